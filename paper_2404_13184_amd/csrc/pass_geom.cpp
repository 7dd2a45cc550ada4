// Host side of the multi-superoperator passes: the process-wide pass limit and the geometry of
// one pass (tile bits, runs of fixed bits, per-superoperator tile offsets and the LDS swizzle,
// which a seeded search picks so that each superoperator's MFMA accesses avoid bank conflicts).
// The kernels are in pass.hip.
#include <algorithm>
#include <atomic>
#include <cstring>

#include "internal.hpp"

namespace tanq {

int pass_tile_bits(tanq_prec p) { return p == TANQ_F64 ? kPassTileBitsF64 : kPassTileBitsF32; }
int pass_max(tanq_prec p) { return p == TANQ_F64 ? kPassMaxF64 : kPassMaxF32; }

static std::atomic<int> g_pass_limit{kPassMax};
int pass_limit() { return g_pass_limit.load(); }
void set_pass_limit(int m) {
  if (m < 1 || m > kPassMax) fail(TANQ_E_ARG, "pass limit must be 1..8");
  g_pass_limit.store(m);
}

// ------------------------------------------------------------------------------------
// host: geometry and swizzle of one pass
// ------------------------------------------------------------------------------------

namespace {

int gf2_rank(uint32_t* v, int cnt) {
  int r = 0;
  for (int bit = 31; bit >= 0 && r < cnt; --bit) {
    int piv = -1;
    for (int i = r; i < cnt; ++i)
      if ((v[i] >> bit) & 1u) {
        piv = i;
        break;
      }
    if (piv < 0) continue;
    std::swap(v[r], v[piv]);
    for (int i = 0; i < cnt; ++i)
      if (i != r && ((v[i] >> bit) & 1u)) v[i] ^= v[r];
    ++r;
  }
  return r;
}

struct SwzProblem {
  int W, V, m;
  uint32_t fbits[kPassMax][4];  // lowest four free tile bits of each superoperator
  uint32_t t1[kPassMax], t2[kPassMax];
};

uint32_t low_of(uint32_t x, const uint8_t* xcol, int W) {
  uint32_t r = x & ((1u << W) - 1u);
  for (int b = W; b < 16; ++b)
    if ((x >> b) & 1u) r ^= xcol[b];
  return r;
}

// Number of bank-conflict-free access patterns under xcol (2 per superoperator).
int swz_score(const SwzProblem& P, const uint8_t* xcol) {
  int score = 0;
  for (int j = 0; j < P.m; ++j) {
    uint32_t v[5];
    if (P.W == 4) {
      for (int q = 0; q < 4; ++q) v[q] = low_of(1u << P.fbits[j][q], xcol, 4);
      score += 2 * (gf2_rank(v, 4) == 4);
    } else {
      for (int q = 0; q < 4; ++q) v[q] = low_of(1u << P.fbits[j][q], xcol, 5);
      v[4] = low_of(P.t1[j], xcol, 5);
      score += gf2_rank(v, 5) == 5;
      for (int q = 0; q < 4; ++q) v[q] = low_of(1u << P.fbits[j][q], xcol, 5);
      v[4] = low_of(P.t2[j], xcol, 5);
      score += gf2_rank(v, 5) == 5;
    }
  }
  return score;
}

// Upper bound of swz_score over all swizzles: a pattern's vectors from bits inside the window
// are fixed unit vectors; those from bits above it can be any vectors of the allowed columns
// (FP32 columns never set bit 0, so an FP32 pattern spans bit 0 only through tile bit 0).
int swz_bound(const SwzProblem& P) {
  auto ok = [&](const uint32_t* bits, int cnt) {
    uint32_t fixed = 0;
    int above = 0;
    for (int q = 0; q < cnt; ++q) {
      if (bits[q] < (uint32_t)P.W) {
        if ((fixed >> bits[q]) & 1u) return false;  // a repeated unit vector
        fixed |= 1u << bits[q];
      } else {
        ++above;
      }
    }
    if (P.W == 5) return (fixed & 1u) && above <= 4 - __builtin_popcount(fixed & ~1u);
    return above <= P.W - __builtin_popcount(fixed);
  };
  int b = 0;
  for (int j = 0; j < P.m; ++j) {
    uint32_t v[5];
    for (int q = 0; q < 4; ++q) v[q] = P.fbits[j][q];
    if (P.W == 4) {
      b += 2 * ok(v, 4);
    } else {
      v[4] = (uint32_t)__builtin_ctz(P.t1[j]);
      b += ok(v, 5);
      v[4] = (uint32_t)__builtin_ctz(P.t2[j]);
      b += ok(v, 5);
    }
  }
  return b;
}

uint64_t splitmix(uint64_t& s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

}  // namespace

PassGeom make_pass_geom(int n, int m, const int* qubits, const uint32_t* op_off, tanq_prec p, int* conflict_free,
                        int* achievable) {
  if (m < 1 || m > kPassMax) fail(TANQ_E_ARG, "pass length outside 1..kPassMax");
  PassGeom g;
  std::memset(&g, 0, sizeof(g));
  const int nb = 2 * n;
  const int V = pass_tile_bits(p);
  if (nb < V) fail(TANQ_E_ARG, "state too small for a pass tile");
  uint64_t vmask = 0;
  for (int j = 0; j < m; ++j)
    for (int t = 0; t < 2; ++t) {
      const int q = qubits[2 * j + t];
      if (q < 0 || q >= n) fail(TANQ_E_ARG, "pass qubit out of range");
      vmask |= (1ull << q) | (1ull << (q + n));
    }
  if (__builtin_popcountll(vmask) > V) fail(TANQ_E_ARG, "pass qubits do not fit one tile");
  for (int b = 0, need = V - __builtin_popcountll(vmask); b < nb && need > 0; ++b)
    if (!((vmask >> b) & 1ull)) {
      vmask |= 1ull << b;
      --need;
    }
  int cnt = 0;
  int local_of[64];
  int vpos[16];  // tile bit -> global bit (ascending)
  for (int b = 0; b < nb; ++b) {
    local_of[b] = -1;
    if ((vmask >> b) & 1ull) {
      local_of[b] = cnt;
      vpos[cnt++] = b;
    }
  }
  if (cnt != V) fail(TANQ_E_STATE, "pass tile bit count");
  // FP32 moves two elements per 16-byte slot: global bit 0 must be tile bit 0
  if (p != TANQ_F64 && vpos[0] != 0) fail(TANQ_E_STATE, "pass tile without global bit 0");
  g.V = V;
  g.m = m;

  uint32_t tj[kPassMax][16], free_mask[kPassMax];
  SwzProblem P{};
  P.W = (p == TANQ_F64) ? 4 : 5;
  P.V = V;
  P.m = m;
  for (int j = 0; j < m; ++j) {
    const int tgt[4] = {qubits[2 * j], qubits[2 * j + 1], qubits[2 * j] + n, qubits[2 * j + 1] + n};
    uint32_t tmask = 0;
    int tpos[4];
    for (int t = 0; t < 4; ++t) {
      tpos[t] = local_of[tgt[t]];
      tmask |= 1u << tpos[t];
    }
    if (__builtin_popcount(tmask) != 4) fail(TANQ_E_ARG, "a pass superoperator repeats a qubit");
    for (int l = 0; l < 16; ++l) {
      uint32_t r = 0;
      for (int t = 0; t < 4; ++t)
        if ((l >> t) & 1) r |= 1u << tpos[t];
      tj[j][l] = r;
    }
    free_mask[j] = ((1u << V) - 1u) & ~tmask;
    g.op_off[j] = op_off[j];
    int q = 0;
    for (int b = 0; b < V && q < 4; ++b)
      if ((free_mask[j] >> b) & 1u) P.fbits[j][q++] = (uint32_t)b;
    P.t1[j] = tj[j][1];  // FP32 operand reads: lanes 0-31 cover rows 0 and 1
    P.t2[j] = tj[j][4];  // FP32 result writes: lanes 0-31 cover rows 0-3 and 4-7
  }

  // swizzle: the identity first, then seeded random candidates, keeping the best (reaching the
  // bound ends the search)
  uint8_t best[16] = {0};
  int best_score = swz_score(P, best);
  const int perfect = swz_bound(P);
  uint64_t seed = 0x7A3Cull ^ ((uint64_t)n << 32) ^ (uint64_t)m;
  // FP32 columns never set bit 0: a 16-byte slot's two elements keep their order, as the
  // global-to-LDS loads require
  const uint32_t wmask = ((1u << P.W) - 1u) & (p == TANQ_F64 ? ~0u : ~1u);
  for (int trial = 0; trial < 4000 && best_score < perfect; ++trial) {
    uint8_t cand[16] = {0};
    const uint64_t r0 = splitmix(seed), r1 = splitmix(seed);
    for (int b = P.W; b < V; ++b) {
      const uint64_t r = (b < 8 + P.W) ? (r0 >> (8 * (b - P.W))) : (r1 >> (8 * (b - P.W - 8)));
      cand[b] = (uint8_t)((uint32_t)r & wmask);
    }
    const int sc = swz_score(P, cand);
    if (sc > best_score) {
      best_score = sc;
      std::memcpy(best, cand, sizeof(best));
    }
  }
  if (conflict_free) *conflict_free = best_score;
  if (achievable) *achievable = perfect;
  auto S = [&](uint32_t e) {
    uint32_t x = e;
    for (int b = P.W; b < 16; ++b)
      if ((e >> b) & 1u) x ^= best[b];
    return x;
  };
  // S and the deposit of a tile element into the state's index bits are linear over GF(2): the kernels form
  // any offset from the images of single bits
  for (int b = 0; b < V; ++b) {
    const uint32_t e = S(1u << b);
    for (int t = 0; t < V; ++t)
      if ((e >> t) & 1u) g.goff[b] |= 1ull << vpos[t];
  }
  for (int j = 0; j < m; ++j) {
    for (int l = 0; l < 16; ++l) g.stj[j][l] = S(tj[j][l]);
    int f = 0;
    for (int b = 0; b < V; ++b)
      if ((free_mask[j] >> b) & 1u) g.fb[j][f++] = (uint16_t)S(1u << b);
  }
  // S(e) = e ^ X(e) with X linear in the bits above the window and valued inside it, so S is an
  // involution of [0, 2^V) exactly when every column lies inside the window (and, in FP32, never
  // flips bit 0, which keeps slot pairs whole and in order); columns of bits >= V are unused
  for (int b = 0; b < 16; ++b)
    if ((b < P.W && best[b]) || (best[b] >> P.W) || (b >= V && best[b]) || (p != TANQ_F64 && (best[b] & 1u)))
      fail(TANQ_E_STATE, "pass swizzle column outside the bank window");

  // runs of fixed bits: the maximal runs of global bits outside the tile, lowest first, each
  // taking the next tile-index bits; so a tile's base is the tile index deposited into those
  // bits, which the FP64 pass kernel relies on to step from one tile's base to the next
  int src = 0, nr = 0;
  for (int b = 0; b < nb;) {
    if ((vmask >> b) & 1ull) {
      ++b;
      continue;
    }
    int e = b;
    while (e < nb && !((vmask >> e) & 1ull)) ++e;
    if (nr >= 16) fail(TANQ_E_STATE, "too many runs of fixed bits");
    g.run_src[nr] = (uint8_t)src;
    g.run_len[nr] = (uint8_t)(e - b);
    g.run_dst[nr] = (uint8_t)b;
    src += e - b;
    ++nr;
    b = e;
  }
  g.nruns = nr;
  g.ntiles = 1ull << (nb - V);
  return g;
}

// ------------------------------------------------------------------------------------
// real-form passes
// ------------------------------------------------------------------------------------

// address bit of index bit b (internal.hpp)
static int real_addr_bit(int b, int n) { return b == 2 * n - 1 ? 0 : b + 1; }

// Address bits a pass over these qubits holds: their row and column bits and the four lowest bits
// (whole 128-byte lines of the state).
static uint64_t real_pass_held(uint64_t qmask, int n) {
  uint64_t held = 15;
  for (int q = 0; q < n; ++q)
    if ((qmask >> q) & 1ull) held |= (1ull << real_addr_bit(q, n)) | (1ull << real_addr_bit(q + n, n));
  return held;
}

bool real_pass_fits(uint64_t qmask, int n) { return __builtin_popcountll(real_pass_held(qmask, n)) <= kRealPassBits; }

// Sets of window vectors (one bit per vector of GF(2)^5): the set moved by v, and the span of it and v.
static uint32_t set_moved(uint32_t set, uint32_t v) {
  if (v & 1u) set = ((set & 0x55555555u) << 1) | ((set >> 1) & 0x55555555u);
  if (v & 2u) set = ((set & 0x33333333u) << 2) | ((set >> 2) & 0x33333333u);
  if (v & 4u) set = ((set & 0x0f0f0f0fu) << 4) | ((set >> 4) & 0x0f0f0f0fu);
  if (v & 8u) set = ((set & 0x00ff00ffu) << 8) | ((set >> 8) & 0x00ff00ffu);
  if (v & 16u) set = (set << 16) | (set >> 16);
  return set;
}

// Columns of a real pass's swizzle: tile bit b above the 32-bank window is XORed into the window as xcol[b].  A
// superoperator's access is free of bank conflicts if its five lane bits (four of the groups, the lowest target) map
// to independent window vectors.  For one column at a time the values that keep every superoperator using it
// independent of its other columns are a set, found for all 32 values at once; a value is taken that suits as many
// of them as possible, and a few rounds over the columns in rotated order repair what the first left.  2.7 us
// for a pass on average, 22 at worst; up to 4000 random trials reached the same number of conflict-free accesses in
// 63 us on average and up to 12 ms, which the first application of every list paid.
static void real_swizzle(const SwzProblem& P, uint8_t* xcol) {
  constexpr int kRounds = 24;
  // columns never set bit 0 (the two elements of a 16-byte slot stay together)
  uint32_t values = 0;
  for (uint32_t v = 0; v < 32; v += 2) values |= 1u << v;
  uint32_t bits[kPassMax];  // lane bits of each superoperator
  for (int j = 0; j < P.m; ++j) {
    bits[j] = P.t1[j];
    for (int q = 0; q < 4; ++q) bits[j] |= 1u << P.fbits[j][q];
  }
  const uint32_t window = (1u << P.W) - 1u;
  uint8_t cur[16] = {0};
  uint32_t chosen = 0;  // columns with a value
  // span of superoperator j's lane bits but `but`; 0 if they are not independent (unchosen ones left out)
  auto span = [&](int j, int but) {
    uint32_t set = 1u;
    for (uint32_t r = bits[j] & (window | chosen) & ~(1u << but); r; r &= r - 1) {
      const int b = __builtin_ctz(r);
      const uint32_t v = b < P.W ? 1u << b : cur[b];
      if ((set >> v) & 1u) return 0u;
      set |= set_moved(set, v);
    }
    return set;
  };
  int best_score = -1;
  for (int round = 0; round < kRounds && best_score < P.m; ++round) {
    for (int i = 0; i < P.V - P.W; ++i) {
      const int b = P.W + (i + round) % (P.V - P.W);
      uint32_t good = values;
      for (int u = 0; u < P.m; ++u) {
        const int j = (u + round) % P.m;
        if (!((bits[j] >> b) & 1u)) continue;
        const uint32_t set = span(j, b);
        if (set && (good & ~set)) good &= ~set;
      }
      if (round > 0 && ((good >> cur[b]) & 1u)) continue;  // as good as any
      // another of the good values each round
      int skip = round % __builtin_popcount(good);
      while (skip-- > 0) good &= good - 1;
      cur[b] = (uint8_t)__builtin_ctz(good);
      chosen |= 1u << b;
    }
    int score = 0;
    for (int j = 0; j < P.m; ++j) score += span(j, 31) != 0;
    if (score > best_score) {
      best_score = score;
      std::memcpy(xcol, cur, sizeof(cur));
    }
  }
}

RealPassGeom make_real_pass_geom(int n, int m, const int* k, const int* qubits, const uint32_t* op_off) {
  if (m < 1 || m > kRealPassMax) fail(TANQ_E_STATE, "real pass length");
  RealPassGeom g{};
  const int nb = 2 * n, V = kRealPassBits, W = 5;
  uint64_t qmask = 0;
  for (int j = 0; j < m; ++j)
    for (int t = 0; t < k[j]; ++t) qmask |= 1ull << qubits[3 * j + t];
  // one-qubit operands need a second qubit that the pass holds
  if (__builtin_popcountll(qmask) == 1) qmask |= (qmask & 1ull) ? 2ull : 1ull;
  uint64_t held = real_pass_held(qmask, n);
  if (__builtin_popcountll(held) > V) fail(TANQ_E_STATE, "real pass qubits do not fit one tile");
  for (int b = 0; b < nb && __builtin_popcountll(held) < V; ++b) held |= 1ull << b;
  int vpos[kRealPassBits], local_of[64], cnt = 0;
  for (int b = 0; b < nb; ++b)
    if ((held >> b) & 1ull) {
      local_of[b] = cnt;
      vpos[cnt++] = b;
    }
  g.m = m;
  g.ntiles = 1ull << (nb - V);
  g.dmask = ((1ull << nb) - 1ull) & ~held;

  int tpos[kRealPassMax][4], fpos[kRealPassMax][9];
  uint32_t tmask[kRealPassMax];
  SwzProblem P{};
  P.W = W;
  P.V = V;
  P.m = m;
  for (int j = 0; j < m; ++j) {
    int q0 = qubits[3 * j], q1 = k[j] == 2 ? qubits[3 * j + 1] : __builtin_ctzll(qmask & ~(1ull << q0));
    const int bits[4] = {q0, q0 + n, q1, q1 + n};
    uint32_t tm = 0;
    for (int t = 0; t < 4; ++t) tm |= 1u << local_of[real_addr_bit(bits[t], n)];
    tmask[j] = tm;
    int nt = 0;
    for (int b = 0; b < V; ++b)
      if ((tm >> b) & 1u) tpos[j][nt++] = b;
    if (nt != 4) fail(TANQ_E_STATE, "a real pass superoperator repeats a qubit");
    g.op_off[j] = op_off[j];
    if (k[j] == 1) {
      // the operand's two local bits among the four, lowest address first
      int e[2], ne = 0;
      for (int t = 0; t < 4; ++t)
        if (tpos[j][t] == local_of[real_addr_bit(q0, n)] || tpos[j][t] == local_of[real_addr_bit(q0 + n, n)]) e[ne++] = t;
      g.emb[j] = (uint8_t)(16 | e[0] | (e[1] << 2));
    }
  }
  // Three bits pick the wave.  Superoperators in a row that leave the same three bits alone share them, so that a
  // wave reads only what it wrote and they need no barrier between them.  Never bit 0, without which a wave's
  // lanes would reach half of the banks.
  for (int j = 0; j < m;) {
    uint32_t targets = tmask[j] | 1u;
    int e = j + 1;
    while (e < m && __builtin_popcount(targets | tmask[e]) <= V - 3) targets |= tmask[e++];
    uint32_t waves = 0;  // the highest bits, so that the lanes keep the lowest
    for (int b = V - 1; __builtin_popcount(waves) < 3; --b)
      if (!((targets >> b) & 1u)) waves |= 1u << b;
    if (e < m) g.sync |= 1u << (e - 1);
    for (; j < e; ++j) {
      int lanes[6], nl = 0, nw = 4;
      for (int b = 0; b < V; ++b) {
        if ((waves >> b) & 1u)
          fpos[j][nw++] = b;
        else if (!((tmask[j] >> b) & 1u))
          lanes[nl++] = b;
      }
      for (int t = 0; t < 4; ++t) fpos[j][t] = lanes[t];
      for (int t = 0; t < 2; ++t) fpos[j][7 + t] = lanes[4 + t];
      // 32 lanes of 8 bytes: 16 groups and the lowest target bit
      for (int t = 0; t < 4; ++t) P.fbits[j][t] = (uint32_t)fpos[j][t];
      P.t1[j] = P.t2[j] = 1u << tpos[j][0];
    }
  }
  uint8_t best[16];
  real_swizzle(P, best);
  // S(e) = e ^ X(e), X from the bits above the window into the window: linear and an involution
  auto S = [&](uint32_t e) {
    uint32_t x = e;
    for (int b = W; b < V; ++b)
      if ((e >> b) & 1u) x ^= best[b];
    return x;
  };
  for (int b = 0; b < 12; ++b) {
    const uint32_t e = S(2u << b);
    uint64_t o = 0;
    for (int t = 0; t < V; ++t)
      if ((e >> t) & 1u) o |= 1ull << vpos[t];
    g.goff[b] = o;
  }
  for (int j = 0; j < m; ++j) {
    for (int b = 0; b < 9; ++b) g.sbit[j][b] = (uint16_t)(8 * S(1u << fpos[j][b]));
    for (int t = 0; t < 4; ++t) g.sbit[j][9 + t] = (uint16_t)(8 * S(1u << tpos[j][t]));
  }
  return g;
}

}  // namespace tanq

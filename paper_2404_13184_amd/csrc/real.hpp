// Real form of Hermitian states, shared by the serving kernels and the Hermitian passes (gfx950).
//
// A Hermitian rho of n qubits is 4^n real numbers, its coefficients over the products of the one-qubit
// matrices |0><0|, |1><1|, X and Y:
//   rho = sum w[r' + c' 2^n] B,  qubit t of B being |0><0|, X, Y or |1><1| for (r'_t, c'_t) = (0,0),
//   (1,0), (0,1) or (1,1).
// The basis factorises over the qubits, so a map on k qubits acts on the same 2k index bits as in
// vec(rho), and a map that keeps Hermiticity (every Kraus set does) is a real 4^k x 4^k matrix R.
// Against vec(rho) that is half the bytes and, per superoperator, one real product in place of
// the three of the 3M form.
//
// The populations rho[x][x] are coefficients themselves (r' = c' = x), and R takes populations to
// populations by the superoperator's own entries.  So rare outcomes keep their relative accuracy and
// outcomes that cannot occur stay exact zeros, as in vec(rho) (the Pauli basis, whose expectations are all
// of order one, turns both into rounding of the trace), the trace moves by the Kraus sets' own rounding and
// nothing else, and errors against 64 bits are no larger than the 3M form's.  A coherence of m qubits is a
// sum of 2^m coefficients, so it is known to the rounding of the largest coherence of the same
// qubits.
//
// Tiles, groups and swizzle follow tile.hpp with real elements: a workgroup owns 2^V elements (the
// 2k target bits plus the lowest free bits).  Each wave owns 16-group column blocks and holds all
// of R in registers (4^k/16 m-tiles x 4^k/4 k-steps of 16x16x4 MFMA fragments), so it reads a
// group's elements once, multiplies, and writes them back in place with no barrier in between --
// also for k = 3, where the 3M operands of the complex form (three times the registers) have to
// be spread over four waves that each read the whole tile.
#pragma once

#include "tile.hpp"

namespace tanq {

// S(e) = e ^ X(e), X copying the lane bits above the 256-byte bank window into the window bits that
// no lane bit covers (make_real_geom), so the 64 lanes of an operand access (16 groups x 4
// rows) fall on distinct banks.  X is linear over GF(2): S(a ^ b) = S(a) ^ S(b).
__device__ inline uint32_t real_swz(uint32_t e, const RealGeom& g) {
  uint32_t x = e;
#pragma unroll
  for (int p = 0; p < kRealSwzPairs; ++p) x ^= ((e >> g.xsrc[p]) & 1u) << g.xdst[p];
  return x;
}

// 16-byte slots a thread moves: global element offset and swizzled LDS slot, the same for every
// tile of one geometry.  has<true>: full tiles, no per-slot guard.
template <int VMAX, int NT>
struct RealIo {
  static constexpr int EPS = 2;  // elements per slot
  static constexpr int SLOTS = (1 << VMAX) / EPS;
  static constexpr int ITERS = (SLOTS + NT - 1) / NT;
  uint32_t off[ITERS];  // elements (states of up to 2^32 elements)
  uint32_t lslot[ITERS];
  int slots;

  __device__ inline void init(const RealGeom& g, int tid) {
    slots = (1 << g.V) / EPS;
#pragma unroll
    for (int it = 0; it < ITERS; ++it) {
      const uint32_t j = (uint32_t)((it * NT + tid) * EPS);
      uint32_t o = 0;
      for (int b = 0; b < g.V; ++b) o |= ((j >> b) & 1u) << g.vpos[b];
      off[it] = o;
      lslot[it] = real_swz(j, g) / EPS;
    }
  }
  template <bool FULL>
  __device__ inline bool has(int it, int tid) const { return FULL || it * NT + tid < slots; }
};

// One superoperator in real form on the tile in LDS, in place: y = R x.  R fragment (m, s) of lane l is
// R[row(m, l % 16)][4 s + l / 16]; accumulator value r of lane l holds row 16 m + l / 16 + 4 r, so the elements a
// lane writes are the ones it read: one set of addresses serves both.
template <int K, int VMAX, int NT>
struct OpReal {
  using M = Mfma<double>;
  using acc_t = typename M::acc_t;
  static constexpr int D = 1 << (2 * K), MT = D / 16, KS = D / 4;
  static constexpr int NW = NT / 64;
  static constexpr int NB_MAX = (1 << (VMAX - 2 * K)) / 16;  // column blocks of a full tile
  static_assert(NB_MAX % NW == 0, "full tiles give every wave the same number of blocks");
  static constexpr int NBW = NB_MAX / NW;
  // column blocks multiplied together: k = 2 has one accumulation chain per block, so pairs keep
  // the matrix unit from waiting for the previous product of the chain
  static constexpr int STEP = (K == 2 && NBW % 2 == 0) ? 2 : 1;
  double a[MT][KS];
  uint32_t lb[NBW];  // S(group part ^ row part l / 16) of this lane in each of its column blocks
  bool act[NBW];
  uint32_t tb[2 * K - 2];  // S(tile offset of local index bit b + 2), uniform
  int nblk;

  __device__ inline void load(const double* __restrict__ frag_in, int lane) {
    const auto* frag = global_ptr(frag_in);
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int s = 0; s < KS; ++s) a[m][s] = frag[(m * KS + s) * 64 + lane];
  }

  __device__ inline void prepare(const RealGeom& g, int lane, int wave) {
    nblk = (g.G + 15) >> 4;
    const int kk = lane >> 4;
    const uint32_t row = ((kk & 1) ? 1u << g.tpos[0] : 0u) | ((kk & 2) ? 1u << g.tpos[1] : 0u);
#pragma unroll
    for (int b = 0; b < 2 * K - 2; ++b)
      tb[b] = (uint32_t)__builtin_amdgcn_readfirstlane((int)real_swz(1u << g.tpos[b + 2], g));
#pragma unroll
    for (int i = 0; i < NBW; ++i) {
      const int gi = (wave + i * NW) * 16 + (lane & 15);
      act[i] = gi < g.G;
      // lanes past the last group (partial tiles) read group 0, which is in the tile, and write nothing
      lb[i] = real_swz((act[i] ? pdep32((uint32_t)gi, g.free_mask) : 0u) | row, g);
    }
  }

  // S(tile offset of local index 4 s)
  __device__ inline uint32_t ts(int s) const {
    uint32_t x = 0;
#pragma unroll
    for (int b = 0; b < 2 * K - 2; ++b)
      if ((s >> b) & 1) x ^= tb[b];
    return x;
  }

  template <bool FULL>
  __device__ inline void compute(double* lds) const {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
#pragma unroll
    for (int i0 = 0; i0 < NBW; i0 += STEP) {
      if (!FULL && wave + i0 * NW >= nblk) break;  // uniform per wave
      double b[STEP][KS];
#pragma unroll
      for (int u = 0; u < STEP; ++u)
#pragma unroll
        for (int s = 0; s < KS; ++s) b[u][s] = lds[ts(s) ^ lb[i0 + u]];
      // m-tiles two at a time: every element is in registers by then, and four accumulators would spill
      constexpr int MP = MT < 2 ? MT : 2;
#pragma unroll
      for (int m0 = 0; m0 < MT; m0 += MP) {
        acc_t acc[STEP][MP];
#pragma unroll
        for (int u = 0; u < STEP; ++u)
#pragma unroll
          for (int m = 0; m < MP; ++m) acc[u][m] = acc_t{0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
          for (int u = 0; u < STEP; ++u)
#pragma unroll
            for (int m = 0; m < MP; ++m) acc[u][m] = M::mma(a[m0 + m][s], b[u][s], acc[u][m]);
#pragma unroll
        for (int u = 0; u < STEP; ++u)
          if (FULL || act[i0 + u]) {
#pragma unroll
            for (int m = 0; m < MP; ++m)
#pragma unroll
              for (int r = 0; r < 4; ++r) lds[ts(4 * (m0 + m) + r) ^ lb[i0 + u]] = acc[u][m][r];
          }
      }
    }
  }
};

// The tiles [t0, t1) of one state, in place: the next tile is prefetched into registers while the
// current one is multiplied in one of two LDS buffers.  A wave multiplies its own groups in place,
// so a tile takes two barriers: one between the multiplication and the store phase (which also
// fills the other buffer with the next tile), one after it.
template <bool FULL, typename IO, typename Op, typename Base>
__device__ inline void real_tiles(double* __restrict__ rho, const IO& io, const Op& op, const Base& base, u32x4 (&lds)[2][IO::SLOTS], uint32_t t0, uint32_t t1, int tid) {
  uint32_t cur = base(t0);
  u32x4 buf[IO::ITERS];
#pragma unroll
  for (int it = 0; it < IO::ITERS; ++it)
    if (io.template has<FULL>(it, tid)) buf[it] = *global_ptr(reinterpret_cast<const u32x4*>(rho + (cur + io.off[it])));
#pragma unroll
  for (int it = 0; it < IO::ITERS; ++it)
    if (io.template has<FULL>(it, tid)) lds[0][io.lslot[it]] = buf[it];
  lds_barrier();
  int b = 0;
  for (uint32_t t = t0;;) {
    const bool more = t + 1 < t1;
    uint32_t nbase = 0;
    if (more) {
      nbase = base(t + 1);
#pragma unroll
      for (int it = 0; it < IO::ITERS; ++it)
        if (io.template has<FULL>(it, tid))
          buf[it] = *global_ptr(reinterpret_cast<const u32x4*>(rho + (nbase + io.off[it])));
    }
    op.template compute<FULL>(reinterpret_cast<double*>(lds[b]));
    lds_barrier();  // results complete
#pragma unroll
    for (int it = 0; it < IO::ITERS; ++it)
      if (io.template has<FULL>(it, tid)) *global_ptr(reinterpret_cast<u32x4*>(rho + (cur + io.off[it]))) = lds[b][io.lslot[it]];
    if (more) {
#pragma unroll
      for (int it = 0; it < IO::ITERS; ++it)
        if (io.template has<FULL>(it, tid)) lds[b ^ 1][io.lslot[it]] = buf[it];
    }
    lds_barrier();  // this buffer is read out, the other one filled (or both free)
    if (!more) break;
    ++t;
    b ^= 1;
    cur = nbase;
  }
}

// ------------------------------------------------------------------------------------
// real form of a superoperator
// ------------------------------------------------------------------------------------

__device__ inline int ycount(uint32_t a, int k) {
  const uint32_t m = (1u << k) - 1u;
  return __popc(~a & (a >> k) & m);
}

// R[a][b] of a superoperator S (4^k x 4^k complex): Re((-i)^(y_a - y_b) 2^-m_a sum_{u,v} +-
// S[i(a,u)][i(b,v)]), u and v running over the 2^m choices of (row, column) = (1, 0) or (0, 1) on the m qubits where
// the index is X or Y, a factor -1 for every Y at (0, 1).  For S = sum_i conj(K_i) (x) K_i the imaginary part
// is zero.  Between populations it is one entry of S; summed without rounding loss and rounded once.
__device__ inline double real_entry(const f64x2* S, int k, uint32_t a, uint32_t b) {
  const uint32_t m = (1u << k) - 1u;
  const uint32_t ra = a & m, ca = a >> k, rb = b & m, cb = b >> k;
  const uint32_t xa = ra ^ ca, xb = rb ^ cb, ya = ~ra & ca, yb = ~rb & cb;
  const int d = (ycount(a, k) - ycount(b, k)) & 3;  // Re((-i)^d (x + i y)) = x, y, -x, -y
  const double scale = 1.0 / (double)(1u << __popc(xa));
  double h = 0.0, l = 0.0;
  for (uint32_t u = xa;; u = (u - 1) & xa) {  // the subsets of xa
    const uint32_t row = ((ra & ca) | u) + (((ra & ca) | (xa & ~u)) << k);
    for (uint32_t v = xb;; v = (v - 1) & xb) {
      const f64x2 x = S[(row << (2 * k)) + ((rb & cb) | v) + (((rb & cb) | (xb & ~v)) << k)];
      const bool neg = ((__popc(ya & ~u) + __popc(yb & ~v)) & 1) != (d >> 1);
      double t = ((d & 1) ? x[1] : x[0]) * scale;
      t = neg ? -t : t;
      const double s = h + t, bb = s - h;  // s + the error term is the exact sum
      l += (h - (s - bb)) + (t - bb);
      h = s;
      if (v == 0) break;
    }
    if (u == 0) break;
  }
  return h + l;
}

// fragment element e of a packed real operand: its row and column (real.hpp, OpReal)
__device__ inline void real_frag_index(int e, int KS, int* row, int* col) {
  const int lane = e & 63, rest = e >> 6, s = rest % KS, m = rest / KS, i = lane & 15;
  *row = 16 * m + i;
  *col = 4 * s + (lane >> 4);
}


// ------------------------------------------------------------------------------------
// real-form passes (herm.hip)
// ------------------------------------------------------------------------------------

__device__ inline uint64_t pdep64(uint64_t x, uint64_t mask) {
  uint64_t r = 0;
  for (uint64_t m = mask; m; m &= m - 1) {
    if (x & 1u) r |= m & (0 - m);
    x >>= 1;
  }
  return r;
}

// A run of up to eight one- and two-qubit superoperators on each tile of 2^13 reals (64 KiB) while it
// is in LDS, as apply_pass_kernel: one workgroup per CU, eight waves that all multiply and each load
// their share of the next tile into the other buffer.  A real operand is a third of a 3M operand,
// so every operand and offset stays in registers for twice the superoperators.
//
// Three tile bits pick the wave, and superoperators in a row that all leave three bits alone share them
// (make_real_pass_geom), so a wave reads what it wrote itself and goes on to the next superoperator
// without a barrier, out of step with the other wave on its SIMD, whose products cover its
// LDS accesses.  Of seven gaps between eight superoperators about one needs a barrier.  At 14 qubits
// a pass takes about 150 + 160 m us for m superoperators where memory does not bound it (150 + 190 m
// with a barrier in every gap; the products alone are 139 m), and not less than 700 to 900 (4.3 GB),
// so up to four superoperators it is bound by memory.
__device__ inline void real_pass_tiles(double* __restrict__ w, const double* __restrict__ packed, const RealPassGeom& g,
                                       u32x4* ldsA, u32x4* ldsB) {
  constexpr int NT = kRealPassThreads, ITERS = 8, NBW = 4, MMAX = kRealPassMax;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  // Tiles one after the other (first, first + 1, ..) or a grid apart, so that those in flight on the card lie next
  // to each other.  20 layers of random U3/CX, contiguous -> apart: 12 qubits 2.88 -> 2.76 ms, 13 qubits
  // 9.92 -> 9.46 ms; from 14 qubits on the two are within 1%, at 16 apart is 2% slower.
  const bool apart = g.ntiles < (1ull << 15);
  const uint64_t per = (g.ntiles + gridDim.x - 1) / gridDim.x;
  const uint64_t first = apart ? blockIdx.x : (uint64_t)blockIdx.x * per, by = apart ? gridDim.x : 1;
  const uint64_t end = apart || first + per > g.ntiles ? g.ntiles : first + per;
  if (first >= end) return;  // uniform per workgroup
  const uint64_t step = pdep64(by, g.dmask);

  // slot it * 512 + tid; offsets are linear over GF(2) in the slot index
  uint64_t off_t = 0;
#pragma unroll
  for (int b = 0; b < 9; ++b)
    if ((tid >> b) & 1) off_t ^= g.goff[b];
  auto off = [&](int it) {
    return off_t ^ ((it & 1) ? g.goff[9] : 0) ^ ((it & 2) ? g.goff[10] : 0) ^ ((it & 4) ? g.goff[11] : 0);
  };
  uint64_t cur = pdep64(first, g.dmask);
  {
    const uint32_t ab = lds_addr(ldsA) + (uint32_t)wave * 1024u;
#pragma unroll
    for (int it = 0; it < ITERS; ++it) pass_dma16(w + cur + off(it), ab + (uint32_t)(it * NT * 16));
  }

  // operands and offsets of every superoperator (real.hpp: fragment and row order of OpReal)
  double a[MMAX][4];
  uint32_t lb[MMAX][NBW];  // LDS byte offset of this lane's group and row in each column block
  const int kk = lane >> 4, li = lane & 15;
#pragma unroll
  for (int j = 0; j < MMAX; ++j) {
    if (j < g.m) {
      const double* P = packed + g.op_off[j];
      const uint32_t em = g.emb[j];
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if (em == 0) {
          a[j][s] = P[s * 64 + lane];
        } else {
          const int e0 = em & 3, e1 = (em >> 2) & 3, row = li, col = 4 * s + kk;
          const int keep = 15 & ~((1 << e0) | (1 << e1));
          const int r4 = ((row >> e0) & 1) | (((row >> e1) & 1) << 1), c4 = ((col >> e0) & 1) | (((col >> e1) & 1) << 1);
          a[j][s] = ((row ^ col) & keep) ? 0.0 : P[r4 * 4 + c4];
        }
      }
      uint32_t l = 0;
#pragma unroll
      for (int b = 0; b < 4; ++b)
        if ((li >> b) & 1) l ^= g.sbit[j][b];
      if (kk & 1) l ^= g.sbit[j][9];
      if (kk & 2) l ^= g.sbit[j][10];
#pragma unroll
      for (int b = 0; b < 3; ++b)
        if ((wave >> b) & 1) l ^= g.sbit[j][4 + b];
#pragma unroll
      for (int i = 0; i < NBW; ++i)
        lb[j][i] = l ^ ((i & 1) ? (uint32_t)g.sbit[j][7] : 0u) ^ ((i & 2) ? (uint32_t)g.sbit[j][8] : 0u);
    }
  }
  vm_wait<0>();
  raw_barrier();  // the first tile is in LDS

  const int m = g.m;
  auto tile_step = [&](u32x4* buf, u32x4* other, uint64_t nbase, bool more) {
    char* L = reinterpret_cast<char*>(buf);
    if (more) {
      const uint32_t ob = lds_addr(other) + (uint32_t)wave * 1024u;
#pragma unroll
      for (int it = 0; it < ITERS; ++it) pass_dma16(w + nbase + off(it), ob + (uint32_t)(it * NT * 16));
    }
#pragma unroll
    for (int j = 0; j < MMAX; ++j) {
      if (j >= m) break;  // uniform
      const uint32_t t1 = g.sbit[j][11], t2 = g.sbit[j][12];
      // formed anew for every tile: hoisted out of the tile loop, the 16 addresses per superoperator
      // would take the registers that the operands need
      uint32_t l[NBW];
#pragma unroll
      for (int i = 0; i < NBW; ++i) {
        l[i] = lb[j][i];
        asm volatile("" : "+v"(l[i]));
      }
      auto at = [&](int i, int s) -> double& {
        return *reinterpret_cast<double*>(L + (l[i] ^ ((s & 1) ? t1 : 0u) ^ ((s & 2) ? t2 : 0u)));
      };
      double b[NBW][4];
#pragma unroll
      for (int i = 0; i < NBW; ++i)
#pragma unroll
        for (int s = 0; s < 4; ++s) b[i][s] = at(i, s);
      __builtin_amdgcn_sched_barrier(0);
      f64x4 acc[2];
#pragma unroll
      for (int i = 0; i < NBW; ++i) {
        f64x4 c = {0, 0, 0, 0};
#pragma unroll
        for (int s = 0; s < 4; ++s) c = Mfma<double>::mma(a[j][s], b[i][s], c);
        acc[i & 1] = c;
        // the results of block i - 1 are written while block i is multiplied
        if (i > 0) {
#pragma unroll
          for (int r = 0; r < 4; ++r) at(i - 1, r) = acc[(i - 1) & 1][r];
        }
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) at(NBW - 1, r) = acc[(NBW - 1) & 1][r];
      if ((g.sync >> j) & 1u)
        raw_barrier();  // the next superoperator reads what other waves wrote
      else
        asm volatile("" ::: "memory");  // it reads what this wave wrote; LDS accesses of a wave stay in order
    }
    raw_barrier();  // the store reads what other waves wrote
#pragma unroll
    for (int it = 0; it < ITERS; ++it)
      __builtin_nontemporal_store(buf[it * NT + tid], reinterpret_cast<u32x4*>(w + cur + off(it)));
  };
  bool odd = false;
  for (uint64_t tile = first;; tile += by) {
    const bool more = tile + by < end;
    // the base of the next tile: a sum under the mask of the bits outside the tile
    const uint64_t nbase = more ? ((cur | ~g.dmask) + step) & g.dmask : 0;
    if (odd)
      tile_step(ldsB, ldsA, nbase, more);
    else
      tile_step(ldsA, ldsB, nbase, more);
    if (!more) break;
    vm_wait<ITERS>();  // this wave's loads of the next tile (issued before its stores)
    raw_barrier();     // the next tile is in LDS; this buffer is read out
    cur = nbase;
    odd = !odd;
  }
}

}  // namespace tanq

// Runs of superoperators on small states (gfx950): consecutive blocks of any width applied to each tile of
// vec(rho) while it is in LDS, one launch per run instead of one per block.
//
// A small state's apply is bound by its launch: 4.4 us each at 8 qubits in FP64 for 0.5 us of products
// (one workgroup per tile, every CU with at most one).  So a run takes every following block whose qubits fit
// the tile, and the tile is small (2^10 elements in FP64, 2^11 in FP32: 16 KiB, five qubits), which
// spreads a state over many CUs.  Larger tiles hold more blocks but multiply longer on fewer CUs: 2^12
// elements need 1.9 us per two-qubit block against 0.5.
//
// Each block is multiplied as its single apply multiplies it (k = 1 on the vector ALU, k = 2 in
// real-block form, k = 3 in 3M form, from the same packed operands and in the same order), so the
// results are those of the blocks one by one, bit for bit.
//
// What is left is a serial chain of short steps with one wave per SIMD, so latencies count.  Operands of one-
// and two-qubit blocks are loaded into LDS together at the start, those of three-qubit blocks touched there
// (their loads later hit the L2); the table of blocks is copied from the kernel's arguments into LDS in
// one go; a block's entry and operand are read from LDS while the one before is multiplied; blocks one after
// the other on one qubit keep their amplitudes in registers.  The 640 single-operation blocks of the
// 8-qubit plain circuit: 640 launches, 2.81 ms, one by one; 59 launches, 0.81 ms, in runs (12.2 us each,
// 3.4 us of it the start).  A 6-qubit list of 23 two-qubit blocks: 150 -> 55 us.
// Touching the three-qubit operands: a 6-qubit FP32 list with 22 of them, operands out of the L2: 266 us where the
// last third of each was left out, 227 us (213 and 216 us where they are in the L2).
#include <cstddef>

#include "real.hpp"

namespace tanq {

namespace {

template <typename T>
struct RunShape;
template <>
struct RunShape<double> { static constexpr int V = kRunBitsF64; };
template <>
struct RunShape<float> { static constexpr int V = kRunBitsF32; };
constexpr int kRunThreads = 256;

// LDS place of tile element e: linear over GF(2), every bit above the 256-byte window XORed into it
template <typename T>
__host__ __device__ inline uint32_t run_place(uint32_t e) {
  if constexpr (sizeof(T) == 8) return e ^ ((e >> 4) & 15u) ^ ((e >> 8) & 15u);
  // FP32 keeps bit 0 (the two elements of a 16-byte slot stay together)
  return e ^ ((e >> 4) & 30u) ^ ((e >> 8) & 30u);
}

__device__ inline uint32_t uniform(uint32_t x) { return (uint32_t)__builtin_amdgcn_readfirstlane((int)x); }
__device__ inline void uniform_all(RunOp& o) {
  static_assert(sizeof(RunOp) % 4 == 0, "copied as dwords");
  uint32_t w[sizeof(RunOp) / 4];
  __builtin_memcpy(w, &o, sizeof(o));
#pragma unroll
  for (int i = 0; i < (int)(sizeof(RunOp) / 4); ++i) w[i] = uniform(w[i]);
  __builtin_memcpy(&o, w, sizeof(o));
}
// offset of the geometry among the kernel's arguments (after two pointers)
constexpr int kRunArgAt = 16;

}  // namespace

template <typename T>
__global__ __launch_bounds__(kRunThreads) void apply_run_kernel(T* __restrict__ rho,
                                                                const unsigned char* __restrict__ packed,
                                                                const RunGeom g) {
  using M = Mfma<T>;
  using acc_t = typename M::acc_t;
  using c2 = typename M::c2;
  constexpr int V = RunShape<T>::V, NT = kRunThreads, NW = NT / 64;
  constexpr int EPS = 16 / (2 * (int)sizeof(T)), SLOTS = (1 << V) / EPS, ITERS = SLOTS / NT;
  constexpr int OPE = 1024;  // elements of a two-qubit operand
  constexpr int LINES3 = packed_elems(3) * (int)sizeof(T) / 128;  // cache lines of a three-qubit one
  __shared__ u32x4 tile4[SLOTS];
  __shared__ RunOp tab[kRunMax];
  __shared__ T opl1[kRunMax][32];
  __shared__ __align__(16) T opl2[kRunMax2][OPE];
  T* L = reinterpret_cast<T*>(tile4);
  c2* C = reinterpret_cast<c2*>(tile4);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kk = lane >> 4;
  const int slots = (1 << g.V) / EPS;

  // The head of the geometry comes from scalar registers; the table of blocks is copied into LDS in one go
  // (kernel arguments may lie in host memory: a scalar load per block that misses costs more than
  // the block).
  uint32_t bit[8];  // all ones where the bit of tid is set
#pragma unroll
  for (int b = 0; b < 8; ++b) bit[b] = 0u - ((uint32_t)(tid >> b) & 1u);
  constexpr int EB = EPS == 2 ? 1 : 0;  // tile bits inside a slot
  uint32_t off_t = pdep32(blockIdx.x, g.dmask);
#pragma unroll
  for (int b = 0; b < 8; ++b) off_t |= b + EB < g.V ? bit[b] & g.goff[b + EB] : 0u;
  uint32_t off[ITERS];
  u32x4 buf[ITERS];
#pragma unroll
  for (int it = 0; it < ITERS; ++it) {
    off[it] = off_t | ((it & 1) ? g.goff[8 + EB] : 0u) | ((it & 2) ? g.goff[9 + EB] : 0u);
    if (it * NT + tid < slots) buf[it] = *reinterpret_cast<const u32x4*>(rho + 2 * (uint64_t)off[it]);
  }
#pragma unroll
  for (int j = 0; j < kRunMax2; ++j) {
    if (j >= g.m2) break;  // uniform
    const unsigned char* P = packed + (size_t)g.off2[j] * 256;
    const uint32_t to = lds_addr(opl2[j]) + (uint32_t)wave * 1024u;
#pragma unroll
    for (int u = 0; u < OPE * (int)sizeof(T) / 16 / NT; ++u) pass_dma16(P + (u * NT + tid) * 16, to + (uint32_t)(u * NT * 16));
  }
#pragma unroll
  for (int j = 0; j < kRunMax3; ++j) {
    if (j >= g.m3) break;
    const unsigned char* P = packed + (size_t)g.off3[j] * 256;
#pragma unroll
    for (int u = 0; u < (LINES3 + NT - 1) / NT; ++u) {
      if (u * NT + tid >= LINES3) break;
      const uint32_t x = *reinterpret_cast<const uint32_t*>(P + (u * NT + tid) * 128);
      asm volatile("" ::"v"(x));
    }
  }
  const uint32_t* arg = reinterpret_cast<const uint32_t*>(
      (const unsigned char*)__builtin_amdgcn_kernarg_segment_ptr() + kRunArgAt + offsetof(RunGeom, op));
  for (int i = tid; i < g.m * (int)(sizeof(RunOp) / 4); i += NT) reinterpret_cast<uint32_t*>(tab)[i] = arg[i];
  lds_barrier();
  for (int idx = tid; idx < g.m * 32; idx += NT)
    if (tab[idx / 32].k == 1)
      opl1[idx / 32][idx % 32] = (T)reinterpret_cast<const double*>(packed + (size_t)tab[idx / 32].off * 256)[idx % 32];
#pragma unroll
  for (int it = 0; it < ITERS; ++it)
    if (it * NT + tid < slots) tile4[run_place<T>((uint32_t)(it * NT + tid) * EPS) / EPS] = buf[it];
  vm_wait<0>();  // this wave's operand loads (the compiler does not count the direct ones)
  lds_barrier();

  // The next block's table entry and operand are read from LDS while the current one is multiplied: of a
  // one-qubit block each lane holds one of the 32 values, of a two-qubit block its fragments.
  RunOp ahead = tab[0];
  T a1 = 0, a2[16];
  auto operand = [&](int j, const RunOp& o) {
    if (o.k == 1) {
      a1 = opl1[j][lane & 31];
    } else if (o.k == 2) {
#pragma unroll
      for (int i = 0; i < 16; ++i) a2[i] = opl2[o.aux][i * 64 + lane];
    }
  };
  uniform_all(ahead);
  operand(0, ahead);
  for (int j = 0; j < g.m;) {
    const RunOp o = ahead;
    uint32_t tb[6];  // LDS place of each local index bit
#pragma unroll
    for (int t = 0; t < 6; ++t) tb[t] = o.tb[t];
    // place of group 16 c + lane % 16 (c uniform)
    const uint32_t lanes = (bit[0] & o.fb[0]) ^ (bit[1] & o.fb[1]) ^ (bit[2] & o.fb[2]) ^ (bit[3] & o.fb[3]);
    auto column = [&](int c) {
      return ((c & 1) ? o.fb[4] : 0u) ^ ((c & 2) ? o.fb[5] : 0u) ^ ((c & 4) ? o.fb[6] : 0u);
    };
    auto place = [&](int l) {  // of local index l
      uint32_t x = 0;
#pragma unroll
      for (int t = 0; t < 6; ++t)
        if ((l >> t) & 1) x ^= tb[t];
      return x;
    };
    const int G = 1 << (g.V - 2 * o.k);
    int jn = j + 1;  // the block after this one (or after a chain of blocks on one qubit)
    if (o.k == 1) jn += o.aux;
    RunOp next = tab[jn < g.m ? jn : 0];
    if (o.k == 1) {
      uint32_t e0 = lanes;
#pragma unroll
      for (int b = 4; b < 8; ++b) e0 ^= bit[b] & o.fb[b];
      constexpr int GT = (1 << (V - 2)) / NT;  // groups of a thread
      uint32_t e[GT];
      c2 x[GT][4];
#pragma unroll
      for (int u = 0; u < GT; ++u) {
        const bool act = u * NT + tid < G;
        e[u] = act ? e0 ^ (u ? o.fb[8] : 0u) : 0u;
        x[u][0] = C[e[u]];
        x[u][1] = C[e[u] ^ tb[0]];
        x[u][2] = C[e[u] ^ tb[1]];
        x[u][3] = C[e[u] ^ tb[0] ^ tb[1]];
      }
      // following blocks on the same qubit act on the same groups: they stay in registers
      for (int c = j; c < jn; ++c) {
        T sr[16], si[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          sr[i] = lane_value(a1, 2 * i);
          si[i] = lane_value(a1, 2 * i + 1);
        }
        if (c + 1 < jn) a1 = opl1[c + 1][lane & 31];
#pragma unroll
        for (int u = 0; u < GT; ++u) {
          c2 y[4];
          c1_group<T>(sr, si, x[u], y);
#pragma unroll
          for (int i = 0; i < 4; ++i) x[u][i] = y[i];
        }
      }
#pragma unroll
      for (int u = 0; u < GT; ++u)
        if (u * NT + tid < G) {
          C[e[u]] = x[u][0];
          C[e[u] ^ tb[0]] = x[u][1];
          C[e[u] ^ tb[1]] = x[u][2];
          C[e[u] ^ tb[0] ^ tb[1]] = x[u][3];
        }
    } else if (o.k == 2) {
      const int cc = kk & 1, hb = kk >> 1;
      for (int blk = wave; blk * 16 < G; blk += NW) {
        const int gi = blk * 16 + (lane & 15);
        const bool act = gi < G;  // lanes past the last group read group 0 and write nothing
        const uint32_t e = act ? lanes ^ column(blk) : 0u;
        T b[8];
#pragma unroll
        for (int s = 0; s < 8; ++s) b[s] = L[2 * (e ^ place(2 * s + hb)) + cc];
        acc_t acc[2] = {acc_t{0, 0, 0, 0}, acc_t{0, 0, 0, 0}};
#pragma unroll
        for (int s = 0; s < 8; ++s)
#pragma unroll
          for (int m = 0; m < 2; ++m) acc[m] = M::mma(a2[m * 8 + s], b[s], acc[m]);
        if (act) {
#pragma unroll
          for (int m = 0; m < 2; ++m) {
            if constexpr (M::kRowsStrided) {
              // value r = component cc of output 8 m + 2 r + hb
#pragma unroll
              for (int r = 0; r < 4; ++r) L[2 * (e ^ place(8 * m + 2 * r + hb)) + cc] = acc[m][r];
            } else {
              // values (0, 1), (2, 3) = outputs 8 m + 2 kk and the next
              const uint32_t e0 = e ^ place(8 * m) ^ ((kk & 1) ? tb[1] : 0u) ^ ((kk & 2) ? tb[2] : 0u);
              C[e0] = c2{acc[m][0], acc[m][1]};
              C[e0 ^ tb[0]] = c2{acc[m][2], acc[m][3]};
            }
          }
        }
      }
    } else {
      // each wave multiplies one 16-row m-tile with every column block; the tile is read by every wave
      // before any of them writes
      constexpr int NBW = ((1 << (V - 6)) + 15) / 16;
      const T* F = reinterpret_cast<const T*>(packed + (size_t)o.off * 256);
      const int mt = wave;
      acc_t p1[NBW], p2[NBW], p3[NBW];
      uint32_t e[NBW];
#pragma unroll
      for (int i = 0; i < NBW; ++i) {
        const int gi = i * 16 + (lane & 15);
        e[i] = gi < G ? lanes ^ column(i) : 0u;
        p1[i] = p2[i] = p3[i] = acc_t{0, 0, 0, 0};
      }
      const uint32_t rk = ((kk & 1) ? tb[0] : 0u) ^ ((kk & 2) ? tb[1] : 0u);
#pragma unroll
      for (int s = 0; s < 16; ++s) {
        const T ar = F[((mt * 16 + s) * 3 + 0) * 64 + lane], ai = F[((mt * 16 + s) * 3 + 1) * 64 + lane],
                as = F[((mt * 16 + s) * 3 + 2) * 64 + lane];
#pragma unroll
        for (int i = 0; i < NBW; ++i) {
          if (i * 16 >= G) continue;
          const c2 v = C[e[i] ^ rk ^ place(4 * s)];
          const T br = v[0], bi = v[1];
          const T bs = br + bi;
          p1[i] = M::mma(ar, br, p1[i]);
          p2[i] = M::mma(ai, bi, p2[i]);
          p3[i] = M::mma(as, bs, p3[i]);
        }
      }
      lds_barrier();
#pragma unroll
      for (int i = 0; i < NBW; ++i) {
        if (i * 16 + (lane & 15) >= G) continue;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          uint32_t row;
          if constexpr (M::kRowsStrided)
            row = place(16 * mt + 4 * r) ^ rk;
          else
            row = place(16 * mt + r) ^ ((kk & 1) ? tb[2] : 0u) ^ ((kk & 2) ? tb[3] : 0u);
          const T re = p1[i][r] - p2[i][r];
          const T im = p3[i][r] - p1[i][r] - p2[i][r];
          C[e[i] ^ row] = c2{re, im};
        }
      }
    }
    uniform_all(next);
    ahead = next;
    if (jn < g.m) operand(jn, ahead);
    lds_barrier();
    j = jn;
  }
#pragma unroll
  for (int it = 0; it < ITERS; ++it)
    if (it * NT + tid < slots)
      *reinterpret_cast<u32x4*>(rho + 2 * (uint64_t)off[it]) = tile4[run_place<T>((uint32_t)(it * NT + tid) * EPS) / EPS];
}

void launch_run(void* rho, int n, tanq_prec p, int m, const RunBlock* blocks, const void* packed, hipStream_t s) {
  if (m < 1 || m > kRunMax || n > run_max_n(p)) fail(TANQ_E_STATE, "run of superoperators out of range");
  RunGeom g{};
  const int nb = 2 * n, V = run_tile_bits(p) < nb ? run_tile_bits(p) : nb;
  uint32_t held = 0;
  for (int j = 0; j < m; ++j)
    for (int t = 0; t < blocks[j].k; ++t) held |= (1u << blocks[j].qubits[t]) | (1u << (blocks[j].qubits[t] + n));
  if (__builtin_popcount(held) > V) fail(TANQ_E_STATE, "run qubits do not fit one tile");
  for (int b = 0; b < nb && __builtin_popcount(held) < V; ++b) held |= 1u << b;
  // FP32 moves two elements per 16-byte slot
  if (p != TANQ_F64 && !(held & 1u)) fail(TANQ_E_STATE, "run tile without index bit 0");
  int local_of[32] = {0}, cnt = 0;
  for (int b = 0; b < nb; ++b)
    if ((held >> b) & 1u) {
      local_of[b] = cnt;
      g.goff[cnt++] = 1u << b;
    }
  g.V = V;
  g.m = m;
  g.dmask = ((1u << nb) - 1u) & ~held;
  auto place = [&](int b) { return (uint16_t)(p == TANQ_F64 ? run_place<double>(1u << b) : run_place<float>(1u << b)); };
  for (int j = 0; j < m; ++j) {
    const RunBlock& b = blocks[j];
    RunOp& o = g.op[j];
    if (b.k == 2) {
      if (g.m2 >= kRunMax2) fail(TANQ_E_STATE, "too many two-qubit blocks in a run");
      o.aux = (uint16_t)g.m2;
      g.off2[g.m2++] = (uint32_t)(b.pack_off / 256);
    } else if (b.k == 3) {
      if (g.m3 >= kRunMax3) fail(TANQ_E_STATE, "too many three-qubit blocks in a run");
      g.off3[g.m3++] = (uint32_t)(b.pack_off / 256);
    } else {
      while (j + o.aux + 1 < m && blocks[j + o.aux + 1].k == 1 && blocks[j + o.aux + 1].qubits[0] == b.qubits[0]) ++o.aux;
    }
    o.off = (uint32_t)(b.pack_off / 256);
    o.k = (uint16_t)b.k;
    uint32_t tm = 0;
    for (int t = 0; t < b.k; ++t) {
      const int r = local_of[b.qubits[t]], c = local_of[b.qubits[t] + n];
      o.tb[t] = place(r);
      o.tb[b.k + t] = place(c);
      tm |= (1u << r) | (1u << c);
    }
    int f = 0;
    for (int t = 0; t < V; ++t)
      if (!((tm >> t) & 1u)) o.fb[f++] = place(t);
  }
  const unsigned grid = 1u << (nb - V);
  if (p == TANQ_F64)
    hipLaunchKernelGGL(apply_run_kernel<double>, dim3(grid), dim3(kRunThreads), 0, s, (double*)rho,
                       (const unsigned char*)packed, g);
  else
    hipLaunchKernelGGL(apply_run_kernel<float>, dim3(grid), dim3(kRunThreads), 0, s, (float*)rho,
                       (const unsigned char*)packed, g);
  TANQ_HIP(hipGetLastError());
}

}  // namespace tanq

// Real (Pauli) form of Hermitian states, shared by the serving kernels and the Hermitian passes
// (gfx950).
//
// A Hermitian rho of n qubits is 4^n real numbers: w[r' + c' 2^n] = Tr(P rho) for the Pauli string
// whose character on qubit t is I, X, Y or Z for (r'_t, c'_t) = (0,0), (1,0), (0,1), (1,1).  In
// terms of vec(rho)
//   w[r', c'] = (-i)^{y} sum_u (-1)^{u . c'} rho[u ^ r' ^ c'][u],   y = popcount(~r' & c'),
// which factorises over the qubits, so a map on k qubits acts on the same 2k index bits as in
// vec(rho), and a map that keeps Hermiticity (every Kraus set does) is a real 4^k x 4^k matrix R.
// Against vec(rho) that is half the bytes and, per superoperator, one real product in place of
// the three of the 3M form.  Everything stays in the precision of the state.
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
template <typename T, int VMAX, int NT>
struct RealIo {
  static constexpr int EPS = 16 / (int)sizeof(T);  // elements per slot
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

// One superoperator in real form on the tile in LDS, in place.  R fragment (m, s) of lane l is
// R[row(m, l % 16)][4 s + l / 16]; accumulator value r of lane l holds row 16 m + l / 16 + 4 r in both
// precisions (the FP32 packing permutes the rows within an m-tile), so the elements a lane writes
// are the ones it read and one set of addresses serves both.
template <typename T, int K, int VMAX, int NT>
struct OpReal {
  using M = Mfma<T>;
  using acc_t = typename M::acc_t;
  static constexpr int D = 1 << (2 * K), MT = D / 16, KS = D / 4;
  static constexpr int NW = NT / 64;
  static constexpr int NB_MAX = (1 << (VMAX - 2 * K)) / 16;  // column blocks of a full tile
  static_assert(NB_MAX % NW == 0, "full tiles give every wave the same number of blocks");
  static constexpr int NBW = NB_MAX / NW;
  // column blocks multiplied together: k = 2 has one accumulation chain per block, so pairs keep
  // the matrix unit from waiting for the previous product of the chain
  static constexpr int STEP = (K == 2 && NBW % 2 == 0) ? 2 : 1;
  T a[MT][KS];
  uint32_t lb[NBW];  // S(group part ^ row part l / 16) of this lane in each of its column blocks
  bool act[NBW];
  uint32_t tb[2 * K - 2];  // S(tile offset of local index bit b + 2), uniform
  int nblk;

  __device__ inline void load(const T* __restrict__ frag_in, int lane) {
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
  __device__ inline void compute(T* lds) const {
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
#pragma unroll
    for (int i0 = 0; i0 < NBW; i0 += STEP) {
      if (!FULL && wave + i0 * NW >= nblk) break;  // uniform per wave
      T b[STEP][KS];
      acc_t acc[STEP][MT];
#pragma unroll
      for (int u = 0; u < STEP; ++u)
#pragma unroll
        for (int s = 0; s < KS; ++s) b[u][s] = lds[ts(s) ^ lb[i0 + u]];
#pragma unroll
      for (int u = 0; u < STEP; ++u)
#pragma unroll
        for (int m = 0; m < MT; ++m) acc[u][m] = acc_t{0, 0, 0, 0};
#pragma unroll
      for (int s = 0; s < KS; ++s)
#pragma unroll
        for (int u = 0; u < STEP; ++u)
#pragma unroll
          for (int m = 0; m < MT; ++m) acc[u][m] = M::mma(a[m][s], b[u][s], acc[u][m]);
#pragma unroll
      for (int u = 0; u < STEP; ++u)
        if (FULL || act[i0 + u]) {
#pragma unroll
          for (int m = 0; m < MT; ++m)
#pragma unroll
            for (int r = 0; r < 4; ++r) lds[ts(4 * m + r) ^ lb[i0 + u]] = acc[u][m][r];
        }
    }
  }
};

}  // namespace tanq

// Feeding a block's operations to the composition kernels (kernels.hip, real.hip): the chain over a block's
// operations is serial and each step is short, so it must not wait for memory.  A ring of 64 entries of the
// block's operation table is kept in LDS, and the superoperators stream into a ring of four LDS buffers
// with direct global-to-LDS loads issued three operations ahead.
#pragma once

#include "tile.hpp"

namespace tanq {

// E: element of a superoperator (f64x2 complex, double real).  256 threads; operations of at most two qubits
// come through the ring (D^2 <= 256 elements), three-qubit ones are read from memory by the caller.
template <typename E>
struct ComposeFeed {
  static constexpr int kTab = 64, kRing = 4, kAhead = 3;
  static constexpr int PER16 = 16 / (int)sizeof(E);     // elements per 16-byte load
  static constexpr int WAVES = 256 / PER16 / 64;        // waves that take part in a load
  struct Lds {
    FuseOpDev tab[kTab];
    __align__(16) E ring[kRing][256];
  };

  Lds& lds;
  const FuseOpDev* ops;  // of the block
  const E* sops;
  int count, tid, wave;

  __device__ ComposeFeed(Lds& l, const FuseOpDev* o, const E* s, int n)
      : lds(l), ops(o), sops(s), count(n), tid(threadIdx.x), wave(__builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6)) {}

  __device__ inline void table(int first, int end) {  // entries [first, end), at most 64
    if (end > count) end = count;
    const uint32_t* src = reinterpret_cast<const uint32_t*>(ops);
    uint32_t* dst = reinterpret_cast<uint32_t*>(lds.tab);
    constexpr int W = (int)(sizeof(FuseOpDev) / 4);
    for (int i = first * W + tid; i < end * W; i += 256) dst[i % (kTab * W)] = src[i];
  }
  // one load per wave that takes part, whatever the operation (lanes past its end repeat the last 16 bytes),
  // so that waits can count them
  __device__ inline void issue(int oi) {
    if (oi >= count || wave >= WAVES) return;  // uniform per wave
    const FuseOpDev& op = lds.tab[oi % kTab];
    const int j = __builtin_amdgcn_readfirstlane(op.j);
    const int last = (1 << (4 * (j < 2 ? j : 2))) / PER16 - 1;
    const int t = tid < last ? tid : last;
    const int64_t off = op.sop_off;
    pass_dma16(sops + off + (int64_t)t * PER16, lds_addr(lds.ring[oi % kRing]) + (uint32_t)wave * 1024u);
  }
  // before the first operation
  __device__ inline void start() {
    table(0, kTab);
    __syncthreads();
    for (int oi = 0; oi < kAhead; ++oi) issue(oi);
    wait(0);
    raw_barrier();
  }
  // this wave's load of operation oi is done when at most the later ones are outstanding
  __device__ inline void wait(int oi) {
    const int later = count - 1 - oi;  // issued after it: at most two
    if (later >= 2)
      vm_wait<2>();
    else if (later == 1)
      vm_wait<1>();
    else
      vm_wait<0>();
  }
  // At the start of operation oi: requests the one three ahead; every 32 operations, refills the half of
  // the table ring that has been used.
  __device__ inline void request(int oi) {
    if (oi > 0 && oi % (kTab / 2) == 0) table(oi + kTab / 2, oi + kTab);
    issue(oi + kAhead);
  }
  // at the end of operation oi: the next one's matrix is in LDS for every wave
  __device__ inline void next(int oi) {
    wait(oi + 1);
    raw_barrier();
  }
};

// ------------------------------------------------------------------------------------
// packing of FP64 superoperators into the apply kernels' A-operand lane layouts
// ------------------------------------------------------------------------------------

// k = 2, real block: R[m'][k'] for m' = 2a + cm, k' = 2b + ck is
//   (cm, ck) = (0,0): Re S[a][b]   (0,1): -Im S[a][b]   (1,0): Im S[a][b]   (1,1): Re S[a][b]
// stored as P[(mt * 8 + ks) * 64 + lane] = R[16 mt + lane % 16][4 ks + lane / 16].
// k = 3, 3M: P[((mt * 16 + ks) * 3 + c) * 64 + lane] = C_c[16 mt + lane % 16][4 ks + lane / 16]
//   with C_0 = Re S, C_1 = Im S, C_2 = Re S + Im S (summed in FP64, rounded once).
// k = 1: the FP64 superoperator itself (32 doubles), for both precisions.
// ld: elements per row of S (k = 3), which holds the columns from c0 on; nc of them, a multiple of four, are packed.
template <typename T>
__device__ void pack_block(int k, const double* __restrict__ S, unsigned char* __restrict__ out, int ld = 64, int c0 = 0,
                           int nc = 64) {
  if (k == 1) {
    double* P = reinterpret_cast<double*>(out);
    for (int e = threadIdx.x; e < 32; e += blockDim.x) P[e] = S[e];
  } else if (k == 2) {
    T* P = reinterpret_cast<T*>(out);
    for (int e = threadIdx.x; e < 2 * 8 * 64; e += blockDim.x) {
      const int lane = e & 63, rest = e >> 6;
      const int ks = rest % 8, mt = rest / 8;
      const int mrow = 16 * mt + (lane & 15), kcol = 4 * ks + (lane >> 4);
      const int a = mrow >> 1, cm = mrow & 1, b = kcol >> 1, ck = kcol & 1;
      const double re = S[2 * (a * 16 + b)], im = S[2 * (a * 16 + b) + 1];
      P[e] = (T)((cm == ck) ? re : (cm == 0 ? -im : im));
    }
  } else {
    T* P = reinterpret_cast<T*>(out);
    const int per = nc / 4 * 3;  // fragments per m-tile
    for (int e = threadIdx.x; e < 4 * per * 64; e += blockDim.x) {
      const int lane = e & 63, rest = e >> 6;
      const int mt = rest / per, f = c0 / 4 * 3 + rest % per, c = f % 3, ks = f / 3;
      const int a = 16 * mt + (lane & 15), b = 4 * ks + (lane >> 4) - c0;
      const double re = S[2 * (a * ld + b)], im = S[2 * (a * ld + b) + 1];
      P[(mt * 48 + f) * 64 + lane] = (T)(c == 0 ? re : (c == 1 ? im : re + im));
    }
  }
}

}  // namespace tanq

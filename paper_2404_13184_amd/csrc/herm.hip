// Long fused lists on Hermitian FP64 states, in real form (real.hpp): vec(rho) is checked,
// transformed in place to 4^n reals in the lower half of its memory, multiplied there, and
// transformed back.  A pass over the state then moves half the bytes and executes a third of the
// products of the 3M form.
//
// Whether the state is Hermitian is known only on the device, and applying a list never waits for
// the device, so the check leaves a flag that every kernel here reads at its start: they do nothing
// unless it is set, and the kernels of the complex form, queued beside them, do nothing if it is
// (apply.hip, pass.hip).
//
// The transform.  X = Re rho + Im rho is a real matrix that determines a Hermitian rho (Re is its
// symmetric part, Im its antisymmetric one), and the real form is the per-qubit butterfly of X,
// (x10, x01) -> half of (sum, difference) and x00, x11 as they are, up to a sign: of the two parts of each
// coefficient the butterflies of Re and Im give, one is zero, and (-i)^y takes the other to the coefficient up
// to (-1) when y mod 4 is 2 or 3 (y: the number of Y).  The inverse is (sum, difference).  Populations pass
// through unchanged, sums of exactly Hermitian input are exactly real, and the way back gives an exactly
// Hermitian matrix.
// The first step of the way in compacts (two complex elements that differ in the top column bit become
// one 16-byte pair of reals in the place of the lower one) on the qubits 0-4 and n - 1, which hold
// that bit and whole 128-byte lines; the others take up to five qubits each.  Way in and out together
// move as many bytes as about three passes of the complex form.
#include "real.hpp"

namespace tanq {

namespace {

// Entries beyond this could overflow where they are added; such a state keeps the complex form.
constexpr double kHermRange = 1e280;

__device__ inline bool flag_set(const uint32_t* flag) { return __builtin_amdgcn_readfirstlane((int)*flag) != 0; }

}  // namespace

__global__ void herm_flag_kernel(uint32_t* flag) { *flag = 1; }

// rho[r][c] = conj(rho[c][r]) over 32 x 32 blocks of the matrix and their mirror images: the block
// is read along its contiguous rows into LDS, the mirror along its own, so both reads are 512-byte
// runs.  Bound by reading the state once; a state that fails ends it early.
__global__ __launch_bounds__(256) void herm_check_kernel(const f64x2* __restrict__ rho, int n, uint32_t* flag) {
  __shared__ f64x2 blk[32][33];
  __shared__ uint32_t on;
  const int tid = threadIdx.x, i = tid & 31, j0 = tid >> 5;
  const uint32_t nb = 1u << (n - 5);  // blocks per side
  const uint64_t total = (uint64_t)nb * nb;
  for (uint64_t t = blockIdx.x; t < total; t += gridDim.x) {
    const uint32_t R = (uint32_t)(t & (nb - 1)), C = (uint32_t)(t >> (n - 5));
    if (R > C) continue;
    __syncthreads();  // the previous block is no longer read
    if (tid == 0) on = *(volatile const uint32_t*)flag;  // may still be the old value: it then checks on
    __syncthreads();
    if (!on) return;
    f64x2 a[4], b[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint64_t j = (uint64_t)(j0 + 8 * u);
      a[u] = rho[((uint64_t)R * 32 + i) + (((uint64_t)C * 32 + j) << n)];
      b[u] = rho[((uint64_t)C * 32 + i) + (((uint64_t)R * 32 + j) << n)];
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) blk[j0 + 8 * u][i] = a[u];
    __syncthreads();
    bool bad = false;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const f64x2 x = blk[i][j0 + 8 * u], y = b[u];  // rho[R*32 + j][C*32 + i] against its mirror
      bad |= !(x[0] == y[0] && x[1] == -y[1] && fabs(x[0]) < kHermRange && fabs(x[1]) < kHermRange);
    }
    if (__syncthreads_or(bad) && tid == 0) *(volatile uint32_t*)flag = 0;
  }
}

// One qubit's butterfly; INV: on the way back.
template <bool INV>
__device__ inline void butterfly2(double& x10, double& x01) {
  const double x = x10 + x01, y = x10 - x01;
  x10 = INV ? x : 0.5 * x;
  x01 = INV ? y : 0.5 * y;
}

// One or two qubits' butterflies on the tile in LDS: each group of 16 (or 4) elements by one thread.
// ra, ca, rb, cb: tile bits of the row and column bit of qubit A and B (rb < 0: one qubit).  ph: LDS
// place of a tile element, linear over GF(2), against bank conflicts.
template <bool INV, int V, int NT, typename Ph>
__device__ inline void tile_butterflies(double* t, int ra, int ca, int rb, int cb, int tid, Ph ph) {
  const uint32_t pra = ph(1u << ra), pca = ph(1u << ca);
  if (rb >= 0) {
    const uint32_t prb = ph(1u << rb), pcb = ph(1u << cb);
    const uint32_t fm = ((1u << V) - 1u) & ~((1u << ra) | (1u << ca) | (1u << rb) | (1u << cb));
    for (int g = tid; g < (1 << (V - 4)); g += NT) {
      const uint32_t base = ph(pdep32((uint32_t)g, fm));
      double x[16];  // l: bits of (row A, column A, row B, column B)
#pragma unroll
      for (int l = 0; l < 16; ++l)
        x[l] = t[base ^ ((l & 1) ? pra : 0u) ^ ((l & 2) ? pca : 0u) ^ ((l & 4) ? prb : 0u) ^ ((l & 8) ? pcb : 0u)];
#pragma unroll
      for (int h = 0; h < 4; ++h) butterfly2<INV>(x[4 * h + 1], x[4 * h + 2]);
#pragma unroll
      for (int h = 0; h < 4; ++h) butterfly2<INV>(x[h + 4], x[h + 8]);
#pragma unroll
      for (int l = 0; l < 16; ++l)
        t[base ^ ((l & 1) ? pra : 0u) ^ ((l & 2) ? pca : 0u) ^ ((l & 4) ? prb : 0u) ^ ((l & 8) ? pcb : 0u)] = x[l];
    }
  } else {
    const uint32_t fm = ((1u << V) - 1u) & ~((1u << ra) | (1u << ca));
    for (int g = tid; g < (1 << (V - 2)); g += NT) {
      const uint32_t e = ph(pdep32((uint32_t)g, fm));
      butterfly2<INV>(t[e ^ pra], t[e ^ pca]);
    }
  }
}

// Tile of the first step: index bits of the qubits 0-4 and n - 1 in vec(rho).  Tile bit order:
// rows 0-4, columns 0-4, row n - 1, column n - 1; so tile bits 0-10 with the top bit 0 are the pair's
// lower element.  Outside bits: rows and columns of the qubits 5..n-2.
constexpr int kEdgeV = 12, kEdgeNT = 512;

__device__ inline uint64_t edge_off(uint32_t e, int n) {  // tile element -> index
  return (uint64_t)(e & 31u) | ((uint64_t)((e >> 5) & 31u) << n) | ((uint64_t)((e >> 10) & 1u) << (n - 1)) |
         ((uint64_t)((e >> 11) & 1u) << (2 * n - 1));
}
__device__ inline uint64_t edge_base(uint32_t ro, uint32_t co, int n) {
  return ((uint64_t)ro << 5) | ((uint64_t)co << (n + 5));
}
// tile bits 7-9 go to bank bits 0-2 and 5-6 to 3-4, so that the lanes of the first butterflies (on tile
// bits 0, 1, 5, 6) fall on distinct banks
__device__ inline uint32_t edge_place(uint32_t e) { return e ^ ((e >> 7) & 7u) ^ (((e >> 5) & 3u) << 3); }
template <bool INV>
__device__ inline void edge_butterflies(double* t, int tid) {
  auto ph = [](uint32_t e) { return edge_place(e); };
  tile_butterflies<INV, kEdgeV, kEdgeNT>(t, 0, 5, 1, 6, tid, ph);
  __syncthreads();
  tile_butterflies<INV, kEdgeV, kEdgeNT>(t, 2, 7, 3, 8, tid, ph);
  __syncthreads();
  tile_butterflies<INV, kEdgeV, kEdgeNT>(t, 4, 9, 10, 11, tid, ph);
  __syncthreads();
}

__global__ __launch_bounds__(kEdgeNT) void herm_in_kernel(f64x2* __restrict__ rho, int n, const uint32_t* flag) {
  __shared__ double t[1 << kEdgeV];
  if (!flag_set(flag)) return;
  const int tid = threadIdx.x;
  const int no = n - 6;
  const uint64_t ntiles = 1ull << (2 * no);
  for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint64_t base = edge_base((uint32_t)(tile & ((1u << no) - 1u)), (uint32_t)(tile >> no), n);
    f64x2 v[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) v[u] = __builtin_nontemporal_load(rho + base + edge_off((uint32_t)(u * kEdgeNT + tid), n));
#pragma unroll
    for (int u = 0; u < 8; ++u) t[edge_place((uint32_t)(u * kEdgeNT + tid))] = v[u][0] + v[u][1];
    __syncthreads();
    edge_butterflies<false>(t, tid);
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const uint32_t e = (uint32_t)(u * kEdgeNT + tid);  // top column bit 0
      rho[base + edge_off(e, n)] = f64x2{t[edge_place(e)], t[edge_place(e | 2048u)]};
    }
    __syncthreads();
  }
}

// The last step of the way back: a tile and its mirror image (rows and columns of the outside bits
// exchanged) together, since rho[r][c] takes X[r][c] and X[c][r].
__global__ __launch_bounds__(kEdgeNT) void herm_out_kernel(f64x2* __restrict__ rho, int n,
                                                           const uint32_t* flag) {
  __shared__ double t[2][1 << kEdgeV];
  if (!flag_set(flag)) return;
  const int tid = threadIdx.x;
  const int no = n - 6;
  const uint64_t ntiles = 1ull << (2 * no);
  for (uint64_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
    const uint32_t ro = (uint32_t)(tile & ((1u << no) - 1u)), co = (uint32_t)(tile >> no);
    if (ro > co) continue;  // done with its mirror image
    const int sides = ro == co ? 1 : 2;
    const uint64_t base[2] = {edge_base(ro, co, n), edge_base(co, ro, n)};
    for (int s = 0; s < sides; ++s) {
      f64x2 v[4];
#pragma unroll
      for (int u = 0; u < 4; ++u) v[u] = rho[base[s] + edge_off((uint32_t)(u * kEdgeNT + tid), n)];
#pragma unroll
      for (int u = 0; u < 4; ++u) {
        const uint32_t e = (uint32_t)(u * kEdgeNT + tid);
        t[s][edge_place(e)] = v[u][0];
        t[s][edge_place(e | 2048u)] = v[u][1];
      }
    }
    __syncthreads();
    for (int s = 0; s < sides; ++s) edge_butterflies<true>(t[s], tid);
    for (int s = 0; s < sides; ++s) {
      const double* a = t[s];
      const double* b = t[sides == 2 ? s ^ 1 : 0];
#pragma unroll
      for (int u = 0; u < 8; ++u) {
        const uint32_t e = (uint32_t)(u * kEdgeNT + tid);
        // rows and columns exchanged inside the tile
        const uint32_t m = ((e & 31u) << 5) | ((e >> 5) & 31u) | ((e & 1024u) << 1) | ((e & 2048u) >> 1);
        const double x = a[edge_place(e)], y = b[edge_place(m)];
        __builtin_nontemporal_store(f64x2{0.5 * (x + y), 0.5 * (x - y)}, rho + base[s] + edge_off(e, n));
      }
    }
    __syncthreads();
  }
}

// Butterflies of the qubits q0..q0 + nq - 1 (at most five, from 5..n-2) on the reals.  A tile holds their
// row and column bits and the lowest other address bits up to 2^14 elements, so that five qubits leave
// whole 128-byte lines (with tiles of 2^13 the five-qubit steps at 16 qubits ran on half lines: 25 ms
// each instead of 13).  128 KiB of LDS, one workgroup of 16 waves per CU; the next tile is prefetched into
// registers.  Bound by memory: one read and one write of the reals.  sign: the factor -1 of
// the elements with y mod 4 in {2, 3} -- 1: after (the last step in), 2: before (the first step out).  INV: a step
// of the way back.
constexpr int kMidBits = 14, kMidNT = 1024;
struct HermMid {
  uint64_t dmask;     // address bits outside the tile
  uint64_t ntiles;
  uint8_t vpos[16];   // tile bit -> address bit
  int8_t rbit[6], cbit[6];  // tile bits of each qubit
  int32_t n, nq, sign;
};

template <bool INV>
__global__ __launch_bounds__(kMidNT) void herm_mid_kernel(double* __restrict__ w, const HermMid g, const uint32_t* flag) {
  constexpr int V = kMidBits, NT = kMidNT, IT = (1 << V) / 2 / NT;
  __shared__ f64x2 t2[(1 << V) / 2];
  if (!flag_set(flag)) return;
  double* t = reinterpret_cast<double*>(t2);
  const int tid = threadIdx.x;
  // tile bit 6 to bank bit 4 (the lanes of a five-qubit step's first butterflies)
  auto ph = [](uint32_t e) { return e ^ (((e >> 6) & 1u) << 4); };
  auto sign = [&](uint64_t a) {  // a: element address
    const uint64_t idx = (a >> 1) | ((a & 1ull) << (2 * g.n - 1));
    const uint64_t r = idx & ((1ull << g.n) - 1ull), c = idx >> g.n;
    return (__popcll(~r & c) & 2) ? -1.0 : 1.0;
  };
  // address offset of slot u * NT + tid: the bits of u and of tid are disjoint
  uint64_t off_t = 0;
#pragma unroll
  for (int b = 0; b < 10; ++b)
    if ((tid >> b) & 1) off_t |= 1ull << g.vpos[b + 1];
  auto off = [&](int u) {
    return off_t | ((u & 1) ? 1ull << g.vpos[11] : 0) | ((u & 2) ? 1ull << g.vpos[12] : 0) | ((u & 4) ? 1ull << g.vpos[13] : 0);
  };
  const uint64_t per = (g.ntiles + gridDim.x - 1) / gridDim.x;
  const uint64_t first = (uint64_t)blockIdx.x * per;
  const uint64_t end = first + per < g.ntiles ? first + per : g.ntiles;
  if (first >= end) return;  // uniform per workgroup
  uint64_t cur = pdep64(first, g.dmask);
  f64x2 v[IT];
#pragma unroll
  for (int u = 0; u < IT; ++u) v[u] = *reinterpret_cast<const f64x2*>(w + cur + off(u));
  for (uint64_t tile = first;; ++tile) {
    if (g.sign == 2) {
#pragma unroll
      for (int u = 0; u < IT; ++u) {
        v[u][0] *= sign(cur + off(u));
        v[u][1] *= sign(cur + off(u) + 1);
      }
    }
#pragma unroll
    for (int u = 0; u < IT; ++u) t2[ph((uint32_t)(u * NT + tid) * 2u) >> 1] = v[u];
    lds_barrier();
    const bool more = tile + 1 < end;
    const uint64_t next = more ? ((cur | ~g.dmask) + 1ull) & g.dmask : 0;
    if (more) {
#pragma unroll
      for (int u = 0; u < IT; ++u) v[u] = *reinterpret_cast<const f64x2*>(w + next + off(u));
    }
    for (int q = 0; q < g.nq; q += 2) {
      const bool two = q + 1 < g.nq;
      tile_butterflies<INV, V, NT>(t, g.rbit[q], g.cbit[q], two ? g.rbit[q + 1] : -1, two ? g.cbit[q + 1] : -1, tid, ph);
      lds_barrier();
    }
#pragma unroll
    for (int u = 0; u < IT; ++u) {
      f64x2 x = t2[ph((uint32_t)(u * NT + tid) * 2u) >> 1];
      if (g.sign == 1) {
        x[0] *= sign(cur + off(u));
        x[1] *= sign(cur + off(u) + 1);
      }
      *reinterpret_cast<f64x2*>(w + cur + off(u)) = x;
    }
    if (!more) break;
    lds_barrier();  // this tile is read out of LDS
    cur = next;
  }
}

// ------------------------------------------------------------------------------------
// superoperators
// ------------------------------------------------------------------------------------

// A three-qubit superoperator: tiles of 2^12 reals (32 KiB) prefetched through registers into the
// other of two LDS buffers while a wave multiplies its own 16 groups in place (OpReal).
__global__ __launch_bounds__(256, 2) void real_apply3_kernel(double* __restrict__ w, const double* __restrict__ frag,
                                                             const RealGeom g, const uint32_t* flag) {
  constexpr int V = 12, NT = 256;
  using IO = RealIo<V, NT>;
  using Op = OpReal<3, V, NT>;
  __shared__ u32x4 lds[2][IO::SLOTS];
  if (!flag_set(flag)) return;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const uint32_t per = (g.ntiles + gridDim.x - 1) / gridDim.x;
  const uint32_t first = blockIdx.x * per;
  const uint32_t end = first + per < g.ntiles ? first + per : g.ntiles;
  if (first >= end) return;
  IO io;
  io.init(g, tid);
  Op op;
  op.load(frag, lane);
  op.prepare(g, lane, wave);
  real_tiles<true>(w, io, op, [&](uint32_t t) { return (uint32_t)tile_base(g, t); }, lds, first, end, tid);
}

// ------------------------------------------------------------------------------------
// operands
// ------------------------------------------------------------------------------------

__global__ __launch_bounds__(256) void pack_herm_kernel(const RealPackDev* __restrict__ blocks,
                                                        const double* __restrict__ raw, double* __restrict__ packed) {
  const RealPackDev b = blocks[blockIdx.x];
  const f64x2* S = reinterpret_cast<const f64x2*>(raw + 2 * b.raw_off);
  double* P = packed + b.pack_off;
  const int D = 1 << (2 * b.k);
  auto local = [&](int x) {
    uint32_t r = 0;
    for (int t = 0; t < 2 * b.k; ++t) r |= (uint32_t)((x >> t) & 1) << b.perm[t];
    return r;
  };
  for (int e = threadIdx.x; e < D * D; e += blockDim.x) {
    int row = e / D, col = e % D;
    if (b.k > 1) real_frag_index(e, D / 4, &row, &col);
    P[e] = real_entry(S, b.k, local(row), local(col));
  }
}

// ------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------

void launch_pack_herm(const RealPackDev* blocks, int nblocks, const double* raw, double* packed, hipStream_t s) {
  if (nblocks <= 0) return;
  hipLaunchKernelGGL(pack_herm_kernel, dim3(nblocks), dim3(256), 0, s, blocks, raw, packed);
  TANQ_HIP(hipGetLastError());
}

static unsigned herm_grid(uint64_t tiles, int per_cu) {
  const uint64_t cap = (uint64_t)device_cu_count() * (uint64_t)per_cu;
  return (unsigned)(tiles < cap ? tiles : cap);
}

void launch_herm_check(const void* rho, int n, uint32_t* flag, hipStream_t s) {
  if (n < kHermMinN || n > kHermMaxN) fail(TANQ_E_STATE, "real form: qubit count");
  hipLaunchKernelGGL(herm_flag_kernel, dim3(1), dim3(1), 0, s, flag);
  TANQ_HIP(hipGetLastError());
  hipLaunchKernelGGL(herm_check_kernel, dim3(herm_grid(1ull << (2 * (n - 5)), 32)), dim3(256), 0, s,
                     (const f64x2*)rho, n, flag);
  TANQ_HIP(hipGetLastError());
}

template <bool INV>
static void launch_herm_mid(void* rho, int n, int q0, int nq, int sign, const uint32_t* flag, hipStream_t s) {
  HermMid g{};
  g.n = n;
  g.nq = nq;
  g.sign = sign;
  uint64_t held = 0;
  for (int i = 0; i < nq; ++i) held |= (1ull << (q0 + i + 1)) | (1ull << (q0 + i + n + 1));
  for (int b = 0; __builtin_popcountll(held) < kMidBits; ++b) held |= 1ull << b;
  int cnt = 0, local_of[64] = {0};
  for (int b = 0; b < 2 * n; ++b)
    if ((held >> b) & 1ull) {
      local_of[b] = cnt;
      g.vpos[cnt++] = (uint8_t)b;
    }
  for (int i = 0; i < nq; ++i) {
    g.rbit[i] = (int8_t)local_of[q0 + i + 1];
    g.cbit[i] = (int8_t)local_of[q0 + i + n + 1];
  }
  g.dmask = ((1ull << (2 * n)) - 1ull) & ~held;
  g.ntiles = 1ull << (2 * n - kMidBits);
  hipLaunchKernelGGL(herm_mid_kernel<INV>, dim3(herm_grid(g.ntiles, 1)), dim3(kMidNT), 0, s, (double*)rho, g, flag);
  TANQ_HIP(hipGetLastError());
}

// the qubits 5..n-2 in steps of at most five, as evenly as they come
static int herm_steps(int n) { return (n - 6 + 4) / 5; }

void launch_herm_in(void* rho, int n, const uint32_t* flag, hipStream_t s) {
  hipLaunchKernelGGL(herm_in_kernel, dim3(herm_grid(1ull << (2 * (n - 6)), 4)), dim3(kEdgeNT), 0, s, (f64x2*)rho, n, flag);
  TANQ_HIP(hipGetLastError());
  const int steps = herm_steps(n), total = n - 6;
  for (int i = 0, q = 5; i < steps; ++i) {
    const int nq = total / steps + (i < total % steps ? 1 : 0);
    launch_herm_mid<false>(rho, n, q, nq, i + 1 == steps ? 1 : 0, flag, s);
    q += nq;
  }
}

void launch_herm_out(void* rho, int n, const uint32_t* flag, hipStream_t s) {
  const int steps = herm_steps(n), total = n - 6;
  for (int i = 0, q = 5; i < steps; ++i) {
    const int nq = total / steps + (i < total % steps ? 1 : 0);
    launch_herm_mid<true>(rho, n, q, nq, i == 0 ? 2 : 0, flag, s);
    q += nq;
  }
  hipLaunchKernelGGL(herm_out_kernel, dim3(herm_grid(1ull << (2 * (n - 6)), 2)), dim3(kEdgeNT), 0, s, (f64x2*)rho, n,
                     flag);
  TANQ_HIP(hipGetLastError());
}

void launch_real_apply3(void* rho, int n, const int* qubits, const double* packed, const uint32_t* flag, hipStream_t s) {
  int tbits[6];
  for (int t = 0; t < 3; ++t) {
    tbits[t] = qubits[t] + 1;
    tbits[3 + t] = qubits[t] == n - 1 ? 0 : qubits[t] + n + 1;
  }
  const RealGeom g = make_real_geom(2 * n, 3, tbits, 12);
  hipLaunchKernelGGL(real_apply3_kernel, dim3(herm_grid(g.ntiles, 2)), dim3(256), 0, s, (double*)rho, packed, g, flag);
  TANQ_HIP(hipGetLastError());
}

}  // namespace tanq

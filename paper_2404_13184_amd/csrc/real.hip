// Kernels of the real (Pauli) form (real.hpp): operands, initial state and outputs.
//
// The form's basis change per qubit is a butterfly of (rho_00, rho_11) and (rho_10, rho_01), so a
// superoperator S becomes R[a][b] = Re((-i)^(y_a - y_b) 2^-k sum_{u,v} (-1)^(u.c_a + v.c_b)
// S[i(a,u)][i(b,v)]), i(a, u) = (u ^ r_a ^ c_a) + 2^k u, where (r, c) are a local index's row and
// column halves and y = popcount(~r & c).  For S = sum_i conj(K_i) (x) K_i the imaginary part of
// that expression is zero.
#include "real.hpp"

namespace tanq {

// One workgroup per operation: S in LDS, then its real form.
__global__ __launch_bounds__(256) void build_real_kernel(const FuseOpDev* __restrict__ ops,
                                                         const double* __restrict__ kraus, double* __restrict__ sops) {
  __shared__ f64x2 S[64 * 64];
  const FuseOpDev op = ops[blockIdx.x];
  const int j = op.j, d = 1 << j, dd = d * d;
  const double* K = kraus + 2 * op.kraus_off;
  for (int e = threadIdx.x; e < dd * dd; e += blockDim.x) {
    const int a = e / dd, b = e % dd;
    const int ar = a & (d - 1), ac = a >> j, br = b & (d - 1), bc = b >> j;
    double sr = 0.0, si = 0.0;
    for (int i = 0; i < op.m; ++i) {
      const double* Ki = K + 2 * (size_t)i * d * d;
      const double xr = Ki[2 * (ac * d + bc)], xi = -Ki[2 * (ac * d + bc) + 1];  // conj
      const double yr = Ki[2 * (ar * d + br)], yi = Ki[2 * (ar * d + br) + 1];
      sr += xr * yr - xi * yi;
      si += xr * yi + xi * yr;
    }
    S[e] = f64x2{sr, si};
  }
  __syncthreads();
  for (int e = threadIdx.x; e < dd * dd; e += blockDim.x)
    sops[op.sop_off + e] = real_entry(S, j, (uint32_t)(e / dd), (uint32_t)(e % dd));
}

// One workgroup per block: M <- R_op(embedded) M in circuit order from M = I, out of place between
// two LDS buffers (one barrier per operation), then M in the operand layout.  The chain over a
// block's operations is serial and each step is short, so what counts is its latency: the next
// operation's matrix is loaded into registers while the current one is applied.  Thread t works
// on column t % D; the 256 / D threads of a column share its groups and outputs.
template <typename T, int K>
__global__ __launch_bounds__(256) void compose_real_kernel(const FuseBlockDev* __restrict__ blocks,
                                                           const FuseOpDev* __restrict__ ops,
                                                           const double* __restrict__ sops,
                                                           unsigned char* __restrict__ packed) {
  constexpr int D = 1 << (2 * K), SLOTS = 256 / D;
  __shared__ double M[2][D * D];
  __shared__ double Sl[2][256];
  const FuseBlockDev blk = blocks[blockIdx.x];
  const int tid = threadIdx.x, c = tid % D, slot = tid / D;
  for (int e = tid; e < D * D; e += 256) M[0][e] = (e / D) == (e % D) ? 1.0 : 0.0;
  FuseOpDev op = ops[blk.op_begin];
  if (blk.op_count > 0 && op.j <= 2 && tid < (1 << (4 * op.j))) Sl[0][tid] = sops[op.sop_off + tid];
  __syncthreads();
  int cur = 0;
  for (int oi = 0; oi < blk.op_count; ++oi) {
    const bool more = oi + 1 < blk.op_count;
    const FuseOpDev nop = more ? ops[blk.op_begin + oi + 1] : op;
    double pre = 0.0;
    const bool fetch = more && nop.j <= 2 && tid < (1 << (4 * nop.j));
    if (fetch) pre = sops[nop.sop_off + tid];

    const double* X = M[cur];
    double* Y = M[cur ^ 1];
    const double* S = Sl[oi & 1];
    const int j = op.j, Dj = 1 << (2 * j);
    // row bits (within M) of the operation's local index bits
    uint32_t tbit[6] = {0, 0, 0, 0, 0, 0}, tmask = 0;
    for (int t = 0; t < j; ++t) {
      tbit[t] = 1u << op.pos[t];
      tbit[j + t] = 1u << (K + op.pos[t]);
      tmask |= tbit[t] | tbit[j + t];
    }
    auto dep = [&](int l) {
      uint32_t r = 0;
      for (int t = 0; t < 2 * j; ++t)
        if ((l >> t) & 1) r |= tbit[t];
      return r;
    };
    const uint32_t freemask = (uint32_t)(D - 1) & ~tmask;
    if (j <= 2) {
      // work items of a column: (group, run of outputs); as many runs per group as the threads of a
      // column need to have one each
      const int groups = D / Dj;
      const int split = groups < SLOTS ? SLOTS / groups : 1;
      const int outs = Dj / split;  // at least 1: SLOTS <= D
      for (int it = slot; it < groups * split; it += SLOTS) {
        const uint32_t base = pdep32((uint32_t)(it / split), freemask);
        const int a0 = (it % split) * outs;
        if (j == 1) {
          double x[4];
#pragma unroll
          for (int b = 0; b < 4; ++b) x[b] = X[(base | dep(b)) * D + c];
          for (int a = a0; a < a0 + outs; ++a) {
            double y = 0.0;
#pragma unroll
            for (int b = 0; b < 4; ++b) y += S[a * 4 + b] * x[b];
            Y[(base | dep(a)) * D + c] = y;
          }
        } else {
          double x[16];
#pragma unroll
          for (int b = 0; b < 16; ++b) x[b] = X[(base | dep(b)) * D + c];
          for (int a = a0; a < a0 + outs; ++a) {
            double y = 0.0;
#pragma unroll
            for (int b = 0; b < 16; ++b) y += S[a * 16 + b] * x[b];
            Y[(base | dep(a)) * D + c] = y;
          }
        }
      }
    } else if constexpr (K == 3) {
      const double* Sg = sops + op.sop_off;
      for (int a = slot; a < D; a += SLOTS) {
        double y = 0.0;
        for (int b = 0; b < D; ++b) y += Sg[a * D + b] * X[dep(b) * D + c];
        Y[dep(a) * D + c] = y;
      }
    }
    if (fetch) Sl[(oi + 1) & 1][tid] = pre;
    __syncthreads();
    cur ^= 1;
    op = nop;
  }
  T* P = reinterpret_cast<T*>(packed + blk.pack_off);
  for (int e = tid; e < D * D; e += 256) {
    int row, col;
    real_frag_index<T>(e, D / 4, &row, &col);
    P[e] = (T)M[cur][row * D + col];
  }
}

// |0..0><0..0| has expectation 1 for every string of I and Z (r' = c') and 0 for the others.
template <typename T>
__global__ void real_init_kernel(T* __restrict__ w, int n) {
  const uint64_t nel = 1ull << (2 * n), dim = 1ull << n;
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nel; i += (uint64_t)gridDim.x * blockDim.x)
    w[i] = (i & (dim - 1)) == (i >> n) ? T(1) : T(0);
}

// One workgroup: p_x = 2^-n sum_z (-1)^(x.z) w[z, z] is a Walsh-Hadamard transform of the diagonal (in
// LDS, FP64); every other output is one element of w.
template <typename T, int NMAX>
__global__ __launch_bounds__(1024) void real_outputs_kernel(const T* __restrict__ w, int n, int want_probs, int count,
                                                            const uint64_t* __restrict__ masks,
                                                            double* __restrict__ out) {
  __shared__ double p[1 << NMAX];
  const uint32_t dim = 1u << n;
  const double tr = (double)w[0];
  if (threadIdx.x == 0) out[0] = tr;
  double* res = out + 1;
  if (want_probs) {
    for (uint32_t z = threadIdx.x; z < dim; z += 1024) p[z] = (double)w[z + ((uint64_t)z << n)];
    __syncthreads();
    for (int t = 0; t < n; ++t) {
      for (uint32_t i = threadIdx.x; i < dim / 2; i += 1024) {
        const uint32_t lo = i & ((1u << t) - 1u), x0 = ((i >> t) << (t + 1)) | lo, x1 = x0 | (1u << t);
        const double a = p[x0], b = p[x1];
        p[x0] = a + b;
        p[x1] = a - b;
      }
      __syncthreads();
    }
    const double inv = 1.0 / tr, scale = 1.0 / (double)dim;
    for (uint32_t x = threadIdx.x; x < dim; x += 1024) res[x] = (p[x] * scale) * inv;
    res += dim;
  }
  for (int i = threadIdx.x; i < count; i += 1024) {
    const uint64_t xm = masks[3 * i], zm = masks[3 * i + 1];
    res[2 * i] = (double)w[(xm ^ zm) + (zm << n)];
    res[2 * i + 1] = 0.0;  // rho is Hermitian
  }
}

// ------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------

RealGeom make_real_geom(int nb, int k, const int* tbits, int vbits, tanq_prec p) {
  RealGeom g{};
  const int V = vbits < nb ? vbits : nb;
  uint64_t tmask = 0;
  for (int t = 0; t < 2 * k; ++t) tmask |= 1ull << tbits[t];
  uint64_t vmask = tmask;
  for (int b = 0, need = V - 2 * k; b < nb && need > 0; ++b)
    if (!((vmask >> b) & 1ull)) {
      vmask |= 1ull << b;
      --need;
    }
  int cnt = 0, nt = 0;
  uint32_t tlocal = 0;
  for (int b = 0; b < nb; ++b) {
    if (!((vmask >> b) & 1ull)) continue;
    if ((tmask >> b) & 1ull) {
      g.tpos[nt++] = (uint8_t)cnt;
      tlocal |= 1u << cnt;
    }
    g.vpos[cnt++] = (uint8_t)b;
  }
  g.V = V;
  g.G = 1 << (V - 2 * k);
  g.free_mask = ((1u << V) - 1u) & ~tlocal;
  // LDS swizzle.  The bits that differ between the lanes of one access are the four lowest free bits
  // (16 groups) and the lowest target bits (rows l / 16: two of them over 64 lanes of 4 bytes, one
  // over 32 lanes of 8 bytes).  Those above the 256-byte window are XORed into the window bits that
  // none of them covers.  Bits inside a 16-byte slot are never destinations: such a bit is free
  // (then it is among the lowest four) or a target (then it is among the lowest).
  const int w = p == TANQ_F64 ? 5 : 6, lo = p == TANQ_F64 ? 1 : 2;
  uint32_t lanes = 0;
  int nf = 0;
  for (int b = 0; b < V && nf < 4; ++b)
    if ((g.free_mask >> b) & 1u) {
      lanes |= 1u << b;
      ++nf;
    }
  for (int t = 0; t < w - 4; ++t) lanes |= 1u << g.tpos[t];
  int np = 0;
  for (int p2 = 0; p2 < kRealSwzPairs; ++p2) g.xsrc[p2] = 31;
  for (int b = w, d = lo; b < V; ++b) {
    if (!((lanes >> b) & 1u)) continue;
    while (d < w && ((lanes >> d) & 1u)) ++d;
    if (d >= w || np >= kRealSwzPairs) break;
    g.xsrc[np] = (uint8_t)b;
    g.xdst[np++] = (uint8_t)d++;
  }
  int src = 0, nr = 0;
  for (int b = 0; b < nb;) {
    if ((vmask >> b) & 1ull) {
      ++b;
      continue;
    }
    int e = b;
    while (e < nb && !((vmask >> e) & 1ull)) ++e;
    g.run_src[nr] = (uint8_t)src;
    g.run_len[nr] = (uint8_t)(e - b);
    g.run_dst[nr] = (uint8_t)b;
    src += e - b;
    ++nr;
    b = e;
  }
  g.nruns = nr;
  g.ntiles = 1u << (nb - V);
  return g;
}

void launch_build_real(const FuseOpDev* ops, int nops, const double* kraus, double* sops, hipStream_t s) {
  if (nops <= 0) return;
  hipLaunchKernelGGL(build_real_kernel, dim3(nops), dim3(256), 0, s, ops, kraus, sops);
  TANQ_HIP(hipGetLastError());
}

template <typename T>
static void compose_real_typed(const FuseBlockDev* blocks, int nblocks, int k, const FuseOpDev* ops,
                               const double* sops, void* packed, hipStream_t s) {
  if (k == 2)
    hipLaunchKernelGGL((compose_real_kernel<T, 2>), dim3(nblocks), dim3(256), 0, s, blocks, ops, sops,
                       (unsigned char*)packed);
  else if (k == 3)
    hipLaunchKernelGGL((compose_real_kernel<T, 3>), dim3(nblocks), dim3(256), 0, s, blocks, ops, sops,
                       (unsigned char*)packed);
  else
    fail(TANQ_E_ARG, "real blocks have two or three qubits");
  TANQ_HIP(hipGetLastError());
}

void launch_compose_real(const FuseBlockDev* blocks, int nblocks, int k, const FuseOpDev* ops, const double* sops,
                         void* packed, tanq_prec p, hipStream_t s) {
  if (nblocks <= 0) return;
  if (p == TANQ_F64)
    compose_real_typed<double>(blocks, nblocks, k, ops, sops, packed, s);
  else
    compose_real_typed<float>(blocks, nblocks, k, ops, sops, packed, s);
}

void launch_real_init(void* w, int n, tanq_prec p, hipStream_t s) {
  uint64_t blocks = ((1ull << (2 * n)) + 1023) / 1024;
  const uint64_t cap = (uint64_t)device_cu_count() * 16;
  if (blocks > cap) blocks = cap;
  if (p == TANQ_F64)
    hipLaunchKernelGGL(real_init_kernel<double>, dim3((unsigned)blocks), dim3(256), 0, s, (double*)w, n);
  else
    hipLaunchKernelGGL(real_init_kernel<float>, dim3((unsigned)blocks), dim3(256), 0, s, (float*)w, n);
  TANQ_HIP(hipGetLastError());
}

template <typename T>
static void real_outputs_typed(const void* w, int n, int want_probs, int count, const uint64_t* masks, double* out,
                               hipStream_t s) {
  // two LDS sizes: up to 12 qubits (32 KiB) and up to 14 (128 KiB)
  if (n <= 12)
    hipLaunchKernelGGL((real_outputs_kernel<T, 12>), dim3(1), dim3(1024), 0, s, (const T*)w, n, want_probs, count,
                       masks, out);
  else
    hipLaunchKernelGGL((real_outputs_kernel<T, kRealOutMaxN>), dim3(1), dim3(1024), 0, s, (const T*)w, n, want_probs,
                       count, masks, out);
  TANQ_HIP(hipGetLastError());
}

void launch_real_outputs(const void* w, int n, tanq_prec p, int want_probs, int count, const uint64_t* masks,
                         double* out, hipStream_t s) {
  if (n > kRealOutMaxN) fail(TANQ_E_ARG, "outputs of a real-form state: too many qubits");
  if (p == TANQ_F64)
    real_outputs_typed<double>(w, n, want_probs, count, masks, out, s);
  else
    real_outputs_typed<float>(w, n, want_probs, count, masks, out, s);
}

}  // namespace tanq

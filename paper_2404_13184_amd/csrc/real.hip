// Kernels of the real form (real.hpp): operands, initial state and outputs.
#include "compose.hpp"
#include "real.hpp"

namespace tanq {

// One workgroup per operation: S in LDS, then R.
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

// One workgroup per block: M <- R_op(embedded) M in circuit order from M = I, out of place between two LDS buffers (one
// barrier per operation), then the operand's fragments.  Thread t works on column t % D; the 256 / D threads of a
// column share its groups and outputs.  The chain over a block's operations is serial: ComposeFeed keeps it from
// waiting for memory.
template <int K>
__global__ __launch_bounds__(256) void compose_real_kernel(const FuseBlockDev* __restrict__ blocks,
                                                           const FuseOpDev* __restrict__ ops,
                                                           const double* __restrict__ sops,
                                                           unsigned char* __restrict__ packed) {
  constexpr int D = 1 << (2 * K), SLOTS = 256 / D;
  __shared__ double M[2][D * D];
  __shared__ typename ComposeFeed<double>::Lds fl;
  const FuseBlockDev blk = blocks[blockIdx.x];
  const int tid = threadIdx.x, c = tid % D, slot = tid / D;
  for (int e = tid; e < D * D; e += 256) M[0][e] = e / D == e % D ? 1.0 : 0.0;
  ComposeFeed<double> feed(fl, ops + blk.op_begin, sops, blk.op_count);
  feed.start();
  int cur = 0;
  for (int oi = 0; oi < blk.op_count; ++oi) {
    feed.request(oi);
    const FuseOpDev& op = fl.tab[oi % feed.kTab];
    const double* X = M[cur];
    double* Y = M[cur ^ 1];
    const double* S = fl.ring[oi % feed.kRing];
    const int j = __builtin_amdgcn_readfirstlane(op.j);
    // row bits (within M) of the operation's local index bits
    uint32_t tb[6], tmask = 0;
#pragma unroll
    for (int t = 0; t < 6; ++t) {
      const int q = t < j ? t : t - j;
      tb[t] = t < 2 * j ? 1u << ((t < j ? 0 : K) + __builtin_amdgcn_readfirstlane(op.pos[q < 3 ? q : 0])) : 0u;
      tmask |= tb[t];
    }
    auto dep = [&](int l) {
      uint32_t r = 0;
#pragma unroll
      for (int t = 0; t < 6; ++t)
        if ((l >> t) & 1) r |= tb[t];
      return r;
    };
    const uint32_t fm = (uint32_t)(D - 1) & ~tmask;
    if (j == 1) {
      if constexpr (K == 2) {  // one output each: group slot / 4, output slot % 4
        const uint32_t base = pdep32((uint32_t)(slot >> 2), fm);
        const int a = slot & 3;
        double y = 0.0;
#pragma unroll
        for (int b = 0; b < 4; ++b) y += S[a * 4 + b] * X[(base | dep(b)) * D + c];
        Y[(base | dep(a)) * D + c] = y;
      } else {
        for (int g = slot; g < D / 4; g += SLOTS) {
          const uint32_t base = pdep32((uint32_t)g, fm);
          double x[4];
#pragma unroll
          for (int b = 0; b < 4; ++b) x[b] = X[(base | dep(b)) * D + c];
#pragma unroll
          for (int a = 0; a < 4; ++a) {
            double y = 0.0;
#pragma unroll
            for (int b = 0; b < 4; ++b) y += S[a * 4 + b] * x[b];
            Y[(base | dep(a)) * D + c] = y;
          }
        }
      }
    } else if (j == 2) {
      if constexpr (K == 2) {  // one group; one output each
        double y = 0.0;
#pragma unroll
        for (int b = 0; b < 16; ++b) y += S[slot * 16 + b] * X[dep(b) * D + c];
        Y[dep(slot) * D + c] = y;
      } else {  // one group each, all its outputs
        const uint32_t base = pdep32((uint32_t)slot, fm);
        double x[16];
#pragma unroll
        for (int b = 0; b < 16; ++b) x[b] = X[(base | dep(b)) * D + c];
#pragma unroll 4
        for (int a = 0; a < 16; ++a) {
          double y = 0.0;
#pragma unroll
          for (int b = 0; b < 16; ++b) y += S[a * 16 + b] * x[b];
          Y[(base | dep(a)) * D + c] = y;
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
    feed.next(oi);
    cur ^= 1;
  }
  double* P = reinterpret_cast<double*>(packed + blk.pack_off);
  for (int e = tid; e < D * D; e += 256) {
    int row, col;
    real_frag_index(e, D / 4, &row, &col);
    P[e] = M[cur][row * D + col];
  }
}

// |0..0><0..0| is an element of the basis.
__global__ void real_init_kernel(double* __restrict__ w, int n) {
  const uint64_t nel = 1ull << (2 * n);
  for (uint64_t i = (uint64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nel; i += (uint64_t)gridDim.x * blockDim.x)
    w[i] = i == 0 ? 1.0 : 0.0;
}

// Workgroup 0: the trace and the probabilities, which are coefficients.  Workgroup 1 + i: string i, which is non-zero on
// the basis elements with X and Y where it has them: Tr(P B) = 2 on those qubits and +-1 (Z) or 1 on the
// populations of the others.
__global__ __launch_bounds__(1024) void real_outputs_kernel(const double* __restrict__ w, int n, int want_probs,
                                                            const uint64_t* __restrict__ masks, double* __restrict__ out) {
  constexpr int PER = 1 << (kRealOutMaxN - 10);  // values of a thread
  __shared__ double part[16];
  const uint32_t dim = 1u << n;
  const bool string = blockIdx.x > 0;
  const uint32_t xm = string ? (uint32_t)masks[3 * (blockIdx.x - 1)] : 0u;
  const uint32_t zm = string ? (uint32_t)masks[3 * (blockIdx.x - 1) + 1] : 0u;
  const uint32_t free = (dim - 1u) & ~xm, count = dim >> __popc(xm);
  const uint64_t at = (uint64_t)(xm & ~zm) + ((uint64_t)(xm & zm) << n);
  double v[PER], acc = 0.0;
#pragma unroll
  for (int u = 0; u < PER; ++u) {
    const uint32_t i = u * 1024 + threadIdx.x;
    v[u] = 0.0;
    if (i < count) {
      const uint32_t x = pdep32(i, free);
      const double e = w[at + x + ((uint64_t)x << n)];
      v[u] = (__popc(x & zm) & 1) ? -e : e;
    }
    acc += v[u];
  }
  for (int o = 32; o > 0; o >>= 1) acc += __shfl_down(acc, o, 64);
  if ((threadIdx.x & 63) == 0) part[threadIdx.x >> 6] = acc;
  __syncthreads();
  acc = 0.0;
  for (int i = 0; i < 16; ++i) acc += part[i];
  if (string) {
    double* res = out + 1 + (want_probs ? dim : 0u) + 2 * (blockIdx.x - 1);
    if (threadIdx.x == 0) {
      res[0] = acc * (double)(1u << __popc(xm));
      res[1] = 0.0;  // rho is Hermitian
    }
    return;
  }
  if (threadIdx.x == 0) out[0] = acc;
  if (want_probs) {
    const double inv = 1.0 / acc;
#pragma unroll
    for (int u = 0; u < PER; ++u)
      if (u * 1024 + threadIdx.x < dim) out[1 + u * 1024 + threadIdx.x] = v[u] * inv;
  }
}

// ------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------

RealGeom make_real_geom(int nb, int k, const int* tbits, int vbits) {
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
  // (16 groups) and the lowest target bit (rows l / 16, over 32 lanes).  Those above the 256-byte window are
  // XORed into the window bits that none of them covers.  The bit inside a 16-byte slot is never a
  // destination: it is free (then among the lowest four) or a target (then the lowest).
  constexpr int w = 5, lo = 1;
  uint32_t lanes = 0;
  int nf = 0;
  for (int b = 0; b < V && nf < 4; ++b)
    if ((g.free_mask >> b) & 1u) {
      lanes |= 1u << b;
      ++nf;
    }
  lanes |= 1u << g.tpos[0];
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

void launch_compose_real(const FuseBlockDev* blocks, int nblocks, int k, const FuseOpDev* ops, const double* sops,
                         void* packed, hipStream_t s) {
  if (nblocks <= 0) return;
  if (k == 2)
    hipLaunchKernelGGL(compose_real_kernel<2>, dim3(nblocks), dim3(256), 0, s, blocks, ops, sops, (unsigned char*)packed);
  else if (k == 3)
    hipLaunchKernelGGL(compose_real_kernel<3>, dim3(nblocks), dim3(256), 0, s, blocks, ops, sops, (unsigned char*)packed);
  else
    fail(TANQ_E_ARG, "real blocks have two or three qubits");
  TANQ_HIP(hipGetLastError());
}

void launch_real_init(void* w, int n, hipStream_t s) {
  uint64_t blocks = ((1ull << (2 * n)) + 1023) / 1024;
  const uint64_t cap = (uint64_t)device_cu_count() * 16;
  if (blocks > cap) blocks = cap;
  hipLaunchKernelGGL(real_init_kernel, dim3((unsigned)blocks), dim3(256), 0, s, (double*)w, n);
  TANQ_HIP(hipGetLastError());
}

void launch_real_outputs(const void* w, int n, int want_probs, int count, const uint64_t* masks, double* out, hipStream_t s) {
  if (n > kRealOutMaxN) fail(TANQ_E_ARG, "outputs of a real-form state: too many qubits");
  hipLaunchKernelGGL(real_outputs_kernel, dim3(1 + count), dim3(1024), 0, s, (const double*)w, n, want_probs, masks, out);
  TANQ_HIP(hipGetLastError());
}

}  // namespace tanq

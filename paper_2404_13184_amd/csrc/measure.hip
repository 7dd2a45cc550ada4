// Measurement statistics (gfx950, FP64): probabilities, readout error, shots, Pauli expectations, reduced
// density matrices.
//
// These calls look at 2^n of the 4^n elements (a diagonal, or one generalised diagonal per string), every one
// in a cache line of its own, and wait for the result: on states of up to 13 qubits a call is a few
// microseconds of work, so what counts is the number of launches and copies.  There one workgroup does the
// whole call with the probabilities in LDS (at most 64 KiB), and every kernel writes its results straight
// into the caller's pinned buffer.  Larger states: the diagonal by many workgroups, then the readout error
// of the 12 lowest qubits in LDS together with the normalisation, then that of the others in registers;
// shots from prefix sums within blocks of 4096 outcomes and the blocks' totals.
// One after the other (probabilities, readout error, 1000 shots, 7 strings, a reduced matrix): 7 qubits
// 300 -> 93 us, 16 qubits in FP32 (100,000 shots, 48 strings, three qubits kept) 771 ->
// 330 us (of which the strings, one cache line per element, are about 80, 10 of them the fixed order of the sums).
#include "tile.hpp"

namespace tanq {

namespace {

constexpr int kSmallN = 13;              // one workgroup, 2^13 probabilities in LDS
constexpr uint64_t kSmallShots = 16384;  // shots one workgroup draws
constexpr int kChunkBits = 12;           // larger states: outcomes per workgroup
constexpr int kMaxN = 17;
constexpr int kPartials = 512 * 2 * 64;  // doubles of scratch (reduce_partials)

struct Readout {
  double p01[kMaxN], p10[kMaxN];  // P(0|1), P(1|0)
  int32_t n;                      // 0: none
};

template <typename T>
struct Complex;
template <>
struct Complex<double> { using t = f64x2; };
template <>
struct Complex<float> { using t = f32x2; };

// the sum over the workgroup, in every thread; sh: one double per wave
__device__ inline double all_sum(double v, double* sh) {
  for (int o = 32; o > 0; o >>= 1) v += __shfl_down(v, o, 64);
  const int w = threadIdx.x >> 6, nw = blockDim.x >> 6;
  __syncthreads();
  if ((threadIdx.x & 63) == 0) sh[w] = v;
  __syncthreads();
  double t = 0.0;
  for (int i = 0; i < nw; ++i) t += sh[i];
  return t;
}

// Qubit t is read as 1 when it is 0 with probability p10 and as 0 when it is 1 with p01:
// q[x with bit t = 0] = (1 - p10) p[.0.] + p01 p[.1.],  q[.1.] = p10 p[.0.] + (1 - p01) p[.1.]
__device__ inline void readout_pair(double& a, double& b, double p01, double p10) {
  const double x = (1.0 - p10) * a + p01 * b, y = p10 * a + (1.0 - p01) * b;
  a = x;
  b = y;
}

// readout error of the qubits [0, nq) on 2^bits probabilities in LDS
__device__ inline void readout_lds(double* p, uint32_t dim, int nq, const Readout& r) {
  for (int t = 0; t < nq; ++t) {
    for (uint32_t i = threadIdx.x; i < dim / 2; i += blockDim.x) {
      const uint32_t x0 = ((i >> t) << (t + 1)) | (i & ((1u << t) - 1u));
      readout_pair(p[x0], p[x0 | (1u << t)], r.p01[t], r.p10[t]);
    }
    __syncthreads();
  }
}

// inclusive prefix sums of p[0, dim) in LDS, in place; sh: 2 * 17 doubles
__device__ inline void scan_lds(double* p, uint32_t dim, double* sh) {
  const uint32_t per = (dim + blockDim.x - 1) / blockDim.x;
  const uint32_t b = threadIdx.x * per, e = b + per < dim ? b + per : dim;
  double s = 0.0;
  for (uint32_t x = b; x < e; ++x) s += p[x];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  double v = s;
  for (int o = 1; o < 64; o <<= 1) {
    const double u = __shfl_up(v, o, 64);
    if (lane >= o) v += u;
  }
  if (lane == 63) sh[w] = v;
  __syncthreads();
  double run = __shfl_up(v, 1, 64);  // of this wave's threads before this one
  if (lane == 0) run = 0.0;
  for (int i = 0; i < w; ++i) run += sh[i];
  for (uint32_t x = b; x < e; ++x) {
    run += p[x];
    p[x] = run;
  }
  __syncthreads();
}

__device__ inline uint64_t splitmix64(uint64_t c) {
  uint64_t z = c + 0x9E3779B97F4A7C15ull;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// smallest x in [0, dim) with cdf[x] > u (dim - 1 if none)
__device__ inline uint32_t first_above(const double* cdf, uint32_t dim, double u) {
  uint32_t lo = 0, hi = dim - 1;
  while (lo < hi) {
    const uint32_t mid = (lo + hi) >> 1;
    if (cdf[mid] > u)
      hi = mid;
    else
      lo = mid + 1;
  }
  return lo;
}

}  // namespace

int reduce_partials() { return kPartials; }

// ------------------------------------------------------------------------------------
// up to 13 qubits: one workgroup
// ------------------------------------------------------------------------------------

// p[x] = Re rho[x][x], divided by the trace if renormalize, through the readout error; probs and trace (each
// may be NULL), and shots outcomes: shot i draws u = top 53 bits of SplitMix64((seed << 40) + i) in
// [0, 1) and is the smallest x with cdf[x] > u cdf[dim - 1].
template <typename T>
__global__ __launch_bounds__(1024) void small_stats_kernel(const T* __restrict__ rho, int n, int renormalize,
                                                           const Readout r, double* __restrict__ probs,
                                                           double* __restrict__ trace, uint64_t shots, uint64_t seed,
                                                           uint64_t* __restrict__ samples) {
  __shared__ double p[1 << kSmallN];
  __shared__ double sh[17];
  const uint32_t dim = 1u << n;
  double acc = 0.0;
  for (uint32_t x = threadIdx.x; x < dim; x += 1024) {
    const double v = (double)rho[2 * ((uint64_t)x * (dim + 1))];
    p[x] = v;
    acc += v;
  }
  const double tr = all_sum(acc, sh);
  if (trace && threadIdx.x == 0) *trace = tr;
  if (renormalize) {
    const double inv = 1.0 / tr;
    for (uint32_t x = threadIdx.x; x < dim; x += 1024) p[x] *= inv;
  }
  __syncthreads();
  readout_lds(p, dim, r.n, r);
  if (probs)
    for (uint32_t x = threadIdx.x; x < dim; x += 1024) probs[x] = p[x];
  if (shots) {
    scan_lds(p, dim, sh);
    const double total = p[dim - 1];
    for (uint64_t i = threadIdx.x; i < shots; i += 1024) {
      const double u = (double)(splitmix64((seed << 40) + i) >> 11) * 0x1.0p-53 * total;
      samples[i] = first_above(p, dim, u);
    }
  }
}

// ------------------------------------------------------------------------------------
// larger states
// ------------------------------------------------------------------------------------

template <typename T>
__global__ __launch_bounds__(256) void diag_kernel(const T* __restrict__ rho, int n, double* __restrict__ p,
                                                   double* __restrict__ partials) {
  __shared__ double sh[4];
  const uint64_t dim = 1ull << n;
  const uint64_t x = (uint64_t)blockIdx.x * 256 + threadIdx.x;  // dim is a multiple of 256
  const double v = (double)rho[2 * (x * (dim + 1))];
  p[x] = v;
  const double t = all_sum(v, sh);
  if (threadIdx.x == 0) partials[blockIdx.x] = t;
}

// Chunks of 4096 outcomes: divided by the trace (the sum of the diagonal's partials, formed by every workgroup),
// and the readout error of the qubits inside a chunk.
__global__ __launch_bounds__(1024) void norm_kernel(const double* __restrict__ in, const double* __restrict__ partials,
                                                    int nparts, int renormalize, const Readout r,
                                                    double* __restrict__ out, double* __restrict__ trace) {
  __shared__ double p[1 << kChunkBits];
  __shared__ double sh[16];
  double acc = 0.0;
  for (int i = threadIdx.x; i < nparts; i += 1024) acc += partials[i];
  const double tr = all_sum(acc, sh);
  if (trace && blockIdx.x == 0 && threadIdx.x == 0) *trace = tr;
  const double inv = renormalize ? 1.0 / tr : 1.0;
  const uint64_t base = (uint64_t)blockIdx.x << kChunkBits;
  for (uint32_t x = threadIdx.x; x < (1u << kChunkBits); x += 1024) p[x] = in[base + x] * inv;
  __syncthreads();
  readout_lds(p, 1u << kChunkBits, r.n < kChunkBits ? r.n : kChunkBits, r);
  for (uint32_t x = threadIdx.x; x < (1u << kChunkBits); x += 1024) out[base + x] = p[x];
}

// Readout error of the qubits 12..n-1: a thread holds the 2^(n-12) outcomes that differ in them.
__global__ __launch_bounds__(256) void readout_high_kernel(const double* __restrict__ in, int n, const Readout r,
                                                           double* __restrict__ out) {
  constexpr int H = 1 << (kMaxN - kChunkBits);
  const uint32_t x = blockIdx.x * 256 + threadIdx.x;  // below 2^12
  const int h = n - kChunkBits;
  double v[H];
#pragma unroll
  for (int i = 0; i < H; ++i) v[i] = i < (1 << h) ? in[((uint64_t)i << kChunkBits) | x] : 0.0;
#pragma unroll
  for (int t = 0; t < kMaxN - kChunkBits; ++t) {
    if (t >= h) break;
    const double p01 = r.p01[kChunkBits + t], p10 = r.p10[kChunkBits + t];
#pragma unroll
    for (int i = 0; i < H; ++i)
      if (!((i >> t) & 1)) readout_pair(v[i], v[i | (1 << t)], p01, p10);
  }
#pragma unroll
  for (int i = 0; i < H; ++i)
    if (i < (1 << h)) out[((uint64_t)i << kChunkBits) | x] = v[i];
}

// prefix sums within each chunk of len (at most 4096) outcomes, in place
__global__ __launch_bounds__(1024) void scan_kernel(double* __restrict__ p, uint32_t len) {
  __shared__ double l[1 << kChunkBits];
  __shared__ double sh[17];
  double* g = p + (uint64_t)blockIdx.x * len;
  for (uint32_t x = threadIdx.x; x < len; x += 1024) l[x] = g[x];
  __syncthreads();
  scan_lds(l, len, sh);
  for (uint32_t x = threadIdx.x; x < len; x += 1024) g[x] = l[x];
}

// cdf: prefix sums within chunks of 2^cbits outcomes; the cdf of outcome x is its chunk's start plus that
__global__ __launch_bounds__(256) void draw_kernel(const double* __restrict__ cdf, int n, int cbits, uint64_t shots,
                                                   uint64_t seed, uint64_t* __restrict__ out) {
  constexpr int CM = 1 << (kMaxN - kChunkBits);
  __shared__ double start[CM + 1];
  const int chunks = 1 << (n - cbits);
  const uint32_t clen = 1u << cbits;
  if ((int)threadIdx.x < chunks) start[threadIdx.x + 1] = cdf[((uint64_t)threadIdx.x << cbits) + clen - 1];
  __syncthreads();
  if (threadIdx.x == 0) {
    start[0] = 0.0;
    for (int c = 0; c < chunks; ++c) start[c + 1] += start[c];
  }
  __syncthreads();
  const double total = start[chunks];
  for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < shots; i += (uint64_t)gridDim.x * 256) {
    const double u = (double)(splitmix64((seed << 40) + i) >> 11) * 0x1.0p-53 * total;
    int c = 0;
    while (c < chunks - 1 && !(start[c + 1] > u)) ++c;  // the first chunk that ends above u
    const double* l = cdf + ((uint64_t)c << cbits);
    uint32_t lo = 0, hi = clen - 1;
    while (lo < hi) {
      const uint32_t mid = (lo + hi) >> 1;
      if (start[c] + l[mid] > u)
        hi = mid;
      else
        lo = mid + 1;
    }
    out[i] = ((uint64_t)c << cbits) + lo;
  }
}

// ------------------------------------------------------------------------------------
// Pauli expectations and reduced density matrices
// ------------------------------------------------------------------------------------

// Tr(P rho) = sum_s phase(s) rho[s][s ^ xmask],  phase(s) = i^{#Y} (-1)^{popcount(s & zmask)}
// masks[3 i + 0] = xmask (X or Y), masks[3 i + 1] = zmask (Z or Y), masks[3 i + 2] = #Y mod 4.
//
// An expectation that vanishes by symmetry is the rounding of its sum, so the order of the sum is part of the
// result and does not depend on how the work is split: nparts (at most 512) part sums (part b takes s = 256 b + t + 256 nparts k,
// thread by thread, then wave by wave), added one after the other.  A workgroup forms kPauliParts of them, its four
// groups of 256 threads (one group where there is one part) two each; where it forms all, it adds them and out[2 string + (re, im)] is the
// result, else out[(2 string + (re, im)) nparts + part].
constexpr int kPauliParts = 8;
constexpr int kMaxParts = 512;
template <typename T>
__global__ __launch_bounds__(1024) void pauli_kernel(const T* __restrict__ rho, int n, int nparts,
                                                     const uint64_t* __restrict__ masks, double* __restrict__ out) {
  __shared__ double sh[2][kPauliParts][4];
  const int si = blockIdx.y;
  const uint64_t xm = masks[3 * si], zm = masks[3 * si + 1];
  const int ny = (int)masks[3 * si + 2];
  const uint64_t dim = 1ull << n;
  const auto* v2 = reinterpret_cast<const typename Complex<T>::t*>(rho);
  const int t = threadIdx.x & 255;
  const int first = blockIdx.x * kPauliParts, count = nparts - first < kPauliParts ? nparts - first : kPauliParts;
  double ar[2] = {0.0, 0.0}, ai[2] = {0.0, 0.0};
  int p[2];  // this thread's parts
#pragma unroll
  for (int r = 0; r < 2; ++r) p[r] = (threadIdx.x >> 8) + r * (kPauliParts / 2);
  for (uint64_t k = 0; k < dim; k += (uint64_t)nparts * 256) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      const uint64_t s = k + (uint64_t)(first + p[r]) * 256 + t;
      if (p[r] < count && s < dim) {
        const auto v = v2[s + ((s ^ xm) << n)];
        const double sg = (__popcll(s & zm) & 1) ? -1.0 : 1.0;
        ar[r] += sg * (double)v[0];
        ai[r] += sg * (double)v[1];
      }
    }
  }
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    // multiply by i^{#Y}
    double pr = ar[r], pi = ai[r];
    if (ny == 1) { pr = -ai[r]; pi = ar[r]; }
    else if (ny == 2) { pr = -ar[r]; pi = -ai[r]; }
    else if (ny == 3) { pr = ai[r]; pi = -ar[r]; }
    for (int o = 32; o > 0; o >>= 1) {
      pr += __shfl_down(pr, o, 64);
      pi += __shfl_down(pi, o, 64);
    }
    if (p[r] < count && (t & 63) == 0) {
      sh[0][p[r]][t >> 6] = pr;
      sh[1][p[r]][t >> 6] = pi;
    }
  }
  __syncthreads();
  auto part = [&](int c, int p) {
    double x = 0.0;
    for (int w = 0; w < 4; ++w) x += sh[c][p][w];
    return x;
  };
  if (gridDim.x == 1) {
    if (threadIdx.x < 2) {
      double x = 0.0;
      for (int p = 0; p < count; ++p) x += part(threadIdx.x, p);
      out[2 * (size_t)si + threadIdx.x] = x;
    }
  } else if ((int)threadIdx.x < 2 * count) {
    const int c = threadIdx.x & 1, p = threadIdx.x >> 1;
    out[((size_t)si * 2 + c) * nparts + first + p] = part(c, p);
  }
}

// out[i] = the sum of partials[i * count ..] one after the other, one wave each
__global__ __launch_bounds__(64) void sum_in_order_kernel(const double* __restrict__ partials, int count,
                                                          double* __restrict__ out) {
  const double* p = partials + (size_t)blockIdx.x * count;
  double v[kMaxParts / 64], t = 0.0;
#pragma unroll
  for (int u = 0; u < kMaxParts / 64; ++u) v[u] = u * 64 + (int)threadIdx.x < count ? p[u * 64 + threadIdx.x] : 0.0;
#pragma unroll
  for (int u = 0; u < kMaxParts / 64; ++u) {
    if (u * 64 >= count) break;
    const int m = count - u * 64 < 64 ? count - u * 64 : 64;
    for (int i = 0; i < m; ++i) t += lane_value(v[u], i);
  }
  if (threadIdx.x == 0) out[blockIdx.x] = t;
}

struct Kept {
  int32_t q[4];       // kept qubits, the first the lowest index bit of the result
  int32_t sorted[4];  // ascending
};

// out[a][b] = sum over the other qubits' values f of rho[dep(a) | f][dep(b) | f]: element (a, b) by
// gridDim.y workgroups, out[(element * 2 + part) * gridDim.y + workgroup]
template <typename T>
__global__ __launch_bounds__(256) void reduced_kernel(const T* __restrict__ rho, int n, int k, const Kept kept,
                                                      double* __restrict__ out) {
  __shared__ double sh[4];
  const int D = 1 << k, a = blockIdx.x % D, b = blockIdx.x / D;
  uint64_t ra = 0, rb = 0;
#pragma unroll
  for (int t = 0; t < 4; ++t)
    if (t < k) {
      if ((a >> t) & 1) ra |= 1ull << kept.q[t];
      if ((b >> t) & 1) rb |= 1ull << kept.q[t];
    }
  const uint64_t nf = 1ull << (n - k);
  const auto* v2 = reinterpret_cast<const typename Complex<T>::t*>(rho);
  double sr = 0.0, si = 0.0;
  for (uint64_t f = (uint64_t)blockIdx.y * 256 + threadIdx.x; f < nf; f += (uint64_t)gridDim.y * 256) {
    uint64_t x = f;  // a zero inserted at every kept qubit
#pragma unroll
    for (int t = 0; t < 4; ++t)
      if (t < k) x = ((x >> kept.sorted[t]) << (kept.sorted[t] + 1)) | (x & ((1ull << kept.sorted[t]) - 1ull));
    const auto v = v2[(ra | x) + ((rb | x) << n)];
    sr += (double)v[0];
    si += (double)v[1];
  }
  const double tr = all_sum(sr, sh);
  const double ti = all_sum(si, sh);
  if (threadIdx.x == 0) {
    out[((size_t)(a * D + b) * 2 + 0) * gridDim.y + blockIdx.y] = tr;
    out[((size_t)(a * D + b) * 2 + 1) * gridDim.y + blockIdx.y] = ti;
  }
}

// out[i] = the sum of partials[i * count ..], one wave each
__global__ __launch_bounds__(64) void sum_partials_kernel(const double* __restrict__ partials, int count,
                                                          double* __restrict__ out) {
  double t = 0.0;
  for (int b = threadIdx.x; b < count; b += 64) t += partials[(size_t)blockIdx.x * count + b];
  for (int o = 32; o > 0; o >>= 1) t += __shfl_down(t, o, 64);
  if (threadIdx.x == 0) out[blockIdx.x] = t;
}

// ------------------------------------------------------------------------------------
// host side
// ------------------------------------------------------------------------------------

static Readout make_readout(int n, const double* p01, const double* p10) {
  Readout r{};
  if (p01) {
    r.n = n;
    for (int t = 0; t < n; ++t) {
      r.p01[t] = p01[t];
      r.p10[t] = p10[t];
    }
  }
  return r;
}

template <typename T>
static void small_stats(const void* rho, int n, int renormalize, const Readout& r, double* probs, double* trace,
                        uint64_t shots, uint64_t seed, uint64_t* samples, hipStream_t s) {
  hipLaunchKernelGGL(small_stats_kernel<T>, dim3(1), dim3(1024), 0, s, (const T*)rho, n, renormalize, r, probs, trace,
                     shots, seed, samples);
  TANQ_HIP(hipGetLastError());
}

static void small_stats_any(const void* rho, int n, tanq_prec p, int renormalize, const Readout& r, double* probs,
                            double* trace, uint64_t shots, uint64_t seed, uint64_t* samples, hipStream_t s) {
  if (p == TANQ_F64)
    small_stats<double>(rho, n, renormalize, r, probs, trace, shots, seed, samples, s);
  else
    small_stats<float>(rho, n, renormalize, r, probs, trace, shots, seed, samples, s);
}

void launch_probs(const void* rho, int n, tanq_prec p, int renormalize, const double* p01, const double* p10,
                  double* probs_dev, double* partials, double* out, double* trace, hipStream_t s) {
  if (n > kMaxN) fail(TANQ_E_ARG, "too many qubits");
  const Readout r = make_readout(n, p01, p10);
  if (n <= kSmallN) {
    small_stats_any(rho, n, p, renormalize, r, out, trace, 0, 0, nullptr, s);
    return;
  }
  if (!out) out = probs_dev;  // only the trace is wanted
  const unsigned nb = 1u << (n - 8), chunks = 1u << (n - kChunkBits);
  if (p == TANQ_F64)
    hipLaunchKernelGGL(diag_kernel<double>, dim3(nb), dim3(256), 0, s, (const double*)rho, n, probs_dev, partials);
  else
    hipLaunchKernelGGL(diag_kernel<float>, dim3(nb), dim3(256), 0, s, (const float*)rho, n, probs_dev, partials);
  TANQ_HIP(hipGetLastError());
  hipLaunchKernelGGL(norm_kernel, dim3(chunks), dim3(1024), 0, s, probs_dev, partials, (int)nb, renormalize, r,
                     p01 ? probs_dev : out, trace);
  TANQ_HIP(hipGetLastError());
  if (p01) {
    hipLaunchKernelGGL(readout_high_kernel, dim3((1u << kChunkBits) / 256), dim3(256), 0, s, probs_dev, n, r, out);
    TANQ_HIP(hipGetLastError());
  }
}

void launch_sample(const void* rho, int n, tanq_prec p, const double* p01, const double* p10, double* probs_dev,
                   double* partials, uint64_t shots, uint64_t seed, uint64_t* out, hipStream_t s) {
  if (n <= kSmallN && shots <= kSmallShots) {
    small_stats_any(rho, n, p, 1, make_readout(n, p01, p10), nullptr, nullptr, shots, seed, out, s);
    return;
  }
  launch_probs(rho, n, p, 1, p01, p10, probs_dev, partials, probs_dev, nullptr, s);
  const int cbits = n < kChunkBits ? n : kChunkBits;
  hipLaunchKernelGGL(scan_kernel, dim3(1u << (n - cbits)), dim3(1024), 0, s, probs_dev, 1u << cbits);
  TANQ_HIP(hipGetLastError());
  uint64_t blocks = (shots + 255) / 256;
  if (blocks > 1024) blocks = 1024;
  hipLaunchKernelGGL(draw_kernel, dim3((unsigned)blocks), dim3(256), 0, s, probs_dev, n, cbits, shots, seed, out);
  TANQ_HIP(hipGetLastError());
}

void launch_pauli(const void* rho, int n, tanq_prec p, int count, const uint64_t* masks, double* partials, double* out,
                  hipStream_t s) {
  // 256 elements a part, at most 512 parts, all within the scratch
  const uint64_t dim = 1ull << n;
  int nparts = dim < 256 * kMaxParts ? (int)((dim + 255) / 256) : kMaxParts;
  const int most = kPartials / (2 * count);
  if (nparts > most) nparts = most < 1 ? 1 : most;
  const int groups = (nparts + kPauliParts - 1) / kPauliParts;
  const unsigned nt = nparts == 1 ? 256 : 1024;
  double* to = groups == 1 ? out : partials;
  if (p == TANQ_F64)
    hipLaunchKernelGGL(pauli_kernel<double>, dim3(groups, count), dim3(nt), 0, s, (const double*)rho, n, nparts, masks, to);
  else
    hipLaunchKernelGGL(pauli_kernel<float>, dim3(groups, count), dim3(nt), 0, s, (const float*)rho, n, nparts, masks, to);
  TANQ_HIP(hipGetLastError());
  if (groups > 1) {
    hipLaunchKernelGGL(sum_in_order_kernel, dim3(2 * count), dim3(64), 0, s, partials, nparts, out);
    TANQ_HIP(hipGetLastError());
  }
}

void launch_reduced(const void* rho, int n, tanq_prec p, int k, const int* keep, double* partials, double* out,
                    hipStream_t s) {
  if (k < 1 || k > 4) fail(TANQ_E_ARG, "at most four kept qubits");
  Kept kept{};
  for (int t = 0; t < k; ++t) kept.q[t] = kept.sorted[t] = keep[t];
  for (int i = 1; i < k; ++i)
    for (int j = i; j > 0 && kept.sorted[j] < kept.sorted[j - 1]; --j) {
      const int x = kept.sorted[j];
      kept.sorted[j] = kept.sorted[j - 1];
      kept.sorted[j - 1] = x;
    }
  const uint64_t nf = 1ull << (n - k);
  const unsigned nel = 1u << (2 * k);
  int nb = (int)(nf / 1024 < 1 ? 1 : nf / 1024);
  if (nb > 32) nb = 32;  // 256 elements x 2 parts x 32: within the scratch
  double* to = nb == 1 ? out : partials;
  if (p == TANQ_F64)
    hipLaunchKernelGGL(reduced_kernel<double>, dim3(nel, nb), dim3(256), 0, s, (const double*)rho, n, k, kept, to);
  else
    hipLaunchKernelGGL(reduced_kernel<float>, dim3(nel, nb), dim3(256), 0, s, (const float*)rho, n, k, kept, to);
  TANQ_HIP(hipGetLastError());
  if (nb > 1) {
    hipLaunchKernelGGL(sum_partials_kernel, dim3(2 * nel), dim3(64), 0, s, partials, nb, out);
    TANQ_HIP(hipGetLastError());
  }
}

}  // namespace tanq

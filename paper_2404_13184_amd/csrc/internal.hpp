// Internal declarations shared by the host sources and the HIP kernels of libtanq.
#pragma once

#include <hip/hip_runtime.h>

#include <cstdint>
#include <stdexcept>
#include <string>
#include <vector>

#include "../../include/tanq.h"

namespace tanq {

// ------------------------------------------------------------------------------------
// errors
// ------------------------------------------------------------------------------------

struct Error : std::runtime_error {
  tanq_status code;
  Error(tanq_status c, const std::string& m) : std::runtime_error(m), code(c) {}
};

[[noreturn]] inline void fail(tanq_status c, const std::string& m) { throw Error(c, m); }

#define TANQ_HIP(expr)                                                                      \
  do {                                                                                      \
    hipError_t e_ = (expr);                                                                 \
    if (e_ != hipSuccess)                                                                   \
      ::tanq::fail(TANQ_E_HIP, std::string(#expr) + ": " + hipGetErrorString(e_));          \
  } while (0)

// ------------------------------------------------------------------------------------
// geometry of one superoperator apply (computed on the host, passed by value)
// ------------------------------------------------------------------------------------

// Tiles: a workgroup owns the 2^V elements of vec(rho) whose "varying" bits take every
// value (the 2k target bits plus the lowest free bits), with the remaining ("fixed") bits
// given by the tile id.  Groups of the superoperator lie wholly inside a tile.
struct ApplyGeom {
  uint64_t ntiles;        // number of tiles = 2^(2n - V)
  uint32_t tj[64];        // tile-local index of each superoperator local index l < 4^k
  uint32_t free_mask;     // tile-local bits that index groups inside the tile
  uint32_t xsrc;          // LDS swizzle: group bits above the bank window ...
  uint32_t xdst;          // ... copied (XOR) into these target-bit positions inside it
  int32_t V;              // tile bits
  int32_t G;              // groups per tile = 2^(V - 2k)
  int32_t nruns;          // runs of fixed bits
  uint8_t vpos[16];       // tile-local bit b -> global bit vpos[b] (ascending)
  uint8_t run_src[8];     // first tile-id bit of run r
  uint8_t run_len[8];     // length of run r
  uint8_t run_dst[8];     // first global bit of run r
};

// One-qubit apply (the paper's C1): groups of 4 at s_i + {0, 2^q, 2^(q+n), 2^q + 2^(q+n)}.
struct C1Geom {
  uint64_t ngroups;  // 4^(n-1)
  int32_t q;
  int32_t n;
};

// A pass: up to kPassMax consecutive 2-qubit superoperators applied to each tile while it is in
// LDS.  The tile holds every target bit of the pass (plus the lowest other bits up to V); the
// LDS swizzle is the linear map S(e) = e ^ (XOR of xcol[b] over the set bits b of e above the
// 256-byte bank window).
constexpr int kPassMax = 8;
// Pass tiles: 2^12 FP64 or 2^13 FP32 elements (64 KiB); superoperators one pass holds (their
// 3M operands must fit in LDS beside two tile buffers).
constexpr int kPassTileBitsF64 = 12, kPassTileBitsF32 = 13;
constexpr int kPassMaxF64 = 4, kPassMaxF32 = 6;
struct PassGeom {
  uint64_t ntiles;               // 2^(2n - V)
  int32_t V;                     // tile bits
  int32_t nruns;                 // runs of fixed bits
  int32_t m;                     // superoperators in the pass
  int32_t pad;
  uint32_t op_off[kPassMax];     // element offset of superoperator j's packed operand
  uint32_t stj[kPassMax][16];    // S(tile-local index of local index l) of superoperator j
  uint64_t goff[13];             // global offset of tile element S(2^b)
  uint16_t fb[kPassMax][10];     // S(tile bit) of superoperator j's group index bits
  uint8_t run_src[16];           // runs of fixed bits (up to 13 around 12 target bits)
  uint8_t run_len[16];
  uint8_t run_dst[16];
};

// Real-form passes over one FP64 state (herm.hip).  Address bit A(b) of a state element: index bit
// 2n - 1 (the top column bit) is address bit 0, index bit b is address bit b + 1, so the 4^n reals
// fill the lower half of vec(rho)'s memory and the pair that differs in the top column bit shares
// the 16 bytes of the lower element of the pair.
constexpr int kHermMinN = 11, kHermMaxN = 16;
inline int herm_min_launches(int n) { return n < 13 ? 12 : 8; }
constexpr int kRealPassBits = 13;  // 2^13 reals = 64 KiB
constexpr int kRealPassMax = 8;    // superoperators whose operands fit in registers
constexpr int kRealPassThreads = 512;
struct RealPassGeom {
  uint64_t ntiles;                      // 2^(2n - 13)
  uint64_t dmask;                       // address bits outside the tile
  uint64_t goff[12];                    // address offset of tile element S(2^(b + 1)): bit b of a slot index
  uint32_t op_off[kRealPassMax];        // element offset of superoperator j's operand
  uint16_t sbit[kRealPassMax][13];      // LDS byte offset of index bit b of superoperator j: b < 9 group
                                        // bits (four of the lanes, three of the waves, two of the column
                                        // blocks), then its four local index bits (ascending)
  uint8_t emb[kRealPassMax];            // 0: a 16 x 16 operand; else a one-qubit 4 x 4 operand on the local
                                        // bits emb & 3 and (emb >> 2) & 3, the identity on the others (bit 4 set)
  int32_t m;
  uint32_t sync;                        // bit j: superoperator j + 1 reads what other waves wrote
};

// Runs of superoperators of any width on small states, one launch per run (run.hip).
constexpr int kRunBitsF64 = 10, kRunBitsF32 = 11;
// blocks of a run; two-qubit blocks among them (operands in LDS), three-qubit ones
constexpr int kRunMax = 32, kRunMax2 = 8, kRunMax3 = 8;
inline int run_tile_bits(tanq_prec p) { return p == TANQ_F64 ? kRunBitsF64 : kRunBitsF32; }
// states smaller than those that use passes
inline int run_max_n(tanq_prec p) { return p == TANQ_F64 ? 9 : 10; }
struct RunOp {
  uint32_t off;     // packed operand, in 256 bytes
  uint16_t k;
  uint16_t aux;     // k = 1: blocks after this one on the same qubit (one after the other); k = 2: place of
                    // its operand in LDS
  uint16_t tb[6];   // LDS place (element) of each local index bit
  uint16_t fb[10];  // and of each group index bit
};
struct RunGeom {
  uint32_t dmask;                // index bits outside the tile
  int32_t V, m, m2, m3;          // blocks; two-qubit and three-qubit ones among them
  uint32_t goff[kRunBitsF32];    // index of each tile bit
  uint32_t off2[kRunMax2];       // operands of the two- and three-qubit blocks, as RunOp::off
  uint32_t off3[kRunMax3];
  RunOp op[kRunMax];
};
struct RunBlock {
  int k;
  int qubits[3];
  size_t pack_off;  // bytes
};

// Fusion: a block of consecutive operations on at most k qubits.
struct FuseOpDev {
  int32_t j;          // qubits of the operation
  int32_t m;          // Kraus matrices
  int64_t kraus_off;  // offset (complex elements) of K_0 in the Kraus pool
  int64_t sop_off;    // offset (complex elements) of its superoperator in the pool
  int32_t pos[3];     // block-local position of each of its qubits
  int32_t pad;
};

struct FuseBlockDev {
  int32_t k;          // qubits of the block
  int32_t op_begin;   // first operation (index into the op table)
  int32_t op_count;
  int32_t pad;
  int64_t out_off;    // offset (complex elements) of the 4^k x 4^k FP64 result
  int64_t pack_off;   // offset (elements of the packed precision) of the packed operand
};

// One superoperator apply on a state in real form (real.hpp): tiles as in ApplyGeom, with real
// elements.  Local index bits are the target bits in ascending tile position.
constexpr int kRealSwzPairs = 6;
struct RealGeom {
  uint32_t ntiles;                // 2^(2n - V)
  uint32_t free_mask;             // tile bits that index groups inside the tile
  int32_t V;                      // tile bits
  int32_t G;                      // groups per tile = 2^(V - 2k)
  int32_t nruns;                  // runs of fixed bits
  uint8_t vpos[16];               // tile bit -> global bit (ascending)
  uint8_t tpos[8];                // local index bit -> tile bit (ascending)
  uint8_t xsrc[8];                // LDS swizzle: tile bit xsrc[p] is XORed into bit xdst[p],
  uint8_t xdst[8];                // p < kRealSwzPairs (unused pairs: source bit 31)
  uint8_t run_src[8];             // first tile-id bit of run r
  uint8_t run_len[8];             // length of run r
  uint8_t run_dst[8];             // first global bit of run r
};

// Serving: one batched launch applies one superoperator to each of many states.  Items and
// chunks live in device memory; a chunk is a range of tiles of one item.
union BatchGeom {
  ApplyGeom g;   // FP32: vec(rho)
  RealGeom rg;   // FP64: real form
};
struct BatchItem {
  uint64_t rho;   // device address of the state
  uint64_t frag;  // device address of the packed operand
  BatchGeom geom;
};

struct BatchChunk {
  uint32_t item;
  uint32_t tile_begin;
  uint32_t tile_end;
  uint32_t pad;
};

// Packed operand sizes (elements of T) per superoperator width.
//   k = 1: 4x4 complex FP64 (32 doubles); k = 2: real-block 32 x 32; k = 3: 3M planar
//   (Sr, Si, Sr + Si) as 4 m-tiles x 16 k-steps x 3 x 64 lanes.
constexpr int packed_elems(int k) { return k == 1 ? 32 : (k == 2 ? 32 * 32 : 4 * 16 * 3 * 64); }

// ------------------------------------------------------------------------------------
// launchers (kernels.hip)
// ------------------------------------------------------------------------------------

ApplyGeom make_apply_geom(int n, int k, const int* qubits, int vbits, tanq_prec p);
// Geometry of one k-qubit superoperator on a state in real form: tbits = its 2k target bits in the
// state's element address (any order), nb = 2n.
RealGeom make_real_geom(int nb, int k, const int* tbits, int vbits);

// Apply-kernel variants per (k, precision), k in {2, 3}: count, shape, process-wide choice.
int variant_count(int k, tanq_prec p);
bool variant_describe(int k, tanq_prec p, int index, int* tile_bits, int* threads, int* staging);
bool variant_select(int k, tanq_prec p, int index);
int variant_selected(int k, tanq_prec p);
// autotuned variant per (n, k, precision); -1 = none (the process-wide choice applies)
constexpr int kTunedMaxN = 17;
bool variant_tune(int n, int k, tanq_prec p, int index);
int variant_tuned(int n, int k, tanq_prec p);
int variant_for(int n, int k, tanq_prec p);
int variant_find(int k, tanq_prec p, int tile_bits, int threads, int staging);
// skip (may be NULL): device flag; the launch does nothing where it is set.
void launch_apply_variant(void* rho, int n, tanq_prec p, int k, int index, const int* qubits, const void* packed,
                          hipStream_t s, const uint32_t* skip = nullptr);

// Passes (pass.hip): tile bits per precision; geometry of m superoperators (qubits: m pairs,
// op_off: element offsets of their packed operands); launch on one state.
int pass_tile_bits(tanq_prec p);
// Most superoperators one pass of precision p holds (at most kPassMax).
int pass_max(tanq_prec p);
// conflict_free (optional): access patterns (two per superoperator) whose LDS reads and writes
// are free of bank conflicts under the chosen swizzle; achievable (optional): an upper bound of
// that count over all swizzles of this form.
PassGeom make_pass_geom(int n, int m, const int* qubits, const uint32_t* op_off, tanq_prec p,
                        int* conflict_free = nullptr, int* achievable = nullptr);
void launch_pass(void* rho, tanq_prec p, const PassGeom& g, const void* frags, hipStream_t s);
// One launch for a pass of either form of an FP64 state: where *flag is set the real-form one (rg, rpacked;
// NULL: nothing), else the complex one (g, frags; NULL: nothing).
void launch_pass_either(void* rho, const PassGeom* g, const void* frags, const RealPassGeom* rg, const double* rpacked,
                        const uint32_t* flag, hipStream_t s);
// blocks: m consecutive blocks whose qubits fit one tile (run_tile_bits)
void launch_run(void* rho, int n, tanq_prec p, int m, const RunBlock* blocks, const void* packed, hipStream_t s);
// Process-wide limit on superoperators per pass (1 = no passes).
int pass_limit();
void set_pass_limit(int m);

// Real-form passes over one FP64 state (herm.hip).  qubits: k[j] per superoperator, three apart.
bool real_pass_fits(uint64_t qmask, int n);
RealPassGeom make_real_pass_geom(int n, int m, const int* k, const int* qubits, const uint32_t* op_off);
// Real operands of every block (k = 1: 4 x 4; k = 2, 3: fragments), local index bits in ascending
// address order; elements per block real_pack_elems(k), offset of block b at off[b] (device table).
constexpr int real_pack_elems(int k) { return k == 1 ? 16 : (k == 2 ? 256 : 4096); }
struct RealPackDev {
  int64_t raw_off;   // complex elements
  int64_t pack_off;  // doubles
  int32_t k;
  uint8_t perm[8];   // local bit of the real operand -> local bit of the superoperator
};
void launch_pack_herm(const RealPackDev* blocks, int nblocks, const double* raw, double* packed, hipStream_t s);
// *flag = 1 if vec(rho) is exactly Hermitian and within range, else 0
void launch_herm_check(const void* rho, int n, uint32_t* flag, hipStream_t s);
// vec(rho) -> real form and back in place; nothing where *flag is 0
void launch_herm_in(void* rho, int n, const uint32_t* flag, hipStream_t s);
void launch_herm_out(void* rho, int n, const uint32_t* flag, hipStream_t s);
void launch_real_apply3(void* rho, int n, const int* qubits, const double* packed, const uint32_t* flag, hipStream_t s);

void launch_init_zero(void* rho, int n, tanq_prec p, hipStream_t s);
void launch_gather(const void* rho, tanq_prec p, const uint64_t* idx_dev, size_t count, void* out_dev,
                   hipStream_t s);
void launch_fill_random(void* rho, int n, tanq_prec p, uint64_t seed, hipStream_t s);
void launch_scale(void* rho, int n, tanq_prec p, double f, hipStream_t s);
// Sustained matrix-unit rate (TFLOP/s) of the pass kernels' multiplication loop shape on the
// current device; synchronous.
double mfma_rate_tflops(tanq_prec p);

// All-qubit sampling (tanq_sample and its variant without allocations): argument checks (also returning the
// handle's device and whether its own result buffer holds the outcomes), and the work itself; out_dev:
// device buffer for the outcomes, unused if the handle's holds them.  Synchronises.
void sample_check(tanq_dm d, uint64_t shots, uint64_t seed, const double* p01, const double* p10, uint64_t* host_out,
                  int* n, int* device, bool* own);
void sample_run(tanq_dm d, uint64_t shots, uint64_t seed, const double* p01, const double* p10, uint64_t* out_dev,
                uint64_t* host_out);

// Apply one superoperator whose packed operand is at `packed` (device).
//   k == 1: packed = 4x4 complex FP64 (32 doubles), used for both precisions.
//   k == 2, 3: packed = real-block fragments in precision p.
void launch_apply(void* rho, int n, tanq_prec p, int k, const int* qubits, const void* packed,
                  hipStream_t s, const uint32_t* skip = nullptr);

// Superoperators of every operation (sum_i conj(K_i) (x) K_i), FP64.
void launch_build_superops(const FuseOpDev* ops, int nops, const double* kraus, double* sops,
                           hipStream_t s);
// Compose each block's superoperators in circuit order (FP64) into `out`, and pack them into the apply
// kernels' operand layout of precision p.
void launch_compose(const FuseBlockDev* blocks, int nblocks, int max_k, const FuseOpDev* ops, const double* sops,
                    double* out, void* packed, tanq_prec p, hipStream_t s);
// Pack a single FP64 superoperator of width k (device or pinned host memory).
void launch_pack_one(int k, const double* raw, void* packed, tanq_prec p, hipStream_t s);
// A one-qubit superoperator (host, 4 x 4 complex) that travels with the launch.
void launch_apply_one_qubit(void* rho, int n, tanq_prec p, int qubit, const double* S, hipStream_t s);

// Real form (real.hip).  Superoperators of every operation as real 4^j x 4^j matrices (offset sop_off, in
// doubles), their composition per block in circuit order, packed as the real apply kernels'
// operands; FP64, rounded once.  Every block has k qubits (2 or 3).
void launch_build_real(const FuseOpDev* ops, int nops, const double* kraus, double* sops, hipStream_t s);
void launch_compose_real(const FuseBlockDev* blocks, int nblocks, int k, const FuseOpDev* ops, const double* sops,
                         void* packed, hipStream_t s);
// w = the real form of |0..0><0..0|
void launch_real_init(void* w, int n, hipStream_t s);
// Outputs of a state in real form, n <= kRealOutMaxN: out[0] = the trace, then the 2^n probabilities
// divided by it if want_probs, then (Re, Im) of count Pauli expectations (masks: x, z, #Y mod 4 per
// string, as launch_pauli).  masks and out are device-accessible (pinned host memory).
constexpr int kRealOutMaxN = 14;
void launch_real_outputs(const void* w, int n, int want_probs, int count, const uint64_t* masks, double* out, hipStream_t s);

// Measurement statistics (measure.hip; FP64).  partials: device scratch of at least reduce_partials() doubles;
// probs_dev: of 2^n doubles.  Outputs (out, trace, masks) are device-accessible: device memory or
// pinned host memory.
int reduce_partials();
// out[x] = Re rho[x][x], divided by the trace if renormalize, through the readout error if p01 (host arrays of
// n values); out and trace may be NULL
void launch_probs(const void* rho, int n, tanq_prec p, int renormalize, const double* p01, const double* p10,
                  double* probs_dev, double* partials, double* out, double* trace, hipStream_t s);
// shots outcomes of the renormalised probabilities, through the readout error if p01
void launch_sample(const void* rho, int n, tanq_prec p, const double* p01, const double* p10, double* probs_dev,
                   double* partials, uint64_t shots, uint64_t seed, uint64_t* out, hipStream_t s);
// out: (Re, Im) of count strings (at most 1024); masks: x, z, number of Y mod 4 per string
void launch_pauli(const void* rho, int n, tanq_prec p, int count, const uint64_t* masks, double* partials, double* out,
                  hipStream_t s);
// reduced density matrix on the k <= 4 qubits keep (host), 2 * 4^k doubles
void launch_reduced(const void* rho, int n, tanq_prec p, int k, const int* keep, double* partials, double* out,
                    hipStream_t s);

// vec(rho) = e_idx (rho = |r><c| for idx = r + c 2^n)
void launch_init_basis(void* rho, int n, tanq_prec p, uint64_t idx, hipStream_t s);
// out3 = (||a-b||_F, max|a-b|, ||a||_F); partials: reduce_partials() doubles.
void launch_compare(const void* a, tanq_prec pa, const void* b, tanq_prec pb, uint64_t nel, double* partials,
                    double* result_dev, hipStream_t s);

int device_cu_count();

// Tile bits of the batched kernel of precision p (geometry of the items must be built with this
// value).
int batch_tile_bits(tanq_prec p);
// Workgroups of the batched kernel's persistent grid on the current device.
int batch_grid(int k, tanq_prec p);
// Apply the items of `*count` chunks (count lives in device memory so the launch can be
// captured in a graph and replayed with new contents).
void launch_batch(int k, tanq_prec p, const BatchItem* items, const BatchChunk* chunks, uint32_t* count,
                  hipStream_t s);

}  // namespace tanq

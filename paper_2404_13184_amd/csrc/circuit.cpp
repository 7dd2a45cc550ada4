#include "circuit.hpp"

#include <algorithm>
#include <utility>

namespace tanq {

std::vector<PlanOp> plan_ops(const std::vector<HostOp>& ops) {
  std::vector<PlanOp> p(ops.size());
  for (size_t i = 0; i < ops.size(); ++i) {
    p[i].j = ops[i].j;
    for (int t = 0; t < 3; ++t) p[i].q[t] = ops[i].q[t];
  }
  return p;
}

void widen_plan(std::vector<PlanBlock>& plan, int n, int w) {
  for (auto& b : plan) {
    for (int q = 0; q < n && (int)b.qubits.size() < w; ++q)
      if (std::find(b.qubits.begin(), b.qubits.end(), q) == b.qubits.end()) b.qubits.push_back(q);
    std::sort(b.qubits.begin(), b.qubits.end());
  }
}

FuseLayout make_fuse_layout(const std::vector<HostOp>& ops, const std::vector<PlanBlock>& plan, tanq_prec p,
                            bool real) {
  FuseLayout L;
  // identical Kraus sets (same pool, offset and size, e.g. a noise channel repeated through a
  // circuit) are uploaded once; their superoperators are still built per operation.  Open addressing:
  // entry h holds an operation with that key (its index in L.ops is seen[h]), -1 is free.
  size_t cap = 16;
  while (cap < 2 * ops.size()) cap *= 2;
  std::vector<int> seen(cap, -1), source(ops.size());  // source: operation of each entry of L.ops
  L.ops.reserve(ops.size());
  L.blocks.reserve(plan.size());
  L.host.reserve(plan.size());
  for (const auto& pb : plan) {
    const int k = (int)pb.qubits.size();
    if (k > 3) fail(TANQ_E_UNSUPPORTED, "a block wider than 3 qubits");
    L.max_k = std::max(L.max_k, k);
    FuseBlockDev bd{};
    bd.k = k;
    bd.op_begin = (int)L.ops.size();
    bd.op_count = (int)pb.ops.size();
    bd.out_off = (int64_t)L.raw_elems;
    bd.pack_off = (int64_t)L.pack_bytes;
    FusedBlockHost bh;
    bh.k = k;
    for (int t = 0; t < k; ++t) bh.qubits[t] = pb.qubits[t];
    bh.raw_off = L.raw_elems;
    bh.pack_off = L.pack_bytes;
    L.raw_elems += (size_t)1 << (4 * k);
    L.pack_bytes += align256(real ? real_pack_elems(k) * sizeof(double) : packed_bytes(k, p));
    for (int oi : pb.ops) {
      const HostOp& ho = ops[oi];
      FuseOpDev od{};
      od.j = ho.j;
      od.m = ho.m;
      size_t h = ((uintptr_t)ho.pool.get() / 16 + ho.koff * 0x9E3779B97F4A7C15ull) >> 7 & (cap - 1);
      while (seen[h] >= 0) {
        const HostOp& other = ops[source[seen[h]]];
        if (other.pool == ho.pool && other.koff == ho.koff && other.kdoubles() == ho.kdoubles()) break;
        h = (h + 1) & (cap - 1);
      }
      if (seen[h] < 0) {
        seen[h] = (int)L.ops.size();
        od.kraus_off = (int64_t)(L.kraus.size() / 2);
        L.kraus.insert(L.kraus.end(), ho.K(), ho.K() + ho.kdoubles());
      } else {
        od.kraus_off = L.ops[seen[h]].kraus_off;
      }
      source[L.ops.size()] = oi;
      od.sop_off = (int64_t)L.sop_elems;
      for (int t = 0; t < ho.j; ++t) {
        int pos = -1;
        for (int u = 0; u < k; ++u)
          if (pb.qubits[u] == ho.q[t]) pos = u;
        if (pos < 0) fail(TANQ_E_STATE, "operation qubit outside its block");
        od.pos[t] = pos;
      }
      L.sop_elems += (size_t)1 << (4 * ho.j);
      L.ops.push_back(od);
    }
    L.blocks.push_back(bd);
    L.host.push_back(bh);
    L.count_k[k] += 1;
  }
  return L;
}

void run_fuse_kernels(const FuseLayout& L, const FuseOpDev* d_ops, const FuseBlockDev* d_blk, const double* d_kraus,
                      double* d_sops, double* d_raw, unsigned char* d_packed, tanq_prec p, hipStream_t s) {
  if (L.blocks.empty()) return;
  launch_build_superops(d_ops, (int)L.ops.size(), d_kraus, d_sops, s);
  launch_compose(d_blk, (int)L.blocks.size(), L.max_k, d_ops, d_sops, d_raw, d_packed, p, s);
}

}  // namespace tanq

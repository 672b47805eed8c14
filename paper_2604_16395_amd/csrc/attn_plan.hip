// Device plan kernel: computes the varlen work partition of one step from the device
// length arrays (rules in plan_rules.h, identical to the host's) and stores it at the start
// of the caller's workspace: per-request arrays and one ItemRec per work item (so that an
// attention workgroup finds all it needs in one scalar load).  The piece length comes from the
// host planner, which chose it from its copies of the lengths, and so does, for the binned item
// order, the XCD bin of each (request, kv head) group.
//
// Bound by latency: the lengths, then scans over the requests, then the records.  Every workgroup
// of the grid repeats the scans (a few hundred values, in LDS) and writes a share of the
// records, one a thread, so that no workgroup waits for another; the first one stores the
// header and the request arrays.  One workgroup for all records, re-reading the lengths and
// scanning all eight bins at once, took 4.9 us for one request of 4 items, 10.6 us for 64 binned
// items, 40 us for 64 requests of 4688 items in bins: now 3.8, 5.2 and 6.9 us.
#include <algorithm>

#include "launch.h"
#include "plan_rules.h"

namespace s2l {

namespace {

constexpr int kPlanThreads = 256;
constexpr int kPlanWaves = kPlanThreads / 64;
constexpr int kMaxPlanParts = 256;
constexpr int kLdsReqs = 1024;   // batches up to this size keep their per-request values in LDS
constexpr int kRankReqs = kPlanThreads;   // batches up to this size are laid out longest first
static_assert(kRankReqs == kBinnedMaxReqs, "the binned order needs the ranking");

// Block-wide exclusive scan of N int64 values; returns the block totals in tot[].  The first
// `waves` waves hold nonzero values.  Synchronises once, before the totals are read.
template <int N>
__device__ void block_scan(const int64_t (&v)[N], int64_t (&excl)[N], int64_t (&tot)[N],
                           int64_t (*sh)[kPlanWaves], int waves) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  int64_t x[N];
  for (int k = 0; k < N; ++k) x[k] = v[k];
  if (w < waves)
    for (int o = 1; o < 64; o <<= 1) {
      for (int k = 0; k < N; ++k) {
        const int64_t y = __shfl_up(x[k], o);
        if (lane >= o) x[k] += y;
      }
    }
  if (lane == 63)
    for (int k = 0; k < N; ++k) sh[k][w] = x[k];
  __syncthreads();
  for (int k = 0; k < N; ++k) {
    int64_t before = 0, all = 0;
    for (int i = 0; i < kPlanWaves; ++i) {
      before += i < w ? sh[k][i] : 0;
      all += sh[k][i];
    }
    excl[k] = before + x[k] - v[k];
    tot[k] = all;
  }
}

// Largest r with a[r] <= x, for a non-decreasing a[0..n] with a[0] <= x < a[n].
template <typename A>
__device__ inline int upper_index(const A& a, int n, int x) {
  int lo = 0, hi = n;
  while (hi - lo > 1) {
    int mid = (lo + hi) >> 1;
    if (a[mid] <= x) lo = mid; else hi = mid;
  }
  return lo;
}

// Sum over the block (every thread calls it).
__device__ inline int block_sum(int x) {
  __shared__ int total;
  if (threadIdx.x == 0) total = 0;
  __syncthreads();
  if (x != 0) atomicAdd(&total, x);
  __syncthreads();
  return total;
}

// Item order.  Up to kRankReqs requests are laid out longest first (by P + C, the key range
// of their longest tile; ties by index), so that when the items take several rounds of
// workgroups the longest start first and the dispatcher balances the tail; larger batches
// keep request order.  Pieces per request come from the host's piece length, and a block scan of
// items, partial floats, tiles and tokens over the slots of that order (a contiguous segment per
// thread) gives every offset and total.  kLds: up to kLdsReqs requests, any number of workgroups
// (a multiple of kNumXcds for the binned order); else one workgroup, which keeps the offsets in
// the workspace.
template <bool kLds>
__global__ __launch_bounds__(kPlanThreads) void attn_plan_kernel(PlanLaunch a, PlanPtrs pp) {
  constexpr int kSlots = kLds ? kLdsReqs : 1;
  __shared__ int64_t sh[4][kPlanWaves], sh_bin[1][kPlanWaves];
  __shared__ int32_t s_item_off[kSlots + 1], s_req[kSlots], s_ns[kSlots], s_nqt[kSlots], s_p[kSlots], s_c[kSlots],
      s_cu[kSlots];
  __shared__ int64_t s_part[kSlots];
  __shared__ int64_t s_key[kRankReqs];
  __shared__ int32_t s_rank[kRankReqs];
  __shared__ int32_t s_bin_cnt[kNumXcds], s_gpos[kBinnedMaxGroups], s_gid[kBinnedMaxGroups];
  const int R = a.num_reqs;
  const int G = a.hq / a.hkv;
  const int tq = tile_tokens(G, a.tile_cols);
  const int split_keys = a.split_keys;
  const int t = threadIdx.x;
  const bool first = blockIdx.x == 0;
  const bool ranked = R <= kRankReqs;
  const int32_t cu_end = a.cu_chunk[R];
  auto set_slot = [&](int k, int r, int P, int C, int cu) {
    s_req[k] = r;
    s_p[k] = P;
    s_c[k] = C;
    s_cu[k] = cu;
    s_ns[k] = req_splits(P, C, split_keys, a.max_splits);
    s_nqt[k] = num_qtiles(C, tq);
  };
  if constexpr (kLds) {
    if (t < kNumXcds) s_bin_cnt[t] = 0;
    if (ranked && R > 1) {
      // a request's slot is the number of those before it: longer, or as long with a lower index.
      // Both in one key, and the comparisons of a request spread over kPlanThreads / rows threads.
      int P = 0, C = 0, cu = 0;
      int64_t key = -1;   // past the requests: after all of them
      if (t < R) {
        P = a.prefix_lens[t], C = a.chunk_lens[t], cu = a.cu_chunk[t];
        key = (int64_t)(C > 0 ? P + C + 1 : 0) << 32 | (uint32_t)(kRankReqs - t);
      }
      s_key[t] = key;
      s_rank[t] = 0;
      __syncthreads();
      const int bits = 32 - __clz(R > 1 ? R - 1 : 0);   // rows = 2^bits >= R
      const int own = t & ((1 << bits) - 1), part = t >> bits, parts = kPlanThreads >> bits;
      const int64_t own_key = s_key[own];
      int rank = 0;
#pragma unroll 8
      for (int o = part; o < R; o += parts) rank += s_key[o] > own_key;
      atomicAdd(&s_rank[own], rank);
      __syncthreads();
      if (t < R) set_slot(s_rank[t], t, P, C, cu);
    } else {
      for (int k = t; k < R; k += kPlanThreads) set_slot(k, k, a.prefix_lens[k], a.chunk_lens[k], a.cu_chunk[k]);
    }
    __syncthreads();
  }
  // request of slot k: index, lengths, pieces, tiles
  struct Req {
    int r, P, C, ns, nqt, cu;
  };
  auto req_at = [&](int k) {
    Req q;
    if constexpr (kLds) {
      q = Req{s_req[k], s_p[k], s_c[k], s_ns[k], s_nqt[k], s_cu[k]};
    } else {
      q.r = k, q.P = a.prefix_lens[k], q.C = a.chunk_lens[k], q.cu = a.cu_chunk[k];
      q.ns = req_splits(q.P, q.C, split_keys, a.max_splits);
      q.nqt = num_qtiles(q.C, tq);
    }
    return q;
  };

  const int seg = (R + kPlanThreads - 1) / kPlanThreads;
  const int k0 = min(R, t * seg), k1 = min(R, k0 + seg);
  int64_t v[4] = {0, 0, 0, 0}, excl[4], tot[4];
  int splits = 0;
  for (int k = k0; k < k1; ++k) {
    const Req q = req_at(k);
    const int64_t tiles = (int64_t)a.hkv * q.nqt;
    v[0] += tiles * q.ns;
    v[1] += req_part_floats(q.ns, q.C, a.hq);
    v[2] += tiles;
    v[3] += q.C;
    splits += q.ns > 1 ? 1 : 0;
  }
  block_scan<4>(v, excl, tot, sh, seg > 1 ? kPlanWaves : (R + 63) / 64);
  const int64_t num_items = tot[0], part_floats = tot[1], num_tiles = tot[2];
  int64_t items = excl[0], part = excl[1];
  for (int k = k0; k < k1; ++k) {
    const Req q = req_at(k);
    if (first) {
      pp.item_off[q.r] = (int32_t)items;
      pp.ns[q.r] = q.ns;
      pp.c[q.r] = q.C;
      pp.cu[q.r] = q.cu;
      pp.part_off[q.r] = part;
    }
    if constexpr (kLds) {
      s_item_off[k] = (int32_t)items;
      s_part[k] = part;
    }
    items += (int64_t)a.hkv * q.nqt * q.ns;
    part += req_part_floats(q.ns, q.C, a.hq);
  }
  if constexpr (kLds)
    if (t == 0) s_item_off[R] = (int32_t)num_items;
  // Binned order (plan_rules.h): the host's bin of each (request, kv head) group, groups in
  // ranked order.  Every group's items are counted into its bin; the bins are as long as the
  // longest.  (Above cap_items nothing is counted: the counts could overflow.)
  const int ngroups = R * a.hkv;
  const bool binned = kLds && a.binned != 0 && ranked && ngroups <= kBinnedMaxGroups;
  int64_t records = num_items;
  int bin_len = 0;
  if (binned && num_items <= pp.cap_items) {
    for (int q = t; q < ngroups; q += kPlanThreads) {
      const int k = q / a.hkv;
      atomicAdd(&s_bin_cnt[a.group_bin[q] & (kNumXcds - 1)], s_nqt[k] * s_ns[k]);
    }
    __syncthreads();
    for (int x = 0; x < kNumXcds; ++x) bin_len = max(bin_len, s_bin_cnt[x]);
    records = (int64_t)kNumXcds * bin_len;
  }
  const bool fits = records <= pp.cap_items && num_tiles <= pp.cap_tiles && part_floats <= pp.cap_part_floats;
  const int num_split = first ? block_sum(splits) : 0;
  if (first && t == 0) {
    pp.item_off[R] = (int32_t)num_items;
    pp.cu[R] = cu_end;
    PlanHeader* h = pp.hdr;
    h->magic = kPlanMagic;
    h->num_reqs = R;
    h->hq = a.hq;
    h->hkv = a.hkv;
    h->g = G;
    h->tq = tq;
    h->num_items = fits ? (int32_t)records : 0;
    h->num_split_reqs = num_split;
    h->split_keys = split_keys;
    h->status = fits ? 0 : 1;
    h->tile_cols = a.tile_cols;
    h->num_tiles = (int32_t)num_tiles;
    h->part_floats = part_floats;
    h->total_tokens = tot[3];
  }
  if (!fits) return;
  __syncthreads();   // request arrays (in LDS, or this workgroup's in the workspace) complete

  // The record of item `local` of the request at slot k (request-local items: kv head g, then
  // query tile, then piece).
  auto make_rec = [&](int k, int local) {
    const Req q = req_at(k);
    const Item it = decode_local(local, q.nqt, q.ns);
    ItemRec rec;
    rec.r = q.r;
    rec.g = it.g;
    rec.i0 = it.qt * tq;
    rec.i1 = min(rec.i0 + tq, q.C);
    piece_range(q.P + rec.i1, q.ns, it.s, &rec.lo, &rec.hi);
    rec.s = it.s;
    rec.ns = q.ns;
    rec.p = q.P;
    rec.c = q.C;
    rec.row0 = q.cu;
    rec.part_off = kLds ? s_part[k] : pp.part_off[q.r];
    rec.pad0 = rec.pad1 = rec.pad2 = 0;
    return rec;
  };
  if (binned) {
    // Workgroup b takes records of bin b mod 8: the bin's groups in order (a scan of their number
    // and of their items, packed, over segments of groups) give the first position of each, and a
    // record's group is found by binary search.  Past the bin's items: padding (request -1).
    const int bin = blockIdx.x % kNumXcds;
    const int gseg = (ngroups + kPlanThreads - 1) / kPlanThreads;
    const int q0 = min(ngroups, t * gseg), q1 = min(ngroups, q0 + gseg);
    auto group_items = [&](int q) { const int k = q / a.hkv; return s_nqt[k] * s_ns[k]; };
    int64_t n[1] = {0}, at[1], all[1];
    for (int q = q0; q < q1; ++q)
      if (a.group_bin[q] == bin) n[0] += ((int64_t)group_items(q) << 16) + 1;
    block_scan<1>(n, at, all, sh_bin, kPlanWaves);
    int64_t pos = at[0];
    for (int q = q0; q < q1; ++q)
      if (a.group_bin[q] == bin) {
        s_gpos[pos & 0xffff] = (int32_t)(pos >> 16);
        s_gid[pos & 0xffff] = q;
        pos += ((int64_t)group_items(q) << 16) + 1;
      }
    __syncthreads();
    const int groups = (int)(all[0] & 0xffff), total = (int)(all[0] >> 16);
    const int parts = gridDim.x / kNumXcds;
    for (int w = (int)(blockIdx.x / kNumXcds) * kPlanThreads + t; w < bin_len; w += parts * kPlanThreads) {
      ItemRec rec = {};
      rec.r = -1;
      if (w < total) {
        const int g = upper_index(s_gpos, groups, w), q = s_gid[g], k = q / a.hkv;
        rec = make_rec(k, (q % a.hkv) * (s_nqt[k] * s_ns[k]) + w - s_gpos[g]);
      }
      pp.items[(int64_t)bin * bin_len + w] = rec;
    }
    return;
  }
  // one record per item; the request of item w is found by binary search over item offsets
  for (int w = (int)blockIdx.x * kPlanThreads + t; w < (int)num_items; w += gridDim.x * kPlanThreads) {
    const int k = kLds ? upper_index(s_item_off, R, w) : upper_index(pp.item_off, R, w);
    pp.items[w] = make_rec(k, w - (kLds ? s_item_off[k] : pp.item_off[k]));
  }
}

}  // namespace

hipError_t launch_attn_plan(const PlanLaunch& a, const PlanDims& dims, hipStream_t stream) {
  const PlanPtrs pp = plan_ptrs(a.workspace, dims);
  if (a.num_reqs > kLdsReqs) {
    attn_plan_kernel<false><<<1, kPlanThreads, 0, stream>>>(a, pp);
    return hipGetLastError();
  }
  // one record a thread: bins of equal length, or all items, in workgroups of kPlanThreads
  const int64_t len = a.binned ? dims.num_items / kNumXcds : dims.num_items;
  const int64_t parts = std::min<int64_t>(std::max<int64_t>(ceil_div64(len, kPlanThreads), 1), kMaxPlanParts);
  attn_plan_kernel<true><<<(unsigned)(parts * (a.binned ? kNumXcds : 1)), kPlanThreads, 0, stream>>>(a, pp);
  return hipGetLastError();
}

}  // namespace s2l

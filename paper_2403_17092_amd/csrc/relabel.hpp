// The relabelling state of the neighbour sampler shared with the launch that
// finishes a sampling call (the last hop's edge compaction can run inside the
// next launch of a training step, the feature gather).
#pragma once
#include <hip/hip_runtime.h>

#include <cstdint>

namespace gnn {

// Persistent header of the sampler's workspace: a magic word, the last
// finished epoch, this call's top epoch and the node count the per-node words
// were built for.
constexpr uint32_t kMagic = 0x474E4E53u;  // "GNNS"

struct Header {
  uint32_t magic;
  uint32_t done_epoch;
  uint32_t top_epoch;
  uint32_t pad;
  int64_t num_nodes;
};

// A padded slot holds the node id of a pick, -1 if unused or invalid; the
// scans add kFirstPick to the pick that is its node's first occurrence in the
// hop's src list (node ids are below 2^31 - 1, so the marked id is not -1).
constexpr uint32_t kFirstPick = 0x80000000u;
__host__ __device__ __forceinline__ int32_t pick_node(int32_t slot) {
  return slot == -1 ? -1 : (int32_t)((uint32_t)slot & ~kFirstPick);
}
__host__ __device__ __forceinline__ bool pick_first(int32_t slot) { return slot < -1; }

// Workgroup counters of the src nodes [lo, lo + kSize), in LDS.  Device
// atomics on one address run one after the other (~17 ns each on gfx950), and
// a hub of a power-law graph is picked by thousands of edges of one hop: 462K
// counts over 209K nodes take 20 us spread evenly and 137 us with 1.7% of them
// on one node; with workgroup counters the latter takes 20 us too.  Hubs are
// met early, so they are among the first new nodes of hop 1 and their ids
// among the lowest past the seeds'.
struct HubCounts {
  static constexpr int kSize = 4096;
  int32_t n[kSize];
};
// seeds whose ids the window still covers beside the first new nodes
constexpr int32_t kHubSeeds = HubCounts::kSize / 2;
// A hop's edges go through the window from this many slots, and this many per
// src node, on: the passes' barriers cost 1-4 us (63K edges over 45K nodes: 9.6
// us for the launch without the window, 13.8 with it), the contention of few
// or spread-out edges less (263K edges over 23K nodes: 52 us without, 25 with).
constexpr int64_t kHubSlots = 1 << 16;
constexpr int64_t kHubShare = 6;

// Edge compaction of one hop: padded slot (i, r), r < k_i, becomes
// indices[indptr[i] + r] = local id of its key; src_occ of that id, which the
// scans start at 1, counts every edge but a new node's first one.
struct IndexJob {
  const int32_t* nbr_pad;  // [n_dst x fanout], -1 = unused
  const int32_t* kcount;   // [n_dst]
  const int32_t* indptr;
  const int32_t* counts;   // counts[0] = n_dst
  const int32_t* nid;      // per-node local id
  int32_t* indices;
  int32_t* src_occ;
  int32_t* rank;           // null, or [cap_edges]: the edge's place among its src node's edges
  int32_t fanout;
  int32_t cap_src;
  int32_t hub_lo;          // first id of the window
  int64_t num_nodes;
};

template <bool WINDOW>
__device__ __forceinline__ void index_passes(const IndexJob& j, int32_t n_dst, int64_t block,
                                             int64_t blocks, int threads, HubCounts& hub) {
  // Four slots per pass, their independent loads (count, pick, row start)
  // issued together and then the four id lookups, so a thread waits on two
  // memory round trips per pass rather than three per slot.
  constexpr int kBatch = 4;
  // (32 bits hold every slot, at most INT32_MAX, plus a pass)
  const uint32_t slots = (uint32_t)n_dst * (uint32_t)j.fanout, f = (uint32_t)j.fanout;
  const uint32_t stride = (uint32_t)blocks * threads;
  for (uint32_t base = (uint32_t)block * threads; base < slots; base += kBatch * stride) {
    uint32_t i[kBatch];
    int32_t r[kBatch], kc[kBatch], slot[kBatch], at[kBatch], id[kBatch], place[kBatch], h[kBatch];
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      const uint32_t s = base + threadIdx.x + k * stride;
      const bool live = s < slots;
      i[k] = live ? s / f : 0;
      r[k] = live ? (int32_t)(s - i[k] * f) : 0;  // dead slots: r = kc = 0, skipped
      kc[k] = live ? j.kcount[i[k]] : 0;
      slot[k] = live ? j.nbr_pad[s] : -1;
      at[k] = live ? j.indptr[i[k]] : 0;
    }
    if (WINDOW)
      for (int x = threadIdx.x; x < HubCounts::kSize; x += threads) hub.n[x] = 0;
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      // a pick dropped as an invalid id (device error raised) points at row 0
      const bool ok = r[k] < kc[k] && slot[k] != -1;
      id[k] = ok ? j.nid[pick_node(slot[k])] : 0;
    }
    if (WINDOW) __syncthreads();
#pragma unroll
    for (int k = 0; k < kBatch; ++k) {
      place[k] = 0;
      h[k] = -1;
      if (r[k] >= kc[k]) continue;
      j.indices[at[k] + r[k]] = id[k];
      if (slot[k] == -1 || pick_first(slot[k]) || (uint32_t)id[k] >= (uint32_t)j.cap_src) continue;
      const uint32_t x = (uint32_t)(id[k] - j.hub_lo);
      if (WINDOW && x < (uint32_t)HubCounts::kSize) {
        h[k] = (int32_t)x;
        place[k] = atomicAdd(&hub.n[x], 1);
      } else if (j.rank) {
        place[k] = atomicAdd(&j.src_occ[id[k]], 1);
      } else {
        atomicAdd(&j.src_occ[id[k]], 1);
      }
    }
    if (WINDOW) {
      __syncthreads();
      for (int x = threadIdx.x; x < HubCounts::kSize; x += threads)
        if (hub.n[x]) hub.n[x] = atomicAdd(&j.src_occ[j.hub_lo + x], hub.n[x]);
      __syncthreads();
    }
    if (j.rank) {
#pragma unroll
      for (int k = 0; k < kBatch; ++k) {
        if (r[k] >= kc[k]) continue;
        if (WINDOW && h[k] >= 0) place[k] += hub.n[h[k]];
        // src_occ starts at 1: a dst node's own occurrence, or a new node's
        // first edge (place 0)
        if (id[k] < n_dst) place[k] -= 1;
        j.rank[at[k] + r[k]] = place[k];
      }
    }
    if (WINDOW) __syncthreads();
  }
}

// Block `block` of `blocks` (of `threads` threads each) of the compaction.
__device__ __forceinline__ void index_slots(const IndexJob& j, int64_t block, int64_t blocks, int threads,
                                            HubCounts& hub) {
  if (!j.nbr_pad) return;
  const int32_t n_dst = j.counts[0], n_src = j.counts[1];
  const int64_t slots = (int64_t)n_dst * j.fanout;
  if (slots >= kHubSlots && slots >= kHubShare * n_src)  // (uniform)
    index_passes<true>(j, n_dst, block, blocks, threads, hub);
  else
    index_passes<false>(j, n_dst, block, blocks, threads, hub);
}

// The transpose of a compacted block (per src node u, the dst nodes v of its
// edges), for the backward of the aggregation as a gather.  Built in two
// steps riding on later sampling launches: an exclusive scan of the
// per-src edge counts (src_occ less the dst's own 1) into t_ptr, then a fill
// that writes every edge's v at its place in its u's list (the order the
// compaction counted them in: unspecified).
struct TransposeJob {
  const int32_t* indptr;
  const int32_t* indices;
  const int32_t* counts;   // counts[0] = n_dst, counts[1] = n_src
  const int32_t* src_occ;
  const int32_t* rank;     // [cap_edges] place of an edge among its src node's
  int32_t* t_ptr;          // [cap_src + 1]
  int32_t* t_dst;          // [cap_edges]
  int32_t fanout;
  int32_t cap_src;
};

__device__ __forceinline__ void transpose_fill(const TransposeJob& t, uint32_t first, uint32_t stride) {
  if (!t.t_dst) return;
  const uint32_t slots = (uint32_t)t.counts[0] * (uint32_t)t.fanout, f = (uint32_t)t.fanout;
  for (uint32_t s = first; s < slots; s += stride) {  // (32 bits: as in index_passes)
    const int32_t v = (int32_t)(s / f);
    const int32_t r = (int32_t)(s - v * f);
    const int32_t e0 = t.indptr[v];
    if (r >= t.indptr[v + 1] - e0) continue;
    const int32_t u = t.indices[e0 + r];
    if ((uint32_t)u >= (uint32_t)t.cap_src) continue;
    const int32_t pos = t.t_ptr[u] + t.rank[e0 + r];
    // (a place outside its list only with a device error raised: an invalid
    // pick counted nowhere but pointing at row 0)
    if (pos >= t.t_ptr[u] && pos < t.t_ptr[u + 1]) t.t_dst[pos] = v;
  }
}

// Calls that may follow one another without a begin launch ("chained":
// the previous call's last step has already prepared the next one); the
// epoch check of the begin launch keeps room for that many.
constexpr uint32_t kChainCalls = 1024;

// The last step of a sampling call: the last hop's compaction, the fill of a
// pending transpose, and (by the first thread) the header marking the
// per-node words as built for this node count up to this call's epochs.  It
// also prepares a chained next call: the per-call scan state is cleared and
// the next call's epochs are reserved (a begin launch sets them again).
struct SampleTail {
  IndexJob job;
  Header* hdr;
  TransposeJob tfill;
  int32_t* zero;  // the per-call scan state
  int64_t n_zero;
  uint32_t L;
};

__device__ __forceinline__ void finish_sampling(const SampleTail& t, int64_t block, int64_t blocks,
                                                int threads) {
  __shared__ HubCounts hub;
  index_slots(t.job, block, blocks, threads, hub);
  transpose_fill(t.tfill, (uint32_t)(block * threads + threadIdx.x), (uint32_t)(blocks * threads));
  for (int64_t i = block * threads + threadIdx.x; i < t.n_zero; i += blocks * threads) t.zero[i] = 0;
  if (block == 0 && threadIdx.x == 0) {
    const uint32_t top = t.hdr->top_epoch;
    t.hdr->done_epoch = top;
    t.hdr->top_epoch = top + t.L;
    t.hdr->num_nodes = t.job.num_nodes;
    t.hdr->magic = kMagic;
  }
}

}  // namespace gnn

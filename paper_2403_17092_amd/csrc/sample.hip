// Layer-wise neighbour sampling and block construction.
//
// Per hop h (Neighbor Sampling, paper section 2.2; budgets of section 5.1.2),
// two launches, none of which needs a count on the host:
//   1. sample:  a group of lanes per dst node, four draws each (group_pick);
//               Floyd's algorithm over CSR
//               positions driven by Philox4x64-10 keyed by (rng_key, hop,
//               node); the picks are ranked across the group and written, in
//               ascending position order, into a padded [n_dst x fanout]
//               layout (unused slots hold -1), so sampling does not wait for
//               a prefix sum.  The padded position space is the dst list
//               followed by the padded slots, i.e. (dst index, rank) order.
//               Every key records itself in a per-node word with a 64-bit
//               atomicMax of (epoch << 32 | ~position), so after the launch
//               the word of a node holds the first position at which it
//               occurs in this hop.  The same launch compacts the previous
//               hop's edges (step 3), which needs that hop's local ids.
//   2. scans:   two single-pass scans in one launch: the per-node counts
//               into indptr, and the first-occurrence flags into local ids;
//               each first occurrence writes src_nodes, the initial src_occ
//               (1), its node's local id into a per-node table, and its
//               mark into its slot.
//   3. indices: padded slot (i, r), r < k_i, becomes indices[indptr[i] + r] =
//               the local id of its key, and adds 1 to src_occ of that id
//               unless it is marked.
// The last hop's step 3 is a launch of its own.  Words of earlier hops and
// calls carry smaller epochs and lose every atomicMax, so the per-node arrays
// are cleared only when the workspace header says they were not built by an
// earlier call for this node count.  The result does not depend on thread
// scheduling.
#include <atomic>

#include "internal.hpp"
#include "philox.hpp"
#include "relabel.hpp"
#include "sampler.hpp"
#include "wave.hpp"

namespace gnn {

namespace {

constexpr int kThreads = 256;
constexpr int kSampleThreads = 512;      // the last compaction's blocks
constexpr int kSampleMaxBlocks = 2048;
// beside another stream's work the wide form leaves that work its share of the
// CUs (six pipelined steps of a 16M-node workload: 1,389 us uncapped, 1,356 with
// 256 workgroups, 1,351 with 192, 1,378 with 128; alone, its serial step 255 ->
// 262 us).  Narrow frontiers, a wave per node, are bound by their chain of loads
// and keep their workgroups (three pipelined steps of 536 seeds 267 -> 238 us)
constexpr int kSampleBesideBlocks = 192;
constexpr int kIndexBlocksMax = 1024;
// slots of a hop from which the sampling looks before its atomics
constexpr int64_t kLookSlots = 1 << 16;
constexpr int64_t kResidentWaves = 8192;  // 256 CUs x 32 waves
constexpr int kBeginBlocks = 256;
constexpr int kMaxExtraFills = 4;
// scan blocks (256 threads) of a launch, certainly resident at once: 256 CUs x 4
constexpr int64_t kScanBlocks = 1024;

// single-pass scan tiles: ITEMS per thread, the smallest of 2, 4, 8 whose
// live tiles fit the grid (small tiles keep more workgroups in flight)
constexpr int kScanItemsMin = 2;
constexpr int kScanItemsMax = 8;

// Per-node word of the first-occurrence race: epoch in the high half, the
// complemented position in the low half (so atomicMax keeps the newest epoch
// and, within it, the smallest position).
__device__ __forceinline__ uint64_t occ_word(uint32_t epoch, int64_t pos) {
  return ((uint64_t)epoch << 32) | (uint32_t)~(uint32_t)pos;
}

// ---------------------------------------------------------------------------
// Single-pass exclusive scan (decoupled look-back, Merrill & Garland 2016).
// Status word per tile: flag in the high half (0 empty, 1 tile aggregate, 2
// inclusive prefix).  The first wave looks back over up to 1,024 predecessors
// at once (16 reads per lane), so a scan whose tiles are all in flight waits
// for one round trip after the last aggregate, not for a chain of 64-wide
// windows (a coherent read goes past the XCDs' L2s, ~1.5 us).
// ---------------------------------------------------------------------------
struct ScanState {
  uint64_t* status;
  int* err;  // device error word (a look-back that gives up sets GNN_DEVERR_SYNC)
};

// Look-back reads of an unpublished predecessor before the wait gives up
// (far beyond any live wait: a predecessor that runs publishes within
// microseconds).  Giving up treats the unread predecessors as zero, so every
// prefix stays at or below the true one and every store stays in bounds.
constexpr int32_t kScanSpinLimit = 1 << 22;

__device__ __forceinline__ uint64_t scan_word(uint32_t flag, int32_t v) {
  return ((uint64_t)flag << 32) | (uint32_t)v;
}

__device__ __forceinline__ int32_t wave_sum_i32(int32_t x) {
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) x += __shfl_xor(x, d, WAVE);
  return x;
}

__device__ __forceinline__ int32_t block_scan_excl(int32_t x, int32_t* total, int32_t* wsum) {
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
  const int32_t inc = wave_inclusive_scan(x);
  if (lane == 63) wsum[wid] = inc;
  __syncthreads();
  int32_t off = 0, tot = 0;
#pragma unroll
  for (int w = 0; w < kThreads / 64; ++w) {
    off += (w < wid) ? wsum[w] : 0;
    tot += wsum[w];
  }
  __syncthreads();
  *total = tot;
  return off + inc - x;
}

// The K * 64 tiles below `top` (K per lane of the wave, nearest first in k and
// lane): adds the aggregates down to the nearest inclusive prefix, or all of
// them, to *prefix; true if there was one (tile 0's is).
template <int K>
__device__ __forceinline__ bool look_back_window(ScanState ss, int64_t top, int32_t* prefix) {
  const int lane = threadIdx.x & 63;
  uint64_t w[K];
#pragma unroll
  for (int k = 0; k < K; ++k) w[k] = 0;
  int32_t spins = 0;
  while (true) {  // bounded
    // only what has not been published is read again, and not at once: a
    // launch beside this one shares the memory these reads go to
    bool empty = false;
#pragma unroll
    for (int k = 0; k < K; ++k) {
      const int64_t j = top - 1 - lane - 64 * k;
      if ((w[k] >> 32) == 0)
        w[k] = j >= 0 ? __hip_atomic_load(&ss.status[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                      : scan_word(2, 0);  // before tile 0: an inclusive 0
    }
#pragma unroll
    for (int k = 0; k < K; ++k) empty |= (w[k] >> 32) == 0;
    if (ballot(empty) == 0ull) break;
    if (++spins > kScanSpinLimit) {
      // flag the error and go on with what has been published
      if (lane == 0) set_device_error(ss.err, GNN_DEVERR_SYNC);
      break;
    }
    __builtin_amdgcn_s_sleep(2);
  }
  // the nearest inclusive prefix, by distance (64 K: none in the window)
  int32_t stop = 64 * K;
#pragma unroll
  for (int k = K - 1; k >= 0; --k) stop = (w[k] >> 32) == 2 ? lane + 64 * k : stop;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) stop = min(stop, __shfl_xor(stop, d, WAVE));
  int32_t sum = 0;
#pragma unroll
  for (int k = 0; k < K; ++k) sum += lane + 64 * k <= stop ? (int32_t)(uint32_t)w[k] : 0;
  *prefix += wave_sum_i32(sum);
  return stop < 64 * K;
}

// Exclusive prefix of `tile` given its aggregate; run by the first wave.
template <bool SMALL>
__device__ __forceinline__ int32_t look_back(ScanState ss, int64_t tile, int32_t agg) {
  const int lane = threadIdx.x & 63;
  if (lane == 0)
    __hip_atomic_store(&ss.status[tile], scan_word(tile == 0 ? 2 : 1, agg), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  if (tile == 0) return 0;
  int32_t prefix = 0;
  // (a short form for the few tiles of a small grid)
  constexpr int K = SMALL ? 2 : 16;
  for (int64_t top = tile; !look_back_window<K>(ss, top, &prefix); top -= K * 64) {
  }
  if (lane == 0)
    __hip_atomic_store(&ss.status[tile], scan_word(2, prefix + agg), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  return prefix;
}

// Tile `tile` of a scan of n items in tiles of kThreads * ITEMS.  Item i is
// value(i, raw, word) of raw = load(i) and word = look(i, raw); the two reads of
// a thread's items are each issued together, items past n reading item 0's
// places instead (a read under a condition waits for the one before it).  Calls
// store(i, exclusive prefix, item, raw) for the items i < n, and finish(total)
// if it is the last tile.  Every lower tile's workgroup must be running or done.
template <int ITEMS, bool SMALL, typename Load, typename Look, typename Value, typename Store,
          typename Finish>
__device__ __forceinline__ void tile_scan(ScanState ss, int64_t tile, int64_t n, Load load, Look look,
                                          Value value, Store store, Finish finish) {
  __shared__ int32_t wsum[kThreads / 64];
  __shared__ int32_t s_prefix;
  constexpr int kTile = kThreads * ITEMS;
  const int64_t base = tile * kTile + (int64_t)threadIdx.x * ITEMS;
  int32_t v[ITEMS], raw[ITEMS];
  uint64_t word[ITEMS];
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) raw[i] = load(base + i < n ? base + i : 0);
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) word[i] = look(base + i < n ? base + i : 0, raw[i]);
  int32_t s = 0;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    v[i] = base + i < n ? value(base + i, raw[i], word[i]) : 0;
    s += v[i];
  }
  int32_t agg;
  const int32_t excl = block_scan_excl(s, &agg, wsum);
  if (threadIdx.x < 64) {
    const int32_t prefix = look_back<SMALL>(ss, tile, agg);
    if (threadIdx.x == 0) {
      s_prefix = prefix;
      if ((tile + 1) * kTile >= n) finish(prefix + agg);
    }
  }
  __syncthreads();
  int32_t run = s_prefix + excl;
#pragma unroll
  for (int i = 0; i < ITEMS; ++i) {
    if (base + i < n) store(base + i, run, v[i], raw[i]);
    run += v[i];
  }
}

__host__ __device__ inline int64_t scan_tiles(int64_t n, int items) {
  const int64_t t = (n + (int64_t)kThreads * items - 1) / ((int64_t)kThreads * items);
  return t < 1 ? 1 : t;
}
// status words of a scan of up to `cap` items: with tiles of fewer than
// kScanItemsMax items per thread all tiles are in the grid at once
inline int64_t scan_words(int64_t cap) {
  return std::min(scan_tiles(cap, kScanItemsMin), std::max(kScanBlocks, scan_tiles(cap, kScanItemsMax)));
}

// ---------------------------------------------------------------------------
// 0. begin: clear the per-call scan state.  The persistent header holds a
//    magic word, the last finished epoch and the node count the per-node
//    words were built for; if it does not match (first use, another graph
//    size, epochs too close to wrapping around for kChainCalls more calls) the
//    per-node words are cleared and the epochs restart.  Hop h of this call
//    uses epoch top - L + h, where top (header word 2) is written here and
//    becomes the finished epoch at the end of the call.  A chained call skips
//    this launch: the previous call's last step did the same preparation.
// ---------------------------------------------------------------------------
// Fill ranges of the caller done by the same launch (the training step's
// gradient buffers).
struct FillSet {
  int32_t* p[kMaxExtraFills];
  int64_t n[kMaxExtraFills];
  int32_t v[kMaxExtraFills];
  int32_t count;
};

__global__ void __launch_bounds__(kThreads)
begin_kernel(Header* hdr, uint64_t* occ, int64_t N, int32_t L, int32_t* zero, int64_t n_zero,
             FillSet extra) {
  const uint32_t magic = hdr->magic, done = hdr->done_epoch;
  const int64_t n_old = hdr->num_nodes;
  const bool fresh = magic != kMagic || n_old != N || done > 0xFFFFFFFFu - (kChainCalls + 1) * (uint32_t)L;
  const int64_t tid = (int64_t)blockIdx.x * kThreads + threadIdx.x;
  const int64_t stride = (int64_t)gridDim.x * kThreads;
  for (int64_t i = tid; i < n_zero; i += stride) zero[i] = 0;
  for (int r = 0; r < extra.count; ++r)
    for (int64_t i = tid; i < extra.n[r]; i += stride) extra.p[r][i] = extra.v[r];
  if (fresh)
    for (int64_t i = tid; i < N; i += stride) occ[i] = 0;
  if (blockIdx.x == 0 && threadIdx.x == 0) hdr->top_epoch = (fresh ? 0u : done) + (uint32_t)L;
}

// The last launch of a call when no later launch takes it over.
__global__ void __launch_bounds__(kSampleThreads) indices_kernel(SampleTail t) {
  finish_sampling(t, blockIdx.x, gridDim.x, kSampleThreads);
}

// ---------------------------------------------------------------------------
// 1. sample (+ the previous hop's indices in blocks past the sampling grid)
// ---------------------------------------------------------------------------
template <int P, typename RP>
__global__ void __launch_bounds__(kThreads)
sample_kernel(const RP* __restrict__ rowptr, const int32_t* __restrict__ col, int64_t num_nodes,
              const int32_t* __restrict__ dst, const int32_t* n_dst_dev, int32_t cap_dst,
              int32_t* counts, int32_t fanout, uint64_t rng_key, uint32_t hop,
              const Header* hdr, int32_t L, int32_t* __restrict__ nbr_pad,
              int32_t* __restrict__ kcount, uint64_t* __restrict__ occ, int32_t sample_blocks,
              IndexJob prev, TransposeJob tfill, int* err) {
  if ((int32_t)blockIdx.x >= sample_blocks) {
    __shared__ HubCounts hub;
    const uint32_t b = blockIdx.x - sample_blocks, nb = gridDim.x - sample_blocks;
    index_slots(prev, b, nb, kThreads, hub);
    transpose_fill(tfill, b * kThreads + threadIdx.x, nb * kThreads);
    return;
  }
  const int lane = lane_id();
  const int j = lane & (P - 1);
  // hop 1: the batch (its count is the capacity); later hops: the previous
  // hop's src count, from the device
  int32_t n_dst = n_dst_dev ? *n_dst_dev : cap_dst;
  n_dst = n_dst > cap_dst ? cap_dst : n_dst;
  if (blockIdx.x == 0 && threadIdx.x == 0) counts[0] = n_dst;
  const uint32_t ep = hdr->top_epoch - (uint32_t)L + hop;
  const uint32_t ep1 = hdr->top_epoch - (uint32_t)L + 1;  // the call's first epoch
  // Many picks: look at a node's word before the atomic, which a dst node and
  // a position after one already recorded then skip (the hubs' words would
  // take thousands of atomics one after the other, see HubCounts).  Few: the
  // extra round trip costs more, and the dst nodes record their positions.
  const bool look = (int64_t)n_dst * fanout >= kLookSlots;  // (uniform)
  // records a pick w (checked) at slot `at` of the hop
  auto record = [&](int32_t w, uint64_t seen, int64_t at) {
    const uint64_t word = occ_word(ep, n_dst + at);
    const uint32_t se = (uint32_t)(seen >> 32);
    // a dst node (a word of an earlier hop of this call) is never a first
    // occurrence, nor is a position after one already recorded
    if (look && (seen >= word || (se >= ep1 && se < ep))) return;
    atomicMax(reinterpret_cast<unsigned long long*>(&occ[w]), word);
  };
  auto in_range = [&](int32_t w) { return w >= 0 && (int64_t)w < num_nodes; };
  // the words of picks as they stand, possibly not yet showing what other
  // groups record meanwhile
  auto peek = [&](int32_t w) -> uint64_t { return look && in_range(w) ? occ[w] : 0; };
  // groups of P lanes, one dst node each; the loop bound is wave-uniform
  constexpr int kPerWave = WAVE / P;
  const int64_t wave = ((int64_t)blockIdx.x * kThreads + threadIdx.x) >> 6;
  const int64_t waves = (int64_t)sample_blocks * (kThreads / 64);
  for (int64_t base = wave * kPerWave; base < n_dst; base += waves * kPerWave) {
    const int64_t i = base + lane / P;
    const bool live = i < n_dst;
    const int32_t v = live ? dst[i] : -1;
    const bool valid = live && in_range(v);
    if (live && !valid && j == 0) set_device_error(err, GNN_DEVERR_SEED_RANGE);
    const int64_t row = i * (int64_t)fanout;
    int32_t k = 0;
    if constexpr (P == WAVE) {
      int32_t w = -1;
      if (valid) k = wave_sample(rowptr, col, v, fanout, rng_key, hop, &w);  // (v is wave-uniform)
      if (lane < k && !in_range(w)) {
        set_device_error(err, GNN_DEVERR_GRAPH);
        w = -1;
      }
      const uint64_t seen = peek(w);
      if (lane < fanout) nbr_pad[row + lane] = w;
      if (lane < k && w >= 0) record(w, seen, row + lane);
    } else {
      int64_t start = 0, d = 0;
      if (valid) row_range(rowptr, v, start, d);
      uint32_t pos[4];
      int32_t rank[4];
      k = group_pick<P>(valid, d, v, fanout, rng_key, hop, pos, rank);
      if (!live) continue;
      int32_t w[4];
      uint64_t seen[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) w[e] = 4 * j + e < k ? col[start + pos[e]] : -1;
#pragma unroll
      for (int e = 0; e < 4; ++e) seen[e] = peek(w[e]);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int32_t s = 4 * j + e;
        if (s < k && !in_range(w[e])) {
          set_device_error(err, GNN_DEVERR_GRAPH);
          w[e] = -1;
        }
        // (unused slots, s >= k, hold -1: the used ones have ranks below k)
        if (s < fanout) nbr_pad[row + (s < k ? rank[e] : s)] = w[e];
        if (s < k && w[e] >= 0) record(w[e], seen[e], row + rank[e]);
      }
    }
    if (j == 0) {
      kcount[i] = k;
      // (with `look`, later hops' dst nodes keep their word of an earlier hop)
      if (valid && (hop == 1 || !look))
        atomicMax(reinterpret_cast<unsigned long long*>(&occ[v]), occ_word(ep, i));
    }
  }
}

// ---------------------------------------------------------------------------
// 2. scans: blocks [0, count_blocks) scan the per-node counts into indptr
//    (counts[2] = E); the others scan the first-occurrence flags into local
//    ids (counts[1] = n_src) and emit src_nodes, src_occ and the per-node id.
// ---------------------------------------------------------------------------
struct ScanArgs {
  const int32_t* dst;
  int32_t* nbr_pad;
  int32_t* counts;
  int32_t fanout;
  const int32_t* kcount;
  int32_t* indptr;
  const uint64_t* occ;
  const Header* hdr;
  int32_t L;
  uint32_t hop;
  int64_t num_nodes;
  int32_t* nid;
  int32_t cap_src;
  int32_t* src_nodes;
  int32_t* src_occ;
  ScanState s_cnt, s_flag, s_tr;
  TransposeJob tr;  // (t_ptr set: the previous hop's per-src edge counts are scanned too)
  int32_t* ticket;
  int32_t use_ticket;
  int32_t min_items;  // tiles of fewer items per thread are not used (not SMALL)
  int* err;
};

// Tile t of the launch: the count tiles, the flag tiles, the transpose's.
template <int ITEMS, bool SMALL = false>
__device__ __forceinline__ void scan_tile(const ScanArgs& a, int64_t t, int64_t ct, int64_t ft,
                                          int32_t n_dst, int32_t n_tr) {
  auto no_look = [](int64_t, int32_t) -> uint64_t { return 0; };
  if (t < ct) {
    auto load = [&](int64_t i) -> int32_t { return a.kcount[i]; };
    auto value = [](int64_t, int32_t k, uint64_t) { return k; };
    auto store = [&](int64_t i, int32_t pre, int32_t, int32_t) { a.indptr[i] = pre; };
    auto finish = [&](int32_t total) {
      a.indptr[n_dst] = total;
      a.counts[2] = total;
    };
    tile_scan<ITEMS, SMALL>(a.s_cnt, t, n_dst, load, no_look, value, store, finish);
  } else if (t < ct + ft) {
    const uint32_t ep = a.hdr->top_epoch - (uint32_t)a.L + a.hop;
    auto load = [&](int64_t i) -> int32_t {
      const int32_t* p = i < n_dst ? a.dst + i : a.nbr_pad + (i - n_dst);
      return *p;
    };
    // the word of a pick's node (of node 0 for a dst node or an unused slot)
    auto look = [&](int64_t i, int32_t key) -> uint64_t { return a.occ[i >= n_dst && key >= 0 ? key : 0]; };
    // the dst nodes (distinct) always keep their positions as ids
    auto value = [&](int64_t i, int32_t key, uint64_t word) -> int32_t {
      return i < n_dst || (key >= 0 && word == occ_word(ep, i)) ? 1 : 0;
    };
    auto store = [&](int64_t i, int32_t id, int32_t f, int32_t key) {
      if (!f) return;
      if (id < a.cap_src) {
        a.src_nodes[id] = key;
        a.src_occ[id] = 1;  // the dst node itself, or the new node's first edge
        if (i >= n_dst) a.nbr_pad[i - n_dst] = (int32_t)((uint32_t)key | kFirstPick);
        // (a dst node of a later hop keeps the id it got when it was new)
        if ((i >= n_dst || a.hop == 1) && key >= 0 && (int64_t)key < a.num_nodes) a.nid[key] = id;
      } else {
        set_device_error(a.err, GNN_DEVERR_CAPACITY);
      }
    };
    auto finish = [&](int32_t total) { a.counts[1] = total; };
    tile_scan<ITEMS, SMALL>(a.s_flag, t - ct, (int64_t)n_dst * (1 + a.fanout), load, look, value, store,
                            finish);
  } else {
    const TransposeJob& tr = a.tr;
    const int32_t nd = tr.counts[0];
    auto load = [&](int64_t u) -> int32_t { return tr.src_occ[u]; };
    auto value = [&](int64_t u, int32_t occ, uint64_t) -> int32_t {
      const int32_t c = occ - (u < nd ? 1 : 0);
      return c > 0 ? c : 0;
    };
    auto store = [&](int64_t u, int32_t pre, int32_t, int32_t) { tr.t_ptr[u] = pre; };
    auto finish = [&](int32_t total) { tr.t_ptr[n_tr] = total; };
    tile_scan<ITEMS, SMALL>(a.s_tr, t - ct - ft, n_tr, load, no_look, value, store, finish);
  }
}

// The launch's tiles are laid out over the live counts: tiles of the fewest
// items per thread that fit the grid, one per workgroup, numbered by block id
// (the grid is resident at once, so every tile waits only on running tiles);
// past that, tiles of kScanItemsMax items taken from a ticket counter in
// arrival order until none is left.  The grid is sized by the capacity; tiles
// sized by it left a hop of 96K dst nodes (575K positions of 4.3M) 281 tiles
// of 8 dependent lookups per thread in place of 749 of 4: 54.5 us for the
// launch, now 19.9.
// SMALL: the capacity's tiles of the fewest items fit the grid, so the live
// ones do, and the kernel holds that one form (a short kernel starts sooner).
template <bool SMALL>
__global__ void __launch_bounds__(kThreads) scans_kernel(ScanArgs a) {
  const int32_t n_dst = a.counts[0];
  const int32_t n_tr = a.tr.t_ptr ? a.tr.counts[1] : 0;
  int64_t ct, ft, total;
  auto lay = [&](int items) {
    ct = scan_tiles(n_dst, items);
    ft = scan_tiles((int64_t)n_dst * (1 + a.fanout), items);
    total = ct + ft + (a.tr.t_ptr ? scan_tiles(n_tr, items) : 0);
    return total <= (int64_t)gridDim.x;
  };
  if constexpr (SMALL) {
    lay(kScanItemsMin);
    if (blockIdx.x < total) scan_tile<kScanItemsMin, true>(a, blockIdx.x, ct, ft, n_dst, n_tr);
    return;
  }
  if (!a.use_ticket) {
    const int64_t t = blockIdx.x;
    if (a.min_items <= 2 && lay(2)) {
      if (t < total) scan_tile<2>(a, t, ct, ft, n_dst, n_tr);
      return;
    }
    if (a.min_items <= 4 && lay(4)) {
      if (t < total) scan_tile<4>(a, t, ct, ft, n_dst, n_tr);
      return;
    }
    if (lay(8)) {
      if (t < total) scan_tile<8>(a, t, ct, ft, n_dst, n_tr);
      return;
    }
  }
  lay(kScanItemsMax);
  __shared__ int32_t s_tile;
  while (true) {  // (tickets only grow: at most total + gridDim.x of them)
    if (threadIdx.x == 0) s_tile = atomicAdd(a.ticket, 1);
    __syncthreads();
    const int64_t t = s_tile;
    __syncthreads();
    if (t >= total) return;
    scan_tile<kScanItemsMax>(a, t, ct, ft, n_dst, n_tr);
  }
}

}  // namespace

// Scratch layout of one gnn_sample_blocks call.  Persistent part (kept
// between calls, laid out from N alone): the header, the per-node
// first-occurrence words and the per-node local-id table (a node's id is the
// same in every hop of a call it occurs in).  Per call: tickets and scan
// status (cleared by the begin launch), per-hop counts, two padded edge
// buffers (hops alternate).
struct SampleScratch {
  Header* hdr;
  uint64_t* occ;                         // [N]
  int32_t* nid;                          // [N]
  int32_t* tickets;                      // [L]
  uint64_t* status[3 * GNN_MAX_LAYERS];  // scan tile status (counts, flags, transposed counts)
  void* zero_begin;                      // [zero_begin, zero_end): cleared once per call
  void* zero_end;
  int32_t* kcount[GNN_MAX_LAYERS];       // [cap_dst]
  int32_t* nbr_pad[2];                   // [max cap_edges]
};

static size_t carve_sample(Carver& c, const int32_t* cap_dst, const int32_t* cap_src,
                           const int64_t* cap_edges, int32_t L, int64_t N, SampleScratch* s) {
  s->hdr = c.take<Header>(1);
  s->occ = c.take<uint64_t>(std::max<int64_t>(1, N));
  s->nid = c.take<int32_t>(std::max<int64_t>(1, N));
  s->zero_begin = c.take<char>(0);
  s->tickets = c.take<int32_t>(GNN_MAX_LAYERS);
  for (int h = 0; h < L; ++h) {
    s->status[3 * h] = c.take<uint64_t>(scan_words(cap_dst[h]));
    s->status[3 * h + 1] = c.take<uint64_t>(scan_words((int64_t)cap_dst[h] + cap_edges[h]));
    s->status[3 * h + 2] = c.take<uint64_t>(scan_words(cap_src[h]));
  }
  s->zero_end = c.take<char>(0);
  int64_t max_edges = 1;
  for (int h = 0; h < L; ++h) {
    s->kcount[h] = c.take<int32_t>(std::max<int64_t>(1, cap_dst[h]));
    max_edges = std::max<int64_t>(max_edges, cap_edges[h]);
  }
  s->nbr_pad[0] = c.take<int32_t>(max_edges);
  s->nbr_pad[1] = c.take<int32_t>(max_edges);
  return c.off;
}

size_t sample_scratch_bytes(const int32_t* cap_dst, const int32_t* cap_src,
                            const int64_t* cap_edges, int32_t L, int64_t N) {
  Carver c(nullptr, 0);
  SampleScratch s;
  return carve_sample(c, cap_dst, cap_src, cap_edges, L, N, &s);
}

template <typename RP>
static int sample_hops(const gnn_csr* csr, const RP* rowptr, const int32_t* seeds, int32_t B,
                       const int32_t* fanouts, int32_t L, uint64_t rng_key, gnn_block* blocks,
                       void* ws, size_t ws_bytes, const FillRange* extra, int n_extra,
                       SampleTail* tail, const BlockTranspose* tr, hipStream_t st, bool chained,
                       bool beside) {
  if (n_extra < 0 || n_extra > kMaxExtraFills) return fail(GNN_EINVAL, "sampler: too many fills");
  if (int rc = check_csr_options(csr, "sampler")) return rc;
  int32_t cap_dst[GNN_MAX_LAYERS], cap_src[GNN_MAX_LAYERS];
  int64_t cap_edges[GNN_MAX_LAYERS];
  for (int h = 0; h < L; ++h) {
    cap_src[h] = blocks[h].cap_src;
    cap_dst[h] = blocks[h].cap_dst;
    cap_edges[h] = blocks[h].cap_edges;
    if (cap_edges[h] != (int64_t)cap_dst[h] * fanouts[h])
      return fail(GNN_EINVAL, "gnn_sample_blocks: cap_edges must equal cap_dst * fanout");
  }
  const int64_t N = csr->num_nodes;
  Carver c(ws, ws_bytes);
  SampleScratch sc;
  carve_sample(c, cap_dst, cap_src, cap_edges, L, N, &sc);
  if (!c.fits()) return fail(GNN_EWORKSPACE, "gnn_sample_blocks: workspace %zu < %zu bytes", ws_bytes, c.off);
  int* err = device_error_word();
  if (!err) return fail(GNN_EHIP, "device error word unavailable");

  const int64_t zero_words =
      (static_cast<char*>(sc.zero_end) - static_cast<char*>(sc.zero_begin)) / 4;
  FillSet fs{};
  for (int r = 0; r < n_extra; ++r) {
    fs.p[r] = static_cast<int32_t*>(extra[r].p);
    fs.n[r] = extra[r].p ? extra[r].n_words : 0;
    fs.v[r] = extra[r].value;
  }
  fs.count = n_extra;
  if (blocks[0].cap_dst != B) return fail(GNN_EINVAL, "sampler: hop 1 capacity %d != batch %d", blocks[0].cap_dst, B);
  if (!chained || n_extra > 0)
    launch("begin", begin_kernel, kBeginBlocks, kThreads, 0, st, sc.hdr, sc.occ, N, L,
           static_cast<int32_t*>(sc.zero_begin), zero_words, fs);

  // transposes (hops h < L - 1, if asked for): hop h's counts are scanned in
  // hop h + 1's scans launch and its lists filled by the launch after it
  auto tjob = [&](int h) -> TransposeJob {
    TransposeJob t{};
    if (!tr || h < 0 || h >= L - 1 || !tr[h].t_ptr) return t;
    const gnn_block& b = blocks[h];
    t = TransposeJob{b.indptr, b.indices, b.counts, b.src_occ, tr[h].rank, tr[h].t_ptr,
                     tr[h].t_dst, fanouts[h], b.cap_src};
    return t;
  };
  IndexJob prev{};
  int64_t prev_slots = 0;
  for (int h = 0; h < L; ++h) {
    gnn_block& bk = blocks[h];
    const int32_t* dst = h == 0 ? seeds : blocks[h - 1].src_nodes;
    const int32_t* n_dst_src = h == 0 ? nullptr : blocks[h - 1].counts + 1;
    const int32_t f = fanouts[h];
    int32_t* pad = sc.nbr_pad[h & 1];

    // lanes per dst node: a wave, a draw per lane, while one wave per node fits
    // the resident waves (the shortest chain: 256 dst nodes of 10 picks 6.0 us
    // against 6.8), else four draws per lane (96K dst nodes of 5 picks 43 -> 31
    // us; with a draw per lane, Philox alone took most of it), on more lanes
    // while the capacity's waves are few (idle lanes then spread the nodes'
    // scattered reads over the CUs: 4.9K dst nodes of 3 picks 8.5 -> 7.3 us)
    int P = 1;
    while (4 * P < f || (P < 16 && (int64_t)bk.cap_dst * P < 64 * 4096)) P *= 2;
    if ((int64_t)bk.cap_dst <= kResidentWaves) P = WAVE;
    const int64_t per_block = kThreads / P;
    const int64_t sblocks = std::min<int64_t>(beside && P < WAVE ? kSampleBesideBlocks : kSampleMaxBlocks,
                                              std::max<int64_t>(1, ceil_div(bk.cap_dst, per_block)));
    // extra blocks: hop h - 1's compaction and hop h - 2's transpose fill
    const TransposeJob tfill = tjob(h - 2);
    const int64_t extra_slots = std::max<int64_t>(prev_slots, tfill.t_dst ? blocks[h - 2].cap_edges : 0);
    const int64_t iblocks =
        h == 0 ? 0
               : std::min<int64_t>(kIndexBlocksMax,
                                   std::max<int64_t>(1, ceil_div(extra_slots, kThreads * 4)));
    const unsigned grid = (unsigned)(sblocks + iblocks);
    auto go = [&](auto kernel) {
      launch("sample", kernel, grid, kThreads, 0, st, rowptr, csr->col, N, dst, n_dst_src,
             bk.cap_dst, bk.counts, f, rng_key, (uint32_t)(h + 1), sc.hdr, L, pad, sc.kcount[h],
             sc.occ, (int32_t)sblocks, prev, tfill, err);
    };
    if (P == 1) go(sample_kernel<1, RP>);
    else if (P == 2) go(sample_kernel<2, RP>);
    else if (P == 4) go(sample_kernel<4, RP>);
    else if (P == 8) go(sample_kernel<8, RP>);
    else if (P == 16) go(sample_kernel<16, RP>);
    else go(sample_kernel<WAVE, RP>);
    // hop h - 1's transposed counts (its compaction ran in this hop's sample launch)
    const TransposeJob tscan = tjob(h - 1);
    ScanArgs sa{};
    sa.dst = dst;
    sa.nbr_pad = pad;
    sa.counts = bk.counts;
    sa.fanout = f;
    sa.kcount = sc.kcount[h];
    sa.indptr = bk.indptr;
    sa.occ = sc.occ;
    sa.hdr = sc.hdr;
    sa.L = L;
    sa.hop = (uint32_t)(h + 1);
    sa.num_nodes = N;
    sa.nid = sc.nid;
    sa.cap_src = bk.cap_src;
    sa.src_nodes = bk.src_nodes;
    sa.src_occ = bk.src_occ;
    sa.s_cnt = ScanState{sc.status[3 * h], err};
    sa.s_flag = ScanState{sc.status[3 * h + 1], err};
    sa.s_tr = ScanState{h >= 1 ? sc.status[3 * (h - 1) + 2] : nullptr, err};
    sa.tr = tscan;
    sa.ticket = sc.tickets + h;
    sa.use_ticket = csr->scan_order == 1 ? 1 : 0;
    sa.min_items = beside ? kScanItemsMax : kScanItemsMin;
    sa.err = err;
    const int64_t tiles = scan_tiles(bk.cap_dst, kScanItemsMin) +
                          scan_tiles((int64_t)bk.cap_dst + bk.cap_edges, kScanItemsMin) +
                          (tscan.t_ptr ? scan_tiles(blocks[h - 1].cap_src, kScanItemsMin) : 0);
    if (tiles <= kScanBlocks && !sa.use_ticket)
      launch("scans", scans_kernel<true>, (unsigned)tiles, kThreads, 0, st, sa);
    else
      launch("scans", scans_kernel<false>, (unsigned)std::min(kScanBlocks, tiles), kThreads, 0, st, sa);
    GNN_LAUNCH_CHECK("gnn_sample_blocks");
    prev = IndexJob{pad, sc.kcount[h], bk.indptr, bk.counts, sc.nid, bk.indices, bk.src_occ,
                    tr && h < L - 1 && tr[h].t_ptr ? tr[h].rank : nullptr, f, bk.cap_src, B <= kHubSeeds ? 0 : B, N};
    prev_slots = bk.cap_edges;
  }
  // the last step: the last hop's compaction and hop L - 2's transpose fill
  const SampleTail last{prev, sc.hdr, tjob(L - 2), static_cast<int32_t*>(sc.zero_begin), zero_words,
                        (uint32_t)L};
  if (tail) {  // the caller's next launch finishes the call
    *tail = last;
    return GNN_OK;
  }
  const int64_t tail_slots = std::max<int64_t>(prev_slots, last.tfill.t_dst ? blocks[L - 2].cap_edges : 0);
  const int64_t gx = std::min<int64_t>(kIndexBlocksMax, std::max<int64_t>(1, ceil_div(tail_slots, kSampleThreads * 4)));
  launch("indices", indices_kernel, (unsigned)gx, kSampleThreads, 0, st, last);
  GNN_LAUNCH_CHECK("gnn_sample_blocks indices");
  return GNN_OK;
}

int sample_blocks_impl(const gnn_csr* csr, const int32_t* seeds, int32_t B, const int32_t* fanouts,
                       int32_t L, uint64_t rng_key, gnn_block* blocks, void* ws, size_t ws_bytes,
                       const FillRange* extra, int n_extra, SampleTail* tail, hipStream_t st,
                       const BlockTranspose* tr, bool chained, bool beside) {
  if (csr->rowptr_bits == 64)
    return sample_hops(csr, static_cast<const int64_t*>(csr->rowptr), seeds, B, fanouts, L, rng_key,
                       blocks, ws, ws_bytes, extra, n_extra, tail, tr, st, chained, beside);
  return sample_hops(csr, static_cast<const int32_t*>(csr->rowptr), seeds, B, fanouts, L, rng_key,
                     blocks, ws, ws_bytes, extra, n_extra, tail, tr, st, chained, beside);
}

}  // namespace gnn

// ---------------------------------------------------------------------------
// C ABI
// ---------------------------------------------------------------------------
extern "C" {

int gnn_block_caps(int32_t B, const int32_t* fanouts, int32_t L, int64_t N, int32_t* cap_dst,
                   int32_t* cap_src, int64_t* cap_edges) {
  using namespace gnn;
  if (!fanouts || !cap_dst || !cap_src || !cap_edges) return fail(GNN_EINVAL, "gnn_block_caps: null pointer");
  if (L < 1 || L > GNN_MAX_LAYERS) return fail(GNN_EINVAL, "gnn_block_caps: L=%d not in [1, %d]", L, GNN_MAX_LAYERS);
  if (B < 0 || N < 0) return fail(GNN_EINVAL, "gnn_block_caps: negative size");
  int64_t nd = B;
  for (int h = 0; h < L; ++h) {
    if (fanouts[h] < 1 || fanouts[h] > GNN_MAX_FANOUT)
      return fail(GNN_EINVAL, "gnn_block_caps: fanout %d not in [1, %d]", fanouts[h], GNN_MAX_FANOUT);
    const int64_t e = nd * fanouts[h];
    int64_t ns = nd + e;
    if (ns > N && N >= nd) ns = N;
    if (e > INT32_MAX || ns > INT32_MAX) return fail(GNN_EINVAL, "gnn_block_caps: block too large");
    cap_dst[h] = (int32_t)nd;
    cap_edges[h] = e;
    cap_src[h] = (int32_t)ns;
    nd = ns;
  }
  return GNN_OK;
}

size_t gnn_sample_workspace_bytes(int32_t B, const int32_t* fanouts, int32_t L, int64_t N) {
  int32_t cd[GNN_MAX_LAYERS], cs[GNN_MAX_LAYERS];
  int64_t ce[GNN_MAX_LAYERS];
  if (gnn_block_caps(B, fanouts, L, N, cd, cs, ce) != GNN_OK) return 0;
  return gnn::sample_scratch_bytes(cd, cs, ce, L, N);
}

int gnn_sample_blocks(const gnn_csr* csr, const int32_t* seeds, int32_t B, const int32_t* fanouts,
                      int32_t L, uint64_t rng_key, gnn_block* blocks, void* ws, size_t ws_bytes,
                      void* stream) {
  using namespace gnn;
  if (!csr || !blocks || !fanouts || !ws) return fail(GNN_EINVAL, "gnn_sample_blocks: null pointer");
  if (!csr->rowptr || !csr->col) return fail(GNN_EINVAL, "gnn_sample_blocks: null CSR array");
  if (csr->rowptr_bits != 32 && csr->rowptr_bits != 64)
    return fail(GNN_EINVAL, "gnn_sample_blocks: rowptr_bits must be 32 or 64");
  if (csr->num_nodes < 0 || csr->num_nodes > INT32_MAX)
    return fail(GNN_EINVAL, "gnn_sample_blocks: num_nodes out of range");
  if (int rc = check_csr_options(csr, "gnn_sample_blocks")) return rc;
  if (B < 0 || (B > 0 && !seeds)) return fail(GNN_EINVAL, "gnn_sample_blocks: bad seeds");
  int32_t cd[GNN_MAX_LAYERS], cs[GNN_MAX_LAYERS];
  int64_t ce[GNN_MAX_LAYERS];
  if (int rc = gnn_block_caps(B, fanouts, L, csr->num_nodes, cd, cs, ce)) return rc;
  for (int h = 0; h < L; ++h) {
    const gnn_block& b = blocks[h];
    if (!b.indptr || !b.indices || !b.src_nodes || !b.src_occ || !b.counts)
      return fail(GNN_EINVAL, "gnn_sample_blocks: block %d has a null array", h);
    if (b.cap_dst < cd[h] || b.cap_src < cs[h] || b.cap_edges < ce[h])
      return fail(GNN_EWORKSPACE, "gnn_sample_blocks: block %d capacities below gnn_block_caps", h);
  }
  // the dst list of hop h+1 is the src list of hop h: its capacity must match
  for (int h = 1; h < L; ++h)
    if (blocks[h].cap_dst < blocks[h - 1].cap_src)
      return fail(GNN_EWORKSPACE, "gnn_sample_blocks: block %d cap_dst < block %d cap_src", h, h - 1);
  if (ws_bytes < sample_scratch_bytes(cd, cs, ce, L, csr->num_nodes))
    return fail(GNN_EWORKSPACE, "gnn_sample_blocks: workspace too small");
  // the kernels size their grids from the capacities given in `blocks`
  gnn_block local[GNN_MAX_LAYERS];
  for (int h = 0; h < L; ++h) {
    local[h] = blocks[h];
    local[h].cap_dst = cd[h];
    local[h].cap_src = blocks[h].cap_src;
    local[h].cap_edges = ce[h];
  }
  return sample_blocks_impl(csr, seeds, B, fanouts, L, rng_key, local, ws, ws_bytes, nullptr, 0,
                            nullptr, as_stream(stream));
}

}  // extern "C"

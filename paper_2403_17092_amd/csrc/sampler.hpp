// Uniform neighbour sampling without replacement by a whole wave (ShaDow
// extractor) and by groups of lanes (layer-wise sampler).
#pragma once
#include "philox.hpp"
#include "wave.hpp"

namespace gnn {

template <typename RP>
__device__ __forceinline__ void row_range(const RP* rowptr, int32_t v, int64_t& start, int64_t& deg) {
  start = (int64_t)rowptr[v];
  deg = (int64_t)rowptr[v + 1] - start;
}

// The whole wave samples node v (valid id) at hop `hop`: k = min(fanout, d)
// neighbours.  On return, lane `rank` (rank < k) holds the rank-th chosen
// neighbour in ascending CSR position order in *nbr; the function returns k.
// If d <= fanout all neighbours are taken and no random number is drawn;
// otherwise Floyd's algorithm picks k distinct positions: step s draws t_s
// uniform in [0, j_s], j_s = d - k + s (draw s of Philox4x64-10 at counter
// (1 + s/4, v, hop, 0), key (rng_key, 0)), and keeps t_s unless an earlier
// step chose it, in which case it keeps j_s.  Must be called by all 64 lanes
// (fanout <= 64).
template <typename RP>
__device__ __forceinline__ int32_t wave_sample(const RP* __restrict__ rowptr,
                                               const int32_t* __restrict__ col, int32_t v,
                                               int32_t fanout, uint64_t rng_key, uint32_t hop,
                                               int32_t* nbr) {
  const int lane = lane_id();
  int64_t start, d;
  row_range(rowptr, v, start, d);
  if (d <= fanout) {
    *nbr = lane < d ? col[start + lane] : -1;
    return (int32_t)d;
  }
  const uint32_t du = (uint32_t)d;
  const uint32_t f = (uint32_t)fanout;
  uint32_t t = 0;
  if ((uint32_t)lane < f) {
    const uint64_t r = sample_draw(rng_key, hop, (uint32_t)v, (uint32_t)lane);
    t = bounded_draw(r, du - f + (uint32_t)lane + 1u);
  }
  int32_t pick = -1;
  for (uint32_t s = 0; s < f; ++s) {
    const int32_t ts = read_lane((int32_t)t, (int)s);
    const bool dup = ballot((uint32_t)lane < s && pick == ts) != 0ull;
    const int32_t chosen = dup ? (int32_t)(du - f + s) : ts;
    if ((uint32_t)lane == s) pick = chosen;
  }
  // rank of each pick among the f distinct picks -> ascending position order
  int32_t rank = 0;
  for (uint32_t m = 0; m < f; ++m) {
    const int32_t pm = read_lane(pick, (int)m);
    rank += (pm < pick) ? 1 : 0;
  }
  // move pick of rank r to lane r
  const int32_t w = (uint32_t)lane < f ? col[start + pick] : -1;
  int32_t src_lane = 0;
  for (uint32_t m = 0; m < f; ++m) {
    const int32_t rm = read_lane(rank, (int)m);
    if (rm == lane) src_lane = (int32_t)m;
  }
  const int32_t moved = __shfl(w, src_lane, 64);
  *nbr = (uint32_t)lane < f ? moved : -1;
  return (int32_t)f;
}

// x of lane J of the caller's group of P lanes (P = 1, 2, 4, 8 or 16 lanes of
// a DPP row of 16; every lane of the wave must be active): one VALU move, two
// and a select for P = 8, where a lane read through LDS costs ~100 cycles.
template <int P, int J>
__device__ __forceinline__ uint32_t group_bcast(uint32_t x) {
  static_assert(J < P, "lane of the group");
  if constexpr (P == 1) {
    return x;
  } else if constexpr (P == 2) {
    constexpr int kPerm = J | (J << 2) | ((2 + J) << 4) | ((2 + J) << 6);  // quad_perm
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kPerm, 0xF, 0xF, false);
  } else if constexpr (P == 4) {
    constexpr int kPerm = J | (J << 2) | (J << 4) | (J << 6);
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, kPerm, 0xF, 0xF, false);
  } else if constexpr (P == 8) {
    constexpr int kBcast = 0x150;  // row_newbcast
    const int lo = __builtin_amdgcn_update_dpp(0, (int)x, kBcast + J, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)x, kBcast + 8 + J, 0xF, 0xF, false);
    return (uint32_t)((lane_id() & 8) ? hi : lo);
  } else {
    static_assert(P == 16, "group size");
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x150 + J, 0xF, 0xF, false);
  }
}

// Node sampling for the layer-wise sampler: a group of P lanes (P a power of
// two, 4 P >= fanout) samples node v, so a wave samples 64 / P nodes at once.
// Lane j of the group owns draws 4 j .. 4 j + 3, the four words of one Philox
// block (with a lane per draw, three of four lanes recomputed their
// neighbour's block).
// On return pos[e] and rank[e] (draw s = 4 j + e < k) are a chosen CSR
// position and its rank among the row's k = min(fanout, d) chosen positions;
// the function returns k (0 for valid == false).  The fanout must be the same
// for the whole wave, and every lane of the wave must call it.
template <int P>
struct GroupPick {
  static constexpr uint32_t kNone = 0xFFFFFFFFu;  // no position: larger than any, equal to none
  uint32_t t[4];     // this lane's draws
  uint32_t pick[4];  // its chosen positions
  int32_t below[4];  // picks of the group below each
  uint64_t gmask;    // the group's lanes
  uint32_t first;    // du - f: step s may draw positions up to first + s
  int j;

  // Floyd, steps 4 J .. : step s keeps t_s unless an earlier step of the group chose it
  template <int J>
  __device__ __forceinline__ void choose(uint32_t f) {
    if constexpr (J < P) {
      if (4 * J < f) {  // (uniform)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t s = 4 * J + e;
          const uint32_t ts = group_bcast<P, J>(t[e]);
          bool dup = pick[0] == ts || pick[1] == ts || pick[2] == ts || pick[3] == ts;
          if (P > 1) dup = (ballot(dup) & gmask) != 0ull;
          if (j == J && s < f) pick[e] = dup ? first + s : ts;
        }
        choose<J + 1>(f);
      }
    }
  }
  template <int J>
  __device__ __forceinline__ void count(uint32_t f) {
    if constexpr (J < P) {
      if (4 * J < f) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t pm = group_bcast<P, J>(pick[e]);  // (kNone past the fanout: below none)
#pragma unroll
          for (int i = 0; i < 4; ++i) below[i] += pm < pick[i] ? 1 : 0;
        }
        count<J + 1>(f);
      }
    }
  }
};

template <int P>
__device__ __forceinline__ int32_t group_pick(bool valid, int64_t d, int32_t v, int32_t fanout,
                                              uint64_t rng_key, uint32_t hop, uint32_t (&pos)[4],
                                              int32_t (&rank)[4]) {
  static_assert(P >= 1 && P <= 16 && (P & (P - 1)) == 0, "group size");
  const int lane = lane_id();
  const int j = lane & (P - 1), g0 = lane - j;
  const uint32_t f = (uint32_t)fanout;
  const bool all = !valid || d <= fanout;
  const uint32_t du = (uint32_t)d;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    pos[e] = 4u * j + e;  // every neighbour: position s, rank s
    rank[e] = 4 * j + e;
  }
  if (ballot(!all) != 0ull) {  // (uniform)
    GroupPick<P> g;
    g.j = j;
    g.first = du - f;
    g.gmask = ((1ull << P) - 1ull) << g0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      g.t[e] = g.pick[e] = GroupPick<P>::kNone;
      g.below[e] = 0;
    }
    if (!all && 4u * j < f) {
      const U64x4 y = philox4x64_10(1ull + j, (uint32_t)v, hop, 0ull, rng_key, 0ull);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (4u * j + e < f) g.t[e] = bounded_draw(y.x[e], du - f + 4u * j + e + 1u);
    }
    g.template choose<0>(f);
    g.template count<0>(f);
    if (!all) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        pos[e] = g.pick[e];
        rank[e] = g.below[e];
      }
    }
  }
  return !valid ? 0 : (all ? (int32_t)d : fanout);
}

}  // namespace gnn

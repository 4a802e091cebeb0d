// fp32 products on the bf16 matrix units, for the long operands of gemm.hip
// (included there: it uses its Operand, Out and GemmArgs).
//
// v_mfma_f32_16x16x4_f32 does 64 flops per cycle and SIMD, the bf16 MFMA 1,024.
// An fp32 value is the exact sum of three bf16 values (h = x to nearest even,
// m = x - h to nearest even, l the rest: 3 x 8 bits, the signs make up for the
// rounding), so a b = ah bh + (ah bm + am bh) + (am bm + ah bl + al bh) + terms
// of at most 2^-26 |a b|: six bf16 MFMAs (exact products, fp32 sums) in place of
// eight fp32 ones of twice the cycles.  Against 64 bits the forward and the
// input gradient are closer than with fp32 MFMAs (3.3e-7 against 4.1e-7 over
// 512 products, 2.3e-7 against 2.7e-7 over 256: fewer roundings of the sum), and
// so is the weight gradient with its chunks of rows (9.1e-7 against 1.0e-6 over
// 108K rows in 64 chunks).  Values below ~2^-110 keep fewer bits (their last
// part is subnormal in bf16).  A tile with an infinite or NaN sum -- an operand
// that was, or one that only its rounding to bf16 made infinite -- is done again
// with fp32 arithmetic.
//
// What bounds it: not the MFMAs (1,536 cycles of a 128 x 128 x 32 slab; a
// sixth of them takes 62% of the time) but splitting, LDS and loads around
// them, so the values are split once per workgroup as they are staged, in the
// order the MFMAs read them (conflict-free 16-byte LDS accesses both ways), and
// two or three workgroups share a CU.  Blocks take tiles (and chunks) in a
// loop over the live counts.  108,459 x 512 x 256 (measured on their own, against
// the 64 x 64 fp32 tiles): forward 301 -> 221-243 us, input gradient 317 -> 273,
// weight gradient 300 -> 175; 95,782 x 200 x 128 forward 67 -> 49; 45,354 x 100 x
// 256 44 -> 35.  Up to ~20K rows the fp32 tiles are as fast or faster: more,
// smaller tiles.
#pragma once

typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

constexpr int kSplitBK = 32;     // k of a slab: one 16x16x32 MFMA
constexpr int kSplitFrag = 192;  // 16-byte LDS slots of a fragment: 64 lanes of h, m and l

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(floatx2{a, b}, bf16x2));  // nearest even
}

// eight fp32 values as three groups of eight bf16 values
__device__ __forceinline__ void split8(const float (&x)[8], uint4& h, uint4& m, uint4& l) {
  uint32_t ph[4], pm[4], pl[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    float a = x[2 * i], b = x[2 * i + 1];
    ph[i] = pack_bf16(a, b);
    a -= __uint_as_float(ph[i] << 16);
    b -= __uint_as_float(ph[i] & 0xFFFF0000u);
    pm[i] = pack_bf16(a, b);
    a -= __uint_as_float(pm[i] << 16);
    b -= __uint_as_float(pm[i] & 0xFFFF0000u);
    pl[i] = pack_bf16(a, b);
  }
  h = make_uint4(ph[0], ph[1], ph[2], ph[3]);
  m = make_uint4(pm[0], pm[1], pm[2], pm[3]);
  l = make_uint4(pl[0], pl[1], pl[2], pl[3]);
}

// Staging of one operand: ROWS rows (of A, or columns of B) by a slab.  A unit
// is eight k values of one row, an MFMA lane's; unit u of thread t.  KC: k is
// the contiguous axis (VEC: 16-byte loads), a wave's units are 16 rows by the
// slab; else the rows are, and a wave's loads are 64 consecutive rows of one k.
template <bool KC, bool VEC, bool MASK, int ROWS>
struct SplitStage {
  static constexpr int U = ROWS * 4 / kThreads;
  static_assert(U >= 1, "rows of a tile");
  const float* p;
  const float* mask;
  int64_t ld, r0;
  int32_t lim;  // rows of the operand
  uint32_t off[U];  // byte offset from the tile's origin (kOob for a row past lim)

  __device__ __forceinline__ static int unit_row(int t) { return KC ? (t & 15) | ((t >> 6) << 4) : t % ROWS; }
  __device__ __forceinline__ static int unit_k(int t) { return 8 * (KC ? (t >> 4) & 3 : t / ROWS); }

  __device__ __forceinline__ SplitStage(const Operand& o, int64_t row0, int32_t rows)
      : p(static_cast<const float*>(o.p)), mask(o.mask), ld(o.ld), r0(row0), lim(rows) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int t = threadIdx.x + kThreads * u, row = unit_row(t), k = unit_k(t);
      off[u] = r0 + row < lim ? (uint32_t)((KC ? row * ld + k : k * ld + row) * 4) : kOob;
    }
  }
  __device__ __forceinline__ static int slot(int u) {
    const int t = threadIdx.x + kThreads * u, row = unit_row(t);
    return (row >> 4) * kSplitFrag + unit_k(t) * 2 + (row & 15);
  }
  // k values k0 .. k0 + 31 (those at or past kend read as 0)
  __device__ __forceinline__ void load(int64_t k0, int64_t kend, float (&x)[U][8]) const {
    const int64_t o = KC ? r0 * ld + k0 : k0 * ld + r0;
    // the operand from the slab's origin on: its last row, or k, ends the range
    const int64_t n = k0 >= kend ? o : o + (KC ? (lim - 1 - r0) * ld + (kend - k0) : (kend - 1 - k0) * ld + (lim - r0));
    const __amdgpu_buffer_rsrc_t r = rsrc_from<4>(p, n, o);
    const __amdgpu_buffer_rsrc_t rm = MASK ? rsrc_from<4>(mask, n, o) : r;
    auto one = [](__amdgpu_buffer_rsrc_t b, uint32_t a) {
      return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(b, a, 0, 0));
    };
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t k = k0 + unit_k(threadIdx.x + kThreads * u);
      if constexpr (KC && VEC) {
#pragma unroll
        for (int h = 0; h < 2; ++h) {
          const uint32_t a = k + 4 * h < kend ? off[u] + 16 * h : kOob;
          const auto v = __builtin_amdgcn_raw_buffer_load_b128(r, a, 0, 0);
#pragma unroll
          for (int e = 0; e < 4; ++e) x[u][4 * h + e] = __uint_as_float(v[e]);
          if constexpr (MASK) {
            const auto w = __builtin_amdgcn_raw_buffer_load_b128(rm, a, 0, 0);
#pragma unroll
            for (int e = 0; e < 4; ++e)
              x[u][4 * h + e] = __uint_as_float(w[e]) > 0.f ? x[u][4 * h + e] : 0.f;
          }
        }
      } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          const uint32_t a = KC ? (k + e < kend ? off[u] + 4u * e : kOob)
                                : off[u] + (uint32_t)e * (uint32_t)ld * 4u;
          x[u][e] = one(r, a);
          if constexpr (MASK) x[u][e] = one(rm, a) > 0.f ? x[u][e] : 0.f;
        }
      }
    }
  }
  __device__ __forceinline__ static void store(uint4* s, const float (&x)[U][8]) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      uint4 h, m, l;
      split8(x[u], h, m, l);
      uint4* d = s + slot(u);
      d[0] = h;
      d[64] = m;
      d[128] = l;
    }
  }
  __device__ __forceinline__ float at(int64_t row, int64_t k) const {
    const int64_t o = KC ? row * ld + k : k * ld + row;
    return MASK && !(mask[o] > 0.f) ? 0.f : p[o];
  }
};

// 16-byte LDS words of a tile: the staged slab, or 64 rows of the output
template <int TM, int TN>
constexpr int split_smem() {
  constexpr int ops = (TM + TN) / 16 * kSplitFrag, out = 64 * (TN + 4) / 4;
  return ops > out ? ops : out;
}

// Block bid of nbid of a product in tiles of TM x TN (four waves of TM/2 x TN/2).
template <int FL, int TM, int TN>
__device__ __forceinline__ void split_body(const GemmArgs& ga, int32_t bid, int32_t nbid, uint4* smem) {
  constexpr bool AT = FL & kAT, BT = FL & kBT, AV = FL & kAV, BV = FL & kBV, AM = FL & kAM, BMk = FL & kBM;
  constexpr int FM = TM / 32, FN = TN / 32;  // 16 x 16 MFMA tiles of a wave
  constexpr int AW = TM / 16 * kSplitFrag;
  using StA = SplitStage<!AT, AV, AM, TM>;
  using StB = SplitStage<BT, BV, BMk, TN>;
  if (bid >= ga.gemm_blocks) {
    side_jobs(ga, bid, nbid);
    return;
  }
  int32_t M = ga.m_cap, K = ga.k_cap;
  const int32_t N = ga.N;
  if (ga.m_dev) M = min(M, *ga.m_dev);
  if (ga.k_dev) K = min(K, *ga.k_dev);
  const int gm = (M + TM - 1) / TM, gn = (N + TN - 1) / TN, tiles = gm * gn;
  if (tiles == 0) return;
  // Units of work, unit u on XCD u % 8 as in gemm_body: without splits the
  // column tiles of one row tile, with splits the tiles of one chunk of k
  // are consecutive units of an XCD.
  int parts = 1, chunk = K;
  int64_t units = (int64_t)((gm + kXcds - 1) / kXcds) * kXcds * gn;
  if (ga.nsplit > 1) {
    // about one unit per block, in chunks of at least min_chunk
    parts = min((ga.gemm_blocks + tiles - 1) / tiles, (K + ga.min_chunk - 1) / ga.min_chunk);
    parts = max(1, min(parts, ga.nsplit));
    if (parts > kXcds) parts -= parts % kXcds;
    chunk = ((K + parts - 1) / parts + kSplitBK - 1) / kSplitBK * kSplitBK;
    units = (int64_t)((parts + kXcds - 1) / kXcds) * kXcds * tiles;
  }
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = (wave >> 1) * FM, wn = (wave & 1) * FN;  // the wave's first fragments
  for (int64_t un = bid; un < units; un += ga.gemm_blocks) {
    const int xcd = (int)(un % kXcds);
    const int64_t idx = un / kXcds;
    int64_t mt = (idx / gn) * kXcds + xcd, nt = idx % gn;
    int32_t kbeg = 0, kend = K;
    if (ga.nsplit > 1) {
      const int z = (int)(idx / tiles) * kXcds + xcd;
      mt = (idx % tiles) / gn;
      nt = (idx % tiles) % gn;
      kbeg = z * chunk;
      kend = min(K, kbeg + chunk);
      if (z >= parts || kbeg >= kend) continue;
    }
    const int64_t m0 = mt * TM, n0 = nt * TN;
    if (m0 >= M) continue;
    const StA sa(ga.A, m0, M);
    const StB sb(ga.B, n0, N);
    floatx4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    // one LDS buffer: the registers of slab kt are free once it is staged and
    // take the loads of slab kt + 1
    float ra[StA::U][8], rb[StB::U][8];
    const int nk = (kend - kbeg + kSplitBK - 1) / kSplitBK;
    sa.load(kbeg, kend, ra);
    sb.load(kbeg, kend, rb);
    for (int kt = 0; kt < nk; ++kt) {
      StA::store(smem, ra);
      StB::store(smem + AW, rb);
      const int64_t k1 = kbeg + (int64_t)(kt + 1) * kSplitBK;
      sa.load(k1, kend, ra);
      sb.load(k1, kend, rb);
      __syncthreads();
      bf16x8 a[FM][3], b[FN][3];
#pragma unroll
      for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int q = 0; q < 3; ++q)
          a[i][q] = __builtin_bit_cast(bf16x8, smem[(wm + i) * kSplitFrag + q * 64 + lane]);
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int q = 0; q < 3; ++q)
          b[j][q] = __builtin_bit_cast(bf16x8, smem[AW + (wn + j) * kSplitFrag + q * 64 + lane]);
      constexpr int qa[6] = {2, 0, 1, 1, 0, 0}, qb[6] = {0, 2, 1, 0, 1, 0};  // small terms first
#pragma unroll
      for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i][qa[t]], b[j][qb[t]], acc[i][j], 0, 0, 0);
      __syncthreads();
    }
    bool bad = false;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) bad |= !(__builtin_fabsf(acc[i][j][r]) < __builtin_huge_valf());
    if (__syncthreads_or(bad)) {
      for (int q = tid; q < TM * TN; q += kThreads) {
        const int64_t i = m0 + q / TN, j = n0 + q % TN;
        if (i >= M || j >= N) continue;
        float x = 0.f;
        for (int64_t k = kbeg; k < kend; ++k) x = fmaf(sa.at(i, k), sb.at(j, k), x);
        out_store(ga.C, i, j, x, ga.epilogue);
      }
      continue;
    }
    // 64 rows of the tile at a time through LDS, for whole row pieces
    constexpr int TS = TN + 4;
    float* T = reinterpret_cast<float*>(smem);
    const int g = lane >> 4, c16 = lane & 15;
#pragma unroll
    for (int half = 0; half < TM / 64; ++half) {
      if ((wave >> 1) == half) {
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float x = acc[i][j][r];
              T[(16 * i + 4 * g + r) * TS + (wn + j) * 16 + c16] = ga.epilogue == 1 ? fmaxf(x, 0.f) : x;
            }
      }
      __syncthreads();
      const int64_t mh = m0 + 64 * half;
      if (ga.epilogue == 2) {
        for (int q = tid; q < 64 * TN; q += kThreads) {
          const int64_t i = mh + q / TN, j = n0 + q % TN;
          if (i < M && j < N) out_store(ga.C, i, j, T[(q / TN) * TS + q % TN], 2);
        }
      } else {
        for (int q = tid; q < 64 * TN / 4; q += kThreads) {
          const int row = q / (TN / 4), c4 = q % (TN / 4);
          const int64_t i = mh + row, j = n0 + 4 * c4;
          if (i < M && j < N) out_store4(ga.C, i, j, *reinterpret_cast<const float4*>(&T[row * TS + 4 * c4]), N);
        }
      }
      __syncthreads();
    }
  }
}

// forward and input-gradient products: 128 x 64 tiles, three workgroups per CU
template <int FL>
__global__ void __launch_bounds__(kThreads, (FL & (kAM | kBM)) ? 2 : 3) split_kernel(GemmArgs ga) {
  __shared__ uint4 smem[split_smem<128, 64>()];
  split_body<FL, 128, 64>(ga, (int32_t)blockIdx.x, (int32_t)gridDim.x, smem);
}
// weight gradients: 128 x 128 tiles (longer rows of atomics, half the splitting
// per product), two workgroups per CU
template <int FL>
__global__ void __launch_bounds__(kThreads, 2) split_dw_kernel(GemmArgs ga) {
  __shared__ uint4 smem[split_smem<128, 128>()];
  split_body<FL, 128, 128>(ga, (int32_t)blockIdx.x, (int32_t)gridDim.x, smem);
}
// both of a layer in one grid (as gemm_pair_kernel)
template <int FL1, int FL2>
__global__ void __launch_bounds__(kThreads, 2) split_pair_kernel(GemmArgs g1, GemmArgs g2, int32_t part1) {
  __shared__ uint4 smem[split_smem<128, 128>()];
  const int32_t b = (int32_t)blockIdx.x;
  if (b < part1) split_body<FL1, 128, 128>(g1, b, part1, smem);
  else split_body<FL2, 128, 128>(g2, b - part1, (int32_t)gridDim.x - part1, smem);
}

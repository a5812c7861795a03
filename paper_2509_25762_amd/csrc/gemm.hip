// gfx950 kernels: the layer's fused QKV projection with the rotary embedding and the
// cache write as its epilogue.
//
//   y[m, n] = sum_k x[m, k] * w[n, k]     x: bf16 [rows][hidden], w: bf16 [(Hq + 2 Hkv) D][hidden]
//
// (both operands contiguous along k, fp32 accumulation), and then, per output row m at
// absolute position p and per head: query and key heads are rotated pair by pair
// ((t, t + D/2), angle p * base^(-2t/D): RoFormer Sec. 3.2 / 3.4.2 in the half-split pairing),
// rounded once to bf16 and written to q_out / to the sequence's cache slab; value heads go
// to the cache as they are.  The projection's output never exists in memory.
//
// Workgroup = 256 columns of y by 256, 192, 128 or 64 rows, 8 waves (two per SIMD).
// Tall tiles have a kernel of their own (qkv_proj_phased_kernel, below, v_mfma_f32_16x16x32_bf16);
// passes too thin to give every compute unit such a tile, and short k loops, take qkv_proj_kernel (v_mfma_f32_32x32x16_bf16) with 256, 128 or
// 64 rows (plan_qkv_proj chooses): k advances in tiles of 64 through a ring of LDS stages, one workgroup per compute
// unit; tiles travel global -> LDS directly, the
// XOR swizzle of the LDS rows applied by choosing which 16-byte granule each lane fetches, so
// the fragment reads (ds_read_b128, one row per lane) spread over the banks.  The epilogue
// parks the fp32 tile in the same LDS, 64 rows at a time, from where threads take 8-column pieces of a row and
// their partners D/2 columns further on, rotate them with the (cos, sin) table a small kernel
// made beforehand for the pass's rows, and store 16 bytes at a time.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "oppo_internal.h"

namespace oppo {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kGemmBN = kProjTileCols, kGemmBK = 64;   // the tile's rows BM are chosen per launch
constexpr int kMaxProjItems = 1000;   // 1000 * 24 B + header in the kernel arguments
constexpr int kFewProjItems = 64;     // the short list (see kFewAttnItems): 64 sequences 15.2 us a call, 65 16.4

// Per-row data of a pass, made by proj_rows_kernel in the caller's workspace:
//   dst[rows]            int64  cache row (token slot) the row's keys and values go to
//   cs[rows][D/2]        float2 (cos, sin) of position * base^(-2t/D)
template <int NI>
struct ProjRowsParams {
  int64_t* dst;
  float2* cs;
  double log2_base;
  int32_t half;      // D / 2
  int32_t n_items;
  QkvItem items[NI];
};
static_assert(sizeof(ProjRowsParams<kMaxProjItems>) <= 32768, "kernel arguments are kept within 32 KiB");

// grid = (items, pieces of (256 / half) * RUN tokens); 256 threads.  Angles in double precision (they reach
// tens of thousands of radians for the fastest pair), kept as fp32.  Bound by the double-precision sines: a thread takes
// RUN consecutive tokens of one pair, forms sine and cosine of the first one's angle and of the pair's step, and turns
// the one by the other (some 1e-16 of error a turn, far below the rounding to fp32).  With a sine per token 14,000 rows of
// chunks of 64, hidden 704, took 230 us a layer pass, with runs of 2, 4, 8 225.4, 224.9, 224.0; thin passes (hidden 4096)
// 134.9, 134.1, 134.6, 135.1.  Up to an angle per thread of two full waves on every SIMD (kOneByOne) it is the length of one
// thread's work that counts, and each angle has its own sine: against runs of 4 -0.2 us for 1 .. 64 rows, -0.3 for 513 .. 1024
// (passes of 5 .. 9 us); heads of 128, 1025 .. 2048 rows -0.2 and 2049 .. 4096 rows +0.3, heads of 64 -0.25 and -0.04, 4097 .. 8192 rows
// +0.2, 16,385 .. 40,000 +2.4.
constexpr int kRowsRun = 4;
constexpr int64_t kOneByOne = 256 * 4 * 2 * 64;
template <int NI, int RUN>
__global__ __launch_bounds__(256) void proj_rows_kernel(const ProjRowsParams<NI> P) {
  const QkvItem it = P.items[blockIdx.x];
  const int tok0 = (blockIdx.y * (256 / P.half) + threadIdx.x / P.half) * RUN;
  const int ntok = min(RUN, it.n_tok - tok0);
  if (ntok <= 0) return;
  const int i = threadIdx.x % P.half;
  const int64_t row = (int64_t)it.src_row + tok0;
  const double theta = exp2(-(double)i / P.half * P.log2_base);
  double s, c, st = 0.0, ct = 1.0;
  sincos((double)(it.pos0 + tok0) * theta, &s, &c);
  if (RUN > 1) sincos(theta, &st, &ct);
#pragma unroll
  for (int t = 0; t < RUN; ++t) {
    if (t < ntok) {
      P.cs[(row + t) * P.half + i] = make_float2((float)c, (float)s);
      if (i == 0) P.dst[row + t] = it.dst_row + tok0 + t;
    }
    const double c1 = c * ct - s * st;
    s = s * ct + c * st;
    c = c1;
  }
}

struct ProjParams {
  const uint16_t* x;     // [rows][hidden]
  const uint16_t* w;     // [n_out][hidden]
  uint16_t* q_out;       // [rows][Hq][D]
  uint16_t* cache_k;     // [slots][Hkv][D]
  uint16_t* cache_v;
  const int64_t* dst;    // [rows]
  const float2* cs;      // [rows][D/2]
  int32_t rows, hidden, n_out;
  int32_t Hq, Hkv;
};

// 16 bytes per lane, global -> LDS: lane l reads gbase[voff_bytes .. +16), the data lands at
// lds_addr + 16 * l (gbase and lds_addr wave-uniform).  See the same helper of the attention
// kernel for why it is written as assembly and why M0 is not on a clobber list.
__device__ __forceinline__ void gemm_async_copy16(const void* gbase, uint32_t voff_bytes, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds_addr), "v"(voff_bytes), "s"(gbase) : "memory");
}

__device__ __forceinline__ uint32_t gemm_pack_bf16(float a, float b) {
  bf16x2 p;
  p[0] = (__bf16)a;   // round to nearest even
  p[1] = (__bf16)b;
  return *(uint32_t*)&p;
}

// Which tile the workgroup with number `block` takes.  Workgroups are dealt round-robin to the
// chip's 8 XCDs, each with a level-2 cache of its own.  The tiles are laid out as blocks of 8 row
// tiles x 4 column tiles, one after the other (those at the edges are smaller); a round of 256
// workgroups takes the next 256 of that list, each XCD 32 consecutive ones: they stream through
// k together, so every slice of a block's row tiles and column tiles is fetched into that cache
// once and serves 4 resp. 8 workgroups.  The list has no gaps, so a pass of up to 256 tiles is
// one round whatever its number of row tiles, and the tiles of a last, smaller round are dealt
// evenly to the XCDs (all on a few of them would share those caches' bandwidth: measured 15 %
// slower at 96 tiles).
struct TileOrder {
  int m_tiles, n_tiles;
  __device__ __forceinline__ TileOrder(const ProjParams& P, int bm, int bn)
      : m_tiles((P.rows + bm - 1) / bm), n_tiles((P.n_out + bn - 1) / bn) {}
  // FEW: passes with few tiles come this way too.  A division is a tenth of a microsecond in front of the first
  // request, out of 7 for the smallest passes: those that the pass's size makes trivial are left out.
  template <bool FEW>
  __device__ __forceinline__ bool at(int block, int* tile_m, int* tile_n) const {
    const int first = block & ~255, left = m_tiles * n_tiles - first;
    const int share = left >= 256 ? 32 : (left + 7) / 8;   // an XCD's tiles of this round
    const int mine = (block / 8) % 32, in_round = (block % 8) * share + mine;
    if (mine >= share || in_round >= left) return false;
    const int pos = first + in_round;
    if (FEW && m_tiles == 1) {
      *tile_m = 0;
      *tile_n = pos;
      return true;
    }
    const int strip = FEW && n_tiles <= 4 ? 0 : pos / (4 * m_tiles), in_strip = pos - 4 * m_tiles * strip;   // strips of 4 column tiles
    const int width = min(4, n_tiles - 4 * strip);
    const int mg = FEW && m_tiles <= 8 ? 0 : in_strip / (8 * width), in_group = in_strip - 8 * width * mg;
    const int height = min(8, m_tiles - 8 * mg);
    const int across = FEW && height == 8 ? in_group >> 3 : in_group / height;
    *tile_m = 8 * mg + in_group - height * across;
    *tile_n = 4 * strip + across;
    return true;
  }
};

// Elements 8 g .. of the first half of a head's row (a0, a1) and their partners D / 2 further on
// (b0, b1): rotated (query and key heads), rounded, and stored to q_out or to the row's cache slot.
template <int D>
__device__ __forceinline__ void store_piece(const ProjParams& P, int64_t row, int head, int g, f32x4 a0, f32x4 a1, f32x4 b0,
                                            f32x4 b1) {
  constexpr int HALF = D / 2;
  const float av[8] = {a0[0], a0[1], a0[2], a0[3], a1[0], a1[1], a1[2], a1[3]};
  const float bv[8] = {b0[0], b0[1], b0[2], b0[3], b1[0], b1[1], b1[2], b1[3]};
  uint16_t* dst;
  u32x4 ra, rb;
  if (head >= P.Hq + P.Hkv) {   // a value head: as it is
    dst = P.cache_v + (P.dst[row] * P.Hkv + (head - P.Hq - P.Hkv)) * D;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      ra[w] = gemm_pack_bf16(av[2 * w], av[2 * w + 1]);
      rb[w] = gemm_pack_bf16(bv[2 * w], bv[2 * w + 1]);
    }
  } else {
    dst = head < P.Hq ? P.q_out + (row * P.Hq + head) * D : P.cache_k + (P.dst[row] * P.Hkv + (head - P.Hq)) * D;
    const float2* cs = P.cs + row * HALF + g * 8;
    float ca[8], sa[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const float2 v = cs[e];
      ca[e] = v.x;
      sa[e] = v.y;
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const int e = 2 * w;
      ra[w] = gemm_pack_bf16(av[e] * ca[e] - bv[e] * sa[e], av[e + 1] * ca[e + 1] - bv[e + 1] * sa[e + 1]);
      rb[w] = gemm_pack_bf16(bv[e] * ca[e] + av[e] * sa[e], bv[e + 1] * ca[e + 1] + av[e + 1] * sa[e + 1]);
    }
  }
  *(u32x4*)(dst + g * 8) = ra;
  *(u32x4*)(dst + HALF + g * 8) = rb;
}

template <int D, int BM>
__global__ __launch_bounds__(512) void qkv_proj_kernel(const ProjParams P) {
  constexpr int BN = kGemmBN, BK = kGemmBK;
  constexpr int ROWB = BK * 2;            // bytes of a tile row in LDS (128)
  constexpr int NGR = ROWB / 16;          // 16-byte granules per row (8)
  constexpr int RPL = 1024 / ROWB;        // rows one wave-wide copy covers (8)
  constexpr int TILE_A = BM * ROWB;       // bytes of an x tile (32, 16 or 8 KiB)
  constexpr int TILE_B = BN * ROWB;       // bytes of a w tile (32 KiB)
  constexpr int STAGE = TILE_A + TILE_B;
  constexpr int WR = BM == 256 ? 4 : 2, WC = 8 / WR;   // waves down and across the tile
  constexpr int MI = BM / WR / 32, NJ = BN / WC / 32;  // 32 x 32 blocks of a wave: 2 x 4, 2 x 2 or 1 x 2
  constexpr int CA = BM / RPL / 8, CB = BN / RPL / 8;  // copies per wave and tile: x (4, 2 or 1), w (4)
  static_assert(BN == 256 && BK == 64 && (BM == 256 || BM == 128 || BM == 64), "8 waves, k tiles of 64");
  // stages of the tile ring: two tiles of 256 rows fill the LDS; the smaller tiles run on passes
  // whose k loop is bound by the tiles' latency, and keep two tiles in flight instead of one
  constexpr int NST = BM == 256 ? 2 : 3;   // (four stages of the 64-row tile: measured, no faster)
  static_assert(NST * STAGE >= 64 * BN * 4 && NST * STAGE <= 160 * 1024, "ring and the epilogue's 64 x 256 fp32 strip fit the LDS");
  // [stage][x tile | w tile]; the epilogue reuses it as a 64 x 256 fp32 strip at a time
  __shared__ __attribute__((aligned(1024))) unsigned char smem[NST * STAGE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l32 = lane & 31, hi = lane >> 5;
  const int wm = wave / WC, wn = wave % WC;    // the wave's (32 MI) x (32 NJ) part of the tile
  const TileOrder order(P, BM, BN);
  int tile_m, tile_n;
  if (!order.at<true>((int)blockIdx.x, &tile_m, &tile_n)) return;
  const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;

  // ---- loads: a wave-wide copy moves 8 rows (8 x 128 B); wave w moves rows 8 (w + 8 i) .. of
  // x (i < CA) and of w (i < CB).  A row's eight granules are swizzled by (row / 2) % 8, so that
  // sixteen consecutive rows cover all sixteen 16-byte bank groups.  Rows past the end of x / w
  // repeat the last valid row (their products are never stored).
  const int lrow = lane / NGR, pg = lane % NGR;
  uint32_t offa[CA], offb[CB];
#pragma unroll
  for (int i = 0; i < CB; ++i) {
    const int r = RPL * (wave + 8 * i) + lrow;
    const int64_t ra = min(m0 + r, (int64_t)P.rows - 1) - m0, rb = min(n0 + r, (int64_t)P.n_out - 1) - n0;
    if (i < CA) offa[i] = (uint32_t)(ra * P.hidden + ((pg ^ ((r >> 1) % NGR)) * 8)) * 2u;
    offb[i] = (uint32_t)(rb * P.hidden + ((pg ^ ((r >> 1) % NGR)) * 8)) * 2u;
  }
  const uint16_t* xa = P.x + m0 * P.hidden;
  const uint16_t* wb = P.w + n0 * P.hidden;
  const uint32_t smem0 = (uint32_t)(uintptr_t)((const __attribute__((address_space(3))) unsigned char*)smem);
  const uint32_t wave_u = (uint32_t)__builtin_amdgcn_readfirstlane(wave);
  auto issue = [&](int kt, int stage) __attribute__((always_inline)) {
    const uint16_t* ga = xa + (int64_t)kt * BK;
    const uint16_t* gb = wb + (int64_t)kt * BK;
#pragma unroll
    for (int i = 0; i < CB; ++i) {
      const uint32_t dst = smem0 + (uint32_t)stage * (uint32_t)STAGE + (wave_u + 8u * i) * 1024u;
      if (i < CA) gemm_async_copy16(ga, offa[i], dst);
      gemm_async_copy16(gb, offb[i], dst + TILE_A);
    }
  };
  auto barrier = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // ---- fragments: lane (l32, hi) reads row (block * 32 + l32), elements k = 16 kk + 8 hi ..;
  // per-lane base addresses (the swizzle (row / 2) % 8 is (l32 / 2) % 8 for every block), stage
  // and k-step folded in as immediates / XORs
  typedef const __attribute__((address_space(3))) unsigned char* lds_cptr;
  const uint32_t a_base = smem0 + (uint32_t)((wm * 32 * MI + l32) * ROWB);
  const uint32_t b_base = smem0 + TILE_A + (uint32_t)((wn * 32 * NJ + l32) * ROWB);
  const uint32_t swz = (uint32_t)((l32 >> 1) % NGR);
  auto frag = [&](uint32_t base, int stage, int block, int kk) __attribute__((always_inline)) -> bf16x8 {
    const uint32_t a = base + (uint32_t)stage * (uint32_t)STAGE + (uint32_t)(block * 32 * ROWB) + ((((uint32_t)(kk * 2 + hi)) ^ swz) * 16u);
    return *(const __attribute__((address_space(3))) bf16x8*)(lds_cptr)(uintptr_t)a;
  };

  f32x16 acc[MI][NJ];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;

  const int KT = P.hidden / BK;
  // one tile's 4 k-steps out of ring stage st
  auto compute = [&](int st) __attribute__((always_inline)) {
    bf16x8 a[2][MI], b[2][NJ];   // fragments of k-step kk in [kk & 1]: read one step ahead of their MFMAs
#pragma unroll
    for (int i = 0; i < MI; ++i) a[0][i] = frag(a_base, st, i, 0);
#pragma unroll
    for (int j = 0; j < NJ; ++j) b[0][j] = frag(b_base, st, j, 0);
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      const int c = kk & 1;
      if (kk + 1 < BK / 16) {
#pragma unroll
        for (int i = 0; i < MI; ++i) a[c ^ 1][i] = frag(a_base, st, i, kk + 1);
#pragma unroll
        for (int j = 0; j < NJ; ++j) b[c ^ 1][j] = frag(b_base, st, j, kk + 1);
      }
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NJ; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[c][i], b[c][j], acc[i][j], 0, 0, 0);
    }
  };
  if constexpr (NST == 2) {
    // the next tile is requested in front of this tile's MFMAs (behind the barrier instead: 2-4 % slower)
    issue(0, 0);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0)
    barrier();
    for (int kt = 0; kt < KT; ++kt) {
      const int st = kt & 1;
      if (kt + 1 < KT) issue(kt + 1, st ^ 1);
      compute(st);
      // this wave's share of the next tile is in LDS, and its fragment reads are through with this tile's stage, which
      // the copies requested behind the barrier overwrite (the compiler sinks the last MFMAs below the barrier)
      __builtin_amdgcn_s_waitcnt(0x0070);   // vmcnt(0), lgkmcnt(0)
      barrier();
    }
  } else {
    // tile t lives in stage t % NST; tile kt + 1 stays in flight while tile kt is
    // waited for, and tile kt + 2 is requested into the stage of tile kt - 1 once every wave
    // has passed the barrier behind that tile's MFMAs
    constexpr int CPT = CA + CB;   // copies per wave and tile
#pragma unroll
    for (int t = 0; t < NST - 1; ++t)
      if (t < KT) issue(t, t);
    int st = 0, st_in = NST - 1;
    for (int kt = 0; kt < KT; ++kt) {
      // this wave's copies of tile kt have landed: only those of the later tiles may be outstanding
      if (kt + 1 < KT)
        __builtin_amdgcn_s_waitcnt(0x0F70 | CPT);         // vmcnt(CPT)
      else
        __builtin_amdgcn_s_waitcnt(0x0F70);               // vmcnt(0)
      barrier();
      if (kt + NST - 1 < KT) issue(kt + NST - 1, st_in);
      compute(st);
      st_in = st;
      st = st + 1 == NST ? 0 : st + 1;
    }
    barrier();   // every wave is through with the ring before the epilogue reuses it
  }

  // ---- epilogue, one strip of 64 rows at a time (the waves whose blocks lie in it: one wm, or
  // both for tiles of 64 rows): the fp32 strip into LDS (row-major, 256 floats per row), then out
  // again as row pieces - an item is (row, head of the tile, group of 8 pairs)
  float* ct = (float*)smem;
  constexpr int HALF = D / 2, GPH = HALF / 8, HPT = BN / D;   // groups per head, heads per tile
  const int heads = P.Hq + 2 * P.Hkv;
  for (int strip = 0; strip < (BM + 63) / 64; ++strip) {
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      const int row0 = (wm * MI + i) * 32;   // the block's first row in the tile
      if (row0 / 64 != strip) continue;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          // register r of lane (l32, hi): row 8 (r / 4) + 4 hi + r % 4, column l32 of the 32 x 32 block
          const int m = row0 % 64 + 8 * (r >> 2) + 4 * hi + (r & 3);
          const int n = (wn * NJ + j) * 32 + l32;
          ct[m * BN + n] = acc[i][j][r];
        }
    }
    __syncthreads();
    for (int item = tid; item < 64 * HPT * GPH; item += 512) {
      const int g = item % GPH, hl = (item / GPH) % HPT, m = item / (GPH * HPT);
      const int64_t row = m0 + strip * 64 + m;
      const int head = (int)(n0 / D) + hl;
      if (row >= P.rows || head >= heads) continue;
      const float* src = ct + m * BN + hl * D + g * 8;
      const f32x4 a0 = *(const f32x4*)(src), a1 = *(const f32x4*)(src + 4);
      const f32x4 b0 = *(const f32x4*)(src + HALF), b1 = *(const f32x4*)(src + HALF + 4);
      store_piece<D>(P, row, head, g, a0, a1, b0, b1);
    }
    __syncthreads();
  }
}

// The kernel for tiles of 256 and 192 rows: the same operand tiles, another k loop and another epilogue.
// Bound by the matrix cores; what the loop above loses on this tile is the time in which both
// waves of a SIMD read fragments or request copies (a wave that issues a copy issues no MFMA).
// Here the two take turns: the waves form two groups, one wave of each SIMD in either, and run
// the same sequence of phases one barrier apart, so that one group's MFMAs always run beside the
// other group's memory instructions.  A wave computes 128 x 64, as four quadrants of 64 x 32 (two
// halves of the x tile by two of the w tile), and a phase is
//     read the fragments the quadrant still needs; request one half tile (two copies per wave);
//     barrier; the quadrant's 16 MFMAs (16x16x32); barrier
// with, for k tile t,   phase   reads              quadrant   requests
//                         0     x0                 x0 w0      x1 of tile t + 1
//                         1     w1                 x0 w1      w0 of tile t + 2
//                         2     x1                 x1 w1      x0 of tile t + 2
//                         3     w0 of tile t + 1   x1 w0      w1 of tile t + 2
// (8, 4, 8 and 4 fragments: the LDS delivers one group's eight, 32 KiB, in about the time of the
// other group's MFMAs.)  A half tile is read in one phase only and overwritten two phases later
// at the earliest: the later group waits for its reads behind the barrier that follows them, and
// the requesting group has passed the barrier after that.  A half tile has five phases to arrive:
// a wave waits for its own copies in the phase before the one that reads them, with the five
// requests made since still in flight, and the barrier that follows makes the half tile complete
// for every wave of either group.
// The MFMAs are 16x16x32 ones: the chip runs this loop against its power limit, and they take less of it than
// 32x32x16 ones (on N(0, 1) operands, MFMAs alone: 1990-2050 against 1750 TFLOP/s; this kernel, 4096 -> 6144, 13,000 rows
// back to back: 566 us against 625).
// The product is computed transposed (w rows as the A operand), so a lane owns one row of y per block, and
// the w rows are dealt to LDS rows such that it holds 8 consecutive columns of a head and, in
// the accumulators of the other w half, their rotation partners D/2 further on: rotation and
// stores (16 bytes per row and lane, the four lanes of a row side by side) need neither LDS nor barriers, and workgroups
// stay for several tiles, requesting the next tile's first operands before they store the current one.
// Tiles of 192 rows are the same with a second x half of 64 rows (M1 = 1 block of 32 rows per wave
// instead of 2); its LDS rows stay where the 128-row half has each wave row's first block.
// Measured in one run, -> 6144 columns, tiles of 256 rows in the loop of qkv_proj_kernel / here: 13,510 rows of 4480
// 618 / 531 us (1400 TFLOP/s), 6223 of 4352 330 / 289, 2477 of 4288 119 / 105, 1482 of 3968 93 / 84.  Tiles of 256 rows
// against those of 192: 1482 rows 84 / 75 us, 2477 105 / 155, 5612 of 3968 256 / 229.
// A tile's fixed cost is the price: where the k loop is short, qkv_proj_kernel is faster (plan_qkv_proj).
template <int D, int BM>
__global__ __launch_bounds__(512) void qkv_proj_phased_kernel(const ProjParams P) {
  static_assert(BM == 256 || BM == 192, "x halves of 128 and 128 or 64 rows");
  constexpr int M1 = (BM - 128) / 64, BN = kGemmBN, BK = kGemmBK;
  constexpr int ROWB = BK * 2, NGR = ROWB / 16, RPL = 1024 / ROWB;
  constexpr int HALF_TILE = 128 * ROWB;        // 16 KiB
  constexpr int TILE = 2 * HALF_TILE;          // an x or w tile
  constexpr int B_AREA = 2 * TILE;             // [x: 2 stages][w: 2 stages]: offsets within either area fit 16 bits
  __shared__ __attribute__((aligned(1024))) unsigned char smem[4 * TILE];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int l16 = lane & 15, grp = lane >> 4;
  const uint32_t wave_u = (uint32_t)__builtin_amdgcn_readfirstlane(wave);
  const int wm = (int)(wave_u >> 2), wn = (int)(wave_u & 3);   // wm is also the wave's group
  const TileOrder order(P, BM, BN);
  int tile_m, tile_n;
  int block = (int)blockIdx.x;
  if (!order.at<false>(block, &tile_m, &tile_n)) return;

  // copies: copies 2 h, 2 h + 1 of a wave belong to half h of the tile, 8 LDS rows each, swizzled
  // as in qkv_proj_kernel (a second x half of 64 rows takes one copy per wave).  LDS row 128 j + 32 wn + l
  // of w holds the column that row l % 16 of MFMA block l / 16 of wave column wn and half j stands for: row 4 g + b of
  // block c is column 8 g + 4 c + b of the wave's 32 (the registers of lane group g are then columns 8 g .. 8 g + 7), the
  // halves j are D/2 columns apart.
  // (Lane-dependent values that only matter between tiles are recomputed there from a copy of the
  // lane number that the optimiser cannot see through, instead of living in registers meanwhile.)
  auto lane_now = [&]() __attribute__((always_inline)) -> int {
    int x = lane;
    asm volatile("" : "+v"(x));
    return x;
  };
  uint32_t offa[4], offb[4];
  const uint16_t *xa, *wb;
  auto open_tile = [&]() __attribute__((always_inline)) {
    const int ln = lane_now(), lrow = ln / NGR, pg = ln % NGR;
    const int64_t m0 = (int64_t)tile_m * BM, n0 = (int64_t)tile_n * BN;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int r = RPL * ((int)wave_u + 8 * i) + lrow;
      const int col = 8 * ((r >> 2) & 3) + 4 * ((r >> 4) & 1) + (r & 3), wc = (r >> 5) & 3, j = r >> 7;
      const int n = D == 128 ? (wc >> 1) * 128 + j * 64 + (wc & 1) * 32 + col : wc * 64 + j * 32 + col;
      // rows past the end of x / w repeat the last valid row (their products are never stored)
      const int rx = i < 2 || M1 == 2 ? r : 128 + RPL * (int)wave_u + lrow;   // (32 rows per wave row: 128 + 32 wm + ..)
      const int ra = min(rx, P.rows - 1 - tile_m * BM), rb = min(n, P.n_out - 1 - tile_n * BN);
      offa[i] = ((uint32_t)ra * (uint32_t)P.hidden + (uint32_t)((pg ^ ((r >> 1) % NGR)) * 8)) * 2u;
      offb[i] = ((uint32_t)rb * (uint32_t)P.hidden + (uint32_t)((pg ^ ((r >> 1) % NGR)) * 8)) * 2u;
    }
    xa = P.x + m0 * P.hidden;
    wb = P.w + n0 * P.hidden;
  };
  const uint32_t smem0 = (uint32_t)(uintptr_t)((const __attribute__((address_space(3))) unsigned char*)smem);
  const uint32_t copy0 = smem0 + wave_u * 1024u;
  auto issue_x = [&](int kt, int stage, int h) __attribute__((always_inline)) {
    const uint32_t dst = copy0 + (uint32_t)(stage * TILE + h * HALF_TILE);
    if (h == 1 && M1 == 1) {
      gemm_async_copy16(xa + (int64_t)kt * BK, offa[2], dst + (wave_u >= 4 ? 4096u : 0u));   // LDS rows 0 .. 31 and 64 .. 95
      return;
    }
    gemm_async_copy16(xa + (int64_t)kt * BK, offa[2 * h], dst);
    gemm_async_copy16(xa + (int64_t)kt * BK, offa[2 * h + 1], dst + 8192u);
  };
  auto issue_w = [&](int kt, int stage, int h) __attribute__((always_inline)) {
    const uint32_t dst = copy0 + (uint32_t)(B_AREA + stage * TILE + h * HALF_TILE);
    gemm_async_copy16(wb + (int64_t)kt * BK, offb[2 * h], dst);
    gemm_async_copy16(wb + (int64_t)kt * BK, offb[2 * h + 1], dst + 8192u);
  };
  const int KT = P.hidden / BK;
  auto issue_first = [&]() __attribute__((always_inline)) {   // what the phases before a tile's first would have requested
    issue_w(0, 0, 0);
    issue_x(0, 0, 0);
    issue_w(0, 0, 1);
    issue_x(0, 0, 1);
    if (KT > 1) {
      issue_w(1, 1, 0);
      issue_x(1, 1, 0);
      issue_w(1, 1, 1);
    }
  };
  // nothing moves across a barrier, MFMAs included
  auto barrier = [&]() __attribute__((always_inline)) {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // This wave's copies have landed, except for the five half tiles requested last (N copies), if
  // so many were requested since.  Not needed in a tile's first k step, whose halves and the next
  // step's were waited for before it: there the previous tile's stores may still be on their way.
  // (The second k step's first wait is for everything, so that the counted ones have nothing but
  // copies to count.)
  constexpr std::integral_constant<int, 10 - (2 - M1)> kOneX1{};       // one second x half among the five
  constexpr std::integral_constant<int, 10 - 2 * (2 - M1)> kTwoX1{};   // two
  auto landed = [&](int t, bool five_behind, auto N) __attribute__((always_inline)) {
    if (t == 0) return;
    if (five_behind) __builtin_amdgcn_s_waitcnt(0x0F70 | decltype(N)::value);   // vmcnt(N)
    else __builtin_amdgcn_s_waitcnt(0x0F70);               // vmcnt(0)
  };

  // fragments: rows 16 * block + l16 of the wave's part of a half tile, elements 32 kk + 8 grp ..
  typedef const __attribute__((address_space(3))) unsigned char* lds_cptr;
  lds_cptr pa[2], pb[2];
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    const uint32_t g = (((uint32_t)(kk * 4 + grp)) ^ (uint32_t)((l16 >> 1) % NGR)) * 16u;
    uint32_t a = smem0 + (uint32_t)((wm * 64 + l16) * ROWB) + g;
    uint32_t b = smem0 + (uint32_t)(B_AREA + (wn * 32 + l16) * ROWB) + g;
    asm volatile("" : "+v"(a), "+v"(b));   // (one register each: stage, half and block are immediate offsets)
    pa[kk] = (lds_cptr)(uintptr_t)a;
    pb[kk] = (lds_cptr)(uintptr_t)b;
  }
  // x fragments [block][kk] of the half at hand; w fragments [set][block][kk]: tile t has its w0 in set t & 1, its w1 in the other
  bf16x8 a[4][2], b[2][2][2];
  auto read_x = [&](int stage, int h) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < (h == 0 ? 4 : 2 * M1); ++i)
        a[i][kk] = *(const __attribute__((address_space(3))) bf16x8*)(pa[kk] + stage * TILE + h * HALF_TILE + i * 16 * ROWB);
  };
  auto read_w = [&](int set, int stage, int h) __attribute__((always_inline)) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int c = 0; c < 2; ++c)
        b[set][c][kk] = *(const __attribute__((address_space(3))) bf16x8*)(pb[kk] + stage * TILE + h * HALF_TILE + c * 16 * ROWB);
  };
  auto reads_done = [&]() __attribute__((always_inline)) { __builtin_amdgcn_s_waitcnt(0xC07F); };   // lgkmcnt(0)
  f32x4 acc[2][4][2][2];   // [x half][block of 16 rows][w half][block of 16 w rows]
  auto quadrant = [&](int h, int j, int set) __attribute__((always_inline)) {
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int i = 0; i < (h == 0 ? 4 : 2 * M1); ++i)
#pragma unroll
        for (int c = 0; c < 2; ++c)
          acc[h][i][j][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[set][c][kk], a[i][kk], acc[h][i][j][c], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };
  auto k_tile = [&](int t, auto ST) __attribute__((always_inline)) {
    constexpr int st = decltype(ST)::value;   // t & 1
    const bool one = t + 1 < KT, two = t + 2 < KT;
    read_x(st, 0);
    if (one) issue_x(t + 1, st ^ 1, 1);
    landed(t, one && t > 1, kTwoX1);   // w1 of tile t
    barrier();
    quadrant(0, 0, st);
    barrier();
    read_w(st ^ 1, st, 1);
    if (two) issue_w(t + 2, st, 0);
    landed(t, two, kOneX1);   // x1 of tile t
    barrier();
    quadrant(0, 1, st ^ 1);
    barrier();
    read_x(st, 1);
    if (two) issue_x(t + 2, st, 0);
    landed(t, two, kOneX1);   // w0 of tile t + 1
    barrier();
    quadrant(1, 1, st ^ 1);
    barrier();
    if (one) read_w(st ^ 1, st ^ 1, 0);
    if (two) issue_w(t + 2, st, 1);
    landed(t, two, kOneX1);   // x0 of tile t + 1
    barrier();
    reads_done();     // (the quadrant does not use them)
    quadrant(1, 0, st);
    barrier();
  };

  constexpr int HALF = D / 2;
  const int heads = P.Hq + 2 * P.Hkv;
  open_tile();
  issue_first();
  __builtin_amdgcn_s_waitcnt(0x0F70);
  for (;;) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int c = 0; c < 2; ++c) acc[h][i][j][c] = f32x4{0.f, 0.f, 0.f, 0.f};
    barrier();
    read_w(0, 0, 0);
    reads_done();
    if (wm == 1) barrier();   // the second group runs one barrier behind the first ...
    for (int t = 0; t < KT; t += 2) {
      k_tile(t, std::integral_constant<int, 0>{});
      if (t + 1 < KT) k_tile(t + 1, std::integral_constant<int, 1>{});
    }
    if (wm == 0) barrier();   // ... and both have passed the same number of them here
    // (every fragment read has fed an MFMA in front of a barrier: the LDS is free)

    // ---- the next tile's operands, and this tile's rows: cache slots and rotation angles
    const int ln = lane_now();
    const int row_first = tile_m * BM + (ln & 15);
    const int head = tile_n * (BN / D) + (D == 128 ? wn >> 1 : wn);      // one head per wave
    const int e0 = (D == 128 ? (wn & 1) * 32 : 0) + 8 * (ln >> 4);       // the lane's first column of the head
    block += (int)gridDim.x;   // (past the last tile where every workgroup has one)
    const bool more = order.at<false>(block, &tile_m, &tile_n);
    if (more) {
      open_tile();
      issue_first();
    }
    const bool turned = head < P.Hq + P.Hkv;   // queries and keys
    constexpr int NQ = 4 + 2 * M1;   // row blocks of the wave
    auto row_of = [&](int q) __attribute__((always_inline)) -> int {   // row of row block q of the wave
      return row_first + (q < 4 ? wm * 64 + q * 16 : 128 + wm * 32 * M1 + (q - 4) * 16);
    };
    // row block q: the lane's 8 columns (and their partners); the angles and the cache slot one block ahead
    float2 cs[2][8];
    int64_t slot[2];
    auto load_row = [&](int q) __attribute__((always_inline)) {
      const int64_t row = min(row_of(q), P.rows - 1);
      slot[q & 1] = head < P.Hq ? row : P.dst[row];
      if (!turned) return;
      const float2* src = P.cs + row * HALF + e0;
#pragma unroll
      for (int e = 0; e < 8; ++e) cs[q & 1][e] = src[e];
    };
    uint16_t* const base = head < P.Hq ? P.q_out + (int64_t)head * D + e0
                           : turned    ? P.cache_k + (int64_t)(head - P.Hq) * D + e0
                                       : P.cache_v + (int64_t)(head - P.Hq - P.Hkv) * D + e0;
    const int64_t stride = (int64_t)(head < P.Hq ? P.Hq : P.Hkv) * D;
    load_row(0);
    __builtin_amdgcn_s_waitcnt(0x0F70);   // vmcnt(0), before the first store: see `landed`
#pragma unroll
    for (int q = 0; q < NQ; ++q) {
      const f32x4(&u)[2] = acc[q >> 2][q & 3][0];
      const f32x4(&v)[2] = acc[q >> 2][q & 3][1];
      u32x4 ra, rb;
      if (q + 1 < NQ) load_row(q + 1);
      if (turned) {
        const float2* c = cs[q & 1];
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int e = 2 * w, f = e & 3;
          const f32x4 &x = u[w >> 1], &y = v[w >> 1];
          ra[w] = gemm_pack_bf16(x[f] * c[e].x - y[f] * c[e].y, x[f + 1] * c[e + 1].x - y[f + 1] * c[e + 1].y);
          rb[w] = gemm_pack_bf16(y[f] * c[e].x + x[f] * c[e].y, y[f + 1] * c[e + 1].x + x[f + 1] * c[e + 1].y);
        }
      } else {
#pragma unroll
        for (int w = 0; w < 4; ++w) {
          const int f = 2 * (w & 1);
          ra[w] = gemm_pack_bf16(u[w >> 1][f], u[w >> 1][f + 1]);
          rb[w] = gemm_pack_bf16(v[w >> 1][f], v[w >> 1][f + 1]);
        }
      }
      if (row_of(q) < P.rows && head < heads) {
        uint16_t* out = base + slot[q & 1] * stride;
        *(u32x4*)out = ra;
        *(u32x4*)(out + HALF) = rb;
      }
      __builtin_amdgcn_sched_barrier(0);   // (one block's values at a time in the registers)
    }
    if (!more) break;
  }
}

size_t proj_workspace_bytes(int D, int64_t rows) {
  return (size_t)rows * (sizeof(int64_t) + (size_t)(D / 2) * sizeof(float2));
}

template <int NI>
static int launch_rows_list(int64_t* dst, float2* cs, double log2_base, int half, const QkvItem* items, int n, hipStream_t st) {
  ProjRowsParams<NI> R;
  R.dst = dst;
  R.cs = cs;
  R.log2_base = log2_base;
  R.half = half;
  R.n_items = n;
  int mt = 0;
  int64_t rows = 0;
  for (int i = 0; i < n; ++i) {
    R.items[i] = items[i];
    if (items[i].n_tok > mt) mt = items[i].n_tok;
    rows += items[i].n_tok;
  }
  const bool runs = rows * half > kOneByOne;
  const int block_rows = 256 / half * (runs ? kRowsRun : 1);
  const dim3 grid((unsigned)n, (unsigned)((mt + block_rows - 1) / block_rows)), block(256);
  if (runs) hipLaunchKernelGGL((proj_rows_kernel<NI, kRowsRun>), grid, block, 0, st, R);
  else hipLaunchKernelGGL((proj_rows_kernel<NI, 1>), grid, block, 0, st, R);
  return (int)hipGetLastError();
}

// Whether the stream may use every compute unit (the default streams have no mask; an error counts as yes).
static bool has_whole_chip(hipStream_t st) {
  if (!st || st == hipStreamLegacy || st == hipStreamPerThread) return true;
  uint32_t mask[kProjCUs / 32] = {};
  if (hipExtStreamGetCUMask(st, kProjCUs / 32, mask) != hipSuccess) {
    (void)hipGetLastError();
    return true;
  }
  int n = 0;
  for (uint32_t m : mask) n += __builtin_popcount(m);
  return n >= kProjCUs;
}

// The projection of P.rows rows with tiles of one kind.
template <int D>
static int launch_tiles(const ProjParams& P, ProjTile tile, hipStream_t st) {
  const int64_t tiles = proj_tiles(tile, P.rows, P.n_out);
  const bool whole_chip = tiles <= kProjCUs || !proj_tile_phased(tile) || has_whole_chip(st);
  const dim3 grid((unsigned)proj_workgroups(tile, tiles, whole_chip)), block(512);
  switch (tile) {
    case kTile256Phased: hipLaunchKernelGGL((qkv_proj_phased_kernel<D, 256>), grid, block, 0, st, P); break;
    case kTile192Phased: hipLaunchKernelGGL((qkv_proj_phased_kernel<D, 192>), grid, block, 0, st, P); break;
    case kTile256: hipLaunchKernelGGL((qkv_proj_kernel<D, 256>), grid, block, 0, st, P); break;
    case kTile128: hipLaunchKernelGGL((qkv_proj_kernel<D, 128>), grid, block, 0, st, P); break;
    case kTile64: hipLaunchKernelGGL((qkv_proj_kernel<D, 64>), grid, block, 0, st, P); break;
  }
  return (int)hipGetLastError();
}

int launch_qkv_proj(const LayerShape& ls, const void* x, const void* w, int32_t hidden, int32_t rows, void* q_out,
                    void* cache_k, void* cache_v, const QkvItem* items, int n_items, double theta_base, void* workspace,
                    void* stream) {
  hipStream_t st = (hipStream_t)stream;
  int64_t* dst = (int64_t*)workspace;
  float2* cs = (float2*)((unsigned char*)workspace + (size_t)rows * sizeof(int64_t));
  for (int base = 0; base < n_items; base += kMaxProjItems) {
    const int n = n_items - base < kMaxProjItems ? n_items - base : kMaxProjItems;
    const int e = n <= kFewProjItems ? launch_rows_list<kFewProjItems>(dst, cs, log2(theta_base), ls.D / 2, items + base, n, st)
                                     : launch_rows_list<kMaxProjItems>(dst, cs, log2(theta_base), ls.D / 2, items + base, n, st);
    if (e) return e;
  }
  const int n_out = (ls.Hq + 2 * ls.Hkv) * ls.D;
  const ProjPlan plan = plan_qkv_proj(rows, n_out, hidden);
  int first = 0;
  for (int l = 0; l < plan.n; ++l) {
    ProjParams P;
    P.rows = plan.rows[l];
    P.x = (const uint16_t*)x + (int64_t)first * hidden;
    P.w = (const uint16_t*)w;
    P.q_out = (uint16_t*)q_out + (int64_t)first * ls.Hq * ls.D;
    P.cache_k = (uint16_t*)cache_k;
    P.cache_v = (uint16_t*)cache_v;
    P.dst = dst + first;
    P.cs = cs + (int64_t)first * (ls.D / 2);
    P.hidden = hidden;
    P.n_out = n_out;
    P.Hq = ls.Hq;
    P.Hkv = ls.Hkv;
    const int e = ls.D == 128 ? launch_tiles<128>(P, plan.tile[l], st) : launch_tiles<64>(P, plan.tile[l], st);
    if (e) return e;
    first += plan.rows[l];
  }
  return 0;
}

}  // namespace oppo

// gfx950 kernels: ragged chunked-prefill attention, split-KV merge, KV append.
// (Passes of a few rows per sequence: attn_thin_kernel.h; the 8-bit cache: attn_fp8_kernel.h.)
//
// Attention (per workgroup = one AttnItem x one kv-head), 8 waves of 64 lanes:
//   * the query tile packs TM tokens x G q-heads of the kv-head into 256 rows
//     (row r = head r % G of token r / G);
//     wave w owns rows [32w, 32w+32), or [16w, 16w+16) where no tile of a launch
//     has more than 128.  The transposed product S^T = K Q^T is
//     computed with v_mfma_f32_16x16x32_bf16 (K as the A operand from LDS, Q^T
//     as the B operand held in registers), so one lane owns two query columns (or one):
//     the softmax statistics are per-lane scalars and the probabilities land
//     in the B-operand layout of the second product O^T = V^T P^T without any
//     cross-lane movement.  V^T fragments come from the token-major V tile in
//     LDS through the transposing LDS read (ds_read_b64_tr_b16).
//     (The chip runs this work against its power limit, and a multiplication in this shape
//     takes less of it than in 32x32x16: loops of nothing but MFMAs on N(0, 1) operands
//     sustain 1990-2050 and 1750 TFLOP/s.)
//   * keys are streamed in tiles of 64 with an online softmax (running max and
//     sum in fp32, exp2 domain with the scale folded in).
//   * causal mask aligned to the end of the cache: the tile's token t at
//     absolute position pos0+t sees keys <= pos0+t.
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>
#include <vector>

#include "oppo_internal.h"

namespace oppo {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(2))) int i32x2;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(8))) int i32x8;

// Work lists travel in the kernel arguments, which the host writes anew for every launch, across
// the bus, at their full length however few items are in use.  Each of these kernels therefore exists with
// a short list as well, and the launcher takes the short one whenever the work fits it.  A step of
// 4 sequences x 32 tokens took 16.6 us with the long list and 14.8 with the short one when the call itself took 5 us
// longer than it does now; at the lists' limits,
// one-row sequences, us per call (likewise): 64 / 65 appended 11.5 / 12.0 (8-bit 11.1 / 11.8), attention in 96 / 97 pieces
// 82.6 / 84.3, in 96 / 98 pieces that are merged 36.4 / 38.5.  (Replayed from a captured
// graph both lists take the same time.)
constexpr int kFewAttnItems = 96;
constexpr int kFewItems = 64;    // merge and append items

struct AttnFields {
  const uint16_t* q;
  uint16_t* k;             // keys / values: the cache, or the packed sequences of a one-shot prefill
  uint16_t* v;
  const uint16_t* k_new;   // appending variant only: the chunk's keys / values, rows indexed like q
  const uint16_t* v_new;
  uint16_t* out;
  float* part_o;
  float* part_ml;
  int32_t Hq, Hkv, G, TM;
  float c;
  float out_scale;     // 8-bit cache: the value tensor's scale (the output is the weighted mean of codes times it)
  float q_mult;        // 8-bit cache: c * 2^k, what the queries are multiplied by before they are rounded to E4M3
  int32_t q_scale_byte;   // ... and the E8M0 code of 2^-k (127 - k), the query operand's scale in the MFMA
  int32_t n_queues;
  uint32_t g_magic;    // ceil(2^16 / G): r / G == (r * g_magic) >> 16 for the rows r < 256 of a packed tile
};
template <int NI>
struct AttnParams : AttnFields {
  // queue j runs pieces first[j] .. first[j+1]-1, in that order (a short list has no more queues than pieces)
  uint16_t first[(NI < kMaxQueues ? NI : kMaxQueues) + 1];
  AttnItem items[NI];
};
static_assert(sizeof(AttnParams<kMaxAttnItems>) <= 32768, "kernel arguments are kept within 32 KiB");

template <int NI>
struct CombineParams {
  uint16_t* out;
  const float* part_o;
  const float* part_ml;
  int32_t Hq, Hkv, G, TM;
  float c;
  float out_scale;     // 1, or the value tensor's scale of an 8-bit cache
  int32_t n_items;
  CombineItem items[NI];
};
static_assert(sizeof(CombineParams<kMaxCombineItems>) <= 32768, "kernel arguments are kept within 32 KiB");

template <int NI>
struct AppendParams {
  uint16_t* cache_k;
  uint16_t* cache_v;
  const uint16_t* k_new;
  const uint16_t* v_new;
  int32_t row_granules;  // 16-byte granules per token row = Hkv*D/8
  int32_t n_items;
  AppendItem items[NI];
};
static_assert(sizeof(AppendParams<kMaxAppendItems>) <= 32768, "kernel arguments are kept within 32 KiB");

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

__device__ __forceinline__ s16x4 lds_read_tr16_l(const __attribute__((address_space(3))) unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p));
}

// Exchange of the two 32-lane halves of a wave: every lane receives the value
// held by the lane 32 away (v_permlane32_swap; the compiler's builtin for it
// mis-assigns the second result, so the instruction is written out).
__device__ __forceinline__ float swap_halves(float x) {
  float a = x, b = x;
  asm volatile("s_nop 1\n\tv_permlane32_swap_b32 %0, %1" : "+v"(a), "+v"(b));
  // a = {x[0:31], x[0:31]}, b = {x[32:63], x[32:63]}: pick the other half
  return (threadIdx.x & 32) ? a : b;
}

// LDS byte address of a __shared__ object.
__device__ __forceinline__ uint32_t lds_addr_of(const void* p) {
  return (uint32_t)(uintptr_t)((const __attribute__((address_space(3))) unsigned char*)p);
}

// Direct global -> LDS copy of 16 bytes per lane: lane l of the wave reads
// gbase[voff_bytes .. +16) and the data lands at LDS address lds_addr + 16 * l
// (gbase and lds_addr are wave-uniform).  Completion is tracked by vmcnt.
// Written as inline assembly on purpose: for the intrinsic form the compiler
// cannot tell the ring stages apart and waits for the copy before every later
// LDS read, which would serialise the prefetch; the waits are placed by hand.
// M0 is written here.  It is a reserved register: the compiler sets it before each of its
// own uses (LDS-DMA and GWS instructions, of which this kernel has none besides these), and
// it refuses M0 on a clobber list ("reserved register ... may lead to undefined behaviour"),
// so none is given.  The LDS addresses this produces are pinned by every GPU parity test.
__device__ __forceinline__ void async_copy16(const void* gbase, uint32_t voff_bytes, uint32_t lds_addr) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds_addr), "v"(voff_bytes), "s"(gbase) : "memory");
}

// Transposing LDS read: within each group of 16 lanes, lane j supplies the
// address of 4 consecutive bf16; lane i receives element (i & 3) of the
// pieces supplied by lanes (i >> 2), 4 + (i >> 2), 8 + (i >> 2), 12 + (i >> 2).
__device__ __forceinline__ s16x4 lds_read_tr16(const unsigned char* p) {
  return __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (s16x4 __attribute__((address_space(3)))*)(const_cast<unsigned char*>(p)));
}

// Eight bf16 values times `mult` -> eight E4M3 codes (round to nearest even; products beyond the
// format's largest finite value, 448, are clamped to it first), element i in byte i.
__device__ __forceinline__ long bf16x8_to_fp8x8(bf16x8 x, float mult) {
  union { bf16x8 v; uint32_t w[4]; } u;
  u.v = x;
  int lo = 0, hi = 0;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float a = __builtin_amdgcn_fmed3f(__uint_as_float(u.w[i] << 16) * mult, -448.0f, 448.0f);
    const float b = __builtin_amdgcn_fmed3f(__uint_as_float(u.w[i] & 0xffff0000u) * mult, -448.0f, 448.0f);
    // (the half of the word that is written has to be a literal)
    if (i == 0) lo = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, lo, false);
    else if (i == 1) lo = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, lo, true);
    else if (i == 2) hi = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, hi, false);
    else hi = __builtin_amdgcn_cvt_pk_fp8_f32(a, b, hi, true);
  }
  return (long)(((unsigned long)(uint32_t)hi << 32) | (unsigned long)(uint32_t)lo);
}

// Persistent workgroups: the launch has one workgroup per (queue, kv-head), about
// one per compute unit, and workgroup (queue j, kv-head g) runs the pieces
// first[j] .. first[j+1]-1 of the work list one after the other.
// Eight waves, each owning 32 query columns of the 256-row tile; two waves share
// a SIMD.  On this hardware vector ALU instructions hide under MFMAs only when
// the two are mixed finely (a handful of vector instructions per MFMA), so the
// instruction stream is laid out by hand and fenced with sched_barrier: see the
// main loop.  Operand fragments are read from LDS several steps before the MFMA
// that consumes them (rolling register buffers ka / vf).
// K/V tiles go straight from global memory into a ring of four LDS stages, two
// tiles ahead: the loads of the tile two places further down the workgroup's
// tile stream are issued after the barrier that opens an iteration (with heads of 128, by half of the waves in the
// middle of its first unit), into the stage whose last reader finished before that barrier, and each wave waits for
// its own loads before the barrier that closes it.  The stream runs across piece
// boundaries: the first two tiles of the next piece are requested during the last
// two iterations of the current one, and the next piece's Q fragments are
// requested as soon as the current piece's last S^T MFMA has been issued.
// APPEND: the chunk's own keys and values are not in the cache yet.  The key loop
// takes them from k_new / v_new, and the piece that starts a query tile's key
// range also copies the tile's token rows into the cache (nothing in this launch
// reads those cache rows).
// NCB: 16-column blocks of a wave.  (Four waves of 64 columns would halve the fragment reads; their loop alone, one wave per
// SIMD with nothing to fill its gaps, sustains 1382 TFLOP/s beside 1368 with two blocks, and boundaries would cost more.)
// One block where no tile has more than 128 rows (kernel_rows): with two blocks only one wave of a SIMD would have rows, and a
// wave alone is bound by the issue of its own instructions (64 keys take it 1.0 us, two waves 1.3 us).
template <int D, bool APPEND, int NI, int NCB>
__global__ __launch_bounds__(512) void attn_fwd_kernel(const AttnParams<NI> P) {
  constexpr int NW = 8, NT = 64 * NW;   // waves, threads
  constexpr int WROWS = 16 * NCB;    // packed rows of a wave
  constexpr int NG = D / 8;          // 16-byte granules per K/V row
  constexpr int KK = D / 32;         // k-steps of S^T = K Q^T
  constexpr int DB = D / 16;         // 16-row blocks of O^T
  constexpr int BN = kKeyTile;
  constexpr int ROWB = D * 2;        // bytes per K/V row in LDS
  constexpr int TILE_BYTES = BN * ROWB;
  constexpr int NSTAGE = 4;
  constexpr int RPI = 1024 / ROWB;     // tile rows one wave-wide 16-byte load covers
  constexpr int IPW = BN / RPI / NW;   // such loads per wave, per tile, for K and again for V
  constexpr int KDEPTH = KK;         // K fragments kept in flight (half a unit ahead: four MFMA steps cover the
                                     // LDS latency several times over, and a whole unit costs 16 more registers)
  constexpr int VDEPTH = DB / 2;     // V^T fragments kept in flight
  static_assert(IPW >= 1, "tile smaller than the workgroup");
  static_assert(NCB == 1 || NCB == 2, "staging area, vector work of a step");

  // K stages and V stages are two arrays of at most 64 KiB each, so that every
  // fragment read is "per-lane base register + immediate offset" (the LDS
  // instructions take 16-bit offsets)
  __shared__ __attribute__((aligned(1024))) unsigned char sk[NSTAGE][TILE_BYTES];
  __shared__ __attribute__((aligned(1024))) unsigned char sv[NSTAGE][TILE_BYTES];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int l16 = lane & 15;
  const int grp = lane >> 4;
  const int Hq = P.Hq, Hkv = P.Hkv, G = P.G, TM = P.TM;
  const int kvh = blockIdx.x % Hkv;
  const int queue = blockIdx.x / Hkv;
  const int p_first = P.first[queue];
  const int p_last = P.first[queue + 1];
  if (p_first >= p_last) return;
  const float c = P.c;

  // The queue's piece descriptors are copied from the kernel-argument segment into
  // LDS once: a read of that segment costs microseconds, far too much to pay at
  // every piece boundary.
  __shared__ __attribute__((aligned(16))) AttnItem spiece[NI];
  {
    const u32x4* src = (const u32x4*)(P.items + p_first);
    const int n16 = (p_last - p_first) * (int)(sizeof(AttnItem) / 16);
    for (int i = tid; i < n16; i += NT) ((u32x4*)spiece)[i] = src[i];
    __syncthreads();
  }
  // descriptor of piece p (a wave-uniform value, moved to scalar registers)
  auto piece = [&](int p) __attribute__((always_inline)) -> AttnItem {
    const u32x4* w = (const u32x4*)&spiece[p - p_first];
    const u32x4 a = w[0], b = w[1];
    AttnItem r;
    r.kv_row0 = (int64_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)a[1]) << 32) |
                          (uint32_t)__builtin_amdgcn_readfirstlane((int)a[0]));
    r.q_row0 = __builtin_amdgcn_readfirstlane((int)a[2]);
    r.n_tok = __builtin_amdgcn_readfirstlane((int)a[3]);
    r.pos0 = __builtin_amdgcn_readfirstlane((int)b[0]);
    r.k_begin = __builtin_amdgcn_readfirstlane((int)b[1]);
    r.k_end = __builtin_amdgcn_readfirstlane((int)b[2]);
    r.part = __builtin_amdgcn_readfirstlane((int)b[3]);
    return r;
  };

  // ---- this lane's query columns (rows l16 and 16 + l16 of the wave's 16 or 32) ------
  bf16x8 qf[NCB][KK];

  // ---- cooperative K/V tile loads ------------------------------------------------
  // Tiles travel global -> LDS directly (global_load_lds_dwordx4): a wave-wide
  // load drops 64 x 16 bytes at consecutive LDS addresses, i.e. RPI whole rows;
  // the LDS swizzle is applied by choosing which 16-byte granule of the row each
  // lane fetches.  Wave w moves rows (w + 8i) * RPI .. of the tile.
  const int row_stride = Hkv * D;  // elements between consecutive tokens
  const int lrow = lane / NG;
  const int pg = lane % NG;
  // Swizzle of a value row's granules: the transposing reads take 32 lanes at a time, 32 bytes of each of eight rows, and these
  // then lie in eight different parts of the 64 banks.  (With rows 4 apart in the same one a third of the LDS cycles were
  // conflicts, SQ_LDS_BANK_CONFLICT 1.34e8 of SQ_LDS_IDX_ACTIVE 4.05e8 on 16 x 1024 rows of 64/8 heads; the time of such passes is
  // the same to 0.3 %, the LDS is not what their loop waits for, but 15 x 15 rows on 413 .. 756 keys take 15.9 -> 15.5 us.)
  // The halves of a row's 64-byte pieces change places in the rows x / (NG / 4) % 2 = 1, with heads of 128 in all rows of a
  // wave's load or in none: with every other row so, passes that mostly read are 1 to 2 % slower (us, 32 x 22 rows on 4579 .. 5668
  // keys, 32/8 heads, 137.9 / 135.1, 223 x 6 rows on 1923 .. 5244, 64/8 heads, 637 / 628), others the same.
  auto vswz = [](int r) __attribute__((always_inline)) {
    const int x = r / (256 / ROWB);
    return x % (NG / 4) * 4 + x / (NG / 4) % 2 * 2;
  };
  uint32_t goffk[IPW], goffv[IPW];   // byte offsets of this lane's granules in a full tile
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    const int r = (wave + NW * i) * RPI + lrow;
    goffk[i] = (uint32_t)(r * row_stride + ((pg ^ (r % NG)) * 8)) * 2u;
    goffv[i] = (uint32_t)(r * row_stride + ((pg ^ vswz(r)) * 8)) * 2u;
  }
  const uint32_t wave_rows = (uint32_t)__builtin_amdgcn_readfirstlane(wave) * 1024u;

  // ---- the wave's staging area: turning 32 x D blocks around ----------------------
  // A lane owns one query column, so its share of Q (a B operand) and of the output
  // is 16-byte / 8-byte pieces of one row: moved to and from global memory like
  // that, every instruction would touch 32 or 64 different rows.  Q and O blocks
  // therefore travel as whole row pieces (16 bytes per lane, consecutive lanes on
  // consecutive addresses) and are turned around in LDS, half of D at a time.  The
  // staging area is the part of a ring stage that this very wave fills with its
  // next tile request (2*IPW chunks of 1 KiB, of which NCB*IPW are needed), used at a time when the stage's last
  // readers have passed a barrier: no other wave is involved, no barrier needed.
  constexpr int RB = D;             // bytes of a row per round (half a row)
  constexpr int NS = RB / 16;       // 16-byte slots of a row per round
  constexpr int RPC = 1024 / RB;    // rows per 1 KiB chunk
  constexpr int NCH = NCB * IPW;    // chunks
  typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
  // The lane-dependent offsets below are needed at piece boundaries only.  They are
  // derived from a copy of the lane number that the optimiser cannot see through,
  // so that it recomputes them there instead of keeping them in registers (which
  // the key loop has none to spare) for the whole kernel.
  auto lane_now = [&]() __attribute__((always_inline)) -> int {
    int x = lane;
    asm volatile("" : "+v"(x));
    return x;
  };
  // row-piece side: lane ln handles slot ln % NS of row ln / NS of each chunk
  auto roff_of = [&](int ln) __attribute__((always_inline)) -> uint32_t {
    return (uint32_t)((ln / NS) * RB + (((ln % NS) ^ ((ln / NS) & (NS - 1))) * 16));
  };
  // column side: row 16 * cb + ln % 16 lies in the K part (cb = 0) or the V part (cb = 1) of the area; cx_of = its swizzle
  auto cx_of = [&](int ln) __attribute__((always_inline)) -> uint32_t { return (uint32_t)(ln & (NS - 1)) * 16u; };
  auto area_of = [&](int stage, int k) __attribute__((always_inline)) -> uint32_t {   // chunk k of the area in `stage`
    return ((k / IPW) ? lds_addr_of(&sv[0][0]) : lds_addr_of(&sk[0][0])) + (uint32_t)stage * TILE_BYTES + wave_rows +
           (uint32_t)((k % IPW) * (NW * 1024));
  };
  static_assert(RPC * IPW == 16, "a column block per part");
  auto carea_of = [&](int stage, int cb, int ln) __attribute__((always_inline)) -> uint32_t {   // that row in its chunk
    const int row = ln & 15;
    return (cb ? lds_addr_of(&sv[0][0]) : lds_addr_of(&sk[0][0])) + (uint32_t)stage * TILE_BYTES + wave_rows +
           (uint32_t)(row / RPC * (NW * 1024) + row % RPC * RB);
  };
  // rows wave*WROWS + k*RPC + ln/NS of the packed tile -> (q-head of the group, token):
  // row R is head R % G of token R / G, so the rows of a tile of n tokens are the
  // first n * G ones (and rows from TM * G on, if G does not divide 256, are never used)
  auto row_of = [&](int ln, int k, int* hk, int* tk) __attribute__((always_inline)) {
    const int R = (int)(wave_rows >> 10) * WROWS + ln / NS + k * RPC;   // (wave number as a scalar)
    const int t = (int)(((uint32_t)R * P.g_magic) >> 16);            // R / G
    *tk = t;
    *hk = R - t * G;
  };
  u32x4 qraw[2][NCH];   // Q row pieces on their way: [half of D][chunk]
  auto q_request = [&](const AttnItem& a) __attribute__((always_inline)) {
    const int ln = lane_now();
#pragma unroll
    for (int k = 0; k < NCH; ++k) {
      int hk, tk;
      row_of(ln, k, &hk, &tk);
      // rows beyond the tile repeat a valid row; their columns are never stored
      const uint16_t* qp = P.q + ((int64_t)(a.q_row0 + min(tk, tokens_of(a) - 1)) * Hq + kvh * G + hk) * D + (ln % NS) * 8;
#pragma unroll
      for (int h = 0; h < 2; ++h) qraw[h][k] = *(const u32x4*)(qp + h * (D / 2));
    }
  };
  auto q_collect = [&](int stage) __attribute__((always_inline)) {
    const int ln = lane_now();
    const uint32_t roff = roff_of(ln);
    const uint32_t cxg = cx_of(ln) ^ ((uint32_t)(ln >> 4) * 16u);   // the lane's slots are 4*kl + grp, swizzled
#pragma unroll
    for (int h = 0; h < 2; ++h) {
#pragma unroll
      for (int k = 0; k < NCH; ++k)
        *(__attribute__((address_space(3))) u32x4*)(lds_ptr)(uintptr_t)(area_of(stage, k) + roff) = qraw[h][k];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
        for (int kl = 0; kl < KK / 2; ++kl)
          qf[cb][h * (KK / 2) + kl] = *(const __attribute__((address_space(3))) bf16x8*)(lds_ptr)(uintptr_t)(
              carea_of(stage, cb, ln) + ((uint32_t)(kl * 64) ^ cxg));
    }
  };
  // The request cursor walks the workgroup's tile stream (all tiles of piece
  // p_first, then of the next piece, ...): all of it is wave-uniform.  A run of whole tiles from one source (cache or chunk) costs
  // a request little but its copies, and what else there is to do (a piece's ragged last tile, the one that crosses from
  // cache to chunk, the next run or piece) is out of the way: behind the barrier that opens an iteration no wave has
  // anything else to run, so each instruction here, and above all each branch taken, is time in which the matrix cores idle.
  // For the same reason what comes next is found behind an iteration's first body and not where it is requested: in front of the
  // first body short pieces, which have little but ends of runs, paid for it.  us in one run, there / here: 424 rows on 77 .. 203
  // keys, 8/2 heads of 128, 13.4 / 13.1, 19 x 138 rows on 82 .. 119, 32/8 heads, 20.1 / 19.8, 5 x 93 rows on 465 .. 498, 64/8
  // heads, 19.2 / 19.0; 1024 rows on up to 8192 keys, 64/8 heads, 1772 / 1775.
  int run = 0;                 // tiles left of the run; kOneTile: the next tile belongs to no run; kNoTile: there is none
  constexpr int kOneTile = -1, kNoTile = -2;
  uintptr_t r_k = 0, r_v = 0;  // its next tile's first row, this kv-head
  int c_piece = p_first - 1;   // piece at the cursor
  int c_key = 0, c_n = 0;      // first key behind the run, and end, of its range, counted from the range's start
  int c_cached = 0;            // APPEND: how many of these keys are in the cache (may be negative)
  uintptr_t c_k = 0, c_kn = 0; // key c_key's row in k, and (APPEND) where that row would be in k_new; v is a fixed distance away
  const uintptr_t k_to_v = (uintptr_t)P.v - (uintptr_t)P.k;
  const uintptr_t kn_to_vn = APPEND ? (uintptr_t)P.v_new - (uintptr_t)P.k_new : 0;
  const uint32_t tile_step = (uint32_t)(BN * row_stride) * 2u;
  // (LDS addresses are formed from a copy of the wave's offset that the optimiser
  // cannot see through: otherwise it keeps one precomputed address per stage, array and
  // load in scalar registers for the whole kernel, and those run out)
  auto copy_at = [&](int stage) __attribute__((always_inline)) -> uint32_t {
    uint32_t wave_rows_now = wave_rows;
    asm volatile("" : "+s"(wave_rows_now));
    return wave_rows_now + (uint32_t)stage * TILE_BYTES;
  };
  // The next tile of the run, into `stage`.
  auto request_plain = [&](int stage) __attribute__((always_inline)) {
    const uint32_t at = copy_at(stage);
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      async_copy16((const void*)r_k, goffk[i], lds_addr_of(&sk[0][0]) + at + i * (NW * 1024u));
      async_copy16((const void*)r_v, goffv[i], lds_addr_of(&sv[0][0]) + at + i * (NW * 1024u));
    }
    r_k += tile_step;
    r_v += tile_step;
    --run;
  };
  // At the end of a run (run = 0): finds what comes next.
  auto next_run = [&]() __attribute__((always_inline)) {
    if (c_key >= c_n) {
      if (c_piece + 1 >= p_last) {
        run = kNoTile;
        return;
      }
      const AttnItem a = piece(++c_piece);
      c_key = 0;
      c_n = a.k_end - a.k_begin;
      c_k = (uintptr_t)(P.k + (((int64_t)a.kv_row0 + a.k_begin) * Hkv + kvh) * D);
      if (APPEND) {
        const int j0 = tile_of(a) * TM;          // the tile's first token within its chunk
        c_cached = (a.pos0 - j0) - a.k_begin;    // keys before the chunk are cached
        c_kn = (uintptr_t)(P.k_new + (((int64_t)(a.q_row0 - j0) - c_cached) * Hkv + kvh) * D);
      }
      // (lgkmcnt(0): where the compiler sees a read of this rare path as outstanding, the common one waits for all of its own)
      __builtin_amdgcn_s_waitcnt(0xC07F);
    }
    const bool fresh = APPEND && c_cached <= c_key;
    run = ((APPEND && !fresh ? min(c_n, c_cached) : c_n) - c_key) / BN;
    if (run == 0) {
      run = kOneTile;
      return;
    }
    r_k = fresh ? c_kn : c_k;
    r_v = r_k + (fresh ? kn_to_vn : k_to_v);
    c_key += run * BN;
    c_k += (uintptr_t)run * tile_step;
    if (APPEND) c_kn += (uintptr_t)run * tile_step;
  };
  // The tile that belongs to no run, into `stage`.
  auto request_one = [&](int stage) __attribute__((always_inline)) {
    const int last = c_n - c_key - 1, cached = APPEND ? c_cached - c_key : BN;
    const int ln = lane_now();
    const uint32_t at = copy_at(stage);
#pragma unroll
    for (int i = 0; i < IPW; ++i) {
      const int r = ((int)(wave_rows >> 10) + NW * i) * RPI + ln / NG;
      const int rc = min(r, last);   // ragged last tile: rows past the range repeat the last key
      const uint32_t ok = (uint32_t)(rc * row_stride + (((ln % NG) ^ (r % NG)) * 8)) * 2u;
      const uint32_t ov = (uint32_t)(rc * row_stride + (((ln % NG) ^ vswz(r)) * 8)) * 2u;
      const uint32_t lk = lds_addr_of(&sk[0][0]) + at + i * (NW * 1024u);
      const uint32_t lv = lds_addr_of(&sv[0][0]) + at + i * (NW * 1024u);
      // cache rows, then chunk rows: each lane's 16 bytes land at the LDS address of its
      // lane number, so the two sources fill one tile with complementary lane masks
      if (!APPEND || rc < cached) {
        async_copy16((const void*)c_k, ok, lk);
        async_copy16((const void*)(c_k + k_to_v), ov, lv);
      } else {
        async_copy16((const void*)c_kn, ok, lk);
        async_copy16((const void*)(c_kn + kn_to_vn), ov, lv);
      }
    }
    c_key += BN;
    c_k += tile_step;
    if (APPEND) c_kn += tile_step;
    run = 0;
  };
  auto issue_next = [&](int stage) __attribute__((always_inline)) {
    if (run > 0) request_plain(stage);
    else if (run == kOneTile) request_one(stage);
    if (run == 0) next_run();
  };
  // workgroup barrier without the implied wait for this wave's LDS reads: the only
  // reads still in flight at a barrier are the K fragments of the next tile, whose
  // stage is not overwritten before they have been consumed
  auto wg_barrier = [&]() __attribute__((always_inline)) {
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // per-lane LDS offsets of the operand fragments (the swizzles are XORs, so they
  // are folded here once instead of per read)
  // per-lane base pointers; stage, key half and group then are immediate offsets
  // (made opaque to the optimiser, which would otherwise fold the array address
  // into each read and rebuild the sum with a vector instruction every time)
  typedef const __attribute__((address_space(3))) unsigned char* lds_cptr;
  lds_cptr kptr[KK];   // K fragment of k-step kk, keys 0 .. 15 of a tile
#pragma unroll
  for (int kk = 0; kk < KK; ++kk) {
    uint32_t a = lds_addr_of(&sk[0][0]) + (uint32_t)(l16 * ROWB + (((kk * 4 + grp) ^ (l16 % NG)) * 16));
    asm volatile("" : "+v"(a));
    kptr[kk] = (lds_cptr)(uintptr_t)a;
  }
  lds_cptr vptr[DB];   // V^T fragment of a d-block, keys 4 * grp .. of a tile
  {
    const int vrow = 4 * grp + (l16 >> 2);
#pragma unroll
    for (int j = 0; j < DB; ++j) {
      const int lg = j * 2 + ((l16 & 3) >> 1);
      uint32_t a = lds_addr_of(&sv[0][0]) + (uint32_t)(vrow * ROWB + ((lg ^ vswz(vrow)) * 16) + (l16 & 1) * 8);
      asm volatile("" : "+v"(a));
      vptr[j] = (lds_cptr)(uintptr_t)a;
    }
  }
  // K fragment (A operand of S^T = K Q^T) of step j = (k-step j / 2, 16-key block j % 2) of the 32-key
  // unit (stage, kb): keys kb*32 + (j % 2)*16 + l16, elements (j / 2)*32 + 8*grp..;
  // `off` = stage * TILE_BYTES (an immediate in the main loop)
  auto ldk = [&](int off, int kb, int j) __attribute__((always_inline)) -> bf16x8 {
    return *(const __attribute__((address_space(3))) bf16x8*)(kptr[j / 2] + off + (2 * kb + j % 2) * 16 * ROWB);
  };
  // V^T fragment (A operand of O^T += V^T P^T) of d-block j of the 32-key unit (stage, kb): the eight
  // contraction indices of lane group grp are keys 4*grp .. and 16 + 4*grp .., as S^T leaves them in P^T
  auto ldv = [&](int off, int kb, int j) __attribute__((always_inline)) -> bf16x8 {
    lds_cptr vp = vptr[j] + off + kb * 32 * ROWB;
    union { struct { s16x4 a, b; } h; bf16x8 v; } cat;
    cat.h.a = lds_read_tr16_l(vp);
    cat.h.b = lds_read_tr16_l(vp + 16 * ROWB);
    return cat.v;
  };

  // A column's reference value m_run (the "running max" of the online softmax) is
  // only moved when the partial row sum of a 32-key unit exceeds 2^24: the weights
  // stay far inside the fp32 / bf16 range, relative precision does not depend on
  // the reference, and the maximum is not needed on the common path.
  constexpr float kRowSumLimit = 16777216.0f;

  // ------------------------------------------------------------------------------
  // Main loop, software-pipelined over 32-key units (two per 64-key tile).  The
  // body of unit u issues, interleaved instruction by instruction,
  //   * the MFMAs of S^T for unit u+1            (four dependent chains: two key by two column blocks),
  //   * the MFMAs of O^T += V^T P^T for unit u-1 (2 * DB independent ones),
  //   * the exp2 / bf16 rounding / row-sum vector work of unit u,
  // so the matrix pipe always has an independent MFMA to run and the vector ALU
  // work (five instructions, two of them exp2, per four MFMAs) is spread evenly under it.
  // What is rare in the loop is marked so (__builtin_expect), and the compiler puts it behind the kernel: the common path of an
  // iteration is one straight piece of code.  Behind a barrier both waves of a SIMD run the same scalar code, and every taken
  // branch is a gap in its MFMAs.  One run, us, without / with: 64 x 256 rows on 262 .. 1017 keys 226.5 / 225.3, prompts of
  // 512 .. 2048 tokens 515 / 505, 64/8 heads, 1024 rows on up to 8192 keys 1724 / 1716.
  // Against the same loop on 32x32x16 MFMAs with v_dot2 row sums, one run, us: 64 x 256 rows on 262 .. 1017 keys 243 -> 235,
  // prompts of 512 .. 2048 tokens 555 -> 534, 4 x 512 rows on 4096 .. 9999 keys 169 -> 160, 64/8 heads as above 1827 -> 1738.
  constexpr int QS = 2 * KK;      // K fragments of a unit, two S^T MFMAs (one per column block) each
  constexpr int PS = DB;          // V^T fragments of a unit, two O^T MFMAs each
  constexpr int PPS = NCB == 2 ? 8 / QS : 1;   // two blocks: probability pairs handled per step
  static_assert(QS == PS && QS % KDEPTH == 0 && PS % VDEPTH == 0, "pipeline shape");

  f32x4 o[DB][NCB];                              // [d-block][column block]
  f32x4 s[2][2][NCB];                            // s[u & 1][16-key block][column block] = S^T of unit u
  bf16x8 ka[KDEPTH];                             // K fragments in flight: step j of a unit sits in ka[j % KDEPTH]
  bf16x8 vf[VDEPTH];                             // V^T fragments in flight, likewise
  union { bf16x2 h[4 * NCB]; bf16x8 v[NCB]; } pf[2];   // pf[u & 1].v[column block] = probabilities of unit u, B-operand layout
  float m_run[NCB], l_run[NCB], mc[NCB], rs[NCB];

  // state of the piece being computed
  AttnItem it = piece(p_first);
  int lim[NCB];      // last key each of the lane's columns may see, minus 4 * grp: compared with the key
                     // that lane group 0 has in the same register, see the mask in unit_body
  int min_lim = 0;   // smallest such limit in the wave: units entirely below it need no mask

  // Pair pr of a unit's scores, and so of its probabilities: keys 2 * (pr % 2) and the next of 16-key block
  // (pr / 2) % 2, column block pr / 4.
  auto score = [&](int cur, int pr, int e) __attribute__((always_inline)) -> float {   // its exponent e = 0, 1
    return fmaf(s[cur][(pr / 2) % 2][pr / 4][2 * (pr % 2) + e], c, -mc[pr / 4]);
  };
  auto round_pair = [&](int cur, int pr, float p0, float p1) __attribute__((always_inline)) {
    bf16x2 pk;
    pk[0] = (__bf16)p0;
    pk[1] = (__bf16)p1;
    // (an empty asm statement pins the work to its place in the instruction stream: the
    // results are "used" by it, and such statements keep their order)
    asm volatile("" : "+v"(pk));
    pf[cur].h[pr] = pk;
  };
  // Row sums over the unit's 32 keys, taken over the rounded values like the numerator, by the matrix cores: every
  // lane of a column receives its sum.  The vector unit has no room for it (unpacking and adding is four instructions a
  // pair), and v_dot2_f32_bf16, one instruction a pair, does not run beside MFMAs: a loop of one 32x32x16 MFMA and four
  // of them takes 61 cycles, with four of any other vector instruction 32.  64/8 heads, 1024 rows on up to 8192 keys, one run:
  // unpacked adds 1909 us, v_dot2 at the unit's end 1830, here 1775 (32x32x16 MFMAs with v_dot2 between them: 1886).
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;
  asm volatile("" : "+v"(ones));   // (four registers, not rebuilt in every unit)
  auto row_sum = [&](int cur, int cb) __attribute__((always_inline)) -> float {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[cur].v[cb], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0)[0];
  };

  // Causal / range mask of the unit in s[cur], which starts at key key0, if it crosses a limit.  One register at a time, each
  // pinned: left to itself the compiler forms all comparisons first, and with scalar registers as scarce as in the append
  // variants it parks their results in lanes of a vector register (16 to 18 v_writelane and as many v_readlane per masked unit;
  // 161 scalar spills in the variant for heads of 128 with two column blocks, 35 with the pin and the same cursor).  Time with / without the pin: 4 x 1191
  // rows on 49 .. 91 keys, 4/4 heads of 64, 0.91; 170 x 196 rows on 161 .. 165 keys, the same heads, 0.95; 64 x 256 rows on
  // 262 .. 1017 keys, 32/8 heads of 128, 0.997.
  auto mask = [&](int cur, int key0) __attribute__((always_inline)) {
    if (__builtin_expect(key0 + 31 > min_lim, 0)) {
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        const int left = lim[cb] - key0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
          // register e % 4 of key block e / 4 holds key key0 + 16 * (e / 4) + 4 * grp + e % 4
          float x = s[cur][e / 4][cb][e % 4];
          if (16 * (e / 4) + e % 4 > left) x = -INFINITY;
          asm volatile("" : "+v"(x));
          s[cur][e / 4][cb][e % 4] = x;
        }
      }
    }
  };
  // Largest score of a column in that unit (its keys are spread over the four lanes that share l16).
  auto unit_max = [&](int cur, int cb) __attribute__((always_inline)) -> float {
    const f32x4 &x = s[cur][0][cb], &y = s[cur][1][cb];
    float mx = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(y[0], y[1]), fmaxf(y[2], y[3])));
    mx = fmaxf(mx, swap_halves(mx));
    return fmaxf(mx, __shfl_xor(mx, 16));
  };

  // Body of unit u.  BC = position of the unit in the LDS ring (stage, key half),
  // a compile-time value, so that every fragment read has an immediate offset.
  auto unit_body = [&](auto BC, int u, auto at_step) __attribute__((always_inline)) {
    constexpr int b = decltype(BC)::value;
    constexpr int st_c = b / 2, kb_c = b % 2;                   // unit u
    constexpr int st_n = ((b + 1) % 8) / 2, kb_n = (b + 1) % 2; // unit u+1
    constexpr int st_nn = ((b + 2) % 8) / 2, kb_nn = b % 2;     // unit u+2
    constexpr int st_p = ((b + 7) % 8) / 2, kb_p = (b + 7) % 2; // unit u-1
    constexpr int cur = b % 2, nxt = cur ^ 1;

    mask(cur, it.k_begin + 32 * u);
    // The probabilities of this unit are formed against the reference value m_run
    // the column already has (no maximum is taken first: the first one is that of the piece's first unit, taken in front of the
    // loop, where forming that unit twice took another 0.5 % of a pass); only if a row sum comes out too large, which is rare,
    // the unit is redone against its true maximum, see below.  (A column sees the keys up to its limit, and the first unit holds
    // the piece's first: one that sees none of it sees none of the piece.  Its reference stays -1e30 and its sum 0.)
#pragma unroll
    for (int e = 0; e < 2 * NCB; ++e) s[nxt][e % 2][e / 2] = f32x4{0.f, 0.f, 0.f, 0.f};

    if constexpr (NCB == 1) {
      // A step is two MFMAs and the work of EPS of the unit's eight weights; their exponents are formed one step ahead.
      constexpr int EPS = 8 / QS;
      float y[8], w[8];
#pragma unroll
      for (int e = 0; e < EPS; ++e) y[e] = score(cur, e / 2, e % 2);
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int i = 0; i < QS; ++i) {
        s[nxt][i % 2][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[i % KDEPTH], qf[0][i / 2], s[nxt][i % 2][0], 0, 0, 0);
        ka[i % KDEPTH] = (i + KDEPTH < QS) ? ldk(st_n * TILE_BYTES, kb_n, i + KDEPTH)
                                           : ldk(st_nn * TILE_BYTES, kb_nn, i + KDEPTH - QS);
#pragma unroll
        for (int e = i * EPS; e < (i + 1) * EPS; ++e) {
          w[e] = fast_exp2(y[e]);
          asm volatile("" : "+v"(w[e]));
        }
        __builtin_amdgcn_sched_barrier(0);
        o[i][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[i % VDEPTH], pf[nxt].v[0], o[i][0], 0, 0, 0);
        vf[i % VDEPTH] = (i + VDEPTH < PS) ? ldv(st_p * TILE_BYTES, kb_p, i + VDEPTH)
                                           : ldv(st_c * TILE_BYTES, kb_c, i + VDEPTH - PS);
#pragma unroll
        for (int e = (i + 1) * EPS; e < (i + 2) * EPS && e < 8; ++e) {
          y[e] = score(cur, e / 2, e % 2);
          asm volatile("" : "+v"(y[e]));
        }
#pragma unroll
        for (int e = i * EPS; e < (i + 1) * EPS; ++e)
          if (e % 2 == 1) round_pair(cur, e / 2, w[e - 1], w[e]);
        __builtin_amdgcn_sched_barrier(0);
        at_step(i);
      }
    } else {
      // An MFMA of this shape leaves the vector unit 8 of its 16 cycles: two instructions, or one exp2.  A step is four
      // MFMAs with PPS pairs' work dealt to them accordingly; a pair's exponents are formed one step ahead.
      float y0[PPS], y1[PPS], p0[PPS], p1[PPS];
#pragma unroll
      for (int j = 0; j < PPS; ++j) {
        y0[j] = score(cur, j, 0);
        y1[j] = score(cur, j, 1);
      }
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int i = 0; i < QS; ++i) {
        s[nxt][i % 2][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[i % KDEPTH], qf[0][i / 2], s[nxt][i % 2][0], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < PPS; ++j) {
          p0[j] = fast_exp2(y0[j]);
          asm volatile("" : "+v"(p0[j]));
        }
        __builtin_amdgcn_sched_barrier(0);
        s[nxt][i % 2][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[i % KDEPTH], qf[1][i / 2], s[nxt][i % 2][1], 0, 0, 0);
        ka[i % KDEPTH] = (i + KDEPTH < QS) ? ldk(st_n * TILE_BYTES, kb_n, i + KDEPTH)
                                           : ldk(st_nn * TILE_BYTES, kb_nn, i + KDEPTH - QS);
#pragma unroll
        for (int j = 0; j < PPS; ++j)
          if (i + 1 < QS) {
            y0[j] = score(cur, (i + 1) * PPS + j, 0);
            asm volatile("" : "+v"(y0[j]));
          }
        __builtin_amdgcn_sched_barrier(0);
        o[i][0] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[i % VDEPTH], pf[nxt].v[0], o[i][0], 0, 0, 0);
#pragma unroll
        for (int j = 0; j < PPS; ++j) {
          p1[j] = fast_exp2(y1[j]);
          asm volatile("" : "+v"(p1[j]));
        }
        __builtin_amdgcn_sched_barrier(0);
        o[i][1] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[i % VDEPTH], pf[nxt].v[1], o[i][1], 0, 0, 0);
        vf[i % VDEPTH] = (i + VDEPTH < PS) ? ldv(st_p * TILE_BYTES, kb_p, i + VDEPTH)
                                           : ldv(st_c * TILE_BYTES, kb_c, i + VDEPTH - PS);
#pragma unroll
        for (int j = 0; j < PPS; ++j) {
          if (i + 1 < QS) {
            y1[j] = score(cur, (i + 1) * PPS + j, 1);
            asm volatile("" : "+v"(y1[j]));
          }
          round_pair(cur, i * PPS + j, p0[j], p1[j]);
        }
        __builtin_amdgcn_sched_barrier(0);
        at_step(i);
      }
    }
    __builtin_amdgcn_s_setprio(0);
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) rs[cb] = row_sum(cur, cb);
    // pin the vector work above to this block: without a use here the compiler
    // sinks it below the branch that follows, away from the MFMAs it should hide under
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) asm volatile("" : "+v"(pf[cur].v[cb]), "+v"(rs[cb]));
    __builtin_amdgcn_sched_barrier(0);
    if (__builtin_expect(u == 0, 0)) {
      // the O^T MFMAs of a piece's first body belong to no unit (zero probabilities
      // times whatever the ring stage held): the accumulation starts here
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) o[db][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    if (__builtin_expect(__any(fmaxf(rs[0], rs[NCB - 1]) > kRowSumLimit), 0)) {
      // Some column saw a score far above its reference: take the unit's true maximum, move every
      // column's reference up to it, redo the unit's probabilities, and rescale what has been accumulated
      // so far - unit u-1 included, whose MFMAs above still used the old reference.
      float alpha[NCB];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        const float m_new = fmaxf(m_run[cb], unit_max(cur, cb));
        alpha[cb] = fast_exp2((m_run[cb] - m_new) * c);
        m_run[cb] = m_new;
        mc[cb] = m_new * c;
        l_run[cb] *= alpha[cb];
      }
#pragma unroll
      for (int pr = 0; pr < 4 * NCB; ++pr) round_pair(cur, pr, fast_exp2(score(cur, pr, 0)), fast_exp2(score(cur, pr, 1)));
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) rs[cb] = row_sum(cur, cb);
#pragma unroll
      for (int db = 0; db < DB; ++db)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) o[db][cb] *= alpha[cb];
    }
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) l_run[cb] += rs[cb];
  };

  // iteration = one tile = units 2t and 2t+1 of the piece (U units in all); TC is
  // the tile's ring stage.  The tile two places down the stream is requested in
  // it (see first_half) and awaited at its end, before the barrier after which the next
  // iteration starts reading the tile in between.
  // U: the units of the piece up to the last key that any of the wave's rows may see.  The causal limit of a tile's rows
  // differs by up to its number of tokens, so the first waves are through before the last; they go on requesting
  // tiles and joining barriers and leave the matrix cores, and the power, to the others.  One run, us, every wave to the
  // piece's end / so: prompts of 512 .. 2048 tokens 527 / 520, of 233 .. 570 147 / 144, of 305 .. 737 with 16/4 heads of 64
  // 108 / 104, 64 x 256 rows on 262 .. 1017 keys 232 / 229.
  int U = 0;
  // A wave whose rows all lie beyond the tile's tokens (a short tile fills the
  // first n_tok * G rows only) does none of the arithmetic of the piece: it still
  // requests its share of every key tile and joins the barriers, and leaves the
  // matrix and vector units of its SIMD to the waves that have rows.
  auto has_rows = [&](const AttnItem& a) __attribute__((always_inline)) -> bool {
    return (int)(wave_rows >> 10) * WROWS < tokens_of(a) * G;
  };
  bool act = true;
  // Heads of 128: of the two waves of a SIMD, one requests its share of a tile of a run in front of an iteration's first body and
  // the other in its middle, so that one of them has MFMAs to run while the other's copies are issued (of an iteration's 3300
  // cycles 400 to 590 passed between barrier and first MFMA, in scalar code and copies that all waves issued at once; now 280 of
  // 2920 in one wave and 120 in the other).  Behind the first body instead of in its middle the copies come too late where they
  // come from memory.  With heads of 64 a body is half as long, and the later copies cost more than they give.  Time by turns /
  // all in front, means over random passes (8 to 94 of a kind), contexts up to / from 1500 tokens: two blocks, heads of 128 0.999 /
  // 0.982 (64/8 heads, 1024 rows on up to 8192 keys 1771 -> 1733 us, 32 prompts of 512 .. 2048 tokens 525 -> 519, 64 x 256 rows on
  // 262 .. 1017 keys 232 -> 230), heads of 64 1.008 / 1.006; one block, heads of 128 1.001 / 1.002 (0.98 .. 1.02: both ways are
  // right about as often, so it is left as with two), heads of 64 1.010 / 1.009 (225 x 26 rows on 235 .. 464 keys, 16/4 heads, 26.4 ->
  // 27.3).
  constexpr bool kTurns = D == 128;
  const bool first_half = !kTurns || __builtin_amdgcn_readfirstlane(wave) < 4;
  auto iteration = [&](auto TC, int t) __attribute__((always_inline)) {
    constexpr int ts = decltype(TC)::value;
    const bool plain = run > 0;
    if (__builtin_expect(run == kOneTile, 0)) request_one((ts + 2) % NSTAGE);
    // (the hint: with two column blocks the waves that request later are the ones that the others wait for, and they fall through;
    // with one, tiles of up to 64 rows have rows in the first four waves alone: 45 x 10 rows on 751 .. 1695 keys, 8/2 heads, 23.9 us
    // where these branch away, 23.5 where they do not)
    if (__builtin_expect(first_half && plain, !kTurns || NCB == 1)) request_plain((ts + 2) % NSTAGE);
    unit_body(std::integral_constant<int, 2 * ts>{}, 2 * t, [&](int i) __attribute__((always_inline)) {
      if (i == QS / 2 - 1 && !first_half && plain) request_plain((ts + 2) % NSTAGE);
    });
    if (__builtin_expect(run == 0, 0)) next_run();
    if (__builtin_expect(2 * t + 1 < U, 1)) unit_body(std::integral_constant<int, 2 * ts + 1>{}, 2 * t + 1, [](int) {});
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): this wave's share of the requested tile is in LDS
    wg_barrier();
  };

  // ---- start-up: Q of the first piece, the first two tiles of the stream ------------
  act = has_rows(it);
  q_request(it);
  next_run();
  issue_next(0);
  issue_next(1);
  q_collect(2);
  // Everything issued so far must have landed before the loop; a wait left to the
  // compiler would sit inside the loop, where it would also cover later tiles.
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
  wg_barrier();

  int ph = 0;   // ring stage of the current piece's first tile
  for (int p = p_first;;) {
    // (per-lane values that only matter here are recomputed from an opaque copy of the
    // lane number, see lane_now)
    const int ln_top = lane_now();
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const int r_tile = (int)(wave_rows >> 10) * WROWS + 16 * cb + (ln_top & 15);   // the column's row of the packed tile
      const int tok = (int)(((uint32_t)r_tile * P.g_magic) >> 16);               // its token within the tile (r_tile / G)
      lim[cb] = min(it.pos0 + min(tok, tokens_of(it) - 1), it.k_end - 1) - 4 * (ln_top >> 4);
    }
    const int nkeys = it.k_end - it.k_begin;
    const int nt = (nkeys + BN - 1) / BN;
    {
      const int row0 = (int)(wave_rows >> 10) * WROWS, row1 = min(row0 + WROWS, tokens_of(it) * G) - 1;   // (act: row0 <= row1)
      const int tok0 = (int)(((uint32_t)row0 * P.g_magic) >> 16), tok1 = (int)(((uint32_t)max(row1, 0) * P.g_magic) >> 16);
      min_lim = min(it.pos0 + tok0, it.k_end - 1);
      // (a piece that starts behind what the wave's rows see: one unit, all of it masked)
      U = max(min(it.pos0 + tok1, it.k_end - 1) - it.k_begin, 0) / 32 + 1;
    }
    const int nt_own = act ? (U + 1) / 2 : 0;   // tiles with such a unit
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) m_run[cb] = mc[cb] = l_run[cb] = 0.f;   // (the first two: below, for waves with rows)
    // the accumulators start undefined (they are cleared after the first body, see
    // unit_body); saying so ends their live range at the previous piece's epilogue
#pragma unroll
    for (int db = 0; db < DB; ++db)
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) asm volatile("" : "=v"(o[db][cb]));

    // Whatever this wave still has in flight (the previous piece's stores, the tiles
    // requested ahead) is awaited here, on the path of every wave: left to the compiler,
    // the wait for the stores ends up inside the key loop, where it would cover each
    // newly requested tile as well.
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    // S^T of unit 0 on its own, then the operand buffers as the first body expects
    // them.  The ring stage is a run-time value here (and only here and in the drain).
    if (act) {
      const int off0 = ph * TILE_BYTES;
      const int offm = ((ph + 3) & 3) * TILE_BYTES;   // "unit -1": any stage, see unit_body
#pragma unroll
      for (int j = 0; j < KDEPTH; ++j) ka[j] = ldk(off0, 0, j);
#pragma unroll
      for (int e = 0; e < 2 * NCB; ++e) s[0][e % 2][e / 2] = f32x4{0.f, 0.f, 0.f, 0.f};
      // ring position of unit 0 is 2*ph: s[] and pf[] are indexed by its parity, 0
#pragma unroll
      for (int i = 0; i < QS; ++i) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
          s[0][i % 2][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ka[i % KDEPTH], qf[cb][i / 2], s[0][i % 2][cb], 0, 0, 0);
        ka[i % KDEPTH] = (i + KDEPTH < QS) ? ldk(off0, 0, i + KDEPTH) : ldk(off0, 1, i + KDEPTH - QS);
        __builtin_amdgcn_sched_barrier(0);
      }
      // the columns' first references
      mask(0, it.k_begin);
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        m_run[cb] = fmaxf(-1e30f, unit_max(0, cb));
        mc[cb] = m_run[cb] * c;
      }
#pragma unroll
      for (int j = 0; j < VDEPTH; ++j) vf[j] = ldv(offm, 1, j);
      const bf16x2 z2 = {(__bf16)0.0f, (__bf16)0.0f};
#pragma unroll
      for (int j = 0; j < 4 * NCB; ++j) pf[1].h[j] = z2;
    }

    // tiles of the piece, the loop unrolled over the four ring stages
    // O^T += V^T P^T of the last unit
    auto drain = [&]() __attribute__((always_inline)) {
      const int ul = U - 1;
      const int off = (((ul >> 1) + ph) & 3) * TILE_BYTES;
      const int kb = ul & 1;
      // the fragments preloaded by the last body belong to this unit already; its
      // probabilities are pf[ul & 1] (picked as values: an array indexed at run time
      // would be put into scratch memory)
      const bool odd = (ul & 1) != 0;
      bf16x8 pl[NCB];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        bf16x8 e0 = pf[0].v[cb], d0 = pf[1].v[cb];
        asm volatile("" : "+v"(e0), "+v"(d0));
        pl[cb] = odd ? d0 : e0;
      }
#pragma unroll
      for (int i = 0; i < PS; ++i) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
          o[i][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[i % VDEPTH], pl[cb], o[i][cb], 0, 0, 0);
        if (i + VDEPTH < PS) vf[i % VDEPTH] = ldv(off, kb, i + VDEPTH);
      }
    };
    const int tau1 = ph + nt_own;
    const bool early = act && nt_own < nt;   // (the last unit's values are overwritten two iterations on)
    if (act) {
      for (int tb = 0; tb < tau1; tb += 4) {
        if (__builtin_expect(tb >= ph, 1)) iteration(std::integral_constant<int, 0>{}, tb - ph);
        if (__builtin_expect(tb + 1 >= ph && tb + 1 < tau1, 1)) iteration(std::integral_constant<int, 1>{}, tb + 1 - ph);
        if (__builtin_expect(tb + 2 >= ph && tb + 2 < tau1, 1)) iteration(std::integral_constant<int, 2>{}, tb + 2 - ph);
        if (__builtin_expect(tb + 3 >= ph && tb + 3 < tau1, 1)) iteration(std::integral_constant<int, 3>{}, tb + 3 - ph);
      }
      if (early) {
        drain();
        __builtin_amdgcn_s_waitcnt(0xC07F);   // lgkmcnt(0): its reads are through before the barriers behind which the stage is refilled
      }
    }
    // (the same requests, waits and barriers as `iteration`, nothing else)
    for (int t = nt_own; t < nt; ++t) {
      issue_next((ph + t + 2) & 3);
      __builtin_amdgcn_s_waitcnt(0x0F70);
      wg_barrier();
    }

    // request the next piece's Q rows; they are collected after the epilogue
    const AttnItem done = it;
    const bool more = p + 1 < p_last;
    if (more) {
      it = piece(p + 1);
      act = has_rows(it);
      q_request(it);
    } else {
      // (defined on every path, so that the values are not kept alive across the key loop)
#pragma unroll
      for (int k = 0; k < NCH; ++k) qraw[0][k] = qraw[1][k] = u32x4{0u, 0u, 0u, 0u};
    }
    const int st_area = (ph + nt + 2) & 3;   // the stage the next tile request goes to

    // APPEND: the piece that starts the tile's key range moves the tile's token rows
    // (this kv-head's D elements of each) from k_new / v_new into the cache, 16 bytes
    // per thread and pass of CP_ROWS rows.  The first two passes are requested here
    // and stored after the epilogue; query tiles of more than 2 * CP_ROWS tokens
    // finish in a plain loop.  The data waits in the registers of s[1], which the
    // key loop no longer needs and the next piece's first body clears.
    constexpr int CP_ROWS = NT / NG;   // token rows per pass
    const bool cp_on = APPEND && done.k_begin == 0;
    const int cp_tid = (int)(wave_rows >> 4) + lane_now();   // thread number, recomputed here
    const int cp_row = cp_tid / NG, cp_g = cp_tid % NG;
    auto cp_src = [&](int row) __attribute__((always_inline)) -> int64_t {
      return (((int64_t)done.q_row0 + row) * Hkv + kvh) * D + cp_g * 8;
    };
    auto cp_dst = [&](int row) __attribute__((always_inline)) -> int64_t {
      return (((int64_t)done.kv_row0 + done.pos0 + row) * Hkv + kvh) * D + cp_g * 8;
    };
    auto park = [&](int slot, const u32x4& x) __attribute__((always_inline)) {
#pragma unroll
      for (int e = 0; e < 4; ++e) s[1][slot % 2][slot / 2][e] = __uint_as_float(x[e]);
    };
    auto unpark = [&](int slot) __attribute__((always_inline)) -> u32x4 {
      u32x4 x;
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = __float_as_uint(s[1][slot % 2][slot / 2][e]);
      return x;
    };
    if (cp_on) {
#pragma unroll
      for (int ps = 0; ps < NCB; ++ps) {
        const int row = ps * CP_ROWS + cp_row;
        if (row < tokens_of(done)) {
          park(2 * ps, *(const u32x4*)(P.k_new + cp_src(row)));
          park(2 * ps + 1, *(const u32x4*)(P.v_new + cp_src(row)));
        }
      }
    }

    if (!early) drain();

    // ---- epilogue ---------------------------------------------------------------------
    if (done.part < 0) {
      // final rows, turned around in the wave's staging area.  They (and the appended cache
      // rows further down) are stored with the non-temporal hint: nothing in this launch reads
      // them again, and lines that do not linger dirty in the level-2 cache need no write-back
      // when the kernel ends.
      float inv[NCB];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) inv[cb] = 1.0f / l_run[cb];
      const int ln = lane_now();
      const uint32_t roff = roff_of(ln), cx = cx_of(ln);
      // the lane's four elements of a d-block are half (grp % 2) of slot 2 * (block) + grp / 2
      const uint32_t cxg = cx ^ ((uint32_t)(ln >> 5) * 16u), half8 = (uint32_t)((ln >> 4) & 1) * 8u;
      int grow[NCH];                    // head-row (token * Hq + head) of the row in out, -1: not a row of this tile
#pragma unroll
      for (int k = 0; k < NCH; ++k) {
        int hk, tk;
        row_of(ln, k, &hk, &tk);
        grow[k] = tk < tokens_of(done) ? (done.q_row0 + tk) * Hq + kvh * G + hk : -1;
      }
#pragma unroll
      for (int h = 0; h < 2; ++h) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb)
#pragma unroll
          for (int dbl = 0; dbl < DB / 2; ++dbl) {
            bf16x4 w;
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e] = (__bf16)(o[h * (DB / 2) + dbl][cb][e] * inv[cb]);
            *(__attribute__((address_space(3))) bf16x4*)(lds_ptr)(uintptr_t)(carea_of(st_area, cb, ln) + half8 +
                                                                            ((uint32_t)(dbl * 32) ^ cxg)) = w;
          }
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
          const u32x4 val = *(const __attribute__((address_space(3))) u32x4*)(lds_ptr)(uintptr_t)(
              area_of(st_area, k) + roff);
          if (grow[k] >= 0) __builtin_nontemporal_store(val, (u32x4*)(P.out + (int64_t)grow[k] * D + (ln % NS) * 8 + h * (D / 2)));
        }
      }
    } else {
      const int lnp = lane_now();
      const int64_t slot0 = ((int64_t)done.part * Hkv + kvh) * kTileRows + (int)(wave_rows >> 10) * WROWS + (lnp & 15);
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        float* po = P.part_o + (slot0 + 16 * cb) * D + 4 * (lnp >> 4);
#pragma unroll
        for (int db = 0; db < DB; ++db) *(f32x4*)(po + db * 16) = o[db][cb];
        if (lnp < 16) {
          P.part_ml[(slot0 + 16 * cb) * 2 + 0] = m_run[cb];
          P.part_ml[(slot0 + 16 * cb) * 2 + 1] = l_run[cb];
        }
      }
    }
    if (cp_on) {
#pragma unroll
      for (int ps = 0; ps < NCB; ++ps) {
        const int row = ps * CP_ROWS + cp_row;
        if (row < tokens_of(done)) {
          __builtin_nontemporal_store(unpark(2 * ps), (u32x4*)(P.k + cp_dst(row)));
          __builtin_nontemporal_store(unpark(2 * ps + 1), (u32x4*)(P.v + cp_dst(row)));
        }
      }
      for (int row = NCB * CP_ROWS + cp_row; row < tokens_of(done); row += CP_ROWS) {
        const u32x4 a = *(const u32x4*)(P.k_new + cp_src(row));
        const u32x4 b = *(const u32x4*)(P.v_new + cp_src(row));
        __builtin_nontemporal_store(a, (u32x4*)(P.k + cp_dst(row)));
        __builtin_nontemporal_store(b, (u32x4*)(P.v + cp_dst(row)));
      }
    }
    if (more) q_collect(st_area);
    if (!more) break;
    ++p;
    ph = (ph + nt) & 3;
  }
}

#include "attn_fp8_kernel.h"
#include "attn_thin_kernel.h"

// Merge the partial (max, sum, unnormalised O) of the pieces of a split tile
// (at most kMaxSplit pieces):
// out = sum_s w_s O_s / sum_s w_s l_s with w_s = exp2((m_s - max_s m_s) * c).
// MAXS: upper bound on the pieces of any tile of the launch (4, 8 or MAXS); the per-piece
// arrays live in registers, and fewer of them means more waves in flight to hide the loads.
template <int D, int MAXS, int NI>
__global__ __launch_bounds__(256) void combine_kernel(const CombineParams<NI> P) {
  constexpr int TPR = D / 4;          // threads per row (float4 each)
  constexpr int RPB = 256 / TPR;      // rows per block
  const CombineItem it = P.items[blockIdx.x / P.Hkv];
  const int kvh = blockIdx.x % P.Hkv;
  const int r = blockIdx.y * RPB + threadIdx.x / TPR;
  const int d4 = (threadIdx.x % TPR) * 4;
  const int tok = r / P.G;    // row r of the packed tile is head r % G of token r / G
  const int hh = r - tok * P.G;
  if (tok >= it.n_tok) return;
  // all loads of a batch are issued before the first use, so the merge is bound
  // by bandwidth and not by a chain of dependent memory latencies
  const int64_t slot0 = ((int64_t)it.part0 * P.Hkv + kvh) * kTileRows + r;
  const int64_t sstride = (int64_t)P.Hkv * kTileRows;   // slots between consecutive pieces
  float ms[MAXS], ls[MAXS];
#pragma unroll
  for (int s = 0; s < MAXS; ++s) {
    const bool on = s < it.nsplit;
    const float2 ml = on ? *(const float2*)(P.part_ml + (slot0 + s * sstride) * 2) : float2{-INFINITY, 0.f};
    ms[s] = ml.x;
    ls[s] = ml.y;
  }
  float m_max = -INFINITY;
#pragma unroll
  for (int s = 0; s < MAXS; ++s) m_max = fmaxf(m_max, ms[s]);
  float l = 0.f;
#pragma unroll
  for (int s = 0; s < MAXS; ++s) {
    ms[s] = (s < it.nsplit) ? fast_exp2((ms[s] - m_max) * P.c) : 0.f;   // now the weight of piece s
    l += ms[s] * ls[s];
  }
  float4 acc = {0.f, 0.f, 0.f, 0.f};
  constexpr int BATCH = MAXS < 8 ? MAXS : 8;
#pragma unroll
  for (int s0 = 0; s0 < MAXS; s0 += BATCH) {
    if (s0 >= it.nsplit) break;
    float4 x[BATCH];
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      const int sj = min(s0 + j, it.nsplit - 1);   // clamped pieces carry weight 0 ... see below
      x[j] = *(const float4*)(P.part_o + (slot0 + sj * sstride) * D + d4);
    }
#pragma unroll
    for (int j = 0; j < BATCH; ++j) {
      const float w = (s0 + j < it.nsplit) ? ms[s0 + j] : 0.f;
      acc.x += w * x[j].x;
      acc.y += w * x[j].y;
      acc.z += w * x[j].z;
      acc.w += w * x[j].w;
    }
  }
  const float inv = P.out_scale / l;
  bf16x4 w4;
  w4[0] = (__bf16)(acc.x * inv);
  w4[1] = (__bf16)(acc.y * inv);
  w4[2] = (__bf16)(acc.z * inv);
  w4[3] = (__bf16)(acc.w * inv);
  uint16_t* op = P.out + ((int64_t)(it.q_row0 + tok) * P.Hq + kvh * P.G + hh) * D + d4;
  *(bf16x4*)op = w4;
}

// KV append: each item is one contiguous run of token rows (token-major layout
// makes a sequence's chunk contiguous in both source and destination).
// grid = (items, pieces of kAppendTok tokens, 2 = K/V); 16-byte copies.
constexpr int kAppendTok = 16;
template <int NI>
__global__ __launch_bounds__(256) void kv_append_kernel(const AppendParams<NI> P) {
  const AppendItem it = P.items[blockIdx.x];
  const int tok0 = blockIdx.y * kAppendTok;
  if (tok0 >= it.n_tok) return;
  const int ntok = min(kAppendTok, it.n_tok - tok0);
  const uint16_t* src = (blockIdx.z == 0 ? P.k_new : P.v_new);
  uint16_t* dst = (blockIdx.z == 0 ? P.cache_k : P.cache_v);
  const int64_t rg = P.row_granules;
  const u32x4* s = (const u32x4*)src + ((int64_t)it.src_row + tok0) * rg;
  u32x4* d = (u32x4*)dst + (it.dst_row + tok0) * rg;
  const int64_t n = (int64_t)ntok * rg;
  for (int64_t i = threadIdx.x; i < n; i += 256) d[i] = s[i];
}

// KV append into the 8-bit cache.  A bf16 value x becomes the E4M3 code nearest (ties to even)
// to clamp(fl32(x * inv_scale), -448, 448).  Keys keep the token-major order, one byte per
// element; values go into blocks of 64 tokens, [block][kv-head][element][token % 64], and what is
// left of the last block a run touches is filled with zero bytes.
// grid = (items, 64-token blocks the longest run touches, kv-heads); 2 * D threads.
template <int NI>
struct Append8Params {
  uint8_t* cache_k;
  uint8_t* cache_v;
  const uint16_t* k_new;
  const uint16_t* v_new;
  float k_inv, v_inv;    // fl32(1 / scale) of the two tensors
  int32_t Hkv;
  int32_t n_items;
  AppendItem items[NI];
};
static_assert(sizeof(Append8Params<kMaxAppendItems>) <= 32768, "kernel arguments are kept within 32 KiB");

__device__ __forceinline__ float code_range(uint32_t bf16_bits, float inv) {
  return __builtin_amdgcn_fmed3f(__uint_as_float(bf16_bits << 16) * inv, -448.0f, 448.0f);
}

template <int D, int NI>
__global__ __launch_bounds__(2 * D) void kv_append_fp8_kernel(const Append8Params<NI> P) {
  constexpr int NT = 2 * D;       // one thread per (4 tokens, 8 elements) of a 64-token block
  constexpr int BLK = kKeyTile;   // tokens per value block
  constexpr int NG = D / 8;       // 16-byte granules of a bf16 row of one kv-head
  constexpr int LROW = BLK + 4;   // bytes per element row of the transposed block in LDS (padded: 17 dwords)
  __shared__ __attribute__((aligned(16))) uint32_t vt[D * LROW / 4];
  const AppendItem it = P.items[blockIdx.x];
  const int64_t first = it.dst_row, end = it.dst_row + it.n_tok;   // the run's slots
  const int64_t blk = first / BLK + blockIdx.y;
  if (blk * BLK >= end) return;
  const int kvh = blockIdx.z;
  const int64_t lo = first > blk * BLK ? first : blk * BLK;             // the run's slots inside this block
  const int64_t hi = end < (blk + 1) * BLK ? end : (blk + 1) * BLK;
  const int64_t row_stride = (int64_t)P.Hkv * D;
  // keys: 8 elements (16 bytes in, 8 bytes out) per thread and step
  const int n8 = (int)(hi - lo) * NG;
  for (int idx = threadIdx.x; idx < n8; idx += NT) {
    const int64_t slot = lo + idx / NG;
    const int g = idx % NG;
    const u32x4 raw = *(const u32x4*)(P.k_new + (it.src_row + (slot - first)) * row_stride + kvh * D + g * 8);
    int w0 = 0, w1 = 0;
    w0 = __builtin_amdgcn_cvt_pk_fp8_f32(code_range(raw[0] & 0xffffu, P.k_inv), code_range(raw[0] >> 16, P.k_inv), w0, false);
    w0 = __builtin_amdgcn_cvt_pk_fp8_f32(code_range(raw[1] & 0xffffu, P.k_inv), code_range(raw[1] >> 16, P.k_inv), w0, true);
    w1 = __builtin_amdgcn_cvt_pk_fp8_f32(code_range(raw[2] & 0xffffu, P.k_inv), code_range(raw[2] >> 16, P.k_inv), w1, false);
    w1 = __builtin_amdgcn_cvt_pk_fp8_f32(code_range(raw[3] & 0xffffu, P.k_inv), code_range(raw[3] >> 16, P.k_inv), w1, true);
    *(u32x2*)(P.cache_k + slot * row_stride + kvh * D + g * 8) = u32x2{(uint32_t)w0, (uint32_t)w1};
  }
  // values, step 1: thread (quad, granule) reads 8 elements of the block's tokens 4 * quad .. + 3
  // (whole 16-byte pieces of the token rows), turns each element's four tokens into one 32-bit word
  // of codes (tokens outside the run: zero) and puts it into the transposed block in LDS
  {
    const int quad = threadIdx.x / NG, g = threadIdx.x % NG;
    const int64_t s0 = blk * BLK + 4 * quad;
    u32x4 raw[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int64_t slot = s0 + e;
      raw[e] = u32x4{0u, 0u, 0u, 0u};
      if (slot >= lo && slot < hi)
        raw[e] = *(const u32x4*)(P.v_new + (it.src_row + (slot - first)) * row_stride + kvh * D + g * 8);
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      float x[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) x[e] = code_range((j & 1) ? raw[e][j / 2] >> 16 : raw[e][j / 2] & 0xffffu, P.v_inv);
      int w = 0;
      w = __builtin_amdgcn_cvt_pk_fp8_f32(x[0], x[1], w, false);
      w = __builtin_amdgcn_cvt_pk_fp8_f32(x[2], x[3], w, true);
      vt[((8 * g + j) * LROW) / 4 + quad] = (uint32_t)w;
    }
  }
  __syncthreads();
  // step 2: 16-byte pieces (element d, tokens 16 * tq ..) go out, a wave writing 1 KiB in one piece.
  // Bytes of tokens before the run are kept, bytes of tokens behind it are zero.
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int piece = threadIdx.x + i * NT;
    const int d = piece / 4, tq = piece % 4;
    const int64_t s0 = blk * BLK + tq * 16;
    if (s0 + 16 <= lo) continue;   // all of it was there before
    uint8_t* dst = P.cache_v + ((blk * P.Hkv + kvh) * D + d) * BLK + tq * 16;
    u32x4 res;
#pragma unroll
    for (int j = 0; j < 4; ++j) res[j] = vt[(d * LROW) / 4 + tq * 4 + j];
    if (s0 < lo) {
      const u32x4 old = *(const u32x4*)dst;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        uint32_t keep = 0u;   // bytes of tokens before the run
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (s0 + 4 * j + e < lo) keep |= 0xffu << (8 * e);
        res[j] = (old[j] & keep) | (res[j] & ~keep);
      }
    }
    *(u32x4*)dst = res;
  }
}

// ---------------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------------

// Optional per-kernel timing: HIP events recorded on the launch stream right
// before and after each kernel launch while enabled.  The list of pairs is shared by
// all host threads and guarded by a lock.
struct EventPair { hipEvent_t a, b; int kind; bool closed; };
static std::mutex g_prof_mu;
static bool g_prof_on = false;
static std::vector<EventPair> g_prof_events;

// Returns the index of the pair that was opened, or -1 (profiling off, or no event to be had:
// then the launch is simply not timed).
static int prof_begin(int kind, hipStream_t st) {
  std::lock_guard<std::mutex> lock(g_prof_mu);
  if (!g_prof_on) return -1;
  EventPair p;
  p.kind = kind;
  p.closed = false;
  if (hipEventCreate(&p.a) != hipSuccess) return -1;
  if (hipEventCreate(&p.b) != hipSuccess) {
    (void)hipEventDestroy(p.a);
    return -1;
  }
  (void)hipEventRecord(p.a, st);
  g_prof_events.push_back(p);
  return (int)g_prof_events.size() - 1;
}
static void prof_end(int pair, hipStream_t st) {
  if (pair < 0) return;
  std::lock_guard<std::mutex> lock(g_prof_mu);
  if ((size_t)pair >= g_prof_events.size()) return;   // read (and cleared) by another thread meanwhile
  (void)hipEventRecord(g_prof_events[(size_t)pair].b, st);
  g_prof_events[(size_t)pair].closed = true;
}
// One launch, and nothing else, between the two events (kind < 0: not timed): the arguments are filled in before, and
// what is refused before its launch leaves no pair behind.
template <typename Kernel, typename Params>
static int launch_timed(int kind, Kernel kernel, dim3 grid, dim3 block, hipStream_t st, const Params& P) {
  const int pair = kind >= 0 ? prof_begin(kind, st) : -1;
  hipLaunchKernelGGL(kernel, grid, block, 0, st, P);
  prof_end(pair, st);
  return (int)hipGetLastError();
}
int profile_enable(int on) {
  std::lock_guard<std::mutex> lock(g_prof_mu);
  g_prof_on = on != 0;
  return 0;
}
bool profile_is_on() {
  std::lock_guard<std::mutex> lock(g_prof_mu);
  return g_prof_on;
}
// Waits for the recorded pairs and forgets them.  Sums per kind go to ms / launches; if
// `each_ms` is given, the first max_each launches' own durations and kinds as well, in
// launch order (n_each = how many were written).
int profile_read(double ms[3], int32_t launches[3], double* each_ms, int32_t* each_kind, int32_t max_each,
                 int32_t* n_each) {
  for (int k = 0; k < 3; ++k) ms[k] = 0.0, launches[k] = 0;
  std::vector<EventPair> pairs;
  {
    std::lock_guard<std::mutex> lock(g_prof_mu);
    pairs.swap(g_prof_events);
  }
  int rc = 0;
  int32_t written = 0;
  for (EventPair& p : pairs) {
    if (p.closed) {
      float t = 0.f;
      hipError_t e = hipEventSynchronize(p.b);
      if (e == hipSuccess) e = hipEventElapsedTime(&t, p.a, p.b);
      if (e != hipSuccess) rc = (int)e;
      else if (p.kind >= 0 && p.kind < 3) {
        ms[p.kind] += t, launches[p.kind] += 1;
        if (each_ms && written < max_each) {
          each_ms[written] = t;
          if (each_kind) each_kind[written] = p.kind;
          ++written;
        }
      }
    }
    (void)hipEventDestroy(p.a);
    (void)hipEventDestroy(p.b);
  }
  if (n_each) *n_each = written;
  return rc;
}

// Scratch buffer of the entry point that allocates nothing (partial results of split key
// ranges).  The array's name is a host-side stand-in for the symbol: kernels are given the
// address hipGetSymbolAddress reports for the current device, looked up once per device.
// Nothing in it has to start at zero: every partial row is written before it is read.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];
constexpr int kMaxDevices = 64;
static std::mutex g_scratch_mu;
static void* g_scratch_ptr[kMaxDevices] = {};

int static_scratch(void** ptr) {
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return (int)e;
  if (dev < 0 || dev >= kMaxDevices) return (int)hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return (int)e;
    if (!p) return (int)hipErrorInvalidSymbol;
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return 0;
}

template <int NI>
static int launch_attention_list(const LayerShape& ls, const AttnFields& F, bool append, const AttnItem* items, int n_items,
                                 const uint16_t* first, int n_queues, hipStream_t st, int kind) {
  if (n_items > NI || n_queues > n_items) return (int)hipErrorInvalidValue;
  AttnParams<NI> P;
  static_cast<AttnFields&>(P) = F;
  for (int j = 0; j <= n_queues; ++j) P.first[j] = first[j];
  for (int i = 0; i < n_items; ++i) P.items[i] = items[i];
  const dim3 grid((unsigned)(n_queues * ls.Hkv)), block(512);
  if (ls.fp8) {
    // (the 8-bit cache is filled by its own append kernel)
    if (append) return (int)hipErrorInvalidValue;
    return ls.D == 128 ? launch_timed(kind, attn_fwd_fp8_kernel<128, NI>, grid, block, st, P)
                       : launch_timed(kind, attn_fwd_fp8_kernel<64, NI>, grid, block, st, P);
  }
  const int rows = kernel_rows(ls, items, n_items);
  if (rows == 16)
    return ls.D == 128 ? (append ? launch_timed(kind, attn_thin_kernel<128, true, NI, 1>, grid, block, st, P)
                                 : launch_timed(kind, attn_thin_kernel<128, false, NI, 1>, grid, block, st, P))
                       : (append ? launch_timed(kind, attn_thin_kernel<64, true, NI, 1>, grid, block, st, P)
                                 : launch_timed(kind, attn_thin_kernel<64, false, NI, 1>, grid, block, st, P));
  if (rows == 32)
    return ls.D == 128 ? (append ? launch_timed(kind, attn_thin_kernel<128, true, NI, 2>, grid, block, st, P)
                                 : launch_timed(kind, attn_thin_kernel<128, false, NI, 2>, grid, block, st, P))
                       : (append ? launch_timed(kind, attn_thin_kernel<64, true, NI, 2>, grid, block, st, P)
                                 : launch_timed(kind, attn_thin_kernel<64, false, NI, 2>, grid, block, st, P));
  if (rows == 128)
    return ls.D == 128 ? (append ? launch_timed(kind, attn_fwd_kernel<128, true, NI, 1>, grid, block, st, P)
                                 : launch_timed(kind, attn_fwd_kernel<128, false, NI, 1>, grid, block, st, P))
                       : (append ? launch_timed(kind, attn_fwd_kernel<64, true, NI, 1>, grid, block, st, P)
                                 : launch_timed(kind, attn_fwd_kernel<64, false, NI, 1>, grid, block, st, P));
  if (ls.D == 128)
    return append ? launch_timed(kind, attn_fwd_kernel<128, true, NI, 2>, grid, block, st, P)
                  : launch_timed(kind, attn_fwd_kernel<128, false, NI, 2>, grid, block, st, P);
  return append ? launch_timed(kind, attn_fwd_kernel<64, true, NI, 2>, grid, block, st, P)
                : launch_timed(kind, attn_fwd_kernel<64, false, NI, 2>, grid, block, st, P);
}

int launch_attention(const LayerShape& ls, const void* q, void* k, void* v, const void* k_new, const void* v_new,
                     void* out, float* part_o, float* part_ml, const AttnItem* items, int n_items,
                     const uint16_t* first, int n_queues, void* stream, bool timed) {
  hipStream_t st = (hipStream_t)stream;
  if (n_items <= 0 || n_queues <= 0) return 0;
  if (n_items > kMaxAttnItems || n_queues > kMaxQueues) return (int)hipErrorInvalidValue;
  AttnFields F;
  F.q = (const uint16_t*)q;
  F.k = (uint16_t*)k;
  F.v = (uint16_t*)v;
  F.k_new = (const uint16_t*)k_new;
  F.v_new = (const uint16_t*)v_new;
  F.out = (uint16_t*)out;
  F.part_o = part_o;
  F.part_ml = part_ml;
  F.Hq = ls.Hq;
  F.Hkv = ls.Hkv;
  F.G = ls.G;
  F.TM = ls.TM;
  F.c = ls.c;
  F.out_scale = ls.out_scale;
  F.q_mult = 1.0f;
  F.q_scale_byte = 127;
  if (ls.fp8) {
    // k with 4 <= c * 2^k < 8: queries of magnitude 2^-8 .. 56 stay inside E4M3's normal range
    int e = 0;
    (void)frexpf(ls.c, &e);                  // c = f * 2^e, 0.5 <= f < 1
    const int k = 3 - e;                     // c * 2^k = 8 f, in [4, 8)
    if (k < -120 || k > 120) return (int)hipErrorInvalidValue;
    F.q_mult = ldexpf(ls.c, k);
    F.q_scale_byte = 127 - k;
  }
  F.n_queues = n_queues;
  F.g_magic = (65536u + (uint32_t)ls.G - 1u) / (uint32_t)ls.G;
  const bool append = k_new != nullptr;
  const int kind = timed ? 0 : -1;
  return n_items <= kFewAttnItems
             ? launch_attention_list<kFewAttnItems>(ls, F, append, items, n_items, first, n_queues, st, kind)
             : launch_attention_list<kMaxAttnItems>(ls, F, append, items, n_items, first, n_queues, st, kind);
}

template <int NI>
static int launch_combine_list(const LayerShape& ls, void* out, const float* part_o, const float* part_ml,
                               const CombineItem* items, int n, hipStream_t st, int kind) {
  CombineParams<NI> P;
  P.out = (uint16_t*)out;
  P.part_o = part_o;
  P.part_ml = part_ml;
  P.Hq = ls.Hq;
  P.Hkv = ls.Hkv;
  P.G = ls.G;
  P.TM = ls.TM;
  P.c = ls.fp8 ? 1.0f : ls.c;   // (the 8-bit kernel stores its references in log2 units)
  P.out_scale = ls.out_scale;
  P.n_items = n;
  for (int i = 0; i < n; ++i) P.items[i] = items[i];
  const int rpb = 256 / (ls.D / 4);
  const dim3 grid((unsigned)(n * ls.Hkv), (unsigned)(kTileRows / rpb)), block(256);
  int max_split = 0;
  for (int i = 0; i < n; ++i) max_split = items[i].nsplit > max_split ? items[i].nsplit : max_split;
  if (ls.D == 128)
    return max_split <= 4   ? launch_timed(kind, combine_kernel<128, 4, NI>, grid, block, st, P)
           : max_split <= 8 ? launch_timed(kind, combine_kernel<128, 8, NI>, grid, block, st, P)
                            : launch_timed(kind, combine_kernel<128, kMaxSplit, NI>, grid, block, st, P);
  return max_split <= 4   ? launch_timed(kind, combine_kernel<64, 4, NI>, grid, block, st, P)
         : max_split <= 8 ? launch_timed(kind, combine_kernel<64, 8, NI>, grid, block, st, P)
                          : launch_timed(kind, combine_kernel<64, kMaxSplit, NI>, grid, block, st, P);
}

int launch_combine(const LayerShape& ls, void* out, const float* part_o, const float* part_ml,
                   const CombineItem* items, int n_items, void* stream, bool timed) {
  hipStream_t st = (hipStream_t)stream;
  for (int base = 0; base < n_items; base += kMaxCombineItems) {
    const int n = n_items - base < kMaxCombineItems ? n_items - base : kMaxCombineItems;
    const int kind = timed ? 1 : -1;
    const int e = n <= kFewItems ? launch_combine_list<kFewItems>(ls, out, part_o, part_ml, items + base, n, st, kind)
                                 : launch_combine_list<kMaxCombineItems>(ls, out, part_o, part_ml, items + base, n, st, kind);
    if (e) return e;
  }
  return 0;
}

template <int NI>
static int launch_append_list(const LayerShape& ls, void* cache_k, void* cache_v, const void* k_new, const void* v_new,
                              const AppendItem* items, int n, hipStream_t st) {
  AppendParams<NI> P;
  P.cache_k = (uint16_t*)cache_k;
  P.cache_v = (uint16_t*)cache_v;
  P.k_new = (const uint16_t*)k_new;
  P.v_new = (const uint16_t*)v_new;
  P.row_granules = ls.Hkv * ls.D / 8;
  P.n_items = n;
  int mt = 0;
  for (int i = 0; i < n; ++i) {
    P.items[i] = items[i];
    if (items[i].n_tok > mt) mt = items[i].n_tok;
  }
  const dim3 grid((unsigned)n, (unsigned)((mt + kAppendTok - 1) / kAppendTok), 2), block(256);
  return launch_timed(2, kv_append_kernel<NI>, grid, block, st, P);
}

int launch_append(const LayerShape& ls, void* cache_k, void* cache_v, const void* k_new,
                  const void* v_new, const AppendItem* items, int n_items, int max_tok, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  (void)max_tok;
  for (int base = 0; base < n_items; base += kMaxAppendItems) {
    const int n = n_items - base < kMaxAppendItems ? n_items - base : kMaxAppendItems;
    const int e = n <= kFewItems ? launch_append_list<kFewItems>(ls, cache_k, cache_v, k_new, v_new, items + base, n, st)
                                 : launch_append_list<kMaxAppendItems>(ls, cache_k, cache_v, k_new, v_new, items + base, n, st);
    if (e) return e;
  }
  return 0;
}

template <int NI>
static int launch_append_fp8_list(const LayerShape& ls, void* cache_k, void* cache_v, const void* k_new, const void* v_new,
                                  float k_inv, float v_inv, const AppendItem* items, int n, hipStream_t st) {
  Append8Params<NI> P;
  P.cache_k = (uint8_t*)cache_k;
  P.cache_v = (uint8_t*)cache_v;
  P.k_new = (const uint16_t*)k_new;
  P.v_new = (const uint16_t*)v_new;
  P.k_inv = k_inv;
  P.v_inv = v_inv;
  P.Hkv = ls.Hkv;
  P.n_items = n;
  int64_t blocks = 0;   // 64-token blocks the longest run of this launch touches
  for (int i = 0; i < n; ++i) {
    const AppendItem& a = items[i];
    P.items[i] = a;
    const int64_t nb = (a.dst_row + a.n_tok - 1) / kKeyTile - a.dst_row / kKeyTile + 1;
    if (nb > blocks) blocks = nb;
  }
  if (blocks > 65535) return (int)hipErrorInvalidValue;
  const dim3 grid((unsigned)n, (unsigned)blocks, (unsigned)ls.Hkv);
  return ls.D == 128 ? launch_timed(2, kv_append_fp8_kernel<128, NI>, grid, dim3(256), st, P)
                     : launch_timed(2, kv_append_fp8_kernel<64, NI>, grid, dim3(128), st, P);
}

int launch_append_fp8(const LayerShape& ls, void* cache_k, void* cache_v, const void* k_new, const void* v_new,
                      float k_inv, float v_inv, const AppendItem* items, int n_items, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (ls.D != 128 && ls.D != 64) return (int)hipErrorInvalidValue;
  for (int base = 0; base < n_items; base += kMaxAppendItems) {
    const int n = n_items - base < kMaxAppendItems ? n_items - base : kMaxAppendItems;
    const int e = n <= kFewItems
                      ? launch_append_fp8_list<kFewItems>(ls, cache_k, cache_v, k_new, v_new, k_inv, v_inv, items + base, n, st)
                      : launch_append_fp8_list<kMaxAppendItems>(ls, cache_k, cache_v, k_new, v_new, k_inv, v_inv, items + base, n, st);
    if (e) return e;
  }
  return 0;
}

const char* hip_error_string(int err) { return hipGetErrorString((hipError_t)err); }

}  // namespace oppo

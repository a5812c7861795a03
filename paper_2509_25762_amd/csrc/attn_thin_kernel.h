// Chunked-prefill attention for passes that bring a few rows per sequence: the kernel (device code only; this file is
// included by kernels.hip inside namespace oppo, after the shared helpers and AttnParams).
//
// Such a pass is bound by reading the cache.  attn_fwd_kernel gives a wave 32 rows of the packed tile, so here one wave of
// its eight would do all the arithmetic while every tile of 64 keys, 32 KiB, makes the round from its request to a barrier
// that all eight wait at.  Here a tile has at most 32 rows (kThinRows) and the eight waves share out the piece's keys
// instead: wave w takes units (32 keys) w, w + 8, .. of the range, with no barrier among them, and holds one unit on its
// way while it works on another: 128 KiB in flight per compute unit.  The waves' results are merged in LDS at the end of
// the piece.  32/8 heads of 128, one row on 2048 .. 8192 keys, 64 sequences: 262 -> 245 us (5.7 TB/s; kv-heads whose rows share
// busier memory channels end last, the others' workgroups read at 6.9 TB/s).  Pieces, queues, partial results and the merge of split tiles are those of attn_fwd_kernel, and so are the
// operand layouts: S^T = K Q^T and O^T = V^T P^T in v_mfma_f32_16x16x32_bf16, a lane owning the query columns l16 and
// 16 + l16.  Keys go from memory into the A operand's registers as they are (a lane's 8 elements of a row are contiguous);
// values go through an area of LDS of the wave's own, from where the transposing read takes them.
template <int D, bool APPEND, int NI, int NCB>
__global__ __launch_bounds__(512) void attn_thin_kernel(const AttnParams<NI> P) {
  constexpr int NW = 8, NT = 64 * NW;
  constexpr int ROWS = 16 * NCB;           // packed rows of a tile, at most
  constexpr int UK = 32;                   // keys of a unit
  constexpr int NG = D / 8;                // 16-byte granules of a K/V row
  constexpr int KK = D / 32;               // k-steps of S^T
  constexpr int DB = D / 16;               // 16-row blocks of O^T
  constexpr int ROWB = D * 2;
  constexpr int RPV = 64 / NG;             // value rows a wave-wide load covers
  constexpr int NV = UK / RPV;             // such loads per unit
  constexpr int VSWZ_MASK = NG / 4 - 1;    // the values' swizzle in LDS is attn_fwd_kernel's
  // a wave's area: the values of a unit, and at the end of a piece its share of the output, fp32
  constexpr int AREA = ROWS * D * 4;
  static_assert(ROWS <= kThinRows && UK * ROWB <= AREA, "a unit's values fit the area");
  __shared__ __attribute__((aligned(1024))) unsigned char areas[NW][AREA];
  __shared__ float2 stats[NW][ROWS];  // (reference, row sum) of each wave's share
  __shared__ __attribute__((aligned(16))) AttnItem spiece[NI];
  static_assert(sizeof(areas) + sizeof(stats) + sizeof(spiece) <= 160 * 1024, "a compute unit's LDS");   // (all of it: 128, 960, 2)

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int l16 = lane & 15, grp = lane >> 4;
  const int Hq = P.Hq, Hkv = P.Hkv, G = P.G;
  const int kvh = blockIdx.x % Hkv, queue = blockIdx.x / Hkv;
  const int p_first = P.first[queue], p_last = P.first[queue + 1];
  if (p_first >= p_last) return;
  const float c = P.c;
  {
    const u32x4* src = (const u32x4*)(P.items + p_first);
    const int n16 = (p_last - p_first) * (int)(sizeof(AttnItem) / 16);
    for (int i = tid; i < n16; i += NT) ((u32x4*)spiece)[i] = src[i];
    __syncthreads();
  }
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
  // LDS accesses before it are through; nothing is said about global ones (the next unit is on its way)
  auto barrier = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };

  // ---- requests: this wave's units, piece after piece ---------------------------------
  const uint32_t row_bytes = (uint32_t)(Hkv * D) * 2u;
  const uintptr_t k_to_v = (uintptr_t)P.v - (uintptr_t)P.k;
  const uintptr_t kn_to_vn = APPEND ? (uintptr_t)P.v_new - (uintptr_t)P.k_new : 0;
  int r_piece = p_first, r_left = 0, r_cached = 0;   // keys of the piece from the next unit on; of them in the cache
  uintptr_t r_k = 0, r_kn = 0;                       // the unit's first row in k, and where it would be in k_new
  auto open = [&]() __attribute__((always_inline)) {   // the first piece, from r_piece on, with a unit for this wave
    for (; r_piece < p_last; ++r_piece) {
      const AttnItem a = piece(r_piece);
      const int first = a.k_begin + UK * wave;
      if (first >= a.k_end) continue;
      r_left = a.k_end - first;
      r_k = (uintptr_t)(P.k + (((int64_t)a.kv_row0 + first) * Hkv + kvh) * D);
      if (APPEND) {
        const int chunk0 = a.pos0 - tile_of(a) * P.TM;   // keys before the chunk are cached
        r_cached = chunk0 - first;
        r_kn = (uintptr_t)(P.k_new + (((int64_t)a.q_row0 - (a.pos0 - chunk0) - r_cached) * Hkv + kvh) * D);
      }
      return;
    }
  };
  bf16x8 kf[2][KK];   // K fragments of the unit: [16-key block][k-step]
  u32x4 vr[NV];       // its value rows: lane (row lane / NG of RPV, granule lane % NG)
  auto request = [&]() __attribute__((always_inline)) {
    if (r_piece >= p_last) return;
    const int last = r_left - 1;   // rows past the range repeat the last key
    const bool mixed = APPEND && r_cached > 0 && r_cached < UK && r_cached <= last;
    const bool all_new = APPEND && r_cached <= 0;
    const uintptr_t bk = all_new ? r_kn : r_k, bv = bk + (all_new ? kn_to_vn : k_to_v);
    int ln = lane;
    asm volatile("" : "+v"(ln));   // (offsets are formed here, not kept in registers)
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const int row = min(16 * b + (ln & 15), last);
      const uint32_t off = (uint32_t)row * row_bytes + (uint32_t)(ln >> 4) * 16u;
      const uintptr_t from = mixed && row >= r_cached ? r_kn : bk;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) kf[b][kk] = *(const bf16x8*)(from + off + kk * 64);
    }
#pragma unroll
    for (int i = 0; i < NV; ++i) {
      const int row = min(RPV * i + ln / NG, last);
      const uint32_t off = (uint32_t)row * row_bytes + (uint32_t)(ln % NG) * 16u;
      vr[i] = *(const u32x4*)((mixed && row >= r_cached ? r_kn + kn_to_vn : bv) + off);
    }
    r_left -= UK * NW;
    r_k += (uintptr_t)(UK * NW) * row_bytes;
    if (APPEND) {
      r_kn += (uintptr_t)(UK * NW) * row_bytes;
      r_cached -= UK * NW;
    }
    if (r_left <= 0) {
      ++r_piece;
      open();
    }
  };

  typedef __attribute__((address_space(3))) unsigned char* lds_ptr;
  typedef const __attribute__((address_space(3))) unsigned char* lds_cptr;
  const uint32_t area = lds_addr_of(&areas[0][0]) + (uint32_t)wave * AREA;
  lds_cptr vptr[DB / 2];   // V^T fragments of d-blocks 2 i (and 2 i + 1, 32 bytes on), keys 4 grp .. of the unit
#pragma unroll
  for (int i = 0; i < DB / 2; ++i) {
    const int vrow = 4 * grp + (l16 >> 2), lg = 4 * i + ((l16 & 3) >> 1);
    vptr[i] = (lds_cptr)(uintptr_t)(area + (uint32_t)(vrow * ROWB + ((lg ^ ((vrow & VSWZ_MASK) << 2)) * 16) + (l16 & 1) * 8));
  }
  bf16x8 ones;
#pragma unroll
  for (int e = 0; e < 8; ++e) ones[e] = (__bf16)1.0f;

  bf16x8 qf[NCB][KK];
  auto load_q = [&](const AttnItem& a) __attribute__((always_inline)) {
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      const int row = min(16 * cb + l16, tokens_of(a) * G - 1);   // (columns without a row repeat the last one)
      const int t = (int)(((uint32_t)row * P.g_magic) >> 16);     // row / G
      const uint16_t* src = P.q + ((int64_t)(a.q_row0 + t) * Hq + kvh * G + row - t * G) * D + grp * 8;
#pragma unroll
      for (int kk = 0; kk < KK; ++kk) qf[cb][kk] = *(const bf16x8*)(src + kk * 32);
    }
  };

  // A column's reference is moved when a weight would exceed 2^24 (as in attn_fwd_kernel relative precision does not
  // depend on it): always at its first visible keys, otherwise almost never.
  constexpr float kMaxLog2Weight = 24.0f;
  f32x4 o[DB][NCB];
  float m_run[NCB], l_run[NCB], mc[NCB];   // l_run: row sums over the rounded weights, by MFMAs with a matrix of ones

  AttnItem it = piece(p_first);
  open();
  request();
  load_q(it);
  for (int p = p_first;;) {
    const int n_rows = tokens_of(it) * G;
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      m_run[cb] = -1e30f;
      mc[cb] = -1e30f * c;
      l_run[cb] = 0.f;
#pragma unroll
      for (int db = 0; db < DB; ++db) o[db][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    const int min_lim = min(it.pos0, it.k_end - 1);
    for (int key0 = it.k_begin + UK * wave; key0 < it.k_end; key0 += UK * NW) {
      // the unit's values into the wave's area, its scores, and then the request of the next unit into the same registers
#pragma unroll
      for (int i = 0; i < NV; ++i) {
        const int r = RPV * i + lane / NG;
        *(__attribute__((address_space(3))) u32x4*)(lds_ptr)(uintptr_t)(
            area + (uint32_t)(r * ROWB + (((lane % NG) ^ ((r & VSWZ_MASK) << 2)) * 16))) = vr[i];
      }
      f32x4 s[2][NCB];
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
          s[b][cb] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int kk = 0; kk < KK; ++kk)
            s[b][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[b][kk], qf[cb][kk], s[b][cb], 0, 0, 0);
        }
      asm volatile("" ::: "memory");
      request();
      if (key0 + UK - 1 > min_lim) {
        int ln = lane;
        asm volatile("" : "+v"(ln));   // (the limits are formed here, not kept in registers)
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
          // last key the lane's column may see, minus 4 * grp
          const int t = (int)(((uint32_t)(16 * cb + (ln & 15)) * P.g_magic) >> 16);
          const int lim = min(it.pos0 + min(t, tokens_of(it) - 1), it.k_end - 1) - 4 * (ln >> 4);
#pragma unroll
          for (int e = 0; e < 8; ++e)
            if (key0 + 16 * (e / 4) + e % 4 > lim) s[e / 4][cb][e % 4] = -INFINITY;
        }
      }
      float mx[NCB];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
        const f32x4 &x = s[0][cb], &y = s[1][cb];
        mx[cb] = fmaxf(fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])), fmaxf(fmaxf(y[0], y[1]), fmaxf(y[2], y[3])));
      }
      float top = fmaf(mx[0], c, -mc[0]);
      if (NCB == 2) top = fmaxf(top, fmaf(mx[NCB - 1], c, -mc[NCB - 1]));
      if (__any(top > kMaxLog2Weight)) {
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) {
          float m = fmaxf(mx[cb], swap_halves(mx[cb]));
          m = fmaxf(m_run[cb], fmaxf(m, __shfl_xor(m, 16)));
          const float alpha = fast_exp2((m_run[cb] - m) * c);
          m_run[cb] = m;
          mc[cb] = m * c;
          l_run[cb] *= alpha;
#pragma unroll
          for (int db = 0; db < DB; ++db) o[db][cb] *= alpha;
        }
      }
      union { bf16x2 h[4]; bf16x8 v; } pf[NCB];
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) {
#pragma unroll
        for (int e = 0; e < 8; ++e) pf[cb].h[e / 2][e % 2] = (__bf16)fast_exp2(fmaf(s[e / 4][cb][e % 4], c, -mc[cb]));
        l_run[cb] += __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[cb].v, f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0)[0];
      }
#pragma unroll
      for (int db = 0; db < DB; ++db) {
        lds_cptr vp = vptr[db / 2] + (db % 2) * 32;
        union { struct { s16x4 a, b; } h; bf16x8 v; } cat;
        cat.h.a = lds_read_tr16_l(vp);
        cat.h.b = lds_read_tr16_l(vp + 16 * ROWB);
#pragma unroll
        for (int cb = 0; cb < NCB; ++cb) o[db][cb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(cat.v, pf[cb].v, o[db][cb], 0, 0, 0);
      }
      asm volatile("" ::: "memory");   // (the next unit's values overwrite these)
    }

    // ---- merge of the eight waves' shares ---------------------------------------------
    const AttnItem done = it;
    const bool more = p + 1 < p_last;
    if (more) {
      it = piece(p + 1);
      load_q(it);
    }
    if (grp == 0) {
#pragma unroll
      for (int cb = 0; cb < NCB; ++cb) stats[wave][16 * cb + l16] = float2{m_run[cb], l_run[cb]};
    }
    barrier();
#pragma unroll
    for (int cb = 0; cb < NCB; ++cb) {
      if (16 * cb >= n_rows) continue;
      float m = m_run[cb];
#pragma unroll
      for (int w = 0; w < NW; ++w) m = fmaxf(m, stats[w][16 * cb + l16].x);
      const float f = fast_exp2((m_run[cb] - m) * c);   // 0 for a wave that saw no key of the column (unless none did)
      // 16-byte granule g of row r lies at place g ^ (r % 16) of the row: the 16 rows that lanes write at a time
      // would otherwise share their banks
#pragma unroll
      for (int db = 0; db < DB; ++db)
        *(__attribute__((address_space(3))) f32x4*)(lds_ptr)(uintptr_t)(
            area + (uint32_t)((16 * cb + l16) * D * 4 + ((4 * db + grp) ^ l16) * 16)) = o[db][cb] * f;
    }
    barrier();
    for (int idx = tid; idx < n_rows * (D / 4); idx += NT) {
      const int row = idx / (D / 4), d4 = idx % (D / 4);
      float m = -INFINITY, l = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) m = fmaxf(m, stats[w][row].x);
      f32x4 x = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float2 ml = stats[w][row];
        l += ml.y * fast_exp2((ml.x - m) * c);
        x += *(const f32x4*)&areas[w][row * D * 4 + (d4 ^ (row % 16)) * 16];
      }
      if (done.part < 0) {
        const float inv = 1.0f / l;
        const int t = (int)(((uint32_t)row * P.g_magic) >> 16);
        bf16x4 y;
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = (__bf16)(x[e] * inv);
        *(bf16x4*)(P.out + ((int64_t)(done.q_row0 + t) * Hq + kvh * G + row - t * G) * D + 4 * d4) = y;
      } else {
        const int64_t slot = ((int64_t)done.part * Hkv + kvh) * kTileRows + row;
        *(f32x4*)(P.part_o + slot * D + 4 * d4) = x;
        if (d4 == 0) *(float2*)(P.part_ml + slot * 2) = float2{m, l};
      }
    }
    if (APPEND && done.k_begin == 0) {   // the piece that starts the tile's key range moves its token rows into the cache
      for (int idx = tid; idx < tokens_of(done) * NG; idx += NT) {
        const int row = idx / NG, g = idx % NG;
        const int64_t src = (((int64_t)done.q_row0 + row) * Hkv + kvh) * D + g * 8;
        const int64_t dst = (((int64_t)done.kv_row0 + done.pos0 + row) * Hkv + kvh) * D + g * 8;
        const u32x4 a = *(const u32x4*)(P.k_new + src), b = *(const u32x4*)(P.v_new + src);
        *(u32x4*)(P.k + dst) = a;
        *(u32x4*)(P.v + dst) = b;
      }
    }
    if (!more) break;
    ++p;
    barrier();   // the areas are free again
  }
}

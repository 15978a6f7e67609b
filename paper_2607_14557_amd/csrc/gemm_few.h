// bf16 GEMM for launches of few tiles: C[M,N] = A[M,K] * B[N,K]^T with the
// epilogues of gemm_bf16.hip (included there).
//
// With few rows (a cached step, one request, a small model) 256x256 tiles
// leave most CUs idle.  So a workgroup takes a 128x64 tile (or 128x128) and its
// four waves a quarter of K each, summed in LDS: no barrier in the loop, and
// where the tiles do not fill the chip K is split further over workgroups, whose
// sums go through memory, 32 or 64 KiB a unit, added by the last unit to arrive
// in the same launch.  Where the 128x128 tiles are one round's worth or a little
// more and K is long, 256x256 tiles split over K with a second launch for the
// sums load fewer operand bytes a flop and win (few_us has each form's cost).
//
// What bounds it: at one tile row the weights from HBM (d 4096, 97 rows: gate/up
// 201 MB in 52 us, 3.9 TB/s), at small d the launch and one tile's chain, beyond
// a few tile rows the operand loads from L2 (60-75 GB/s a CU; 128x64 tiles load
// three times the bytes a flop of 256x256 ones), where the larger tiles take
// over.  Times in us, 256x256 tiles alone split over K with a second launch or
// in halves, and now, QKV / O / gate-up / down:
//   d 4096, 97 rows     38 / 25 / 63 / 43    ->  32 / 18 / 50 / 34
//   d 4096, 890 rows    87 / 53 / 160 / 101  ->  86 / 43 / 159 / 102; O and down
//                       under a bound of 2304 rows 65 / 163  ->  43 / 103
//   d 2048, 1280 rows   34 / 33 / 50 / 48    ->  35 / 22 / 50 / 41
//   d 512, 1137 rows    26 / 21 / 25 / 23    ->  10 / 10 / 11 / 11
#pragma once

namespace seer {

constexpr int FEW_ROWS = 128;
constexpr int FEW_STAGE = 64 * ROW_BYTES;           // bytes of one wave's A stage: 64 rows of 64 K values
constexpr int kScopeAgent = 16;                     // buffer cache policy sc1: coherent across the XCDs

// Buffer records of a step `left` past the last (negative: a real step): -1
// (all) or 0 (none).  In scalar registers: a select compiles to a vector one,
// which puts the descriptor in vector registers and a loop around every load.
__device__ __forceinline__ int few_records(int left) {
  asm("s_ashr_i32 %0, %0, 31" : "+s"(left) : : "scc");
  return left;
}

// The epilogue of one wave's 32 rows x 64 packed columns: `a0` and `a1` are the
// column blocks wcol and wcol + 32 (register r: row row0 + lane%32, column
// 8 (r/4) + 4 (lane/32) + r%4 of the block).
template <int EPI>
struct FewEpilogue {
  static constexpr bool kGlu = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_COUNT;
  static constexpr bool kPair = EPI == EPI_RESID_PAIR;
  static constexpr bool kRes = EPI == EPI_RESID_SPLIT || kPair;
  static constexpr bool kScale = EPI == EPI_SCALE || EPI == EPI_SCALE_ROPE;
  float sc = 1.0f;
  int pos = 0;
  u32x4_t r[kRes ? 4 : 1], r2[kPair ? 4 : 1];

  // what the epilogue reads besides the sums, requested ahead of its use
  __device__ __forceinline__ void fetch(const GemmParams& p, int M, int row0, int wcol) {
    const int lane = threadIdx.x & 63, fhalf = lane >> 5;
    int row = row0 + (lane & 31);
    row = row < M ? row : M - 1;                    // rows past M are never stored
    if constexpr (kScale || kGlu) sc = p.rs[row];
    if constexpr (EPI == EPI_SCALE_ROPE) pos = p.rope_pos[row];
    if constexpr (kRes) {
      const uint16_t* rb = static_cast<const uint16_t*>(p.R) + (size_t)row * p.ldr + wcol + 8 * fhalf;
#pragma unroll
      for (int t = 0; t < 4; ++t) r[t] = *reinterpret_cast<const u32x4_t*>(rb + 16 * t);
    }
    if constexpr (kPair) {
      const uint16_t* rb = static_cast<const uint16_t*>(p.R2) + (size_t)row * p.ldr + wcol + 8 * fhalf;
#pragma unroll
      for (int t = 0; t < 4; ++t) r2[t] = *reinterpret_cast<const u32x4_t*>(rb + 16 * t);
    }
  }

  // columns 8q..8q+7 of lanes l and columns 8q+8..8q+15 of lanes l + 32 from the quads (q, q+1)
  static __device__ __forceinline__ u32x4_t join(uint2 a, uint2 b) {
    const u32x2_t sx = __builtin_amdgcn_permlane32_swap(a.x, b.x, false, false);
    const u32x2_t sy = __builtin_amdgcn_permlane32_swap(a.y, b.y, false, false);
    return u32x4_t{sx[0], sy[0], sx[1], sy[1]};
  }
  static __device__ __forceinline__ void split(u32x4_t w, uint2& a, uint2& b) {
    const u32x2_t sx = __builtin_amdgcn_permlane32_swap(w[0], w[2], false, false);
    const u32x2_t sy = __builtin_amdgcn_permlane32_swap(w[1], w[3], false, false);
    a.x = sx[0]; a.y = sy[0];
    b.x = sx[1]; b.y = sy[1];
  }
  static __device__ __forceinline__ void add4(float* v, uint2 w) {
    v[0] += __uint_as_float(w.x << 16);
    v[1] += __uint_as_float(w.x & 0xffff0000u);
    v[2] += __uint_as_float(w.y << 16);
    v[3] += __uint_as_float(w.y & 0xffff0000u);
  }

  __device__ __forceinline__ void apply(const GemmParams& p, int M, int row0, int wcol, f32x16_t a0, f32x16_t a1) {
    const int lane = threadIdx.x & 63, fhalf = lane >> 5;
    const int row = row0 + (lane & 31);
    const bool ok = row < M;
    const int cq = 4 * fhalf;
    if constexpr (kGlu) {
      int nz = 0;
      uint2 pk[4];
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        float a[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          a[e] = silu(a0[4 * q + e] * sc) * (a1[4 * q + e] * sc);
          if constexpr (EPI == EPI_SWIGLU_COUNT) nz += __float_as_uint(fabsf(a[e]) - p.eps) >> 31;
        }
        pk[q].x = pack_bf2(a[0], a[1]);
        pk[q].y = pack_bf2(a[2], a[3]);
      }
      // the swaps are wave-wide: every lane takes part, rows past M store nothing
      const u32x4_t w0 = join(pk[0], pk[1]), w1 = join(pk[2], pk[3]);
      uint16_t* cw = static_cast<uint16_t*>(p.C) + (size_t)row * p.ldc + (wcol >> 1) + 8 * fhalf;
      if (ok) {
        *reinterpret_cast<u32x4_t*>(cw) = w0;
        *reinterpret_cast<u32x4_t*>(cw + 16) = w1;
      }
      if constexpr (EPI == EPI_SWIGLU_COUNT) {
        nz += __shfl_xor(nz, 32, kWave);
        if (ok && fhalf == 0) atomicAdd(p.cnt + row, nz);
      }
    } else {
      // below perm_col1 the two blocks are features (32 h, 64 + 32 h) of one
      // 128-wide head, h = the 64-column half (qk_packed_row)
      const bool perm = kScale && wcol < p.perm_col1;
      const int hsel = (wcol >> 6) & 1;
      if constexpr (EPI == EPI_SCALE_ROPE) {
        if (wcol < p.rope_col1) {
          const double dp = (double)pos;
#pragma unroll
          for (int e = 0; e < 16; ++e) {
            double rv = dp * p.rope_freq[32 * hsel + 8 * (e >> 2) + cq + (e & 3)];
            rv -= floor(rv);
            const float t = (float)rv;              // revolutions in [0, 1)
            const float sn = __builtin_amdgcn_sinf(t), cs = __builtin_amdgcn_cosf(t);
            const float x = a0[e], y = a1[e];
            a0[e] = x * cs - y * sn;
            a1[e] = y * cs + x * sn;
          }
        }
      }
      const bool to_f16 = kScale && p.f16_col0 > 0 && wcol >= p.f16_col0;
      float f16_max = 0.0f;
#pragma unroll
      for (int j = 0; j < 2; ++j) {
        uint2 rv[4], rv2[4];
        if constexpr (kRes) {
          split(r[2 * j], rv[0], rv[1]);
          split(r[2 * j + 1], rv[2], rv[3]);
        }
        if constexpr (kPair) {
          split(r2[2 * j], rv2[0], rv2[1]);
          split(r2[2 * j + 1], rv2[2], rv2[3]);
        }
        uint2 pk[4], lo[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          float v[4];
#pragma unroll
          for (int e = 0; e < 4; ++e) v[e] = (j ? a1[4 * q + e] : a0[4 * q + e]) * (kScale ? sc : 1.0f);
          if constexpr (kRes) add4(v, rv[q]);
          if constexpr (kPair) add4(v, rv2[q]);
          if (kScale && to_f16) {
#pragma unroll
            for (int e = 0; e < 4; ++e) f16_max = fmaxf(f16_max, fabsf(v[e]));
            pk[q].x = pack_h2(v[0], v[1]);
            pk[q].y = pack_h2(v[2], v[3]);
          } else {
            pk[q].x = pack_bf2(v[0], v[1]);
            pk[q].y = pack_bf2(v[2], v[3]);
          }
          if constexpr (EPI == EPI_RESID_SPLIT) {
            // v - bf16(v) is exact in fp32; its bf16 rounding leaves ~2^-17 of v
            lo[q].x = pack_bf2(v[0] - __uint_as_float(pk[q].x << 16), v[1] - __uint_as_float(pk[q].x & 0xffff0000u));
            lo[q].y = pack_bf2(v[2] - __uint_as_float(pk[q].y << 16), v[3] - __uint_as_float(pk[q].y & 0xffff0000u));
          }
        }
        const int col = (perm ? (wcol & ~127) + 32 * (hsel + 2 * j) : wcol + 32 * j) + 8 * fhalf;
        const u32x4_t w0 = join(pk[0], pk[1]), w1 = join(pk[2], pk[3]);
        uint16_t* cw = static_cast<uint16_t*>(p.C) + (size_t)row * p.ldc + col;
        if (ok) {
          *reinterpret_cast<u32x4_t*>(cw) = w0;
          *reinterpret_cast<u32x4_t*>(cw + 16) = w1;
        }
        if constexpr (EPI == EPI_RESID_SPLIT) {
          const u32x4_t l0 = join(lo[0], lo[1]), l1 = join(lo[2], lo[3]);
          uint16_t* cl = static_cast<uint16_t*>(p.C2) + (size_t)row * p.ldc + col;
          if (ok) {
            *reinterpret_cast<u32x4_t*>(cl) = l0;
            *reinterpret_cast<u32x4_t*>(cl + 16) = l1;
          }
        }
      }
      if constexpr (kScale) {
        if (to_f16 && p.status && ok && f16_max > 65504.0f) atomicOr(p.status, SEER_STATUS_V_RANGE);
      }
    }
  }
};

// One 128 x (32 NJ) tile over the 64-wide K tiles [k0, k1), split `sp` of `S`
// of its K range; r is the tile's counter and partial slot.  Wave w multiplies
// the whole tile over the K tiles k0 + w, k0 + w + 4, ..., so the loop has no
// barrier: A goes to an LDS ring of the wave's own with direct-to-LDS loads,
// a half tile (64 rows, whole 128-byte lines) a stage, three stages ahead; B
// (fragment-major) straight to registers, a K tile ahead.
template <int EPI, int NJ>
__device__ __forceinline__ void few_tile(const GemmParams& p, uint8_t* st0, uint8_t* st1, uint8_t* st2, uint8_t* st3,
                                         int* s_last, int M, int m0, int n0, int k0, int k1, int sp, int S, int r) {
  constexpr int NI = FEW_ROWS / 32;
  const int lane = threadIdx.x & 63;
  const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int fr = lane & 31, fhalf = lane >> 5;
  const int n = k1 - k0 - wv > 0 ? (k1 - k0 - wv + 3) >> 2 : 0;   // K tiles of this wave

  // A: instruction i of half h fills rows 8 i .. +7 of the stage (128 bytes
  // each) with tile rows 64 h + 8 i ..; lane l lands at row 8 i + l/8, slot l%8
  // and fetches the 16-byte chunk that the swizzle puts there.  Rows past M
  // re-read row M-1 (never stored).
  uint32_t a_src[16];
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int row = 8 * i + (lane >> 3);
    int ga = m0 + row;
    ga = ga < M ? ga : M - 1;
    a_src[i] = (uint32_t)ga * (uint32_t)p.lda * 2u + (uint32_t)(((lane & 7) ^ swz(row)) << 4);
  }
  uint32_t b_blk[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) b_blk[j] = (uint32_t)((n0 >> 5) + j) * (uint32_t)(p.K >> 4) * 1024u;
  const int b_lane = lane * 16;
  const int a_row = wv * FEW_STAGE + fr * 128;
  const int fsw = swz(fr);

  f32x16_t acc[NI][NJ];
#pragma unroll
  for (int i = 0; i < NI; ++i)
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.0f;
  u32x4_t bq[2][4][NJ];
  bf16x8_t af[2][2];

  // Quarter Q of the loads of A half H of this wave's K tile T into stage ST,
  // and quarter Q of B half HB (slices 2 HB, 2 HB + 1) of its K tile TB into
  // set BS.  A tile past the last has a descriptor of no records: its loads
  // return zeros without touching memory.
#define FEW_A(ST, T, H, Q)                                                                                        \
  {                                                                                                               \
    const __amdgpu_buffer_rsrc_t ra_ =                                                                            \
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.A), 0, few_records((T) - n), 0x00020000);           \
    const uint32_t ko_ = (uint32_t)(k0 + wv + 4 * (T)) * 128u;                                                    \
    _Pragma("unroll") for (int i = 2 * (Q); i < 2 * (Q) + 2; ++i)                                                 \
      __builtin_amdgcn_raw_ptr_buffer_load_lds(ra_, (lds_void_t*)((ST) + wv * FEW_STAGE + i * 1024), 16,          \
                                               a_src[8 * (H) + i], ko_, 0, 0);                                    \
  }
#define FEW_B(BS, TB, KS)                                                                                         \
  {                                                                                                               \
    const __amdgpu_buffer_rsrc_t rb_ =                                                                            \
        __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p.B), 0, few_records((TB) - n), 0x00020000);          \
    const uint32_t ko_ = (uint32_t)(k0 + wv + 4 * (TB)) * 4096u;                                                  \
    _Pragma("unroll") for (int j = 0; j < NJ; ++j)                                                                \
      bq[BS][KS][j] = __builtin_amdgcn_raw_buffer_load_b128(rb_, b_lane + 1024 * (KS), b_blk[j] + ko_, 0);        \
  }
#define FEW_READ(ST, KS, BUF)                                                                                     \
  _Pragma("unroll") for (int i = 0; i < 2; ++i)                                                                   \
    af[BUF][i] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(                                  \
        (ST) + a_row + i * 4096 + (((2 * (KS) + fhalf) ^ fsw) << 4)));
  // Half H of K tile T out of stage SC and B set BS; meanwhile the half three
  // on goes to stage SF (whose fragments were consumed in the step before) and
  // half the slices of tile T + 1 to the other set.  Before the
  // look-ahead read of the next half (stage SN, loaded two steps ago) its
  // loads must have landed: what was issued since, the last step's A and half
  // set of B and this one's but its last quarter of A, may be in flight.
#define FEW_STEP(T, H, SC, SN, SF, BS)                                                                            \
  {                                                                                                               \
    _Pragma("unroll") for (int ks = 0; ks < 4; ++ks) {                                                            \
      if (ks == 3) {                                                                                              \
        __builtin_amdgcn_s_waitcnt(waitcnt_imm(8 + 2 * NJ + 6 + 2 * NJ, 15));                                     \
        __builtin_amdgcn_sched_barrier(0);                                                                        \
      }                                                                                                           \
      FEW_READ(ks < 3 ? SC : SN, (ks + 1) & 3, (ks + 1) & 1);                                                     \
      FEW_A(SF, (T) + 1 + (H), (H) ^ 1, ks);                                                                      \
      if (ks < 2) FEW_B((BS) ^ 1, (T) + 1, 2 * (H) + ks);                                        \
      _Pragma("unroll") for (int i = 0; i < 2; ++i)                                                               \
        _Pragma("unroll") for (int j = 0; j < NJ; ++j)                                                            \
          acc[2 * (H) + i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(                                          \
              __builtin_bit_cast(bf16x8_t, bq[BS][ks][j]), af[ks & 1][i], acc[2 * (H) + i][j], 0, 0, 0);          \
      __builtin_amdgcn_sched_barrier(0);                                                                          \
    }                                                                                                             \
  }

  // in the steps' order, so that their wait covers the first one too: younger
  // than st1's loads are half a set of B, st2's and the first step's
  _Pragma("unroll") for (int q = 0; q < 4; ++q) FEW_A(st0, 0, 0, q);
  _Pragma("unroll") for (int q = 0; q < 2; ++q) FEW_B(0, 0, q);
  __builtin_amdgcn_sched_barrier(0);
  _Pragma("unroll") for (int q = 0; q < 4; ++q) FEW_A(st1, 0, 1, q);
  __builtin_amdgcn_sched_barrier(0);
  _Pragma("unroll") for (int q = 2; q < 4; ++q) FEW_B(0, 0, q);
  _Pragma("unroll") for (int q = 0; q < 4; ++q) FEW_A(st2, 1, 0, q);
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(16 + 4 * NJ, 15));
  __builtin_amdgcn_sched_barrier(0);
  if (n > 0) {
    FEW_READ(st0, 0, 0);
#define FEW_TILE0(T) FEW_STEP(T, 0, st0, st1, st3, 0); FEW_STEP(T, 1, st1, st2, st0, 0);
#define FEW_TILE1(T) FEW_STEP(T, 0, st2, st3, st1, 1); FEW_STEP(T, 1, st3, st0, st2, 1);
    int t = 0;
    for (; t + 2 <= n; t += 2) {
      FEW_TILE0(t);
      FEW_TILE1(t + 1);
    }
    if constexpr (NJ == 2) {                        // an even n otherwise: see gemm_bf16_split_kernel
      if (t < n) { FEW_TILE0(t); }
    }
#undef FEW_TILE0
#undef FEW_TILE1
  }
#undef FEW_A
#undef FEW_B
#undef FEW_READ
#undef FEW_STEP
  __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));    // no load into the stages is left in flight

  // ---- sum the four waves: wave w ends with rows 32 w .. +31, added in wave
  // order through LDS ----------------------------------------------------------
  const int row0 = m0 + 32 * wv;
  FewEpilogue<EPI> epi[NJ / 2];
  if (S == 1 && row0 < M) {
#pragma unroll
    for (int g = 0; g < NJ / 2; ++g) epi[g].fetch(p, M, row0, n0 + 64 * g);
  }
  f32x16_t own[NJ];
  uint8_t* const st[4] = {st0, st1, st2, st3};
  constexpr int PER = 8 / NJ;                       // owners per round: 24 KiB of each stage array in use
#pragma unroll
  for (int o0 = 0; o0 < 4; o0 += PER) {
    __syncthreads();
#pragma unroll
    for (int o = o0; o < o0 + PER; ++o) {
      if (wv == o) continue;
      const int slot = (wv - (wv > o ? 1 : 0)) * 8192 + lane * 16;
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          *reinterpret_cast<f32x4_t*>(st[(o - o0) * (NJ / 2) + j / 2] + slot + ((j & 1) * 4 + q) * 1024) =
              f32x4_t{acc[o][j][4 * q], acc[o][j][4 * q + 1], acc[o][j][4 * q + 2], acc[o][j][4 * q + 3]};
    }
    __syncthreads();
#pragma unroll
    for (int o = o0; o < o0 + PER; ++o) {
      if (wv != o) continue;
#pragma unroll
      for (int v = 0; v < 4; ++v)
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          f32x16_t c = acc[o][j];
          if (v != o) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              const f32x4_t x = *reinterpret_cast<const f32x4_t*>(
                  st[(o - o0) * (NJ / 2) + j / 2] + (v - (v > o ? 1 : 0)) * 8192 + lane * 16 + ((j & 1) * 4 + q) * 1024);
#pragma unroll
              for (int e = 0; e < 4; ++e) c[4 * q + e] = x[e];
            }
          }
          if (v == 0) own[j] = c;
          else own[j] += c;
        }
    }
  }

  // ---- sum the K splits: every split leaves its sums in the scratch, the last
  // to arrive adds them in split order ------------------------------------------
  if (S > 1) {
    constexpr int BLK = NJ * 4096;                  // bytes of one wave's sums
    const __amdgpu_buffer_rsrc_t rp = __builtin_amdgcn_make_buffer_rsrc(p.partial, 0, -1, 0x00020000);
    auto at = [&](int s) { return (uint32_t)((r * S + s) * 4 + wv) * (uint32_t)BLK; };
    if (row0 < M) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q)
          __builtin_amdgcn_raw_buffer_store_b128(
              __builtin_bit_cast(u32x4_t, f32x4_t{own[j][4 * q], own[j][4 * q + 1], own[j][4 * q + 2], own[j][4 * q + 3]}),
              rp, lane * 16 + (j * 4 + q) * 1024, at(sp), kScopeAgent);
    }
    __builtin_amdgcn_s_waitcnt(waitcnt_imm(0, 0));  // this wave's sums are visible to every XCD
    __syncthreads();
    if (threadIdx.x == 0) *s_last = atomicAdd(p.counters + r, 1) == S - 1;
    __syncthreads();
    if (!*s_last || row0 >= M) return;
#pragma unroll
    for (int g = 0; g < NJ / 2; ++g) epi[g].fetch(p, M, row0, n0 + 64 * g);
    f32x16_t tot[NJ];
    for (int s0 = 0; s0 < S; s0 += 2) {
      u32x4_t w[2][NJ * 4];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int s = s0 + u < S ? s0 + u : S - 1;
#pragma unroll
        for (int k = 0; k < NJ * 4; ++k)
          w[u][k] = __builtin_amdgcn_raw_buffer_load_b128(rp, lane * 16 + k * 1024, at(s), kScopeAgent);
      }
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        if (s0 + u >= S) continue;
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const f32x4_t x = __builtin_bit_cast(f32x4_t, w[u][j * 4 + q]);
#pragma unroll
            for (int e = 0; e < 4; ++e) tot[j][4 * q + e] = s0 + u == 0 ? x[e] : tot[j][4 * q + e] + x[e];
          }
      }
    }
#pragma unroll
    for (int j = 0; j < NJ; ++j) own[j] = tot[j];
  }
  if (row0 >= M) return;
#pragma unroll
  for (int g = 0; g < NJ / 2; ++g) epi[g].apply(p, M, row0, n0 + 64 * g, own[2 * g], own[2 * g + 1]);
}

// Unit u over the launch's tiles_m x tiles_n tiles: whole tiles in full rounds,
// then the others, their K split over S units each.  Whether and how a tile's K
// is split follows from its place among all tiles, also when only the tiles of a
// row-tile list are computed, so that a row's result does not depend on the list.
template <int EPI, int NJ>
__device__ __forceinline__ void run_unit_few(const GemmParams& p, uint8_t* st0, uint8_t* st1, uint8_t* st2, uint8_t* st3,
                                             int* s_last, int M, int tiles_m, bool k_split, int u) {
  auto uni = [](int v) { return __builtin_amdgcn_readfirstlane(v); };   // keeps the buffer descriptors scalar
  const int tiles_n = p.N / (32 * NJ), tiles = tiles_m * tiles_n;
  const int full = few_full(p.n_units, tiles), rem = tiles - full;
  const int splits = k_split ? few_k_splits(p.n_units, rem, p.K / BK) : 1;
  int tm, tn, sp = 0, r = 0, S = 1;
  if (p.mtiles) {
    // first every listed tile, whole or its split 0; then the other splits of
    // all split tiles, those not in the list exiting
    // of 2 listed half tiles each, but the last may start past the last row
    const int cnt = p.mtiles[0];
    const int listed = 2 * cnt - (cnt > 0 && 2 * p.mtiles[cnt] + 1 >= tiles_m ? 1 : 0);
    if (u < listed * tiles_n) {
      raster(xcd_remap(u, listed * tiles_n), listed, tiles_n, tm, tn);
      tm = 2 * p.mtiles[1 + (tm >> 1)] + (tm & 1);
      const int lid = raster_of(tm, tn, tiles_m, tiles_n);
      if (lid >= full) { r = lid - full; S = splits; }
    } else {
      const int v = u - listed * tiles_n;
      if (v >= rem * (splits - 1)) return;
      S = splits;
      sp = 1 + v / rem;
      r = v % rem;
      raster(full + r, tiles_m, tiles_n, tm, tn);
      bool found = false;
      for (int k = 0; k < cnt; ++k) found |= p.mtiles[1 + k] == tm >> 1;
      if (!found) return;
    }
  } else if (u < full) {
    raster(xcd_remap(u, full), tiles_m, tiles_n, tm, tn);
  } else {
    if (u >= full + rem * splits) return;
    // split-major, so that the units of one XCD walk the same K range
    const int v = xcd_remap(u - full, rem * splits);
    S = splits;
    sp = S > 1 ? v / rem : 0;
    r = v - sp * rem;
    raster(full + r, tiles_m, tiles_n, tm, tn);
  }
  const int m0 = tm * FEW_ROWS;
  if (m0 >= M) return;
  // the wide tile's loop takes two K tiles a wave: splits of whole 512-wide runs
  constexpr int RUN = NJ == 2 ? 1 : 8;
  const int runs = p.K / BK / RUN;
  const int k0 = S > 1 ? runs * sp / S * RUN : 0, k1 = S > 1 ? runs * (sp + 1) / S * RUN : runs * RUN;
  few_tile<EPI, NJ>(p, st0, st1, st2, st3, s_last, uni(M), uni(m0), uni(tn * 32 * NJ), uni(k0), uni(k1), uni(sp), uni(S),
                    uni(r));
}

// The run of the rule for tiles_m row tiles, 0 (FEW_WHOLE) past the last.
__device__ __forceinline__ unsigned few_run(const FewRuns& w, int tiles_m) {
  unsigned run = 0;
#pragma unroll
  for (int i = kFewRuns - 1; i >= 0; --i)
    if (tiles_m <= few_end(w.run[i])) run = w.run[i];
  return run;
}

// Launches whose 256x256 tiles (of the rows bound) fill at most one round of
// the n_units workgroups that run at once; the form follows from the real row
// count, read on the device.
template <int EPI>
__global__ __launch_bounds__(NT, 1) void gemm_bf16_split_kernel(FewRuns w, GemmParams p) {
  __shared__ __attribute__((aligned(1024))) uint8_t st0[4 * FEW_STAGE];
  __shared__ __attribute__((aligned(1024))) uint8_t st1[4 * FEW_STAGE];
  __shared__ __attribute__((aligned(1024))) uint8_t st2[4 * FEW_STAGE];
  __shared__ __attribute__((aligned(1024))) uint8_t st3[4 * FEW_STAGE];
  __shared__ int s_last;
  const int M = rows_from(p.m_ptr, p.m_ub);
  const int tiles_m = (M + FEW_ROWS - 1) / FEW_ROWS;
  const int u = blockIdx.x;
  const unsigned run = few_run(w, tiles_m);
  const int shape = few_form(run);
  if (__builtin_expect(shape == FEW_WHOLE, 1)) {
    run_unit256<EPI>(p, st0, st1, st2, st3, M, Units256(M, p.N, p.n_units, p.mtiles), u);
  } else if (shape == FEW_WIDE) {
    run_unit_few<EPI, 4>(p, st0, st1, st2, st3, &s_last, M, tiles_m, few_run_splits(run), u);
  } else if (shape == FEW_NARROW) {
    run_unit_few<EPI, 2>(p, st0, st1, st2, st3, &s_last, M, tiles_m, few_run_splits(run), u);
  } else if constexpr (EPI == EPI_RESID_PAIR) {
    const int parts = few_run_parts(run);
    // unit u: part u % parts of tile u / parts; gemm_parts_kernel adds the sums
    const int tm256 = p.mtiles ? p.mtiles[0] : (M + 255) / 256, tiles_n = p.N / 256;
    if (u >= tm256 * tiles_n * parts) return;
    const int tile = u / parts, sp = u - tile * parts;
    const int kts = p.K / BK / parts;
    int tm, tn;
    raster(tile, tm256, tiles_n, tm, tn);
    if (p.mtiles) tm = p.mtiles[1 + tm];
    gemm_tile<EPI, 256, true>(p, st0, st1, st2, st3, M, tm * 256, tn * 256, kts, sp * kts,
                              p.partial + (size_t)sp * (size_t)(tiles_m * FEW_ROWS) * (size_t)p.N);
  }
}

// The second launch of FEW_PARTS with the residual pair's epilogue: a thread adds
// 8 columns of the parts in part order and the residual, and stores them.  Exits
// at once where the rule has another form for the real row count.
__global__ __launch_bounds__(256) void gemm_parts_kernel(FewRuns w, GemmParams p) {
  const int M = rows_from(p.m_ptr, p.m_ub);
  const int tiles_m = (M + FEW_ROWS - 1) / FEW_ROWS;
  const unsigned run = few_run(w, tiles_m);
  if (few_form(run) != FEW_PARTS) return;
  const int parts = few_run_parts(run);
  const int groups = p.N / 8;
  const long long idx = (long long)blockIdx.x * 256 + threadIdx.x;
  int row = (int)(idx / groups);
  const int col = 8 * (int)(idx - (long long)row * groups);
  if (p.mtiles) {
    if ((row >> 8) >= p.mtiles[0]) return;
    row = p.mtiles[1 + (row >> 8)] * 256 + (row & 255);
  }
  if (row >= M) return;
  float v[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) v[e] = 0.0f;
  for (int sp = 0; sp < parts; ++sp) {
    const float* src = p.partial + ((size_t)sp * (size_t)(tiles_m * FEW_ROWS) + (size_t)row) * (size_t)p.N + col;
    const f32x4_t a = *reinterpret_cast<const f32x4_t*>(src);
    const f32x4_t b = *reinterpret_cast<const f32x4_t*>(src + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[e] += a[e];
      v[4 + e] += b[e];
    }
  }
  auto add = [&](const void* rows) {
    const u32x4_t r = *reinterpret_cast<const u32x4_t*>(static_cast<const uint16_t*>(rows) + (size_t)row * p.ldr + col);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      v[2 * e] += __uint_as_float(r[e] << 16);
      v[2 * e + 1] += __uint_as_float(r[e] & 0xffff0000u);
    }
  };
  add(p.R);
  add(p.R2);
  *reinterpret_cast<u32x4_t*>(static_cast<uint16_t*>(p.C) + (size_t)row * p.ldc + col) =
      u32x4_t{pack_bf2(v[0], v[1]), pack_bf2(v[2], v[3]), pack_bf2(v[4], v[5]), pack_bf2(v[6], v[7])};
}

}  // namespace seer

// fp32 variants of the layer kernels (any d_model, d_ff; head_dim <= 128): the
// GEMM with the same fused epilogues as the bf16 path, attention and the
// rotary embedding, on the fp32 matrix instruction (16x16x4: exact products,
// fp32 sums).
#include <math.h>

#include "common.h"
#include "kernels.h"

namespace seer {

namespace {

template <int N>
struct FVec { float v[N]; };

// N consecutive floats at src + c of a row of `n` valid ones, zero past n.
template <int N, bool VEC>
__device__ __forceinline__ FVec<N> load_chunk(const float* src, int c, int n) {
  FVec<N> r;
  if constexpr (VEC) {
    // n % 4 == 0 and c is a multiple of N: the chunk is all in or all out
    typedef float vec_t __attribute__((ext_vector_type(N)));
    const vec_t x = *reinterpret_cast<const vec_t*>(src + (c < n ? c : 0));
#pragma unroll
    for (int e = 0; e < N; ++e) r.v[e] = c < n ? x[e] : 0.0f;
  } else {
#pragma unroll
    for (int e = 0; e < N; ++e) r.v[e] = c + e < n ? src[c + e] : 0.0f;
  }
  return r;
}

}  // namespace

// C[M,N] = A[M,K] B[N,K]^T.  A workgroup owns one square tile of 16 W rows and
// columns; its four waves take a quarter of K each and sum through LDS in wave
// order at the end.  Operands go straight from memory to registers, 16 bytes
// per lane, one 16-wide K step ahead (the summed index of an MFMA may be
// permuted freely, so lane group lane/16 takes K values k0 + 4 (lane/16) .. +3
// for four MFMAs, and a load covers whole 64-byte runs of 16 rows): no LDS and
// no barrier in the loop.  The weights are the first MFMA operand, so lane l
// holds row l%16 and four consecutive columns 4 (l/16) .. +3 of a 16x16 tile.
//
// What bounds it: the chain of one wave (load, MFMAs, the LDS sum) while the
// tiles fit the chip a few times over, hence the four-way K split and the
// small tile; the operand loads from L2 beyond that.  Against a 64x64 LDS-tiled
// vector-ALU kernel (d 256, d_ff 688, times in us for QKV / O / gate-up / down):
// 224 rows 37 / 38 / 58 / 130 -> 6 / 5 / 8 / 9; 2668 rows 40 / 36 / 61 / 126 ->
// 21 / 9 / 30 / 18.  Three K steps ahead instead of one: 30 -> 49 us on that
// gate/up (the loads past a wave's short range are wasted).
// VEC: 16-byte accesses (every row a multiple of 16 bytes, aligned bases).
template <int EPI, int W, bool VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmParams p) {
  constexpr bool kGlu = (EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_COUNT);
  constexpr int NB = kGlu ? 2 : 1;                  // B operands (gate and up)
  constexpr int KS = 4;                             // waves, each a quarter of K
  constexpr int TILE = 16 * W;
  constexpr int CPT = W / 2;                       // 4-column groups per thread and 32-row part
  __shared__ float s_acc[KS * NB][32][TILE + 4];
  const int M = rows_from(p.m_ptr, p.m_ub);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, lq = lane >> 4;
  const int m0 = blockIdx.y * TILE, n0 = blockIdx.x * TILE;
  if (m0 >= M) return;
  const float* ap[W];
  const float* bp[NB][W];
  // rows and columns past the matrix re-read the last one (never stored)
#pragma unroll
  for (int i = 0; i < W; ++i)
    ap[i] = static_cast<const float*>(p.A) + (size_t)min(m0 + 16 * i + li, M - 1) * p.lda;
#pragma unroll
  for (int i = 0; i < W; ++i) {
    const int c = min(n0 + 16 * i + li, p.N - 1);
    bp[0][i] = static_cast<const float*>(p.B) + (size_t)c * p.ldb;
    if constexpr (kGlu) bp[NB - 1][i] = static_cast<const float*>(p.B2) + (size_t)c * p.ldb;
  }
  f32x4_t acc[NB][W][W];
#pragma unroll
  for (int u = 0; u < NB; ++u)
#pragma unroll
    for (int i = 0; i < W; ++i)
#pragma unroll
      for (int j = 0; j < W; ++j) acc[u][i][j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

  // K steps of 16 [t0, t1) of this wave
  const int steps = (p.K + 15) / 16;
  const int per = (steps + KS - 1) / KS;
  const int t0 = min(per * wave, steps), t1 = min(t0 + per, steps);
  struct Frag { FVec<4> a[W], b[NB][W]; };
  auto load = [&](int t, Frag& f) {
    const int k = 16 * t + 4 * lq;
#pragma unroll
    for (int i = 0; i < W; ++i) f.a[i] = load_chunk<4, VEC>(ap[i], k, p.K);
#pragma unroll
    for (int i = 0; i < W; ++i) {
#pragma unroll
      for (int u = 0; u < NB; ++u) f.b[u][i] = load_chunk<4, VEC>(bp[u][i], k, p.K);
    }
  };
  auto mul = [&](const Frag& f) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int u = 0; u < NB; ++u)
#pragma unroll
        for (int i = 0; i < W; ++i)
#pragma unroll
          for (int j = 0; j < W; ++j)
            acc[u][i][j] =
                __builtin_amdgcn_mfma_f32_16x16x4f32(f.b[u][j].v[e], f.a[i].v[e], acc[u][i][j], 0, 0, 0);
  };
  if (t0 < t1) {
    Frag f0, f1;
    load(t0, f0);
    int t = t0;
    for (; t + 2 < t1; t += 2) {
      load(t + 1, f1);
      mul(f0);
      load(t + 2, f0);
      mul(f1);
    }
    if (t + 1 < t1) {
      load(t + 1, f1);
      mul(f0);
      mul(f1);
    } else {
      mul(f0);
    }
  }

  float* C = static_cast<float*>(p.C);
  const float* R = static_cast<const float*>(p.R);
  // the tile in parts of 32 rows: partial sums to LDS, then thread t adds the
  // waves' values of row t / 8 and 4-column groups t % 8 + 8 g
#pragma unroll
  for (int part = 0; part < W / 2; ++part) {
    if (part) __syncthreads();
#pragma unroll
    for (int u = 0; u < NB; ++u)
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < W; ++j)
          *reinterpret_cast<f32x4_t*>(&s_acc[wave * NB + u][16 * i + li][16 * j + 4 * lq]) = acc[u][2 * part + i][j];
    __syncthreads();
    const int r = threadIdx.x >> 3;
    const int row = m0 + 32 * part + r;
    int cnt = 0;
#pragma unroll
    for (int g = 0; g < CPT; ++g) {
      const int c = 4 * ((threadIdx.x & 7) + 8 * g);
      const int col = n0 + c;
      if (row >= M || col >= p.N) continue;
      f32x4_t sum[NB];
#pragma unroll
      for (int u = 0; u < NB; ++u) {
        sum[u] = *reinterpret_cast<const f32x4_t*>(&s_acc[u][r][c]);
#pragma unroll
        for (int w = 1; w < KS; ++w) sum[u] += *reinterpret_cast<const f32x4_t*>(&s_acc[w * NB + u][r][c]);
      }
      f32x4_t v = sum[0];
      if constexpr (EPI == EPI_SCALE) v *= p.rs[row];
      if constexpr (kGlu) {
        const float sc = p.rs[row];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = silu(sum[0][e] * sc) * (sum[NB - 1][e] * sc);
          if (EPI == EPI_SWIGLU_COUNT && col + e < p.N) cnt += fabsf(v[e]) < p.eps ? 1 : 0;
        }
      }
      float* dst = C + (size_t)row * p.ldc + col;
      if constexpr (VEC) {
        if constexpr (EPI == EPI_RESID) v += *reinterpret_cast<const f32x4_t*>(R + (size_t)row * p.ldr + col);
        *reinterpret_cast<f32x4_t*>(dst) = v;
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          if (col + e >= p.N) continue;
          if constexpr (EPI == EPI_RESID) v[e] += R[(size_t)row * p.ldr + col + e];
          dst[e] = v[e];
        }
      }
    }
    if constexpr (EPI == EPI_SWIGLU_COUNT) {
#pragma unroll
      for (int off = 1; off < 8; off <<= 1) cnt += __shfl_xor(cnt, off, kWave);
      if ((threadIdx.x & 7) == 0 && cnt) atomicAdd(p.cnt + row, cnt);
    }
  }
}

template <int EPI>
static void launch_gemm_f32_epi(const GemmParams& p, bool vec, hipStream_t s) {
  // A 64x64 tile halves the operand loads per MFMA but leaves fewer, longer
  // chains.  At 11,600 rows (d 512, 1448 such tiles) O and down take 148
  // against 173 us with it and QKV 231 against 276; at 750 rows (288 tiles)
  // 24 against 31 us without.  SwiGLU's two weights already share one set of
  // activation loads: 399 us against 434 with the wide tile.  Element-wise
  // loads cost four times the instructions, so there it pays earlier and for
  // SwiGLU too (8400 rows, d_ff 687: 184 against 259 us).
  const bool glu = EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_COUNT;
  const long long tiles = (long long)((p.N + 63) / 64) * ((p.m_ub + 63) / 64);
  const bool wide = vec ? !glu && tiles >= 1024 : tiles >= 512;
  const int tile = wide ? 64 : 32;
  dim3 grid((p.N + tile - 1) / tile, (p.m_ub + tile - 1) / tile), block(256);
  if (wide && vec) hipLaunchKernelGGL((gemm_f32_kernel<EPI, 4, true>), grid, block, 0, s, p);
  else if (wide) hipLaunchKernelGGL((gemm_f32_kernel<EPI, 4, false>), grid, block, 0, s, p);
  else if (vec) hipLaunchKernelGGL((gemm_f32_kernel<EPI, 2, true>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((gemm_f32_kernel<EPI, 2, false>), grid, block, 0, s, p);
}

int launch_gemm_f32(int epi, const GemmParams& p, hipStream_t s) {
  auto a16 = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
  const bool vec = p.K % 4 == 0 && p.N % 4 == 0 && p.lda % 4 == 0 && p.ldb % 4 == 0 && p.ldc % 4 == 0 &&
                   p.ldr % 4 == 0 && a16(p.A) && a16(p.B) && a16(p.B2) && a16(p.C) && a16(p.R);
  switch (epi) {
    case EPI_SCALE: launch_gemm_f32_epi<EPI_SCALE>(p, vec, s); break;
    case EPI_RESID: launch_gemm_f32_epi<EPI_RESID>(p, vec, s); break;
    case EPI_SWIGLU: launch_gemm_f32_epi<EPI_SWIGLU>(p, vec, s); break;
    case EPI_SWIGLU_COUNT: launch_gemm_f32_epi<EPI_SWIGLU_COUNT>(p, vec, s); break;
    default: return -1;
  }
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ---------------------------------------------------------------------------
// fp32 attention, one workgroup per (sequence, 16 queries, head).  The batches
// are small, so a launch is bound by the length of one workgroup's chain, not
// by throughput: its four waves take a quarter of the keys each, with an
// online softmax of their own, and merge through LDS at the end.
//
// Scores are computed transposed, S^T = K Q^T, so register r of a 16-key tile
// holds query lane%16 and key 4 (lane/16) + r, which is already the operand
// layout of O^T = V^T P^T: no shuffle of P.  K, Q and V come straight from
// memory (the rows of one head fit L2), 16 bytes per lane: lane group lane/16
// takes dims 16 j + 4 (lane/16) .. +3 of a chunk for four MFMAs, and output
// tile (g, e) holds the dims 16 E g + E i + e, i < 16.
//
// Measured against one lane per query walking every key: one 224-row sequence
// of 4 heads of 64, 327 -> 10 us; 16 sequences of 105-224 rows, 330 -> 22 us.
// 32 queries per workgroup (half the K and V loads per query) took 26 us there
// and 349 against 313 us at 11,600 rows of 8 heads: fewer waves per SIMD.
//
// VEC: 16-byte loads (head_dim % 4 == 0 and aligned rows); otherwise the same
// chunks element by element.
template <int DH, bool VEC>
__global__ __launch_bounds__(256) void attn_f32_kernel(AttnParams p) {
  constexpr int QT = 16;
  constexpr int NJ = DH / 16;                 // 16-dim chunks of a head
  constexpr int E = NJ < 4 ? NJ : 4;          // dims per V load and lane
  constexpr int G = NJ / E;
  __shared__ float s_o[4][QT][DH + 4];
  __shared__ float s_m[4][QT], s_l[4][QT];
  int b, t;
  if (!tile_of(p.cu, p.B, QT, blockIdx.x, b, t)) return;
  const int h = blockIdx.y;
  const int s0 = p.cu[b];
  if (s0 < 0 || s0 >= p.rows_ub) return;
  int len = p.cu[b + 1] - s0;
  len = len > p.rows_ub - s0 ? p.rows_ub - s0 : len;
  if (t * QT >= len) return;
  int used = p.used ? p.used[b] : len;
  used = used < 0 ? 0 : (used > len ? len : used);
  // keys: the cached prefix rows (if any), then the sequence's own used rows
  int P = 0, kv0 = 0;
  if (p.cu_kv) {
    kv0 = p.cu_kv[b];
    P = p.cu_kv[b + 1] - kv0;
    P = P < 0 ? 0 : P;
  }
  const int nk = P + used;

  const int lane = threadIdx.x & 63;
  const int wave = threadIdx.x >> 6;
  const int li = lane & 15, lq = lane >> 4;
  const int hd = p.head_dim;
  const size_t ld = (size_t)3 * p.d;
  const float* qkv = static_cast<const float*>(p.qkv) + h * hd;
  const float* kvc = p.cu_kv ? static_cast<const float*>(p.kv) + h * hd : nullptr;
  // K row of key position k < nk; its V row is d elements further
  auto key_row = [&](int k) {
    return k < P ? kvc + (size_t)(kv0 + k) * 2 * p.d : qkv + (size_t)(s0 + k - P) * ld + p.d;
  };

  f32x4_t qf[NJ];
  {
    int q = t * QT + li;
    q = q < len ? q : len - 1;
    const float* qr = qkv + (size_t)(s0 + q) * ld;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const FVec<4> c = load_chunk<4, VEC>(qr, 16 * j + 4 * lq, hd);
#pragma unroll
      for (int e = 0; e < 4; ++e) qf[j][e] = c.v[e] * p.scale;
    }
  }
  f32x4_t o[NJ];
  float m = -INFINITY, l = 0.0f;
#pragma unroll
  for (int j = 0; j < NJ; ++j) o[j] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};

  // This wave's keys: a quarter of the 16-key tiles, walked two at a time.  A
  // step's V is requested before its scores and the next step's K before its
  // softmax, so that neither latency is on the chain.
  const int per = ((nk + 15) / 16 + 3) / 4;
  const int k_begin = 16 * per * wave, k_end = min(k_begin + 16 * per, nk);
  FVec<4> kf[2][NJ];
  FVec<E> vf[2][4][G];
  auto load_k = [&](int k0) {
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      const int key = k0 + 16 * c + li;
      const float* kr = key_row(key < nk ? key : nk - 1);
#pragma unroll
      for (int j = 0; j < NJ; ++j) kf[c][j] = load_chunk<4, VEC>(kr, 16 * j + 4 * lq, hd);
    }
  };
  if (k_begin < k_end) load_k(k_begin);
  for (int k0 = k_begin; k0 < k_end; k0 += 32) {
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int key = k0 + 16 * c + 4 * lq + r;
        const float* vr = key_row(key < nk ? key : nk - 1) + p.d;
#pragma unroll
        for (int g = 0; g < G; ++g) vf[c][r][g] = load_chunk<E, VEC>(vr, 16 * E * g + E * li, hd);
      }
    f32x4_t s[2];
#pragma unroll
    for (int c = 0; c < 2; ++c) {
      s[c] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e)
          s[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][j].v[e], qf[j][e], s[c], 0, 0, 0);
    }
    if (k0 + 32 < k_end) load_k(k0 + 32);
    if (k0 + 32 > k_end) {
      // masked keys: probability 0, and a zero V so that they add 0 x 0
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (k0 + 16 * c + 4 * lq + r >= k_end) {
            s[c][r] = -INFINITY;
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
              for (int e = 0; e < E; ++e) vf[c][r][g].v[e] = 0.0f;
          }
    }
    // the four lane groups of a query hold 8 of the step's 32 keys each; key
    // k0 is never masked, so the step's maximum covers a real score
    float mt = s[0][0];
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) mt = fmaxf(mt, s[c][r]);
    mt = fmaxf(mt, __shfl_xor(mt, 16, kWave));
    mt = fmaxf(mt, __shfl_xor(mt, 32, kWave));
    const float mn = fmaxf(m, mt);
    const float alpha = __expf(m - mn);
    m = mn;
    l *= alpha;
#pragma unroll
    for (int j = 0; j < NJ; ++j) o[j] *= alpha;
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float pe = __expf(s[c][r] - mn);
        s[c][r] = pe;
        l += pe;
      }
#pragma unroll
    for (int c = 0; c < 2; ++c)
#pragma unroll
      for (int r = 0; r < 4; ++r)
#pragma unroll
        for (int g = 0; g < G; ++g)
#pragma unroll
          for (int e = 0; e < E; ++e)
            o[g * E + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[c][r][g].v[e], s[c][r], o[g * E + e], 0, 0, 0);
  }

  // merge the four waves' states in wave order
  l += __shfl_xor(l, 16, kWave);
  l += __shfl_xor(l, 32, kWave);
  if (lq == 0) {
    s_m[wave][li] = m;
    s_l[wave][li] = l;
  }
#pragma unroll
  for (int g = 0; g < G; ++g)
#pragma unroll
    for (int e = 0; e < E; ++e)
#pragma unroll
      for (int r = 0; r < 4; ++r) s_o[wave][li][16 * E * g + E * (4 * lq + r) + e] = o[g * E + e][r];
  __syncthreads();
  float* out = static_cast<float*>(p.out);
  for (int i = threadIdx.x; i < QT * DH; i += 256) {
    const int q = i / DH, c = i % DH;
    const int q_row = t * QT + q;
    if (q_row >= len || c >= hd) continue;
    float mx = s_m[0][q];
#pragma unroll
    for (int w = 1; w < 4; ++w) mx = fmaxf(mx, s_m[w][q]);
    float num = 0.0f, den = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      // a wave without keys (m = -inf, l = 0) adds nothing
      const float f = s_l[w][q] == 0.0f ? 0.0f : __expf(s_m[w][q] - mx);
      num = fmaf(f, s_o[w][q][c], num);
      den = fmaf(f, s_l[w][q], den);
    }
    const float inv = (q_row < used && den > 0.0f) ? 1.0f / den : 0.0f;
    out[(size_t)(s0 + q_row) * p.d + h * hd + c] = num * inv;
  }
}

template <int DH>
static void launch_attn_f32_dh(const AttnParams& p, bool vec, hipStream_t s) {
  dim3 grid((p.rows_ub + 15) / 16 + p.B, p.n_heads), block(256);
  if (vec) hipLaunchKernelGGL((attn_f32_kernel<DH, true>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((attn_f32_kernel<DH, false>), grid, block, 0, s, p);
}

int launch_attn_f32(const AttnParams& p, hipStream_t s) {
  if (p.cu_kv && !p.kv) return -1;
  auto a16 = [](const void* q) { return (reinterpret_cast<uintptr_t>(q) & 15) == 0; };
  const bool vec = p.head_dim % 4 == 0 && p.d % 4 == 0 && a16(p.qkv) && (!p.cu_kv || a16(p.kv));
  if (p.head_dim <= 32) launch_attn_f32_dh<32>(p, vec, s);
  else if (p.head_dim <= 64) launch_attn_f32_dh<64>(p, vec, s);
  else if (p.head_dim <= 128) launch_attn_f32_dh<128>(p, vec, s);
  else return -1;
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ---------------------------------------------------------------------------
// Rotary embedding of the q and k columns of an fp32 qkv buffer, in place: one
// thread per (row, q|k, head, pair j < head_dim / 2); pair (j, j + head_dim/2)
// of the head turns by 2 pi * frac(pos[r] * freq[j]).
__global__ __launch_bounds__(256) void rope_f32_kernel(float* qkv, int d, int head_dim, const int* m_ptr,
                                                       int m_ub, const int* pos, const double* freq) {
  const int M = rows_from(m_ptr, m_ub);
  const int half = head_dim >> 1;
  const int per_row = d;                 // 2 d columns rotated in pairs: d pairs per row
  const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  const int row = (int)(t / per_row);
  if (row >= M) return;
  const int k = (int)(t % per_row);      // pair index over q and k
  const int head = k / half, j = k % half;
  float* x = qkv + (size_t)row * 3 * d + head * head_dim + j;
  double rv = (double)pos[row] * freq[j];
  rv -= floor(rv);
  const float a = (float)rv;
  const float sn = __builtin_amdgcn_sinf(a), cs = __builtin_amdgcn_cosf(a);
  const float x1 = x[0], x2 = x[half];
  x[0] = x1 * cs - x2 * sn;
  x[half] = x2 * cs + x1 * sn;
}

int launch_rope_f32(float* qkv, int d, int n_heads, int head_dim, const int* m_ptr, int m_ub,
                    const int* pos, const double* freq, hipStream_t s) {
  (void)n_heads;
  if (head_dim % 2 != 0) return -1;
  const long long work = (long long)m_ub * d;
  dim3 grid((unsigned)((work + 255) / 256)), block(256);
  hipLaunchKernelGGL(rope_f32_kernel, grid, block, 0, s, qkv, d, head_dim, m_ptr, m_ub, pos, freq);
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

}  // namespace seer

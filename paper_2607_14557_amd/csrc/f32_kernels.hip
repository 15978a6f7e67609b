// fp32 variants of the layer kernels (any d_model, d_ff; head_dim <= 128): the
// GEMM with the same fused epilogues as the bf16 path, attention and the
// rotary embedding, on the fp32 matrix instruction.
//
// Every sum runs in ascending order of its index, one fused multiply-add a
// term: the near-zero count is a threshold on the activations, so that another
// order of the sums moves it by one now and then (about 2% of the batches of
// 224 rows by 688 columns).  v_mfma_f32_16x16x4 is such a chain over its four
// index values (compared with fmaf bit for bit, denormals included), so the
// chains run on the matrix pipe at its full rate; what is given up is the
// split of one sum over several waves.
#include <math.h>

#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace seer {

namespace {

// 16-byte accesses to memory of any 4-byte alignment.
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));

// Floats c .. c + 3 of a row of n.  What lies past n is some float of the row
// until keep_valid clears it: a select beside the load would wait for it there.
// WHOLE: n % 4 == 0, so that the four (c % 4 == 0) are all in or all out.
template <bool WHOLE>
__device__ __forceinline__ f32x4_t load4(const float* src, int c, int n) {
  if constexpr (WHOLE) return *reinterpret_cast<const f32x4_u*>(src + (c < n ? c : 0));
  f32x4_t r;
#pragma unroll
  for (int e = 0; e < 4; ++e) r[e] = src[c + e < n ? c + e : 0];
  return r;
}

__device__ __forceinline__ f32x4_t keep_valid(f32x4_t v, int c, int n) {
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = c + e < n ? v[e] : 0.0f;
  return v;
}

// Lane l of a 16-row operand loads elements 4 (l/16) .. +3 of row l%16; the
// matrix instruction e of four wants element 4 e + l/16 in register e: the
// 4x4 transpose between the lane groups and the registers.
__device__ __forceinline__ f32x4_t to_index_order(f32x4_t c) {
  uint32_t v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = __float_as_uint(c[e]);
  const u32x2_t a = __builtin_amdgcn_permlane32_swap(v[0], v[2], false, false);
  const u32x2_t b = __builtin_amdgcn_permlane32_swap(v[1], v[3], false, false);
  const u32x2_t lo = __builtin_amdgcn_permlane16_swap(a[0], b[0], false, false);
  const u32x2_t hi = __builtin_amdgcn_permlane16_swap(a[1], b[1], false, false);
  return f32x4_t{__uint_as_float(lo[0]), __uint_as_float(lo[1]), __uint_as_float(hi[0]), __uint_as_float(hi[1])};
}

}  // namespace

// C[M,N] = A[M,K] B[N,K]^T.  A workgroup owns a square tile of 32 W rows and
// columns, each of its four waves a quarter of it (W x W tiles of 16x16) over
// all of K.  Operands go straight from memory to registers, 16 bytes per lane
// (a load covers whole 64-byte runs of 16 rows), PF 16-wide K steps ahead: no
// LDS and no barrier.  The transposes of a step are issued between the MFMAs of
// the step before.  The weights are the first MFMA operand, so lane l holds
// row l%16 and four consecutive columns 4 (l/16) .. +3 of a 16x16 tile.
//
// What bounds it: one wave's chain of MFMAs, 32 cycles each, and the loads
// ahead of it while the tiles fit the chip a few times over, the operand loads
// from L2 beyond that.  Against a 64x64 LDS-tiled vector-ALU kernel (d 256,
// d_ff 688, times in us for QKV / O / gate-up / down): 224 rows 37 / 38 / 58 /
// 130 -> 7 / 6 / 10 / 9; 2700 rows 41 / 37 / 61 / 126 -> 24 / 12 / 29 / 21;
// 14,000 rows with d_ff 687 101 / 53 / 167 / 140 -> 83 / 35 / 122 / 80.  A K
// split over the waves (sums in another order) took 6 / 5 / 8 / 9 at 224 rows.
// The transposes ahead of a step's MFMAs instead of between those of the step
// before, and a select beside each load, cost 8 to 20 us at 2700 rows.
template <int EPI, int W>
__global__ __launch_bounds__(256) void gemm_f32_kernel(GemmParams p) {
  constexpr bool kGlu = (EPI == EPI_SWIGLU || EPI == EPI_SWIGLU_COUNT);
  constexpr int NB = kGlu ? 2 : 1;                  // B operands (gate and up)
  constexpr int PF = W == 1 ? 6 : 2;
  const int M = rows_from(p.m_ptr, p.m_ub);
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int li = lane & 15, lq = lane >> 4;
  const int m0 = (blockIdx.y * 2 + (wave >> 1)) * 16 * W, n0 = (blockIdx.x * 2 + (wave & 1)) * 16 * W;
  if (m0 >= M || n0 >= p.N) return;
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

  struct Frag { f32x4_t a[W], b[NB][W]; };
  const int steps = p.K / 16, part = 16 * steps;    // whole steps; K values from `part` on are a last, partial one
  auto load = [&](int t, Frag& g) {
    const int k = 16 * t + 4 * lq;
#pragma unroll
    for (int i = 0; i < W; ++i) {
      g.a[i] = *reinterpret_cast<const f32x4_u*>(ap[i] + k);
#pragma unroll
      for (int u = 0; u < NB; ++u) g.b[u][i] = *reinterpret_cast<const f32x4_u*>(bp[u][i] + k);
    }
  };
  // operand k of a step's W + NB W, in index order
  auto order = [&](const Frag& g, int k, Frag& r) {
    if (k < W) r.a[k] = to_index_order(g.a[k]);
    else r.b[(k - W) / W][(k - W) % W] = to_index_order(g.b[(k - W) / W][(k - W) % W]);
  };
  // one step; meanwhile the operands of the next go from raw to next
  auto mul = [&](const Frag& g, bool more, const Frag& raw, Frag& next) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      if (more) {
        constexpr int NF = (1 + NB) * W;
#pragma unroll
        for (int k = NF * e / 4; k < NF * (e + 1) / 4; ++k) order(raw, k, next);
      }
#pragma unroll
      for (int u = 0; u < NB; ++u)
#pragma unroll
        for (int i = 0; i < W; ++i)
#pragma unroll
          for (int j = 0; j < W; ++j)
            acc[u][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(g.b[u][j][e], g.a[i][e], acc[u][i][j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  auto order_all = [&](const Frag& g, Frag& r) {
#pragma unroll
    for (int k = 0; k < (1 + NB) * W; ++k) order(g, k, r);
  };
  Frag last;
  if (part < p.K) {
    const int k = part + 4 * lq;
#pragma unroll
    for (int i = 0; i < W; ++i) {
      last.a[i] = load4<false>(ap[i], k, p.K);
#pragma unroll
      for (int u = 0; u < NB; ++u) last.b[u][i] = load4<false>(bp[u][i], k, p.K);
    }
  }
  if (steps > 0) {
    Frag f[PF], now[2];
    // no condition on a load up to the end of the main loop: behind one that may
    // not have been issued, a wait would have to count it as missing
#pragma unroll
    for (int u = 0; u < PF; ++u) load(u < steps ? u : steps - 1, f[u]);
    order_all(f[0], now[0]);
    int t = 0;
    // step t + u multiplies now[u % 2]; f[u] is free, f[(u + 1) % PF] holds the step after
    for (; t + 2 * PF <= steps; t += PF) {
#pragma unroll
      for (int u = 0; u < PF; ++u) {
        load(t + u + PF, f[u]);
        __builtin_amdgcn_sched_barrier(0);
        mul(now[u & 1], true, f[(u + 1) % PF], now[(u + 1) & 1]);
      }
    }
#pragma unroll
    for (int u = 0; u < 2 * PF; ++u)
      if (t + u < steps) {
        if (t + u + PF < steps) load(t + u + PF, f[u % PF]);
        mul(now[u & 1], t + u + 1 < steps, f[(u + 1) % PF], now[(u + 1) & 1]);
      }
  }
  if (part < p.K) {
    const int k = part + 4 * lq;
#pragma unroll
    for (int i = 0; i < W; ++i) {
      last.a[i] = keep_valid(last.a[i], k, p.K);
#pragma unroll
      for (int u = 0; u < NB; ++u) last.b[u][i] = keep_valid(last.b[u][i], k, p.K);
    }
    Frag g;
    order_all(last, g);
    mul(g, false, g, last);
  }

  float* C = static_cast<float*>(p.C);
  const float* R = static_cast<const float*>(p.R);
#pragma unroll
  for (int i = 0; i < W; ++i) {
    const int row = m0 + 16 * i + li;
    const bool row_ok = row < M;
    float sc = 1.0f;
    if constexpr (EPI == EPI_SCALE || kGlu) sc = p.rs[row_ok ? row : M - 1];
    int cnt = 0;
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const int col = n0 + 16 * j + 4 * lq;
      if (!row_ok || col >= p.N) continue;
      f32x4_t v = acc[0][i][j];
      if constexpr (EPI == EPI_SCALE) v *= sc;
      if constexpr (kGlu) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          v[e] = silu(acc[0][i][j][e] * sc) * (acc[NB - 1][i][j][e] * sc);
          if (EPI == EPI_SWIGLU_COUNT && col + e < p.N) cnt += fabsf(v[e]) < p.eps ? 1 : 0;
        }
      }
      float* dst = C + (size_t)row * p.ldc + col;
      if (col + 4 <= p.N) {
        if constexpr (EPI == EPI_RESID) v += *reinterpret_cast<const f32x4_u*>(R + (size_t)row * p.ldr + col);
        *reinterpret_cast<f32x4_u*>(dst) = v;
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
      cnt += __shfl_xor(cnt, 16, kWave);
      cnt += __shfl_xor(cnt, 32, kWave);
      if (row_ok && lq == 0 && cnt) atomicAdd(p.cnt + row, cnt);
    }
  }
}

template <int EPI>
static void launch_gemm_f32_epi(const GemmParams& p, hipStream_t s) {
  // A 64x64 tile halves the operand loads per MFMA but makes a wave's chain four
  // times as long: 10.6 against 7.2 us with 48 such tiles (QKV, 224 rows, d 256),
  // 11.2 against 10.5 with 128 (O, 2000 rows), 15.7 against 19.4 with 132
  // (gate/up, 750 rows), 18.2 against 24.3 with 144 (O, 1100 rows, d 512).
  const bool wide = (long long)((p.N + 63) / 64) * ((p.m_ub + 63) / 64) > 128;
  const int tile = wide ? 64 : 32;
  dim3 grid((p.N + tile - 1) / tile, (p.m_ub + tile - 1) / tile), block(256);
  if (wide) hipLaunchKernelGGL((gemm_f32_kernel<EPI, 2>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((gemm_f32_kernel<EPI, 1>), grid, block, 0, s, p);
}

int launch_gemm_f32(int epi, const GemmParams& p, hipStream_t s) {
  switch (epi) {
    case EPI_SCALE: launch_gemm_f32_epi<EPI_SCALE>(p, s); break;
    case EPI_RESID: launch_gemm_f32_epi<EPI_RESID>(p, s); break;
    case EPI_SWIGLU: launch_gemm_f32_epi<EPI_SWIGLU>(p, s); break;
    case EPI_SWIGLU_COUNT: launch_gemm_f32_epi<EPI_SWIGLU_COUNT>(p, s); break;
    default: return -1;
  }
  return hipGetLastError() == hipSuccess ? 0 : -1;
}

// ---------------------------------------------------------------------------
// fp32 attention, one workgroup per (sequence, 16 queries, head), the keys in
// chunks of KC.  A chunk takes three passes, so that each is parallel in what
// its sums are not: the scores (16-key tiles dealt to four waves); the running
// maximum after every key, by a scan, and with it each key's probability p and
// the factor a of the sums before it; the sums in key order, o = fma(p, v, o a)
// (a wave takes 16 of the head's dims, or two such tiles) and l = fma(l, a, p)
// (one wave).
//
// a is 1 but where a key raises the maximum of one of the 16 queries, so four
// keys go through one MFMA, except in a quad with such a key (about every second
// of the first 200 keys): there each key is a product o a and a 4x4x1 MFMA of 16
// blocks, whose result has the same layout and whose V operand is a permutation
// of the other's.  Cutting the quad instead into MFMAs with the other keys' p
// and v set to zero took 36 us against 26 for the 16 sequences below, the sums
// on the vector ALU 42.
//
// Scores are computed transposed, S^T = K Q^T: lane l holds query l%16 and keys
// 4 (l/16) .. +3 of a tile, one 16-byte LDS store.  K and Q come straight from
// memory, 16 bytes per lane, V one dim per lane (64-byte runs).
//
// What bounds it: the batches are small, so one workgroup's chain of loads and
// MFMAs (32 cycles each), and the quads that raise a maximum.  Measured against
// one lane per query walking every key: one 224-row sequence of 4 heads of 64,
// 327 -> 17 us; 16 sequences of 105-224 rows, 330 -> 26 us; 13 sequences of 900
// rows, 8 heads, 1418 -> 532 us.  The keys split over the waves (sums in another
// order) took 11, 22 and 381 us.
//
// WHOLE: head_dim % 4 == 0; otherwise element loads.
template <int DH, bool WHOLE>
__global__ __launch_bounds__(256, DH > 64 ? 2 : 4) void attn_f32_kernel(AttnParams p) {
  constexpr int QT = 16;
  constexpr int KC = 256;                     // keys of a chunk: 16 a thread in the scan
  constexpr int NJ = DH / 16;                 // 16-dim chunks of a head
  constexpr int NT = NJ > 4 ? NJ / 4 : 1;     // 16-dim output tiles of a wave
  constexpr int KD = 2;                       // K tiles in flight
  constexpr int VG = 2;                       // groups of 16 keys that V is loaded ahead
  __shared__ __attribute__((aligned(16))) float s_p[QT][KC + 4], s_a[QT][KC + 4];
  __shared__ float s_l[QT];
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
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int li = lane & 15, lq = lane >> 4;
  const int hd = p.head_dim;
  const size_t ld = (size_t)3 * p.d;
  const float* qkv = static_cast<const float*>(p.qkv) + h * hd;
  f32x4_t qf[NJ];
  {
    int q = t * QT + li;
    q = q < len ? q : len - 1;
    const float* qr = qkv + (size_t)(s0 + q) * ld;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      const int c = 16 * j + 4 * lq;
      qf[j] = to_index_order(keep_valid(load4<WHOLE>(qr, c, hd), c, hd) * p.scale);
    }
  }
  f32x4_t o[NT];
#pragma unroll
  for (int T = 0; T < NT; ++T) o[T] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
  float m = -INFINITY;                        // running maximum of query threadIdx.x / 16
  float l = 0.0f;                             // wave l_wave: running sum of query li
  const bool has_dims = 16 * wave < hd;
  // the one wave that also adds p: one without dims, or another from tile to tile
  const int l_wave = hd <= 48 ? 3 : t & 3;

  float vf[VG][4][NT];
  // a chunk is of cached rows or of own rows
  for (int c0 = 0, cn; c0 < nk; c0 += cn) {
    const bool cached = c0 < P;
    cn = min(KC, (cached ? P : nk) - c0);
    const int groups = (cn + 15) / 16;
    const uint32_t stride = (cached ? 2u : 3u) * (uint32_t)p.d;
    const float* kb = cached ? static_cast<const float*>(p.kv) + h * hd + (size_t)(kv0 + c0) * stride
                             : qkv + p.d + (size_t)(s0 + c0 - P) * stride;
    const float* vb = kb + p.d;
    auto load_k = [&](int k, f32x4_t* kf) {
      k += li;
      const uint32_t row = (uint32_t)(k < cn ? k : cn - 1) * stride;
#pragma unroll
      for (int j = 0; j < NJ; ++j) kf[j] = load4<WHOLE>(kb + row, 16 * j + 4 * lq, hd);
    };
    auto load_v = [&](int k, float (&g)[4][NT]) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int key = k + 4 * e + lq;
        const uint32_t row = (uint32_t)(key < cn ? key : cn - 1) * stride;
#pragma unroll
        for (int T = 0; T < NT; ++T) {
          const int c = 16 * (wave + 4 * T) + li;
          g[e][T] = (vb + row)[c < hd ? c : hd - 1];
        }
      }
    };
    if (c0) __syncthreads();                  // the last chunk's p and a are read
    // scores; a tile past the last key re-reads it
    if (wave < groups) {
      f32x4_t kf[KD][NJ];
#pragma unroll
      for (int i = 0; i < KD; ++i) load_k(16 * (wave + 4 * i), kf[i]);
#pragma unroll
      for (int i = 0; i < KC / 64; ++i) {
        const int g = wave + 4 * i;
        if (g >= groups) break;
        f32x4_t k4[NJ];
#pragma unroll
        for (int j = 0; j < NJ; ++j) {
          const f32x4_t raw = kf[i % KD][j];
          k4[j] = to_index_order(hd < DH ? keep_valid(raw, 16 * j + 4 * lq, hd) : raw);
        }
        if (i + KD < KC / 64) load_k(16 * (g + 4 * KD), kf[i % KD]);
        __builtin_amdgcn_sched_barrier(0);
        f32x4_t s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int j = 0; j < NJ; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_16x16x4f32(k4[j][e], qf[j][e], s, 0, 0, 0);
        *reinterpret_cast<f32x4_t*>(&s_p[li][16 * g + 4 * lq]) = s;
      }
    }
    if (has_dims) {
#pragma unroll
      for (int u = 0; u < VG; ++u) load_v(16 * u, vf[u]);
    }
    __syncthreads();
    // probabilities: 16 threads a query, 16 keys each
    {
      const int q = threadIdx.x >> 4, k = 16 * (threadIdx.x & 15);
      f32x4_t x[4];
      float top = -INFINITY;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        x[g] = *reinterpret_cast<const f32x4_t*>(&s_p[q][k + 4 * g]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (k + 4 * g + e < cn) top = fmaxf(top, x[g][e]);
      }
      float upto = top;                       // maximum of this thread's keys and those of the threads before
#pragma unroll
      for (int off = 1; off < 16; off <<= 1) {
        const float v = __shfl_up(upto, off, 16);
        if ((threadIdx.x & 15) >= off) upto = fmaxf(v, upto);
      }
      const float before = __shfl_up(upto, 1, 16);
      float mk = (threadIdx.x & 15) ? fmaxf(m, before) : m;
      m = fmaxf(m, __shfl(upto, 15, 16));
      if (k < cn) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          f32x4_t pe, al;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float mn = fmaxf(mk, x[g][e]);
            const bool live = k + 4 * g + e < cn;
            pe[e] = live ? __expf(x[g][e] - mn) : 0.0f;
            al[e] = live ? __expf(mk - mn) : 1.0f;
            mk = live ? mn : mk;
          }
          *reinterpret_cast<f32x4_t*>(&s_p[q][k + 4 * g]) = pe;
          *reinterpret_cast<f32x4_t*>(&s_a[q][k + 4 * g]) = al;
        }
      }
    }
    __syncthreads();
    // weighted sums, in key order: a group's p and a are read while the group
    // before is added
    struct Group { float p[4]; f32x4_t a[4]; };
    auto read_group = [&](int g, Group& r) {
      const int k = 16 * (g < groups ? g : groups - 1);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        r.p[e] = s_p[li][k + 4 * e + lq];
        r.a[e] = *reinterpret_cast<const f32x4_t*>(&s_a[li][k + 4 * e]);
      }
    };
    auto add_group = [&](int g, const Group& r, float (&v)[4][NT]) {
      if (16 * g + 16 > cn) {                 // a key past the last adds 0 x 0
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int T = 0; T < NT; ++T) v[e][T] = 16 * g + 4 * e + lq < cn ? v[e][T] : 0.0f;
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (!__any(r.a[e][0] != 1.0f || r.a[e][1] != 1.0f || r.a[e][2] != 1.0f || r.a[e][3] != 1.0f)) {
#pragma unroll
          for (int T = 0; T < NT; ++T) o[T] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e][T], r.p[e], o[T], 0, 0, 0);
        } else {
          // key j: lane l takes dim 4 (l/16) + l%4 of it, which lane 16 j + that dim holds
          const f32x4_t p4 = *reinterpret_cast<const f32x4_t*>(&s_p[li][16 * g + 4 * e]);
          float vj[4][NT];
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int T = 0; T < NT; ++T) vj[j][T] = __shfl(v[e][T], 16 * j + 4 * lq + (lane & 3), kWave);
#pragma unroll
          for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int T = 0; T < NT; ++T) {
              o[T] *= r.a[e][j];
              o[T] = __builtin_amdgcn_mfma_f32_4x4x1f32(vj[j][T], p4[j], o[T], 0, 0, 0);
            }
        }
      }
      if (wave == l_wave) {
        f32x4_t p4[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) p4[e] = *reinterpret_cast<const f32x4_t*>(&s_p[li][16 * g + 4 * e]);
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
          for (int j = 0; j < 4; ++j) l = fmaf(l, r.a[e][j], p4[e][j]);
      }
    };
    if (has_dims || wave == l_wave) {
      Group r[2];
      read_group(0, r[0]);
      for (int g = 0; g < groups; g += VG) {
#pragma unroll
        for (int u = 0; u < VG; ++u) {
          read_group(g + u + 1, r[(u + 1) & 1]);
          if (g + u < groups) add_group(g + u, r[u & 1], vf[u]);
          load_v(16 * (g + u + VG), vf[u]);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
  }

  if (wave == l_wave && lq == 0) s_l[li] = l;
  __syncthreads();
  const int q_row = t * QT + li;
  if (q_row >= len || !has_dims) return;
  const float lt = s_l[li];
  const float inv = (q_row < used && lt > 0.0f) ? 1.0f / lt : 0.0f;
  float* out = static_cast<float*>(p.out) + (size_t)(s0 + q_row) * p.d + h * hd;
#pragma unroll
  for (int T = 0; T < NT; ++T) {
    const int c = 16 * (wave + 4 * T) + 4 * lq;
    const f32x4_t r = o[T] * inv;
    if (c + 4 <= hd) {
      *reinterpret_cast<f32x4_u*>(out + c) = r;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (c + e < hd) out[c + e] = r[e];
    }
  }
}

template <int DH>
static void launch_attn_f32_dh(const AttnParams& p, hipStream_t s) {
  dim3 grid((p.rows_ub + 15) / 16 + p.B, p.n_heads), block(256);
  if (p.head_dim % 4 == 0) hipLaunchKernelGGL((attn_f32_kernel<DH, true>), grid, block, 0, s, p);
  else hipLaunchKernelGGL((attn_f32_kernel<DH, false>), grid, block, 0, s, p);
}

int launch_attn_f32(const AttnParams& p, hipStream_t s) {
  if (p.cu_kv && !p.kv) return -1;
  if (p.head_dim <= 32) launch_attn_f32_dh<32>(p, s);
  else if (p.head_dim <= 64) launch_attn_f32_dh<64>(p, s);
  else if (p.head_dim <= 128) launch_attn_f32_dh<128>(p, s);
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

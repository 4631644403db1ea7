// float32 kernels of the verification step, for float32 models (small models:
// cache-resident, so launches and latency count, not bandwidth).  Same
// semantics as the bfloat16 path: RMSNorm is applied as (x * gain) followed by
// a per-row scale of the product.
//
// Five launches a layer -- QKV, attention, output projection, gate/up, down
// projection -- each product on v_mfma_f32_16x16x4_f32 (fp32 operands and
// sums) with its neighbours fused: RMSNorm while the operand is loaded, RoPE
// and the cache stores, residual add, SwiGLU, argmax partials.  The tiny
// decoder (2 layers, hidden 256, 25 tree nodes, 128 cached) takes 76 us a
// step; one thread per output and a launch per operation took 527.
#include <algorithm>

#include "ppd_internal.h"

namespace {

__device__ __forceinline__ floatx4 mfma4(float a, float b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0);
}

// elements k .. k + 3 of a row of n (zero past its end).  VEC: n % 4 == 0 and
// the row is 16-byte aligned.
template <bool VEC>
__device__ __forceinline__ floatx4 load4(const float *row, int k, int n) {
  if constexpr (VEC) {
    const floatx4 v = *(const floatx4 *)(row + min(k, n - 4));
    return k < n ? v : floatx4{0.f, 0.f, 0.f, 0.f};
  } else {
    floatx4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float x = row[min(k + e, n - 1)];
      v[e] = k + e < n ? x : 0.f;
    }
    return v;
  }
}

}  // namespace

// ---- out[t][n] = sum_k A[t][k] W[n][k].  Workgroup (16 output rows, 16
// tokens); its four waves deal the columns, 16 at a time: lane l loads columns
// k + 4 (l / 16) .. + 3 of row l % 16 (weights, the A operand) and of token
// l % 16 (the B operand), and instruction e multiplies element e of both, so
// the 16 columns take four instructions.  Every launch here is bound by memory
// round trips, one for each 64 columns (the loop is not unrolled: 4 at 256
// columns, 11 at 688); the 16 x 16 tiles give the chip as many workgroups as
// the matrix has tiles, and the waves' split of the columns shortens each one's
// chain.  The waves' sums meet in LDS; wave 0 finishes the tile.
template <int KIND, bool VEC>
__global__ __launch_bounds__(256) void f32_gemm_kernel(F32Gemm g) {
  constexpr bool kNorm = KIND != GEMM_RESID;
  constexpr int S = KIND == GEMM_SWIGLU ? 2 : 1;
  __shared__ floatx4 red_s[4][S][64];
  __shared__ float ss_s[4][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int K = g.K, half = g.d / 2;
  const int tok = blockIdx.y * 16 + lr;
  // weight row of tile row r.  QKV: rows r and r + 8 (r < 8) are a RoPE pair
  // (dims i and i + d / 2 of a head part), pairs counted over all head parts.
  auto row_of = [&](int r, int q) {
    if constexpr (KIND == GEMM_QKV) {
      const int p = blockIdx.x * 8 + (r & 7);
      return (p / half) * g.d + p % half + (r < 8 ? 0 : half);
    } else {
      return (int)blockIdx.x * 16 + r + q * g.N;
    }
  };
  const int n_rows = KIND == GEMM_SWIGLU ? 2 * g.N : g.N;
  const float *w[S];
#pragma unroll
  for (int q = 0; q < S; ++q) w[q] = g.W + (size_t)min(row_of(lr, q), n_rows - 1) * K;
  const float *a = g.A + (size_t)tok * K;
  floatx4 acc[S];
#pragma unroll
  for (int q = 0; q < S; ++q) acc[q] = floatx4{0.f, 0.f, 0.f, 0.f};
  float ss = 0.f;
  for (int k0 = 16 * wave; k0 < K; k0 += 64) {
    const int k = k0 + 4 * lg;
    floatx4 b = load4<VEC>(a, k, K);
    floatx4 wv[S];
#pragma unroll
    for (int q = 0; q < S; ++q) wv[q] = load4<VEC>(w[q], k, K);
    if constexpr (kNorm) {
      const floatx4 gn = load4<VEC>(g.gain, k, K);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ss = fmaf(b[e], b[e], ss);
        b[e] *= gn[e];
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int q = 0; q < S; ++q) acc[q] = mfma4(wv[q][e], b[e], acc[q]);
  }
#pragma unroll
  for (int q = 0; q < S; ++q) red_s[wave][q][lane] = acc[q];
  if constexpr (kNorm) ss_s[wave][lane] = ss;
  __syncthreads();
  if (wave > 0) return;
  // the lane's rows 4 lg + e of the tile, token tok
#pragma unroll
  for (int q = 0; q < S; ++q)
    acc[q] = (red_s[0][q][lane] + red_s[1][q][lane]) + (red_s[2][q][lane] + red_s[3][q][lane]);
  float rs = 1.f;
  if constexpr (kNorm) {
    float s = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      s += (ss_s[i][lr] + ss_s[i][16 + lr]) + (ss_s[i][32 + lr] + ss_s[i][48 + lr]);
    rs = rsqrtf(s / (float)K + g.eps);
  }
  if constexpr (KIND == GEMM_QKV) {
    const bool upper = lane >= 32;
    const int T_half = (g.nh + 2 * g.nkv) * half;  // pairs
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int p = blockIdx.x * 8 + 4 * (lg & 1) + e;
      const int hp = p / half, i = p % half;
      float v = acc[0][e] * rs;
      // [0]: lane l % 32's value (dim i), [1]: lane l % 32 + 32's (dim i + d / 2)
      const auto pr = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
      const float x0 = __uint_as_float(pr[0]), x1 = __uint_as_float(pr[1]);
      if (p >= T_half || tok >= g.T) continue;
      if (hp < g.nh + g.nkv) {
        const float2 cs = g.rope[(size_t)tok * half + i];
        v = upper ? x1 * cs.x + x0 * cs.y : x0 * cs.x - x1 * cs.y;
      }
      const int dim = i + (upper ? half : 0);
      if (hp < g.nh)
        g.out[((size_t)tok * g.nh + hp) * g.d + dim] = v;
      else if (hp < g.nh + g.nkv)
        g.kc[((size_t)(hp - g.nh) * g.cap + g.L + tok) * g.d + dim] = v;
      else
        g.vc[((size_t)(hp - g.nh - g.nkv) * g.d + dim) * g.cap + g.L + tok] = v;
    }
  } else {
    const int n0 = blockIdx.x * 16 + 4 * lg;
    float bv = 0.f;
    int bi = -1;
    if (tok < g.T) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int n = n0 + e;
        if (n >= g.N) continue;
        const float v = acc[0][e] * rs;
        if constexpr (KIND == GEMM_SWIGLU) {
          g.out[(size_t)tok * g.N + n] = v / (1.f + expf(-v)) * (acc[1][e] * rs);
        } else if constexpr (KIND == GEMM_RESID) {
          g.out[(size_t)tok * g.N + n] += v;
        } else {
          if (g.out) g.out[(size_t)tok * g.N + n] = v;
          if (v != v) {
            atomicOr(g.status, PPD_DEV_NAN_LOGIT);
          } else if (bi < 0 || v > bv) {
            bv = v;
            bi = n;
          }
        }
      }
    }
    if constexpr (KIND == GEMM_LOGITS) {
      // merge over the 4 lane groups: larger value, then smaller index
#pragma unroll
      for (int off = 16; off <= 32; off <<= 1) {
        const float v2 = __shfl_xor(bv, off, 64);
        const int i2 = __shfl_xor(bi, off, 64);
        if (i2 >= 0 && (bi < 0 || v2 > bv || (v2 == bv && i2 < bi))) {
          bv = v2;
          bi = i2;
        }
      }
      if (lane < 16) g.amax[(size_t)blockIdx.x * gridDim.y * 16 + tok] = make_float2(bv, __int_as_float(bi));
    }
  }
}

hipError_t launch_f32_gemm(const F32Gemm &g, hipStream_t s) {
  // QKV: 8 RoPE pairs a tile
  const int tiles = g.kind == GEMM_QKV ? (g.N / 2 + 7) / 8 : (g.N + 15) / 16;
  const dim3 grid(tiles, (g.T + 15) / 16), block(256);
  // 16-byte loads: every row of the operands (A: workspace rows of K) starts on 16 bytes
  const bool vec = g.K % 4 == 0 && (((uintptr_t)g.W | (uintptr_t)g.gain | (uintptr_t)g.A) & 15) == 0;
  void (*kernel)(F32Gemm) = nullptr;
  switch (g.kind) {
    case GEMM_QKV: kernel = vec ? f32_gemm_kernel<GEMM_QKV, true> : f32_gemm_kernel<GEMM_QKV, false>; break;
    case GEMM_RESID: kernel = vec ? f32_gemm_kernel<GEMM_RESID, true> : f32_gemm_kernel<GEMM_RESID, false>; break;
    case GEMM_SWIGLU: kernel = vec ? f32_gemm_kernel<GEMM_SWIGLU, true> : f32_gemm_kernel<GEMM_SWIGLU, false>; break;
    case GEMM_LOGITS: kernel = vec ? f32_gemm_kernel<GEMM_LOGITS, true> : f32_gemm_kernel<GEMM_LOGITS, false>; break;
    default: return hipErrorInvalidValue;
  }
  hipLaunchKernelGGL(kernel, grid, block, 0, s, g);
  return hipGetLastError();
}

// ---- tree attention.  Workgroup (16 queries, head); its eight waves deal the
// 16-key blocks, each with an online softmax of its own, and meet in LDS.
// S^T[key][query] = K Q^T (keys the A operand, 16 dims four instructions, as
// above) leaves a lane with keys 4 (lane / 16) + e of query lane % 16, which is
// the B operand of O^T[dim][query] += V^T P^T with instruction e taking key
// element e of V^T's row (values are position-minor).  ND: 16-dim tiles of the
// head (rounded up to 2, 4 or 8); VK, VV: 16-byte loads of key (and query)
// rows and of value rows.
constexpr int kAttnWaves = 8;

template <int ND, bool VK, bool VV>
__global__ __launch_bounds__(64 * kAttnWaves) void f32_attention_kernel(
    const float *__restrict__ q, const float *__restrict__ kc, const float *__restrict__ vc,
    const uint64_t *__restrict__ mask, int T, int L, int cap, int nh, int nkv, int d, float *__restrict__ out) {
  __shared__ floatx4 o_s[kAttnWaves][ND][64];
  __shared__ float2 ml_s[kAttnWaves][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int lr = lane & 15, lg = lane >> 4;
  const int h = blockIdx.y, kvh = h / (nh / nkv);
  const int t = blockIdx.x * 16 + lr;
  const bool live = t < T;
  const float *kb = kc + (size_t)kvh * cap * d;
  const float *vb = vc + (size_t)kvh * d * cap;
  const float *qr = q + ((size_t)min(t, T - 1) * nh + h) * d;
  const uint64_t m0 = live ? mask[2 * t] : 0ull, m1 = live ? mask[2 * t + 1] : 0ull;
  const float scale = rsqrtf((float)d);
  floatx4 qv[ND], o[ND];
#pragma unroll
  for (int j = 0; j < ND; ++j) {
    qv[j] = load4<VK>(qr, 16 * j + 4 * lg, d);
    o[j] = floatx4{0.f, 0.f, 0.f, 0.f};
  }
  float m_run = -INFINITY, l_run = 0.f;
  const int n_keys = L + T;
  for (int k0 = 16 * wave; k0 < n_keys; k0 += 16 * kAttnWaves) {
    const float *kr = kb + (size_t)min(k0 + lr, n_keys - 1) * d;
    // single-element key loads are used as they come: all of a wide head's, and
    // their addresses, do not fit the registers beside the values
    constexpr bool kAhead = VK || ND < 8;
    floatx4 kv[kAhead ? ND : 1], vv[ND];
    floatx4 s = floatx4{0.f, 0.f, 0.f, 0.f};
    if constexpr (kAhead) {
#pragma unroll
      for (int j = 0; j < ND; ++j) kv[j] = load4<VK>(kr, 16 * j + 4 * lg, d);
    } else {
#pragma unroll
      for (int j = 0; j < ND; ++j) {
        kv[0] = load4<VK>(kr, 16 * j + 4 * lg, d);
#pragma unroll
        for (int e = 0; e < 4; ++e) s = mfma4(kv[0][e], qv[j][e], s);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // values past the last key enter as zeros (the cache there may hold anything)
    const int key = k0 + 4 * lg;
#pragma unroll
    for (int j = 0; j < ND; ++j) {
      int row = min(16 * j + lr, d - 1);
      if constexpr (!kAhead) asm volatile("" : "+v"(row));  // no addresses kept over the loop either
      const float *vr = vb + (size_t)row * cap;
      if constexpr (VV) {
        vv[j] = *(const floatx4 *)(vr + min(key, cap - 4));
#pragma unroll
        for (int e = 0; e < 4; ++e) vv[j][e] = key + e < n_keys ? vv[j][e] : 0.f;
      } else {
        vv[j] = load4<false>(vr, key, n_keys);
      }
    }
    if constexpr (kAhead) {
#pragma unroll
      for (int j = 0; j < ND; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) s = mfma4(kv[j][e], qv[j][e], s);
    }
    float bm = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int jj = key + e - L;
      const bool vis = jj < 0 || (jj < T && (((jj < 64 ? m0 >> jj : m1 >> (jj - 64)) & 1ull) != 0));
      s[e] = vis ? s[e] * scale : -INFINITY;
      bm = fmaxf(bm, s[e]);
    }
    bm = fmaxf(bm, __shfl_xor(bm, 16, 64));
    bm = fmaxf(bm, __shfl_xor(bm, 32, 64));
    const float m_new = fmaxf(m_run, bm);
    const float m_ref = m_new == -INFINITY ? 0.f : m_new;  // nothing visible yet: probabilities 0
    const float alpha = expf(m_run - m_ref);
    m_run = m_new;
    l_run *= alpha;
    floatx4 p;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[e] = expf(s[e] - m_ref);
      l_run += p[e];
    }
    float bad = 0.f;  // NaN if a value of the block is not finite
#pragma unroll
    for (int j = 0; j < ND; ++j) {
      o[j] *= alpha;
#pragma unroll
      for (int e = 0; e < 4; ++e) bad = fmaf(vv[j][e], 0.f, bad);
    }
    if (__any(bad != bad)) {
      // a key of probability 0 adds nothing, whatever its value (a node that
      // overflowed stays invisible to the nodes that do not see it)
      for (int k = 0; k < 16; ++k) {
        const int src = 16 * (k >> 2);
        const float pk = __shfl(k % 4 == 0 ? p[0] : k % 4 == 1 ? p[1] : k % 4 == 2 ? p[2] : p[3], src + lr, 64);
#pragma unroll
        for (int j = 0; j < ND; ++j) {
          const float ve = k % 4 == 0 ? vv[j][0] : k % 4 == 1 ? vv[j][1] : k % 4 == 2 ? vv[j][2] : vv[j][3];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const float v = __shfl(ve, src + 4 * lg + i, 64);
            o[j][i] = pk != 0.f ? fmaf(pk, v, o[j][i]) : o[j][i];
          }
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < ND; ++j)
#pragma unroll
        for (int e = 0; e < 4; ++e) o[j] = mfma4(vv[j][e], p[e], o[j]);
    }
  }
  // the waves meet: (m, l) per query, then wave w adds dim tiles w, w + 8, ..
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  if (lane < 16) ml_s[wave][lane] = make_float2(m_run, l_run);
#pragma unroll
  for (int j = 0; j < ND; ++j) o_s[wave][j][lane] = o[j];
  __syncthreads();
  if (!live) return;
  float M = -INFINITY;
#pragma unroll
  for (int i = 0; i < kAttnWaves; ++i) M = fmaxf(M, ml_s[i][lr].x);
  float sc[kAttnWaves], l = 0.f;  // a query sees itself: M is finite
#pragma unroll
  for (int i = 0; i < kAttnWaves; ++i) {
    sc[i] = expf(ml_s[i][lr].x - M);
    l += sc[i] * ml_s[i][lr].y;
  }
  for (int j = wave; j < ND; j += kAttnWaves) {
    floatx4 v = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < kAttnWaves; ++i) v += sc[i] * o_s[i][j][lane];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int dim = 16 * j + 4 * lg + e;
      if (dim < d) out[((size_t)t * nh + h) * d + dim] = v[e] / l;
    }
  }
}

template <int ND>
static void launch_nd(bool vk, bool vv, dim3 grid, hipStream_t s, const float *q, const float *kc, const float *vc,
                      const uint64_t *mask, int T, int L, int cap, int nh, int nkv, int d, float *out) {
  auto kernel = vk ? (vv ? f32_attention_kernel<ND, true, true> : f32_attention_kernel<ND, true, false>)
                   : (vv ? f32_attention_kernel<ND, false, true> : f32_attention_kernel<ND, false, false>);
  hipLaunchKernelGGL(kernel, grid, dim3(64 * kAttnWaves), 0, s, q, kc, vc, mask, T, L, cap, nh, nkv, d, out);
}

hipError_t launch_f32_attention(const float *q, const float *kc, const float *vc, const uint64_t *mask, int T, int L,
                                int cap, int nh, int nkv, int d, float *out, hipStream_t s) {
  const dim3 grid((T + 15) / 16, nh);
  const bool vk = d % 4 == 0 && (((uintptr_t)kc | (uintptr_t)q) & 15) == 0;
  const bool vv = cap % 4 == 0 && ((uintptr_t)vc & 15) == 0;
  if (d <= 32)
    launch_nd<2>(vk, vv, grid, s, q, kc, vc, mask, T, L, cap, nh, nkv, d, out);
  else if (d <= 64)
    launch_nd<4>(vk, vv, grid, s, q, kc, vc, mask, T, L, cap, nh, nkv, d, out);
  else
    launch_nd<8>(vk, vv, grid, s, q, kc, vc, mask, T, L, cap, nh, nkv, d, out);
  return hipGetLastError();
}

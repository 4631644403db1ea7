// Skinny-M GEMMs of the verification forward pass with fused epilogues.
// out[row][t] = sum_k W[row][k] * A[t][k] for the T <= 128 tree tokens t, on
// the gfx950 matrix cores (v_mfma_f32_16x16x32_bf16: weight rows are the
// 16-row A operand, tokens the 16-column B operand), fp32 accumulation.
//
// Precision.  Weights are bf16.  Activations enter the matrix cores as the
// sum of two bf16 parts (hi = bf16(a), lo = bf16(a - hi): about 16
// significant bits), two products per weight fragment.  A bf16 rounding of
// every activation between layers would make two correct implementations
// drift apart layer after layer (each rounding flip is a full bf16 ulp); with
// the pair the drift stays near fp32 noise at any depth.
//
// The step is bound by streaming the weights from HBM once (~T flop per byte
// at bf16, far below the MI355X ridge), so the kernel is organised around
// keeping that stream in flight from the launch's first cycle to its last:
//  * weights are pre-packed group-major (launch_pack_weight): a group is 16
//    output rows (gate/up: 16 gate rows and the matching 16 up rows), and
//    each 64-column chunk of a group is a run of 1 KB fragments in the lane
//    order of the instruction's A operand;
//  * activations come as operand planes: whoever produces an activation
//    (embedding, attention, a GEMM epilogue) splits it once into (hi, lo) and
//    stores both parts in the lane order of the B operand (plane_off in
//    ppd_internal.h), norm consumers' operands already times the gain.  So
//    the main loop is loads and matrix instructions only: no conversion, no
//    LDS, no barrier;
//  * a workgroup owns a tile of groups and a K slice; its four waves (one per
//    SIMD) all hold the whole tile and deal the slice's 32-column steps among
//    themselves, KP at a time (a slab), so every weight and activation
//    fragment is loaded once per workgroup, straight into the registers of
//    the one wave that multiplies it, and the waves never wait for one
//    another.  A compute unit returns its loads in order, so an L2 hit (the
//    activations, the same for all tiles of an XCD) waits for the HBM loads
//    ahead of it: L2 hits alone reach 130 GB/s on a compute unit, mixed with
//    the weight stream 40, and the activations become the bound from
//    T = 48 on.  The waves' sums are added through
//    LDS at the end.
//  * the groups are dealt to eight workgroup sets b % 8 (each runs on one
//    XCD: the dispatcher deals workgroups round-robin over the XCDs) and,
//    within a set, to TX tiles x s K-slices.  s = 1 needs no exchange between
//    workgroups; s > 1 trades one (partial sums through the XCD's L2 behind a
//    counter, a bounded wait) for 1 / s of the activation bytes per workgroup
//    (plan_gemm chooses; two_slice_gw: tiles with a cheaper exchange);
//  * epilogues: RMSNorm row scale, RoPE + query / key / value stores into the
//    cache (QKV), residual add, the next norm's operand planes and sums of
//    squares (output / down projections), SwiGLU into operand planes
//    (gate/up), logits + per-tile argmax (LM head).
//
// Measured (us a launch; in brackets with fp32 activations, split, staged
// through LDS and behind a barrier per chunk in every workgroup, as this
// kernel did before): 7B, T = 1: QKV 20.0 (25.6), output 11.1 and down
// projection 21.2 (18.2 on average), gate/up 31.6 (37.6); T = 64: QKV 31.1
// (31.3), output 16.7 (18.5), down 30.4 (32.0), gate/up 41.3 (43.7), LM head
// 57.0 (62.7); 13B, T = 128: QKV 60 (77), gate/up 89 (123), LM head 119
// (134).  What bounds it: up to T = 32 the HBM stream (5.7 TB/s over a gate/up
// launch at T = 1), beyond that the compute unit's load path, which the
// activations share.
#include <algorithm>

#include "ppd_internal.h"

namespace {

constexpr int KC = 64;    // columns of a packed chunk: two MFMA k-steps
constexpr int NW = 4;     // waves of a GEMM workgroup
constexpr int NT = 64 * NW;
constexpr int FRAG = 64;  // u32x4 per packed operand fragment (1 KB)

template <int KIND>
constexpr int SUB = KIND == GEMM_SWIGLU ? 2 : 1;  // 16-row sub-tiles per group

__device__ __forceinline__ void amax_merge(float &v, int &i, float v2, int i2) {
  if (i2 >= 0 && (i < 0 || v2 > v || (v2 == v && i2 < i))) {
    v = v2;
    i = i2;
  }
}

// weight row held by row r (< 16) of sub-tile q of group grp; rows past the
// matrix are padding (zero weights, no output)
template <int KIND>
__device__ __forceinline__ int group_row(int grp, int q, int r, int N) {
  if constexpr (KIND == GEMM_SWIGLU) {
    const int f = grp * 16 + r;  // feature
    return f >= N ? 2 * N : q == 0 ? f : N + f;
  } else if constexpr (KIND == GEMM_QKV) {
    // group gs: dims 8 (gs % 8) .. + 7 of head part gs / 8 in rows 0..7 and
    // their RoPE partners (+ 64) in rows 8..15, so a pair lies in lanes l
    // and l + 32 of the accumulator
    return (grp >> 3) * 128 + (r < 8 ? 0 : 64) + 8 * (grp & 7) + (r & 7);
  } else {
    return grp * 16 + r;
  }
}

// ---- RMSNorm row scale r[t] = 1/sqrt(mean(x^2) + eps) from the producer's
// partial sums of squares ss[p][T_pad], p < n_ss: thread (quad of tokens,
// residue j) adds partials j, j + NJ, .. in order, then the NJ sums are added
// in order.  The first RS_N partials of a thread are requested between the
// first slabs (rs_request).
constexpr int RS_N = 8;

template <int MT>
__device__ __forceinline__ void rs_request(const GemmLaunch &g, floatx4 (&v)[RS_N]) {
  constexpr int NQ = MT * 4, NJ = NT / NQ, T_pad = MT * 16;
  const int q = threadIdx.x % NQ, j = threadIdx.x / NQ;
  // past n_ss: beyond the resource, zeros
  const __amdgpu_buffer_rsrc_t r = rsrc_of(g.ss, (uint32_t)(g.n_ss * T_pad * 4));
#pragma unroll
  for (int i = 0; i < RS_N; ++i)
    v[i] = __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(
                                           r, ((j + NJ * i) * T_pad + 4 * q) * 4, 0, 0));
}

template <int MT>
__device__ __forceinline__ void rs_finish(const GemmLaunch &g, const floatx4 (&v)[RS_N], float *tmp,
                                          float *rs_s) {
  constexpr int NQ = MT * 4, NJ = NT / NQ, T_pad = MT * 16;
  const int tid = threadIdx.x, q = tid % NQ, j = tid / NQ;
  floatx4 s = v[0];
#pragma unroll
  for (int i = 1; i < RS_N; ++i) s += v[i];
  if (j < NJ) {
    for (int p = j + NJ * RS_N; p < g.n_ss; p += NJ) s += *(const floatx4 *)(g.ss + (size_t)p * T_pad + 4 * q);
    *(floatx4 *)(tmp + j * T_pad + 4 * q) = s;
  }
  __syncthreads();
  if (tid < T_pad) {
    float t = 0.f;
    for (int i = 0; i < NJ; ++i) t += tmp[i * T_pad + tid];
    rs_s[tid] = rsqrtf(t * g.inv_h + g.eps);
  }
  __syncthreads();
}

// ---- inputs of an item's epilogue that come from memory, requested before
// the sums meet: the residual row and the next norm's gains (output / down
// projections), the RoPE angles (QKV)
template <int KIND>
struct EpiIn {};
template <>
struct EpiIn<GEMM_QKV> {
  floatx4 cs[2];  // (cos, sin) of dims i0 .. i0 + 3
};
template <>
struct EpiIn<GEMM_RESID> {
  floatx4 x;
  uint2 gain;
};

// where the keys and values of one token go (QKV): its sequence's cache and
// the position L + local index.  The lookup is the same for every item of a
// token block, so a wave keeps its last block's.
struct TokenSlot {
  int m = -1;
  bf16_t *k, *v;
  int cap, pos;
};
__device__ __forceinline__ void find_slot(const GemmLaunch &g, int m, TokenSlot &t) {
  if (m == t.m) return;  // uniform
  const int tk = m * 16 + (threadIdx.x & 15);
  t.m = m;
  t.k = g.sb.k[0];
  t.v = g.sb.v[0];
  t.cap = g.sb.cap[0];
  t.pos = g.sb.L[0] + tk;
  for (int j = 1; j < g.sb.B; ++j)
    if (tk >= g.sb.t0[j]) {
      t.k = g.sb.k[j];
      t.v = g.sb.v[j];
      t.cap = g.sb.cap[j];
      t.pos = g.sb.L[j] + tk - g.sb.t0[j];
    }
}

template <int KIND>
__device__ __forceinline__ void epi_load(const GemmLaunch &g, int grp, int m, EpiIn<KIND> &in) {
  const int lane = threadIdx.x & 63;
  const int tk = m * 16 + (lane & 15);
  if constexpr (KIND == GEMM_QKV) {
    const int i0 = 8 * (grp & 7) + 4 * ((lane >> 4) & 1);
    const floatx4 *rp = (const floatx4 *)(g.rope + (size_t)tk * 64 + i0);
    in.cs[0] = rp[0];
    in.cs[1] = rp[1];
  } else if constexpr (KIND == GEMM_RESID) {
    const int n = grp * 16 + (lane >> 4) * 4;  // N is a multiple of 128: always a row of the matrix
    in.x = *(const floatx4 *)(g.x + (size_t)tk * g.N + n);
    in.gain = *(const uint2 *)(g.gain + n);
  }
}

// ---- epilogue of item (group grp, token block m) from its complete sums
// a[q]: the lane holds rows 4 (lane / 16) + e of sub-tile q, token
// 16 m + lane % 16.  One wave, no barriers.  What a reduction over the
// tile's rows needs goes to red[16], one entry per token: the LM head's best
// (value, index), the output / down projections' sum of squares.
template <int KIND>
__device__ __forceinline__ void epilogue(const GemmLaunch &g, int grp, int m, const floatx4 (&a)[SUB<KIND>],
                                         const float *rs_s, const EpiIn<KIND> &in, float2 *red,
                                         const TokenSlot &st) {
  const int lane = threadIdx.x & 63;
  const int lr = lane & 15, r4 = (lane >> 4) * 4;
  const int T = g.T;
  const int tk = m * 16 + lr;
  if constexpr (KIND == GEMM_QKV) {
    const int nh = g.nh, nkv = g.nkv;
    const bool upper = lane >= 32;  // rows 8..15: the RoPE partner dims (+64)
    const float rs = rs_s[tk];      // finite for padding tokens too
    const int hp = grp >> 3;        // head part: q heads, then k, then v
    const int i0 = 8 * (grp & 7) + 4 * ((lane >> 4) & 1);
    const int d0 = i0 + (upper ? 64 : 0);  // this lane's dims d0 .. d0 + 3
    float v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) v[e] = a[0][e] * rs;
    if (hp < nh + nkv) {
      const float cs[8] = {in.cs[0][0], in.cs[0][1], in.cs[0][2], in.cs[0][3],
                           in.cs[1][0], in.cs[1][1], in.cs[1][2], in.cs[1][3]};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        // [0]: lane l % 32's value (dim i), [1]: lane l % 32 + 32's (dim i + 64)
        const auto pr = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[e]), __float_as_uint(v[e]),
                                                         false, false);
        const float x0 = __uint_as_float(pr[0]), x1 = __uint_as_float(pr[1]);
        const float c = cs[2 * e], sn = cs[2 * e + 1];
        v[e] = upper ? x1 * c + x0 * sn : x0 * c - x1 * sn;
      }
    }
    if (tk >= T) return;
    if (hp < nh) {
      store_plane4(g.q, g.MT, tk, hp * 128 + d0, v);
      return;
    }
    const int cap = st.cap, pos = st.pos;
    if (hp < nh + nkv) {
      bf16_t *dst = st.k + ((size_t)(hp - nh) * cap + pos) * 128;
      *(u32x2 *)(dst + d0) = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
    } else {
      bf16_t *vb = st.v + (size_t)(hp - nh - nkv) * 128 * cap + pos;
#pragma unroll
      for (int e = 0; e < 4; ++e) vb[(size_t)(d0 + e) * cap] = f32_to_bf16(v[e]);
    }
  } else if constexpr (KIND == GEMM_SWIGLU) {
    const int f0 = grp * 16 + r4;
    if (tk >= T || f0 >= g.N) return;
    const float rs = rs_s[tk];
    float o[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float gt_ = a[0][e] * rs, up = a[1][e] * rs;
      o[e] = gt_ / (1.f + expf(-gt_)) * up;
    }
    store_plane4(g.planes, g.MT, tk, f0, o);
  } else if constexpr (KIND == GEMM_RESID) {
    const int n = grp * 16 + r4;
    float sq = 0.f;
    if (tk < T) {
      const floatx4 xv = in.x + a[0];
      *(floatx4 *)(g.x + (size_t)tk * g.N + n) = xv;
      sq = (xv[0] * xv[0] + xv[1] * xv[1]) + (xv[2] * xv[2] + xv[3] * xv[3]);
      const float o[4] = {xv[0] * bf16_to_f32(in.gain.x & 0xffff), xv[1] * bf16_to_f32(in.gain.x >> 16),
                          xv[2] * bf16_to_f32(in.gain.y & 0xffff), xv[3] * bf16_to_f32(in.gain.y >> 16)};
      store_plane4(g.planes, g.MT, tk, n, o);
    }
    // the group's 16 rows: one partial sum of squares per token
    sq += __shfl_xor(sq, 16, 64);
    sq += __shfl_xor(sq, 32, 64);
    if (lane < 16) red[lane].x = sq;
  } else {  // GEMM_LOGITS
    const int n = grp * 16 + r4;
    float bv = 0.f;
    int bi = -1;
    if (tk < T) {
      const float rs = rs_s[tk];
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = a[0][e] * rs;
      if (g.logits) {
        if ((g.N & 3) == 0 && n + 3 < g.N) {
          *(floatx4 *)(g.logits + (size_t)tk * g.N + n) = floatx4{v[0], v[1], v[2], v[3]};
        } else {
          for (int e = 0; e < 4; ++e)
            if (n + e < g.N) g.logits[(size_t)tk * g.N + n + e] = v[e];
        }
      }
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        if (n + e < g.N) {
          if (v[e] != v[e]) {
            atomicOr(g.status, PPD_DEV_NAN_LOGIT);
          } else if (bi < 0 || v[e] > bv) {
            bv = v[e];
            bi = n + e;
          }
        }
      }
    }
    // merge over the 4 lane groups: larger value, then smaller index
#pragma unroll
    for (int off = 16; off <= 32; off <<= 1) {
      const float v2 = __shfl_xor(bv, off, 64);
      const int i2 = __shfl_xor(bi, off, 64);
      amax_merge(bv, bi, v2, i2);
    }
    if (lane < 16) red[lane] = make_float2(bv, __int_as_float(bi));
  }
}

// buffer-load offset of a lane whose load is to be dropped: past every
// resource's range (each is below 2 GB), with or without the scalar offset
// added, so the load returns zeros and touches no memory
constexpr uint32_t kDropped = 0x80000000u;

// Register buffers of a wave.  `steps` k-steps of fragments (weights and
// activations) fit beside the accumulators and among the 64 loads a wave can
// have outstanding; they are used as three slabs of KP steps, two where no
// more fit.  Where not even two steps fit (the largest
// tile of 128 tokens), one step's activations and two steps' weights are kept
// (NB = 1).  Measured, 7B layers with T = 64 / 48 / 32 / 1 (us a step of 4): 3
// slabs of 1 / 1 / 2 / 8 steps 613 / 580 / 521 / 464, two of twice the steps
// 613 / 579 / 543 / 481, activations in one buffer and weights in two of 4 to
// 8 steps 642 / 605 / 546 / 479.
constexpr int buf_steps(int MT, int WF) {
  // twelve weight fragments a step or more: ten registers of addresses more
  // (gate/up tiles of 6 groups with four token blocks spilled 12 bytes a lane
  // and took 28.3 us a launch at 4096 x 4288, 65.6 at 4096 x 20480, T = 64; now
  // 26.8 and 61.9)
  return std::min((WF < 12 ? 440 : 430) - 4 * WF * MT, 4 * 66) / (4 * (WF + 2 * MT));
}
constexpr int slab_steps(int MT, int WF) {
  return std::max(1, std::min({(MT == 1 ? 16 : 8) / (2 * MT), buf_steps(MT, WF) / 3}));
}
constexpr int slab_bufs(int MT, int WF) {
  return std::min(3, std::max(1, buf_steps(MT, WF) / slab_steps(MT, WF)));
}

// ---- the GEMM.  Workgroup b: XCD x = b % 8, slot j = b / 8 -> tile
// t = j / s (groups [ga, gb) of the XCD's range, at most GW), K slice
// ks = j % s (k-steps [u0, u1)).
// TWO: the tile comes in two slices, each keeping the sums it finishes in LDS.
template <int MT, int KIND, int GW, bool FEW, bool TWO>
__global__ __launch_bounds__(NT, 1) void gemm_bf16_kernel(GemmLaunch g) {
  constexpr int T_pad = MT * 16;
  constexpr int S = SUB<KIND>, WF = GW * S;
  constexpr int KP = slab_steps(MT, WF), NB = slab_bufs(MT, WF);
  constexpr bool kNorm = KIND != GEMM_RESID;  // rows scaled in the epilogue
  // the waves' sums meet in LDS, MR token blocks a round (at most 96 KB)
  constexpr int MR = std::max(1, std::min(MT, 96 / (NW * WF)));
  constexpr int ITEMS = GW * MR;  // per round
  constexpr int PI = (ITEMS + NW - 1) / NW;
  __shared__ __attribute__((aligned(16))) float red_s[NW * WF * MR * 256];
  __shared__ float rs_tmp[NT * 4];
  __shared__ float rs_s[T_pad];
  constexpr bool kRows = KIND == GEMM_LOGITS || KIND == GEMM_RESID;  // reductions over the tile's rows
  __shared__ float2 item_s[kRows ? GW * MT * 16 : 1];
  // TWO: the sums of the items this slice finishes
  __shared__ __attribute__((aligned(16))) float own_s[TWO ? (GW * MT + 1) / 2 * S * 256 : 4];

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int x = blockIdx.x & 7, j = blockIdx.x >> 3;
  // slot j -> tile t, slice ks (s = 1 << ls); the XCD's groups [g0, g0 + nx)
  // in TX runs of nx / TX groups, the first nx % TX of one more (nx is one of
  // two values: both quotients come from the host)
  const int ls = g.ls, s = 1 << ls;
  const int t = j >> ls, ks = j & (s - 1);
  const int gt = x * g.TX + t;  // global tile index
  const int g0 = (g.G * x) >> 3, nx = ((g.G * (x + 1)) >> 3) - g0;
  const bool more = nx > (g.G >> 3);
  const int hq = more ? g.q1 : g.q0, hr = more ? g.r1 : g.r0;
  const int ga = g0 + t * hq + min(t, hr), ng = hq + (t < hr ? 1 : 0), gb = ga + ng;
  const int kc = g.kc;
  const int u0 = (2 * kc * ks) >> ls, u1 = (2 * kc * (ks + 1)) >> ls;
  // Which slice finishes item (group i, token block m) of a split tile: the
  // items in turn; where the tile's rows are reduced, (m R + i % R) % s with
  // R = ceil(s / MT), so that the reduction of a token block over groups
  // i % R = r, one output row per (tile, r), stays in one slice.
  const int R = kRows ? (s + MT - 1) / MT : 1;
  auto row_slice = [&](int i, int m) { return (m * R + i % R) & (s - 1); };
  auto rows_out = [&](int n) {  // the tile's reductions, from its items in item_s
    for (int o = tid; o < R * T_pad; o += NT) {
      const int r = o / T_pad, tk = o % T_pad, m = tk >> 4;
      if (row_slice(r, m) != ks) continue;
      const size_t at = (size_t)(gt * R + r) * T_pad + tk;
      if constexpr (KIND == GEMM_RESID) {
        float v = 0.f;
        for (int i = r; i < n; i += R) v += item_s[(i * MT + m) * 16 + (tk & 15)].x;
        g.ss_out[at] = v;
      } else {
        float v = 0.f;
        int bi = -1;
        for (int i = r; i < n; i += R) {
          const float2 c = item_s[(i * MT + m) * 16 + (tk & 15)];
          amax_merge(v, bi, c.x, __float_as_int(c.y));
        }
        g.amax[at] = make_float2(v, __int_as_float(bi));
      }
    }
  };
  if (ng <= 0) {  // no groups on this tile: neutral rows
    if constexpr (kRows) rows_out(0);
    return;
  }

  // ---- the wave's k-steps u0 + (slab NW + wave) KP + k, k < KP: weight
  // fragments (group i, sub-tile q) and activation fragments (token block m,
  // part p).  Steps past the slice and groups past the tile are dropped loads
  // (zeros), so every slab issues the same instructions.
  const __amdgpu_buffer_rsrc_t wrs = rsrc_of(g.W, g.w_bytes), ars = rsrc_of(g.A, g.a_bytes);
  uint32_t wo[GW];
  int wg[GW];  // the group's first fragment
#pragma unroll
  for (int i = 0; i < GW; ++i) {
    wo[i] = i < ng ? lane * 16 : kDropped;
    wg[i] = min(ga + i, gb - 1) * kc * 2 * S;
  }
  // FEW: lanes of padding tokens load nothing
  const uint32_t ao = !FEW || (lane & 15) < g.T ? lane * 16 : kDropped;
  const int n_slab = __builtin_amdgcn_readfirstlane((u1 - u0 + NW * KP - 1) / (NW * KP));
  u32x4 wr[NB == 1 ? 2 : NB][KP][WF], ar[NB][KP][2 * MT];
  auto request_w = [&](int n, u32x4(&w)[KP][WF]) {
#pragma unroll
    for (int k = 0; k < KP; ++k) {
      const int u = u0 + (n * NW + wave) * KP + k, uc = min(u, u1 - 1);
      const uint32_t drop = u < u1 ? 0u : kDropped;
#pragma unroll
      for (int i = 0; i < GW; ++i)
#pragma unroll
        for (int q = 0; q < S; ++q)
          w[k][i * S + q] = __builtin_amdgcn_raw_buffer_load_b128(
              wrs, (int)(wo[i] | drop), (wg[i] + (uc >> 1) * 2 * S + 2 * q + (uc & 1)) << 10, 2);
    }
  };
  auto request_a = [&](int n, u32x4(&a)[KP][2 * MT]) {
    const int u = u0 + (n * NW + wave) * KP;
#pragma unroll
    for (int k = 0; k < KP; ++k) {
      const int uc = min(u + k, u1 - 1);
      const uint32_t drop = u + k < u1 ? 0u : kDropped;
#pragma unroll
      for (int m = 0; m < 2 * MT; ++m)
        a[k][m] = __builtin_amdgcn_raw_buffer_load_b128(ars, (int)(ao | drop), (uc * 2 * MT + m) << 10, 0);
    }
  };
  floatx4 acc[GW][S][MT];
#pragma unroll
  for (int i = 0; i < GW; ++i)
#pragma unroll
    for (int q = 0; q < S; ++q)
#pragma unroll
      for (int m = 0; m < MT; ++m) acc[i][q][m] = floatx4{0.f, 0.f, 0.f, 0.f};

  // one slab: the smaller parts' products first, then the larger parts', so
  // that consecutive instructions add to different accumulators
  auto multiply = [&](const u32x4(&w)[KP][WF], const u32x4(&a)[KP][2 * MT]) {
#pragma unroll
    for (int k = 0; k < KP; ++k)
#pragma unroll
      for (int p = 1; p >= 0; --p)
#pragma unroll
        for (int i = 0; i < GW; ++i)
#pragma unroll
          for (int q = 0; q < S; ++q)
#pragma unroll
            for (int m = 0; m < MT; ++m)
              acc[i][q][m] = mfma16x16x32(as_bf16x8(w[k][i * S + q]), as_bf16x8(a[k][2 * m + p]), acc[i][q][m]);
  };

  [[maybe_unused]] floatx4 ssv[RS_N];
#pragma unroll
  for (int d = 0; d < NB; ++d) {
    request_a(d, ar[d]);
    __builtin_amdgcn_sched_barrier(0);
    request_w(d, wr[d]);
    __builtin_amdgcn_sched_barrier(0);
    // behind the first slab: the stream starts first, and the row scales wait
    // for no more than the first products do
    if constexpr (kNorm)
      if (d == 0) rs_request<MT>(g, ssv);
    __builtin_amdgcn_sched_barrier(0);
  }
  if constexpr (NB == 1) request_w(1, wr[1]);
  __builtin_amdgcn_sched_barrier(0);
  if constexpr (kNorm) rs_finish<MT>(g, ssv, rs_tmp, rs_s);

  // ---- main loop: multiply slab n, then request slab n + NB into its
  // registers (NB = 1: the next activations and the weights after next)
  int n = 0;
  if constexpr (NB > 1) {
    for (; n + NB <= n_slab; n += NB) {
#pragma unroll
      for (int d = 0; d < NB; ++d) {
        multiply(wr[d], ar[d]);
        __builtin_amdgcn_sched_barrier(0);
        request_a(n + d + NB, ar[d]);
        __builtin_amdgcn_sched_barrier(0);
        request_w(n + d + NB, wr[d]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
#pragma unroll
    for (int d = 0; d < NB - 1; ++d)
      if (n + d < n_slab) multiply(wr[d], ar[d]);
  } else {
    auto turn = [&](int i, u32x4(&w)[KP][WF]) {
      multiply(w, ar[0]);
      __builtin_amdgcn_sched_barrier(0);
      request_a(i + 1, ar[0]);
      __builtin_amdgcn_sched_barrier(0);
      request_w(i + 2, w);
      __builtin_amdgcn_sched_barrier(0);
    };
    for (; n + 2 <= n_slab; n += 2) {
      turn(n, wr[0]);
      turn(n + 1, wr[1]);
    }
    if (n < n_slab) multiply(wr[0], ar[0]);
  }

  // ---- the waves' sums meet: item idx = (group i, token block m) of a
  // round; wave (idx / s) % NW adds its NW parts in wave order.  s = 1: it
  // then finishes the item.  s > 1: it stores the sum to the XCD's L2; after
  // the tile's slices have met at the counter, slice idx % s (of the whole
  // tile's items) adds the s sums in slice order and finishes the item.  Partial sums: [tile][slice][item][q][lane] floatx4.
  [[maybe_unused]] TokenSlot slot;
  // (TWO: one sum an item, the slice's that does not finish it: [tile][item][q][lane])
  constexpr int kPart = GW * MT * S * 256;  // floats per workgroup
  float *part = g.part + (TWO ? (size_t)gt : (size_t)gt * s + ks) * kPart;
#pragma unroll
  for (int m0 = 0; m0 < MT; m0 += MR) {
    if (m0 > 0) __syncthreads();
    EpiIn<KIND> in[PI];
    if (s == 1) {
#pragma unroll
      for (int jj = 0; jj < PI; ++jj) {
        const int idx = min(jj * NW + wave, ITEMS - 1);
        if (KIND == GEMM_QKV && jj == 0) find_slot(g, min(m0 + idx % MR, MT - 1), slot);
        epi_load<KIND>(g, min(ga + idx / MR, gb - 1), min(m0 + idx % MR, MT - 1), in[jj]);
      }
    }
#pragma unroll
    for (int i = 0; i < GW; ++i)
#pragma unroll
      for (int r = 0; r < MR; ++r)
        if (m0 + r < MT) {
#pragma unroll
          for (int q = 0; q < S; ++q)
            *(floatx4 *)(red_s + (((wave * GW + i) * MR + r) * S + q) * 256 + lane * 4) = acc[i][q][m0 + r < MT ? m0 + r : 0];
        }
    __syncthreads();
    auto sum_item = [&](int idx, floatx4(&a)[S]) {
#pragma unroll
      for (int q = 0; q < S; ++q) {
        a[q] = *(const floatx4 *)(red_s + (idx * S + q) * 256 + lane * 4);
#pragma unroll
        for (int w = 1; w < NW; ++w)
          a[q] += *(const floatx4 *)(red_s + ((w * ITEMS + idx) * S + q) * 256 + lane * 4);
      }
    };
    if (s == 1) {
#pragma unroll
      for (int jj = 0; jj < PI; ++jj) {
        const int idx = jj * NW + wave;
        const int i = idx / MR, m = m0 + idx % MR;
        if (idx < ITEMS && i < ng && m < MT) {
          floatx4 a[S];
          sum_item(idx, a);
          if constexpr (KIND == GEMM_QKV) find_slot(g, m, slot);
          epilogue<KIND>(g, ga + i, m, a, rs_s, in[jj], item_s + (kRows ? (i * MT + m) * 16 : 0), slot);
        }
      }
      continue;
    }
    for (int o = 0; o < ITEMS; o += s * NW)  // this wave's items: o + wave s + (0 .. s - 1)
      for (int sl = 0; sl < s; ++sl) {
        const int idx = o + wave * s + sl;
        const int i = idx / MR, m = m0 + idx % MR;
        if (idx >= ITEMS || i >= ng || m >= MT) continue;
        floatx4 a[S];
        sum_item(idx, a);
        float *dst = part + (size_t)(i * MT + m) * S * 256;
        if constexpr (TWO)
          if (((i * MT + m) & 1) == ks) dst = own_s + ((i * MT + m) >> 1) * S * 256;
#pragma unroll
        for (int q = 0; q < S; ++q) *(floatx4 *)(dst + q * 256 + lane * 4) = a[q];
      }
  }
  if (s > 1) {
    // this slice's items, dealt to its waves in turn: the s partial sums are
    // added in slice order; the next item's are requested while this one is
    // finished.  Its own sums make the round trip with the others' (one code
    // for every s: where s is 4 or 8 that costs nothing measurable), except
    // with TWO
    const int nb = (ng + R - 1) / R;  // groups of a class (m, i % R)
    const int n_own = kRows ? ((MT * R - ks + s - 1) >> ls) * nb : (ng * MT - ks + s - 1) >> ls;
    auto item_at = [&](int n, int &i, int &m) {
      if constexpr (kRows) {
        const int c = ks + s * (n / nb);
        m = c / R;
        i = c % R + R * (n % nb);
      } else {
        i = (ks + s * n) / MT;
        m = (ks + s * n) % MT;
      }
      return i < ng;
    };
    EpiIn<KIND> in[2];
    constexpr int NP = TWO ? 1 : 8;  // sums that come from L2 (TWO: the other slice's)
    floatx4 buf[2][NP][S];
    const __amdgpu_buffer_rsrc_t rp = rsrc_of(g.part + (size_t)gt * (TWO ? 1 : s) * kPart,
                                               (uint32_t)(TWO ? 1 : s) * kPart * 4);
    auto ask_sums = [&](int n, floatx4(&d)[NP][S]) {
      int i, m;
      const uint32_t drop = n < n_own && item_at(n, i, m) ? 0u : kDropped;
      if (drop) i = m = 0;
#pragma unroll
      for (int sl = 0; sl < NP; ++sl)
#pragma unroll
        for (int q = 0; q < S; ++q)  // past the last slice: beyond the resource, zeros
          d[sl][q] = load_l2(rp, (uint32_t)(sl * kPart * 4 + ((i * MT + m) * S + q) * 1024 + lane * 16) | drop);
    };
    auto ask_inputs = [&](int n, EpiIn<KIND> &e) {
      int i, m;
      if (n < n_own && item_at(n, i, m)) epi_load<KIND>(g, ga + i, m, e);
    };
    auto finish = [&](int n, const floatx4(&d)[NP][S], const EpiIn<KIND> &e) {
      int i, m;
      if (n >= n_own || !item_at(n, i, m)) return;
      floatx4 a[S];
#pragma unroll
      for (int q = 0; q < S; ++q) {
        a[q] = d[0][q];
        if constexpr (TWO) a[q] += *(const floatx4 *)(own_s + (n * S + q) * 256 + lane * 4);
#pragma unroll
        for (int sl = 1; sl < NP; ++sl) a[q] += d[sl][q];
      }
      if constexpr (KIND == GEMM_QKV) find_slot(g, m, slot);
      epilogue<KIND>(g, ga + i, m, a, rs_s, e, item_s + (kRows ? (i * MT + m) * 16 : 0), slot);
    };
    ask_inputs(wave, in[0]);
    ask_inputs(wave + NW, in[1]);
    asm volatile("" ::: "memory");
    __builtin_amdgcn_s_waitcnt(0);  // this thread's partial stores have reached L2
    __syncthreads();
    // one 128-byte line of counters per group of XCD slots
    if (tid == 0) xcd_arrive_wait(g.ctr + x * 32 + t, x, (uint32_t)s, g.spin_limit, g.status);
    __syncthreads();
    ask_sums(wave, buf[0]);
    for (int n = wave; n < n_own; n += 2 * NW) {
      ask_sums(n + NW, buf[1]);
      __builtin_amdgcn_sched_barrier(0);
      finish(n, buf[0], in[0]);
      ask_sums(n + 2 * NW, buf[0]);
      ask_inputs(n + 2 * NW, in[0]);
      __builtin_amdgcn_sched_barrier(0);
      finish(n + NW, buf[1], in[1]);
      ask_inputs(n + 3 * NW, in[1]);
    }
  }
  if constexpr (kRows) {
    __syncthreads();
    rows_out(ng);
  }
}

template <int MT, int KIND, int GW, bool FEW = false, bool TWO = false>
hipError_t launch_one(const GemmLaunch &g, hipStream_t s) {
  const dim3 grid(8 * g.TX << g.ls), block(NT);
  hipEvent_t ev0 = (hipEvent_t)g.ev_start, ev1 = (hipEvent_t)g.ev_stop;
  if (ev0)
    hipExtLaunchKernelGGL((gemm_bf16_kernel<MT, KIND, GW, FEW, TWO>), grid, block, 0, s, ev0, ev1, 0, g);
  else
    hipLaunchKernelGGL((gemm_bf16_kernel<MT, KIND, GW, FEW, TWO>), grid, block, 0, s, g);
  return hipGetLastError();
}

// groups per tile instantiated for S sub-tiles and MT token tiles: the
// accumulators (4 GW S MT registers), a step's activations and two steps'
// weights must fit one wave's registers
constexpr int gw_limit(int S, int MT) { return S == 1 ? (MT <= 7 ? 8 : 6) : MT <= 4 ? 6 : 4; }

// Tiles of seven groups or more in two slices (TWO): QKV with two to seven token
// blocks, gate/up with four.  The sums a slice finishes stay in its LDS; with
// all of them on the round trip through L2, and six dropped loads an item, two
// slices were not worth it.  13B, T = 56, us a launch whole, in two slices, so:
// QKV 42.1, 40.5, 39.7; gate/up 59.5, 59.2, 57.9; a step of 40 layers 7450 ->
// 7240.  Not for smaller tiles (7B, T = 96, QKV: 0.5 us a layer lost) nor
// gate/up with three token blocks (4608 and 5120 columns: 0.6 to 1 % of a step
// lost).
constexpr int two_slice_gw(int kind, int MT) {
  return kind == GEMM_QKV && MT >= 2 && MT <= 7 ? 8 : kind == GEMM_SWIGLU && MT == 4 ? 7 : 0;
}

// Up to this many tokens (one block, half of it padding or more) the padding
// tokens' lanes of the activation loads are masked (FEW): with one token a
// workgroup of the 7B down projection otherwise loads twice its weight bytes
// for 15 tokens that do not exist.  Four 7B layers, us a step with the mask
// (without): T = 1 430.7 (442.0).  Beyond, little is saved and the masked
// offset costs: T = 16 of the 1.4B width 241.9 (239.0), 7B T = 32 501.4
// (499.1), 1.4B T = 80 1890 (1876).
constexpr int kFewTokens = 8;

template <int MT, int KIND>
hipError_t launch_mt(const GemmLaunch &g, hipStream_t s) {
  constexpr int LIM = gw_limit(SUB<KIND>, MT), TGW = two_slice_gw(KIND, MT);
  if constexpr (TGW > 0)
    if (g.gw == TGW && g.ls == 1) return launch_one<MT, KIND, TGW, false, true>(g, s);
  switch (g.gw) {
#define PPD_GW(n)                                                        \
  case n:                                                                \
    if constexpr (MT == 1 && LIM >= n)                                   \
      if (g.T <= kFewTokens) return launch_one<MT, KIND, n, true>(g, s); \
    if constexpr (LIM >= n) return launch_one<MT, KIND, n>(g, s);        \
    break;
    PPD_GW(1) PPD_GW(2) PPD_GW(3) PPD_GW(4) PPD_GW(6) PPD_GW(8)
#undef PPD_GW
  }
  return hipErrorInvalidValue;
}

template <int KIND>
hipError_t launch_kind(const GemmLaunch &g, hipStream_t s) {
  switch (g.MT) {
    case 1: return launch_mt<1, KIND>(g, s);
    case 2: return launch_mt<2, KIND>(g, s);
    case 3: return launch_mt<3, KIND>(g, s);
    case 4: return launch_mt<4, KIND>(g, s);
    case 5: return launch_mt<5, KIND>(g, s);
    case 6: return launch_mt<6, KIND>(g, s);
    case 7: return launch_mt<7, KIND>(g, s);
    case 8: return launch_mt<8, KIND>(g, s);
  }
  return hipErrorInvalidValue;
}

// ---- weight packing.  Packed 16-byte item (group, chunk, sub-tile q < S,
// k-step s < 2, lane l < 64) holds the 8 bf16 of weight row
// group_row(group, q, l % 16) at columns 64 chunk + 32 s + 8 (l / 16) .. + 7;
// rows past the matrix are zero.
template <int KIND>
__global__ __launch_bounds__(256) void pack_kernel(const bf16_t *__restrict__ src, u32x4 *__restrict__ dst,
                                                   int N, int K, int rows_total, int kc, long n_items) {
  constexpr int S = SUB<KIND>;
  for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n_items;
       i += (long)gridDim.x * blockDim.x) {
    const int l = (int)(i & 63);
    const long f = i >> 6;  // fragment ((group kc + chunk) S + q) 2 + s
    const int st = (int)(f & 1), q = (int)((f >> 1) % S);
    const long gc = f / (2 * S);
    const int chunk = (int)(gc % kc), grp = (int)(gc / kc);
    const int row = group_row<KIND>(grp, q, l & 15, N);
    const int col = chunk * KC + 32 * st + 8 * (l >> 4);
    u32x4 v = u32x4{0u, 0u, 0u, 0u};
    if (row < rows_total && col < K) v = *(const u32x4 *)(src + (size_t)row * K + col);
    dst[i] = v;
  }
}

template <int KIND>
hipError_t launch_pack_kind(int N, int K, const bf16_t *src, bf16_t *dst, hipStream_t s) {
  const int G = gemm_groups_of(KIND, N), kc = K / KC;
  const long n_items = (long)G * kc * SUB<KIND> * 2 * FRAG;
  const int rows_total = KIND == GEMM_SWIGLU ? 2 * N : N;
  const dim3 grid((unsigned)std::min<long>(8192, (n_items + 255) / 256)), block(256);
  hipLaunchKernelGGL((pack_kernel<KIND>), grid, block, 0, s, src, (u32x4 *)dst, N, K, rows_total, kc,
                     n_items);
  return hipGetLastError();
}

}  // namespace

int gemm_groups_of(int kind, int N) {
  // QKV: N / 16 (head_dim 128); gate/up: 16 features per group; others 16 rows
  return (N + 15) / 16;
}

int gemm_sub_of(int kind) { return kind == GEMM_SWIGLU ? 2 : 1; }

int gemm_gw_max(int kind, int MT) { return gw_limit(gemm_sub_of(kind), MT); }
int gemm_two_slice_gw(int kind, int MT) { return two_slice_gw(kind, MT); }

hipError_t launch_pack_weight(int kind, int N, int K, const bf16_t *src, bf16_t *dst, hipStream_t s) {
  if (K % KC) return hipErrorInvalidValue;
  switch (kind) {
    case GEMM_QKV: return launch_pack_kind<GEMM_QKV>(N, K, src, dst, s);
    case GEMM_RESID: return launch_pack_kind<GEMM_RESID>(N, K, src, dst, s);
    case GEMM_SWIGLU: return launch_pack_kind<GEMM_SWIGLU>(N, K, src, dst, s);
    case GEMM_LOGITS: return launch_pack_kind<GEMM_LOGITS>(N, K, src, dst, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm_bf16(const GemmLaunch &g, hipStream_t s) {
  switch (g.kind) {
    case GEMM_QKV: return launch_kind<GEMM_QKV>(g, s);
    case GEMM_RESID: return launch_kind<GEMM_RESID>(g, s);
    case GEMM_SWIGLU: return launch_kind<GEMM_SWIGLU>(g, s);
    case GEMM_LOGITS: return launch_kind<GEMM_LOGITS>(g, s);
  }
  return hipErrorInvalidValue;
}

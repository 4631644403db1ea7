// Internal declarations shared by the HIP kernels and the host driver of
// libppd.  Device helpers: bfloat16 bit conversions (round to nearest even),
// MFMA operand types, wavefront reductions.
#pragma once

#include <hip/hip_ext.h>
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/ppd.h"

typedef uint16_t bf16_t;  // raw bfloat16 storage word
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));

#define PPD_WAVE 64

__device__ __forceinline__ float bf16_to_f32(bf16_t h) {
  return __uint_as_float(((uint32_t)h) << 16);
}

// float -> bfloat16, round to nearest, ties to even (NaN stays NaN): the
// gfx950 conversion instruction (v_cvt_pk_bf16_f32) in the default rounding
// mode
typedef __bf16 hw_bf16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ bf16_t f32_to_bf16(float f) {
  return __builtin_bit_cast(bf16_t, (__bf16)f);
}

__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
  const hw_bf16x2 v = {(__bf16)lo, (__bf16)hi};
  return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ floatx4 mfma16x16x32(bf16x8 a, bf16x8 b, floatx4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// buffer resource over a whole workspace region (raw, untyped loads)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_of(const void *p, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), (short)0, (int)bytes, 0x00020000);
}
// 16-byte load that misses L1 (sc0): data written by another compute unit of
// this XCD is read from the shared L2 (each address is read once per
// dispatch, after the writers' arrival)
__device__ __forceinline__ floatx4 load_l2(__amdgpu_buffer_rsrc_t r, uint32_t byte_off) {
  return __builtin_bit_cast(floatx4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)byte_off, 0, 1));
}

// ---- operand planes: a bf16 GEMM's activations [T_pad][K] as the B operand
// of v_mfma_f32_16x16x32_bf16, each element the sum of two bf16 parts.
// Fragment (k-step u = column / 32, token block m = token / 16, part p: 0 hi,
// 1 lo) is 1 KB; its lane l holds token 16 m + l % 16, columns 32 u + 8 (l /
// 16) .. + 7.  Order [u][m][p]; T_pad x K x 4 bytes, as fp32.
__host__ __device__ __forceinline__ size_t plane_off(int MT, int tok, int col) {
  return ((size_t)((col >> 5) * MT + (tok >> 4)) << 11) + (((tok & 15) + 16 * ((col >> 3) & 3)) << 4) +
         2 * (col & 7);
}
constexpr int kPlaneLo = 1024;  // bytes from an element's hi part to its lo part
// columns col .. col + 3 (col % 4 == 0) of token tok
__device__ __forceinline__ void store_plane4(unsigned char *planes, int MT, int tok, int col, const float (&v)[4]) {
  float lo[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) lo[e] = v[e] - bf16_to_f32(f32_to_bf16(v[e]));
  unsigned char *d = planes + plane_off(MT, tok, col);
  *(u32x2 *)d = u32x2{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3])};
  *(u32x2 *)(d + kPlaneLo) = u32x2{pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3])};
}
// columns col .. col + 7 (col % 8 == 0)
__device__ __forceinline__ void store_plane8(unsigned char *planes, int MT, int tok, int col, const float (&v)[8]) {
  float lo[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) lo[e] = v[e] - bf16_to_f32(f32_to_bf16(v[e]));
  unsigned char *d = planes + plane_off(MT, tok, col);
  *(u32x4 *)d = u32x4{pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]),
                      pack_bf16x2(v[6], v[7])};
  *(u32x4 *)(d + kPlaneLo) = u32x4{pack_bf16x2(lo[0], lo[1]), pack_bf16x2(lo[2], lo[3]),
                                   pack_bf16x2(lo[4], lo[5]), pack_bf16x2(lo[6], lo[7])};
}

// the XCD this wave runs on
__device__ __forceinline__ unsigned xcc_id() {
  unsigned v;
  asm volatile("s_getreg_b32 %0, hwreg(HW_REG_XCC_ID)" : "=s"(v));
  return v & 0xf;
}

// Arrival at an XCD-local counter shared by n workgroups of one dispatch
// (one thread per workgroup, after its results have reached L2), then a
// bounded wait for the other n - 1.  Workgroup b runs on XCD (b + o) % 8, o
// being the dispatcher's offset (round-robin from wherever the previous
// dispatch left it: the same for every workgroup of this one), so each
// arrival adds 1 + 256 o, o = (this XCD - set) mod 8; a final count whose
// high part is not n o means the workgroups did not share an XCD.  Agent
// scope: a workgroup-scope load may be served by this compute unit's L1,
// which keeps the line of the first poll.
__device__ __forceinline__ void xcd_arrive_wait(uint32_t *ctr, int set, uint32_t n, int spin_limit,
                                                uint32_t *status) {
  const uint32_t o = (xcc_id() - (unsigned)set) & 7u;
  __hip_atomic_fetch_add(ctr, 1u + (o << 8), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  int it = 0;
  uint32_t v;
  while (((v = __hip_atomic_load(ctr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) & 0xffu) < n) {
    if (++it > spin_limit) {
      atomicOr(status, PPD_DEV_SYNC_TIMEOUT);
      break;
    }
    __builtin_amdgcn_s_sleep(2);
  }
  if ((v >> 8) != o * n) atomicOr(status, PPD_DEV_XCD_PLACEMENT);
}

__device__ __forceinline__ float wave_sum(float v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, PPD_WAVE);
  return v;
}

// ---------------------------------------------------------------------------
// workspace layout (computed on the host, passed to kernels as pointers)

struct WsLayout {
  size_t status;      // uint32 [4], the workspace's header (256 bytes)
  size_t x;           // float  [T_pad][H]        residual stream
  size_t xg;          // x * gain of the next norm: operand planes [T_pad][H] (bf16 models)
  size_t ss;          // float  [max_ss][T_pad]   sum-of-squares partials
  size_t q;           // operand planes [T_pad][nh d] queries after RoPE (fp32 path: float)
  size_t attn_o;      // operand planes [T_pad][nh d] attention output (fp32 path: float)
  size_t act;         // operand planes [T_pad][F] SwiGLU output (fp32 path: float)
  size_t attn_part;   // float  [nh][max_splits][T_pad][PPD_ATTN_OROW]; the same memory as xg
  size_t gemm_part;   // partial sums of split GEMMs
  size_t amax;        // float2 [max_amax_tiles][T_pad]
  size_t rope;        // float2 [T_pad][d/2]      (cos, sin)
  size_t ctr;         // uint32 [n_ctr]           tile / head counters (zeroed per step)
  size_t n_ctr;
  size_t total;
  int max_ss, max_splits, max_amax_tiles;
};

#define PPD_ATTN_MAX_SPLITS 64

// ---------------------------------------------------------------------------
// kernel launchers (defined in the .hip files, called by the host driver)

// Skinny GEMM partition (k_gemm.hip).  Weights are packed group-major: a
// group is 16 output rows (gate/up: 16 features, i.e. 16 gate and 16 up
// rows), each of its K / 64 chunks a run of 1 KB MFMA fragments.  The groups
// are dealt to the 8 XCDs (XCD x: groups [G x / 8, G (x + 1) / 8)); on each XCD,
// TX tiles (consecutive groups, at most gw) x s K-slices take its TX s
// workgroups (workgroup b runs on XCD b % 8, slot b / 8 = tile s + slice).
// A tile split over s > 1 slices is finished inside the kernel: partial sums
// to L2, an XCD-local counter, each slice finishing its share of the tile's
// items.  One workgroup per compute unit; grid = 8 TX s, with s > 1 at most
// 256 (workgroups that wait for each other are resident together).

// The sequences of one (batched) step: their tree tokens are packed in
// sequence order, sequence s owning tokens [t0[s], t0[s + 1]); each has its
// own cache and cached length.
struct SeqBatch {
  int B;
  int t0[PPD_BATCH_MAX + 1];  // t0[B]: all tokens
  int L[PPD_BATCH_MAX];       // tokens already in the sequence's cache
  int cap[PPD_BATCH_MAX];     // its capacity
  bf16_t *k[PPD_BATCH_MAX];   // this layer's keys [nkv][cap][128]
  bf16_t *v[PPD_BATCH_MAX];   // this layer's values [nkv][128][cap]
};

// (What a workgroup needs before its first load comes first: few cache lines
// of kernel arguments.)
struct GemmLaunch {
  // operands
  const bf16_t *W;      // packed weight (ppd_pack_weight)
  const unsigned char *A;  // operand planes [T_pad][K] (norm consumers: of x * gain)
  uint32_t w_bytes, a_bytes;  // their sizes
  // partition (see above)
  int kc;               // K / 64
  int TX, ls;           // tiles per XCD, log2 of the K slices per tile
  int G;                // groups; an XCD has G / 8 or one more of them, of which
  int q0, r0, q1, r1;   // a tile holds q0 = (G / 8) / TX, the first r0 = (G / 8) % TX
                        // one more (q1, r1: for G / 8 + 1)
  int T;                // tokens
  // norm partials for row scaling (QKV, SwiGLU, LOGITS): [n_ss][T_pad]
  int n_ss;
  const float *ss;
  float inv_h, eps;
  int N, K, MT;         // N = output rows (SwiGLU: F), MT = T_pad / 16
  float *part;          // s > 1: [8 TX][s][gw MT S][64] floatx4 partial sums (gemm_two_slice_gw tiles: no [s])
  uint32_t *ctr;        // s > 1: tile counters, XCD x's at ctr + 32 x (zeroed per step)
  uint32_t *status;
  int spin_limit;       // bounded wait for a tile's other slices
  // QKV outputs
  int nh, nkv;
  const float2 *rope;   // [T_pad][64]
  unsigned char *q;     // operand planes [T_pad][nh 128]
  // RESID
  float *x;
  float *ss_out;        // [8 TX R][T_pad]: sums of squares, R = ceil(s / MT) rows a tile
  const bf16_t *gain;   // the next norm's gain [N]
  // RESID: x * gain, SWIGLU: the activation, as the next GEMM's operand [T_pad][N]
  unsigned char *planes;
  // LOGITS
  float *logits;        // [T][N] or null
  float2 *amax;         // [8 TX R][T_pad]
  SeqBatch sb;          // QKV: caches, positions: token t of sequence s goes to L[s] + t - t0[s]
  // host side
  int kind;             // GemmKind
  int gw;               // most groups a tile holds
  void *ev_start, *ev_stop;  // optional events at the dispatch's start / end
};

enum GemmKind { GEMM_QKV = 0, GEMM_RESID = 1, GEMM_SWIGLU = 2, GEMM_LOGITS = 3 };

int gemm_groups_of(int kind, int N);  // groups of a GEMM with N output rows (gate/up: features)
int gemm_sub_of(int kind);            // 16-row sub-tiles per group (2 for gate/up)
int gemm_gw_max(int kind, int MT);    // largest tile (in groups) instantiated for MT token tiles
int gemm_two_slice_gw(int kind, int MT);  // tile (seven groups or more) with an exchange of its own in two slices, or 0
hipError_t launch_pack_weight(int kind, int N, int K, const bf16_t *src, bf16_t *dst, hipStream_t s);
hipError_t launch_gemm_bf16(const GemmLaunch &g, hipStream_t s);

#define PPD_ATTN_OROW 132  // floats per partial row: 128 dims, m, l, padding

struct AttnLaunch {
  const unsigned char *q;  // operand planes [T_pad][nh d]
  const uint64_t *mask; // [T][2], bits over the token's own tree
  unsigned char *out;   // operand planes [T_pad][nh d]
  float *part;          // [nh][max_splits][T_pad][PPD_ATTN_OROW] (splits > 1)
  int T_pad, nh, nkv, max_splits;
  int tiles;            // most 16-query tiles of a sequence
  SeqBatch sb;
  // Workgroup b: XCD set x = b % 8 (heads [nh x / 8, nh (x + 1) / 8)), slot
  // b / 8; sequence s takes the slots from slot0[s] on: ceil(nh / 8) heads x
  // splits[s], a split holding chunk[s] 32-key blocks.  meet: a head's splits
  // meet in the kernel, at counter ctr + 32 x + ctr0[s] + local head (zeroed per
  // step); all slots of an XCD are on its 32 compute units together (they wait
  // for each other), in sequence order.  Else the sequences with the longest
  // splits come first and a second launch adds the splits, if any.
  int slot0[PPD_BATCH_MAX], splits[PPD_BATCH_MAX], chunk[PPD_BATCH_MAX], ctr0[PPD_BATCH_MAX];
  int n_slots, meet;
  uint32_t *ctr;
  int spin_limit;
  uint32_t *status;
  float scale_log2;     // log2(e) / sqrt(d)
  void *ev_start, *ev_stop;  // optional events at the dispatch's start / end
};
int attn_blocks_per_step(int tiles);  // blocks a workgroup multiplies together
hipError_t launch_attn_bf16(const AttnLaunch &a, hipStream_t s);

// next-step candidate generation (k_next.hip)
#define PPD_NEXT_MAX_DEPTH 15
struct NextTreeLaunch {
  const int32_t *parent, *ids;  // this step's tree
  int T, vocab;
  int n_ept;                    // EPT groups per prompt token (1: plain chains)
  const float *logits;          // [T][vocab]
  const int32_t *path, *n_path, *next_tok;
  int32_t *next_ids;            // [tpl_T]
  uint32_t *status;
  int tpl_T;
  int8_t tpl_depth[PPD_T_MAX];  // template node depth (root 0)
  int16_t tpl_kind[PPD_T_MAX];  // rank of a candidate, or -1 - prompt id
  int k_of_depth[PPD_NEXT_MAX_DEPTH + 1];  // ranks needed at each depth (0: none)
  void *ev_start, *ev_stop;     // optional events on the dispatch (profiling)
};
hipError_t launch_next_tree(const NextTreeLaunch &p, int n_depths, hipStream_t s);

// The partition a step of T tokens takes for a GEMM of GemmKind `kind` (N output
// rows, gate/up: features; K columns) on a device of `cus` compute units, for
// the tests that must reach a given one: plan = {groups of the largest tile,
// tiles per XCD, K slices}.  Host only.
extern "C" void ppd_plan_gemm(int32_t kind, int32_t N, int32_t K, int32_t T, int32_t cus, int32_t plan[3]);

// The same for the attention: splits[s] and chunk[s] (in 32-key blocks) of a
// batch's sequences with L[s] cached and T[s] tree tokens, info = {slots an
// XCD's compute units share, 1 where splits, if any, meet in the kernel}.
extern "C" void ppd_plan_attention(int32_t nh, int32_t nkv, int32_t B, const int32_t *L, const int32_t *T,
                                   int32_t cus, int32_t *splits, int32_t *chunk, int32_t info[2]);

// records the thread's error message (ppd_last_error) and returns s
ppd_status ppd_fail(ppd_status s, const char *fmt, ...);

// embedding rows into x (fp32), rows T..T_pad-1 zero, and the rotary
// table [T_pad][d / 2] (cos, sin); bf16 models also write the first norm's
// operand planes (x * gain) and sums of squares (ss, one per row) and zero
// the n_ctr tile / head counters
hipError_t launch_embed(int dtype, const void *tok_emb, const void *prompt_emb, const int32_t *ids,
                        const int32_t *depth, const SeqBatch &sb, int d, float base, float2 *rope,
                        int vocab, int n_prompt, int H, float *x, const bf16_t *gain,
                        unsigned char *planes, float *ss, uint32_t *ctr, size_t n_ctr,
                        uint32_t *status, hipStream_t s);
hipError_t launch_argmax_final(const float2 *amax, int n_tiles, int T, int T_pad, int32_t *pred,
                               uint32_t *status, hipStream_t s);
hipError_t launch_accept(int T, const int32_t *parent, const int32_t *ids, const int32_t *pred,
                         int vocab, int32_t *path, int32_t *n_path, int32_t *next_tok,
                         uint32_t *status, hipStream_t s);
hipError_t launch_kv_compact(int dtype, void *k, void *v, int n_layers, int nkv, int cap, int d,
                             int L, const int32_t *path, int path_len, const int32_t *n_path,
                             int32_t *len_dev, hipStream_t s);
hipError_t launch_ws_init(void *ws, size_t n_words, hipStream_t s);
hipError_t launch_read_probe(const void *buf, size_t bytes, uint32_t *sink, hipStream_t s);

// fp32 path (float32 models): one product with its neighbours fused, kinds as
// GemmKind
struct F32Gemm {
  int kind;
  const float *A;     // [T_pad][K]
  const float *W;     // row-major [N][K] (SwiGLU: [2 N][K], gate rows then up rows)
  const float *gain;  // norm kinds: the norm gain [K]
  int T, N, K;
  float eps;
  float *out;  // QKV: q [T][nh][d]; RESID: x [T][N], added to; SwiGLU: [T][N]; LOGITS: [T][N] or null
  // QKV
  const float2 *rope;
  float *kc, *vc;
  int nh, nkv, d, cap, L;
  // LOGITS: best (value, index) of each 16 rows, [ceil(N / 16)][T_pad]
  float2 *amax;
  uint32_t *status;
};
hipError_t launch_f32_gemm(const F32Gemm &g, hipStream_t s);
hipError_t launch_f32_attention(const float *q, const float *kc, const float *vc,
                                const uint64_t *mask, int T, int L, int cap, int nh, int nkv,
                                int d, float *out, hipStream_t s);

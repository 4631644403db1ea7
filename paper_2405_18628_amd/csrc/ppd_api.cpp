// Host side of libppd: argument validation, workspace layout and the launch
// sequence of the verification step.  Everything is enqueued on the caller's
// stream; nothing is allocated, copied or synchronised (except in
// ppd_device_status, which is documented as synchronous).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <functional>
#include <string>

#include "ppd_internal.h"

namespace {

thread_local std::string g_err;

// optional per-thread kernel timer (ppd_set_kernel_timer)
struct KernelTimer {
  int kind = -1;
  void *const *start = nullptr;
  void *const *stop = nullptr;
  int n = 0;
  int next = 0;  // launches of `kind` seen in the current step
};
thread_local KernelTimer g_timer;

enum TimedKind { TK_QKV = 0, TK_ATTN = 1, TK_O = 2, TK_GATEUP = 3, TK_DOWN = 4, TK_LM = 5, TK_NEXT = 6 };

// Events of the next timed launch of `kind` (both null when not timed).  The
// kernel is then launched with hipExtLaunchKernelGGL, which records them at
// the dispatch's own start and end, so they measure the kernel alone.
void timer_events(int kind, void **start, void **stop) {
  *start = *stop = nullptr;
  if (g_timer.kind != kind || g_timer.next >= g_timer.n) return;
  *start = g_timer.start[g_timer.next];
  *stop = g_timer.stop[g_timer.next];
  ++g_timer.next;
}

ppd_status fail(ppd_status s, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return s;
}

}  // namespace

// the same for the library's other translation units
ppd_status ppd_fail(ppd_status s, const char *fmt, ...) {
  char buf[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(buf, sizeof buf, fmt, ap);
  va_end(ap);
  g_err = buf;
  return s;
}

namespace {

#define PPD_TRY_HIP(call)                                                               \
  do {                                                                                  \
    hipError_t e_ = (call);                                                             \
    if (e_ != hipSuccess) return fail(PPD_EDEVICE, "%s: %s", #call, hipGetErrorString(e_)); \
  } while (0)

constexpr int kCUs = 256;          // MI355X compute units
constexpr size_t kAlign = 256;
constexpr size_t kMaxPackedBytes = 0x7ffffff0u;  // one buffer resource per packed weight

size_t align_up(size_t v) { return (v + kAlign - 1) & ~(kAlign - 1); }
int t_pad_of(int T) { return (T + 15) & ~15; }

ppd_status pack_args(int kind, int rows, int cols, int *gk, int *N);

ppd_status check_model(const ppd_model *m) {
  if (!m) return fail(PPD_EINVAL, "model is NULL");
  if (m->n_layers < 1 || m->hidden < 1 || m->n_heads < 1 || m->n_kv_heads < 1 ||
      m->head_dim < 2 || m->ffn < 1 || m->vocab < 1 || m->n_prompt < 0)
    return fail(PPD_EINVAL, "model sizes must be positive");
  if (m->n_heads % m->n_kv_heads) return fail(PPD_EINVAL, "n_kv_heads must divide n_heads");
  if (m->head_dim % 2 || m->head_dim > 128)
    return fail(PPD_EUNSUPPORTED, "head_dim must be even and <= 128");
  if (!(m->rms_eps >= 0.f) || !(m->rope_base > 0.f))
    return fail(PPD_EINVAL, "rms_eps must be >= 0 and rope_base > 0");
  if (m->dtype != PPD_F32 && m->dtype != PPD_BF16) return fail(PPD_EINVAL, "unknown dtype");
  if (m->dtype == PPD_BF16) {
    if (m->head_dim != 128) return fail(PPD_EUNSUPPORTED, "bf16 kernels need head_dim 128");
    if (m->hidden % 128) return fail(PPD_EUNSUPPORTED, "bf16 kernels need hidden %% 128 == 0");
    if (m->ffn % 64) return fail(PPD_EUNSUPPORTED, "bf16 kernels need ffn %% 64 == 0");
    const int shapes[5][3] = {{PPD_W_QKV, (m->n_heads + 2 * m->n_kv_heads) * 128, m->hidden},
                              {PPD_W_O, m->hidden, m->n_heads * 128},
                              {PPD_W_GATE_UP, 2 * m->ffn, m->hidden},
                              {PPD_W_DOWN, m->hidden, m->ffn},
                              {PPD_W_LM_HEAD, m->vocab, m->hidden}};
    for (const auto &w : shapes) {
      int gk, N;
      const ppd_status st = pack_args(w[0], w[1], w[2], &gk, &N);
      if (st != PPD_OK) return st;
    }
  }
  if (!m->tok_emb || !m->lm_head || !m->final_norm || (m->n_prompt > 0 && !m->prompt_emb))
    return fail(PPD_EINVAL, "embedding, LM head and final norm pointers must be set");
  const void *const *arrs[6] = {m->attn_norm, m->w_qkv, m->w_o, m->mlp_norm, m->w_gate_up,
                                m->w_down};
  for (int a = 0; a < 6; ++a) {
    if (!arrs[a]) return fail(PPD_EINVAL, "per-layer pointer array %d is NULL", a);
    for (int l = 0; l < m->n_layers; ++l)
      if (!arrs[a][l]) return fail(PPD_EINVAL, "per-layer pointer %d of layer %d is NULL", a, l);
  }
  return PPD_OK;
}

int qkv_rows(const ppd_model *m) { return (m->n_heads + 2 * m->n_kv_heads) * m->head_dim; }

// ---- launch shapes (also used to size the workspace)

// Compute units of the current device (one workgroup per compute unit; the
// XCD-local tile finish needs the MI355X layout of 8 XCDs x 32 CUs with
// round-robin dispatch, else every tile is finished whole, without waits).
int device_cus() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess) return 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  return n;
}

struct GemmShape {
  int kind, N, K;
};

// Partition of one GEMM for MT token tiles (see GemmLaunch).  For each number
// s of K slices the XCD's 32 workgroups take TX = 32 / s tiles (s = 1: 32, 64,
// .. tiles, as few as the largest instantiated tile allows; each further 32
// are a round of workgroups that follows) of h groups, and the cheapest by a
// model of the slowest workgroup's time is taken.  The model's rates are the
// MI355X compute unit's load path, measured: it returns loads in order, so a
// workgroup's weight bytes cost ~36 GB/s (HBM latency over what a compute
// unit can have outstanding) and its activation bytes, L2 hits, ~110 GB/s on
// top of that, and all weights together stream at 6.2 TB/s at most.  s > 1
// divides the activation bytes by s and adds the exchange of the partial
// sums: ~2 us of latency and ~4 GB/s for a workgroup's sums; two slices of a
// tile of seven groups or more, whose own sums stay in LDS, 2.5 us and ~13.5
// GB/s, part of it while the stream still runs.
// Compared with every plan that fits, the steps timed with one GEMM changed at
// a time (270 (shape, kind, T) of the 1.4B, 7B, 13B, GQA and two narrower
// widths, T = 1 .. 128), the choice is the fastest or within 2 us of it in all
// but a dozen: projections 2560 or 1024 wide with T = 48 .. 96 run whole and
// would gain up to 5 us in 4 slices.
struct GemmPlan {
  int gw = 1, TX = 32, s = 1;
  // rows of the tiles' reductions (sums of squares, argmax)
  int rows(int MT) const { return 8 * TX * ((s + MT - 1) / MT); }
};

// Columns from which the cheaper exchange of two slices is counted on (us a step
// of three layers, whole tiles -> two slices, T = 64 and 96: 3072 columns 380.7 ->
// 385.5, 467.9 -> 476.4; 4096 475.9 -> 475.3, 574.5 -> 578.0; 4608 494.6 -> 492.9,
// 610.2 -> 607.2; 5120 538.5 -> 532.5, 660.7 -> 653.5).
constexpr int kTwoSliceK = 4608;

GemmPlan plan_gemm(const GemmShape &sh, int MT, bool xcd_sync) {
  GemmPlan best;
  const int G = gemm_groups_of(sh.kind, sh.N), S = gemm_sub_of(sh.kind), kc = sh.K / 64;
  const int nx = (G + 7) / 8;
  const int gmax = gemm_gw_max(sh.kind, MT);
  const double hbm = 2.0 * G * 16 * S * sh.K / 6.2e12;
  double best_t = 1e30;
  for (int s = 1; s <= 8; s *= 2) {
    if (s > kc || (s > 1 && !xcd_sync)) break;
    int TX = 32 / s, h = std::max(1, (nx + TX - 1) / TX);
    if (s == 1)
      for (; h > gmax; h = (nx + TX - 1) / TX) TX += 32;
    // a tile of seven groups or more in two slices has a cheaper exchange
    const int two_gw = s == 2 && sh.K >= kTwoSliceK ? gemm_two_slice_gw(sh.kind, MT) : 0;
    const bool two = h >= 7 && h <= two_gw;
    const int gw = two ? two_gw : h == 5 ? 6 : h == 7 ? 8 : h;
    if (gw > gmax && !two) continue;
    const double cols = (double)((kc + s - 1) / s) * 64;
    const double wb = 2.0 * h * 16 * S * cols, ab = 4.0 * MT * 16 * cols, pb = 1024.0 * h * S * MT;
    const double load = (TX + 31) / 32 * (wb / 36e9 + ab / 110e9);
    const double t = two     ? std::max(load + 2.5e-6 + pb / 13.5e9, hbm + 2e-6)
                     : s > 1 ? std::max(load, hbm) + 2e-6 + pb / 4e9
                             : std::max(load, hbm);
    if (t < best_t) {
      best_t = t;
      best.gw = gw;
      best.TX = TX;
      best.s = s;
    }
  }
  return best;
}

enum { SH_QKV = 0, SH_O = 1, SH_GATE_UP = 2, SH_DOWN = 3, SH_LM = 4 };

void gemm_shapes(const ppd_model *m, GemmShape out[5]) {
  out[SH_QKV] = {GEMM_QKV, qkv_rows(m), m->hidden};
  out[SH_O] = {GEMM_RESID, m->hidden, m->n_heads * 128};
  out[SH_GATE_UP] = {GEMM_SWIGLU, m->ffn, m->hidden};
  out[SH_DOWN] = {GEMM_RESID, m->hidden, m->ffn};
  out[SH_LM] = {GEMM_LOGITS, m->vocab, m->hidden};
}

// bytes of the partial sums of a plan (0 when every tile is whole)
size_t plan_part_bytes(const GemmShape &sh, const GemmPlan &p, int MT) {
  if (p.s == 1) return 0;
  const bool two = p.s == 2 && p.gw == gemm_two_slice_gw(sh.kind, MT);
  return (size_t)8 * p.TX * (two ? 1 : p.s) * p.gw * gemm_sub_of(sh.kind) * MT * 64 * 16;
}

constexpr int kSpinLimit = 1 << 14;  // bounded wait of a tile's slices (~10-20 ms)

// Key splits of a head: at most what puts one workgroup of each of its XCD's
// heads and splits on one of the XCD's 32 compute units.
int attn_max_splits(int nh) { return std::max(1, std::min(PPD_ATTN_MAX_SPLITS, kCUs / nh)); }

// The attention's key splits.  Either the splits of a head meet in the kernel,
// or a second launch adds them.
//
// Meeting needs an XCD's heads x splits of all sequences on its 32 compute
// units together: the slots left are given one by one to the sequence with the
// most blocks per split, as long as a split keeps kAttnMinBlocks 32-key blocks.
// A batch's heads take at most kAttnMeetBatch splits: workgroups start in
// order, so a launch holds at most one incomplete head an XCD, and two launches
// of two streams (2 x 15 waiting workgroups) always leave compute units for the
// ones they wait for.
//
// Where that leaves a batch unbalanced (no slot left for a sequence much longer
// than the others, or a second round of a few workgroups) every sequence is cut
// into chunks of an even share of all blocks, in one round or two, and a second
// launch adds the splits.  The cheaper by the time of the last workgroup is
// taken, each counted as its blocks and kAttnSlotBlocks for what it does
// besides, the second launch as kAttnMergeBlocks: a block of a 16-token tree
// takes ~0.33 us, and no less than twice that while all 256 compute units read
// keys of their own (6.2 TB/s).  us a launch, 16-token trees, meeting (second
// launch): 7B, eight sequences of 16384 and 7 x 256 tokens 177.7 (75.8), 13B,
// six of 8192 and 5 x 512 98.0 (52.1), 13B, two of 32768 and 256 113 (123).
constexpr int kAttnMinBlocks = 4, kAttnMeetBatch = 16, kAttnSlotBlocks = 16, kAttnMergeBlocks = 16;

struct AttnPlan {
  int splits[PPD_BATCH_MAX], chunk[PPD_BATCH_MAX], order[PPD_BATCH_MAX];  // order: longest chunk first
  int slots;
  bool meet;
};

// chunks and slots of a plan whose splits are wanted so: each sequence takes the
// fewest splits that need no more steps of the kernel
void attn_chunks(AttnPlan &p, int B, const int *nblk, int step, int unit) {
  p.slots = 0;
  for (int j = 0; j < B; ++j) {
    const int per = (nblk[j] + p.splits[j] - 1) / p.splits[j];
    p.chunk[j] = (per + step - 1) / step * step;
    p.splits[j] = (nblk[j] + p.chunk[j] - 1) / p.chunk[j];
    p.slots += unit * p.splits[j];
    p.order[j] = j;
  }
  std::stable_sort(p.order, p.order + B, [&](int a, int b) { return p.chunk[a] > p.chunk[b]; });
}

// when the last of an XCD's workgroups ends, in blocks: each starts, in order,
// on the compute unit that is free first
int attn_makespan(const AttnPlan &p, int B, const int *nblk, int unit) {
  int busy[32] = {0}, end = 0;  // a min-heap
  for (int i = 0; i < B; ++i) {
    const int j = p.order[i];
    const int t = kAttnSlotBlocks + std::min(p.chunk[j], nblk[j]);
    for (int w = 0; w < unit * p.splits[j]; ++w) {
      std::pop_heap(busy, busy + 32, std::greater<int>());
      end = std::max(end, busy[31] += t);
      std::push_heap(busy, busy + 32, std::greater<int>());
    }
  }
  return end;
}

AttnPlan plan_attn(int nh, int nkv, int B, const int *nblk, int step, bool xcd_sync) {
  const int unit = (nh + 7) / 8, max_splits = attn_max_splits(nh);
  AttnPlan best{};
  best.meet = true;
  int used = B * unit, total = 0;
  for (int j = 0; j < B; ++j) {
    best.splits[j] = 1;
    total += unit * nblk[j];
  }
  const int cap = B > 1 ? std::min(max_splits, kAttnMeetBatch) : max_splits;
  for (; xcd_sync && used + unit <= 32; used += unit) {
    int longest = -1;
    for (int j = 0; j < B; ++j)
      if (nblk[j] >= (best.splits[j] + 1) * kAttnMinBlocks && best.splits[j] < cap &&
          (longest < 0 || (long)nblk[j] * best.splits[longest] > (long)nblk[longest] * best.splits[j]))
        longest = j;
    if (longest < 0) break;
    ++best.splits[longest];
  }
  attn_chunks(best, B, nblk, step, unit);
  if (B == 1 && xcd_sync) return best;
  best.meet = xcd_sync && best.slots <= 32;  // else nothing is split so far
  const int stream = (int)(2L * total * nkv / (32 * nh));
  // (of plans that the stream bounds alike the shorter one)
  auto cost = [&](int span) { return 8 * std::max(stream, span) + span; };
  int best_t = cost(attn_makespan(best, B, nblk, unit));
  for (int rounds = 1; rounds <= 2; ++rounds) {
    const int share = std::max(kAttnMinBlocks, (total + 32 * rounds - 1) / (32 * rounds));
    if (cost(share + kAttnSlotBlocks) + 8 * kAttnMergeBlocks >= best_t) continue;
    AttnPlan p{};
    for (int j = 0; j < B; ++j) p.splits[j] = std::max(1, std::min(max_splits, (nblk[j] + share - 1) / share));
    attn_chunks(p, B, nblk, step, unit);
    const int t = cost(attn_makespan(p, B, nblk, unit)) + 8 * kAttnMergeBlocks;
    if (t < best_t) best_t = t, best = p;
  }
  return best;
}

// 32-key blocks of the sequences, and the most 16-query tiles one has
int attn_blocks(int B, const int *L, const int *T, int *nblk) {
  int tiles = 1;
  for (int j = 0; j < B; ++j) {
    tiles = std::max(tiles, (T[j] + 15) / 16);
    nblk[j] = (L[j] + T[j] + 31) / 32;
  }
  return tiles;
}

void set_attn_plan(AttnLaunch &a, const int *L, const int *T, bool xcd_sync) {
  const int B = a.sb.B, unit = (a.nh + 7) / 8;
  int nblk[PPD_BATCH_MAX];
  a.tiles = attn_blocks(B, L, T, nblk);
  const AttnPlan p = plan_attn(a.nh, a.nkv, B, nblk, attn_blocks_per_step(a.tiles), xcd_sync);
  a.meet = p.meet;
  a.n_slots = 0;
  for (int i = 0; i < B; ++i) {
    const int j = p.meet ? i : p.order[i];
    a.splits[j] = p.splits[j];
    a.chunk[j] = p.chunk[j];
    a.slot0[j] = a.n_slots;
    a.n_slots += unit * p.splits[j];
    a.ctr0[j] = j * unit;  // used only where splits meet: then all slots fit 32, and so do the counters
  }
}

WsLayout layout_of(const ppd_model *m, int T) {
  WsLayout w{};
  const int Tp = t_pad_of(T);
  const bool bf16 = m->dtype == PPD_BF16;
  const int H = m->hidden, F = m->ffn, nh = m->n_heads, d = m->head_dim;
  size_t off = 0;
  auto take = [&](size_t bytes) {
    size_t o = off;
    off = align_up(off + bytes);
    return o;
  };
  w.status = take(16);
  w.x = take(sizeof(float) * Tp * H);
  // activations take 4 bytes an element on both paths (bf16 models: fp32 x,
  // operand planes of two bf16 parts elsewhere).  x * gain lives from the GEMM
  // that writes it to the one that reads it, the attention's split rows within
  // one launch between the two: they share memory, so that a step needs no
  // more of it for the operand planes
  w.max_splits = bf16 ? attn_max_splits(nh) : 0;
  const size_t split_rows = sizeof(float) * (size_t)nh * w.max_splits * Tp * PPD_ATTN_OROW;
  w.xg = w.attn_part = take(bf16 ? std::max(sizeof(float) * Tp * H, split_rows) : 0);
  w.max_ss = 1;
  w.max_amax_tiles = bf16 ? 1 : (m->vocab + 15) / 16;
  size_t part = 0;
  if (bf16) {
    GemmShape gs[5];
    gemm_shapes(m, gs);
    const bool sync = device_cus() == kCUs;
    for (int mt = 1; mt <= Tp / 16; ++mt)
      for (int i = 0; i < 5; ++i) {
        const GemmPlan p = plan_gemm(gs[i], mt, sync);
        part = std::max(part, plan_part_bytes(gs[i], p, mt));
        if (gs[i].kind == GEMM_RESID) w.max_ss = std::max(w.max_ss, p.rows(mt));
        if (gs[i].kind == GEMM_LOGITS) w.max_amax_tiles = std::max(w.max_amax_tiles, p.rows(mt));
      }
  }
  w.ss = take(sizeof(float) * w.max_ss * Tp);
  w.q = take(sizeof(float) * Tp * nh * d);
  w.attn_o = take(sizeof(float) * Tp * nh * d);
  w.act = take(sizeof(float) * Tp * F);
  w.gemm_part = take(part);
  w.amax = take(sizeof(float2) * w.max_amax_tiles * Tp);
  w.rope = take(sizeof(float2) * Tp * (d / 2));
  // counters: one 1 KB block (8 XCDs x one 128-byte line) per GEMM launch
  // (tiles) and per attention launch (heads)
  w.n_ctr = bf16 ? (size_t)(5 * m->n_layers + 1) * 256 : 0;
  w.ctr = take(sizeof(uint32_t) * w.n_ctr);
  w.total = off;
  return w;
}

template <typename P>
P *at(void *ws, size_t off) {
  return (P *)((char *)ws + off);
}

ppd_status check_kv(const ppd_model *m, const ppd_kv *kv) {
  if (!kv || !kv->k || !kv->v) return fail(PPD_EINVAL, "kv cache pointers must be set");
  if (kv->capacity < 1) return fail(PPD_EINVAL, "kv capacity must be positive");
  if (m->dtype == PPD_BF16 && kv->capacity % 8)
    return fail(PPD_EUNSUPPORTED, "bf16 caches need capacity %% 8 == 0");
  if (kv->capacity > PPD_CAPACITY_MAX)  // per-head offsets are 32-bit in the kernels
    return fail(PPD_EUNSUPPORTED, "capacity %d > %d", kv->capacity, PPD_CAPACITY_MAX);
  return PPD_OK;
}

// the sequences of a step, with this layer's cache slices
SeqBatch seq_batch(const ppd_model *m, int B, const ppd_kv *kvs, const int32_t *Ls,
                   const int32_t *Ts, int layer) {
  SeqBatch sb{};
  sb.B = B;
  for (int j = 0; j < B; ++j) {
    sb.t0[j + 1] = sb.t0[j] + Ts[j];
    sb.L[j] = Ls[j];
    sb.cap[j] = kvs[j].capacity;
    const size_t per_layer = (size_t)m->n_kv_heads * kvs[j].capacity * m->head_dim;
    sb.k[j] = (bf16_t *)kvs[j].k + (size_t)layer * per_layer;
    sb.v[j] = (bf16_t *)kvs[j].v + (size_t)layer * per_layer;
  }
  return sb;
}

ppd_status step_bf16(const ppd_model *m, int B, const ppd_kv *kvs, const int32_t *Ls,
                     const int32_t *Ts, const int32_t *ids, const int32_t *depth,
                     const uint64_t *mask, void *ws, const WsLayout &w, float *logits,
                     int32_t *pred, hipStream_t s) {
  const int H = m->hidden, nh = m->n_heads, nkv = m->n_kv_heads;
  int T = 0;
  for (int j = 0; j < B; ++j) T += Ts[j];
  const int Tp = t_pad_of(T), MT = Tp / 16;
  uint32_t *status = at<uint32_t>(ws, w.status);
  float *x = at<float>(ws, w.x);
  float *ss = at<float>(ws, w.ss);
  unsigned char *q = at<unsigned char>(ws, w.q);
  unsigned char *xg = at<unsigned char>(ws, w.xg);
  unsigned char *attn_o = at<unsigned char>(ws, w.attn_o);
  unsigned char *act = at<unsigned char>(ws, w.act);
  float *part = at<float>(ws, w.gemm_part);
  float2 *amax = at<float2>(ws, w.amax);
  float2 *rope = at<float2>(ws, w.rope);
  uint32_t *ctr = at<uint32_t>(ws, w.ctr);
  GemmShape gs[5];
  gemm_shapes(m, gs);
  const bool sync = device_cus() == kCUs;
  GemmPlan plan[5];
  for (int i = 0; i < 5; ++i) plan[i] = plan_gemm(gs[i], MT, sync);
  int launch = 0;  // GEMM launches of this step: counter block `launch`
  auto setup = [&](GemmLaunch &g, int i) {
    g.kind = gs[i].kind;
    g.N = gs[i].N;
    g.K = gs[i].K;
    g.kc = gs[i].K / 64;
    g.w_bytes = (uint32_t)((size_t)gemm_groups_of(g.kind, g.N) * gemm_sub_of(g.kind) * 16 * g.K * sizeof(bf16_t));
    g.a_bytes = (uint32_t)(sizeof(float) * Tp * g.K);
    g.gw = plan[i].gw;
    g.TX = plan[i].TX;
    g.ls = 0;
    while ((1 << g.ls) < plan[i].s) ++g.ls;
    g.G = gemm_groups_of(g.kind, g.N);
    g.q0 = g.G / 8 / g.TX;
    g.r0 = g.G / 8 % g.TX;
    g.q1 = (g.G / 8 + 1) / g.TX;
    g.r1 = (g.G / 8 + 1) % g.TX;
    g.ctr = ctr + (size_t)launch++ * 256;
  };

  // embedding, the first norm's operand and sums of squares (one partial per
  // row), rotary table, zeroed counters
  PPD_TRY_HIP(launch_embed(PPD_BF16, m->tok_emb, m->prompt_emb, ids, depth,
                           seq_batch(m, B, kvs, Ls, Ts, 0), m->head_dim, m->rope_base, rope,
                           m->vocab, m->n_prompt, H, x, (const bf16_t *)m->attn_norm[0], xg, ss, ctr,
                           w.n_ctr, status, s));
  int n_ss = 1;
  AttnLaunch a{};
  a.q = q;
  a.mask = mask;
  a.out = attn_o;
  a.part = at<float>(ws, w.attn_part);
  a.T_pad = Tp;
  a.nh = nh;
  a.nkv = nkv;
  a.max_splits = w.max_splits;
  a.spin_limit = kSpinLimit;
  a.status = status;
  a.scale_log2 = (float)(1.4426950408889634 / std::sqrt(128.0));
  a.sb = seq_batch(m, B, kvs, Ls, Ts, 0);
  set_attn_plan(a, Ls, Ts, sync);
  uint32_t *attn_ctr = ctr + (size_t)(4 * m->n_layers + 1) * 256;
  const float inv_h = 1.0f / (float)H;

  for (int l = 0; l < m->n_layers; ++l) {
    const SeqBatch sb = seq_batch(m, B, kvs, Ls, Ts, l);
    GemmLaunch g{};
    g.T = T;
    g.MT = MT;
    g.part = part;
    g.inv_h = inv_h;
    g.eps = m->rms_eps;
    g.status = status;
    g.spin_limit = kSpinLimit;
    // QKV + RoPE + cache stores; operand x * attn_norm
    GemmLaunch qg = g;
    setup(qg, SH_QKV);
    qg.W = (const bf16_t *)m->w_qkv[l];
    qg.A = xg;
    qg.ss = ss;
    qg.n_ss = n_ss;
    qg.rope = rope;
    qg.q = q;
    qg.nh = nh;
    qg.nkv = nkv;
    qg.sb = sb;
    timer_events(TK_QKV, &qg.ev_start, &qg.ev_stop);
    PPD_TRY_HIP(launch_gemm_bf16(qg, s));
    // tree attention
    a.sb = sb;
    a.ctr = attn_ctr + (size_t)l * 256;
    timer_events(TK_ATTN, &a.ev_start, &a.ev_stop);
    PPD_TRY_HIP(launch_attn_bf16(a, s));
    // O projection + residual; the MLP norm's operand and sums of squares
    GemmLaunch o = g;
    setup(o, SH_O);
    o.W = (const bf16_t *)m->w_o[l];
    o.A = attn_o;
    o.x = x;
    o.ss_out = ss;
    o.gain = (const bf16_t *)m->mlp_norm[l];
    o.planes = xg;
    timer_events(TK_O, &o.ev_start, &o.ev_stop);
    PPD_TRY_HIP(launch_gemm_bf16(o, s));
    n_ss = plan[SH_O].rows(MT);
    // gate/up + SwiGLU; operand x * mlp_norm
    GemmLaunch u = g;
    setup(u, SH_GATE_UP);
    u.W = (const bf16_t *)m->w_gate_up[l];
    u.A = xg;
    u.ss = ss;
    u.n_ss = n_ss;
    u.planes = act;
    timer_events(TK_GATEUP, &u.ev_start, &u.ev_stop);
    PPD_TRY_HIP(launch_gemm_bf16(u, s));
    // down projection + residual; the next norm's operand and sums of squares
    GemmLaunch dn = g;
    setup(dn, SH_DOWN);
    dn.W = (const bf16_t *)m->w_down[l];
    dn.A = act;
    dn.x = x;
    dn.ss_out = ss;
    dn.gain = (const bf16_t *)(l + 1 < m->n_layers ? m->attn_norm[l + 1] : m->final_norm);
    dn.planes = xg;
    timer_events(TK_DOWN, &dn.ev_start, &dn.ev_stop);
    PPD_TRY_HIP(launch_gemm_bf16(dn, s));
    n_ss = plan[SH_DOWN].rows(MT);
  }
  // final norm + LM head + greedy partials; operand x * final_norm
  GemmLaunch lm{};
  setup(lm, SH_LM);
  lm.W = (const bf16_t *)m->lm_head;
  lm.A = xg;
  lm.T = T;
  lm.MT = MT;
  lm.part = part;
  lm.ss = ss;
  lm.n_ss = n_ss;
  lm.inv_h = inv_h;
  lm.eps = m->rms_eps;
  lm.logits = logits;
  lm.amax = amax;
  lm.status = status;
  lm.spin_limit = kSpinLimit;
  timer_events(TK_LM, &lm.ev_start, &lm.ev_stop);
  PPD_TRY_HIP(launch_gemm_bf16(lm, s));
  PPD_TRY_HIP(launch_argmax_final(amax, plan[SH_LM].rows(MT), T, Tp, pred, status, s));
  return PPD_OK;
}

ppd_status step_f32(const ppd_model *m, const ppd_kv *kv, int L, int T, const int32_t *ids,
                    const int32_t *depth, const uint64_t *mask, void *ws, const WsLayout &w,
                    float *logits, int32_t *pred, hipStream_t s) {
  const int H = m->hidden, F = m->ffn, nh = m->n_heads, nkv = m->n_kv_heads, d = m->head_dim;
  const int cap = kv->capacity;
  uint32_t *status = at<uint32_t>(ws, w.status);
  float *x = at<float>(ws, w.x);
  float *q = at<float>(ws, w.q);
  float *attn_o = at<float>(ws, w.attn_o);
  float *act = at<float>(ws, w.act);
  float2 *amax = at<float2>(ws, w.amax);
  float2 *rope = at<float2>(ws, w.rope);

  SeqBatch one{};
  one.B = 1;
  one.t0[1] = T;
  one.L[0] = L;
  PPD_TRY_HIP(launch_embed(PPD_F32, m->tok_emb, m->prompt_emb, ids, depth, one, d, m->rope_base, rope,
                           m->vocab, m->n_prompt, H, x, nullptr, nullptr, nullptr, nullptr, 0, status, s));
  F32Gemm g{};
  g.T = T;
  g.eps = m->rms_eps;
  g.rope = rope;
  g.nh = nh;
  g.nkv = nkv;
  g.d = d;
  g.cap = cap;
  g.L = L;
  g.status = status;
  auto gemm = [&](int kind, const float *A, const void *W, const void *gain, int N, int K, float *out) {
    g.kind = kind;
    g.A = A;
    g.W = (const float *)W;
    g.gain = (const float *)gain;
    g.N = N;
    g.K = K;
    g.out = out;
    return launch_f32_gemm(g, s);
  };
  for (int l = 0; l < m->n_layers; ++l) {
    g.kc = (float *)kv->k + (size_t)l * nkv * cap * d;
    g.vc = (float *)kv->v + (size_t)l * nkv * d * cap;
    PPD_TRY_HIP(gemm(GEMM_QKV, x, m->w_qkv[l], m->attn_norm[l], qkv_rows(m), H, q));
    PPD_TRY_HIP(launch_f32_attention(q, g.kc, g.vc, mask, T, L, cap, nh, nkv, d, attn_o, s));
    PPD_TRY_HIP(gemm(GEMM_RESID, attn_o, m->w_o[l], nullptr, H, nh * d, x));
    PPD_TRY_HIP(gemm(GEMM_SWIGLU, x, m->w_gate_up[l], m->mlp_norm[l], F, H, act));
    PPD_TRY_HIP(gemm(GEMM_RESID, act, m->w_down[l], nullptr, H, F, x));
  }
  g.amax = amax;
  PPD_TRY_HIP(gemm(GEMM_LOGITS, x, m->lm_head, m->final_norm, m->vocab, H, logits));
  PPD_TRY_HIP(launch_argmax_final(amax, (m->vocab + 15) / 16, T, t_pad_of(T), pred, status, s));
  return PPD_OK;
}

// GEMM kind and output-row count of a weight given as a row-major
// [rows][cols] matrix
ppd_status pack_args(int kind, int rows, int cols, int *gk, int *N) {
  if (rows < 1 || cols < 1) return fail(PPD_EINVAL, "weight sizes must be positive");
  if (cols % 64) return fail(PPD_EUNSUPPORTED, "packed weights need cols %% 64 == 0");
  switch (kind) {
    case PPD_W_QKV:
      if (rows % 128) return fail(PPD_EUNSUPPORTED, "w_qkv needs rows %% 128 == 0 (head_dim 128)");
      *gk = GEMM_QKV, *N = rows;
      break;
    case PPD_W_O:
    case PPD_W_DOWN:
      if (rows % 128) return fail(PPD_EUNSUPPORTED, "w_o / w_down need rows (hidden) %% 128 == 0");
      *gk = GEMM_RESID, *N = rows;
      break;
    case PPD_W_GATE_UP:
      if (rows % 128) return fail(PPD_EUNSUPPORTED, "w_gate_up needs rows (2 ffn) %% 128 == 0");
      *gk = GEMM_SWIGLU, *N = rows / 2;
      break;
    case PPD_W_LM_HEAD:
      *gk = GEMM_LOGITS, *N = rows;
      break;
    default:
      return fail(PPD_EINVAL, "unknown weight kind %d", kind);
  }
  // the GEMM reads a packed weight through one buffer resource: < 2 GB
  const size_t bytes = (size_t)gemm_groups_of(*gk, *N) * gemm_sub_of(*gk) * 16 * cols * sizeof(bf16_t);
  if (bytes > kMaxPackedBytes)
    return fail(PPD_EUNSUPPORTED, "a packed weight of %zu bytes exceeds %zu", bytes, kMaxPackedBytes);
  return PPD_OK;
}

}  // namespace

extern "C" {

size_t ppd_workspace_bytes(const ppd_model *model, int32_t t_max, int32_t max_len) {
  if (check_model(model) != PPD_OK) return 0;
  if (t_max < 1 || t_max > PPD_T_MAX || max_len < 0) {
    fail(PPD_EINVAL, "t_max must be in [1, %d] and max_len >= 0", PPD_T_MAX);
    return 0;
  }
  return layout_of(model, t_max).total;
}

ppd_status ppd_workspace_init(void *ws, size_t ws_bytes, void *stream) {
  const size_t need = align_up(16);  // the header: the status word
  if (!ws || ws_bytes < need) return fail(PPD_EWORKSPACE, "workspace needs at least %zu bytes", need);
  PPD_TRY_HIP(launch_ws_init(ws, need / 4, (hipStream_t)stream));
  return PPD_OK;
}

ppd_status ppd_build_tree_mask(int32_t T, const int32_t *parent, int32_t *depth_out,
                               uint64_t *mask_out) {
  if (T < 1 || T > PPD_T_MAX) return fail(PPD_EINVAL, "T=%d outside [1, %d]", T, PPD_T_MAX);
  if (!parent || !depth_out || !mask_out) return fail(PPD_EINVAL, "NULL argument");
  if (parent[0] != -1) return fail(PPD_ETREE, "parent[0] must be -1 (root)");
  for (int i = 1; i < T; ++i)
    if (parent[i] < 0 || parent[i] >= i)
      return fail(PPD_ETREE, "parent[%d]=%d is not an earlier node", i, parent[i]);
  for (int i = 0; i < T; ++i) {
    uint64_t row[PPD_MASK_WORDS] = {0, 0};
    int dep = -1;
    for (int j = i; j != -1; j = parent[j]) {
      row[j >> 6] |= 1ull << (j & 63);
      ++dep;
    }
    depth_out[i] = dep;
    mask_out[i * PPD_MASK_WORDS + 0] = row[0];
    mask_out[i * PPD_MASK_WORDS + 1] = row[1];
  }
  return PPD_OK;
}

ppd_status ppd_verify_batch(const ppd_model *model, int32_t B, const ppd_kv *kvs,
                            const int32_t *L, const int32_t *T, const int32_t *ids,
                            const int32_t *depth, const uint64_t *mask, void *ws, size_t ws_bytes,
                            float *logits, int32_t *pred, void *stream) {
  ppd_status st = check_model(model);
  if (st != PPD_OK) return st;
  if (B < 1 || B > PPD_BATCH_MAX)
    return fail(PPD_EINVAL, "B=%d outside [1, %d]", B, PPD_BATCH_MAX);
  if (!kvs || !L || !T) return fail(PPD_EINVAL, "NULL sequence arrays");
  if (B > 1 && model->dtype != PPD_BF16)
    return fail(PPD_EUNSUPPORTED, "batched steps need a bf16 model");
  int64_t total = 0;
  for (int j = 0; j < B; ++j) {
    if ((st = check_kv(model, &kvs[j])) != PPD_OK) return st;
    if (T[j] < 1) return fail(PPD_EINVAL, "T[%d]=%d must be >= 1", j, T[j]);
    if (L[j] < 0) return fail(PPD_EINVAL, "L[%d] must be >= 0", j);
    if ((int64_t)L[j] + T[j] > kvs[j].capacity)
      return fail(PPD_ECAPACITY, "sequence %d: L + T = %lld exceeds capacity %d", j,
                  (long long)L[j] + T[j], kvs[j].capacity);
    total += T[j];
  }
  if (total > PPD_T_MAX)
    return fail(PPD_EINVAL, "%lld tree tokens in all > %d", (long long)total, PPD_T_MAX);
  if (!ids || !depth || !mask || !pred) return fail(PPD_EINVAL, "NULL tree or output pointer");
  const WsLayout w = layout_of(model, (int)total);
  if (!ws || ws_bytes < w.total)
    return fail(PPD_EWORKSPACE, "workspace of %zu bytes is smaller than the %zu required", ws_bytes,
                w.total);
  hipStream_t s = (hipStream_t)stream;
  g_timer.next = 0;
  if (model->dtype == PPD_BF16)
    return step_bf16(model, B, kvs, L, T, ids, depth, mask, ws, w, logits, pred, s);
  return step_f32(model, &kvs[0], L[0], T[0], ids, depth, mask, ws, w, logits, pred, s);
}

ppd_status ppd_verify_step(const ppd_model *model, const ppd_kv *kv, int32_t L, int32_t T,
                           const int32_t *ids, const int32_t *depth, const uint64_t *mask,
                           void *ws, size_t ws_bytes, float *logits, int32_t *pred,
                           void *stream) {
  if (!kv) return fail(PPD_EINVAL, "kv cache pointers must be set");
  if (T < 1 || T > PPD_T_MAX) return fail(PPD_EINVAL, "T=%d outside [1, %d]", T, PPD_T_MAX);
  return ppd_verify_batch(model, 1, kv, &L, &T, ids, depth, mask, ws, ws_bytes, logits, pred,
                          stream);
}

ppd_status ppd_accept(int32_t T, const int32_t *parent, const int32_t *ids, const int32_t *pred,
                      int32_t vocab, int32_t *path, int32_t *n_path, int32_t *next_tok, void *ws,
                      size_t ws_bytes, void *stream) {
  if (T < 1 || T > PPD_T_MAX) return fail(PPD_EINVAL, "T=%d outside [1, %d]", T, PPD_T_MAX);
  if (vocab < 1) return fail(PPD_EINVAL, "vocab must be positive");
  if (!parent || !ids || !pred || !path || !n_path || !next_tok)
    return fail(PPD_EINVAL, "NULL argument");
  if (!ws || ws_bytes < 16) return fail(PPD_EWORKSPACE, "workspace (status word) required");
  PPD_TRY_HIP(launch_accept(T, parent, ids, pred, vocab, path, n_path, next_tok, (uint32_t *)ws,
                            (hipStream_t)stream));
  return PPD_OK;
}

ppd_status ppd_kv_compact(const ppd_model *model, const ppd_kv *kv, int32_t L,
                          const int32_t *path, int32_t path_len, const int32_t *n_path,
                          void *stream) {
  ppd_status st = check_model(model);
  if (st != PPD_OK) return st;
  if ((st = check_kv(model, kv)) != PPD_OK) return st;
  if (L < 0 || L >= kv->capacity)
    return fail(PPD_ECAPACITY, "L=%d must be in [0, capacity=%d)", L, kv->capacity);
  if (!path || !n_path) return fail(PPD_EINVAL, "NULL path");
  if (path_len < 1 || path_len > PPD_T_MAX)
    return fail(PPD_EINVAL, "path_len=%d outside [1, %d]", path_len, PPD_T_MAX);
  PPD_TRY_HIP(launch_kv_compact(model->dtype, kv->k, kv->v, model->n_layers, model->n_kv_heads,
                                kv->capacity, model->head_dim, L, path, path_len, n_path,
                                kv->len_dev, (hipStream_t)stream));
  return PPD_OK;
}

ppd_status ppd_next_tree(int32_t T, const int32_t *parent, const int32_t *ids, int32_t vocab,
                         int32_t n_prompt, int32_t n_ept, const float *logits, const int32_t *path,
                         const int32_t *n_path, const int32_t *next_tok, int32_t tpl_T,
                         const int32_t *tpl_parent, const int32_t *tpl_kind, int32_t *next_ids,
                         void *ws, size_t ws_bytes, void *stream) {
  if (T < 1 || T > PPD_T_MAX) return fail(PPD_EINVAL, "T=%d outside [1, %d]", T, PPD_T_MAX);
  if (tpl_T < 1 || tpl_T > PPD_T_MAX)
    return fail(PPD_EINVAL, "template size %d outside [1, %d]", tpl_T, PPD_T_MAX);
  if (vocab < 1 || n_prompt < 0) return fail(PPD_EINVAL, "vocab must be positive, n_prompt >= 0");
  if (n_ept < 1 || n_ept > PPD_EPT_MAX || (int64_t)n_prompt * n_ept > 32767)
    return fail(PPD_EINVAL, "n_ept=%d outside [1, %d] or too many prompt ids", n_ept, PPD_EPT_MAX);
  if (!parent || !ids || !logits || !path || !n_path || !next_tok || !tpl_parent || !tpl_kind ||
      !next_ids)
    return fail(PPD_EINVAL, "NULL argument");
  if (!ws || ws_bytes < 16) return fail(PPD_EWORKSPACE, "workspace (status word) required");
  NextTreeLaunch p{};
  p.parent = parent;
  p.ids = ids;
  p.T = T;
  p.vocab = vocab;
  p.n_ept = n_ept;
  p.logits = logits;
  p.path = path;
  p.n_path = n_path;
  p.next_tok = next_tok;
  p.next_ids = next_ids;
  p.status = (uint32_t *)ws;
  p.tpl_T = tpl_T;
  // the template: topological, candidates under the root or candidates,
  // one prompt chain per EPT group under candidates, in token-distance order
  if (tpl_parent[0] != -1) return fail(PPD_EINVAL, "template: tpl_parent[0] must be -1");
  int n_depths = 0;
  for (int i = 0; i < tpl_T; ++i) {
    const int par = tpl_parent[i], kind = tpl_kind[i];
    int depth = 0;
    if (i > 0) {
      if (par < 0 || par >= i)
        return fail(PPD_EINVAL, "template: tpl_parent[%d]=%d is not an earlier node", i, par);
      const int pk = par > 0 ? tpl_kind[par] : 0;  // the root counts as a candidate
      depth = p.tpl_depth[par] + 1;
      if (kind >= 0) {
        if (pk < 0) return fail(PPD_EINVAL, "template: candidate %d under a prompt token", i);
        if (kind >= PPD_TOPK_MAX || kind >= vocab)
          return fail(PPD_EINVAL, "template: rank %d of node %d too large", kind, i);
        if (depth > PPD_NEXT_MAX_DEPTH)
          return fail(PPD_EINVAL, "template: candidate depth %d > %d", depth, PPD_NEXT_MAX_DEPTH);
        p.k_of_depth[depth] = std::max(p.k_of_depth[depth], kind + 1);
        n_depths = std::max(n_depths, depth);
      } else {
        const int q = -kind - 1;  // prompt embedding: token distance j + 1, EPT group g
        const int j = q / n_ept, g = q % n_ept;
        if (kind < -32767 || j >= n_prompt)
          return fail(PPD_EINVAL, "template: prompt id %d beyond %d token distances", q, n_prompt);
        if (j == 0 ? pk < 0 : pk != -1 - ((j - 1) * n_ept + g))
          return fail(PPD_EINVAL, "template: prompt token %d of node %d out of chain order", q, i);
      }
    }
    if (depth > 127) return fail(PPD_EINVAL, "template too deep");
    p.tpl_depth[i] = (int8_t)depth;
    p.tpl_kind[i] = (int16_t)(i == 0 ? 0 : std::max(kind, -32768));
  }
  if (g_timer.kind == TK_NEXT) g_timer.next = 0;  // one timed launch per call
  timer_events(TK_NEXT, &p.ev_start, &p.ev_stop);
  PPD_TRY_HIP(launch_next_tree(p, n_depths, (hipStream_t)stream));
  return PPD_OK;
}

ppd_status ppd_read_probe(const void *buf, size_t bytes, uint32_t *sink, void *stream) {
  if (!buf || !sink) return fail(PPD_EINVAL, "NULL argument");
  if (bytes % 16 || ((uintptr_t)buf & 15)) return fail(PPD_EINVAL, "buf and bytes must be 16-byte aligned");
  PPD_TRY_HIP(launch_read_probe(buf, bytes, sink, (hipStream_t)stream));
  return PPD_OK;
}

ppd_status ppd_device_status(void *ws, size_t ws_bytes, uint32_t *status_out, int32_t clear,
                             void *stream) {
  if (!ws || ws_bytes < 16 || !status_out) return fail(PPD_EINVAL, "NULL or short workspace");
  hipStream_t s = (hipStream_t)stream;
  PPD_TRY_HIP(hipMemcpyAsync(status_out, ws, sizeof(uint32_t), hipMemcpyDeviceToHost, s));
  PPD_TRY_HIP(hipStreamSynchronize(s));
  if (clear) PPD_TRY_HIP(launch_ws_init(ws, 4, s));
  return PPD_OK;
}

ppd_status ppd_set_kernel_timer(int32_t kind, void *const *start_events, void *const *stop_events,
                                int32_t n_events) {
  if (n_events <= 0) {
    g_timer = KernelTimer{};
    return PPD_OK;
  }
  if (kind < TK_QKV || kind > TK_NEXT || !start_events || !stop_events)
    return fail(PPD_EINVAL, "bad kernel timer arguments");
  g_timer.kind = kind;
  g_timer.start = start_events;
  g_timer.stop = stop_events;
  g_timer.n = n_events;
  g_timer.next = 0;
  return PPD_OK;
}

void ppd_plan_gemm(int32_t kind, int32_t N, int32_t K, int32_t T, int32_t cus, int32_t plan[3]) {
  const GemmPlan p = plan_gemm({kind, N, K}, t_pad_of(T) / 16, cus == kCUs);
  plan[0] = p.gw, plan[1] = p.TX, plan[2] = p.s;
}

void ppd_plan_attention(int32_t nh, int32_t nkv, int32_t B, const int32_t *L, const int32_t *T, int32_t cus,
                        int32_t *splits, int32_t *chunk, int32_t info[2]) {
  int nblk[PPD_BATCH_MAX];
  const int tiles = attn_blocks(B, L, T, nblk);
  const AttnPlan p = plan_attn(nh, nkv, B, nblk, attn_blocks_per_step(tiles), cus == kCUs);
  std::copy(p.splits, p.splits + B, splits);
  std::copy(p.chunk, p.chunk + B, chunk);
  info[0] = p.slots, info[1] = p.meet;
}

const char *ppd_last_error(void) { return g_err.c_str(); }

size_t ppd_packed_weight_bytes(int32_t kind, int32_t rows, int32_t cols) {
  int gk, N;
  if (pack_args(kind, rows, cols, &gk, &N) != PPD_OK) return 0;
  return (size_t)gemm_groups_of(gk, N) * gemm_sub_of(gk) * 16 * cols * sizeof(bf16_t);
}

ppd_status ppd_pack_weight(int32_t kind, int32_t rows, int32_t cols, const void *src, void *dst,
                           void *stream) {
  int gk, N;
  ppd_status st = pack_args(kind, rows, cols, &gk, &N);
  if (st != PPD_OK) return st;
  if (!src || !dst) return fail(PPD_EINVAL, "NULL weight pointer");
  PPD_TRY_HIP(launch_pack_weight(gk, N, cols, (const bf16_t *)src, (bf16_t *)dst, (hipStream_t)stream));
  return PPD_OK;
}

}  // extern "C"

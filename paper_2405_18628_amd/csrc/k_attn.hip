// Split-KV tree attention on the gfx950 matrix cores (Section 4.1: every tree
// node attends to the cached prefix, to its ancestors and to itself).
//
// Keys of one kv head occupy cache positions [0, L + T): the accepted prefix
// [0, L) -- visible to every node -- followed by the tree nodes' own keys
// (written at L + i by the QKV epilogue), visible to node t iff bit i of its
// ancestor mask is set.  The key range is cut into 32-key blocks.
//
// Work decomposition.  A workgroup owns one sequence (a batched step packs
// several, each with its own cache and tree), one head, one of KS contiguous
// key splits and all of that sequence's queries, so each key/value block is
// read once per head.  Its eight waves load the split PARS blocks at a time
// (16-byte non-temporal loads of whole 128-byte lines, the next PARS blocks
// requested while the current ones are multiplied), stage them in a
// double-buffered LDS slot, and multiply: wave w takes block w / QW with
// the 16-query tiles w % QW + QW i, i < NQ, keeping one online softmax per
// query.  A wave reads each key and value fragment from LDS once for all its
// tiles.  (QW, PARS, NQ) follow the tile count so that waves are busy: (2, 4,
// 1) for one tile (1.4B, T = 16: 9.2 us against 9.8 with (4, 2, 1)), (4, 2, 1)
// up to four (7B, T = 64: 18.4 us; (2, 4, 2) 20.5), (4, 2, 2) up to eight.
// The waves' blocks are merged through LDS at the end.  With KS > 1 each
// query's (O, m, l) is stored and the splits are added in split order: inside
// the kernel where an XCD's workgroups are resident together (a head's splits
// share an XCD, so they meet in its L2; each split, once all have arrived at
// the head's counter, merges its share of the queries), else -- batches of
// unequal lengths with more heads than compute units -- by a second launch.
//
// Per 32-key block and query tile, on the matrix cores
// (v_mfma_f32_16x16x32_bf16):
//   S^T[key][query] = K Q^T      keys are the 16-row A operand, queries the B
//                                operand (operand planes written by the QKV
//                                epilogue: two bf16 parts, hi and lo)
//   O^T[d][query]  += V^T P^T    values (stored position-minor, so V^T rows
//                                are contiguous) are the A operand; P^T comes
//                                straight from S^T's accumulator layout: row
//                                m of key tile kt holds key 8 (m / 4) + 4 kt +
//                                (m % 4), so each lane's 8 probabilities are 8
//                                consecutive keys, i.e. a valid B operand.
// Softmax runs in fp32 in the log2 domain against a lazily moved reference
// (rescaling only when a block's maximum exceeds it by more than 2^8); P
// enters the PV product as the sum of two bf16 parts (hi, lo), i.e. to about
// 16 significant bits.
//
// Measured (us a launch, in brackets before two tiles shared a wave's LDS
// reads, batches merged in the kernel and the queries came as operand planes):
// 13B, T = 128, L = 4096 35.8 (41.0), 13B, T = 88 33.8 (36.5), four sequences
// of 16 nodes at 7B 28.0 (31.9 and a merge launch of 5.2), 7B, T = 64, L = 2048
// 18.3 (18.3), L = 32768 109.5 (109.3: 4.9 TB/s, the stream).  At 2k keys a
// launch is bound by its matrix, vector and LDS work (~1.4 us per two blocks)
// and the split exchange (~4 us).  Loading keys and values straight into the
// registers of the wave that multiplies them, four tiles to a wave and one wave
// per SIMD, was slower (7B, T = 64: 23.2 us): nothing hides the softmax there.
#include <algorithm>

#include "ppd_internal.h"

namespace {

constexpr int OROW = PPD_ATTN_OROW;  // partial row: 128 dims, m, l, padding (floats)
constexpr int NT = 512;              // eight waves, two per SIMD
constexpr int KSLOT = 8192;          // 32 keys x 256 bytes
constexpr int SLOT = 2 * KSLOT;      // one block in LDS: keys, then values (128 dims x 64 bytes)

// LDS row of the K slot holding key j (j < 32) of a block: MFMA row m of key
// tile kt holds key 8 (m / 4) + 4 kt + (m % 4)
__device__ __forceinline__ int row_of_key(int j) {
  const int a = j >> 3, kt = (j >> 2) & 1, e = j & 3;
  return kt * 16 + a * 4 + e;
}

// Reductions over the four 16-lane groups of a wave (lanes l, l ^ 16,
// l ^ 32, l ^ 48) with the gfx950 lane-swap instructions: swapping a value
// with itself across 16-lane (32-lane) halves gives each lane its partner's
// value in one of the two results and its own in the other.
__device__ __forceinline__ float quad_max(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float quad_sum(float v) {
  auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// one 16-query tile of a wave
struct QTile {
  u32x4 q[4][2];  // queries (B operand), dims 32 ds + 8 (lane / 16) .. + 7, parts hi, lo
  uint64_t mk0, mk1;
  floatx4 o[8];  // O^T tiles: dims 16 dt + 4 (lane / 16) + e, query lane % 16
  float m_run;   // reference of the exponentials (log2 domain, scaled)
  float l_run;
};

// Merge of one query's KS split rows, 4 dims of a row: the rows are read 8
// at a time (one round trip per batch) and added in split order, scaled to
// the running maximum.  rows(s0, ml, r) loads splits s0 .. s0 + 7 (those
// below KS): ml[v] = (m, l, -, -), r[v] = the 4 dims.
constexpr int MERGE_B = 8;
template <typename ROWS>
__device__ __forceinline__ floatx4 merge_splits(int KS, ROWS rows) {
  constexpr int B = MERGE_B;
  float M = -INFINITY, lsum = 0.f;
  floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
  for (int s0 = 0; s0 < KS; s0 += B) {
    floatx4 ml[B], r[B];
    rows(s0, ml, r);
    float mb = -INFINITY;
#pragma unroll
    for (int v = 0; v < B; ++v)
      if (s0 + v < KS) mb = fmaxf(mb, ml[v][0]);
    if (mb > M) {
      const float f = exp2f(M - mb);  // 0 while M = -inf (nothing accumulated)
      acc *= f;
      lsum *= f;
      M = mb;
    }
#pragma unroll
    for (int v = 0; v < B; ++v) {
      if (s0 + v < KS) {
        const float sc = ml[v][0] == -INFINITY ? 0.f : exp2f(ml[v][0] - M);
        lsum += sc * ml[v][1];
        acc += sc * r[v];
      }
    }
  }
  return acc * (1.f / lsum);
}

// MEET: the splits meet in the kernel (slots in sequence order)
template <int NQ, int QW, int PARS, bool MEET>
__global__ __launch_bounds__(NT, 1) void attn_bf16_kernel(AttnLaunch p) {
  static_assert(QW * PARS * 64 == NT, "one block and tile set per wave");
  constexpr int kRows = PARS * QW * NQ * 16 * OROW * 4;  // bytes of the waves' rows
  constexpr int kRing = 2 * PARS * SLOT;
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kRows > kRing ? kRows : kRing];
  float *rows_s = (float *)lds;  // [PARS][16 QW NQ][OROW], after the main loop

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qw = wave % QW, par = wave / QW;
  const int lr = lane & 15, lg = lane >> 4;
  // this workgroup's XCD set xs and slot -> sequence, head, split
  const int xs = blockIdx.x & 7, slot = blockIdx.x >> 3;
  int sq = 0;
  if constexpr (MEET) {
    for (int j = 1; j < p.sb.B; ++j) sq = slot >= p.slot0[j] ? j : sq;
  } else {
    const int unit = (p.nh + 7) / 8;
    for (int j = 1; j < p.sb.B; ++j) sq = (unsigned)(slot - p.slot0[j]) < (unsigned)(unit * p.splits[j]) ? j : sq;
  }
  const int KS = p.splits[sq];
  const int local = slot - p.slot0[sq];
  const int ks = local % KS, hl = local / KS;
  const int h0 = p.nh * xs / 8, h = h0 + hl;
  if (h >= p.nh * (xs + 1) / 8) return;  // a slot past the XCD's heads
  const int kvh = h / (p.nh / p.nkv);
  const int t0 = p.sb.t0[sq], T = p.sb.t0[sq + 1] - t0, L = p.sb.L[sq], cap = p.sb.cap[sq];
  const int MT = p.T_pad >> 4;
  const int n_keys = L + T;
  const int nblk = (n_keys + 31) >> 5;
  const int b0 = min(nblk, ks * p.chunk[sq]), b1 = min(nblk, b0 + p.chunk[sq]);
  const int nb = b1 - b0;
  const int nsteps = (nb + PARS - 1) / PARS;
  const bf16_t *kbase = p.sb.k[sq] + (size_t)kvh * cap * 128;
  const bf16_t *vbase = p.sb.v[sq] + (size_t)kvh * 128 * cap;

  // ---- this wave's query tiles that exist (tokens t0 + tile 16 + lr)
  const int n_live = min(NQ, ((T + 15) / 16 - qw + QW - 1) / QW);
  QTile qt[NQ];
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const int tl = (qw + QW * i) * 16 + lr;
    const bool live = tl < T;
    const int tq = t0 + min(tl, T - 1);
#pragma unroll
    for (int ds = 0; ds < 4; ++ds) {
      const unsigned char *src = p.q + plane_off(MT, tq, h * 128 + ds * 32 + lg * 8);
      qt[i].q[ds][0] = *(const u32x4 *)src;
      qt[i].q[ds][1] = *(const u32x4 *)(src + kPlaneLo);
    }
    qt[i].mk0 = live ? p.mask[2 * tq] : 0ull;
    qt[i].mk1 = live ? p.mask[2 * tq + 1] : 0ull;
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) qt[i].o[dt] = floatx4{0.f, 0.f, 0.f, 0.f};
    qt[i].m_run = -INFINITY;
    qt[i].l_run = 0.f;
  }
  __builtin_amdgcn_sched_barrier(0);

  // ---- cooperative loads of PARS blocks: K chunk n = tid + 512 i (i < PARS)
  // is key n / 16, column n % 16; V^T chunk n is dim row n / (4 PARS), keys
  // 8 (n % (4 PARS)) .. + 7.  Key rows past the cache capacity are clamped
  // into it (such keys are never visible, and their values are cleared when
  // staged).  Past the split every lane reads the head's first 16 bytes
  // (offsets masked to 0: one line per load), so every step issues the same
  // loads.
  const int b_last = nb > 0 ? b1 - 1 : 0;
  u32x4 kr[PARS], vr[PARS];
  auto request = [&](int st) {
    const int kp0 = min(b0 + PARS * st, b_last) * 32;
    // opaque to the compiler, so that it issues the same loads on every path
    int keep = __builtin_amdgcn_readfirstlane(st < nsteps ? -1 : 0);
    asm volatile("" : "+s"(keep));
#pragma unroll
    for (int i = 0; i < PARS; ++i) {
      const int n = tid + NT * i;
      const int key = min(kp0 + (n >> 4), cap - 1);
      kr[i] = __builtin_nontemporal_load((const u32x4 *)(kbase + ((key * 128 + (n & 15) * 8) & keep)));
      const int g0 = min(kp0 + n % (4 * PARS) * 8, cap - 8);
      vr[i] = __builtin_nontemporal_load((const u32x4 *)(vbase + (((n / (4 * PARS)) * cap + g0) & keep)));
    }
  };
  // LDS destinations of this thread's chunks: block and byte offset within the
  // block slot.  K row R = row_of_key(key % 32), physical 16-byte column =
  // logical ^ (R % 16); V^T row = dim ^ block (two blocks: ^ 2 block), so that
  // the stores of one 16-lane group -- one dim row of four blocks, or two rows
  // of two -- fall into different banks, physical column = logical ^
  // ((dim / 4) % 4)
  constexpr int kVShift = PARS == 2 ? 1 : 0;
  int kofs[PARS], vofs[PARS], kblk[PARS], vblk[PARS], vgrp[PARS];
#pragma unroll
  for (int i = 0; i < PARS; ++i) {
    const int n = tid + NT * i;
    const int k = n >> 4, R = row_of_key(k & 31);
    kblk[i] = k >> 5;
    kofs[i] = R * 256 + (((n & 15) ^ (R & 15)) * 16);
    const int d = n / (4 * PARS), g = n % (4 * PARS);
    vblk[i] = g >> 2;
    vgrp[i] = g & 3;
    vofs[i] = KSLOT + (d ^ (vblk[i] << kVShift)) * 64 + (((g & 3) ^ ((d >> 2) & 3)) * 16);
  }
  // block index of step st, wave block q (past the split: beyond the last key)
  auto block_of = [&](int st, int q) { return PARS * st + q < nb ? b0 + PARS * st + q : nblk + PARS; };
  auto stage = [&](int st) {
    unsigned char *base = lds + (st & 1) * PARS * SLOT;
#pragma unroll
    for (int i = 0; i < PARS; ++i) {
      *(u32x4 *)(base + kblk[i] * SLOT + kofs[i]) = kr[i];
      *(u32x4 *)(base + vblk[i] * SLOT + vofs[i]) = vr[i];
    }
    // a step reaching past the last key: clear the values of keys >= n_keys
    // in LDS (their probabilities are 0, but the cache there may hold
    // anything); each thread rewrites only its own chunks
    if (PARS * st + PARS > nb || n_keys - (b0 + PARS * st) * 32 < 32 * PARS) {
#pragma unroll
      for (int i = 0; i < PARS; ++i) {
        const int keep_n = n_keys - block_of(st, vblk[i]) * 32 - vgrp[i] * 8;
        if (keep_n < 8) {
          u32x4 v = vr[i];
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const uint32_t keep =
                (2 * w < keep_n ? 0xffffu : 0u) | (2 * w + 1 < keep_n ? 0xffff0000u : 0u);
            v[w] &= keep;
          }
          *(u32x4 *)(base + vblk[i] * SLOT + vofs[i]) = v;
        }
      }
    }
  };

  request(0);
  __builtin_amdgcn_sched_barrier(0);

  const float c = p.scale_log2;
  // one block for the wave's tiles
  auto multiply = [&](const unsigned char *sl, int key0) {
    const unsigned char *vs_l = sl + KSLOT;
    // S^T for the two 16-key tiles; the queries' smaller parts first
    floatx4 sc[NQ][2];
#pragma unroll
    for (int i = 0; i < NQ; ++i) sc[i][0] = sc[i][1] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int ds = 0; ds < 4; ++ds) {
      u32x4 ka[2];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
        ka[kt] = *(const u32x4 *)(sl + (kt * 16 + lr) * 256 + (((ds * 4 + lg) ^ lr) * 16));
#pragma unroll
      for (int part = 1; part >= 0; --part)
#pragma unroll
        for (int i = 0; i < NQ; ++i)
#pragma unroll
          for (int kt = 0; kt < 2; ++kt)
            sc[i][kt] = mfma16x16x32(as_bf16x8(ka[kt]), as_bf16x8(qt[i].q[ds][part]), sc[i][kt]);
    }
    u32x4 pb[NQ], pl[NQ];
#pragma unroll
    for (int i = 0; i < NQ; ++i) {
      QTile &Q = qt[i];
      const floatx4 (&s)[2] = sc[i];
      // mask and block max: this lane holds keys key0 + 8 lg + 4 kt + e of its
      // query; scores stay unscaled here (the scale c > 0 keeps the order)
      float sv[8];
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int e = 0; e < 4; ++e) sv[kt * 4 + e] = s[kt][e];
      if (key0 + 32 > L) {
        // this lane's 8 keys key0 + 8 lg .. + 7 (bit u = key j0 + u): visible
        // if in the cached prefix, or a tree key (j - L < T) whose bit j - L of
        // the ancestor mask is set; blocks wholly in the prefix skip this
        const int j0 = key0 + lg * 8;
        const int sh = j0 - L;  // ancestor-mask bit of key j0
        const uint32_t pre = (1u << min(8, max(0, -sh))) - 1u;
        const uint32_t valid = (1u << min(8, max(0, n_keys - j0))) - 1u;
        uint64_t win;  // mask bits sh .. sh + 7 in its low byte (0 below bit 0)
        if (sh >= 128)
          win = 0ull;
        else if (sh >= 64)
          win = Q.mk1 >> (sh - 64);
        else if (sh >= 0)
          win = (Q.mk0 >> sh) | (sh > 56 ? Q.mk1 << (64 - sh) : 0ull);
        else
          win = sh > -8 ? Q.mk0 << -sh : 0ull;
        const uint32_t vis = pre | ((uint32_t)win & valid & 0xffu);
#pragma unroll
        for (int u = 0; u < 8; ++u) sv[u] = (vis >> u) & 1u ? sv[u] : -INFINITY;
      }
      const float lmax = c * fmaxf(fmaxf(fmaxf(sv[0], sv[1]), fmaxf(sv[2], sv[3])),
                                   fmaxf(fmaxf(sv[4], sv[5]), fmaxf(sv[6], sv[7])));
      // Lazy rescaling: the exponentials are taken against a reference (m_run)
      // that moves only when a block's maximum exceeds it by more than 8 (log2
      // units), so probabilities stay below 2^8 and the accumulators are
      // rescaled only then.  The common case needs no exchange between lanes:
      // only when some lane's own maximum exceeds the reference does the wave
      // (all together) reduce the block maximum over each query's four lane
      // groups and move the reference of the queries that need it.
      if (__ballot(lmax > Q.m_run + 8.f)) {
        const float bmax = quad_max(lmax);
        const bool need = bmax > Q.m_run + 8.f;  // the same in a query's four lanes
        // 0 when leaving -inf (nothing accumulated yet), 1 where kept
        const float alpha = need ? __builtin_amdgcn_exp2f(Q.m_run - bmax) : 1.f;
#pragma unroll
        for (int dt = 0; dt < 8; ++dt) Q.o[dt] *= alpha;
        Q.l_run *= alpha;
        Q.m_run = need ? bmax : Q.m_run;
      }
      // a query with nothing visible yet keeps reference -inf: use 0 so that
      // its probabilities are exactly 0
      const float m_eff = Q.m_run == -INFINITY ? 0.f : Q.m_run;
      float pv[8];
      float psum = 0.f;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        pv[e] = __builtin_amdgcn_exp2f(fmaf(sv[e], c, -m_eff));
        psum += pv[e];
      }
      Q.l_run += psum;
      // P = hi + lo, both bf16 (lo the rounding of what hi leaves): the PV
      // product carries P to ~16 significant bits, as the activations are
      // carried (two MFMAs per tile, the smaller part first)
      float plo[8];
#pragma unroll
      for (int e = 0; e < 8; ++e) plo[e] = pv[e] - bf16_to_f32(f32_to_bf16(pv[e]));
      pb[i] = u32x4{pack_bf16x2(pv[0], pv[1]), pack_bf16x2(pv[2], pv[3]), pack_bf16x2(pv[4], pv[5]),
                    pack_bf16x2(pv[6], pv[7])};
      pl[i] = u32x4{pack_bf16x2(plo[0], plo[1]), pack_bf16x2(plo[2], plo[3]), pack_bf16x2(plo[4], plo[5]),
                    pack_bf16x2(plo[6], plo[7])};
    }
#pragma unroll
    for (int dt = 0; dt < 8; ++dt) {
      const int r = dt * 16 + lr;
      const u32x4 va = *(const u32x4 *)(vs_l + (r ^ (par << kVShift)) * 64 + ((lg ^ ((lr >> 2) & 3)) * 16));
#pragma unroll
      for (int i = 0; i < NQ; ++i) qt[i].o[dt] = mfma16x16x32(as_bf16x8(va), as_bf16x8(pl[i]), qt[i].o[dt]);
#pragma unroll
      for (int i = 0; i < NQ; ++i) qt[i].o[dt] = mfma16x16x32(as_bf16x8(va), as_bf16x8(pb[i]), qt[i].o[dt]);
    }
  };

  // ---- main loop.  Step st: stage its blocks (requested a step ago) into LDS
  // slot st & 1 and request step st + 1's into the freed registers; barrier;
  // every wave multiplies its query tiles with its block.  The slot staged
  // here was last read for step st - 2, which every wave finished before step
  // st - 1's barrier.  Blocks past the split lie beyond the last key (values
  // cleared, nothing visible).
  for (int st = 0; st < nsteps; ++st) {
    stage(st);
    __builtin_amdgcn_sched_barrier(0);
    request(st + 1);
    __builtin_amdgcn_sched_barrier(0);
    __syncthreads();
    if (n_live > 0) multiply(lds + ((st & 1) * PARS + par) * SLOT, block_of(st, par) * 32);
  }

  // ---- the waves meet in LDS: thread -> query tid / 32 + 16 n, dims 4 (tid %
  // 32) .. + 3; the output (KS = 1) or this split's row
  __syncthreads();  // the blocks' LDS is free
#pragma unroll
  for (int i = 0; i < NQ; ++i) {
    const float l = quad_sum(qt[i].l_run);
    if (i < n_live) {
      float *row = rows_s + ((size_t)par * (16 * QW * NQ) + (qw + QW * i) * 16 + lr) * OROW;
#pragma unroll
      for (int dt = 0; dt < 8; ++dt) *(floatx4 *)(row + dt * 16 + lg * 4) = qt[i].o[dt];
      if (lg == 0) *(float2 *)(row + 128) = float2{qt[i].m_run, l};
    }
  }
  __syncthreads();
  const int d4 = (tid & 31) * 4;
  const size_t split_floats = (size_t)p.T_pad * OROW;
  float *hp = p.part + (size_t)h * p.max_splits * split_floats + (size_t)t0 * OROW;
  for (int ql = tid >> 5; ql < T; ql += NT / 32) {
    float2 ml[PARS];
    float M = -INFINITY;
#pragma unroll
    for (int w = 0; w < PARS; ++w) {
      ml[w] = *(const float2 *)(rows_s + ((size_t)w * (16 * QW * NQ) + ql) * OROW + 128);
      M = fmaxf(M, ml[w].x);
    }
    float l = 0.f;
    floatx4 o = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < PARS; ++w) {
      const float f = ml[w].x == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ml[w].x - M);
      l += f * ml[w].y;
      o += f * *(const floatx4 *)(rows_s + ((size_t)w * (16 * QW * NQ) + ql) * OROW + d4);
    }
    if (KS == 1) {
      const float inv = 1.f / l;
      store_plane4(p.out, MT, t0 + ql, h * 128 + d4, {o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv});
    } else {
      float *row = hp + (size_t)ks * split_floats + (size_t)ql * OROW;
      *(floatx4 *)(row + d4) = o;
      if (d4 == 0) *(float2 *)(row + 128) = float2{M, l};
    }
  }
  if (!MEET || KS == 1) return;
  // every split of the head stores its rows (in this XCD's L2) and arrives at
  // the head's counter; then each merges queries [T ks / KS, T (ks + 1) / KS)
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_waitcnt(0);  // this thread's row stores have reached L2
  __syncthreads();
  if (tid == 0) xcd_arrive_wait(p.ctr + xs * 32 + p.ctr0[sq] + hl, xs, (uint32_t)KS, p.spin_limit, p.status);
  __syncthreads();
  const __amdgpu_buffer_rsrc_t rp = rsrc_of(hp, (uint32_t)(KS * split_floats * 4));
  for (int ql = T * ks / KS + (tid >> 5); ql < T * (ks + 1) / KS; ql += NT / 32) {
    const floatx4 o = merge_splits(KS, [&](int s0, floatx4(&ml)[MERGE_B], floatx4(&r)[MERGE_B]) {
#pragma unroll
      for (int v = 0; v < MERGE_B; ++v) {
        const size_t row = (size_t)min(s0 + v, KS - 1) * split_floats + (size_t)ql * OROW;
        ml[v] = load_l2(rp, (uint32_t)((row + 128) * 4));
        r[v] = load_l2(rp, (uint32_t)((row + d4) * 4));
      }
    });
    store_plane4(p.out, MT, t0 + ql, h * 128 + d4, {o[0], o[1], o[2], o[3]});
  }
}

// ---- the second launch where a head's splits do not meet: workgroup
// (sequence and head, 16-query tile); thread -> query tid / 32, dims 4 (tid %
// 32) .. + 3.  A launch and one round trip, ~5 us; for it a sequence much longer
// than the rest of its batch is read by several compute units a head: 7B, 16384
// and 7 x 256 cached tokens, 16-node trees, both launches 75.8 us, one workgroup
// a head and sequence 177.7.
__global__ __launch_bounds__(NT) void attn_merge_kernel(AttnLaunch p) {
  const int sq = blockIdx.x / p.nh, h = blockIdx.x % p.nh;
  const int ql = blockIdx.y * 16 + (threadIdx.x >> 5), d4 = (threadIdx.x & 31) * 4;
  const int KS = p.splits[sq], t0 = p.sb.t0[sq];
  if (KS == 1 || ql >= p.sb.t0[sq + 1] - t0) return;  // one split: already final
  const size_t split_floats = (size_t)p.T_pad * OROW;
  const float *hp = p.part + (size_t)h * p.max_splits * split_floats + (size_t)(t0 + ql) * OROW;
  const floatx4 o = merge_splits(KS, [&](int s0, floatx4(&ml)[MERGE_B], floatx4(&r)[MERGE_B]) {
#pragma unroll
    for (int v = 0; v < MERGE_B; ++v) {
      const float *row = hp + (size_t)min(s0 + v, KS - 1) * split_floats;
      ml[v] = *(const floatx4 *)(row + 128);
      r[v] = *(const floatx4 *)(row + d4);
    }
  });
  store_plane4(p.out, p.T_pad >> 4, t0 + ql, h * 128 + d4, {o[0], o[1], o[2], o[3]});
}

}  // namespace

int attn_blocks_per_step(int tiles) { return tiles <= 1 ? 4 : 2; }

hipError_t launch_attn_bf16(const AttnLaunch &a, hipStream_t s) {
  const dim3 grid(8 * a.n_slots), block(NT);
  auto kernel = a.tiles <= 1   ? (a.meet ? attn_bf16_kernel<1, 2, 4, true> : attn_bf16_kernel<1, 2, 4, false>)
                : a.tiles <= 4 ? (a.meet ? attn_bf16_kernel<1, 4, 2, true> : attn_bf16_kernel<1, 4, 2, false>)
                               : (a.meet ? attn_bf16_kernel<2, 4, 2, true> : attn_bf16_kernel<2, 4, 2, false>);
  const bool merge = !a.meet && *std::max_element(a.splits, a.splits + a.sb.B) > 1;
  const hipEvent_t ev0 = (hipEvent_t)a.ev_start, ev1 = (hipEvent_t)a.ev_stop;
  if (ev0)
    hipExtLaunchKernelGGL(kernel, grid, block, 0, s, ev0, merge ? (hipEvent_t) nullptr : ev1, 0, a);
  else
    hipLaunchKernelGGL(kernel, grid, block, 0, s, a);
  if (merge) {
    const dim3 mgrid(a.sb.B * a.nh, a.tiles);
    if (ev1)
      hipExtLaunchKernelGGL(attn_merge_kernel, mgrid, block, 0, s, (hipEvent_t) nullptr, ev1, 0, a);
    else
      hipLaunchKernelGGL(attn_merge_kernel, mgrid, block, 0, s, a);
  }
  return hipGetLastError();
}

// ctx_prefill_attn.hip -- causal prefill attention for gfx950 (MI355X),
// behind ctx_prefill_attn_run in the C ABI declared in include/ctx_decode_attn.h.
//
// Causal prefill of each sequence's newest tokens (the reference next
// observation the fast action conditions on) against its cache, which already
// holds their K/V rows.  The columns of the 16-column MFMA tiles are the
// consecutive (query position, head) pairs of one KV group, column c being
// position c / g and head c % g, so every column carries work for any group
// size g (a position's heads may straddle two workgroups).  32-token K/V blocks,
// up to the workgroup's last query position, are loaded straight into LDS.  Two
// kinds of workgroup, both of kPrefillWaves waves with 48 columns per wave:
//   * wide (kSplitKv false): its waves cover kPrefillCols = 192 columns of one
//     (sequence, KV head) and share every block through a three-stage tile,
//     loaded two blocks ahead of the math;
//   * narrow (kSplitKv true), for calls with too few columns to fill the chip
//     with wide ones: all its waves cover the same kSplitCols = 48 columns, each
//     for a quarter of the blocks through tiles of its own, and their partial
//     results are merged through LDS in a fixed order.  No workspace, no second
//     launch.  One request with 301 new tokens over 8,000: 212 us (56 wide
//     workgroups on 256 CUs, one wave per SIMD) against 81 us.
// Per 32 tokens and 16 columns a wave computes
//   S^T = K Q^T                 (8 MFMA 16x16x32, K rows straight from LDS)
//   causal mask, lazy online softmax
//   O^T += V^T P^T              (8 MFMA 16x16x32 per bf16 term of P)
// where the V^T operand comes from the row-major LDS tile through the LDS
// transpose read, whose 4 values per lane are tokens 4c..4c+3 of one
// dimension -- the rows the S^T tile gives each lane.  P enters the product
// either as one bf16 term (rounded to nearest even; the row sum is taken over
// the rounded weights, so each output row stays a convex combination of V
// rows) or, with CTX_PREFILL_SPLIT_P, as P_hi + P_lo (16 significant bits, a
// second set of 8 MFMAs).

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdint>

#include "ctx_attn_common.h"

namespace {

// K/V block loads use the default (cached) policy: the query tiles of one
// (sequence, KV head) re-read the same blocks, mostly from L2.
constexpr int kPrefillLoadAux = 0;

typedef __attribute__((address_space(3))) void lds_void;
constexpr int kPrefillWaves = 4;  // waves per workgroup
constexpr int kPrefillTiles = 3;  // 16-column tiles per wave
constexpr int kPrefillCols = kPrefillWaves * kPrefillTiles * 16;
constexpr int kSplitCols = kPrefillTiles * 16;  // columns of a workgroup whose waves share the tokens out
constexpr int kPrefillBlock = 32;  // tokens per block
constexpr int kBlockElems = kPrefillBlock * kHeadDim;

// s_waitcnt vmcnt(n) with expcnt and lgkmcnt left open
constexpr int wait_vmcnt(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

struct PrefillPlan {
  int32_t hq;
  int32_t hkv;
  int32_t group;
  int32_t tiles;  // workgroups per (sequence, KV head)
  int32_t units;  // sequences x KV heads
  int32_t last_first;  // the tiles of a unit in falling order
  float scale_log2;
};

// Workgroup barrier with no memory fence: the caller has already waited for
// its own loads into LDS that the other waves will read, and a fence would
// also wait for the loads of later blocks still in flight.  The memory clobber
// keeps the compiler from moving LDS accesses across it.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_barrier" ::: "memory"); }

// 16 bytes per lane from voff in r straight to LDS base + 16 * lane
__device__ __forceinline__ void load16_to_lds(__amdgpu_buffer_rsrc_t r, uint16_t* base, int voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_void*)base, 16, voff, 0, 0, kPrefillLoadAux);
}

// Split a pair of non-negative floats into bf16 hi = the value with its low 16
// bits cleared and bf16 lo = round-to-nearest-even of the exact remainder, so
// that hi + lo carries 16 significant bits; both packed as (a, b).
__device__ __forceinline__ void split_bf16x2(float a, float b, uint32_t* hi, uint32_t* lo) {
  const uint32_t ua = __float_as_uint(a), ub = __float_as_uint(b);
  *hi = __builtin_amdgcn_perm(ub, ua, 0x07060302u);  // high halves of a and b
  *lo = pack_bf16x2(a - __uint_as_float(ua & 0xffff0000u), b - __uint_as_float(ub & 0xffff0000u));
}

// Largest of 8 logits with the NaN-propagating maximum, which gfx950 has as a
// three-input instruction (fmaxf would first quiet each input).  A NaN logit
// gives a NaN weight either way.
__device__ __forceinline__ float max8(float a, float b, float c, float d, float e, float f, float g, float h) {
  const auto mx = [](float x, float y) { return __builtin_elementwise_maximum(x, y); };
  // grouped so that the three-input form covers it in 4 instructions
  return mx(mx(mx(mx(a, b), c), mx(mx(d, e), f)), mx(g, h));
}

template <typename OutT, bool kSplitP, bool kSplitKv, bool kShort>
__global__ __launch_bounds__(64 * kPrefillWaves) __attribute__((amdgpu_waves_per_eu(2))) void prefill_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ kc, const uint16_t* __restrict__ vc,
    const int32_t* __restrict__ offs, const int32_t* __restrict__ lens,
    const int32_t* __restrict__ q_starts, const int32_t* __restrict__ q_lens, PrefillPlan pp,
    OutT* __restrict__ out) {
  // columns of the workgroup, and the part of it that stages a block together:
  // the whole workgroup, or each wave for itself
  constexpr int kTiles = kPrefillTiles;
  constexpr int kCols = kSplitKv ? kSplitCols : kPrefillCols;
  constexpr int kStagers = kSplitKv ? 1 : kPrefillWaves;
  // 16-byte chunks each thread stages per K (and per V) block
  constexpr int kLoads = kPrefillBlock * 16 / (64 * kStagers);
  static_assert(kLoads >= 1 && kLoads * 64 * kStagers == kPrefillBlock * 16, "a block's chunks must divide evenly");
  // all but this wave's newest block of loads have landed
  constexpr int kWaitBlock = wait_vmcnt(2 * kLoads);
  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int col_wave = kSplitKv ? 0 : wave;    // this wave's columns in the workgroup
  const int stage_wave = kSplitKv ? 0 : wave;  // its part of the staging
  const int n = lane & 15;
  const int c = lane >> 4;
  const int g = pp.group;
  // consecutive workgroups go to different XCDs; keep every tile of a unit on
  // one XCD so that its L2 serves the tiles' re-reads of the unit's K/V
  const int slot = blockIdx.x / kXcds;
  // In a grid that is not resident at once, last tile first: it sees the most
  // tokens, and started last it ran on alone (12 fresh prompts of 200..2,000
  // tokens 132 -> 124 us).
  const int tile = pp.last_first ? pp.tiles - 1 - slot % pp.tiles : slot % pp.tiles;
  const int unit = (slot / pp.tiles) * kXcds + (int)(blockIdx.x % kXcds);
  if (unit >= pp.units) return;
  const int kv = unit % pp.hkv;
  const int b = unit / pp.hkv;
  const int nq = q_lens[b];
  // query positions of the workgroup's columns, tile * kCols onwards
  const int first_q = tile * kCols / g;
  if (first_q >= nq) return;  // the whole workgroup: nothing to do
  const int seq_len = lens[b];
  const int hist = seq_len - nq;  // position of query 0
  // one past the last column's position; min(q_end, nq) - 1 rather than
  // min(q_end - 1, nq - 1), a form that compiles to 8 more registers
  const int q_end = (tile * kCols + kCols - 1) / g + 1;
  const int last_q = (q_end < nq ? q_end : nq) - 1;
  const int kv_end = hist + last_q + 1;  // tokens any query of the workgroup attends to
  const size_t row_elems = (size_t)pp.hkv * kHeadDim;
  const int row_bytes = (int)(row_elems * 2);
  const uint16_t* kseq = kc + (size_t)offs[b] * row_elems + (size_t)kv * kHeadDim;
  const uint16_t* vseq = vc + (size_t)offs[b] * row_elems + (size_t)kv * kHeadDim;

  // blocks per stage: one shared by the workgroup, or one per wave
  constexpr int kStageElems = (kSplitKv ? kPrefillWaves : 1) * kBlockElems;
  __shared__ __attribute__((aligned(16))) uint16_t lds_k0[kStageElems];
  __shared__ __attribute__((aligned(16))) uint16_t lds_v0[kStageElems];

  // logits in log2 units are s * cs with cs >= 0: a negative scale flips the
  // sign of q instead (exact in bf16), so that max(s) * cs = max(s * cs)
  const float cs = fabsf(pp.scale_log2);
  const uint32_t qflip = pp.scale_log2 < 0.f ? 0x80008000u : 0u;

  // this lane's query column in each tile: query index qi, head kv * g + hh,
  // attending to positions 0 .. last_pos (columns past the last query attend
  // to the whole block range and are not written)
  int qi[kTiles], hh[kTiles], last_pos[kTiles];
  bf16x8 qb[kTiles][4];
#pragma unroll
  for (int ct = 0; ct < kTiles; ++ct) {
    const int col = tile * kCols + (col_wave * kTiles + ct) * 16 + n;
    qi[ct] = col / g;
    hh[ct] = col - qi[ct] * g;
    const bool valid = qi[ct] < nq;
    last_pos[ct] = valid ? hist + qi[ct] : kv_end - 1;
    if (valid) {
      const uint16_t* qrow =
          q + ((size_t)(q_starts[b] + qi[ct]) * pp.hq + (size_t)kv * g + hh[ct]) * kHeadDim + 8 * c;
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) qb[ct][kk] = as_bf16x8(load16(qrow + 32 * kk) ^ qflip);
    } else {
#pragma unroll
      for (int kk = 0; kk < 4; ++kk) qb[ct][kk] = as_bf16x8(u32x4{0u, 0u, 0u, 0u});
    }
  }
  // the wave's query positions: tokens at or below mask_from are seen by every
  // column; tokens from wave_end on by none (a wave past the last query idles)
  const int wave_q0 = (tile * kCols + col_wave * kTiles * 16) / g;
  const int wave_q1 = (tile * kCols + (col_wave + 1) * kTiles * 16 - 1) / g;
  const bool wave_active = wave_q0 < nq;
  const int mask_from = hist + wave_q0;
  const int wave_end = hist + (wave_q1 < last_q ? wave_q1 : last_q) + 1;

  Softmax st[kTiles];
  f32x4 o[kTiles][8];
  // lazy-rescale thresholds: the running max plus 2^8, in log2 units (for
  // masked blocks, whose logits are scaled first) and divided by cs (for the
  // raw logits of unmasked blocks); both move only with the running max
  float thr[kTiles], thr_raw[kTiles];
#pragma unroll
  for (int ct = 0; ct < kTiles; ++ct) {
    thr[ct] = -INFINITY;
    thr_raw[ct] = -INFINITY;
    st[ct] = Softmax{-INFINITY, 0.f};
#pragma unroll
    for (int nb = 0; nb < 8; ++nb) o[ct][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  // Block loads go straight from memory into the LDS tile (buffer loads with
  // the LDS flag, no registers held).  Such a load writes lane L's 16 bytes at
  // LDS base + 16 L: wave w's round r fills slots 0..15 of tokens
  // 16 r + 4 w + L / 16, so each lane fetches the chunk that the swizzle puts
  // at its slot.  Past kv_end the buffer bound writes zeros.
  int dvo[kLoads];
#pragma unroll
  for (int r = 0; r < kLoads; ++r) {
    const int t = ((kSplitKv ? lane : tid) >> 4) + r * 4 * kStagers;
    dvo[r] = t * row_bytes + (((tid & 15) ^ tile_swizzle(t)) << 4);
  }
  // the resource of the block at tb: past kv_end an empty range (no memory access, zeros in LDS)
  auto block_rsrc = [&](const uint16_t* seq, int tb) {
    const int rem = kv_end - tb;
    const uint32_t bytes = (uint32_t)((rem <= 0 ? 0 : rem < kPrefillBlock ? rem : kPrefillBlock) * row_bytes);
    return make_rsrc(seq + (size_t)tb * row_elems, bytes);
  };
  auto lds_row = [&](uint16_t* dst, int r) { return dst + (r * 4 * kStagers + 4 * stage_wave) * kHeadDim; };

  // per-lane LDS offsets of the operand reads within a 16-token half block
  int k_off[4];
#pragma unroll
  for (int kk = 0; kk < 4; ++kk) k_off[kk] = n * kHeadDim + (((4 * kk + c) ^ tile_swizzle(n)) << 3);
  const int v_tok = 4 * c + (n >> 2);
  const int v_row = v_tok * kHeadDim + 4 * (n & 1);
  const int v_swz = tile_swizzle(v_tok);
  const int v_ch = (n & 3) >> 1;

  // S^T of a staged block: tokens 16 h + 4c + i (i < 4) for every column tile
  auto scores = [&](const uint16_t* kt, f32x4 (&sc)[kTiles][2]) __attribute__((always_inline)) {
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      u32x4 kr[4];
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
        kr[kk] = *reinterpret_cast<const u32x4*>(kt + 16 * h * kHeadDim + k_off[kk]);
#pragma unroll
      for (int ct = 0; ct < kTiles; ++ct) sc[ct][h] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kk = 0; kk < 4; ++kk)
#pragma unroll
        for (int ct = 0; ct < kTiles; ++ct)
          sc[ct][h] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(as_bf16x8(kr[kk]), qb[ct][kk], sc[ct][h], 0, 0, 0);
    }
  };
  // Blocks on the causal diagonal (or past kv_end) are scaled and masked first;
  // their logits then count as they are (factor 1, threshold thr), those of the
  // other blocks with the factor cs (threshold thr_raw).
  auto is_masked = [&](int t0) { return t0 + kPrefillBlock - 1 > mask_from; };
  // The block's logits ready for the softmax, and each lane's largest ones; true
  // if some logit of the wave exceeds its running maximum by 2^8.  One test for
  // all tiles: with a branch per tile, and the masked logits in an array of their
  // own, the compiler moved that array through registers in every block (burst
  // prefill 10.76 -> 10.28 ms, one wave per SIMD 247 -> 219 us).  The thresholds
  // are read before the choice between them, a choice between the arrays would put
  // them in memory.
  auto maxima = [&](int t0, f32x4 (&sc)[kTiles][2], float (&lm)[kTiles]) __attribute__((always_inline)) {
    const bool masked = is_masked(t0);
    if (masked) {
#pragma unroll
      for (int ct = 0; ct < kTiles; ++ct)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int i = 0; i < 4; ++i)
            sc[ct][h][i] = (t0 + 16 * h + 4 * c + i > last_pos[ct]) ? -INFINITY : sc[ct][h][i] * cs;
    }
    float over = -INFINITY;
#pragma unroll
    for (int ct = 0; ct < kTiles; ++ct) {
      const f32x4 a = sc[ct][0], e = sc[ct][1];
      lm[ct] = max8(a[0], a[1], a[2], a[3], e[0], e[1], e[2], e[3]);
      const float t1 = thr[ct], t2 = thr_raw[ct];
      over = fmaxf(over, lm[ct] - (masked ? t1 : t2));
    }
    return __any(over > 0.f);
  };
  // the largest of a column, whose tokens are spread over the 4 rows of 16 lanes
  // (swaps of rows and halves between two copies: register moves, no trip through LDS)
  auto column_max = [&](float x) {
    const uint32_t a = __float_as_uint(x);
    const auto rows = __builtin_amdgcn_permlane16_swap(a, a, false, false);
    const uint32_t b = __float_as_uint(fmaxf(__uint_as_float(rows[0]), __uint_as_float(rows[1])));
    const auto halves = __builtin_amdgcn_permlane32_swap(b, b, false, false);
    return fmaxf(__uint_as_float(halves[0]), __uint_as_float(halves[1]));
  };
  // tile ct's running maximum becomes m; fresh: nothing has been summed yet
  auto rescale = [&](int ct, float m, bool fresh) __attribute__((always_inline)) {
    if (!fresh) {
      const float alpha = fast_exp2(st[ct].m - m);
      st[ct].l *= alpha;
#pragma unroll
      for (int nb = 0; nb < 8; ++nb) o[ct][nb] *= alpha;
    }
    st[ct].m = m;
    thr[ct] = m + kLazyRescale;
    thr_raw[ct] = thr[ct] / cs;
  };
  // the block's softmax weights (one or two bf16 terms)
  auto weights = [&](int t0, const f32x4 (&sc)[kTiles][2], u32x4 (&phi)[kTiles], u32x4 (&plo)[kTiles])
      __attribute__((always_inline)) {
    const float factor = is_masked(t0) ? 1.f : cs;
#pragma unroll
    for (int ct = 0; ct < kTiles; ++ct) {
      float pr[8];
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int i = 0; i < 4; ++i) pr[4 * h + i] = fast_exp2(fmaf(sc[ct][h][i], factor, -st[ct].m));
      if (kSplitP) {
        st[ct].l += ((pr[0] + pr[1]) + (pr[2] + pr[3])) + ((pr[4] + pr[5]) + (pr[6] + pr[7]));
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          uint32_t hw, lw;
          split_bf16x2(pr[2 * j], pr[2 * j + 1], &hw, &lw);
          phi[ct][j] = hw;
          plo[ct][j] = lw;
        }
      } else {
        // one bf16 term; the row sum adds the rounded weights the product
        // uses, a pair per dot product with (1, 1)
        const bf16x2 ones = {(__bf16)1.0f, (__bf16)1.0f};
        float l = st[ct].l;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const bf16x2 pair = {(__bf16)pr[2 * j], (__bf16)pr[2 * j + 1]};  // round to nearest even
          phi[ct][j] = __builtin_bit_cast(uint32_t, pair);
          l = __builtin_amdgcn_fdot2_f32_bf16(pair, ones, l, false);
        }
        st[ct].l = l;
      }
    }
  };
  auto values = [&](const uint16_t* vt, const u32x4 (&phi)[kTiles], const u32x4 (&plo)[kTiles])
      __attribute__((always_inline)) {
    // O^T += V^T P^T: the K dimension holds tokens 4c..4c+3 of both halves.
    // The MFMA stream runs at raised wave priority, so that the other wave
    // on this SIMD fills the matrix core's issue gaps with its softmax.
    __builtin_amdgcn_s_setprio(1);
    // The V^T reads of dimension group nb + 1 are issued before the
    // products of group nb (the scheduling barrier keeps the compiler from
    // sinking them to their use), so their latency hides behind those.
    auto read_vt = [&](int nb, s16x4& v0, s16x4& v1) {
      const int off = v_row + (((2 * nb + v_ch) ^ v_swz) << 3);
      v0 = lds_read_tr16(vt + off);
      v1 = lds_read_tr16(vt + 16 * kHeadDim + off);
    };
    s16x4 nv0, nv1;
    read_vt(0, nv0, nv1);
#pragma unroll
    for (int nb = 0; nb < 8; ++nb) {
      const bf16x8 va = __builtin_bit_cast(bf16x8, __builtin_shufflevector(nv0, nv1, 0, 1, 2, 3, 4, 5, 6, 7));
      if (nb + 1 < 8) read_vt(nb + 1, nv0, nv1);
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int ct = 0; ct < kTiles; ++ct)
        o[ct][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, as_bf16x8(phi[ct]), o[ct][nb], 0, 0, 0);
      if (kSplitP) {
#pragma unroll
        for (int ct = 0; ct < kTiles; ++ct)
          o[ct][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(va, as_bf16x8(plo[ct]), o[ct][nb], 0, 0, 0);
      }
    }
    __builtin_amdgcn_s_setprio(0);
  };
  // a staged block after those before it
  auto attend = [&](int t0, const uint16_t* kt, const uint16_t* vt) __attribute__((always_inline)) {
    f32x4 sc[kTiles][2];
    u32x4 phi[kTiles], plo[kTiles];
    float lm[kTiles];
    scores(kt, sc);
    // lazy rescale: the column maxima are taken only then
    if (maxima(t0, sc, lm)) {
      const bool masked = is_masked(t0);
#pragma unroll
      for (int ct = 0; ct < kTiles; ++ct) {
        // A tile whose own logits stay below its thresholds keeps its maxima: a
        // row's weights are rounded as they would be without the other tiles'
        // rows (and rescaling all three took 10.09 ms against 10.03 for the burst).
        const float t1 = thr[ct], t2 = thr_raw[ct];
        if (!__any(lm[ct] > (masked ? t1 : t2))) continue;
        rescale(ct, fmaxf(st[ct].m, column_max(lm[ct] * (masked ? 1.f : cs))), false);
      }
    }
    weights(t0, sc, phi, plo);
    values(vt, phi, plo);
  };
  // the wave's output rows, where it has seen all of their tokens
  auto finish = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int ct = 0; ct < kTiles; ++ct) {
      float l_tot = st[ct].l + __shfl_xor(st[ct].l, 16);
      l_tot += __shfl_xor(l_tot, 32);
      if (qi[ct] < nq) {
        const float inv = 1.0f / l_tot;
        OutT* orow = out + ((size_t)(q_starts[b] + qi[ct]) * pp.hq + (size_t)kv * g + hh[ct]) * kHeadDim + 4 * c;
#pragma unroll
        for (int nb = 0; nb < 8; ++nb) store4<OutT>(orow + 16 * nb, o[ct][nb] * inv);
      }
    }
  };
  if constexpr (!kSplitKv) {
    __shared__ __attribute__((aligned(16))) uint16_t lds_k1[kStageElems];
    __shared__ __attribute__((aligned(16))) uint16_t lds_v1[kStageElems];
    __shared__ __attribute__((aligned(16))) uint16_t lds_k2[kStageElems];
    __shared__ __attribute__((aligned(16))) uint16_t lds_v2[kStageElems];
    auto issue = [&](int tb, uint16_t* dk, uint16_t* dv) {
      const __amdgpu_buffer_rsrc_t rk = block_rsrc(kseq, tb), rv = block_rsrc(vseq, tb);
#pragma unroll
      for (int r = 0; r < kLoads; ++r) {
        load16_to_lds(rk, lds_row(dk, r), dvo[r]);
        load16_to_lds(rv, lds_row(dv, r), dvo[r]);
      }
    };
    // One 32-token block: wait for this wave's loads of it, then the barrier
    // (every wave's loads have landed, and every wave is done with the stage
    // read in the previous step); the loads of the block two ahead go into that
    // stage, in flight for two steps of math.  The three stages are distinct LDS
    // arrays named at compile time, so the compiler's wait before the reads
    // covers only this stage's loads.
    auto step = [&](int t0, const uint16_t* kt, const uint16_t* vt, uint16_t* nk, uint16_t* nv) __attribute__((always_inline)) {
      // Every step issues the loads of the block two ahead (an empty range past
      // kv_end), so this wave's loads of this block are all but its newest
      // block's worth; the barrier then makes everyone's visible.
      __builtin_amdgcn_s_waitcnt(kWaitBlock);
      lds_barrier();
      issue(t0 + 2 * kPrefillBlock, nk, nv);
      if (wave_active && t0 < wave_end) attend(t0, kt, vt);
    };
    issue(0, lds_k0, lds_v0);
    issue(kPrefillBlock, lds_k1, lds_v1);
    // Block j in stage j % 3; step j issues block j + 2 into stage (j + 2) % 3.
    // An exit in the middle of the loop would join its head and make the compiler
    // wait there for loads that no path to it leaves unfinished, so the loop runs
    // whole rounds of three steps, the last of them on empty blocks.  For short
    // contexts, where those count, the last one or two blocks come after the loop
    // (134 fresh prompts of 37..92 tokens 65.5 -> 62.5 us; the longer code costs
    // the burst over long histories 10.28 -> 10.60 ms).
    if constexpr (kShort) {
      int t0 = 0;
      for (; t0 + 2 * kPrefillBlock < kv_end; t0 += 3 * kPrefillBlock) {
        step(t0, lds_k0, lds_v0, lds_k2, lds_v2);
        step(t0 + kPrefillBlock, lds_k1, lds_v1, lds_k0, lds_v0);
        step(t0 + 2 * kPrefillBlock, lds_k2, lds_v2, lds_k1, lds_v1);
      }
      if (t0 < kv_end) {
        step(t0, lds_k0, lds_v0, lds_k2, lds_v2);
        if (t0 + kPrefillBlock < kv_end) step(t0 + kPrefillBlock, lds_k1, lds_v1, lds_k0, lds_v0);
      }
    } else {
      for (int t0 = 0; t0 < kv_end; t0 += 3 * kPrefillBlock) {
        step(t0, lds_k0, lds_v0, lds_k2, lds_v2);
        step(t0 + kPrefillBlock, lds_k1, lds_v1, lds_k0, lds_v0);
        step(t0 + 2 * kPrefillBlock, lds_k2, lds_v2, lds_k1, lds_v1);
      }
    }
    // no load may land in LDS after the workgroup has released it
    __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));
    finish();
  } else {
    // Wave w takes blocks w, w + 4, w + 8, ... of the workgroup's token range
    // through its own K and V tiles.  A tile is refilled with the wave's next
    // block as soon as it has been read: K while the softmax and P.V run, V while
    // the next block's K Q^T and softmax do.
    // Every wave weighs a block against the running maximum that a pass over all
    // blocks in order would have there, so the rounded weights are those of a wide
    // workgroup and a row differs between the two kinds only by the order of its
    // fp32 sums.  The maxima move rarely: of every block its wave publishes which
    // tiles have a logit past their thresholds, and the column maxima of those, and
    // a wave reads what the three blocks before its own have published.  The waves
    // need not be in step for that.  301 new tokens over 8,000 with keys of equal
    // size: 67 us, 82 with a barrier per round; 59 where each wave had maxima of its
    // own, and weights rounded differently from a wide workgroup's.
    constexpr int kStride = kPrefillWaves * kPrefillBlock;
    // Of block j in slot j mod kSlots: (j + 1) << kTiles | bits of the tiles.  A wave
    // overwrites a slot four of its blocks later, when it has read of every other
    // wave a block that follows, in that wave's order, its last look at the slot.
    constexpr int kSlots = 4 * kPrefillWaves;
    __shared__ uint32_t lds_over[kSlots];
    __shared__ float lds_max[kSlots][kCols];
    uint16_t* const kt = lds_k0 + wave * kBlockElems;
    uint16_t* const vt = lds_v0 + wave * kBlockElems;
    auto issue = [&](const uint16_t* seq, int tb, uint16_t* dst) {
      const __amdgpu_buffer_rsrc_t rs = block_rsrc(seq, tb);
#pragma unroll
      for (int r = 0; r < kLoads; ++r) load16_to_lds(rs, lds_row(dst, r), dvo[r]);
    };
    // Contexts of up to kAlone blocks are one wave's, in order, without the exchange
    // and the merge; the tiles hold its next four blocks.  A prompt of 12 tokens 6.1
    // us, shared by the waves 9.0 (wide 6.0); 12 tokens over 140 9.5 and 10.2.  With
    // a limit of 8, 12 over 240 11.9 against 10.1.
    constexpr int kAlone = 6;
    if (kv_end <= kAlone * kPrefillBlock) {
      if (wave > 0) return;
      auto fill = [&](int t0, int slot) {
        issue(kseq, t0, lds_k0 + slot * kBlockElems);
        issue(vseq, t0, lds_v0 + slot * kBlockElems);
      };
      for (int t0 = 0; t0 < kv_end && t0 < kStride; t0 += kPrefillBlock) fill(t0, t0 / kPrefillBlock);
#pragma nounroll
      for (int t0 = 0; t0 < kv_end; t0 += kPrefillBlock) {
        const int slot = t0 / kPrefillBlock % kPrefillWaves;
        // all loads have landed but those of the blocks after this one
        if (t0 + 3 * kPrefillBlock < kv_end)
          __builtin_amdgcn_s_waitcnt(wait_vmcnt(3 * 2 * kLoads));
        else if (t0 + 2 * kPrefillBlock < kv_end)
          __builtin_amdgcn_s_waitcnt(wait_vmcnt(2 * 2 * kLoads));
        else if (t0 + kPrefillBlock < kv_end)
          __builtin_amdgcn_s_waitcnt(wait_vmcnt(2 * kLoads));
        else
          __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));
        asm volatile("" ::: "memory");
        attend(t0, lds_k0 + slot * kBlockElems, lds_v0 + slot * kBlockElems);
        // the tiles' reads have returned before their refill is issued
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        if (t0 + kStride < kv_end) fill(t0 + kStride, slot);
      }
      finish();
      return;
    }
    // What the blocks before blk have published, one per lane, 0 past them.  Plain
    // accesses between compiler fences: before an atomic one the compiler waits for
    // all loads into LDS, the tiles' among them.
    constexpr int kAhead = kPrefillWaves - 1;
    auto published = [&](int blk) {
      asm volatile("" ::: "memory");
      const uint32_t word = lds_over[(blk - kAhead + lane) & (kSlots - 1)];
      asm volatile("" ::: "memory");
      return lane < kAhead ? word : 0u;
    };
    // Running maxima past the kPrefillWaves blocks from `first` of which `seen`, lane i
    // for block first + i, has the bits of tiles with a logit past older
    // thresholds.  Those only rise, so that no other block moves anything.
    auto advance = [&](int first, uint32_t seen, bool fresh) __attribute__((always_inline)) {
      // row c of 16 lanes holds block first + c, so that one test finds the next that moves
      const bool row_masked = is_masked((first + c) * kPrefillBlock);
      float row_max[kTiles];
#pragma unroll
      for (int ct = 0; ct < kTiles; ++ct) row_max[ct] = lds_max[(first + c) & (kSlots - 1)][ct * 16 + n];
#pragma unroll
      for (int ct = 0; ct < kTiles; ++ct) {
        uint32_t over = (uint32_t)__ballot(seen >> ct & 1);
        if (over == 0) continue;
        float m = st[ct].m, t1 = thr[ct], t2 = thr_raw[ct];
        bool moved = false;
#pragma nounroll
        while (true) {
          const unsigned long long past = __ballot((over >> c & 1) && row_max[ct] > (row_masked ? t1 : t2));
          if (past == 0) break;
          const int i = __builtin_ctzll(past) >> 4;
          const float mx = column_max(c == i ? row_max[ct] : -INFINITY);  // row i's to every row
          m = fmaxf(m, is_masked((first + i) * kPrefillBlock) ? mx : mx * cs);
          t1 = m + kLazyRescale;
          t2 = t1 / cs;
          moved = true;
          over &= ~((2u << i) - 1);
        }
        if (moved) rescale(ct, m, fresh);
      }
    };
    if (tid < kSlots) lds_over[tid] = 0;
    issue(kseq, wave * kPrefillBlock, kt);
    issue(vseq, wave * kPrefillBlock, vt);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");  // the words are zero; the loads stay in flight
    // Every query of the workgroup is a column of every wave, so no block below
    // kv_end is without work; one past it, in the last round, is masked for all.
    int blk = wave;
    for (int r0 = 0; r0 < kv_end; r0 += kStride, blk += kPrefillWaves) {
      const int t0 = blk * kPrefillBlock;
      f32x4 sc[kTiles][2];
      u32x4 phi[kTiles], plo[kTiles];
      float lm[kTiles];
      __builtin_amdgcn_s_waitcnt(wait_vmcnt(kLoads));  // this block's K; its V is still on the way
      asm volatile("" ::: "memory");
      scores(kt, sc);
      // the tile's reads have returned before its refill is issued
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      issue(kseq, t0 + kStride, kt);
      uint32_t seen = published(blk);  // on its way during the test
      uint32_t mine = 0;
      if (maxima(t0, sc, lm)) {
        const bool masked = is_masked(t0);
#pragma unroll
        for (int ct = 0; ct < kTiles; ++ct) {
          const float t1 = thr[ct], t2 = thr_raw[ct];
          if (!__any(lm[ct] > (masked ? t1 : t2))) continue;
          mine |= 1u << ct;
          const float mx = column_max(lm[ct]);
          if (c == 0) lds_max[blk & (kSlots - 1)][ct * 16 + n] = mx;
        }
      }
      // the wave's LDS accesses execute in order: who sees the word sees the maxima
      asm volatile("" ::: "memory");
      lds_over[blk & (kSlots - 1)] = (uint32_t)(blk + 1) << kTiles | mine;
      asm volatile("" ::: "memory");
      // Every wave publishes its blocks in order and waits only for earlier ones,
      // and all are resident: the wave with the earliest block goes on.
      const uint32_t want = lane < kAhead && blk - kAhead + lane >= 0 ? blk - kAhead + lane + 1 : 0;
      if (mine != 0 || !__all(seen == want << kTiles)) {
        while (!__all(seen >> kTiles == want)) seen = published(blk);
        if (mine != 0 || !__all(seen == want << kTiles)) advance(blk - kAhead, lane == kAhead ? mine : seen, r0 == 0);
      }
      weights(t0, sc, phi, plo);
      __builtin_amdgcn_s_waitcnt(wait_vmcnt(kLoads));  // this block's V
      asm volatile("" ::: "memory");
      values(vt, phi, plo);
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      issue(vseq, t0 + kStride, vt);
    }
    __builtin_amdgcn_s_waitcnt(wait_vmcnt(0));
    __syncthreads();
    // past the blocks of the last round that follow this wave's
    {
      const int first = blk - kPrefillWaves + 1;
      const uint32_t seen = lane < kAhead - wave ? lds_over[(first + lane) & (kSlots - 1)] : 0u;
      if (__any(seen & ((1u << kTiles) - 1))) advance(first, seen, false);
    }
    // the tiles now take the waves' partial results

    // Merge of the waves' partial results, all relative to the same maxima, one
    // half of the dimensions at a time: wave w puts its columns' sums and
    // unnormalised outputs into its part of the tiles, 16-byte chunk ch of column j
    // at slot ch ^ (j & 15) (conflict-free writes), and every thread adds up 4
    // dimensions of some columns.
    constexpr int kHalf = kHeadDim / 2;
    constexpr int kChunks = kHalf / 4;
    constexpr int kPartFloats = kCols * kHalf;  // then the sums
    static_assert((kPartFloats + kCols) * 4 <= 2 * kBlockElems * 2,
                  "a wave's partial results must fit half of a tile array");
    auto part_of = [&](int w) {
      return reinterpret_cast<float*>((w < 2 ? lds_k0 : lds_v0) + (w & 1) * 2 * kBlockElems);
    };
    float* const mine = part_of(wave);
#pragma unroll
    for (int ct = 0; ct < kTiles; ++ct) {
      float l_tot = st[ct].l + __shfl_xor(st[ct].l, 16);
      l_tot += __shfl_xor(l_tot, 32);
      if (c == 0) mine[kPartFloats + ct * 16 + n] = l_tot;
    }
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      if (half > 0) __syncthreads();  // the first half has been read
#pragma unroll
      for (int ct = 0; ct < kTiles; ++ct)
#pragma unroll
        for (int nb = 0; nb < 4; ++nb)
          *reinterpret_cast<f32x4*>(mine + (ct * 16 + n) * kHalf + (((4 * nb + c) ^ n) << 2)) = o[ct][4 * half + nb];
      __syncthreads();
      const int ch = tid % kChunks;
#pragma unroll
      for (int j = tid / kChunks; j < kCols; j += 64 * kPrefillWaves / kChunks) {
        const int col = tile * kCols + j;
        const int q_idx = col / g;
        if (q_idx >= nq) continue;
        float l = 0.f;
        f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < kPrefillWaves; ++w) {
          l += part_of(w)[kPartFloats + j];
          acc += *reinterpret_cast<const f32x4*>(part_of(w) + j * kHalf + ((ch ^ (j & 15)) << 2));
        }
        const float inv = 1.0f / l;
        OutT* orow = out + ((size_t)(q_starts[b] + q_idx) * pp.hq + (size_t)kv * g + (col - q_idx * g)) * kHeadDim;
        store4<OutT>(orow + half * kHalf + 4 * ch, acc * inv);
      }
    }
  }
}

struct PrefillArgs {
  const uint16_t *q, *kc, *vc;
  const int32_t *offs, *lens, *q_starts, *q_lens;
  PrefillPlan plan;
  void* out;
  unsigned grid;
  hipStream_t stream;
};

template <typename OutT, bool kSplitP, bool kSplitKv, bool kShort>
void launch_one(const PrefillArgs& a) {
  hipLaunchKernelGGL((prefill_kernel<OutT, kSplitP, kSplitKv, kShort>), dim3(a.grid), dim3(64 * kPrefillWaves), 0,
                     a.stream, a.q, a.kc, a.vc, a.offs, a.lens, a.q_starts, a.q_lens, a.plan,
                     static_cast<OutT*>(a.out));
}

template <typename OutT, bool kSplitP>
void launch_prefill(const PrefillArgs& a, bool split_kv, bool short_kv) {
  if (split_kv)
    launch_one<OutT, kSplitP, true, false>(a);
  else if (short_kv)
    launch_one<OutT, kSplitP, false, true>(a);
  else
    launch_one<OutT, kSplitP, false, false>(a);
}

}  // namespace

extern "C" int ctx_prefill_attn_run(ctx_decode_attn* h, const void* q, const void* k_cache, const void* v_cache,
                         const int32_t* seq_offsets, const int32_t* seq_lens, const int32_t* q_starts,
                         const int32_t* q_lens, int32_t num_seqs, int32_t max_q_len, float scale,
                         uint32_t flags, void* out, void* stream) {
  int rc = check_common(h, num_seqs, scale);
  if (rc != CTX_OK) return rc;
  const ctx_decode_attn_desc& d = h->desc;
  const int g = d.num_q_heads / d.num_kv_heads;
  if (max_q_len < 0) return fail(CTX_ERR_INVALID_ARG, "max_q_len %d < 0", max_q_len);
  if ((flags & ~CTX_PREFILL_SPLIT_P) != 0) return fail(CTX_ERR_INVALID_ARG, "unknown prefill flags 0x%x", flags);
  if (num_seqs == 0 || max_q_len == 0) return CTX_OK;
  if (q == nullptr || k_cache == nullptr || v_cache == nullptr || seq_offsets == nullptr ||
      seq_lens == nullptr || q_starts == nullptr || q_lens == nullptr || out == nullptr)
    return fail(CTX_ERR_INVALID_ARG, "NULL data pointer");
  if (!aligned16(q) || !aligned16(k_cache) || !aligned16(v_cache) || !aligned16(out))
    return fail(CTX_ERR_ALIGNMENT, "q, k_cache, v_cache and out must be 16-byte aligned");
  rc = check_device(h);
  if (rc != CTX_OK) return rc;
  PrefillPlan pp;
  pp.hq = d.num_q_heads;
  pp.hkv = d.num_kv_heads;
  pp.group = g;
  pp.scale_log2 = (float)((double)scale * 1.4426950408889634);
  pp.units = num_seqs * d.num_kv_heads;
  const int64_t cols = (int64_t)max_q_len * g;
  const int64_t units = round_up(pp.units, kXcds);  // padded to whole XCD rounds
  const int64_t whole = units * ((cols + kPrefillCols - 1) / kPrefillCols);
  // A CU holds two workgroups of either kind.  As long as the narrow ones (up to 4
  // times as many, each wave through a quarter of the tokens) are all resident at
  // once, they finish first but for the shortest contexts: one request with 301 new
  // tokens over 8,000 (208 narrow workgroups) 81 us against 212, with 60 over 600
  // 14.4 and 22.5; two fresh prompts of 301 15.0 and 14.1.  In a second round each
  // pays its start and its merge again, which only long contexts win back, and
  // their length is not known here: 4 requests over 4,096..12,288 tokens 222 against
  // 286 us, but 8 fresh prompts of 300 tokens 40.7 against 21.7, 30 requests with
  // 60..90 over 1,200 97 against 58.
  // The fewer waves of the wide ones are idle, the less there is to win.  Where the
  // narrow ones are no more than the wide, one per CU is the limit (64 requests with
  // up to 12 new tokens over up to 400 19.2 against 17.5 us); where they are twice as
  // many, three for two CUs (13..16 new tokens over 2,000: 24 requests 46 against 53
  // us, 28 51 and 53, 32 63 and 54; over 300 28 requests 18.2 and 15.6, 32 18.7 and
  // 15.7); one per CU also where the handle's bound says that no wave can have three
  // blocks (16 requests with 30..36 over up to 220 14.1 against 12.8).
  const int64_t narrow = units * ((cols + kSplitCols - 1) / kSplitCols);
  const bool one_per_cu = narrow <= whole || d.max_seq_len <= 2 * kPrefillWaves * kPrefillBlock;
  const int per_two_cus = one_per_cu ? 2 : narrow <= 2 * whole ? 3 : 4;
  const bool split_kv = 2 * narrow <= per_two_cus * (int64_t)h->num_cus;
  // up to 16 blocks at most: the last two steps of the wide kernel's loop count
  const bool short_kv = d.max_seq_len <= 16 * kPrefillBlock;
  const int64_t blocks = split_kv ? narrow : whole;
  pp.last_first = blocks > 2 * (int64_t)h->num_cus;
  pp.tiles = (int32_t)(blocks / units);
  if (whole > INT32_MAX) return fail(CTX_ERR_INVALID_ARG, "prefill grid too large");
  const PrefillArgs a{static_cast<const uint16_t*>(q), static_cast<const uint16_t*>(k_cache),
                      static_cast<const uint16_t*>(v_cache), seq_offsets, seq_lens, q_starts, q_lens, pp, out,
                      (unsigned)blocks, reinterpret_cast<hipStream_t>(stream)};
  const bool split_p = (flags & CTX_PREFILL_SPLIT_P) != 0;
  if (d.out_dtype == CTX_DTYPE_F32)
    split_p ? launch_prefill<float, true>(a, split_kv, short_kv) : launch_prefill<float, false>(a, split_kv, short_kv);
  else
    split_p ? launch_prefill<uint16_t, true>(a, split_kv, short_kv) : launch_prefill<uint16_t, false>(a, split_kv, short_kv);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return hip_fail(e, "kernel launch");
  return CTX_OK;
}

// ctx_opd_loss.hip -- fused OPD token loss and logits gradient for gfx950
// (MI355X), behind the C ABI declared in include/ctx_opd_loss.h.
//
// The loss of App. OPD Optimization needs, per supervised token, the
// student's log-probability of the sampled token, i.e. a log-sum-exp over the
// whole vocabulary row (151,936 bf16 logits = 297 KiB for the Qwen3 students),
// and back-propagation writes a gradient row of the same size.  Everything
// else is a handful of scalars per token, so the work is bound by HBM, and
// the least traffic is one read of each logits row and one write of each
// gradient row.
//
// Design:
//   * opd_weight_kernel: one workgroup per response counts its supervised
//     tokens and writes w_j = m_j / (B (M_b + eps)).
//   * opd_row_kernel: persistent workgroups walk the token rows; each holds a
//     whole row in registers (thread t owns the 16-byte chunks t + kThreads k,
//     k < C: coalesced, non-temporal loads) and has 256, 512 or 1024 threads, the
//     fewest that can (up to 19 chunks per thread; 26 of 512 threads), so that a CU
//     works on 4, 2 or 1 rows (8 short ones) at different stages.  It reduces the row maximum and
//     the sum of exp over the registers (lane moves, then the waves' partials
//     through LDS, always in the same order), forms lp, the clipped ratio, the
//     dual-clip loss and the per-row gradient scale g, and writes the gradient
//     row g (onehot - softmax) from the same registers, rounded to bf16.  A row
//     whose g is 0 (a flat clipping regime or A = 0) writes zeros without the
//     second exp pass; a masked row is not read at all.  The next row's loads are
//     issued chunk by chunk as the last pass frees the registers: the gradient
//     pass, or for the loss alone the sum pass (5,716 rows of 151,936 columns:
//     355 us when it waited for the row's end, 288 then, 271 with row_max's packed
//     words, 6.35 TB/s).
//   * opd_reduce_kernel: loss = sum_j w_j l_j in double precision, one
//     workgroup, fixed order (deterministic, no atomics).

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdarg>
#include <cstdint>
#include <cstdio>

#include "ctx_opd_loss.h"

// the library's per-thread last-error message (defined with the attention entry points)
__attribute__((visibility("hidden"))) int ctx_report_error(int code, const char* msg);
__attribute__((visibility("hidden"))) void ctx_clear_error();

namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxRowThreads = 1024;
constexpr int kChunk = 8;  // bf16 per 16-byte chunk
constexpr int kMaxChunksPerThread = 19;  // 76 VGPRs of row data: 128 VGPRs at 16 waves per CU
// most chunks per thread of a 512-thread workgroup: still 128 VGPRs, 16 waves per CU
constexpr int kMaxChunks512 = 26;
constexpr int64_t kMaxVocab = (int64_t)kMaxRowThreads * kChunk * kMaxChunksPerThread;  // 155,648
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

// Chunks per thread up to which a CU takes 32 waves of rows instead of 16: with
// so little work per row the reductions' latency is what more rows hide (2,000
// columns, 18,387 rows: 59 us with 32 waves, 65 with 16; with 7 chunks, 12,944
// columns, 90 and 87).
constexpr int kLightChunks = 4;

// Calls of up to kOwnWeightTokens tokens whose rows take 256 threads find each
// row's weight in the row kernel, which saves the launch of opd_weight_kernel (a
// small call is bound by its launches) for at most one read of the mask, 2 KiB
// from L2, and of as many response bounds per row; with more responses than that,
// most of them empty, the search would grow past it.  Longer rows keep the launch: the work would take them past
// the registers that let two workgroups share a CU.
constexpr int32_t kOwnWeightTokens = 2048;
constexpr int kOwnWeightThreads = 256;

struct OpdParams {
  float clip_log;
  float delta;
  float kappa;
  float eps;
};

__device__ __forceinline__ float lo_bf16(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi_bf16(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// round to nearest even, two floats into one word (a low, b high)
__device__ __forceinline__ uint32_t pack_bf16x2(float a, float b) {
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  bf16x2 v = {(__bf16)a, (__bf16)b};
  return __builtin_bit_cast(uint32_t, v);
}

// x of the lane kBy further round in the row of 16
template <int kBy>
__device__ __forceinline__ float row_rotate(float x) {
  return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x120 + kBy, 0xf, 0xf, false));
}

// Reduction over the wave, in a fixed order: halves of 32 and 16 lanes by
// shuffles, then of 8, 4, 2 and 1 by rotations of the rows, where the lanes that
// far apart hold the same (register moves instead of trips through LDS).  Every
// lane ends with the result.
template <typename Op>
__device__ __forceinline__ float wave_reduce(float x, Op op) {
  x = op(x, __shfl_xor(x, 32));
  x = op(x, __shfl_xor(x, 16));
  x = op(x, row_rotate<8>(x));
  x = op(x, row_rotate<4>(x));
  x = op(x, row_rotate<2>(x));
  return op(x, row_rotate<1>(x));
}

// The same over a workgroup of kThreads threads: the waves' results in wave order.
template <int kThreads, typename Op>
__device__ __forceinline__ float block_reduce(float x, float* red, Op op) {
  x = wave_reduce(x, op);
  __syncthreads();  // red is free (previous reduction read it)
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = x;
  __syncthreads();
  float r = red[0];
#pragma unroll
  for (int w = 1; w < kThreads / 64; ++w) r = op(r, red[w]);
  return r;
}

template <int kThreads>
__device__ __forceinline__ float block_max(float x, float* red) {
  return block_reduce<kThreads>(x, red, [](float a, float b) { return fmaxf(a, b); });
}

template <int kThreads>
__device__ __forceinline__ float block_sum(float x, float* red) {
  return block_reduce<kThreads>(x, red, [](float a, float b) { return a + b; });
}

__global__ __launch_bounds__(256) void opd_weight_kernel(const uint8_t* __restrict__ mask,
                                                         const int32_t* __restrict__ seq_starts,
                                                         int32_t num_seqs, float eps,
                                                         float* __restrict__ weight) {
  __shared__ int red[4];
  const int b = blockIdx.x;
  const int s0 = seq_starts[b], s1 = seq_starts[b + 1];
  int cnt = 0;
  for (int j = s0 + (int)threadIdx.x; j < s1; j += 256) cnt += mask[j] ? 1 : 0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) cnt += __shfl_xor(cnt, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = cnt;
  __syncthreads();
  const int mb = red[0] + red[1] + red[2] + red[3];
  const float w = (float)(1.0 / ((double)num_seqs * ((double)mb + (double)eps)));
  for (int j = s0 + (int)threadIdx.x; j < s1; j += 256) weight[j] = mask[j] ? w : 0.f;
}

// w_j of a supervised row j, by one wave: the row's response (the first that ends
// after it) and a count of its supervised tokens, as opd_weight_kernel has them.
__device__ __forceinline__ float row_weight(const uint8_t* __restrict__ mask, const int32_t* __restrict__ seq_starts,
                                            int32_t num_seqs, float eps, int j) {
  const int lane = threadIdx.x & 63;
  int b = 0;
  for (int base = 0; base < num_seqs; base += 64) {
    const unsigned long long after = __ballot(base + lane < num_seqs && seq_starts[base + lane + 1] > j);
    if (after != 0) {
      b = base + __builtin_ctzll(after);
      break;
    }
  }
  const int s0 = seq_starts[b], s1 = seq_starts[b + 1];
  int mb = 0;
  for (int base = s0; base < s1; base += 64) {
    const int i = base + lane;
    mb += __builtin_popcountll(__ballot(i < s1 && mask[i < s1 ? i : s0] != 0));
  }
  return (float)(1.0 / ((double)num_seqs * ((double)mb + (double)eps)));
}

// eq:opd-dual-clip for one token: the loss and d loss / d rho
__device__ __forceinline__ void dual_clip_loss(float rho, float a, const OpdParams& p, float* loss,
                                               float* dloss) {
  const float lo = 1.f - p.delta, hi = 1.f + p.delta;
  const float clipped = fminf(fmaxf(rho, lo), hi);
  const float dclipped = (rho > lo && rho < hi) ? 1.f : 0.f;
  const float unclipped_term = rho * a, clipped_term = clipped * a;
  float l, d;
  if (unclipped_term <= clipped_term) {
    l = -unclipped_term;
    d = -a;
  } else {
    l = -clipped_term;
    d = -a * dclipped;
  }
  if (a < 0.f && -p.kappa * a < l) {
    l = -p.kappa * a;
    d = 0.f;
  }
  *loss = l;
  *dloss = d;
}

// Buffer resource over `bytes` bytes from a wave-uniform base: loads past
// the end return zeros and stores past it are dropped.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t row_rsrc(const void* base, uint32_t bytes) {
  const uint64_t a = reinterpret_cast<uint64_t>(base);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
  const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
  const uint64_t u = ((uint64_t)hi << 32) | lo;
  return __builtin_amdgcn_make_buffer_rsrc(reinterpret_cast<void*>(u), (short)0,
                                           (int)__builtin_amdgcn_readfirstlane(bytes), 0x00020000);
}

constexpr int kNonTemporal = 2;  // buffer cache-policy bits: streamed once
// Chunk offsets go in the VGPR offset, which the buffer range check covers;
// the SGPR offset stays 0.
constexpr int kWaitVmcnt0 = 0x0F70;  // s_waitcnt vmcnt(0), expcnt and lgkmcnt left open

// An empty asm that "may change" every chunk of the row: the compiler then
// recomputes the cheap bf16 -> fp32 unpacking in each pass instead of keeping
// eight unpacked floats per chunk alive across passes (two rows' worth of
// registers).  It emits no instruction.
template <int C>
__device__ __forceinline__ void opaque(u32x4 (&x)[C]) {
#pragma unroll
  for (int k = 0; k < C; ++k) asm volatile("" : "+v"(x[k]));
}

// The largest logit of the row that the workgroup holds in x.
// The high half of a word needs no unpacking: as a float the word lies between
// its high bf16 and the next one further from zero, so the largest word has the
// largest high half (the loss alone over 5,716 rows of 151,936 columns 289 -> 269
// us: this pass overlaps no loads).  Over a non-zero low half an infinity reads
// as NaN; a row with such a word, a NaN or +inf takes a second pass over both
// halves unpacked.
template <int C, int kThreads>
__device__ __forceinline__ float row_max(const u32x4 (&x)[C], int t, int vocab, float* red) {
  float mx = -INFINITY, mw = -INFINITY;
#pragma unroll
  for (int k = 0; k < C - 1; ++k) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      mx = fmaxf(mx, lo_bf16(x[k][i]));
      mw = __builtin_elementwise_maximum(mw, __uint_as_float(x[k][i]));  // keeps a NaN
    }
    __builtin_amdgcn_sched_barrier(0);  // chunk by chunk: bounded live ranges
  }
  // the last round may pass the vocabulary
  const int c0 = (t + (C - 1) * kThreads) * kChunk;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (c0 + 2 * i < vocab) mx = fmaxf(mx, lo_bf16(x[C - 1][i]));
    if (c0 + 2 * i + 1 < vocab) mx = fmaxf(mx, hi_bf16(x[C - 1][i]));
  }
  const float m = block_max<kThreads>(mw == mw ? fmaxf(mx, hi_bf16(__float_as_uint(mw))) : INFINITY, red);
  if (C == 1 || m < INFINITY) return m;
#pragma unroll
  for (int k = 0; k < C - 1; ++k) {
#pragma unroll
    for (int i = 0; i < 4; ++i) mx = fmaxf(mx, hi_bf16(x[k][i]));
    __builtin_amdgcn_sched_barrier(0);
  }
  return block_max<kThreads>(mx, red);
}

template <int C, int kThreads, bool kGrad>
__global__ __launch_bounds__(kThreads) void opd_row_kernel(
    const uint16_t* __restrict__ logits, int64_t row_stride, int32_t vocab, int32_t num_rows,
    const int32_t* __restrict__ tokens, const float* __restrict__ old_logp,
    const float* __restrict__ teacher_logp, const uint8_t* __restrict__ mask,
    float* __restrict__ weight, const int32_t* __restrict__ seq_starts, int32_t num_seqs, OpdParams prm,
    float* __restrict__ token_logp, float* __restrict__ token_loss, uint16_t* __restrict__ grad,
    int64_t grad_stride) {
  __shared__ float red[kThreads / 64];
  // a row's weight computed here, or read as opd_weight_kernel has written it
  const bool own_weights = kThreads == kOwnWeightThreads && seq_starts != nullptr;
  const int tid = threadIdx.x;
  const int nchunks = (vocab + kChunk - 1) / kChunk;
  const int nwhole = vocab / kChunk;  // chunks with 8 columns below vocab
  // C = ceil(nchunks / kThreads): rounds k < C - 1 give every thread a whole
  // chunk; only the last round tests chunks and columns against vocab
  constexpr int kwhole = C - 1;
  const uint32_t load_bytes = (uint32_t)nchunks * 16u;   // loads: every chunk (the partial one padded)
  const uint32_t store_bytes = (uint32_t)nwhole * 16u;   // stores: whole chunks; a partial one apart
  const int voff = tid * 16;

  // Persistent: rows blockIdx.x, + gridDim.x, ...  The row is held in x; the
  // next row's loads are issued chunk by chunk as the last pass over x (the
  // gradient's, or without one the sum's) frees it.
  u32x4 x[C];
  int j = blockIdx.x;
  if (j >= num_rows) return;
  bool sup = mask[j] != 0;
  if (sup) {
    const __amdgpu_buffer_rsrc_t rr = row_rsrc(logits + (size_t)j * row_stride, load_bytes);
#pragma unroll
    for (int k = 0; k < C; ++k)
      x[k] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(rr, voff + k * kThreads * 16, 0,
                                                                              kNonTemporal));
  }
#pragma nounroll
  for (; j < num_rows; j += gridDim.x) {
    // per-row copy of the lane index, opaque to the compiler: lane-dependent
    // masks and offsets are recomputed per row (a few instructions) instead of
    // being hoisted out of the row loop, where they would occupy registers
    int t = tid;
    asm volatile("" : "+v"(t));
    const int vo = t * 16;
    const int jn = j + (int)gridDim.x;
    const bool next_sup = jn < num_rows && mask[jn] != 0;
    const __amdgpu_buffer_rsrc_t nr = row_rsrc(logits + (size_t)(next_sup ? jn : j) * row_stride, next_sup ? load_bytes : 0u);
    auto refill = [&](int k) {
      x[k] = __builtin_bit_cast(u32x4, __builtin_amdgcn_raw_buffer_load_b128(nr, vo + k * kThreads * 16, 0,
                                                                              kNonTemporal));
    };
    float g = 0.f, lse2 = 0.f;
    int tok = -1;
    if (sup) {
      // the token's values, asked for before the passes that they are needed after
      tok = tokens[j];
      const bool tok_ok = tok >= 0 && tok < vocab;
      const float zt = tok_ok ? __uint_as_float((uint32_t)logits[(size_t)j * row_stride + tok] << 16)
                              : __builtin_nanf("");
      const float old = old_logp[j], teacher = teacher_logp[j];
      const float wj = own_weights ? row_weight(mask, seq_starts, num_seqs, prm.eps, j) : weight[j];
      float m2 = row_max<C, kThreads>(x, t, vocab, red) * kLog2e;
      asm volatile("" : "+v"(m2));  // rounded: not fused into a sum here or there, the modes agree bit for bit
      opaque(x);
      float s = 0.f;
      // as below: the row has landed, the refills need not wait for each other
      if (!kGrad) __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
#pragma unroll
      for (int k = 0; k < C; ++k) {
        if (k < kwhole) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            s += __builtin_amdgcn_exp2f(fmaf(lo_bf16(x[k][i]), kLog2e, -m2)) +
                 __builtin_amdgcn_exp2f(fmaf(hi_bf16(x[k][i]), kLog2e, -m2));
        } else {
          const int c0 = (t + k * kThreads) * kChunk;
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            if (c0 + 2 * i < vocab) s += __builtin_amdgcn_exp2f(fmaf(lo_bf16(x[k][i]), kLog2e, -m2));
            if (c0 + 2 * i + 1 < vocab) s += __builtin_amdgcn_exp2f(fmaf(hi_bf16(x[k][i]), kLog2e, -m2));
          }
        }
        if (!kGrad) refill(k);
        __builtin_amdgcn_sched_barrier(0);
      }
      lse2 = m2 + __log2f(block_sum<kThreads>(s, red));  // log2 of sum_v exp(z_v)
      if (kGrad) opaque(x);

      // per-token scalars (every thread computes them; they are uniform)
      const float lp = fmaf(-lse2, kLn2, zt);
      const float a = teacher - old;
      const float r = lp - old;
      const float rc = fminf(fmaxf(r, -prm.clip_log), prm.clip_log);
      const float rho = expf(rc);
      const float drho = (r > -prm.clip_log && r < prm.clip_log) ? rho : 0.f;
      float l, dl;
      dual_clip_loss(rho, a, prm, &l, &dl);
      g = wj * dl * drho;
      if (t == 0) {
        if (token_logp != nullptr) token_logp[j] = lp;
        token_loss[j] = l;
        if (own_weights) weight[j] = wj;
      }
    } else if (t == 0) {  // no loss, no gradient, logits not read
      if (token_logp != nullptr) token_logp[j] = 0.f;
      token_loss[j] = 0.f;
      if (own_weights) weight[j] = 0.f;
    }

    if (kGrad) {
      // gradient row g (onehot(tok) - exp(z - lse)); zeros when g = 0 (masked
      // rows, flat clipping regimes); then the next row's chunk k into x[k]
      const __amdgpu_buffer_rsrc_t gr = row_rsrc(grad + (size_t)j * grad_stride, store_bytes);
      const float ng = -g;
      // Every load of this row has landed (the passes above read them); saying
      // so here lets the compiler issue the chunk-by-chunk refills below without
      // waiting on each other (on the masked-row path it could not tell).
      __builtin_amdgcn_s_waitcnt(kWaitVmcnt0);
#pragma unroll
      for (int k = 0; k < C; ++k) {
        const int q = t + k * kThreads;
        u32x4 o = {0u, 0u, 0u, 0u};
        if (g != 0.f) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
            o[i] = pack_bf16x2(ng * __builtin_amdgcn_exp2f(fmaf(lo_bf16(x[k][i]), kLog2e, -lse2)),
                               ng * __builtin_amdgcn_exp2f(fmaf(hi_bf16(x[k][i]), kLog2e, -lse2)));
          if (q == tok / kChunk) {  // the sampled token's entry: g (1 - p)
            const int e = tok - q * kChunk;
            const uint32_t w = o[e >> 1];
            const float zv = (e & 1) ? hi_bf16(x[k][e >> 1]) : lo_bf16(x[k][e >> 1]);
            const float gv = fmaf(ng, __builtin_amdgcn_exp2f(fmaf(zv, kLog2e, -lse2)), g);
            const uint32_t hv = pack_bf16x2(gv, gv) & 0xffffu;
            o[e >> 1] = (e & 1) ? (w & 0xffffu) | (hv << 16) : (w & 0xffff0000u) | hv;
          }
        }
        if (k < C - 1 || q < nwhole) {
          __builtin_amdgcn_raw_buffer_store_b128(
              __builtin_bit_cast(__attribute__((ext_vector_type(4))) unsigned, o), gr, vo + k * kThreads * 16, 0,
              kNonTemporal);
        } else if (q == nwhole && nwhole < nchunks) {  // the partial chunk: its columns below vocab
          uint16_t* gp = grad + (size_t)j * grad_stride + (size_t)nwhole * kChunk;
          for (int e = 0; e < vocab - nwhole * kChunk; ++e)
            gp[e] = (uint16_t)(e & 1 ? o[e >> 1] >> 16 : o[e >> 1] & 0xffffu);
        }
        refill(k);
        // keep the refill of x[k] after its last use: hoisting the loads would
        // need a second row's worth of registers
        __builtin_amdgcn_sched_barrier(0);
      }
    } else if (!sup && next_sup) {
#pragma unroll
      for (int k = 0; k < C; ++k) refill(k);
    }
    sup = next_sup;
  }
}

__global__ __launch_bounds__(1024) void opd_reduce_kernel(const float* __restrict__ weight,
                                                          const float* __restrict__ token_loss,
                                                          int32_t n, float* __restrict__ loss) {
  __shared__ double red[16];
  double acc = 0.0;
  for (int j = threadIdx.x; j < n; j += 1024) acc += (double)weight[j] * (double)token_loss[j];
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int w = 0; w < 16; ++w) t += red[w];
    *loss = (float)t;
  }
}

int fail(int code, const char* fmt, ...) {
  char msg[512];
  va_list ap;
  va_start(ap, fmt);
  vsnprintf(msg, sizeof msg, fmt, ap);
  va_end(ap);
  return ctx_report_error(code, msg);
}

bool aligned16(const void* ptr) { return (reinterpret_cast<uintptr_t>(ptr) & 15u) == 0; }

struct RowArgs {
  const uint16_t* logits;
  int64_t stride;
  int32_t vocab, n;
  const int32_t* tokens;
  const float *old_lp, *tea_lp;
  const uint8_t* mask;
  float* weight;
  const int32_t* seq_starts;  // null: the weights are there already
  int32_t num_seqs;
  OpdParams prm;
  float *token_logp, *token_loss;
  uint16_t* grad;
  int64_t grad_stride;
  int cus;
  hipStream_t stream;
};

template <int C, int kThreads, bool kGrad>
void launch_rows(const RowArgs& a) {
  // resident workgroups
  constexpr int kPerCu = (C <= kLightChunks ? 2048 : 1024) / kThreads;
  const int64_t most = (int64_t)a.cus * kPerCu;
  const unsigned grid = (unsigned)(a.n < most ? a.n : most);
  hipLaunchKernelGGL((opd_row_kernel<C, kThreads, kGrad>), dim3(grid), dim3(kThreads), 0, a.stream, a.logits, a.stride,
                     a.vocab, a.n, a.tokens, a.old_lp, a.tea_lp, a.mask, a.weight, a.seq_starts, a.num_seqs, a.prm,
                     a.token_logp, a.token_loss, a.grad, a.grad_stride);
}

// The kernel with exactly ceil(chunks / kThreads) chunks per thread, kLo <= that <= kHi.
template <int kThreads, int kLo, int kHi>
void launch_rows_of(int per_thread, const RowArgs& a) {
  if constexpr (kLo < kHi) {
    if (per_thread > kLo) return launch_rows_of<kThreads, kLo + 1, kHi>(per_thread, a);
  }
  a.grad != nullptr ? launch_rows<kLo, kThreads, true>(a) : launch_rows<kLo, kThreads, false>(a);
}

}  // namespace

extern "C" int ctx_opd_loss_run(const void* logits, int64_t row_stride, int32_t vocab, const int32_t* tokens,
                                const float* old_logp, const float* teacher_logp, const uint8_t* mask,
                                const int32_t* seq_starts, int32_t num_seqs, int32_t num_tokens,
                                const ctx_opd_loss_params* params, float* token_logp, float* token_weight,
                                float* token_loss, float* loss, void* grad_logits, int64_t grad_row_stride,
                                void* stream) {
  ctx_clear_error();
  if (params == nullptr) return fail(CTX_ERR_INVALID_ARG, "params is NULL");
  const ctx_opd_loss_params p = *params;
  if (!(std::isfinite(p.log_ratio_clip) && p.log_ratio_clip > 0.f))
    return fail(CTX_ERR_INVALID_ARG, "log_ratio_clip must be finite and > 0");
  if (!(std::isfinite(p.clip_delta) && p.clip_delta >= 0.f && p.clip_delta < 1.f))
    return fail(CTX_ERR_INVALID_ARG, "clip_delta must be in [0, 1)");
  if (!(std::isfinite(p.dual_clip) && p.dual_clip > 1.f))
    return fail(CTX_ERR_INVALID_ARG, "dual_clip must be finite and > 1");
  if (!(std::isfinite(p.eps) && p.eps >= 0.f)) return fail(CTX_ERR_INVALID_ARG, "eps must be finite and >= 0");
  if (num_seqs < 0 || num_tokens < 0) return fail(CTX_ERR_INVALID_ARG, "negative num_seqs or num_tokens");
  if (num_seqs == 0 && num_tokens > 0) return fail(CTX_ERR_INVALID_ARG, "tokens without responses");
  if (vocab <= 0) return fail(CTX_ERR_INVALID_ARG, "vocab %d <= 0", vocab);
  if (vocab > kMaxVocab) return fail(CTX_ERR_UNSUPPORTED, "vocab %d > %lld", vocab, (long long)kMaxVocab);
  if (row_stride < vocab || row_stride % kChunk != 0)
    return fail(CTX_ERR_INVALID_ARG, "row_stride %lld must be >= vocab and a multiple of 8", (long long)row_stride);
  if (loss == nullptr || seq_starts == nullptr) return fail(CTX_ERR_INVALID_ARG, "NULL loss or seq_starts");
  // per-token arrays of an empty batch are never touched and may be NULL
  if (num_tokens > 0 && (token_weight == nullptr || token_loss == nullptr))
    return fail(CTX_ERR_INVALID_ARG, "NULL token_weight or token_loss");
  if (num_tokens > 0 && (logits == nullptr || tokens == nullptr || old_logp == nullptr ||
                         teacher_logp == nullptr || mask == nullptr))
    return fail(CTX_ERR_INVALID_ARG, "NULL per-token input");
  if (grad_logits != nullptr && (grad_row_stride < vocab || grad_row_stride % kChunk != 0))
    return fail(CTX_ERR_INVALID_ARG, "grad_row_stride %lld must be >= vocab and a multiple of 8",
                (long long)grad_row_stride);
  if ((logits != nullptr && !aligned16(logits)) || (grad_logits != nullptr && !aligned16(grad_logits)))
    return fail(CTX_ERR_ALIGNMENT, "logits and grad_logits must be 16-byte aligned");
  hipStream_t s = reinterpret_cast<hipStream_t>(stream);
  const OpdParams prm{p.log_ratio_clip, p.clip_delta, p.dual_clip, p.eps};
  if (num_tokens > 0) {
    int device = 0, cus = 0;
    hipError_t e = hipGetDevice(&device);
    if (e == hipSuccess) e = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, device);
    if (e != hipSuccess) return fail(CTX_ERR_HIP, "device query: %s", hipGetErrorString(e));
    const int chunks = (vocab + kChunk - 1) / kChunk;
    const auto per_thread = [&](int threads) { return (chunks + threads - 1) / threads; };
    const bool own =
        num_tokens <= kOwnWeightTokens && num_seqs <= kOwnWeightTokens && per_thread(kOwnWeightThreads) <= kMaxChunksPerThread;
    if (!own)
      hipLaunchKernelGGL(opd_weight_kernel, dim3((unsigned)num_seqs), dim3(256), 0, s, mask, seq_starts, num_seqs,
                         p.eps, token_weight);
    const RowArgs a{static_cast<const uint16_t*>(logits), row_stride, vocab, num_tokens, tokens, old_logp, teacher_logp,
                    mask, token_weight, own ? seq_starts : nullptr, num_seqs, prm, token_logp, token_loss,
                    static_cast<uint16_t*>(grad_logits), grad_row_stride, cus, s};
    // The fewest threads whose registers hold a row: several workgroups per CU
    // are then in different passes over their rows, where one of 1024 threads
    // leaves the memory idle while it reduces.  Against 1024 threads: 12,944
    // columns 90 and 133 us, 32,000 130 and 153 (512 threads: 139), the loss alone
    // 61 and 69; 50,257 columns with 512 threads 229 and 242, 100,277 (25 chunks
    // per thread) 466 and 476, alone 179 and 193.  With 256 threads 20 to 26
    // chunks gain nothing: 45,000 columns 206 and (512 threads) 203.  Those are
    // batches of thousands of rows; with fewer rows than CUs, where a row is alone on
    // its CU, the fewer waves lose nothing either: against 1024 threads 16 rows of
    // 32,000 columns 9.3 and 10.8 us with the gradient, 100 of 50,257 14.0 and 14.8,
    // 256 of 100,277 29.9 and 29.3 (the loss alone 19.4 and 20.0).
    if (per_thread(256) <= kMaxChunksPerThread)
      launch_rows_of<256, 1, kMaxChunksPerThread>(per_thread(256), a);
    else if (per_thread(512) <= kMaxChunks512)
      launch_rows_of<512, kMaxChunksPerThread / 2 + 1, kMaxChunks512>(per_thread(512), a);
    else
      launch_rows_of<1024, kMaxChunks512 / 2 + 1, kMaxChunksPerThread>(per_thread(1024), a);
  }
  hipLaunchKernelGGL(opd_reduce_kernel, dim3(1), dim3(1024), 0, s, token_weight, token_loss, num_tokens, loss);
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(CTX_ERR_HIP, "kernel launch: %s", hipGetErrorString(e));
  return CTX_OK;
}

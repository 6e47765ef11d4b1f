// LM head + log-softmax + KL (Algorithm 1, WindowKL; Eq. sample-response).
//
// KL_t = sum_v P_v (log P_v - log Q_v) with P = softmax(a), Q = softmax(b),
// a = x_clean W^T, b = x_pert W^T.  With delta = a - b, A_t = logsumexp(a) and
// p_v = exp(a_v - A_t):
//   KL_t = sum_v p_v delta_v + log(sum_v p_v e^{-delta_v})
//        = sum_v p_v delta_v + log1p(S_t),  S_t = sum_v p_v (e^{-delta_v} - 1)
//        = sum_v p_v f(delta_v) - g(S_t),  f(x) = x + expm1(-x), g(y) = y - log1p(y).
// The fused kernel accumulates the first form (cheap: no clean max or sums
// beyond A_t, delta = 0 gives exactly 0); the unfused kernel uses the last form,
// whose terms are all non-negative (f and g by series near 0), as a cross-check.
//
// Fused path (bf16): logits never reach HBM.  The clean pass runs lm_lse once per
// batch (A_t).  lm_kl then computes, per 128-token x 128-vocab tile, the clean
// logits once and the logits of G perturbed passes against the same W tile, and
// folds each into per-lane (F, S) partials.  The tile is computed transposed
// (vocab rows = MFMA M, tokens = MFMA N), so a lane owns one token and all its
// vocab reductions are lane-local.  Vocab is split into chunks across
// workgroups; a fixed-order merge kernel combines the chunk partials.
// Unfused path (any dtype): KL over two materialised fp32 logit tensors.
#include <math.h>

#include "mfma_tile.h"

#include <type_traits>

namespace rk {

// f(x) = x + expm1(-x) = x^2/2 - x^3/6 + ...  (>= 0)
__device__ __forceinline__ float kl_f(float x) {
  if (fabsf(x) < 0.25f) {
    float p = x * (1.0f / 40320.0f) - (1.0f / 5040.0f);
    p = fmaf(p, x, 1.0f / 720.0f);
    p = fmaf(p, x, -1.0f / 120.0f);
    p = fmaf(p, x, 1.0f / 24.0f);
    p = fmaf(p, x, -1.0f / 6.0f);
    p = fmaf(p, x, 0.5f);
    return p * x * x;
  }
  return (expf(-fmaxf(x, -80.0f)) - 1.0f) + x;
}

// --------------------------------------------------------------------------- clean log-sum-exp
// The chunk merges: L lanes per row, lane j takes chunks j, j + L, ... in order, and a
// fixed butterfly adds the lanes (double).  16 lanes: one thread per row walking all chunks is
// a serial chain of loads (64 us for 250 chunks of 509 rows, 526 us for 1002 of 16 rows).
constexpr int kMergeLanes = 16, kMergeRows = 256 / kMergeLanes;

template <typename T, int L = kMergeLanes>
__device__ __forceinline__ T merge_sum(T v) {
#pragma unroll
  for (int m = L / 2; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// Folds n pairs per row into the row's running pair (none yet if `first`); `last`
// writes the log-sum-exp instead of the pair.
__global__ __launch_bounds__(256) void lse_merge_kernel(const float2* __restrict__ part, int n, int rows, bool first,
                                                        bool last, float2* run, float* __restrict__ lse) {
  const int r = blockIdx.x * kMergeRows + threadIdx.x / kMergeLanes, j = threadIdx.x % kMergeLanes;
  const int rr = min(r, rows - 1);
  const float2 prev = first ? make_float2(-INFINITY, 0.f) : run[rr];
  float M = prev.x;
  for (int c = j; c < n; c += kMergeLanes) M = fmaxf(M, part[(int64_t)c * rows + rr].x);
#pragma unroll
  for (int m = kMergeLanes / 2; m >= 1; m >>= 1) M = fmaxf(M, __shfl_xor(M, m, 64));
  double z = j == 0 && prev.y > 0.f ? (double)prev.y * exp((double)prev.x - (double)M) : 0.0;
  for (int c = j; c < n; c += kMergeLanes) {
    const float2 p = part[(int64_t)c * rows + rr];
    if (p.y > 0.f) z += (double)p.y * exp((double)p.x - (double)M);
  }
  z = merge_sum(z);
  if (j == 0 && r < rows) {
    if (last) lse[r] = (float)((double)M + log(z));
    else run[r] = make_float2(M, (float)z);
  }
}

// --------------------------------------------------------------------------- fused KL
// Per (token t, pass g): T1 = sum_v p_v delta_v and S = sum_v p_v (e^{-delta_v} - 1)
// with p_v = exp(a_v - A_t), so KL_t = T1 + log1p(S) (= sum p (a - b) - A + B
// without forming A and B).  delta = 0 gives exactly T1 = S = 0.  p is recomputed
// per pass instead of being held, which keeps the kernel at two waves per SIMD.
//
// A workgroup of 8 waves owns 256 tokens and a chunk of 128-wide vocab tiles.  For
// each vocab tile it computes the clean logit tile (kept in registers as `a`) and
// then the G perturbed tiles against the same W rows, folding each into the
// per-lane (T1, S) of its pass.  All the k-steps of all these tiles form one
// stream through a 3-stage LDS ring, so the copies run ahead across tile
// boundaries.  Wave w owns 64 tokens (64 (w / 2) .., the MFMA N side) and 64 vocab rows
// of the tile (half w % 2, M side): four fragments per four MFMAs, where 128 rows x 32
// tokens take five; its reductions over vocab stay in its lanes until the two halves
// meet at the end.  Against that, in calls on two cards: d = 4096, V = 32000, 32768 tokens, one
// pass 16.5-17.4 -> 16.0-16.9 ms; d = 768, 16384 tokens, 12 passes 11.4-11.6 -> 11.2-11.4 ms;
// V = 128256, 3000 tokens 7.68 -> 7.41.  Bound: the copies (48 KB per 1024 MFMA cycles) and their latency; the projections'
// alternating schedule, whose copies have two phases to land here instead of four, was slower
// (19.8 and 12.7 ms).
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kKlTok = 256;     // tokens per workgroup

// One 16-byte global->LDS copy per lane through a raw buffer descriptor over
// [base, base + nrec): lanes whose offset falls outside read zeros.
__device__ __forceinline__ void dma16_rows(const void* base, uint32_t nrec, uint32_t voff, int32_t soff,
                                           uint32_t lds) {
  const uint64_t b = (uint64_t)base;
  i32x4_t rsrc;
  rsrc[0] = __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)b);
  rsrc[1] = __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)(b >> 32));
  rsrc[2] = __builtin_amdgcn_readfirstlane((int32_t)nrec);
  rsrc[3] = 0x00020000;   // raw buffer, 32-bit data format
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               :
               : "v"(voff), "s"(rsrc), "s"(soff), "{m0}"(lds)
               : "memory");
}

template <int GMAX, int BK, int ST>
__global__ __launch_bounds__(512) void lm_kl_kernel(const bf16_t* __restrict__ Xc, const bf16_t* __restrict__ Xp,
                                                    int64_t pass_stride, int G, const bf16_t* __restrict__ W,
                                                    int rows, int d, int n_vt, int n_chunks,
                                                    const float* __restrict__ lse, float2* __restrict__ part) {
  constexpr int CH = BK / 8;                     // 16-byte chunks per k row of a stage
  constexpr int RPI = 64 / CH;                   // rows per wave copy instruction
  constexpr int WS = 128 * CH, XS = kKlTok * CH, SS = WS + XS;   // 16-byte slots per stage
  constexpr int NLW = WS / 512, NLX = XS / 512, NL = NLW + NLX;  // copies per thread and stage
  constexpr int NKS = BK / 16;                   // k-slices per k-step
  static_assert(WS % 512 == 0 && (ST - 2) * NL < 16 && ST * SS * 16 <= 160 * 1024, "stage geometry");
  __shared__ __attribute__((aligned(16))) v4u smem[ST * SS];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, l32 = lane & 31;
  const int vh = w & 1, tq = w >> 1;
  // Workgroup -> (token block, vocab chunk): the 32 workgroups an XCD runs at once
  // cover 4 token blocks x 8 chunks, so one pass's X rows (4 x 384 KB at d = 768)
  // and the W tiles in use (8 x 192 KB) stay in that XCD's L2 through the passes.
  int tb, chunk;
  xcd_tile((int)blockIdx.x, (rows + kKlTok - 1) / kKlTok, n_chunks, 4, &tb, &chunk);
  const int t0 = tb * kKlTok;
  const int vt0 = (int)((int64_t)chunk * n_vt / n_chunks), vt1 = (int)((int64_t)(chunk + 1) * n_vt / n_chunks);
  const int nk = d / BK;
  const int nsteps = (vt1 - vt0) * (G + 1) * nk;
  const int token = t0 + tq * 64 + l32;   // and token + 32
  float Ac[2];
#pragma unroll
  for (int tb2 = 0; tb2 < 2; ++tb2) {
    Ac[tb2] = lse[min(token + tb2 * 32, rows - 1)] * kLog2e;
    asm volatile("" : "+v"(Ac[tb2]));   // loaded before the copies start: no vector-memory wait inside the loop
  }

  // Copy geometry: in round j a wave instruction fills rows 8 RPI j + RPI w ..
  // + RPI - 1 of a tile, lane -> (row 8 RPI j + RPI w + lane / CH, swizzled chunk);
  // rounds advance by a multiple of 16 rows, which leaves the row swizzle unchanged.
  const int r0 = w * RPI + lane / CH;
  const uint32_t voff0 = (uint32_t)(r0 * d * 2 + (((lane % CH) ^ swz<CH>(r0)) * 16));
  const uint32_t round_bytes = (uint32_t)(8 * RPI * d * 2);
  const uint32_t x_nrec = (uint32_t)(max(0, min(rows - t0, kKlTok)) * d * 2);
  const uint32_t w_nrec = (uint32_t)(128 * d * 2);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) v4u*)smem;

  // producer position: the next k-step to copy
  int p_kt = 0, p_g = -1, p_vt = vt0, issued = 0;
  auto issue_one = [&](int j, int slot) {
    const uint32_t lds = lds0 + (uint32_t)(slot * SS * 16);
    const int32_t soff = p_kt * BK * 2;
    if (j < NLW) {
      dma16_rows(W + (int64_t)p_vt * 128 * d, w_nrec, voff0 + j * round_bytes, soff,
                 lds + (uint32_t)((j * 8 + w) * 64 * 16));
    } else {
      const int jx = j - NLW;
      const bf16_t* xb = (p_g < 0 ? Xc : Xp + (int64_t)p_g * pass_stride) + (int64_t)t0 * d;
      dma16_rows(xb, x_nrec, voff0 + jx * round_bytes, soff, lds + (uint32_t)((WS + (jx * 8 + w) * 64) * 16));
    }
  };
  auto advance = [&]() {
    ++issued;
    if (++p_kt == nk) {
      p_kt = 0;
      if (++p_g == G) { p_g = -1; ++p_vt; }
    }
  };
#pragma unroll
  for (int q = 0; q < ST - 1; ++q)
    if (issued < nsteps) {
#pragma unroll
      for (int j = 0; j < NL; ++j) issue_one(j, q);
      advance();
    }

  float T1[2][GMAX], S[2][GMAX];
#pragma unroll
  for (int g = 0; g < GMAX; ++g) { T1[0][g] = T1[1][g] = 0.f; S[0][g] = S[1][g] = 0.f; }
  f32x16_t a[4], b[4];   // block 2 x + y: vocabulary block x, token block y
  int kt = 0, g = -1, slot = 0, pslot = ST - 1;
  constexpr int PER = (NL + NKS - 1) / NKS;   // copies issued per k-slice
  // One k-step of the stream from LDS slot `slot`; COPY: it also issues its share
  // of the copies of the step ST - 1 ahead.  The copying steps and the last ST - 1
  // (which copy nothing) run as two loops, so each k-slice's reads, copies and
  // MFMAs form one basic block.
  int s = 0;
  auto kstep = [&](auto COPY) {
    constexpr bool CP = decltype(COPY)::value;
    if constexpr (CP) wait_vmem_le<(ST - 2) * NL>(); else wait_steps_ahead<NL, ST - 2>(issued - 1 - s);
    __syncthreads();   // k-step s is in LDS for every wave; the slot of s - 1 is free
    if (kt == 0) {
#pragma unroll
      for (int vb = 0; vb < 4; ++vb)
#pragma unroll
        for (int i = 0; i < 16; ++i) b[vb][i] = 0.f;
    }
    const v4u* Wt = smem + slot * SS;
    const v4u* Xt = Wt + WS;
    bf16x8_t wf[2][2], xf[2][2];
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      wf[0][q] = frag<CH>(Wt, vh * 64 + q * 32 + l32, 0, lane);
      xf[0][q] = frag<CH>(Xt, tq * 64 + q * 32 + l32, 0, lane);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
      const int c = ks & 1;
      if (ks + 1 < NKS) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          wf[c ^ 1][q] = frag<CH>(Wt, vh * 64 + q * 32 + l32, ks + 1, lane);
          xf[c ^ 1][q] = frag<CH>(Xt, tq * 64 + q * 32 + l32, ks + 1, lane);
        }
      }
      if constexpr (CP) {
#pragma unroll
        for (int j = ks * PER; j < (ks + 1) * PER; ++j)
          if (j < NL) issue_one(j, pslot);
      }
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int vb = 0; vb < 4; ++vb)
        b[vb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(wf[c][vb >> 1], xf[c][vb & 1], b[vb], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);
    }
    if constexpr (CP) {
      advance();
      pslot = pslot == ST - 1 ? 0 : pslot + 1;
    }
    slot = slot == ST - 1 ? 0 : slot + 1;
  };
  // after each k-step: a complete logit tile is kept (clean) or folded (a pass)
  auto tile_done = [&]() {
    if (++kt < nk) return;
    kt = 0;
    if (g < 0) {
#pragma unroll
      for (int vb = 0; vb < 4; ++vb) a[vb] = b[vb];
    } else {
      float t1[2] = {0.f, 0.f}, s2[2] = {0.f, 0.f};
#pragma unroll
      for (int vb = 0; vb < 4; ++vb)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float av = a[vb][i];
          const float p = __builtin_amdgcn_exp2f(fmaf(av, kLog2e, -Ac[vb & 1]));
          const float dl = av - b[vb][i];
          const float e = __builtin_amdgcn_exp2f(-dl * kLog2e) - 1.0f;
          t1[vb & 1] = fmaf(p, dl, t1[vb & 1]);
          s2[vb & 1] = fmaf(p, e, s2[vb & 1]);
        }
#pragma unroll
      for (int j = 0; j < GMAX; ++j)
        if (j == g) {
#pragma unroll
          for (int y = 0; y < 2; ++y) { T1[y][j] += t1[y]; S[y][j] += s2[y]; }
        }
    }
    if (++g == G) g = -1;
  };
  for (; s < nsteps - (ST - 1); ++s) {
    kstep(std::true_type{});
    tile_done();
  }
  for (; s < nsteps; ++s) {
    kstep(std::false_type{});
    tile_done();
  }
  // the half-waves hold other vocabulary rows of the same tokens, the waves vh = 0 and 1
  // the two halves of the tile: added in that order through LDS
  __syncthreads();
  float2* red = reinterpret_cast<float2*>(smem);
#pragma unroll
  for (int g2 = 0; g2 < GMAX; ++g2)
    if (g2 < G) {
#pragma unroll
      for (int y = 0; y < 2; ++y) {
        const float tx = T1[y][g2] + __shfl_xor(T1[y][g2], 32, 64), sx = S[y][g2] + __shfl_xor(S[y][g2], 32, 64);
        if (lane < 32) red[(g2 * 2 + vh) * kKlTok + tq * 64 + y * 32 + l32] = make_float2(tx, sx);
      }
    }
  __syncthreads();
  for (int q = tid; q < G * kKlTok; q += 512) {
    const int g2 = q / kKlTok, tk = q % kKlTok;
    if (t0 + tk < rows) {
      const float2 x = red[(g2 * 2) * kKlTok + tk], y = red[(g2 * 2 + 1) * kKlTok + tk];
      part[((int64_t)chunk * G + g2) * rows + t0 + tk] = make_float2(x.x + y.x, x.y + y.y);
    }
  }
}

// kl[g * rows + r] = sum_c T1 + log1p(sum_c S), fixed chunk order, double.
template <int L>
__global__ __launch_bounds__(256) void kl_merge_kernel(const float2* __restrict__ part, int n_chunks, int G, int rows,
                                                       float* __restrict__ kl) {
  const int r = blockIdx.x * (256 / L) + threadIdx.x / L, j = threadIdx.x % L, g = blockIdx.y;
  const int rr = min(r, rows - 1);
  double t1 = 0.0, s = 0.0;
  for (int c = j; c < n_chunks; c += L) {
    const float2 v = part[((int64_t)c * G + g) * rows + rr];
    t1 += v.x;
    s += v.y;
  }
  t1 = merge_sum<double, L>(t1);
  s = merge_sum<double, L>(s);
  if (j == 0 && r < rows) kl[(int64_t)g * rows + r] = (float)(t1 + log1p(s));
}

// chunks of the fused KL kernel: about 1024 workgroups of 256 tokens; chunk c
// takes vocab tiles [c n_vt / chunks, (c + 1) n_vt / chunks)
int lm_kl_chunks(int rows, int vocab) {
  const int n_vt = vocab / 128, n_tb = (rows + kKlTok - 1) / kKlTok;
  const int chunks = (1024 + n_tb - 1) / n_tb;
  return chunks > n_vt ? n_vt : (chunks < 1 ? 1 : chunks);
}

// The logits of the column blocks run on the projections' 8-wave tiles (EpiLse), their
// pairs are merged per row.  The scratch holds the pairs of `fit` column blocks; a
// larger vocabulary goes in several launches.  Bound: the matrix cores.  Against tiles
// of 128 tokens that waited on every k-step: 22636 rows, d = 4096, V = 32000 7.85 ms (0.76
// PFLOP/s) -> 4.5, 16384 rows, d = 768 1.03 -> 0.75 ms.
hipError_t launch_lm_lse(const bf16_t* x, const bf16_t* W, int rows, int d, int vocab, void* scratch,
                         size_t scratch_bytes, float2* run, float* lse, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const int cols = lse_tile_cols(vocab), n = vocab / cols;
  const int64_t fit = (int64_t)(scratch_bytes / ((size_t)rows * sizeof(float2)));
  if (fit < 1 || d % 64 != 0 || vocab % 128 != 0) return hipErrorInvalidValue;
  float2* part = (float2*)scratch;
  for (int b = 0; b < n;) {
    const int nb = (int)(fit < n - b ? fit : n - b);
    hipError_t e = launch_lse_tiles(x, W + (int64_t)b * cols * d, rows, d, nb * cols, cols, part, s);
    if (e != hipSuccess) return e;
    lse_merge_kernel<<<(rows + kMergeRows - 1) / kMergeRows, 256, 0, s>>>(part, nb, rows, b == 0, b + nb == n, run, lse);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    b += nb;
  }
  return hipSuccess;
}

hipError_t launch_lm_kl(const bf16_t* xc, const bf16_t* xp, int64_t pass_stride, int G, const bf16_t* W, int rows,
                        int d, int vocab, const float* lse, float2* part, float* kl, hipStream_t s) {
  if (rows <= 0 || G <= 0) return hipSuccess;
  if (d % 64 != 0 || vocab % 128 != 0 || (int64_t)kKlTok * d * 2 > 0x7fffffff) return hipErrorInvalidValue;
  const int chunks = lm_kl_chunks(rows, vocab);
  const int grid = (rows + kKlTok - 1) / kKlTok * chunks;
#ifndef RK_KL_BK
#define RK_KL_BK 64
#define RK_KL_ST 3
#endif
  constexpr int BK = RK_KL_BK, ST = RK_KL_ST;
  if (d % BK != 0) return hipErrorInvalidValue;
  if (G <= 4)
    lm_kl_kernel<4, BK, ST><<<grid, 512, 0, s>>>(xc, xp, pass_stride, G, W, rows, d, vocab / 128, chunks, lse, part);
  else if (G <= 8)
    lm_kl_kernel<8, BK, ST><<<grid, 512, 0, s>>>(xc, xp, pass_stride, G, W, rows, d, vocab / 128, chunks, lse, part);
  else if (G <= RK_MAX_GROUP)
    lm_kl_kernel<RK_MAX_GROUP, BK, ST><<<grid, 512, 0, s>>>(xc, xp, pass_stride, G, W, rows, d, vocab / 128, chunks, lse,
                                                             part);
  else
    return hipErrorInvalidValue;
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  // up to 16 chunks (many rows): a thread per row, whose loads are whole lines of neighbouring rows
  // (12 passes of 16384 rows, 16 chunks: 10 us against 19 with 16 lanes; 32768 rows, 8 chunks 8
  // against 36)
  if (chunks <= kMergeLanes)
    kl_merge_kernel<1><<<dim3((rows + 255) / 256, G), 256, 0, s>>>(part, chunks, G, rows, kl);
  else
    kl_merge_kernel<kMergeLanes><<<dim3((rows + kMergeRows - 1) / kMergeRows, G), 256, 0, s>>>(part, chunks, G, rows, kl);
  return hipGetLastError();
}

// --------------------------------------------------------------------------- unfused KL
// One workgroup (16 waves) per row scores every pass of the group: one sweep over
// the clean row gives its log-sum-exp A (running max and rescaled sum per thread,
// merged in a fixed order); when the row fits (vocab <= kKlLdsRow) it stays in
// LDS, so every pass reads only its own row from memory, once (p_v =
// 2^(a_v log2 e - A log2 e) with the hardware exp2, as in the fused kernel).  Per
// thread F and S are summed in fp32 over its vocab / 1024 entries, then across
// the workgroup in double, in a fixed order (lane tree, then waves in order).
constexpr int kKlThreads = 1024;
constexpr int kKlLdsRow = 36864;   // longest row kept in LDS (144 KB of fp32)

template <typename T>
__device__ __forceinline__ T wave_sum(T v) {
#pragma unroll
  for (int m = 32; m >= 1; m >>= 1) v += __shfl_xor(v, m, 64);
  return v;
}

// sum over the workgroup: every thread gets the same value
__device__ __forceinline__ double block_sum(double v, double* red) {
  const int w = threadIdx.x >> 6;
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[w] = v;
  __syncthreads();
  double r = 0.0;
  for (int i = 0; i < kKlThreads / 64; ++i) r += red[i];
  __syncthreads();
  return r;
}

// merge of two (max, sum of exp(x - max)) pairs
__device__ __forceinline__ void lse_merge(float& m, double& z, float m2, double z2) {
  if (m2 == -INFINITY) return;
  if (m == -INFINITY) { m = m2; z = z2; return; }
  const float mn = fmaxf(m, m2);
  z = z * (double)expf(m - mn) + z2 * (double)expf(m2 - mn);
  m = mn;
}

// one step of the running (max, sum) of a thread
__device__ __forceinline__ void lse_add(float& m, double& z, float x) {
  if (x > m) { z = z * (double)expf(m - x) + 1.0; m = x; }   // expf(-inf) = 0 on the first element
  else z += (double)expf(x - m);
}

__device__ __forceinline__ float block_lse(float m, double z, double* red, float* redm) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
#pragma unroll
  for (int d = 32; d >= 1; d >>= 1) lse_merge(m, z, __shfl_xor(m, d, 64), __shfl_xor(z, d, 64));
  if (lane == 0) { redm[w] = m; red[w] = z; }
  __syncthreads();
  float M = -INFINITY;
  double Z = 0.0;
  for (int i = 0; i < kKlThreads / 64; ++i) lse_merge(M, Z, redm[i], red[i]);
  __syncthreads();
  return (float)((double)M + log(Z));
}

// F and S terms of one entry: clean logit x, pass logit y
__device__ __forceinline__ void kl_terms(float x, float y, float Al, float& f1, float& s1) {
  const float p = __builtin_amdgcn_exp2f(fmaf(x, kLog2e, -Al));
  const float dl = x - y;
  const float f = kl_f(dl);
  f1 = fmaf(p, f, f1);
  s1 = fmaf(p, f - dl, s1);
}

// Rows are read as 16-byte groups of four entries (vocab is a multiple of 128),
// four groups per thread in flight.
template <bool IN_LDS>
__global__ __launch_bounds__(kKlThreads) void kl_logits_kernel(const float* __restrict__ lc,
                                                               const float* __restrict__ lp, int64_t pass_stride,
                                                               int G, int rows, int vocab, float* __restrict__ kl) {
  __shared__ float4 row[IN_LDS ? kKlLdsRow / 4 : 1];
  __shared__ double red[kKlThreads / 64];
  __shared__ float redm[kKlThreads / 64];
  constexpr int U = 4;
  const int r = blockIdx.x, t = threadIdx.x, n4 = vocab / 4;
  const float4* a = reinterpret_cast<const float4*>(lc + (int64_t)r * vocab);
  float m = -INFINITY;
  double z = 0.0;
  for (int q0 = t; q0 < n4; q0 += U * kKlThreads) {
    float4 x[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = q0 + u * kKlThreads;
      if (q < n4) x[u] = a[q];
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int q = q0 + u * kKlThreads;
      if (q < n4) {
        if (IN_LDS) row[q] = x[u];
        lse_add(m, z, x[u].x);
        lse_add(m, z, x[u].y);
        lse_add(m, z, x[u].z);
        lse_add(m, z, x[u].w);
      }
    }
  }
  const float A = block_lse(m, z, red, redm);   // its barriers also publish the LDS row
  const float Al = A * kLog2e;
  for (int g = 0; g < G; ++g) {
    const float4* b = reinterpret_cast<const float4*>(lp + (int64_t)g * pass_stride + (int64_t)r * vocab);
    float f1 = 0.f, s1 = 0.f;
    for (int q0 = t; q0 < n4; q0 += U * kKlThreads) {
      float4 y[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = q0 + u * kKlThreads;
        if (q < n4) y[u] = b[q];
      }
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int q = q0 + u * kKlThreads;
        if (q < n4) {
          const float4 x = IN_LDS ? row[q] : a[q];
          kl_terms(x.x, y[u].x, Al, f1, s1);
          kl_terms(x.y, y[u].y, Al, f1, s1);
          kl_terms(x.z, y[u].z, Al, f1, s1);
          kl_terms(x.w, y[u].w, Al, f1, s1);
        }
      }
    }
    const double F = block_sum((double)f1, red);
    const double S = block_sum((double)s1, red);
    if (t == 0) kl[(int64_t)g * rows + r] = (float)(F - (S - log1p(S)));
  }
}

hipError_t launch_kl_logits(const float* lc, const float* lp, int64_t pass_stride, int G, int rows, int vocab,
                            float* kl, hipStream_t s) {
  if (rows <= 0 || G <= 0) return hipSuccess;
  if (vocab % 4 != 0 || pass_stride % 4 != 0 || ((uintptr_t)lc | (uintptr_t)lp) % 16 != 0) return hipErrorInvalidValue;
  if (vocab <= kKlLdsRow)
    kl_logits_kernel<true><<<rows, kKlThreads, 0, s>>>(lc, lp, pass_stride, G, rows, vocab, kl);
  else
    kl_logits_kernel<false><<<rows, kKlThreads, 0, s>>>(lc, lp, pass_stride, G, rows, vocab, kl);
  return hipGetLastError();
}

}  // namespace rk

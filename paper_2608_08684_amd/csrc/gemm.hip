// Projection GEMMs of the decoder block, C[M, N] = A[M, K] * B[N, K]^T, with the
// block's elementwise work fused into the epilogue:
//   q|k|v projection  -> rotate-half rotary embedding on the q and k columns,
//   output / down     -> residual add into the fp32 stream,
//   gate|up           -> SwiGLU (silu(gate) * up), written as one [M, d_ff] tile,
//   LM head (unfused) -> plain fp32 logits.
// bf16 path: BM x BN block tiles (256 rows on 8 waves for many rows, 32 or 64 rows
// with a deep ring for few; pick_tile), v_mfma_f32_32x32x16_bf16,
// K-steps streamed global -> LDS by buffer loads into rings of LDS stages (see
// mfma_tile.h).  The finished tile leaves through LDS so the global accesses are
// whole rows; a rotary pair j, j + d_h/2 or a gate/up pair always lies inside one tile.
// fp32 path: the deep-ring tiles on v_mfma_f32_32x32x2_f32.
#include "mfma_tile.h"

#include <algorithm>
#include <cstdint>
#include <type_traits>

namespace rk {

// --------------------------------------------------------------------------- stores of 8 values
__device__ __forceinline__ void store8(float* p, const float* v) {
  reinterpret_cast<float4*>(p)[0] = make_float4(v[0], v[1], v[2], v[3]);
  reinterpret_cast<float4*>(p)[1] = make_float4(v[4], v[5], v[6], v[7]);
}

// 4 values to 4 consecutive elements (16 bytes fp32, 8 bytes bf16)
__device__ __forceinline__ void store4(float* p, float4 v) { *reinterpret_cast<float4*>(p) = v; }
__device__ __forceinline__ void store4(bf16_t* p, float4 v) {
  uint2 u;
  u.x = (uint32_t)f2bf(v.x) | ((uint32_t)f2bf(v.y) << 16);
  u.y = (uint32_t)f2bf(v.z) | ((uint32_t)f2bf(v.w) << 16);
  *reinterpret_cast<uint2*>(p) = u;
}
// 16 bytes between LDS and global memory (the LDS side 8-byte aligned for bf16 rows)
__device__ __forceinline__ void copy16(float* dst, const float* src) {
  *reinterpret_cast<float4*>(dst) = *reinterpret_cast<const float4*>(src);
}
__device__ __forceinline__ void copy16(bf16_t* dst, const bf16_t* src) {
  const uint2 a = reinterpret_cast<const uint2*>(src)[0], b = reinterpret_cast<const uint2*>(src)[1];
  *reinterpret_cast<uint4*>(dst) = make_uint4(a.x, a.y, b.x, b.y);
}

// --------------------------------------------------------------------------- epilogues
// The two runs of columns that a split-K tile holds: rows of B (b0 .., b1 ..) and
// the output columns they end in.
struct ColRuns {
  int b0, b1, o0, o1;
};
// Called per (row, 8 consecutive output columns starting at c0) with cs = the
// staged fp32 row of a BN-wide tile.  out_cols(BN) = output columns per tile.
template <typename O>
struct EpiRope {
  static constexpr int out_cols(int BN) { return BN; }
  static constexpr bool kPaired = true;
  static constexpr int pair_dist(int, int head_dim) { return head_dim / 2; }
  // tab[pos * head_dim/2 + j] = (cos, sin) of position pos, pair j; pos[row] = position of the row
  O* out; int64_t ldo; int rope_cols; int head_dim; const float2* tab; const int32_t* pos; int q_cols; float q_scale;
  // register form: x = tile columns tc..tc+3 (first half of a head), y = their
  // partners head_dim/2 further on; o0, o1 = the outputs at the same columns
  using stage_t = O;
  static constexpr int kOut = 2;
  template <int BN>
  __device__ __forceinline__ void pair(int row, int bn, int tc, float4 x, float4 y, float4& o0, float4& o1) const {
    const int gc = bn * BN + tc, half = head_dim >> 1;
    if (gc >= rope_cols) {  // value columns: no rotation
      o0 = x;
      o1 = y;
      return;
    }
    const float4* t4 = reinterpret_cast<const float4*>(tab + (int64_t)pos[row] * half + (gc & (head_dim - 1)));
    const float4 t01 = t4[0], t23 = t4[1];   // (cos, sin) of pairs j .. j+3
    const float sc = gc < q_cols ? q_scale : 1.0f;
    o0 = make_float4(fmaf(-y.x, t01.y, x.x * t01.x) * sc, fmaf(-y.y, t01.w, x.y * t01.z) * sc,
                     fmaf(-y.z, t23.y, x.z * t23.x) * sc, fmaf(-y.w, t23.w, x.w * t23.z) * sc);
    o1 = make_float4(fmaf(x.x, t01.y, y.x * t01.x) * sc, fmaf(x.y, t01.w, y.y * t01.z) * sc,
                     fmaf(x.z, t23.y, y.z * t23.x) * sc, fmaf(x.w, t23.w, y.w * t23.z) * sc);
  }
  // HB columns of the first half of a head and their partners (q|k|v width: whole heads)
  template <int HB>
  __device__ __forceinline__ ColRuns runs(int bn, int) const {
    const int half = head_dim >> 1, per = half / HB, c = bn / per * head_dim + bn % per * HB;
    return {c, c + half, c, c + half};
  }
  __device__ __forceinline__ void put(int row, const ColRuns& cr, int c, float4 x, float4 y) const {
    float4 p, q;
    pair<1>(row, 0, cr.o0 + c, x, y, p, q);
    store4(out + (int64_t)row * ldo + cr.o0 + c, p);
    store4(out + (int64_t)row * ldo + cr.o1 + c, q);
  }
};

struct EpiResidual {
  static constexpr int out_cols(int BN) { return BN; }
  static constexpr bool kPaired = false;
  float* out; int64_t ldo; const float* res; int64_t ldr;
  using stage_t = float;
  template <int HB>
  __device__ __forceinline__ ColRuns runs(int bn, int) const {
    return {bn * 2 * HB, bn * 2 * HB + HB, bn * 2 * HB, bn * 2 * HB + HB};
  }
  __device__ __forceinline__ void put(int row, const ColRuns& cr, int c, float4 x, float4 y) const {
    const float4 a = *reinterpret_cast<const float4*>(res + (int64_t)row * ldr + cr.o0 + c);
    const float4 b = *reinterpret_cast<const float4*>(res + (int64_t)row * ldr + cr.o1 + c);
    store4(out + (int64_t)row * ldo + cr.o0 + c, make_float4(a.x + x.x, a.y + x.y, a.z + x.z, a.w + x.w));
    store4(out + (int64_t)row * ldo + cr.o1 + c, make_float4(b.x + y.x, b.y + y.y, b.z + y.z, b.w + y.w));
  }
  template <int BN>
  __device__ void apply(int row, int bn, int c0, const float* cs) const {
    const int64_t n = (int64_t)bn * BN + c0;
    const float4* r4 = reinterpret_cast<const float4*>(res + (int64_t)row * ldr + n);
    const float4 a = r4[0], b = r4[1];
    float v[8] = {a.x + cs[c0 + 0], a.y + cs[c0 + 1], a.z + cs[c0 + 2], a.w + cs[c0 + 3],
                  b.x + cs[c0 + 4], b.y + cs[c0 + 5], b.z + cs[c0 + 6], b.w + cs[c0 + 7]};
    store8(out + (int64_t)row * ldo + n, v);
  }
};

template <typename O>
struct EpiSwiGLU {
  static constexpr int out_cols(int BN) { return BN / 2; }  // tile columns [0, BN/2) gate, [BN/2, BN) up
  static constexpr bool kPaired = true;
  static constexpr int pair_dist(int BN, int) { return BN / 2; }
  O* out; int64_t ldo;
  // silu(g) u, silu(g) = g / (1 + e^-g) with the hardware exp2 and reciprocal (about 1
  // ulp each)
  static __device__ __forceinline__ float silu_mul(float g, float u) {
    return g * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(-g * 1.4426950408889634f)) * u;
  }
  // register form: gate = tile columns tc..tc+3 (< BN/2), up = the same columns + BN/2;
  // o0 = output columns tc..tc+3 of this tile
  using stage_t = O;
  static constexpr int kOut = 1;
  template <int BN>
  __device__ __forceinline__ void pair(int, int, int, float4 g, float4 u, float4& o0, float4&) const {
    o0 = make_float4(silu_mul(g.x, u.x), silu_mul(g.y, u.y), silu_mul(g.z, u.z), silu_mul(g.w, u.w));
  }
  template <int HB>
  __device__ __forceinline__ ColRuns runs(int bn, int d_ff) const {
    return {bn * HB, d_ff + bn * HB, bn * HB, bn * HB};
  }
  __device__ __forceinline__ void put(int row, const ColRuns& cr, int c, float4 x, float4 y) const {
    store4(out + (int64_t)row * ldo + cr.o0 + c, make_float4(silu_mul(x.x, y.x), silu_mul(x.y, y.y),
                                                             silu_mul(x.z, y.z), silu_mul(x.w, y.w)));
  }
};

struct EpiStoreF32 {
  static constexpr int out_cols(int BN) { return BN; }
  static constexpr bool kPaired = false;
  float* out; int64_t ldo;
  float* out2;   // output of the second rows (GemmArgs.A2)
  using stage_t = float;
  template <int HB>
  __device__ __forceinline__ ColRuns runs(int bn, int) const {
    return {bn * 2 * HB, bn * 2 * HB + HB, bn * 2 * HB, bn * 2 * HB + HB};
  }
  __device__ __forceinline__ void put(int row, const ColRuns& cr, int c, float4 x, float4 y) const {
    store4(out + (int64_t)row * ldo + cr.o0 + c, x);
    store4(out + (int64_t)row * ldo + cr.o1 + c, y);
  }
  template <int BN>
  __device__ void apply(int row, int bn, int c0, const float* cs) const {
    store8(out + (int64_t)row * ldo + (int64_t)bn * BN + c0, cs + c0);
  }
};

// LM head, log-sum-exp only: the tile's logits never leave the registers.  Each row of
// the tile ends as one (max, sum of e^(x - max)) pair of its BN columns.
struct EpiLse {
  static constexpr int out_cols(int BN) { return BN; }
  static constexpr bool kPaired = false;
  using stage_t = float;
  float2* part;   // [column block][rows]
};

// --------------------------------------------------------------------------- bf16 MFMA kernels
// Wave layout.  PD: distance in tile columns between the two values an epilogue
// combines (a rotary pair, gate/up).  A wave with NI = 2 P column blocks (P = 1 or
// 2) holds P pairs: pair p is the blocks at c_p and c_p + PD, so each lane holds
// both values in registers.  With PD >= 32 P the first members are contiguous, c_p
// = wcol + 32 p with wcol = (wn / (PD / 32P)) * 2 PD + (wn % (PD / 32P)) * 32 P;
// with PD = 32 < 32 P the pairs are adjacent, c_p = wcol + 64 p, wcol = 128 wn.
// PD = 32 with P = 1 is the plain layout (wave wn: columns 64 wn ..).  Waves with
// three column blocks (NI = 3) take the plain layout, and paired epilogues then
// combine their values from the staged fp32 tile instead.
template <int BM_, int BN_, int BK_, int NWM_, int NWN_, int PD_, class E>
struct TileGeom {
  static constexpr int BM = BM_, BN = BN_, BK = BK_, NWM = NWM_, NWN = NWN_, PD = PD_;
  static constexpr int NW = NWM * NWN, NT = 64 * NW;
  static constexpr int WTM = BM / NWM, WTN = BN / NWN;   // wave tile
  static constexpr int MI = WTM / 32, NI = WTN / 32;     // 32x32 blocks per wave
  static constexpr int CH = BK / 8;                      // 16-byte chunks per tile row
  static constexpr int AS = BM * CH, BS = BN * CH;       // 16-byte slots of one stage's A and B tiles
  static constexpr bool REG_PAIR = E::kPaired && (NI == 2 || NI == 4);   // pairs combined in registers
  static constexpr int NP = NI == 3 ? 1 : NI / 2;                        // pairs per wave
  static constexpr int PSTEP = PD >= 32 * NP ? 32 : 2 * PD;              // column step between pairs
  static_assert(((NI == 2 || NI == 4) && BN % (2 * PD) == 0 && PD % 32 == 0 && (PD >= 32 * NP || PD == 32)) ||
                    (NI == 3 && PD == 32),
                "column blocks");
  // Epilogue staging: register-paired epilogues stage their outputs (type O), the
  // others the fp32 accumulators; rows padded by 4 elements.
  using SO = typename std::conditional<REG_PAIR, typename E::stage_t, float>::type;
  static constexpr int OC = REG_PAIR ? E::out_cols(BN) : BN, SP = OC + 4;
  static constexpr int ROW_BYTES = SP * (int)sizeof(SO);
  // fewest staging rounds (1, 2 or 4, each a whole number of every wave's 32-row
  // blocks) whose rows fit in `bytes`; 0 if none does
  static constexpr int rounds_for(int bytes) {
    return BM * ROW_BYTES <= bytes                        ? 1
           : (MI % 2 == 0 && BM / 2 * ROW_BYTES <= bytes) ? 2
           : (MI % 4 == 0 && BM / 4 * ROW_BYTES <= bytes) ? 4
                                                          : 0;
  }
  // copy instructions per thread and stage (A tile, then B tile or its gate and up halves)
  static constexpr int NA = BM * CH / (64 * NW), NB = BN * CH / (64 * NW), NL = NA + NB;
  static constexpr int NKS = BK / 16;   // k-slices per k-step
  static __device__ __forceinline__ int wave_col(int wn) {
    return NI == 3 ? wn * WTN
                   : (PD >= 32 * NP ? (wn / (PD / (32 * NP))) * (2 * PD) + (wn % (PD / (32 * NP))) * (32 * NP)
                                    : wn * WTN);
  }
  // tile column of column block ni (blocks ni < NP: first members, ni >= NP: partners)
  static __device__ __forceinline__ int colblk(int wcol, int ni) {
    return NI == 3 ? wcol + ni * 32 : wcol + (ni % NP) * PSTEP + (ni / NP) * PD;
  }
};

// Epilogue of one tile, staged in ROUNDS passes through the LDS at `stage`.  The
// MFMAs take B as the first operand, so acc[mi][ni] is the transposed 32x32 block:
// lane l holds row l % 32 and, in elements 4g..4g+3, the four consecutive columns
// 8 g + 4 (l / 32) .. +3 of the block.  Paired epilogues combine their two blocks
// in registers; the results go through LDS so the global accesses are whole
// rows.  The caller has freed the staging area (barrier) and must place a barrier
// before the area is written again.
template <class G, int ROUNDS, class E>
__device__ __forceinline__ void tile_epilogue(const f32x16_t (&acc)[G::MI][G::NI], v4u* stage, int m0, int bn, int M,
                                              const E& e, int wm, int wcol, int tid) {
  using SO = typename G::SO;
  constexpr int MI = G::MI, NI = G::NI, NP = G::NP, OC = G::OC, SP = G::SP, NT = G::NT, BN = G::BN;
  static_assert(ROUNDS >= 1 && MI % ROUNDS == 0, "staging rounds split each wave's rows evenly");
  const int lane = tid & 63, l32 = lane & 31;
  SO* Cs = reinterpret_cast<SO*>(stage);
  constexpr int WR = G::WTM / ROUNDS, MIR = MI / ROUNDS;   // rows per wave and round, blocks per round
#pragma unroll
  for (int h = 0; h < ROUNDS; ++h) {
    if (h) __syncthreads();   // the previous round has been written out
#pragma unroll
    for (int q = 0; q < MIR; ++q) {
      const int mi = h * MIR + q;
      const int row = m0 + wm * G::WTM + mi * 32 + l32;
      SO* cs = Cs + (wm * WR + q * 32 + l32) * SP;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int q4 = g * 8 + (lane >> 5) * 4;
        if constexpr (G::REG_PAIR) {
#pragma unroll
          for (int pp = 0; pp < NP; ++pp) {
            const int tc = G::colblk(wcol, pp) + q4;
            const f32x16_t& ax = acc[mi][pp];
            const f32x16_t& ay = acc[mi][pp + NP];
            const float4 x = make_float4(ax[4 * g], ax[4 * g + 1], ax[4 * g + 2], ax[4 * g + 3]);
            const float4 y = make_float4(ay[4 * g], ay[4 * g + 1], ay[4 * g + 2], ay[4 * g + 3]);
            float4 o0 = make_float4(0.f, 0.f, 0.f, 0.f), o1 = o0;
            if (row < M) e.template pair<BN>(row, bn, tc, x, y, o0, o1);
            store4(cs + tc, o0);   // SwiGLU: gate columns [0, PD) are the output columns
            if constexpr (E::kOut == 2) store4(cs + tc + G::PD, o1);
          }
        } else {
#pragma unroll
          for (int ni = 0; ni < NI; ++ni)
            store4(cs + G::colblk(wcol, ni) + q4, make_float4(acc[mi][ni][4 * g], acc[mi][ni][4 * g + 1],
                                                              acc[mi][ni][4 * g + 2], acc[mi][ni][4 * g + 3]));
        }
      }
    }
    __syncthreads();
    // staged row r is tile row (r / WR) * WTM + h * WR + r % WR
    if constexpr (G::REG_PAIR) {
      constexpr int CE = 16 / (int)sizeof(SO), CPR = OC / CE, RPP = NT / CPR;
      const int c = (tid % CPR) * CE;
      if (tid < RPP * CPR)
        for (int r = tid / CPR; r < G::BM / ROUNDS; r += RPP) {
          const int row = m0 + (r / WR) * G::WTM + h * WR + r % WR;
          if (row < M) copy16(e.out + (int64_t)row * e.ldo + (int64_t)bn * OC + c, Cs + r * SP + c);
        }
    } else {
      constexpr int TPR = E::out_cols(BN) / 8, RPP = NT / TPR;
      const int c0 = (tid % TPR) * 8;
      if (tid < RPP * TPR)
        for (int r = tid / TPR; r < G::BM / ROUNDS; r += RPP) {
          const int row = m0 + (r / WR) * G::WTM + h * WR + r % WR;
          if (row < M) e.template apply<BN>(row, bn, c0, Cs + r * SP);
        }
    }
  }
}

// (max, sum of e^(x - max)) of every row of the tile over its columns; red: the ring's
// LDS, freed by the caller.
template <class G>
__device__ __forceinline__ void tile_lse(const f32x16_t (&acc)[G::MI][G::NI], float2* red, int m0, int bn, int M,
                                         float2* part, int wm, int wn, int tid) {
  constexpr float kLog2e = 1.4426950408889634f;
  constexpr int NWN = G::NWN;
  const int lane = tid & 63;
#pragma unroll
  for (int mi = 0; mi < G::MI; ++mi) {
    float m = -INFINITY;
#pragma unroll
    for (int ni = 0; ni < G::NI; ++ni)
#pragma unroll
      for (int i = 0; i < 16; ++i) m = fmaxf(m, acc[mi][ni][i]);
    m = fmaxf(m, __shfl_xor(m, 32, 64));   // the half-waves hold the same rows
    // from the exact difference: e^(x - m) as 2^(x log2 e - m log2 e) would carry the rounding of m log2 e,
    // as large as that of the whole log-sum-exp to fp32
    float z = 0.f;
#pragma unroll
    for (int ni = 0; ni < G::NI; ++ni)
#pragma unroll
      for (int i = 0; i < 16; ++i) z += __builtin_amdgcn_exp2f((acc[mi][ni][i] - m) * kLog2e);
    z += __shfl_xor(z, 32, 64);
    if (lane < 32) red[(wm * G::WTM + mi * 32 + lane) * NWN + wn] = make_float2(m, z);
  }
  __syncthreads();
  for (int r = tid; r < G::BM; r += G::NT) {
    if (m0 + r >= M) break;
    float m = red[r * NWN].x, z = 0.f;
#pragma unroll
    for (int q = 1; q < NWN; ++q) m = fmaxf(m, red[r * NWN + q].x);
#pragma unroll
    for (int q = 0; q < NWN; ++q) z += red[r * NWN + q].y * __builtin_amdgcn_exp2f((red[r * NWN + q].x - m) * kLog2e);
    part[(int64_t)bn * M + m0 + r] = make_float2(m, z);
  }
}

// --------------------------------------------------------------------------- alternating 8-wave kernel
// The 8-wave tiles in two groups of four waves, one wave of each group per SIMD,
// half a phase apart: while one group runs the MFMAs of half a k-step, the other
// reads its next fragments from LDS and issues copies, and a workgroup barrier
// closes every phase.  Without the alternation both waves of a SIMD read, wait
// and multiply at the same times, and the matrix cores idle through the reads.
//
// A k-step of a wave is P0 M0 P1 M1:
//   P0  reads every B fragment and the A fragments of the wave's first MI / 2 row
//       blocks; copies the second half of A of k-step t + 1;
//   M0  multiplies them;
//   P1  reads the A fragments of the other row blocks (into the same registers);
//       copies B and the first half of A of k-step t + 2;
//   M1  multiplies them.
// Ring of two stages.  A phase ends with its LDS reads done, so after the barrier
// that follows P0 (P1) of the later group a region may be written again: B and the
// first half of A of stage t from P1(t) on, the second half from P0(t + 1) on.
// Each P phase ends by waiting for what the next P phase reads, which was issued
// four phases before; the copies issued in between stay in flight.
// Bound: the matrix cores through the reads, waits and barriers of the other
// group.  Against both groups in step, kernel times inside calls on two cards (the cards
// differ by 5%): d = 4096, 32768 rows: gate|up 1252-1319 -> 1373-1439 TFLOP/s, down (K = 14336)
// 1160-1192 -> 1330-1389, q|k|v 1136-1178 -> 1222-1284, output 1108-1139 -> 1193-1237;
// d = 768, 65536 rows: down (K = 3072) 910-926 -> 1050-1083, gate|up 1019-1082 -> 1051-1095,
// q|k|v 790-833 -> 819-852, output 569-586 -> 589-603; bitwise the same.
// Spreading the reads evenly over P0 and P1 (a quarter of B one phase early) and
// leaving out the priorities measured the same within 1%.
template <int BM, int BN, int NWM, int NWN, int PD, class E, bool SWIGLU>
__global__ __launch_bounds__(512) void gemm_alt_kernel(const bf16_t* __restrict__ A, int64_t lda,
                                                       const bf16_t* __restrict__ B, int64_t ldb, int M, int K,
                                                       int d_ff, int n_bn, int group_m, E e) {
  using G = TileGeom<BM, BN, kBK, NWM, NWN, PD, E>;
  constexpr int MI = G::MI, NI = G::NI, MH = MI / 2, CH = G::CH, HW = G::WTM / 2;
  constexpr int PIPE = 2 * (G::AS + G::BS);
  constexpr int ROUNDS = G::rounds_for(160 * 1024);
  static_assert(ROUNDS > 0, "staging");
  constexpr int STG = G::BM / ROUNDS * G::ROW_BYTES / 16;
  static_assert(PIPE * 16 <= 160 * 1024 && STG * 16 <= 160 * 1024, "LDS");
  static_assert(!SWIGLU || G::REG_PAIR, "SwiGLU tiles pair gate and up in registers");
  static_assert(NWM * NWN == 8 && NWM % 2 == 0 && MI % 2 == 0 && HW % 16 == 0 && CH == 8, "two groups of four waves");
  constexpr int NAH = G::NA / 2, NB = G::NB;   // copies per wave: half of A, all of B
  static_assert(G::NA % 2 == 0 && (!SWIGLU || NB % 2 == 0), "copies split evenly");
  __shared__ __attribute__((aligned(16))) v4u smem[PIPE > STG ? PIPE : STG];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w / NWN, wn = w % NWN;
  const int wcol = G::wave_col(wn);
  int bm_, bn;
  xcd_tile((int)blockIdx.x, (M + BM - 1) / BM, n_bn, group_m, &bm_, &bn);
  const int m0 = bm_ * BM;
  RowGroupSrc sa, sb, su;
  sa.init(A + (int64_t)m0 * lda, lda, w, lane);
  if (SWIGLU) {
    sb.init(B + (int64_t)bn * (BN / 2) * ldb, ldb, w, lane);
    su.init(B + ((int64_t)d_ff + (int64_t)bn * (BN / 2)) * ldb, ldb, w, lane);
  } else {
    sb.init(B + (int64_t)bn * BN * ldb, ldb, w, lane);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) v4u*)smem;
  auto copy_b = [&](int kt, int st) {
    const uint32_t Bs = lds0 + (2 * G::AS + st * G::BS) * 16;
#pragma unroll
    for (int j = 0; j < NB; ++j) {
      const int g = j * 8 + w;   // 8-row group of the B tile
      if (SWIGLU && j >= NB / 2) su.load_at(kt, g - NB / 2 * 8, Bs + g * 1024);
      else sb.load_at(kt, g, Bs + g * 1024);
    }
  };
  // half h of A: of each wave's WTM rows the h-th HW
  auto copy_a = [&](int kt, int st, int h) {
    const uint32_t As = lds0 + st * G::AS * 16;
#pragma unroll
    for (int j = 0; j < NAH; ++j) {
      const int q = j * 8 + w;
      const int g = q / (HW / 8) * (G::WTM / 8) + h * (HW / 8) + q % (HW / 8);
      sa.load_at(kt, g, As + g * 1024);
    }
  };

  f32x16_t acc[MI][NI];
#pragma unroll
  for (int mi = 0; mi < MI; ++mi)
#pragma unroll
    for (int ni = 0; ni < NI; ++ni)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[mi][ni][i] = 0.f;
  bf16x8_t af[MH][G::NKS], bfr[NI][G::NKS];
  auto read_b = [&](int st) {
    const v4u* Bt = smem + 2 * G::AS + st * G::BS;
#pragma unroll
    for (int ks = 0; ks < G::NKS; ++ks)
#pragma unroll
      for (int ni = 0; ni < NI; ++ni) bfr[ni][ks] = frag<CH>(Bt, G::colblk(wcol, ni) + l32, ks, lane);
  };
  auto read_a = [&](int st, int h) {
    const v4u* At = smem + st * G::AS;
#pragma unroll
    for (int ks = 0; ks < G::NKS; ++ks)
#pragma unroll
      for (int mi = 0; mi < MH; ++mi) af[mi][ks] = frag<CH>(At, wm * G::WTM + h * HW + mi * 32 + l32, ks, lane);
  };
  auto mma = [&](auto H) {
    constexpr int h = decltype(H)::value;
    __builtin_amdgcn_s_setprio(1);
#pragma unroll
    for (int ks = 0; ks < G::NKS; ++ks)
#pragma unroll
      for (int mi = 0; mi < MH; ++mi)
#pragma unroll
        for (int ni = 0; ni < NI; ++ni)
          acc[h * MH + mi][ni] =
              __builtin_amdgcn_mfma_f32_32x32x16_bf16(bfr[ni][ks], af[mi][ks], acc[h * MH + mi][ni], 0, 0, 0);
    __builtin_amdgcn_s_setprio(0);
  };
  typedef std::integral_constant<int, 0> H0;
  typedef std::integral_constant<int, 1> H1;

  const int nk = K / kBK;
  copy_b(0, 0);
  copy_a(0, 0, 0);
  copy_a(0, 0, 1);
  if (nk > 1) {
    copy_b(1, 1);
    copy_a(1, 1, 0);
    wait_vmem_le<NB + 2 * NAH>();   // B and the first half of A of k-step 0
  } else {
    wait_vmem();
  }
  phase_barrier();
  if (w >= 4) phase_barrier();   // the second group runs one phase behind
  int t = 0;
  for (; t < nk - 2; ++t) {
    const int st = t & 1;
    read_b(st);
    read_a(st, 0);
    copy_a(t + 1, st ^ 1, 1);
    wait_reads_and_copies<NB + 2 * NAH>();   // second half of A of k-step t
    phase_barrier();
    mma(H0{});
    phase_barrier();
    read_a(st, 1);
    copy_b(t + 2, st);
    copy_a(t + 2, st, 0);
    wait_reads_and_copies<NB + 2 * NAH>();   // B and the first half of A of k-step t + 1
    phase_barrier();
    mma(H1{});
    phase_barrier();
  }
  for (; t < nk; ++t) {   // the last two k-steps: at most one half of A is left to copy
    const int st = t & 1;
    read_b(st);
    read_a(st, 0);
    if (t + 1 < nk) {
      copy_a(t + 1, st ^ 1, 1);
      wait_reads_and_copies<NB + 2 * NAH>();
    } else {
      wait_reads_and_copies<0>();
    }
    phase_barrier();
    mma(H0{});
    phase_barrier();
    read_a(st, 1);
    wait_reads_and_copies<NAH>();
    phase_barrier();
    mma(H1{});
    phase_barrier();
  }
  if (w < 4) phase_barrier();
  __syncthreads();   // the staging area overlaps the ring
  if constexpr (std::is_same<E, EpiLse>::value)
    tile_lse<G>(acc, reinterpret_cast<float2*>(smem), m0, bn, M, e.part, wm, wn, tid);
  else
    tile_epilogue<G, ROUNDS>(acc, smem, m0, bn, M, e, wm, wcol, tid);
}

// --------------------------------------------------------------------------- deep-ring kernel
// Few rows: BM x BN tiles of one 32x32 block per multiplying wave, streamed through a
// ring of S stages.  NW waves copy; the first (BM / 32) (BN / 32) of them multiply,
// reading the fragments of k-step i + 1 under the MFMAs of k-step i.  K is summed in
// order, as in the 8-wave tiles, so an element does not depend on the number of
// rows or the tile.  The tile's columns are two runs of BN / 2 that the epilogue
// pairs: gate and up, the two halves of a head, or (no pairs) neighbours.
// Bound: the copies' latency (about 1.1 us) against the bytes in flight per CU, and
// the serial MFMA chain of a k-step; so small tiles to fill the grid, rings of 72-144
// KB, copies spread over waves that do not multiply, and no wait on the reads just
// issued.  Against 128x128 tiles with 32 KB in flight, inside calls (weights from memory):
// 16 rows, N = 4096, K = 14336 230 -> 37 us, N = 6144, K = 4096 67 -> 15; 300 rows, N = 4096,
// K = 14336 222 -> 106; 509 rows, N = 768, K = 3072 51 -> 13; 2048 rows, the same weights, 52 ->
// 25.  Splitting K between wave groups gained at most 4 us at 16 rows and made sums depend
// on the tile.
// fp32 (T = float): the same with 128-byte k-steps of 32 values and
// v_mfma_f32_32x32x2_f32; each k-step is summed from zero and then added, so the
// rounding error grows with K / 32 + 32 terms, not K.  Bound: the matrix cores (a k-step
// is 1024 cycles per block, 157 TFLOP/s over the chip).  Against the vector units
// with a 64x128 tile: 1801 rows, N = 32000, K = 768 73 -> 99 TFLOP/s, N = 768, K = 3072 27 -> 71;
// 256 rows, N = 256, K = 1024 105 -> 22 us.
template <typename T, int BM, int BN, int NW, int S, class E>
__global__ __launch_bounds__(64 * NW) void gemm_ring_kernel(const T* __restrict__ A, const T* __restrict__ A2,
                                                            int64_t lda, const T* __restrict__ B, int64_t ldb, int M,
                                                            int K, int d_ff, int n_bn, E e) {
  constexpr bool F32 = sizeof(T) == 4;
  constexpr int WN = BN < 32 ? 1 : BN / 32;          // 32-column blocks (a 16-wide tile fills half of one)
  constexpr int GW = (BM / 32) * WN, NT = 64 * NW, HB = BN / 2, CH = 8;
  constexpr int SA = BM * CH, SS = (BM + BN) * CH;   // 16-byte slots of a stage's A tile, of a stage
  constexpr int PAD = (WN * 32 - BN) * CH;           // read past a 16-wide tile's last stage, never used
  constexpr int NG = (BM + BN) / 8, NL = NG / NW;    // 8-row groups of a stage, copies per wave
  static_assert(NW >= GW && NG % NW == 0 && S >= 3 && (S - 2) * NL < 64, "copies split evenly");
  constexpr int SP = BN + 4;                         // staged row in floats
  static_assert((S * SS + PAD) * 16 <= 160 * 1024 && BM * SP * 4 <= S * SS * 16, "LDS");
  __shared__ __attribute__((aligned(16))) v4u smem[S * SS + PAD];
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = w / WN, wn = w % WN;
  int bm_, bn;
  const int n_bm = (M + BM - 1) / BM, n_m = A2 ? 2 * n_bm : n_bm;
  xcd_tile((int)blockIdx.x, n_m, n_bn, n_m, &bm_, &bn);   // the row tiles of one column block together
  if constexpr (std::is_same<E, EpiStoreF32>::value) {
    if (bm_ >= n_bm) {   // the second rows
      bm_ -= n_bm;
      A = A2;
      e.out = e.out2;
    }
  }
  const int m0 = bm_ * BM;
  const ColRuns cr = e.template runs<HB>(bn, d_ff);
  // this wave's 8-row groups: from A, or from either run of B
  RowGroupSrc src[NL];
#pragma unroll
  for (int j = 0; j < NL; ++j) {
    const int g = j * NW + w, rb = (g - BM / 8) * 8;
    const bool isa = g < BM / 8;
    const T* p = isa ? A + (int64_t)(m0 + g * 8) * lda
                     : B + (int64_t)(rb < HB ? cr.b0 + rb : cr.b1 + rb - HB) * ldb;
    src[j].init(reinterpret_cast<const bf16_t*>(p), (isa ? lda : ldb) * (sizeof(T) / 2), g, lane);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) v4u*)smem + w * 1024;
  const int nk = K / (128 / (int)sizeof(T));
  auto issue = [&](int kt, int slot) {
#pragma unroll
    for (int j = 0; j < NL; ++j) src[j].load_at(kt, 0, lds0 + slot * (SS * 16) + j * (NW * 1024));
  };
  f32x16_t acc;
#pragma unroll
  for (int i = 0; i < 16; ++i) acc[i] = 0.f;
  bf16x8_t af[2][4], bf[2][4];
#pragma unroll
  for (int p = 0; p < S - 1; ++p)
    if (p < nk) issue(p, p);
  wait_steps_ahead<NL, S - 2>(min(nk, S - 1) - 1);
  phase_barrier();
  // Step i: stage i + 1 is in LDS for every wave and k-step i in registers; the slot
  // of i - 1 is free (its fragments were multiplied before the barrier).  The
  // copying steps and the last S - 1 run as separate loops.
  auto run = [&](auto MUL) {
    constexpr bool mul = decltype(MUL)::value;
    int nxt = S - 1, rd = 0, i = 0;
    auto read = [&](int h) {
      const v4u* At = smem + rd * SS;
      const v4u* Bt = At + SA;
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) {
        bf[h][ks] = frag<CH>(Bt, wn * 32 + l32, ks, lane);
        af[h][ks] = frag<CH>(At, wm * 32 + l32, ks, lane);
      }
      rd = rd == S - 1 ? 0 : rd + 1;
      __builtin_amdgcn_sched_barrier(0);
    };
    auto mma = [&](int h) {
      if constexpr (F32) {
        f32x16_t part;
#pragma unroll
        for (int q = 0; q < 16; ++q) part[q] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const f32x4_t x = __builtin_bit_cast(f32x4_t, af[h][ks]), y = __builtin_bit_cast(f32x4_t, bf[h][ks]);
#pragma unroll
          for (int q = 0; q < 4; ++q) part = __builtin_amdgcn_mfma_f32_32x32x2f32(y[q], x[q], part, 0, 0, 0);
        }
#pragma unroll
        for (int q = 0; q < 16; ++q) acc[q] += part[q];
      } else {
#pragma unroll
        for (int ks = 0; ks < 4; ++ks)
          acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[h][ks], af[h][ks], acc, 0, 0, 0);
      }
    };
    auto step = [&](int h) {
      wait_vmem_le<(S - 3) * NL>();
      phase_barrier();
      if constexpr (mul) read(h ^ 1);
      issue(i + S - 1, nxt);
      if constexpr (mul) mma(h);
      nxt = nxt == S - 1 ? 0 : nxt + 1;
      ++i;
    };
    auto last = [&](int h) {   // no more stages to copy
      wait_steps_ahead<NL, S - 3>(nk - 2 - i);
      phase_barrier();
      if constexpr (mul) {
        read(h ^ 1);
        mma(h);
      }
      ++i;
    };
    if constexpr (mul) read(0);
    while (i + S < nk) {
      step(0);
      step(1);
    }
    int h = 0;   // parity of i (even here)
    if (i + S - 1 < nk) {
      step(0);
      h = 1;
    }
    if (h) {
      while (i < nk - 2) {
        last(1);
        last(0);
      }
    } else {
      while (i < nk - 2) {
        last(0);
        last(1);
      }
    }
    if (i < nk - 1) {
      if (h) last(1); else last(0);
      h ^= 1;
    }
    if constexpr (mul) {
      if (h) mma(1); else mma(0);
    }
  };
  if (NW == GW || w < GW) run(std::true_type{});
  else run(std::false_type{});
  __syncthreads();   // the staging area overlaps the ring
  float* Cs = reinterpret_cast<float*>(smem);
  if (NW == GW || w < GW) {
    // acc is the transposed block: lane l holds row l % 32, columns 8 g + 4 (l / 32) .. + 3
    float* cs = Cs + (wm * 32 + l32) * SP + wn * 32 + (lane >> 5) * 4;
#pragma unroll
    for (int g = 0; g < (BN < 32 ? BN / 8 : 4); ++g)
      store4(cs + g * 8, make_float4(acc[4 * g], acc[4 * g + 1], acc[4 * g + 2], acc[4 * g + 3]));
  }
  __syncthreads();
  constexpr int QPR = HB / 4;   // four-column units per run
  for (int u = tid; u < BM * QPR; u += NT) {
    const int r = u / QPR, c = u % QPR * 4, row = m0 + r;
    if (row >= M) break;   // u grows with r
    const float* cs = Cs + r * SP + c;
    e.put(row, cr, c, *reinterpret_cast<const float4*>(cs), *reinterpret_cast<const float4*>(cs + HB));
  }
}

// --------------------------------------------------------------------------- dispatch
static int cu_count() {
  static int n = 0;
  if (n == 0) {
    int dev = 0, v = 0;
    if (hipGetDevice(&dev) == hipSuccess && hipDeviceGetAttribute(&v, hipDeviceAttributeMultiprocessorCount, dev) == hipSuccess && v > 0)
      n = v;
    else
      n = 256;
  }
  return n;
}

// The tile with the least estimated time.  A round of workgroups takes fixed + k-steps x step
// microseconds, a ring tile's last round by how many tiles are left in it, an 8-wave tile's every
// round alike; the constants are fits to launches inside clean passes (weights and rows from
// memory), M = 17 .. 24576 at the widths 768 and 4096.  There the tile taken is the best at nine
// sizes of ten and within 25% of it at all, and its estimate within 6% at half of them, 20% at
// nine of ten and 40% at all.  Fits to single launches, and every round of ring tiles counted as
// full, put 32x64 and 64x64 where rounds of them wait on L2: 768 rows, N = 4096, K = 14336
// 257 us (now 199), 512 rows, N = 6144, K = 4096 75.7 (60), 4096 rows, N = 768, K = 3072 57 (43),
// 4608 rows, N = K = 768 23 (20); two LM heads of 48 rows, N = 128256, K = 4096 400 (272).
// The 8-wave tiles: 256x256 fixed 11.5, step 0.89 with a few tiles, up to 1.25 with every
// CU busy; 256x192 11 and 0.78; 256x128 7.5 and 0.61.  The ring tiles: 64x128 2.5, 0.3 and up to
// 0.39; two workgroups per CU, step with one and with both: 64x64 1.4, 0.28, 0.52; 32x64
// 0.65, 0.22, 0.36; 32x32 1.2, 0.15, 0.24.  No tile beats the time the weights take from
// memory (4.9 TB/s); among equals the one listed first is taken.
enum class Tile { k32x16, k32x64, k32x32, k64x64, k64x128, k256x128, k256x192, k256x256 };

static Tile pick_tile(const GemmArgs& a, bool swiglu) {
  const int64_t ncu = cu_count(), nk = a.K / kBK;
  const double mem = (double)a.N * a.K * 2 / 4.9e6;   // microseconds
  double best = 1e30;
  Tile tile = Tile::k32x64;
  auto offer = [&](Tile t, double us) {
    if (us < mem) us = mem;
    if (us < best) { best = us; tile = t; }
  };
  auto tiles = [&](int bm, int bn) { return ((a.M + bm - 1) / bm) * (int64_t)(a.N / bn); };
  // ring tiles, `per` workgroups per CU: full rounds, and one of the tiles left
  auto ring = [&](Tile t, int bm, int bn, int per, double fixed, double alone, double full) {
    const int64_t n = tiles(bm, bn) * (a.A2 ? 2 : 1), nf = n / (per * ncu), rem = n % (per * ncu);
    const double step = per == 2 ? (rem <= ncu ? alone : full) : alone + (full - alone) * ((double)rem / ncu);
    offer(t, nf * (fixed + nk * full) + (rem ? fixed + nk * step : 0.0));
  };
  auto one = [&](Tile t, int bm, int bn, double fixed, double step, double load) {
    const int64_t n = tiles(bm, bn);
    const double rounds = (double)((n + ncu - 1) / ncu);
    const double us = rounds * (fixed + nk * step * (1.0 + load * (n < ncu ? (double)n / ncu : 1.0)));
    offer(t, a.A2 ? 2.0 * std::max(us, mem) : us);   // a launch for each set of rows
  };
  // 32x16 tiles put twice the CUs on weights that stream from memory; worth it where K is
  // long enough for their 24-stage ring (16 rows, N = 4096, cold weights: K = 14336 41.6 -> 37
  // us, K = 4096 12.6 -> 14.2; a decode step of 8 blocks 1.41 -> 1.38 ms)
  if (nk >= 128 && tiles(32, 16) <= ncu) one(Tile::k32x16, 32, 16, 3.0, 0.1, 0.0);
  ring(Tile::k32x64, 32, 64, 2, 0.65, 0.22, 0.36);
  ring(Tile::k32x32, 32, 32, 2, 1.2, 0.15, 0.24);
  ring(Tile::k64x64, 64, 64, 2, 1.4, 0.28, 0.52);
  // a 64-wide run does not fit a 64-wide head's half
  if (a.epi != Epi::kStoreRope || a.head_dim == 128) ring(Tile::k64x128, 64, 128, 1, 2.5, 0.3, 0.39);
  one(Tile::k256x128, 256, 128, 7.5, 0.61, 0.4);
  // 192-wide tiles have three column blocks per wave: no pairs in registers
  if (!swiglu && a.epi != Epi::kStoreRope && a.N % 192 == 0) one(Tile::k256x192, 256, 192, 11.0, 0.78, 0.4);
  if (swiglu ? a.d_ff % 128 == 0 : a.N % 256 == 0) one(Tile::k256x256, 256, 256, 11.5, 0.89, 0.4);
  return tile;
}

template <typename T, int BM, int BN, int NW, int S, class E>
static hipError_t go_ring(const GemmArgs& a, const E& e, hipStream_t s) {
  const int nbn = a.N / BN;
  gemm_ring_kernel<T, BM, BN, NW, S, E><<<(a.M + BM - 1) / BM * nbn * (a.A2 ? 2 : 1), 64 * NW, 0, s>>>(
      (const T*)a.A, (const T*)a.A2, a.lda, (const T*)a.B, a.ldb, a.M, a.K, a.d_ff, nbn, e);
  return hipGetLastError();
}

template <int BM, int BN, int NWM, int NWN, int PD, class E, bool SWIGLU>
static void go_pd(const GemmArgs& a, const E& e, hipStream_t s) {
  const int nbn = SWIGLU ? a.d_ff / (BN / 2) : a.N / BN;
  const int nbm = (a.M + BM - 1) / BM;
  // tile-rows per L2 group: 4 for the long-K projections of the 8B-scale models
  // (1-2% faster than 8 on q|k|v, output and down at 32768 rows, equal on
  // gate|up), 8 for short K
  const int group_m = a.K >= 4096 ? 4 : 8;
  gemm_alt_kernel<BM, BN, NWM, NWN, PD, E, SWIGLU><<<nbm * nbn, 512, 0, s>>>(
      (const bf16_t*)a.A, a.lda, (const bf16_t*)a.B, a.ldb, a.M, a.K, a.d_ff, nbn, group_m, e);
}

// the pair distance each epilogue needs (plain layout when it pairs nothing)
template <int BM, int BN, class E, bool SWIGLU, int NWM, int NWN>
static hipError_t go_bf16(const GemmArgs& a, const E& e, hipStream_t s) {
  if constexpr (!E::kPaired) {
    go_pd<BM, BN, NWM, NWN, 32, E, SWIGLU>(a, e, s);
  } else if constexpr (BN % 128 != 0) {
    return hipErrorInvalidValue;   // three column blocks per wave: no pairs in registers
  } else if constexpr (SWIGLU) {
    go_pd<BM, BN, NWM, NWN, BN / 2, E, SWIGLU>(a, e, s);
  } else {
    if (a.head_dim == 64) go_pd<BM, BN, NWM, NWN, 32, E, SWIGLU>(a, e, s);
    else if (a.head_dim == 128) go_pd<BM, BN, NWM, NWN, 64, E, SWIGLU>(a, e, s);
    else return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

template <typename T, class E, bool SWIGLU>
static hipError_t go(const GemmArgs& a, const E& e, hipStream_t s) {
  if constexpr (sizeof(T) == 2) {
    if (E::kPaired && !SWIGLU && a.head_dim != 64 && a.head_dim != 128) return hipErrorInvalidValue;
    const Tile tile = pick_tile(a, SWIGLU);
    // the 8-wave tiles take the second rows (the LM head only) in a launch of their own
    if (a.A2 && tile != Tile::k32x16 && tile != Tile::k32x64 && tile != Tile::k32x32 && tile != Tile::k64x64 && tile != Tile::k64x128) {
      if constexpr (std::is_same<E, EpiStoreF32>::value) {
        GemmArgs one = a;
        one.A2 = nullptr;
        hipError_t r = go<T, E, SWIGLU>(one, e, s);
        if (r != hipSuccess) return r;
        one.A = a.A2;
        return go<T, E, SWIGLU>(one, EpiStoreF32{e.out2, e.ldo, nullptr}, s);
      }
      return hipErrorInvalidValue;
    }
    switch (tile) {
      case Tile::k32x16: return go_ring<bf16_t, 32, 16, 6, 24>(a, e, s);
      case Tile::k32x64: return go_ring<bf16_t, 32, 64, 4, 6>(a, e, s);
      case Tile::k32x32: return go_ring<bf16_t, 32, 32, 4, 9>(a, e, s);
      case Tile::k64x64: return go_ring<bf16_t, 64, 64, 4, 5>(a, e, s);
      case Tile::k64x128: return go_ring<bf16_t, 64, 128, 8, 6>(a, e, s);
      case Tile::k256x128: return go_bf16<256, 128, E, SWIGLU, 4, 2>(a, e, s);
      case Tile::k256x192: return go_bf16<256, 192, E, SWIGLU, 4, 2>(a, e, s);
      case Tile::k256x256: return go_bf16<256, 256, E, SWIGLU, 2, 4>(a, e, s);
    }
    return hipErrorInvalidValue;
  } else {
    // 64x64 tiles keep the four matrix cores of a CU busy; with fewer tiles than CUs,
    // 32x32 tiles spread the work over four times as many (a block's serial chain is
    // the same).  The two runs of a 32-wide head's halves are 16 columns.
    const int64_t n64 = (int64_t)((a.M + 63) / 64) * (a.N / 64);
    if (n64 < cu_count()) return go_ring<float, 32, 32, 4, 9>(a, e, s);
    if constexpr (E::kPaired && !SWIGLU)
      if (a.head_dim < 64) return go_ring<float, 64, 32, 4, 6>(a, e, s);
    return go_ring<float, 64, 64, 4, 5>(a, e, s);
  }
}

int lse_tile_cols(int vocab) { return vocab % 256 == 0 ? 256 : 128; }

hipError_t launch_lse_tiles(const bf16_t* x, const bf16_t* W, int rows, int d, int cols, int tile_cols, float2* part,
                            hipStream_t s) {
  GemmArgs a{};
  a.A = x; a.lda = d; a.B = W; a.ldb = d; a.M = rows; a.N = cols; a.K = d;
  const EpiLse e{part};
  if (tile_cols == 256) go_pd<256, 256, 2, 4, 32, EpiLse, false>(a, e, s);
  else go_pd<256, 128, 4, 2, 32, EpiLse, false>(a, e, s);
  return hipGetLastError();
}

template <typename T>
static hipError_t gemm_of(const GemmArgs& a, hipStream_t s) {
  switch (a.epi) {
    case Epi::kStoreRope:
      return go<T, EpiRope<T>, false>(
          a, {(T*)a.out, a.ldo, a.rope_cols, a.head_dim, a.rope_tab, a.rope_pos, a.q_cols, a.q_scale}, s);
    case Epi::kResidual: return go<T, EpiResidual, false>(a, {(float*)a.out, a.ldo, a.res, a.ldr}, s);
    case Epi::kSwiGLU: return go<T, EpiSwiGLU<T>, true>(a, {(T*)a.out, a.ldo}, s);
    case Epi::kStoreF32: return go<T, EpiStoreF32, false>(a, {(float*)a.out, a.ldo, (float*)a.out2}, s);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm(const GemmArgs& a, bool bf16, hipStream_t s) {
  if (a.M <= 0) return hipSuccess;
  if (a.A2 && a.epi != Epi::kStoreF32) return hipErrorInvalidValue;
  return bf16 ? gemm_of<bf16_t>(a, s) : gemm_of<float>(a, s);
}

}  // namespace rk

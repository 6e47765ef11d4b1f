// Causal grouped-query attention of one decoder block (Section 4.1), reading the
// (possibly perturbed) Values of the q|k|v buffer: o = softmax(q k^T / sqrt(d_h)) v
// with key u visible from query t iff u <= t; query head hq reads KV head
// hq / (H / H_kv).  With the Keys fixed the attention weights of the perturbed
// layer equal the clean ones (Section 4.3); only the aggregated Values change.
//
// bf16 kernel (flash attention, fp32 online softmax in base 2):
//   * the queries arrive pre-multiplied by log2(e) / sqrt(d_h) (the q|k|v
//     projection's epilogue does it before rounding), so a score is already
//     the exponent of 2;
//   * one workgroup = 4 waves (d_h 64) or 8 waves (d_h 128) x 32 queries of one
//     head; it runs a pair of query blocks (nqb - 1 - x, then x) so all pairs of
//     a sequence cost the same, longest sequences first (one block per workgroup
//     when the rows sit behind a cached prefix, which every block reads in full);
//   * 64-key tiles of K and V go global -> LDS by buffer_load ... lds (no
//     staging registers; rows past the sequence read as zero) through a
//     ring of 2-3 stages;
//   * S^T = K Q^T on v_mfma_f32_32x32x16_bf16 with the accumulator started at
//     -m (the running max), so each lane owns one query column and exp2 is
//     applied to the MFMA result directly; m is raised lazily (only when a
//     tile's max exceeds it by 2^8), with one exchange with the partner
//     half-wave (v_permlane32_swap); the two 32-key halves of a tile run as two
//     interleaved accumulator chains;
//   * O^T = V^T P^T: P^T is the lane's own S^T registers rounded to bf16, and
//     the V^T operand comes from the row-major V tile through ds_read_b64_tr_b16
//     in the same key order; the softmax denominator is summed from the rounded
//     P with v_dot2_f32_bf16, so the weights applied to V sum to one;
//   * masks only on diagonal / ragged tiles;
//   * the K fragment reads of a tile are issued up to six ahead of the MFMAs
//     that consume them (scheduling groups), not each right before its use.
// fp32 kernel: 32 queries of a head per workgroup on fp32 MFMAs.
#include <math.h>

#include <algorithm>

#include "rk_internal.h"

namespace rk {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4_t __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef short s16x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t v2u __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) void lds_void;
typedef __attribute__((address_space(3))) s16x4_t lds_s16x4;

// A score may exceed the running max by up to 2^kLazy before m is raised.
constexpr float kLazy = 8.0f;

typedef int32_t i32x4_t __attribute__((ext_vector_type(4)));

// 16-byte global -> LDS copy of one wave (lane l lands at lds_base + 16 l); rows
// past the descriptor's range read as zero.  Issued as inline assembly so the
// compiler does not tie later LDS reads of the other buffer to it: the caller
// waits with s_waitcnt vmcnt(0) and a barrier before the data is read.
__device__ __forceinline__ void dma16(i32x4_t rsrc, uint32_t lds_base, uint32_t voff, int32_t soff) {
  asm volatile("s_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
               :
               : "v"(voff), "s"(rsrc), "s"(soff), "{m0}"(lds_base)
               : "memory");
}

// s_waitcnt vmcnt(0) (gfx9 encoding: expcnt and lgkmcnt fields at their maximum)
// as a builtin, so the compiler also knows that its own earlier loads are done
__device__ __forceinline__ void wait_vm0() { __builtin_amdgcn_s_waitcnt(0x0F70); }
// s_waitcnt vmcnt(N), N < 16
template <int N>
__device__ __forceinline__ void wait_vm() {
  static_assert(N >= 0 && N < 16, "vmcnt field");
  __builtin_amdgcn_s_waitcnt(0x0F70 | N);
}

// s_waitcnt vmcnt(N), N < 64
template <int N>
__device__ __forceinline__ void wait_vmem_few() {
  static_assert(N >= 0 && N < 64, "vmcnt field");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// 16-byte chunk swizzles that keep the LDS reads free of bank conflicts (64
// banks of 4 bytes): the K tile is read as 16 rows x one chunk per quarter-wave,
// the V tile by ds_read_b64_tr_b16 as 4 rows x 4 chunks per half-wave.
template <int DH>
__device__ __forceinline__ int k_swz(int row) { return DH == 128 ? (row & 15) : ((row >> 1) & 7); }
template <int DH>
__device__ __forceinline__ int v_swz(int row) { return DH == 128 ? ((row & 3) << 2) : (((row >> 1) & 1) << 2); }

// max / sum of a lane's value and that of lane l ^ 32 (the other half-wave):
// v_permlane32_swap with both operands x hands lanes 0-31 the upper half's x and
// lanes 32-63 the lower half's, each keeping its own in the other result.
__device__ __forceinline__ float max_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float sum_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// Workgroup shape per head size.  d_h = 64: 4 waves (128 queries), a three-stage
// K/V ring (prefetch two tiles ahead), three workgroups per CU.  d_h = 128: 8 waves
// (256 queries) share one two-stage ring, one workgroup per CU (two waves per SIMD
// either way; the wider group halves the copies per query).
template <int DH>
struct AttnTraits {
  static constexpr int kWaves = DH == 64 ? 4 : 8;
  static constexpr int kStages = DH == 64 ? 3 : 2;
  static constexpr int kMinBlocks = DH == 64 ? 3 : 1;
};

template <int DH, bool PREFIX>
__global__ __launch_bounds__(64 * AttnTraits<DH>::kWaves, AttnTraits<DH>::kMinBlocks) void attn_bf16_kernel(const bf16_t* __restrict__ qkv, int64_t ldq,
                                                        bf16_t* __restrict__ out, int64_t ldo, SeqTable st,
                                                        AttnWork wk, int H, int Hkv, int n_items, int paired,
                                                        KvPrefix pk) {
  constexpr int NW = AttnTraits<DH>::kWaves;
  constexpr int BQ = 32 * NW, BKV = 64;
  constexpr int CH = DH / 8;                // 16-byte chunks per row
  constexpr int NKS = DH / 16;              // k-steps of S^T
  constexpr int NDB = DH / 32;              // 32-row blocks of O^T
  constexpr int SLOTS = BKV * CH;           // 16-byte slots per tile
  constexpr int NLD = SLOTS / (64 * NW);    // DMA instructions per thread, per tile and matrix
  constexpr int ROWB = DH * 2;              // bytes per tile row
  constexpr int S = AttnTraits<DH>::kStages;
  __shared__ __attribute__((aligned(16))) v4u Ks[S][SLOTS];
  __shared__ __attribute__((aligned(16))) v4u Vs[S][SLOTS];

  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

  // ---- work item: XCD-grouped so the query heads of one KV head share an L2
  const int grp = H / Hkv;
  int t_item;
  {
    const int g = blockIdx.x, x = g & 7, n = g >> 3;
    t_item = (n / grp) * (8 * grp) + x * grp + n % grp;
  }
  if (t_item >= n_items) return;
  const int item = t_item / H, hq = t_item - item * H, hk = hq / grp;
  int j = 0;
  {
    int lo = 0, hi = st.n - 1;
    while (lo < hi) {
      const int mid = (lo + hi + 1) >> 1;
      if (wk.cum[mid] <= item) lo = mid; else hi = mid - 1;
    }
    j = lo;
  }
  const int k = wk.order[j], x = item - wk.cum[j];
  const int row0 = st.off[k], T = st.off[k + 1] - row0;
  const int nqb = (T + BQ - 1) / BQ;

  // buffer descriptor over this sequence's rows (raw, stride 0): reads past row T - 1 return zero
  auto make_rsrc = [](const bf16_t* base_ptr, int64_t bytes) {
    i32x4_t r;
    const uint64_t base = (uint64_t)base_ptr;
    r[0] = __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)base);
    r[1] = __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)(base >> 32));
    r[2] = __builtin_amdgcn_readfirstlane((int32_t)bytes);
    r[3] = 0x00020000;
    return r;
  };
  const i32x4_t rsrc = make_rsrc(qkv + (int64_t)row0 * ldq, (int64_t)T * ldq * 2);
  const int kcol = (H + hk) * DH, vcol = (H + Hkv + hk) * DH;
  uint32_t koff[NLD], voff[NLD];
#pragma unroll
  for (int i = 0; i < NLD; ++i) {
    const int slot = (i * NW + w) * 64 + lane, r = slot / CH, ph = slot % CH;
    koff[i] = (uint32_t)(r * ldq * 2 + (kcol + (ph ^ k_swz<DH>(r)) * 8) * 2);
    voff[i] = (uint32_t)(r * ldq * 2 + (vcol + (ph ^ v_swz<DH>(r)) * 8) * 2);
  }
  // cached prefix of this sequence (PREFIX): rows k * P .. k * P + P - 1 of the K and V caches
  const int P = PREFIX ? pk.P : 0;
  i32x4_t rk_p = rsrc, rv_p = rsrc;
  uint32_t koff_p[PREFIX ? NLD : 1], voff_p[PREFIX ? NLD : 1];
  int64_t ldv_p = pk.ldv;
  if constexpr (PREFIX) {
    // the prefix of this sequence (of sequence k % n_seq when several passes share a launch)
    const int ps = pk.n_seq > 0 ? k % pk.n_seq : k;
    const bool alt = pk.n_seq > 0 && k / pk.n_seq == pk.alt_pass;
    const bf16_t* vb = alt ? pk.v_alt : pk.v;
    ldv_p = alt ? pk.ldv_alt : pk.ldv;
    rk_p = make_rsrc(pk.k + (int64_t)ps * P * pk.ldk, (int64_t)P * pk.ldk * 2);
    rv_p = make_rsrc(vb + (int64_t)ps * P * ldv_p, (int64_t)P * ldv_p * 2);
#pragma unroll
    for (int i = 0; i < NLD; ++i) {
      const int slot = (i * NW + w) * 64 + lane, r = slot / CH, ph = slot % CH;
      koff_p[i] = (uint32_t)(r * pk.ldk * 2 + (hk * DH + (ph ^ k_swz<DH>(r)) * 8) * 2);
      voff_p[i] = (uint32_t)(r * ldv_p * 2 + (hk * DH + (ph ^ v_swz<DH>(r)) * 8) * 2);
    }
  }
  const int n_pre = (P + BKV - 1) / BKV;   // prefix tiles, visited before the window's own
  const uint32_t ks_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) v4u*)&Ks[0][0];
  const uint32_t vs_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) v4u*)&Vs[0][0];
  // tile t: prefix tile t (t < n_pre), else the sequence's own tile t - n_pre
  auto issue = [&](int t, int b) {
    if (PREFIX && t < n_pre) {
      const int sk = __builtin_amdgcn_readfirstlane(t * BKV * (int)pk.ldk * 2);
      const int sv = __builtin_amdgcn_readfirstlane(t * BKV * (int)ldv_p * 2);
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const uint32_t o = (uint32_t)((b * SLOTS + (i * NW + w) * 64) * 16);
        dma16(rk_p, __builtin_amdgcn_readfirstlane(ks_lds + o), koff_p[i], sk);
        dma16(rv_p, __builtin_amdgcn_readfirstlane(vs_lds + o), voff_p[i], sv);
      }
    } else {
      const int so = __builtin_amdgcn_readfirstlane((t - n_pre) * BKV * (int)ldq * 2);
#pragma unroll
      for (int i = 0; i < NLD; ++i) {
        const uint32_t o = (uint32_t)((b * SLOTS + (i * NW + w) * 64) * 16);
        dma16(rsrc, __builtin_amdgcn_readfirstlane(ks_lds + o), koff[i], so);
        dma16(rsrc, __builtin_amdgcn_readfirstlane(vs_lds + o), voff[i], so);
      }
    }
  };

  // per-lane LDS byte offsets of the K fragments (row l32 of a 32-row block, chunk 2 ks + hf)
  // and of the V^T fragments (ds_read_b64_tr_b16: lane (G, jj) reads row 4 (G / 2) + jj / 4
  // of an 8-row group, columns db * 32 + 16 (G % 2) + 4 (jj % 4))
  int kfo[NKS];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) kfo[ks] = l32 * ROWB + (((2 * ks + hf) ^ k_swz<DH>(l32)) << 4);
  int vfo[NDB];
  {
    const int G = lane >> 4, jj = lane & 15, r = 4 * (G >> 1) + (jj >> 2);
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      const int ch = 4 * db + 2 * (G & 1) + ((jj & 3) >> 1);
      vfo[db] = r * ROWB + ((ch ^ v_swz<DH>(r)) << 4) + (jj & 1) * 8;
    }
  }

  const bf16x2_t ones = {(__bf16)1.0f, (__bf16)1.0f};
  // causal rows: the pair (nqb - 1 - x, x); behind a cached prefix every q-block
  // costs about the same, so one q-block per item; also where the pairs leave CUs idle
  const int n_blocks = PREFIX || !paired ? 1 : ((x == nqb - 1 - x) ? 1 : 2);
  for (int bi = 0; bi < n_blocks; ++bi) {
    const int qb = (PREFIX || bi == 0) ? nqb - 1 - x : x;
    const int q0 = qb * BQ;
    const int my_q = min(q0 + w * 32 + l32, T - 1);   // rows past T duplicate row T - 1
    bf16x8_t qf[NKS];
    {
      const bf16_t* qp = qkv + (int64_t)(row0 + my_q) * ldq + (int64_t)hq * DH + hf * 8;
#pragma unroll
      for (int ks = 0; ks < NKS; ++ks)
        qf[ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const v4u*>(qp + ks * 16));
    }
    const int kv_end = min(T, q0 + BQ);
    const int n_tiles = n_pre + (kv_end + BKV - 1) / BKV;
    const int wave_qmin = q0 + w * 32, wave_qmax = wave_qmin + 31;

    f32x16_t o[NDB], negm;
#pragma unroll
    for (int i = 0; i < 16; ++i) negm[i] = 0.f;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
    float l_run = 0.f;

    wait_vm0();   // the query fragments are in registers before the ring starts
#pragma unroll
    for (int p = 0; p < S - 1; ++p)
      if (p < n_tiles) issue(p, p);
    int buf = 0, nbuf = S - 1;   // ring slots of tile t and of tile t + S - 1
    for (int t = 0; t < n_tiles; ++t) {
      const bool pre = PREFIX && t < n_pre;
      const int k0 = (pre ? t : t - n_pre) * BKV;   // first key of the tile within its segment
      // tile t has landed once at most the S - 2 later tiles are in flight
      if (t + S - 2 < n_tiles) wait_vm<(S - 2) * 2 * NLD>(); else wait_vm0();
      __syncthreads();   // ... for every wave; and tile t - 1's slot is free again
      if (t + S - 1 < n_tiles) issue(t + S - 1, nbuf);
      if (pre || k0 <= wave_qmax) {
        const char* kt = reinterpret_cast<const char*>(Ks[buf]);
        f32x16_t s[2] = {negm, negm};
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks)
#pragma unroll
          for (int rb = 0; rb < 2; ++rb) {
            const bf16x8_t a = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const v4u*>(kt + rb * 32 * ROWB + kfo[ks]));
            s[rb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[ks], s[rb], 0, 0, 0);
          }
        {
          // schedule: the K fragment reads run up to three MFMA pairs ahead of their
          // MFMAs (the compiler's own order waits on each read right before its use)
          constexpr int AHEAD = NKS >= 8 ? 6 : 4, N = 2 * NKS;
          __builtin_amdgcn_sched_group_barrier(0x100, AHEAD, 0);   // LDS reads
#pragma unroll
          for (int p = 0; p < (N - AHEAD) / 2; ++p) {
            __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);     // MFMAs
            __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
          }
          __builtin_amdgcn_sched_group_barrier(0x008, AHEAD, 0);
        }
        // masks only where a key can exceed the query or the segment (wave-uniform test);
        // every cached prefix key precedes every query of the sequence's own rows
        if (pre ? (k0 + BKV > P) : (k0 + BKV - 1 > wave_qmin || k0 + BKV > T)) {
          const int qlim = pre ? P - 1 : my_q, klim = pre ? P : T;
#pragma unroll
          for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
              const int key = k0 + rb * 32 + (i >> 2) * 8 + hf * 4 + (i & 3);
              if (key > qlim || key >= klim) s[rb][i] = -INFINITY;
            }
        }
        float mx = fmaxf(s[0][0], s[0][1]);
#pragma unroll
        for (int i = 2; i < 16; i += 2) mx = fmaxf(mx, fmaxf(s[0][i], s[0][i + 1]));
#pragma unroll
        for (int i = 0; i < 16; i += 2) mx = fmaxf(mx, fmaxf(s[1][i], s[1][i + 1]));
        mx = max_halves(mx);
        if (t == 0 || __any(mx > kLazy)) {
          // raise the running max: by the tile max on the first tile, else where it grew past 2^kLazy
          const float dm = (t == 0 || mx > kLazy) ? mx : 0.f;
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            s[0][i] -= dm;
            s[1][i] -= dm;
            negm[i] -= dm;
          }
          if (t != 0) {
            const float corr = __builtin_amdgcn_exp2f(-dm);
            l_run *= corr;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
              for (int i = 0; i < 16; ++i) o[db][i] *= corr;
          }
        }
        const char* vt = reinterpret_cast<const char*>(Vs[buf]);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
          for (int ss = 0; ss < 2; ++ss) {
            bf16x8_t pb;
#pragma unroll
            for (int e = 0; e < 8; ++e) pb[e] = (__bf16)__builtin_amdgcn_exp2f(s[rb][8 * ss + e]);
#pragma unroll
            for (int e = 0; e < 8; e += 2) {
              const bf16x2_t pr = {pb[e], pb[e + 1]};
              l_run = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, l_run, false);
            }
            // k-slot hf * 8 + e of this MFMA is key rb*32 + ss*16 + 8 (e / 4) + 4 hf + e % 4
            const int kr = (rb * 32 + ss * 16) * ROWB;
#pragma unroll
            for (int db = 0; db < NDB; ++db) {
              const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vt + kr + vfo[db]));
              const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vt + kr + 8 * ROWB + vfo[db]));
              const v4u vv = {__builtin_bit_cast(v2u, lo)[0], __builtin_bit_cast(v2u, lo)[1],
                              __builtin_bit_cast(v2u, hi)[0], __builtin_bit_cast(v2u, hi)[1]};
              o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, vv), pb, o[db], 0, 0, 0);
            }
          }
      }
      buf = buf == S - 1 ? 0 : buf + 1;
      nbuf = nbuf == S - 1 ? 0 : nbuf + 1;
    }
    __syncthreads();   // the next q-block refills the ring

    const float l = sum_halves(l_run);
    const float inv = 1.0f / l;
    const int q_out = q0 + w * 32 + l32;
    if (q_out < T) {
      bf16_t* op = out + (int64_t)(row0 + q_out) * ldo + (int64_t)hq * DH;
#pragma unroll
      for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          bf16x4_t u;
#pragma unroll
          for (int e = 0; e < 4; ++e) u[e] = (__bf16)(o[db][g * 4 + e] * inv);
          *reinterpret_cast<bf16x4_t*>(op + db * 32 + g * 8 + hf * 4) = u;
        }
    }
  }
}

// Few query rows behind a cached prefix (a decode step, short windows): the rows of
// all query heads of one KV head together are at most 32 columns, so one workgroup =
// 4 waves serves a (sequence, KV head).  The waves share out the 32-key blocks (wave w
// takes blocks w, w + 4, ...: the prefix's, then the rows' own), each through a two-stage
// ring of its own (it alone writes and reads it, so it waits on its own copies and
// needs no barrier), with its own running maximum, denominator and output; merged through
// LDS in wave order.  A prefix restricted to retained positions is read in place: the
// positions lie in LDS and give each copied row its offset.
// Bound: latency of the copies and of a block's chain; 128 KB of copies in flight per CU.
// With one workgroup of 8 waves per query head, of whose 256 query columns one was
// used, 16 sequences, 32 / 8 heads of 128, 300 to 510 keys: 49 us and 12 us for gathering
// them; now 11 to 15 in all.
constexpr int kFewRows = 32, kFewPos = 4096;

template <int DH>
__global__ __launch_bounds__(256) void attn_few_kernel(const bf16_t* __restrict__ qkv, int64_t ldq,
                                                       bf16_t* __restrict__ out, int64_t ldo, SeqTable st, int H,
                                                       int Hkv, KvPrefix pk) {
  constexpr int CH = DH / 8, NKS = DH / 16, NDB = DH / 32, ROWB = DH * 2, SP = DH + 4;
  constexpr int SLOTS = 32 * CH, NI = SLOTS / 64, RPI = 64 / CH;   // copies per block and matrix, rows per copy
  // per wave: two stages of K and V blocks; the outputs of the waves at the end
  __shared__ __attribute__((aligned(16))) v4u ring[4][2][2][SLOTS];
  __shared__ float sm[4][32], sl[4][32];
  __shared__ int32_t spos[kFewPos];
  static_assert(4 * 32 * SP * 4 <= (int)sizeof(ring), "merge area");
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int k = blockIdx.x / Hkv, hk = blockIdx.x - k * Hkv, grp = H / Hkv;
  const int row0 = st.off[k], T = st.off[k + 1] - row0;
  if (T <= 0 || (int64_t)T * grp > kFewRows) return;   // the whole workgroup: such a sequence is attn_bf16_kernel's
  const int ps = pk.n_seq > 0 ? k % pk.n_seq : k;
  const bool alt = pk.n_seq > 0 && k / pk.n_seq == pk.alt_pass;
  const int P = pk.P, PR = pk.pos ? pk.full_P : P;   // keys, cached rows per sequence
  if (pk.pos) {
    const int32_t* pp = pk.pos + (int64_t)ps * pk.pos_stride + (int64_t)hk * P;
    for (int j = tid; j < P; j += 256) spos[j] = min(max(pp[j], 0), PR - 1);
    __syncthreads();
  }
  const int64_t ldv = alt ? pk.ldv_alt : pk.ldv;
  auto make_rsrc = [](const bf16_t* base_ptr, int64_t bytes) {
    i32x4_t r;
    const uint64_t base = (uint64_t)base_ptr;
    r[0] = __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)base);
    r[1] = __builtin_amdgcn_readfirstlane((int32_t)(uint32_t)(base >> 32));
    r[2] = __builtin_amdgcn_readfirstlane((int32_t)bytes);
    r[3] = 0x00020000;
    return r;
  };
  const i32x4_t rk_p = make_rsrc(pk.k + (int64_t)ps * PR * pk.ldk, (int64_t)PR * pk.ldk * 2);
  const i32x4_t rv_p = make_rsrc((alt ? pk.v_alt : pk.v) + (int64_t)ps * PR * ldv, (int64_t)PR * ldv * 2);
  const i32x4_t rsrc = make_rsrc(qkv + (int64_t)row0 * ldq, (int64_t)T * ldq * 2);
  const uint32_t lds_k = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) v4u*)&ring[w][0][0][0];
  const int n_pre = (P + 31) / 32, n_blk = n_pre + (T + 31) / 32;
  // block b into stage st_: rows past the prefix or the sequence read as zero (a prefix
  // block's rows past P are other rows or zero: masked)
  auto issue = [&](int b, int stage) {
    const bool pre = b < n_pre;
    const int k0 = (pre ? b : b - n_pre) * 32;
    const uint32_t ldk2 = (uint32_t)((pre ? pk.ldk : ldq) * 2), ldv2 = (uint32_t)((pre ? ldv : ldq) * 2);
    const uint32_t kc = (uint32_t)((pre ? hk : H + hk) * ROWB), vc = (uint32_t)((pre ? hk : H + Hkv + hk) * ROWB);
    const uint32_t base = lds_k + (uint32_t)(stage * 2 * SLOTS * 16);
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = i * RPI + lane / CH, ph = lane % CH;
      int row = k0 + r;
      if (pre && pk.pos) row = spos[min(row, P - 1)];
      const uint32_t ko = (uint32_t)row * ldk2 + kc + (uint32_t)((ph ^ k_swz<DH>(r)) * 16);
      const uint32_t vo = (uint32_t)row * ldv2 + vc + (uint32_t)((ph ^ v_swz<DH>(r)) * 16);
      const uint32_t lk = __builtin_amdgcn_readfirstlane(base + i * 1024);
      if (pre) {
        dma16(rk_p, lk, ko, 0);
        dma16(rv_p, lk + SLOTS * 16, vo, 0);
      } else {
        dma16(rsrc, lk, ko, 0);
        dma16(rsrc, lk + SLOTS * 16, vo, 0);
      }
    }
  };
  // column c = l32: query head c / T of the group, row c % T (columns past grp * T repeat the last)
  const int c = min(l32, grp * T - 1), my_t = c % T, hq = hk * grp + c / T;
  bf16x8_t qf[NKS];
  {
    const bf16_t* qp = qkv + (int64_t)(row0 + my_t) * ldq + (int64_t)hq * DH + hf * 8;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) qf[ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const v4u*>(qp + ks * 16));
  }
  int kfo[NKS], vfo[NDB];
#pragma unroll
  for (int ks = 0; ks < NKS; ++ks) kfo[ks] = l32 * ROWB + (((2 * ks + hf) ^ k_swz<DH>(l32)) << 4);
  {
    const int G = lane >> 4, jj = lane & 15, r = 4 * (G >> 1) + (jj >> 2);
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      const int chv = 4 * db + 2 * (G & 1) + ((jj & 3) >> 1);
      vfo[db] = r * ROWB + ((chv ^ v_swz<DH>(r)) << 4) + (jj & 1) * 8;
    }
  }
  const bf16x2_t ones = {(__bf16)1.0f, (__bf16)1.0f};
  f32x16_t o[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
  float m = -INFINITY, l = 0.f;
  wait_vm0();   // the query fragments are in registers before the ring starts
  if (w < n_blk) issue(w, 0);
  int stage = 0;
  for (int b = w; b < n_blk; b += 4) {
    if (b + 4 < n_blk) {
      issue(b + 4, stage ^ 1);
      wait_vmem_few<2 * NI>();
    } else {
      wait_vm0();
    }
    asm volatile("" ::: "memory");
    const bool pre = b < n_pre;
    const int k0 = (pre ? b : b - n_pre) * 32;
    const char* kt = reinterpret_cast<const char*>(&ring[w][stage][0][0]);
    const char* vt = reinterpret_cast<const char*>(&ring[w][stage][1][0]);
    f32x16_t s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks)
      s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
          __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const v4u*>(kt + kfo[ks])), qf[ks], s, 0, 0, 0);
    const int lim = pre ? P - 1 : my_t;   // last visible key of the segment
    if (pre ? k0 + 32 > P : true) {
#pragma unroll
      for (int i = 0; i < 16; ++i)
        if (k0 + (i >> 2) * 8 + hf * 4 + (i & 3) > lim) s[i] = -INFINITY;
    }
    float mx = s[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = fmaxf(mx, s[i]);
    const float m_new = fmaxf(m, max_halves(mx));
    const float ref = m_new == -INFINITY ? 0.f : m_new;   // an own block past the query's row
    const float corr = __builtin_amdgcn_exp2f(m - ref);   // 0 on the first block (m = -inf)
    m = m_new;
    l *= corr;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[db][i] *= corr;
#pragma unroll
    for (int ss = 0; ss < 2; ++ss) {
      bf16x8_t pb;
#pragma unroll
      for (int e = 0; e < 8; ++e) pb[e] = (__bf16)__builtin_amdgcn_exp2f(s[8 * ss + e] - ref);
#pragma unroll
      for (int e = 0; e < 8; e += 2) {
        const bf16x2_t pr = {pb[e], pb[e + 1]};
        l = __builtin_amdgcn_fdot2_f32_bf16(pr, ones, l, false);
      }
      const int kr = ss * 16 * ROWB;
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        const s16x4_t lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vt + kr + vfo[db]));
        const s16x4_t hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(vt + kr + 8 * ROWB + vfo[db]));
        const v4u vv = {__builtin_bit_cast(v2u, lo)[0], __builtin_bit_cast(v2u, lo)[1], __builtin_bit_cast(v2u, hi)[0],
                        __builtin_bit_cast(v2u, hi)[1]};
        o[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, vv), pb, o[db], 0, 0, 0);
      }
    }
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this stage is copied into next
    stage ^= 1;
  }
  l = sum_halves(l);
  if (hf == 0) {
    sm[w][l32] = m;
    sl[w][l32] = l;
  }
  __syncthreads();   // every ring is drained: its area holds the outputs now
  float* so = reinterpret_cast<float*>(&ring[0][0][0][0]);
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4_t*>(so + (w * 32 + l32) * SP + db * 32 + g * 8 + hf * 4) =
          f32x4_t{o[db][4 * g], o[db][4 * g + 1], o[db][4 * g + 2], o[db][4 * g + 3]};
  __syncthreads();
  const int q = tid >> 3;
  if (q >= grp * T) return;
  float M = sm[0][q];
#pragma unroll
  for (int j = 1; j < 4; ++j) M = fmaxf(M, sm[j][q]);   // finite: a row sees its own key
  float f[4], L = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    f[j] = __builtin_amdgcn_exp2f(sm[j][q] - M);
    L += sl[j][q] * f[j];
  }
  const float inv = 1.0f / L;
  bf16_t* op = out + (int64_t)(row0 + q % T) * ldo + (int64_t)(hk * grp + q / T) * DH;
#pragma unroll
  for (int cc = (tid & 7) * 4; cc < DH; cc += 32) {
    f32x4_t a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f32x4_t x = *reinterpret_cast<const f32x4_t*>(so + (j * 32 + q) * SP + cc);
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] += x[e] * f[j];
    }
    bf16x4_t u;
#pragma unroll
    for (int e = 0; e < 4; ++e) u[e] = (__bf16)(a[e] * inv);
    *reinterpret_cast<bf16x4_t*>(op + cc) = u;
  }
}

// infinite or NaN, by its bits (opaque to the compiler, which takes floats here not to be NaN)
__device__ __forceinline__ bool nonfinite(float x) {
  uint32_t bits = __builtin_bit_cast(uint32_t, x);
  asm volatile("" : "+v"(bits));
  return (bits & 0x7f800000u) == 0x7f800000u;
}

// fp32, one row of a sequence (rows at base) and head, key by key: lane sub of eight holds the
// dimensions 4 sub + 32 j .. + 3.  hq, hk, hv: the head's places in a row, in heads.
template <int DH>
__device__ __forceinline__ void attn_f32_row(const float* base, int64_t ldq, int row, int hq, int hk, int hv,
                                             float scale, int sub, float* op) {
  constexpr int N = DH / 32;
  f32x4_t q[N], acc[N];
#pragma unroll
  for (int j = 0; j < N; ++j) {
    q[j] = *reinterpret_cast<const f32x4_t*>(base + (int64_t)row * ldq + hq * DH + j * 32 + sub * 4);
    acc[j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }
  float m = -INFINITY, l = 0.f;
  for (int u = 0; u <= row; ++u) {
    const float* kp = base + (int64_t)u * ldq + hk * DH + sub * 4;
    const float* vp = base + (int64_t)u * ldq + hv * DH + sub * 4;
    float s = 0.f;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const f32x4_t kf = *reinterpret_cast<const f32x4_t*>(kp + j * 32);
#pragma unroll
      for (int e = 0; e < 4; ++e) s = fmaf(q[j][e], kf[e], s);
    }
#pragma unroll
    for (int x = 1; x < 8; x <<= 1) s += __shfl_xor(s, x, 64);
    s *= scale;
    const float m_new = fmaxf(m, s), corr = expf(m - m_new), p = expf(s - m_new);
    l = l * corr + p;
    m = m_new;
#pragma unroll
    for (int j = 0; j < N; ++j) {
      const f32x4_t vf = *reinterpret_cast<const f32x4_t*>(vp + j * 32);
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[j][e] = fmaf(p, vf[e], acc[j][e] * corr);
    }
  }
  const float inv = 1.0f / l;
#pragma unroll
  for (int j = 0; j < N; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) op[j * 32 + sub * 4 + e] = acc[j][e] * inv;
}

// fp32: one workgroup = 4 waves for 32 queries of one head.  The waves share out the
// 32-key blocks (wave w takes blocks w, w + 4, ...), each with its own running
// maximum, denominator and output, merged through LDS in wave order.  S^T = K Q^T and
// O^T = V^T P^T on v_mfma_f32_32x32x2_f32, softmax with expf.  In S^T a half-wave
// holds the dimensions hf d_h / 2 .. of its row, so K and Q rows are read as 16-byte
// pieces; lane l then owns query l % 32 and the keys 8 (i / 4) + 4 hf + i % 4, and the key
// order of O^T is that of those registers.
// Bound: latency of a block's two MFMA chains (2 x d_h x 32 cycles) and of its loads.
// Against one thread per (row, head) walking the keys: 256 rows, 4 heads of 64 278 -> 13 us,
// 1024 + 777 rows, 12 heads of 64 1181 -> 57.
// CLEAN: Values of the diagonal block that are infinite or NaN (tested by their bits: this
// file is compiled as if there were no NaN) count as zero, and the rows from the first of
// them on, which see it, are walked key by key.  Returns whether any of the thread's
// outputs is infinite or NaN.
template <int DH, bool CLEAN>
__device__ __forceinline__ bool attn_f32_tile(const float* __restrict__ qkv, int64_t ldq, float* __restrict__ out,
                                              int64_t ldo, const SeqTable& st, const AttnWork& wk, int H, int Hkv,
                                              float scale, float (&so)[4][32 * (DH + 4)], float (&sm)[4][32],
                                              float (&sl)[4][32], int32_t& sbad) {
  constexpr int HD = DH / 2, NDB = DH / 32, SP = DH + 4;
  const int tid = threadIdx.x, lane = tid & 63, l32 = lane & 31, hf = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int item = blockIdx.x / H, hq = blockIdx.x - item * H, hk = hq / (H / Hkv);
  int lo = 0, hi = st.n - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (wk.cum[mid] <= item) lo = mid; else hi = mid - 1;
  }
  const int k = wk.order[lo], row0 = st.off[k], T = st.off[k + 1] - row0;
  const int qb = (T + 31) / 32 - 1 - (item - wk.cum[lo]), q0 = qb * 32;   // longest first
  const int my_q = min(q0 + l32, T - 1);   // rows past T duplicate row T - 1
  const float* kbase = qkv + (int64_t)row0 * ldq + (int64_t)(H + hk) * DH;
  const float* vbase = kbase + (int64_t)Hkv * DH;
  f32x4_t qf[HD / 4];
  {
    const float* qp = qkv + (int64_t)(row0 + my_q) * ldq + (int64_t)hq * DH + hf * HD;
#pragma unroll
    for (int j = 0; j < HD / 4; ++j) qf[j] = *reinterpret_cast<const f32x4_t*>(qp + 4 * j);
  }
  f32x16_t o[NDB];
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[db][i] = 0.f;
  float m = -INFINITY, l = 0.f;
  for (int kb = w; kb <= qb; kb += 4) {
    const int k0 = kb * 32;
    f32x16_t s;
#pragma unroll
    for (int i = 0; i < 16; ++i) s[i] = 0.f;
    const float* kp = kbase + (int64_t)min(k0 + l32, T - 1) * ldq + hf * HD;
#pragma unroll
    for (int j = 0; j < HD / 4; ++j) {
      const f32x4_t kf = *reinterpret_cast<const f32x4_t*>(kp + 4 * j);
#pragma unroll
      for (int e = 0; e < 4; ++e) s = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[e], qf[j][e], s, 0, 0, 0);
    }
    float mx = -INFINITY;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int key = k0 + (i >> 2) * 8 + hf * 4 + (i & 3);
      s[i] = key <= my_q ? s[i] * scale : -INFINITY;
      mx = fmaxf(mx, s[i]);
    }
    mx = max_halves(mx);
    const float m_new = fmaxf(m, mx);   // block 0 holds a key of every query; later blocks follow a finite m or start one
    const float ref = m_new == -INFINITY ? 0.f : m_new;
    const float corr = m == -INFINITY ? 0.f : expf(m - ref);
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s[i] = expf(s[i] - ref);
      sum += s[i];
    }
    l = l * corr + sum;
    m = m_new;
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[db][i] *= corr;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float* vp = vbase + (int64_t)min(k0 + (i >> 2) * 8 + hf * 4 + (i & 3), T - 1) * ldq + l32;
#pragma unroll
      for (int db = 0; db < NDB; ++db) {
        float x = vp[db * 32];
        if constexpr (CLEAN)
          if (kb == qb && nonfinite(x)) x = 0.f;
        o[db] = __builtin_amdgcn_mfma_f32_32x32x2f32(x, s[i], o[db], 0, 0, 0);
      }
    }
    if constexpr (CLEAN)
      if (kb == qb) {   // one wave's
        int first = INT32_MAX;
        for (int u = min(k0 + 31, T - 1); u >= k0; --u) {
          bool bad = false;
          for (int j = lane; j < DH; j += 64) bad |= nonfinite(vbase[(int64_t)u * ldq + j]);
          if (__any(bad)) first = u;
        }
        if (lane == 0) sbad = first;
      }
  }
  l = sum_halves(l);
  if (hf == 0) {
    sm[w][l32] = m;
    sl[w][l32] = l;
  }
#pragma unroll
  for (int db = 0; db < NDB; ++db)
#pragma unroll
    for (int g = 0; g < 4; ++g)
      *reinterpret_cast<f32x4_t*>(&so[w][l32 * SP + db * 32 + g * 8 + hf * 4]) =
          f32x4_t{o[db][4 * g], o[db][4 * g + 1], o[db][4 * g + 2], o[db][4 * g + 3]};
  __syncthreads();
  const int q = tid >> 3, row = q0 + q;
  if (row >= T) return false;
  float M = sm[0][q];   // wave 0 holds block 0: finite
#pragma unroll
  for (int j = 1; j < 4; ++j) M = fmaxf(M, sm[j][q]);
  float f[4], L = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    f[j] = sm[j][q] == -INFINITY ? 0.f : expf(sm[j][q] - M);
    L += sl[j][q] * f[j];
  }
  const float inv = 1.0f / L;
  float* op = out + (int64_t)(row0 + row) * ldo + (int64_t)hq * DH;
  bool bad = false;
#pragma unroll
  for (int c = (tid & 7) * 4; c < DH; c += 32) {
    f32x4_t a = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const f32x4_t x = *reinterpret_cast<const f32x4_t*>(&so[j][q * SP + c]);
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] += x[e] * f[j];
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      a[e] *= inv;
      bad |= nonfinite(a[e]);
    }
    *reinterpret_cast<f32x4_t*>(op + c) = a;
  }
  if constexpr (CLEAN)
    if (row >= sbad) attn_f32_row<DH>(qkv + (int64_t)row0 * ldq, ldq, row, hq, H + hk, H + Hkv + hk, scale, tid & 7, op);
  return bad;
}

template <int DH>
__global__ __launch_bounds__(256) void attn_f32_kernel(const float* __restrict__ qkv, int64_t ldq,
                                                       float* __restrict__ out, int64_t ldo, SeqTable st, AttnWork wk,
                                                       int H, int Hkv, float scale) {
  __shared__ __attribute__((aligned(16))) float so[4][32 * (DH + 4)];
  __shared__ float sm[4][32], sl[4][32];
  __shared__ int32_t sbad;
  const bool bad = attn_f32_tile<DH, false>(qkv, ldq, out, ldo, st, wk, H, Hkv, scale, so, sm, sl, sbad);
  // A masked key's zero weight times a non-finite Value is NaN, which would reach rows that do
  // not see the key: such a tile is run again.
  if (__syncthreads_or(bad)) attn_f32_tile<DH, true>(qkv, ldq, out, ldo, st, wk, H, Hkv, scale, so, sm, sl, sbad);
}

// Work items of a launch: sequences by decreasing length; items[k] per sequence.
template <class F>
static AttnWork attn_work(const SeqTable& st, const F& items) {
  AttnWork wk;
  for (int k = 0; k < st.n; ++k) wk.order[k] = k;
  for (int a = 1; a < st.n; ++a) {  // insertion sort, stable
    const int v = wk.order[a], len = st.off[v + 1] - st.off[v];
    int b = a;
    while (b > 0 && st.off[wk.order[b - 1] + 1] - st.off[wk.order[b - 1]] < len) {
      wk.order[b] = wk.order[b - 1];
      --b;
    }
    wk.order[b] = v;
  }
  wk.cum[0] = 0;
  for (int j = 0; j < st.n; ++j) {
    const int k = wk.order[j];
    wk.cum[j + 1] = wk.cum[j] + items(st.off[k + 1] - st.off[k]);
  }
  wk.total = wk.cum[st.n];
  return wk;
}

// Whether a sequence of len rows behind a cached prefix takes attn_few_kernel.  By its own
// length: the two kernels round differently, and a sequence's result is the same beside
// any others.
static bool few_rows(int len, int n_heads, int n_kv_heads) {
  return (int64_t)len * (n_heads / n_kv_heads) <= kFewRows;
}

// Only attn_few_kernel takes positions; beside longer sequences all read gathered caches,
// with the same result.
bool attention_takes_positions(const SeqTable& st, int n_heads, int n_kv_heads, int keep, int full_P, int64_t ld) {
  return few_rows(st.max_len, n_heads, n_kv_heads) && keep <= kFewPos && (int64_t)full_P * ld * 2 < ((int64_t)1 << 31);
}

hipError_t launch_attention(const void* qkv, int64_t ldq, void* out, int64_t ldo, const SeqTable& st, int n_heads,
                            int n_kv_heads, int head_dim, bool bf16, hipStream_t s, const KvPrefix* prefix) {
  if (st.rows <= 0) return hipSuccess;
  if (bf16) {
    const bool pre = prefix && prefix->P > 0;
    const int bq = 32 * (head_dim == 64 ? AttnTraits<64>::kWaves : AttnTraits<128>::kWaves);   // queries per block
    // Items = pairs of q-blocks.  Single q-blocks behind a cached prefix, and where all
    // single blocks run at once (one workgroup on each of 256 CUs): a pair's second block only
    // adds to the longest item's time (509 rows, 12 heads of 64: 24 pairs of up to 10 tiles
    // 14.1 us, 48 blocks of up to 8 tiles 10.8).
    int64_t blocks = 0;
    int n_few = 0;   // sequences of attn_few_kernel: no items here
    for (int k = 0; k < st.n; ++k) {
      const int len = st.off[k + 1] - st.off[k];
      blocks += (len + bq - 1) / bq;
      if (pre && len > 0 && few_rows(len, n_heads, n_kv_heads)) ++n_few;
    }
    const bool paired = !pre && blocks * n_heads > 256;
    const AttnWork wk = attn_work(st, [&](int len) {
      const int nqb = (len + bq - 1) / bq;
      if (pre && few_rows(len, n_heads, n_kv_heads)) return 0;
      return paired ? (nqb + 1) / 2 : nqb;
    });
    if (wk.total == 0 && n_few == 0) return hipSuccess;
    // the buffer descriptor covers one sequence's rows with 32-bit byte offsets
    if ((int64_t)st.max_len * ldq * 2 >= ((int64_t)1 << 31) || n_heads % n_kv_heads != 0) return hipErrorInvalidValue;
    const int grp = n_heads / n_kv_heads;
    const int n_items = wk.total * n_heads;
    const int grid = (n_items + 8 * grp - 1) / (8 * grp) * (8 * grp);
    KvPrefix pk{};
    if (pre) {
      pk = *prefix;
      if (pk.pos && !attention_takes_positions(st, n_heads, n_kv_heads, pk.P, pk.full_P, std::max(pk.ldk, pk.ldv)))
        return hipErrorInvalidValue;
      // one descriptor per sequence's cached prefix, also with 32-bit byte offsets
      const int64_t ld = std::max(std::max(pk.ldk, pk.ldv), pk.alt_pass >= 0 && pk.n_seq > 0 ? pk.ldv_alt : 0);
      if ((int64_t)pk.P * ld * 2 >= ((int64_t)1 << 31)) return hipErrorInvalidValue;
      if (pk.n_seq > 0 && (st.n % pk.n_seq != 0 || (pk.alt_pass >= 0 && !pk.v_alt))) return hipErrorInvalidValue;
    }
    if (n_few > 0) {
      if (head_dim == 128)
        attn_few_kernel<128><<<st.n * n_kv_heads, 256, 0, s>>>((const bf16_t*)qkv, ldq, (bf16_t*)out, ldo, st, n_heads,
                                                               n_kv_heads, pk);
      else if (head_dim == 64)
        attn_few_kernel<64><<<st.n * n_kv_heads, 256, 0, s>>>((const bf16_t*)qkv, ldq, (bf16_t*)out, ldo, st, n_heads,
                                                              n_kv_heads, pk);
      else return hipErrorInvalidValue;
      if (wk.total == 0) return hipGetLastError();
    }
#define RK_ATTN(D, PRE)                                                                                      \
  attn_bf16_kernel<D, PRE><<<grid, 64 * AttnTraits<D>::kWaves, 0, s>>>((const bf16_t*)qkv, ldq, (bf16_t*)out, ldo, \
                                                                      st, wk, n_heads, n_kv_heads, n_items, paired ? 1 : 0, pk)
    if (head_dim == 128) { if (pre) RK_ATTN(128, true); else RK_ATTN(128, false); }
    else if (head_dim == 64) { if (pre) RK_ATTN(64, true); else RK_ATTN(64, false); }
    else return hipErrorInvalidValue;
#undef RK_ATTN
  } else {
    if (prefix && prefix->P > 0) return hipErrorInvalidValue;   // cached prefixes: bf16 path only
    const float scale = (float)(1.0 / sqrt((double)head_dim));
    const AttnWork wk = attn_work(st, [](int len) { return (len + 31) / 32; });
    if (n_heads % n_kv_heads != 0 || (int64_t)wk.total * n_heads > INT32_MAX) return hipErrorInvalidValue;
    const int grid = wk.total * n_heads;
#define RK_ATTN32(D)                                                                                        \
  attn_f32_kernel<D><<<grid, 256, 0, s>>>((const float*)qkv, ldq, (float*)out, ldo, st, wk, n_heads, n_kv_heads, \
                                          scale)
    if (head_dim == 32) RK_ATTN32(32);
    else if (head_dim == 64) RK_ATTN32(64);
    else if (head_dim == 128) RK_ATTN32(128);
    else return hipErrorInvalidValue;
#undef RK_ATTN32
  }
  return hipGetLastError();
}

}  // namespace rk

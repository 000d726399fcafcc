// Device code of the update's decisions (Eq. 7-9) that more than one kernel runs: the retention of a head by one
// workgroup (retain_kernel; the extra workgroups of the attention launch that takes the decisions beside the
// attention), and the scoring of a whole head by one workgroup (those extra workgroups only).
//
// Every fp32 operation here is exactly the one written (the arithmetic that decides block sets and slots is
// specified operation by operation in pbsa.h): the functions switch contraction off for themselves, and every
// file that includes this one is compiled with correctly rounded fp32 division.
#pragma once

#include <type_traits>
#include <utility>

#include "pbsa_internal.h"

namespace pbsa {
namespace plan_dev {

__device__ __forceinline__ int lanes_below(uint64_t mask) {   // set bits of `mask` in lanes below this one
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// exp(x) for x <= 0 from fp32 mul / fma / rint only (steps fixed in pbsa.h).  Without a branch: several run side by side.
__device__ __forceinline__ float pexp(float x0) {
  const bool none = x0 < -64.0f;
  const float x = none ? -64.0f : x0;
  float n = __builtin_rintf(x * 0x1.715476p+0f);
  float r = __builtin_fmaf(n, -0x1.630000p-1f, x);
  r = __builtin_fmaf(n, 0x1.bd0106p-13f, r);
  float p = 0x1.6c16c2p-10f;
  p = __builtin_fmaf(p, r, 0x1.111112p-7f);
  p = __builtin_fmaf(p, r, 0x1.555556p-5f);
  p = __builtin_fmaf(p, r, 0x1.555556p-3f);
  p = __builtin_fmaf(p, r, 0.5f);
  p = __builtin_fmaf(p, r, 1.0f);
  p = __builtin_fmaf(p, r, 1.0f);
  const float e = p * __uint_as_float((uint32_t)((int)n + 127) << 23);
  return none ? 0.0f : e;
}

struct ScoreArgs {
  int H, nqb, nqb_pad, n_loc, n_loc_cap, C, nU_max, n_evict;
  float scale;
  const float* Kc_l;
  const float* Kc_p;
  const float* Qc;
  const float* Zl;          // optional: scaled local logits [H][nqb][n_loc] from the selection call
  const int32_t* l_map;
  const int32_t* p_len;
  float* A;
};

constexpr int kMaxCand = PBSA_MAX_C + PBSA_MAX_N_LOC_AUX;

struct RetainArgs {
  int H, nqb, nqb_pad, n_loc, n_loc_cap, C, n_sink, n_evict, nU_max, d, B, fold;
  int fine, Nq;             // fine: A is the attention-mass matrix [H][C+1+n_loc][nqb_pad], one row per key block
                            // (slots 0..C, then the local blocks), and a score is its row sum over Nq
  const float* A;           // A^T [H][nU_max][nqb_pad]
  const float* Kc_l;
  float* Kc_p;
  const int32_t* p_len;
  int32_t* p_len_out;       // [H][C + 1] lengths after the update (the fold kernel commits them)
  int64_t* p_id;
  int32_t* S_cnt;
  const int32_t* l_len;
  const int32_t* l_map;
  const int64_t* l_id;
  float* scores;
  int32_t* slot_src;
  int32_t* fold_n;
  int32_t* fold_src;        // dropped candidate: < C persistent slot, else C + PHYSICAL local slot
  int32_t* fold_len;
  int32_t* promo_slot;      // [H][C] physical local slot a persistent slot is refilled from, or -1
};

// position of the n-th (0-based) set bit of mask
__device__ __forceinline__ int nth_set_bit(uint64_t mask, int n) {
  for (int i = 0; i < n; ++i) mask &= mask - 1;
  return __ffsll((unsigned long long)mask) - 1;
}

// What retain_body needs of a head's metadata, in registers: asked for before anything else, so that it arrives while the
// scores are computed.
template <int NT>
struct RetainPre {
  static constexpr int EV = (PBSA_MAX_N_LOC_AUX + NT - 1) / NT;
  int e_len[EV], e_map[EV], slot_len, cnt;
  long long e_id[EV];
};
template <int NT>
__device__ __forceinline__ RetainPre<NT> retain_prefetch(const RetainArgs& a, const int h) {
  static_assert(NT >= 128 && NT > PBSA_MAX_C, "one thread per position of a block, and per slot");
  RetainPre<NT> pre;
  pre.slot_len = (int)threadIdx.x <= a.C ? a.p_len[(size_t)h * (a.C + 1) + threadIdx.x] : 0;
#pragma unroll
  for (int u = 0; u < RetainPre<NT>::EV; ++u) {
    const int e = threadIdx.x + u * NT;
    pre.e_len[u] = e < a.n_evict ? a.l_len[e] : 0;
    pre.e_map[u] = e < a.n_evict ? a.l_map[e] : 0;
    pre.e_id[u] = e < a.n_evict ? a.l_id[e] : 0;
  }
  pre.cnt = a.fold && (int)threadIdx.x < a.B ? a.S_cnt[(size_t)h * a.B + threadIdx.x] : 0;
  return pre;
}

// LDS of retain_body
struct RetainLds {
  alignas(16) float cs[kMaxCand + 4];   // candidate scores
  float s[kMaxCand];   // mean column score of slot / evicted-block columns, U order
  int cand[kMaxCand];   // < C: slot, else C + local block
  unsigned char win[kMaxCand];
  int rank_s[kMaxCand];
  unsigned char vac_s[PBSA_MAX_C];   // slot whose occupant is dropped
  int old_len[PBSA_MAX_C + 1];
  int src_s[PBSA_MAX_C];
  int flen[kMaxCand];   // valid tokens of each dropped candidate
  int e_len[PBSA_MAX_N_LOC_AUX];   // valid tokens / physical slot of the evicted blocks
  int e_map[PBSA_MAX_N_LOC_AUX];
  long long e_id[PBSA_MAX_N_LOC_AUX];   // global ids of the evicted blocks
  int nf_s, npos_s;
};

// Retention (Eq. 8-9) of head h by one workgroup of NT threads (a multiple of 64, at least 128).  A: the head's matrix, columns
// nqb_pad floats apart, in global memory or (in_lds) in LDS outside L.
template <int NT>
__device__ inline void retain_body(const RetainArgs& a, const int h, const RetainPre<NT>& pre, const float* A, const bool in_lds, RetainLds& L) {
#pragma clang fp contract(off)
  auto& cs = L.cs;
  auto& s = L.s;
  auto& cand = L.cand;
  auto& win = L.win;
  auto& rank_s = L.rank_s;
  auto& vac_s = L.vac_s;
  auto& old_len = L.old_len;
  auto& src_s = L.src_s;
  auto& flen = L.flen;
  auto& e_len = L.e_len;
  auto& e_map = L.e_map;
  auto& e_id = L.e_id;
  int& nf_s = L.nf_s;
  int& npos_s = L.npos_s;
  const int C = a.C, C1 = a.C + 1;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  if ((int)threadIdx.x < C1) old_len[threadIdx.x] = pre.slot_len;
#pragma unroll
  for (int u = 0; u < RetainPre<NT>::EV; ++u) {
    const int e = threadIdx.x + u * NT;
    if (e < a.n_evict) {
      e_len[e] = max(0, min(pre.e_len[u], a.B));
      e_map[e] = min(max(pre.e_map[u], 0), a.n_loc_cap - 1);
      e_id[e] = pre.e_id[u];
    }
  }
  const int cnt_mine = pre.cnt;            // the summary's count of position threadIdx.x, needed at the very end
  if (threadIdx.x == 0) npos_s = 0;
  __syncthreads();
  // occupied slots: U position of slot c = number of occupied slots below it (C <= 64: one ballot)
  const bool occ = lane < C && old_len[lane] > 0;
  const uint64_t occ_mask = __ballot(occ);
  const int nP = __popcll(occ_mask), u_pos = lanes_below(occ_mask);
  // Column means (Eq. 8) of the columns that can be candidates: the occupied slots and the evicted
  // blocks, i.e. the first nP + n_evict columns of U.
  const int n_need = nP + a.n_evict;
  // A column is contiguous in A^T: its rows are fetched 64 at a time and added in ascending order.
  for (int j = threadIdx.x; j < n_need; j += NT) {
    float acc = 0.0f;
    // where column j of U sits: the coarse matrix is in U order (occupied slots, then local blocks); the mass
    // matrix has a row for every slot, the summary included
    const int at = !a.fine ? j : j < nP ? nth_set_bit(occ_mask, j) : C + 1 + (j - nP);
    const float4* col = reinterpret_cast<const float4*>(A + (size_t)at * a.nqb_pad);
    auto add4 = [&](const float4& v, int i) {
      acc = acc + v.x;
      if (i + 1 < a.nqb) acc = acc + v.y;
      if (i + 2 < a.nqb) acc = acc + v.z;
      if (i + 3 < a.nqb) acc = acc + v.w;
    };
    if (in_lds) {
#pragma unroll 1
      for (int i = 0; i < a.nqb; i += 4) add4(col[i / 4], i);
    } else {                               // 64 rows in flight together
#pragma unroll 1
      for (int i0 = 0; i0 < a.nqb; i0 += 64) {
        float4 v[16];
#pragma unroll
        for (int u = 0; u < 16; ++u) v[u] = i0 + 4 * u < a.nqb ? col[i0 / 4 + u] : make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
        for (int u = 0; u < 16; ++u)
          if (i0 + 4 * u < a.nqb) add4(v[u], i0 + 4 * u);
      }
    }
    s[j] = acc / (float)(a.fine ? a.Nq : a.nqb);
  }
  __syncthreads();
  // candidates: occupants of slots >= n_sink in slot order, then the evicted blocks
  const int ncand_max = C + a.n_evict;
  const bool is_cand = occ && lane >= a.n_sink;
  const uint64_t cand_mask = __ballot(is_cand);
  const int ncP = __popcll(cand_mask), nc = ncP + a.n_evict, places = C - a.n_sink;
  if (wave == 0) {
    if (lane < C && a.scores) a.scores[(size_t)h * ncand_max + lane] = occ ? s[u_pos] : 0.0f;
    if (is_cand) {
      const int x = lanes_below(cand_mask);
      cand[x] = lane;
      cs[x] = s[u_pos];
    }
  }
  for (int e = threadIdx.x; e < a.n_evict; e += NT) {
    if (a.scores) a.scores[(size_t)h * ncand_max + C + e] = s[nP + e];
    cand[ncP + e] = C + e;
    cs[ncP + e] = s[nP + e];
  }
  __syncthreads();
  // rank of a candidate = how many beat it (higher score, or equal score and lower index).  All threads
  // take part: with P = NT / nc threads per candidate each counts over its share of the others
  // (several 16-byte reads in flight), and the shares meet in an integer counter.
  for (int x = threadIdx.x; x < nc; x += NT) rank_s[x] = 0;
  __syncthreads();
  {
    const int P = max(1, NT / max(nc, 1)), n4 = (nc + 3) / 4, per = (n4 + P - 1) / P;
    const float4* c4 = reinterpret_cast<const float4*>(cs);
    for (int idx = threadIdx.x; idx < nc * P; idx += NT) {
      const int x = idx % nc, part = idx / nc;
      const float mine = cs[x];
      int rank = 0;
      const int q_end = min(n4, (part + 1) * per);
#pragma unroll 1
      for (int q = part * per; q < q_end; ++q) {
        const float4 v = c4[q];
        const int y = 4 * q;
        // without branches: (in range) and (higher, or equal and earlier)
        rank += (int)(y + 0 < nc) & ((int)(v.x > mine) | ((int)(v.x == mine) & (int)(y + 0 < x)));
        rank += (int)(y + 1 < nc) & ((int)(v.y > mine) | ((int)(v.y == mine) & (int)(y + 1 < x)));
        rank += (int)(y + 2 < nc) & ((int)(v.z > mine) | ((int)(v.z == mine) & (int)(y + 2 < x)));
        rank += (int)(y + 3 < nc) & ((int)(v.w > mine) | ((int)(v.w == mine) & (int)(y + 3 < x)));
      }
      if (rank) atomicAdd(&rank_s[x], rank);
    }
  }
  __syncthreads();
  for (int x = threadIdx.x; x < nc; x += NT) win[x] = rank_s[x] < places;
  for (int c = threadIdx.x; c < C; c += NT) vac_s[c] = 0;
  __syncthreads();
  // wave 0: dropped candidates, in candidate order, go to the fold list; then kept newcomers, in
  // ascending block order, take the vacated and empty slots in ascending slot order
  if (wave == 0) {
    int nf = 0;
    for (int x0 = 0; x0 < nc; x0 += 64) {
      const int x = x0 + lane;
      const bool lose = x < nc && !win[x];
      const uint64_t lm = __ballot(lose);
      if (lose) {
        const int f = nf + lanes_below(lm);
        const bool slot_cand = cand[x] < C;
        const int len = slot_cand ? old_len[cand[x]] : e_len[cand[x] - C];
        a.fold_src[(size_t)h * ncand_max + f] = slot_cand ? cand[x] : C + e_map[cand[x] - C];
        a.fold_len[(size_t)h * ncand_max + f] = len;
        flen[f] = len;
        if (slot_cand) vac_s[cand[x]] = 1;
      }
      nf += __popcll(lm);
    }
    if (lane == 0) { a.fold_n[h] = nf; nf_s = nf; }
    // free slots = (empty or vacated) and >= n_sink (vac_s: written above by this wave, LDS keeps a wave's order)
    const bool vacated = lane < C && vac_s[lane];
    const bool is_free = lane < C && lane >= a.n_sink && (old_len[lane] <= 0 || vacated);
    const uint64_t free_mask = __ballot(is_free);
    if (lane < C) {
      src_s[lane] = -1;
      if (vacated) old_len[lane] = 0;
    }
    int taken = 0;
    for (int x0 = ncP; x0 < nc; x0 += 64) {
      const int x = x0 + lane;
      const bool keep = x < nc && win[x];
      const uint64_t km = __ballot(keep);
      if (keep) {
        const int r = taken + lanes_below(km);       // r-th kept newcomer takes the r-th free slot
        if (r < __popcll(free_mask)) {
          const int slot = nth_set_bit(free_mask, r);
          const int e = cand[x] - C;
          old_len[slot] = e_len[e];
          src_s[slot] = e;
        }
      }
      taken += __popcll(km);
    }
  }
  __syncthreads();
  // per-position counts of the summary: every dropped block adds one to each position it has
  if (a.fold && nf_s > 0) {
    if (threadIdx.x < a.B) {
      const int t = threadIdx.x;
      int cnt = cnt_mine;
#pragma unroll 8
      for (int f = 0; f < nf_s; ++f) cnt += (int)(t < flen[f]);
      a.S_cnt[(size_t)h * a.B + t] = cnt;
      if (cnt > 0) atomicAdd(&npos_s, 1);
    }
    __syncthreads();
    if (threadIdx.x == 0) old_len[C] = npos_s;
    __syncthreads();
  }
  for (int c = threadIdx.x; c < C1; c += NT) a.p_len_out[(size_t)h * C1 + c] = old_len[c];
  for (int c = threadIdx.x; c < C; c += NT) {
    const int e = src_s[c];
    a.slot_src[(size_t)h * C + c] = e;
    a.promo_slot[(size_t)h * C + c] = e >= 0 ? e_map[e] : -1;
    if (e >= 0) a.p_id[(size_t)h * C + c] = e_id[e];
    else if (c >= a.n_sink && old_len[c] == 0) a.p_id[(size_t)h * C + c] = -1;
  }
  // pooled keys move with the promoted blocks: independent float4 copies
  const int d4 = a.d / 4;
  for (int idx = threadIdx.x; idx < C * d4; idx += NT) {
    const int c = idx / d4, x = idx % d4;
    const int e = src_s[c];
    if (e >= 0)
      reinterpret_cast<float4*>(a.Kc_p + ((size_t)h * C + c) * a.d)[x] =
          reinterpret_cast<const float4*>(a.Kc_l + ((size_t)h * a.n_loc_cap + e_map[e]) * a.d)[x];
  }
}

// v_mfma_f32_4x4x1_16b_f32: sixteen 4 x 4 products of one contraction index.  With A of block X broadcast to all blocks (cbsz
// 4), lane L's element r of the result is fma(a of lane 4 X + r, b of lane L, c of element r), rounded once, denormals and
// infinities included; a NaN in any of them is a NaN in the result.
typedef __attribute__((ext_vector_type(4))) float vec4;
template <int X>
__device__ __forceinline__ vec4 fma_4_rows(float a, float b, vec4 c) {
  return __builtin_amdgcn_mfma_f32_4x4x1f32(a, b, c, 4, X, 0);
}
template <typename F, int... I>
__device__ __forceinline__ void unroll(F f, std::integer_sequence<int, I...>) {     // f(0), f(1), .. with the number as a constant
  (f(std::integral_constant<int, I>{}), ...);
}

// The largest of the wave's numbers (a NaN counts as none), of four such at a time: the steps of one are as far apart as a
// number must be from the data-parallel step that reads it.
__device__ __forceinline__ void wave_max4(float (&x)[4]) {
#define PBSA_STEP(HOW)                                                                                                  \
  "v_max_f32_dpp %0, %0, %0 " HOW "\n\tv_max_f32_dpp %1, %1, %1 " HOW "\n\tv_max_f32_dpp %2, %2, %2 " HOW                \
  "\n\tv_max_f32_dpp %3, %3, %3 " HOW "\n\t"
  asm volatile("s_nop 1\n\t"
               PBSA_STEP("row_shr:1 row_mask:0xf bank_mask:0xf")    // the lane 1, 2, 4, 8 places down in the row of 16
               PBSA_STEP("row_shr:2 row_mask:0xf bank_mask:0xf")
               PBSA_STEP("row_shr:4 row_mask:0xf bank_mask:0xf")
               PBSA_STEP("row_shr:8 row_mask:0xf bank_mask:0xf")
               PBSA_STEP("row_bcast:15 row_mask:0xa bank_mask:0xf") // the last lane of the row before
               PBSA_STEP("row_bcast:31 row_mask:0xc bank_mask:0xf") // lane 31
               "s_nop 1"
               : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
#undef PBSA_STEP
#pragma unroll
  for (int r = 0; r < 4; ++r) x[r] = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x[r]), 63));
}

// One wave-wide global -> LDS load of 4 or 16 bytes per lane: LDS bytes [lds_off, lds_off + 64 * that) receive the lanes' bytes,
// fetched from base + voff, side by side.  Completion is tracked by the issuing wave's vmcnt.
__device__ __forceinline__ void stage4(const void* base, uint32_t voff, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2" : : "s"(lds_off), "v"(voff), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void stage16(const void* base, uint32_t voff, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_off), "v"(voff), "s"(base) : "memory", "m0");
}

// Rows of the block-level softmax (Eq. 7) of a whole head by one workgroup of NT threads, given the scaled local
// logits Zl the selection call left: the same operations in the same order as score_rows_kernel (per row the chain of each
// persistent column, the row maximum, the exponentials, their sum in column order, the quotients stored column-major into
// A, nqb_pad floats a column).  Pooled keys, queries and logits reach LDS by direct loads that are all in flight together, as
// many rows at a time as fit; then each wave works on four rows at a time: lane c runs the chains of slot c as rows of one
// matrix instruction per dimension (slots' keys lie there as the selection's do), and adds up row c of the wave's rows.
// Bound by latency, and much of that is fetching instructions that run once: nothing is unrolled but the four rows that a wave
// works on side by side.  Both halves of the decisions, workgroups of 256 threads, by time stamps: 9.4 -> 7.4 us at 2 heads x 4
// blocks of 64, longer than the attention beside them before; with rows and columns unrolled and more asked for at
// once 11.6.  A chained step of 15 x 1386 x 64 whose 128 threads decide for 22 blocks, 46.3 -> 34.8; a step of 9 x 4458 x 128 with
// 70 blocks and 280 columns and a short attention 134 -> 93.
template <int D>
struct ScoreGeo {
  static constexpr int key_round(int C) { return ((C + 7) & ~7) * 128; }        // bytes of 32 dimensions of the slots' pooled keys
  static constexpr int keys(int C) { return D / 32 * key_round(C); }
  static constexpr int row_floats(int n_loc) { return 64 * ((n_loc + 63) / 64) + 65; }   // logits, then the slots', an odd pitch
  // rows at a time in so many bytes; the queries' last load may run up to 1 KiB over
  static constexpr int rows(int bytes, int C, int n_loc) { return (bytes - keys(C) - 1024) / ((D + row_floats(n_loc)) * 4) & ~3; }
};
template <int D>
constexpr bool score_fits(int bytes) { return ScoreGeo<D>::rows(bytes, PBSA_MAX_C, PBSA_MAX_N_LOC_AUX) >= 4; }

template <int D, int NT>
__device__ inline void score_head_body(const ScoreArgs& a, const int h, unsigned char* lds, const int lds_bytes, float* A) {
#pragma clang fp contract(off)
  constexpr int NW = NT / 64;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int nml = (a.n_loc + 63) / 64, EP = ScoreGeo<D>::row_floats(a.n_loc);
  const int cap = min((a.nqb + 3) & ~3, ScoreGeo<D>::rows(lds_bytes, a.C, a.n_loc)), key_round = ScoreGeo<D>::key_round(a.C);
  float* const qs = reinterpret_cast<float*>(lds + ScoreGeo<D>::keys(a.C));     // [cap][D]
  float* const er = qs + cap * D + 256;                                         // [cap][EP]
  const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)lds);
  const uint32_t qs0 = lds0 + ScoreGeo<D>::keys(a.C), er0 = qs0 + cap * D * 4 + 1024;
  const int slot_len = lane < a.C ? a.p_len[(size_t)h * (a.C + 1) + lane] : 0;
  {
    // 1 KiB a load: eight slots' 32 dimensions 32 r .. (128 bytes a slot, 16-byte chunk c of slot j at c ^ ((j / 2) % 8))
    const float* const kp = a.Kc_p + (size_t)h * a.C * D;
    const int n8 = (a.C + 7) / 8;
#pragma unroll 1
    for (int n = wave; n < n8; n += NW) {
      const int j = 8 * n + (lane >> 3), chunk = (lane & 7) ^ ((j >> 1) & 7);
#pragma unroll 1
      for (int r = 0; r < D / 32; ++r)
        stage16(kp + 32 * r, (uint32_t)(min(j, a.C - 1) * D * 4 + chunk * 16), lds0 + r * key_round + n * 1024);
    }
  }
  uint64_t occ_mask = 0;
  int nP = 0, at = 0;                                                           // occupied slots; this lane's place among them
#pragma unroll 1
  for (int r0 = 0; r0 < a.nqb; r0 += cap) {
    const int rows = min(cap, a.nqb - r0);
    if (r0 > 0) __syncthreads();                                                // the rows before are done with
    const float* const q = a.Qc + ((size_t)h * a.nqb + r0) * D;
#pragma unroll 1
    for (int n = wave; n * 256 < rows * D; n += NW) stage16(q, (uint32_t)(min(n * 256 + lane * 4, rows * D - 4) * 4), qs0 + n * 1024);
    const float* const z = a.Zl + ((size_t)h * a.nqb + r0) * a.n_loc;
#pragma unroll 1
    for (int m = 0; m < nml; ++m) {
      const uint32_t voff = (uint32_t)(min(64 * m + lane, a.n_loc - 1) * 4);
      const float* zr = z + (size_t)wave * a.n_loc;
      uint32_t to = er0 + (wave * EP + 64 * m) * 4;
#pragma unroll 1
      for (int r = wave; r < rows; r += NW, zr += (size_t)NW * a.n_loc, to += NW * EP * 4) stage4(zr, voff, to);
    }
    if (r0 == 0) {
      occ_mask = __ballot(slot_len > 0);
      nP = __popcll(occ_mask);
      at = lanes_below(occ_mask);
    }
    const bool occ = slot_len > 0;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    const int sw = (lane >> 1) & 7;
    float s = 0.0f;
#pragma unroll 1
    for (int g = wave; 4 * g < rows; g += NW) {
      vec4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 1
      for (int m = 0; m < D / 16; ++m) {
        const float qv = qs[(4 * g + (lane & 3)) * D + 16 * m + (lane >> 2)];
        const unsigned char* kb = lds + (m >> 1) * key_round + min(lane, max((a.C + 7) & ~7, 8) - 1) * 128;
        float4 k[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) k[c] = *reinterpret_cast<const float4*>(kb + (((4 * (m & 1) + c) ^ sw) << 4));
        asm volatile("" : "+v"(k[0].x), "+v"(k[1].x), "+v"(k[2].x), "+v"(k[3].x));     // all on their way before the first is used
        unroll([&](auto C) {
          constexpr int c = decltype(C)::value;
          acc = fma_4_rows<4 * c + 0>(qv, k[c].x, acc);
          acc = fma_4_rows<4 * c + 1>(qv, k[c].y, acc);
          acc = fma_4_rows<4 * c + 2>(qv, k[c].z, acc);
          acc = fma_4_rows<4 * c + 3>(qv, k[c].w, acc);
        }, std::make_integer_sequence<int, 4>{});
      }
      float* const e4 = er + 4 * g * EP;
      float zp[4], mx[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        zp[r] = acc[r] * a.scale;
        mx[r] = occ ? zp[r] : -INFINITY;
      }
      float x[4];
      auto four = [&](int j) {             // of column j, on their way before the first is used
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = e4[r * EP + j];
        asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
      };
#pragma unroll 1
      for (int j = lane; j < a.n_loc; j += 64) {
        four(j);
#pragma unroll
        for (int r = 0; r < 4; ++r) mx[r] = fmaxf(mx[r], x[r]);
      }
      wave_max4(mx);
      // the exponentials of a column's four rows, side by side; the slots' first
#pragma unroll
      for (int r = 0; r < 4; ++r) x[r] = zp[r];
      for (int j = occ ? at + 64 * nml : -1, next = lane;; j = next, next += 64) {
        if (j >= 0) {
          if (j < 64 * nml) four(j);
#pragma unroll
          for (int r = 0; r < 4; ++r) x[r] = pexp(x[r] - mx[r]);
          asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]));
#pragma unroll
          for (int r = 0; r < 4; ++r) e4[r * EP + j] = x[r];
        }
        if (next >= a.n_loc) break;
      }
    }
    // the rest reads what other lanes of this wave wrote, in LDS that no other wave touches: in order for the hardware, and so
    // for the compiler
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
    // the sums: lane l adds up row l % 4 of the wave's group l / 4 (rows beyond the last have a place in LDS as well)
    {
      const int r = 4 * (wave + NW * (lane >> 2)) + (lane & 3);
      if (r < rows) {
        const float* const row = er + r * EP;
#pragma unroll 8
        for (int j = 0; j < nP; ++j) s = s + row[64 * nml + j];
#pragma unroll 16
        for (int j = 0; j < a.n_loc; ++j) s = s + row[j];
      }
    }
    // the quotients of four rows side by side (padding rows as well, which nobody reads)
    auto sum_of = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(s), l)); };
#pragma unroll 1
    for (int g = wave, l = 0; 4 * g < rows; g += NW, l += 4) {
      const float* const e4 = er + 4 * g * EP;
#pragma unroll 1
      for (int u = lane; u < nP + a.n_evict; u += 64) {
        const float* const e = e4 + (u < nP ? 64 * nml + u : u - nP);
        float4 v;
        v.x = e[0] / sum_of(l);
        v.y = e[EP] / sum_of(l + 1);
        v.z = e[2 * EP] / sum_of(l + 2);
        v.w = e[3 * EP] / sum_of(l + 3);
        *reinterpret_cast<float4*>(A + (size_t)u * a.nqb_pad + r0 + 4 * g) = v;
      }
    }
  }
}

// Both for head h, in the lds_bytes at lds.  The matrix between them stays in LDS where it leaves the scores room, and goes
// through the workspace where not.
template <int D, int NT>
__device__ __forceinline__ void decide_body(const ScoreArgs& sa, const RetainArgs& ra, const int h, unsigned char* lds, const int lds_bytes) {
  const RetainPre<NT> pre = retain_prefetch<NT>(ra, h);
  const int a_bytes = (sa.C + sa.n_evict) * sa.nqb_pad * 4, used = (lds_bytes - a_bytes) & ~15;
  const bool fits = used >= (int)sizeof(RetainLds) && ScoreGeo<D>::rows(used, sa.C, sa.n_loc) >= min(sa.nqb_pad, 16);
  float* const A = fits ? reinterpret_cast<float*>(lds + used) : sa.A + (size_t)h * sa.nU_max * sa.nqb_pad;
  score_head_body<D, NT>(sa, h, lds, fits ? used : lds_bytes, A);
  __syncthreads();                         // the head's rows are written, and the scoring scratch is dead
  retain_body<NT>(ra, h, pre, A, fits, *reinterpret_cast<RetainLds*>(lds));
}

// The two argument blocks of the update's decisions, from the caller's pointers and the workspace
inline ScoreArgs make_score_args(const pbsa_params& p, const float* Qc, const float* Kc_l, const float* Zl,
                                 const float* Kc_p, const int32_t* p_len, const int32_t* l_map, const UpdateWs& ws) {
  return ScoreArgs{p.H, p.nqb, (p.nqb + 3) & ~3, p.n_loc, p.n_loc_cap, p.C, p.C + p.n_loc, p.n_evict, p.scale,
                   Kc_l, Kc_p, Qc, Zl, l_map, p_len, ws.A};
}
// A: the matrix whose row sums are the scores (the coarse matrix in the workspace, or the mass matrix), n_rows of it per head
inline RetainArgs make_retain_args(const pbsa_params& p, const float* A, int n_rows, int fine, const float* Kc_l,
                                   float* Kc_p, const int32_t* p_len, int64_t* p_id, int32_t* S_cnt, int fold,
                                   const int32_t* l_len, const int32_t* l_map, const int64_t* l_id, float* scores,
                                   int32_t* slot_src, const UpdateWs& ws) {
  return RetainArgs{p.H, p.nqb, (p.nqb + 3) & ~3, p.n_loc, p.n_loc_cap, p.C, p.n_sink, p.n_evict, n_rows, p.d, p.B,
                    fold, fine, p.Nq, A, Kc_l, Kc_p, p_len, ws.plen_new, p_id, S_cnt, l_len, l_map, l_id, scores,
                    slot_src, ws.fold_n, ws.fold_src, ws.fold_len, ws.promo_slot};
}

}  // namespace plan_dev
}  // namespace pbsa

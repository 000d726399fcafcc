// PBSA fine stage for launches with few query rows: one workgroup = W waves (2 or 4) = 64 consecutive query rows of one
// head, all in one query block, and the waves share out the keys.
//
// With 128 rows to a workgroup of two waves (pbsa_attention.hip) a chunk of a few hundred or thousand rows leaves most of the
// chip idle while every wave walks a whole list.  Here the tiles of the list -- every non-empty 64-key tile of the persistent
// slots, then of the selected local blocks, ascending -- are dealt to the waves in turn.  A wave brings its tiles through
// rings of its own (OwnRing) and meets the others only at the end, where the O^T of all of them, left in the place of
// their rings, are added up through LDS, weighted as their softmax references ask for.  No second launch, no scratch.
// parts > 1: the tiles are dealt to the waves of `parts` workgroups; combine_kernel puts those together.
//
// Bound by latency.  By time stamps, 5 heads x 1000 x 64 with 26 tiles: metadata 1.3 us, list 0.5, first loads and product
// 1.5, seven tiles 7.3, O^T to LDS 0.5, sum and output 0.9.  When a launch goes this way and what it gains: attn_team.
#include "pbsa_attention_device.h"

namespace pbsa {
namespace {

constexpr int kTeamTiles = 2 * (PBSA_MAX_C_ATTEND + 1) + 2 * PBSA_MAX_N_LOC;   // the longest list

template <int W>
struct TeamLds {
  unsigned char ring[W * 32 * 1024];                 // OwnRing of each wave; scratch of the workgroups that take decisions
  float2 ml[W * 64];                                 // per wave and row: softmax reference, sum of probabilities
  uint32_t list[W][(kTeamTiles + W - 1) / W];        // bit 31: local, bits 7..: slot * (B / 64) + tile of it, bits 0..6: valid keys
  uint32_t blk[PBSA_MAX_C_ATTEND + 1 + PBSA_MAX_N_LOC];   // slots 0 .. C, then the local blocks: physical slot << 8 | length
  uint32_t picked[(PBSA_MAX_N_LOC + 31) / 32];       // the local blocks that the query block selected
};
static_assert(sizeof(TeamLds<4>) <= 160 * 1024 && 2 * sizeof(TeamLds<2>) <= 160 * 1024, "four waves on a compute unit");

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wuninitialized"
// PLAN: as in attention_kernel, workgroups ahead of the others that take the decisions of the memory update.
template <int D, int W, bool MASS, bool PLAN>
__global__ void __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(1, 1)))
attention_team_kernel(AttnArgs a, PlanArgs<PLAN> pl) {
  using R = OwnRing<D>;
  constexpr int NT = 64 * W, N = R::N;
  constexpr int KS = Geo<D>::KS, DT = Geo<D>::DT, ROW = Geo<D>::ROW, SUB1 = Geo<D>::SUB_BYTES;
  constexpr int CH = D / 8, RPI = 64 / CH, NIW = DmaPlan<D>::NIW;
  __shared__ __align__(1024) TeamLds<W> L;

  const int n_plan = PLAN ? 8 * ((a.H + 7) / 8) : 0;
  if constexpr (PLAN) {
    if ((int)blockIdx.x < n_plan) {
      const int hp = (int)blockIdx.x;
      if (hp >= a.H) return;
      static_assert(plan_dev::score_fits<D>(sizeof(L.ring)) && sizeof(plan_dev::RetainLds) <= sizeof(L.ring), "scratch must fit");
      plan_dev::decide_body<D, NT>(pl.sa, pl.ra, hp, L.ring, sizeof(L.ring));
      return;
    }
  }
  // consecutive workgroup ids go round-robin to the 8 XCDs: each XCD takes a contiguous range of (unit, part) pairs
  const int bx = (int)blockIdx.x - n_plan;
  const int n_ut = (a.Nq + 63) / 64, nu = a.H * n_ut * a.parts;
  const int lu = (bx % 8) * ((nu + 7) / 8) + bx / 8;
  if (bx / 8 >= (nu + 7) / 8 || lu >= nu) return;
  const int unit = lu / a.parts, part = lu % a.parts;
  const int h = unit / n_ut, T0 = (unit % n_ut) * 64;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int qn = lane & 31, half = lane >> 5;
  const int sub_bits = a.B == 128 ? 1 : 0;           // 64-key tiles per block, as a shift

  // ---- metadata: one parallel round; the queries behind it ----------------------------------------
  constexpr int kLocPer = 512 / NT, kPersPer = 128 / NT > 0 ? 128 / NT : 1, kSelPer = 256 / NT;
  const int32_t* const sel_row = a.sel + ((size_t)h * a.nqb + T0 / a.B) * a.k;
  const int32_t* const plen_h = a.p_len + (size_t)h * (a.C + 1);
  if (tid < (int)(sizeof(L.picked) / 4)) L.picked[tid] = 0;
  int llen_v[kLocPer], lmap_v[kLocPer], plen_v[kPersPer], selv[kSelPer];
#pragma unroll
  for (int u = 0; u < kLocPer; ++u) {
    const int l = min(tid + u * NT, a.n_loc - 1);
    llen_v[u] = a.l_len[l];
    lmap_v[u] = a.l_map[l];
  }
#pragma unroll
  for (int u = 0; u < kPersPer; ++u) plen_v[u] = plen_h[min(tid + u * NT, a.C)];
#pragma unroll
  for (int u = 0; u < kSelPer; ++u) selv[u] = tid + u * NT < a.k ? sel_row[tid + u * NT] : -1;
  const int tok0 = T0 + qn;                // row group g holds token tok0 + 32 g
  bf16x8 qf[2][KS];
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const bf16_t* qrow = a.Q + (size_t)h * a.q_stride_h + (size_t)min(tok0 + 32 * g, a.Nq - 1) * a.q_stride_t + 8 * half;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[g][ks] = *reinterpret_cast<const bf16x8*>(qrow + 16 * ks);
  }
  __syncthreads();                         // the marks are clear
  auto put_local = [&](int l, int slot, int len) {
    if (l < a.n_loc) L.blk[a.C + 1 + l] = (unsigned)slot < (unsigned)a.n_loc_cap ? ((uint32_t)slot << 8) | (uint32_t)min(max(len, 0), a.B) : 0u;
  };
  auto put_slot = [&](int c, int len) {
    if (c <= a.C) L.blk[c] = ((uint32_t)c << 8) | (uint32_t)min(max(len, 0), a.B);
  };
  auto pick = [&](int l) {
    if (l >= 0 && l < a.n_loc) atomicOr(&L.picked[l >> 5], 1u << (l & 31));
  };
#pragma unroll
  for (int u = 0; u < kLocPer; ++u) put_local(tid + u * NT, lmap_v[u], llen_v[u]);
#pragma unroll 1
  for (int l = tid + kLocPer * NT; l < a.n_loc; l += NT) put_local(l, a.l_map[l], a.l_len[l]);
#pragma unroll
  for (int u = 0; u < kPersPer; ++u) put_slot(tid + u * NT, plen_v[u]);
#pragma unroll 1
  for (int c = tid + kPersPer * NT; c <= a.C; c += NT) put_slot(c, plen_h[c]);
#pragma unroll
  for (int u = 0; u < kSelPer; ++u) pick(selv[u]);
#pragma unroll 1
  for (int j = tid + kSelPer * NT; j < a.k; j += NT) pick(sel_row[j]);
  __syncthreads();

  // ---- this wave's tiles: every wave looks at all blocks, 64 at a time, and keeps its own ---------
  const int share = part * W + wave, n_shares = W * a.parts;
  const size_t rec = (size_t)(h * ((a.Nq + 127) / 128) + T0 / 128) * 2 + (T0 / 64) % 2;     // MASS: MassRows' 64 rows
  int32_t* const rlist = MASS ? a.Rlist + rec / 2 * a.list_cap : nullptr;
  int n_all = 0;
  const int n_cand = a.C + 1 + a.n_loc;
  const uint32_t inv_parts = (65536u + (uint32_t)a.parts - 1) / (uint32_t)a.parts;   // q / parts for q <= kTeamTiles, parts <= kMaxParts
  static_assert(kTeamTiles * (kMaxParts - 1) < 65536, "the quotient is exact");
#pragma unroll 1
  for (int r0 = 0; r0 < n_cand; r0 += 64) {
    const int c = r0 + lane, l = c - (a.C + 1);
    int len = 0;
    uint32_t src = 0;
    if (c < n_cand) {
      const uint32_t w = L.blk[c];
      const bool on = l < 0 || ((L.picked[l >> 5] >> (l & 31)) & 1u);
      len = on ? (int)(w & 0xFFu) : 0;
      src = ((w >> 8) << (7 + sub_bits)) | (l < 0 ? 0u : 0x80000000u);
    }
    const unsigned long long m1 = __ballot(len > 0), m2 = __ballot(len > 64);
    const int q0 = n_all + lanes_below(m1) + lanes_below(m2);
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      const int q = q0 + s, tl = min(len - 64 * s, 64);
      if (tl > 0) {
        if constexpr (MASS) {              // the later pass walks the whole list, whoever walked its tiles
          if (share == 0 && q < a.list_cap - 4)
            reinterpret_cast<uint16_t*>(rlist + 4)[(rec % 2) * (a.list_cap - 4) + q] = (uint16_t)(c << 1 | s);
        }
        if (q % W == wave) {
          const uint32_t r = (uint32_t)(q / W), at = (r * inv_parts) >> 16;
          if (r - at * (uint32_t)a.parts == (uint32_t)part) L.list[wave][at] = src | ((uint32_t)s << 7) | (uint32_t)tl;
        }
      }
    }
    n_all += __popcll(m1) + __popcll(m2);
  }
  // tile q of the list goes to wave q % W of part q / W % parts
  int n = 0;
  {
    const int rows_w = (n_all - wave + W - 1) / W;   // tiles of waves of this number, over all parts
    n = rows_w > part ? (rows_w - part + a.parts - 1) / a.parts : 0;
  }
  n = __builtin_amdgcn_readfirstlane(n);
  asm volatile("" ::: "memory");
  // The Q fragments are only ever MFMA operands: keep them in the accumulator half of the register file.
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(qf[g][ks]));

  f32x16 o[2][DT];
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
      for (int v = 0; v < 16; ++v) o[g][dt][v] = 0.0f;
      asm volatile("" : "+a"(o[g][dt]));
    }
  f32x16 sA[2], sB[2];                     // S^T of even / odd half tiles
  PTile pA, pB;                            // P^T of even / odd half tiles (bf16 pairs)
  const float c2 = a.scale * 1.4426950408889634f, lift = kLift / c2;
  SoftmaxRun sr{{kInitMax, kInitMax}, {-kInitMax * c2, -kInitMax * c2}, {0.0f, 0.0f, 0.0f, 0.0f},
                {sum_selector(lane, 0), sum_selector(lane, 1)}, 0ull, c2, lift, false};
  MassOut mo{nullptr, 0, 64 * n_shares, lane, lane >= 32, 0.0f, 0.0f};
  if constexpr (MASS) {
    if (share == 0 && lane == 0) rlist[rec % 2] = n_all;
    // (the first step's product of nothing leaves a record too: where the first tile's will be)
    mo.rp = a.R + (rec * a.r_slots + part * W + wave) * 64;
  }

  const uint32_t ring_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)L.ring;
  const uint32_t kring = __builtin_amdgcn_readfirstlane(ring_lds + wave * R::WAVE_BYTES), vring = kring + R::RING_BYTES;
  if (n > 0) {
    bf16x8 frag[2 * KS];
    const int lim0[2] = {0, 0};
    // ---- operand addresses, as in attention_kernel: K in ring entry 0, V two entries on where there are four ------
    uint32_t kx[KS], vx[DT];
    {
      const int kb = qn * ROW + ((half ^ k_swz<D>(qn)) << 4);
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        kx[ks] = kring + (uint32_t)(kb ^ (ks << 5));
        asm volatile("" : "+v"(kx[ks]));
      }
      const int s16 = lane & 15, q16 = (lane >> 4) & 1;
      const int v_row0 = 4 * half + (s16 >> 2);
      const int v_sub = 2 * q16 + ((s16 & 3) >> 1), v_lo = (s16 & 1) * 8;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        vx[dt] = vring + (N == 4 ? 2 * SUB1 : 0) + (uint32_t)(v_row0 * ROW + (((4 * dt + v_sub) ^ v_swz<D>(v_row0)) << 4) + v_lo);
        asm volatile("" : "+v"(vx[dt]));
      }
    }
    // ---- staging ------------------------------------------------------------------------------
    const int rl = lane / CH, vchk = ((lane % CH) ^ v_swz<D>(rl)) << 4;
    DmaPlan<D> plan;
#pragma unroll
    for (int k = 0; k < 4; ++k) plan.kpat[k] = rl * ROW + (((lane % CH) ^ k_swz<D>(RPI * k + rl)) << 4);
    plan.vpat = rl * ROW + vchk;
    plan.vragged = false;
#pragma unroll
    for (int i = 0; i < NIW; ++i) plan.voff[i] = 0;
    const unsigned char* const kl = reinterpret_cast<const unsigned char*>(a.Kl) + (size_t)h * a.n_loc_cap * a.B * ROW;
    const unsigned char* const vl = reinterpret_cast<const unsigned char*>(a.Vl) + (size_t)h * a.n_loc_cap * a.B * ROW;
    const unsigned char* const kp = reinterpret_cast<const unsigned char*>(a.Kp) + (size_t)h * (a.C + 1) * a.B * ROW;
    const unsigned char* const vp = reinterpret_cast<const unsigned char*>(a.Vp) + (size_t)h * (a.C + 1) * a.B * ROW;
    const uint32_t* const list = L.list[wave];
    // the plan that brings half HALF of tile KD of K into K ring entry KENTRY, and of tile VD of V into V entry VENTRY
#define PBSA_OWN_K(KD, HALF, KENTRY)                                                                    \
  {                                                                                                     \
    plan.kp = ((KD) >> 31 ? kl : kp) + (size_t)(((KD) & 0x7FFFFFFFu) >> 7) * (kTile * ROW) + (HALF) * SUB1; \
    plan.klds = kring + (KENTRY) * SUB1;                                                                \
  }
#define PBSA_OWN_V(VD, HALF, VENTRY)                                                                    \
  {                                                                                                     \
    plan.vtile = ((VD) >> 31 ? vl : vp) + (size_t)(((VD) & 0x7FFFFFFFu) >> 7) * (kTile * ROW);           \
    plan.vp = plan.vtile + (HALF) * SUB1;                                                               \
    plan.vlds = vring + (VENTRY) * SUB1;                                                                \
  }
    // rows past the valid length of a V tile must not reach LDS (p = 0 times whatever they hold): the last valid row instead
#define PBSA_OWN_VRAGGED(VD, HALF)                                                                      \
  {                                                                                                     \
    int last_ = (int)((VD) & 127u) - 1;                                                                 \
    plan.vragged = last_ < kTile - 1;                                                                   \
    if (plan.vragged) {                                                                                 \
      /* (an address register is left alone until the load that uses it is back) */                     \
      asm volatile("s_waitcnt vmcnt(0)" : "+s"(last_) : : "memory");                                    \
      _Pragma("unroll") for (int i_ = 0; i_ < NIW; ++i_)                                                \
        plan.voff[i_] = min(32 * (HALF) + RPI * i_ + rl, last_) * ROW + vchk;                           \
    }                                                                                                   \
  }
    // keys of half HALF of the tile that do not exist: a score below all others
#define PBSA_OWN_MASK(S, DESC, HALF)                                                                    \
  {                                                                                                     \
    const int valid_ = (int)((DESC) & 127u) - 32 * (HALF);                                              \
    if (valid_ < 32) {                                                                                  \
      const int lim_ = valid_ - 4 * half;                                                               \
      _Pragma("unroll") for (int g_ = 0; g_ < 2; ++g_)                                                  \
        _Pragma("unroll") for (int v_ = 0; v_ < 16; ++v_)                                               \
          if (8 * (v_ / 4) + (v_ % 4) >= lim_) S[g_][v_] = kMasked;                                     \
    }                                                                                                   \
  }
    auto tile = [&](int t) -> uint32_t { return (uint32_t)__builtin_amdgcn_readfirstlane((int)list[min(t, n - 1)]); };
    // ---- the halves the first steps need, in the order they need them ---------------------------
    uint32_t d_cur = tile(0), d_k = tile(N / 2), d_v = tile(N / 2 - 1);   // tile walked; those whose K / V are loaded next
    uint32_t d_next = d_cur;
    int d_ahead = (int)list[min(N / 2 + 1, n - 1)];
    PBSA_OWN_K(d_cur, 0, 0)
    dma_all<D>(plan, true, false);
    PBSA_OWN_K(d_cur, 1, 1)
    dma_all<D>(plan, true, false);
    if constexpr (N == 4) {
      const uint32_t d1 = tile(1);
      PBSA_OWN_V(d_cur, 0, 0)
      PBSA_OWN_VRAGGED(d_cur, 0)
      PBSA_OWN_K(d1, 0, 2)
      dma_all<D>(plan, true, true);
      PBSA_OWN_V(d_cur, 1, 1)
      PBSA_OWN_VRAGGED(d_cur, 1)
      PBSA_OWN_K(d1, 1, 3)
      dma_all<D>(plan, true, true);
    }
    // The first step has the product of the half tile before it as all others do, with probabilities of zero; the V it
    // meets is zero as well (one step without a second product would be a kilobyte of code more to fetch).
    {
      typedef __attribute__((address_space(3))) u32x4* lds_w_t;
      const u32x4 z = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int i = 0; i < SUB1 / 1024; ++i) *(lds_w_t)(uintptr_t)(vring + (N - 1) * SUB1 + i * 1024 + lane * 16) = z;
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int e = 0; e < 4; ++e) pB[g][j][e] = 0u;
    }
    NoMid nomid;
    typedef StepKind<true, true, SUB1, SUB1> KindA;          // first half of a tile: K one entry on, V one entry back
    typedef StepKind<true, true, 0, 0> KindB;                // second half
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((N == 4 ? 5 : 1) * NIW) : "memory");
    step<D, false, false, false, kNoLoads, StepKind<false, true, 0, 0>, false, kNextNone, void, NoMid>(
        vx, kx, qf, o, sB, sA, pB, pA, sr, lim0, plan, mo, frag, 0, 0, nomid);
    PBSA_OWN_MASK(sA, d_cur, 0)
    seed_reference(sA, sr);
    // loads of the steps of tile t: K of tile t + N / 2, V of tile t + N / 2 - 1, half by half
    PBSA_OWN_K(d_k, 0, 0)
    PBSA_OWN_V(d_v, 0, N == 4 ? 2 : 0)
    PBSA_OWN_VRAGGED(d_v, 0)
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((N == 4 ? 4 : 0) * NIW) : "memory");
    preload_frags<D, KindA>(frag, vx, kx);
    for (int t = 0; t < n; ++t) {
      const int odd = t & 1, flip = N == 4 ? (odd ? -2 * SUB1 : 2 * SUB1) : 0;
      auto mid_a = [&](auto piece) {       // behind the loads of the first half: the plan of the second
        constexpr int pc = decltype(piece)::value;
        if constexpr (pc == 0) {
          plan.kp += SUB1;
          plan.klds += SUB1;
        }
        if constexpr (pc == 1) {
          plan.vp += SUB1;
          plan.vlds += SUB1;
        }
        if constexpr (pc == 2) PBSA_OWN_VRAGGED(d_v, 1)
        if constexpr (pc == 3) d_next = (uint32_t)(N == 4 ? d_v : d_k);
      };
      step<D, MASS, true, false, kLoads, KindA, true, N == 4 ? kNextOwnMove : kNextOwn, KindB, decltype(mid_a)>(
          vx, kx, qf, o, sA, sB, pA, pB, sr, lim0, plan, mo, frag, flip, -flip, mid_a);
      PBSA_OWN_MASK(sB, d_cur, 1)
      auto mid_b = [&](auto piece) {       // and of the first half of the next tile
        constexpr int pc = decltype(piece)::value;
        if constexpr (pc == 0) {
          d_v = d_k;
          d_k = (uint32_t)__builtin_amdgcn_readfirstlane(d_ahead);
        }
        if constexpr (pc == 1) PBSA_OWN_K(d_k, 0, N == 4 && !odd ? 2 : 0)
        if constexpr (pc == 2) PBSA_OWN_V(d_v, 0, N == 4 && odd ? 2 : 0)
        if constexpr (pc == 3) PBSA_OWN_VRAGGED(d_v, 0)
        if constexpr (pc == 4) d_ahead = (int)list[min(t + N / 2 + 2, n - 1)];
      };
      step<D, MASS, true, false, kLoads, KindB, true, kNextOwn, KindA, decltype(mid_b)>(
          vx, kx, qf, o, sB, sA, pB, pA, sr, lim0, plan, mo, frag, 0, 0, mid_b);
      d_cur = d_next;
      PBSA_OWN_MASK(sA, d_cur, 0)
    }
    step<D, MASS, false, false, kNoLoads, StepKind<true, false, 0, SUB1>, false, kNextNone, void, NoMid>(
        vx, kx, qf, o, sA, sB, pA, pB, sr, lim0, plan, mo, frag, 0, 0, nomid);
    // between runs the compiler may copy the accumulators to other registers: let the matrix pipe drain first
    acc_settle<DT>(o[0]);
    acc_settle<DT>(o[1]);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the trailing loads land before their place is used again
  }
  acc_settle<DT>(o[0]);
  acc_settle<DT>(o[1]);
  sum_settle(sr.l_run);

  // ---- the waves' O^T, in the accumulators' own order (1 KiB pieces [row group][DT][4][lane][4]), added up --------
  unsigned char* const mine = L.ring + wave * R::WAVE_BYTES;
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *reinterpret_cast<float4*>(mine + ((g * DT + dt) * 4 + q4) * 1024 + lane * 16) =
            make_float4(o[g][dt][4 * q4], o[g][dt][4 * q4 + 1], o[g][dt][4 * q4 + 2], o[g][dt][4 * q4 + 3]);
  L.ml[wave * 64 + lane] = make_float2(lane < 32 ? sr.m_ref[0] : sr.m_ref[1], sr.l_run[0]);
  __syncthreads();
  // wave w: row group w / (W / 2), an equal share of its pieces
  constexpr int WG2 = W / 2, PER = DT * 4 / WG2;
  const int g = wave / WG2, p0 = (wave % WG2) * PER, row = 32 * g + qn;
  float wgt[W], m_all = kInitMax, l_tot = 0.0f;
  float2 ml[W];
#pragma unroll
  for (int j = 0; j < W; ++j) {
    ml[j] = L.ml[j * 64 + row];
    if (ml[j].y != 0.0f) m_all = fmaxf(m_all, ml[j].x);
  }
#pragma unroll
  for (int j = 0; j < W; ++j) {
    wgt[j] = ml[j].y != 0.0f ? __builtin_amdgcn_exp2f((ml[j].x - m_all) * c2) : 0.0f;
    l_tot = __builtin_fmaf(wgt[j], ml[j].y, l_tot);
  }
  const int tok = T0 + row;
  const bool split = a.parts > 1, writes_row = p0 == 0 && half == 0;
  const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
  const size_t slot = (size_t)unit * a.parts + part;
  float* const po = a.part_o + slot * (64 * D) + lane * 4;
  bf16_t* const orow = a.O + (size_t)h * a.o_stride_h + (size_t)min(tok, a.Nq - 1) * a.o_stride_t + 4 * half;
#pragma unroll
  for (int i = 0; i < PER; ++i) {
    const int piece = g * (DT * 4) + p0 + i;
    float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int j = 0; j < W; ++j) {
      const float4 v = *reinterpret_cast<const float4*>(L.ring + j * R::WAVE_BYTES + piece * 1024 + lane * 16);
      acc.x = __builtin_fmaf(wgt[j], v.x, acc.x);
      acc.y = __builtin_fmaf(wgt[j], v.y, acc.y);
      acc.z = __builtin_fmaf(wgt[j], v.z, acc.z);
      acc.w = __builtin_fmaf(wgt[j], v.w, acc.w);
    }
    if (split) {
      *reinterpret_cast<float4*>(po + piece * 256) = acc;
    } else if (tok < a.Nq) {
      bf16x4 w;
      w[0] = (__bf16)(acc.x * inv);
      w[1] = (__bf16)(acc.y * inv);
      w[2] = (__bf16)(acc.z * inv);
      w[3] = (__bf16)(acc.w * inv);
      *reinterpret_cast<bf16x4*>(orow + 8 * (p0 + i)) = w;       // piece p0 + i: columns 32 dt + 8 q4 + 4 half ..
    }
  }
  if (writes_row) {
    if (split) *reinterpret_cast<float2*>(a.part_ml + (slot * 64 + row) * 2) = make_float2(m_all, l_tot);
    else if (a.lse && tok < a.Nq) a.lse[(size_t)h * a.Nq + tok] = l_tot > 0.0f ? m_all * a.scale + __logf(l_tot) : -INFINITY;
  }
}
#pragma clang diagnostic pop

}  // namespace

template <int D, int W, bool MASS, bool PLAN>
static hipError_t launch_t(const AttnArgs& a, const PlanArgs<PLAN>& pl, int n_plan, hipStream_t stream) {
  const int nu = a.H * ((a.Nq + 63) / 64) * a.parts;
  hipLaunchKernelGGL((attention_team_kernel<D, W, MASS, PLAN>), dim3(n_plan + 8 * ((nu + 7) / 8)), dim3(64 * W), 0, stream, a, pl);
  return hipGetLastError();
}

template <bool MASS, bool PLAN>
hipError_t launch_attention_team(const pbsa_params& p, const AttnArgs& a, const PlanArgs<PLAN>& pl, int waves, int n_plan, hipStream_t stream) {
  if (p.d == 128)
    return waves == 4 ? launch_t<128, 4, MASS, PLAN>(a, pl, n_plan, stream) : launch_t<128, 2, MASS, PLAN>(a, pl, n_plan, stream);
  return waves == 4 ? launch_t<64, 4, MASS, PLAN>(a, pl, n_plan, stream) : launch_t<64, 2, MASS, PLAN>(a, pl, n_plan, stream);
}
template hipError_t launch_attention_team<false, false>(const pbsa_params&, const AttnArgs&, const PlanArgs<false>&, int, int, hipStream_t);
template hipError_t launch_attention_team<true, false>(const pbsa_params&, const AttnArgs&, const PlanArgs<false>&, int, int, hipStream_t);
template hipError_t launch_attention_team<false, true>(const pbsa_params&, const AttnArgs&, const PlanArgs<true>&, int, int, hipStream_t);

}  // namespace pbsa

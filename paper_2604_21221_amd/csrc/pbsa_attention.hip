// PBSA fine stage (Eq. 3-5) for gfx950: block-sparse flash attention on bf16 MFMA.
//
// One workgroup = 2 waves = 128 consecutive query tokens of one head (one query block when B = 128,
// two when B = 64).  Wave w owns rows 64 w .. 64 w + 63 of the workgroup as two row groups of 32, so
// with B = 64 a wave is exactly one query block.  Two workgroups share a CU, one wave per SIMD, so a
// wave has the whole 512-entry register file of its SIMD.
//
// The workgroup walks a list of 64-key tiles: every non-empty persistent slot (the dense part of the
// mask, visible to all rows) and the union of the local blocks selected by its query blocks, sorted by
// who attends a tile:
//   shared  full tiles both waves attend, then the ragged tiles (fewer than 64 valid keys, masked per
//           wave).  The waves stage each tile together, two tiles per operand in flight, and meet at a
//           barrier once per tile.
//   solo    full tiles only one wave attends (B = 64: a block one query block selected and its
//           neighbour did not).  After the shared part each wave streams its own tiles through its own
//           half of the LDS in 32-key halves, with no barrier: both waves run at full width on different
//           tiles, and since every query block selects the same number of blocks the two waves, and all
//           workgroups, have the same amount of work however the selections overlap.
// The order of keys does not matter to an online softmax.  K/V tiles go from global memory straight
// into LDS (global_load_lds, no register round trip).
//
// MFMA arrangement (v_mfma_f32_32x32x16_bf16, wave64):
//   S^T = K Q^T   A = K tile rows (32 keys x 16 dims), B = Q^T (16 dims x 32 query rows).
//                 The accumulator then holds, per lane, 16 keys of ONE query row (column lane%32),
//                 so the softmax row reductions are in-lane plus one exchange with lane^32.
//   O^T = V^T P^T A = V^T (32 dims x 16 keys), B = P^T (16 keys x 32 query rows) taken straight
//                 from the S^T accumulators: the contraction index (key) is enumerated in the order
//                 the accumulator holds it, and V^T is read from LDS with the same enumeration.
//   A K or V^T fragment read from LDS feeds the MFMAs of both row groups, which halves the LDS
//   traffic per flop.  (At one fragment per MFMA -- 32 rows per wave, two waves per SIMD -- four matrix
//   pipes ask the LDS for 128 bytes per clock, about half of what it delivers to reads alone; with the
//   staging loads and the barrier beside them that arrangement measured no faster in a probe, and it
//   needs the whole step in 256 registers.)
//
// Software pipeline.  The unit is a sub-tile of 32 keys.  In step u a wave runs, as one straight
// stretch of code cut into slots (one MFMA plus a slice of vector work each), the softmax of
// sub-tile u (one fma and one exp2 per score, one conversion per pair; S^T(u) -> P^T(u)) together with
// the MFMAs that do not depend on it: O^T += V^T P^T of sub-tile u-1 and S^T = K Q^T of sub-tile u+1.
// S^T and P^T are double buffered.  Each part of the list (shared full, shared ragged, solo) is one
// pipelined run with its own template instance; the pipeline drains between them.  Softmax is online,
// fp32, base 2 (scale and log2 e folded into one fma), against a reference that a step takes as given.
// The row sums (over the bf16-rounded probabilities, the numbers the second product uses) are four small
// MFMAs per step whose A operand selects the rows (sum_mfma); the check that the reference still serves is
// one OR per two pairs inside the slots and one compare at the end of the step, and the rare step that
// fails it is redone in place (softmax_redo).  A step loads the first operand fragments of the step after
// it during its last slots and hands them over in registers, so no step starts by waiting for LDS; the
// barrier that turns the rings over sits in the middle of a tile's second step, under its MFMAs.
#include "pbsa_attention_device.h"

namespace pbsa {
namespace {

#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Wuninitialized"
// PLAN: the grid has H more workgroups ahead of those of the attention, one per head, which take the decisions of
// the memory update (Eq. 7-9: scoring, retention, slot assignment) while the attention runs.  They read the
// cache's metadata and pooled keys and what the selection call left, never K / V or the attention's output, and
// a one-round launch leaves them SIMDs to run on (two workgroups per CU, 128 rows each: at 4680 rows and 12
// heads 444 of 512 places are taken).
//
// SPLIT: the workgroups of the last round -- all of them where the launch has less than one -- are shared out over the
// places that round would leave empty: the tile list of a query tile goes to `parts` workgroups, an equal share of
// every class to each, which leave O^T unnormalised with its reference and sum to combine_kernel (attn_split).
template <int D, int B, bool MASS, bool PLAN, bool SPLIT>
__global__ void __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(1, 1)))
attention_kernel(AttnArgs a, PlanArgs<PLAN> pl) {
  constexpr int G = kRowsPerWg / B;        // query blocks per workgroup
  constexpr int SUB = B / kTile;           // 64-key tiles per block
  constexpr int KS = Geo<D>::KS, DT = Geo<D>::DT, TILE = Geo<D>::TILE_BYTES, ROW = Geo<D>::ROW;
  constexpr int SUB1 = Geo<D>::SUB_BYTES;
  constexpr int CH = D / 8, RPI = 64 / CH;          // 16-byte chunks per row, rows per wave instruction
  constexpr int NIW = (kTile / RPI) / 2;            // global_load_lds instructions per wave per tile
  // K ring (2 tiles), V ring (2 tiles); the decisions' workgroups have use for more than d = 64 needs
  constexpr int SMEM = PLAN ? 64 * 1024 : 4 * TILE;
  static_assert(PBSA_MAX_N_LOC * 8 + (PBSA_MAX_C_ATTEND + 1 + 8) * 4 <= SMEM, "setup scratch must fit");
  // the plain call takes the larger limits and keeps the list within two workgroups' share of a CU's LDS by
  // storing 16-bit descriptors (the mass variant's carry the key block as well)
  constexpr bool kAux = MASS || PLAN;
  constexpr int kTilesMax = kAux ? kMaxTilesAux : kMaxTiles;
  constexpr int kLocMax = kAux ? PBSA_MAX_N_LOC_AUX : PBSA_MAX_N_LOC;
  using meta_t = std::conditional_t<kAux, int, uint16_t>;

  __shared__ __align__(1024) unsigned char smem[SMEM];
  __shared__ int t_src[kTilesMax];         // bit 31: local, bits 0..: (slot * SUB + sub)
  __shared__ meta_t t_meta[kTilesMax];     // valid keys (bits 0..7) | waves that attend (bits 8, 9)
  // setup scratch, dead before the first tile is staged: per local block its physical slot and, in one word, its length
  // (0: it is nowhere) and from bit 16 the waves that attend it; the slots' lengths; each wave's counts
  int2* lblk = reinterpret_cast<int2*>(smem);

  // XCD-aware mapping: consecutive workgroup ids go round-robin to the 8 XCDs, so give XCD x the
  // contiguous range [x * per, (x+1) * per) of (head, query tile) pairs: neighbours share K/V in L2.
  const int n_qt = (a.Nq + kRowsPerWg - 1) / kRowsPerWg;
  const int n_wg = a.H * n_qt;
  const int per = (n_wg + 7) / 8;
  // the workgroups that take the decisions come first in the grid (whole rows of 8, so that the XCD of the others is
  // still their index mod 8): they start with the launch however many rounds the attention needs
  const int n_plan = PLAN ? 8 * ((a.H + 7) / 8) : 0;
  if constexpr (PLAN) {
    if ((int)blockIdx.x < n_plan) {
      const int hp = (int)blockIdx.x;
      if (hp >= a.H) return;
      static_assert(plan_dev::score_fits<D>(SMEM) && sizeof(plan_dev::RetainLds) <= SMEM, "scratch must fit");
      plan_dev::decide_body<D, kThreads>(pl.sa, pl.ra, hp, smem, SMEM);
      return;
    }
  }
  const int bx = (int)blockIdx.x - n_plan;
  int logical, part = 0, n_parts = 1;
  if constexpr (SPLIT) {
    if (bx < a.n_full) {                   // a whole number of rounds
      logical = (bx % 8) * (a.n_full / 8) + bx / 8;
    } else {
      const int nu = (n_wg - a.n_full) * a.parts, u = bx - a.n_full, lu = (u % 8) * ((nu + 7) / 8) + u / 8;
      if (u / 8 >= (nu + 7) / 8 || lu >= nu) return;
      logical = a.n_full + lu / a.parts;
      part = lu % a.parts;
      n_parts = a.parts;
    }
  } else {
    logical = (bx % 8) * per + bx / 8;
    if (logical >= n_wg) return;
  }
  const int h = logical / n_qt;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int T0 = (logical % n_qt) * kRowsPerWg;
  const int i0 = T0 / B;
  const int qn = lane & 31, half = lane >> 5;

  // ---- tile list --------------------------------------------------------------------------------
  // Everything the list needs is fetched from global memory in one parallel round into LDS scratch:
  // per local block the set of waves whose query block selected it, its length and its physical slot;
  // per persistent slot its length.  The candidates -- the 64-key tiles of the persistent slots, then
  // of the local blocks, in ascending order -- are then classified 64 at a time, the first half of them by wave 0: full
  // tiles of both waves, ragged tiles, full tiles of wave 0 only, of wave 1 only.  Every part of the list is in ascending
  // candidate order.  With each wave sweeping all candidates, three LDS words each, and a division per selected block in a
  // loop unrolled for the largest shape the list took 3.4 us of a launch of 12 heads x 4680 rows, now 2.1 (four denoising
  // passes at 8 + 16 blocks of 128 497.9 -> 485.7 us, select, forward and backward of 3 x 1500 x 64 44.8 -> 43.4; nothing
  // beyond noise in a chained step, whose launch holds the decisions too: 111.3 -> 109.7 and, at 32 + 48 blocks of 64,
  // 175.0 -> 175.5).
  int* plen_s = reinterpret_cast<int*>(lblk + kLocMax);
  int* cnt_s = plen_s + PBSA_MAX_C_ATTEND + 1;
  // The first of each are fetched together (up to 384 local blocks, 128 slots, 256 selected blocks); the rest, at shapes beyond
  // those, in loops of their own: this code runs once per workgroup, and instructions that have to be fetched cost more than
  // the loads they issue (the same list with everything unrolled gained nothing, and a step of 2 x 256 x 64 lost 1 us).
  constexpr int kLocPer = 3, kSelPer = 2;
  const int n_sel = G * a.k;
  const int32_t* const sel_wg = a.sel + ((size_t)h * a.nqb + i0) * a.k;         // the rows lie one behind the other
  const int32_t* const plen_h = a.p_len + (size_t)h * (a.C + 1);
  const int n_sel_here = G == 1 || i0 + 1 < a.nqb ? n_sel : a.k;
  int llen_v[kLocPer], lmap_v[kLocPer], selv[kSelPer];
  // (loads return in order: anything asked for after the queries would wait for them)
#pragma unroll
  for (int u = 0; u < kLocPer; ++u) {
    const int l = min(tid + u * kThreads, a.n_loc - 1);
    llen_v[u] = a.l_len[l];
    lmap_v[u] = a.l_map[l];
  }
  const int plen_v = plen_h[min(tid, a.C)];
#pragma unroll
  for (int u = 0; u < kSelPer; ++u) selv[u] = tid + u * kThreads < n_sel_here ? sel_wg[tid + u * kThreads] : -1;

  // ---- Q fragments (B operand of S^T = K Q^T): row group g, query row lane % 32, dims 16 ks + 8 (lane/32) ..+8.
  // Issued after the few loads the tile list waits for and not touched until the list is built: the
  // chunk's queries come from HBM while every workgroup of the launch asks for its own at the same time.
  const int tok0 = T0 + wave * 64 + qn;                 // row group g holds token tok0 + 32 g
  bf16x8 qf[2][KS];
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    const int tok_c = min(tok0 + 32 * g, a.Nq - 1);
    const bf16_t* qrow = a.Q + (size_t)h * a.q_stride_h + (size_t)tok_c * a.q_stride_t + 8 * half;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qf[g][ks] = *reinterpret_cast<const bf16x8*>(qrow + 16 * ks);
  }
  auto put_block = [&](int l, int slot, int len) {
    if (l < a.n_loc) lblk[l] = make_int2(slot, (unsigned)slot < (unsigned)a.n_loc_cap ? min(max(len, 0), B) : 0);
  };
#pragma unroll
  for (int u = 0; u < kLocPer; ++u) put_block(tid + u * kThreads, lmap_v[u], llen_v[u]);
#pragma unroll 1
  for (int l = tid + kLocPer * kThreads; l < a.n_loc; l += kThreads) put_block(l, a.l_map[l], a.l_len[l]);
  if (tid <= a.C) plen_s[tid] = min(max(plen_v, 0), B);
#pragma unroll 1
  for (int c = tid + kThreads; c <= a.C; c += kThreads) plen_s[c] = min(max(plen_h[c], 0), B);
  __syncthreads();
  auto flag = [&](int idx, int l) {        // with one query block per workgroup both waves belong to it
    if (l >= 0 && l < a.n_loc) atomicOr(&lblk[l].y, (G == 1 ? 3 : idx < a.k ? 1 : 2) << 16);
  };
#pragma unroll
  for (int u = 0; u < kSelPer; ++u) flag(tid + u * kThreads, selv[u]);
#pragma unroll 1
  for (int idx = tid + kSelPer * kThreads; idx < n_sel_here; idx += kThreads) flag(idx, sel_wg[idx]);
  __syncthreads();
  const int n_pers = (a.C + 1) * SUB, n_cand = n_pers + a.n_loc * SUB;
  // candidate i -> its class (-1: no tile) and its list entry
  auto classify = [&](int i, int& src, int& meta) -> int {
    if (i >= n_cand) return -1;
    if (i < n_pers) {
      const int c = i / SUB, sub = i % SUB;
      const int tl = min(max(plen_s[c] - sub * kTile, 0), kTile);
      src = i;
      meta = tl | (3 << 8);
      if constexpr (MASS) meta |= (c << 10) | (sub << 20);       // the key block the tile belongs to, and which tile of it
      return tl == 0 ? -1 : tl == kTile ? 0 : 1;
    }
    const int l = (i - n_pers) / SUB, sub = (i - n_pers) % SUB;
    const int2 blk = lblk[l];
    const int f = blk.y >> 16, tl = min(max((blk.y & 0xFFFF) - sub * kTile, 0), kTile);
    src = (int)(0x80000000u | (uint32_t)(blk.x * SUB + sub));
    meta = tl | (f << 8);
    if constexpr (MASS) meta |= ((a.C + 1 + l) << 10) | (sub << 20);
    return f == 0 || tl == 0 ? -1 : tl < kTile ? 1 : f == 3 ? 0 : f + 1;      // f is 1 or 2 otherwise
  };
  // A wave classifies its candidates twice: the first sweep gives the sizes of the four parts, the second the places, with
  // the running counts in scalar registers (ballots).
  const int n_rounds = (n_cand + 63) / 64, r_mid = (n_rounds + 1) / 2;
  const int r_begin = wave == 0 ? 0 : r_mid, r_end = wave == 0 ? r_mid : n_rounds;
  int tot[4] = {0, 0, 0, 0};
#pragma unroll 1
  for (int r = r_begin; r < r_end; ++r) {
    int src, meta;
    const int cls = classify(r * 64 + lane, src, meta);
#pragma unroll
    for (int c = 0; c < 4; ++c) tot[c] += __popcll(__ballot(cls == c));
  }
  if (lane == 0)
#pragma unroll
    for (int c = 0; c < 4; ++c) cnt_s[4 * wave + c] = tot[c];
  __syncthreads();
  int before[4];                           // what the candidates of wave 0 put ahead of this wave's
#pragma unroll
  for (int c = 0; c < 4; ++c) {
    const int other = __builtin_amdgcn_readfirstlane(cnt_s[4 * (wave ^ 1) + c]);
    before[c] = wave == 0 ? 0 : other;
    tot[c] += other;
  }
  // this workgroup's tiles of each class: all of them, or ranks lo .. lo + num - 1 (the classes take the parts in opposite
  // orders, so that the remainders do not meet in one part)
  int lo[4] = {0, 0, 0, 0}, num[4] = {tot[0], tot[1], tot[2], tot[3]};
  if constexpr (SPLIT) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const int p = c == 0 ? part : n_parts - 1 - part;
      lo[c] = tot[c] * p / n_parts;
      num[c] = tot[c] * (p + 1) / n_parts - lo[c];
    }
  }
  const int first[4] = {0, num[0], num[0] + num[1], num[0] + num[1] + num[2]};
  const int cls_end[4] = {first[1], first[2], first[3], first[3] + num[3]};
  int base[4];
#pragma unroll
  for (int c = 0; c < 4; ++c) base[c] = first[c] - lo[c] + before[c];
  int32_t* mass_list = MASS ? a.Rlist + (size_t)logical * a.list_cap : nullptr;
  auto place = [&](int cls, int src, int meta) {
#pragma unroll
    for (int c = 0; c < 4; ++c) {
      const unsigned long long m = __ballot(cls == c);
      if (cls == c) {
        const int pos = base[c] + lanes_below(m);
        if (!SPLIT || (pos >= first[c] && pos < cls_end[c])) {
          t_src[pos] = src;
          t_meta[pos] = (meta_t)meta;
        }
        if constexpr (SPLIT && MASS) {     // the later pass walks the whole list, whoever walked its parts
          const int at = pos - first[c] + lo[c] + (c > 0 ? tot[0] : 0) + (c > 1 ? tot[1] : 0) + (c > 2 ? tot[2] : 0);
          if (part == 0 && at < a.list_cap - 4) mass_list[4 + at] = meta;
        }
      }
      base[c] += __popcll(m);
    }
  };
#pragma unroll 1
  for (int r = r_begin; r < r_end; ++r) {
    int src = 0, meta = 0;
    const int cls = classify(r * 64 + lane, src, meta);
    place(cls, src, meta);
  }
  __syncthreads();
  // The Q fragments are only ever MFMA operands, which may come from the accumulator half of the
  // register file: define them there, leaving the architectural half to the softmax and the outputs.
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(qf[g][ks]));

  MassOut mo{nullptr, 64, 64, lane, lane >= 32, 0.0f, 0.0f};
  if constexpr (MASS) {
    // the later pass walks the same list: the ends of its four parts, then a descriptor per tile
    if (tid == 0 && part == 0) {
      mass_list[0] = tot[0];
      mass_list[1] = tot[0] + tot[1];
      mass_list[2] = tot[0] + tot[1] + tot[2];
      mass_list[3] = tot[0] + tot[1] + tot[2] + tot[3];
    }
    if constexpr (!SPLIT)
      for (int i = tid; i < cls_end[3] && i < a.list_cap - 4; i += kThreads) mass_list[4 + i] = t_meta[i];
    mo.rp = a.R + ((size_t)logical * 2 + wave) * a.r_slots * 64;
  }
  // the records of a split walk go where the whole walk would leave them
  float* const rec0 = mo.rp;
#define PBSA_RECORDS_AT(TILE_)                                                                          \
  if constexpr (SPLIT && MASS) mo.rp = rec0 + (size_t)(TILE_) * 64;
  const int e0 = cls_end[0];               // shared full tiles [0, e0)
  const int n_tiles = cls_end[1];          // shared ragged tiles [e0, n_tiles): the end of the shared list
  const int solo_b = wave == 0 ? n_tiles : cls_end[2];         // this wave's solo tiles [solo_b, solo_e)
  const int solo_e = wave == 0 ? cls_end[2] : cls_end[3];

  f32x16 o[2][DT];
#pragma unroll
  for (int g = 0; g < 2; ++g)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
      for (int v = 0; v < 16; ++v) o[g][dt][v] = 0.0f;
      asm volatile("" : "+a"(o[g][dt]));
    }
  f32x16 sA[2], sB[2];                     // S^T of even / odd sub-tiles
  PTile pA, pB;                            // P^T of even / odd sub-tiles (bf16 pairs)
  const float c2 = a.scale * 1.4426950408889634f, lift = kLift / c2;
  SoftmaxRun sr{{kInitMax, kInitMax}, {-kInitMax * c2, -kInitMax * c2}, {0.0f, 0.0f, 0.0f, 0.0f},
                {sum_selector(lane, 0), sum_selector(lane, 1)}, 0ull, c2, lift, false};
  bf16x8 frag[2 * KS];                     // operand fragments, handed from step to step
  NoMid nomid;

  // ---- operand addresses ------------------------------------------------------------------------
  // this lane's fragment addresses inside ring entry 0, sub-tile 0 (LDS byte addresses)
  const uint32_t smem_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  uint32_t ka0[KS], va0[DT];
  {
    const int kb = qn * ROW + ((half ^ k_swz<D>(qn)) << 4);        // chunk (2 ks + half) ^ f = (half ^ f) ^ 2 ks
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) ka0[ks] = smem_lds + (uint32_t)(kb ^ (ks << 5));
    const int s16 = lane & 15, q16 = (lane >> 4) & 1;
    const int v_row0 = 4 * half + (s16 >> 2);                      // address row within 16 keys
    const int v_sub = 2 * q16 + ((s16 & 3) >> 1), v_lo = (s16 & 1) * 8;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
      va0[dt] = smem_lds + 2 * TILE + (uint32_t)(v_row0 * ROW + (((4 * dt + v_sub) ^ v_swz<D>(v_row0)) << 4) + v_lo);
  }

  // ---- staging --------------------------------------------------------------------------------
  // A wave instruction fills one KiB of a tile: RPI consecutive rows, lane i -> row i / CH, physical
  // chunk i % CH, i.e. the logical chunk (i % CH) ^ f(row) of that row.  Since f has period 16 in the row
  // (K) or depends on the row within the piece only (V), the per-lane source offsets within a piece are
  // four patterns for K (the pieces of 16 rows) and one for V, whatever rows a load brings.  In the
  // shared part wave w brings rows 32 w .. 32 w + 31 of every tile.  A ragged V tile must not bring rows
  // past its valid length into LDS (they meet p = 0 in the MFMA, and 0 x NaN-or-Inf pattern is NaN): the
  // lanes of such rows fetch the last valid row instead.
  const int rl = lane / CH, vchk = ((lane % CH) ^ v_swz<D>(rl)) << 4;
  DmaPlan<D> plan;
#pragma unroll
  for (int k = 0; k < 4; ++k) plan.kpat[k] = rl * ROW + (((lane % CH) ^ k_swz<D>(RPI * k + rl)) << 4);
  plan.vpat = rl * ROW + vchk;
  plan.vragged = false;
#pragma unroll
  for (int i = 0; i < NIW; ++i) plan.voff[i] = 0;
  const uint32_t smem_s = __builtin_amdgcn_readfirstlane(smem_lds);
  const size_t head_l = (size_t)h * a.n_loc_cap * B * D * 2, head_p = (size_t)h * (a.C + 1) * B * D * 2;
#define PBSA_TILE_PTR(SRC, BASE_L, BASE_P)                                                              \
  ((SRC) < 0 ? reinterpret_cast<const unsigned char*>(BASE_L) + head_l + (size_t)((SRC) & 0x7FFFFFFF) * (kTile * D * 2) \
             : reinterpret_cast<const unsigned char*>(BASE_P) + head_p + (size_t)(SRC) * (kTile * D * 2))
  // the plan that brings this wave's half of K tile KSRC into K ring entry KENTRY and of V tile VSRC
  // (descriptor words of the list) into V ring entry VENTRY
#define PBSA_PLAN_K(KSRC, KENTRY)                                                                       \
  {                                                                                                     \
    const int ksrc_ = __builtin_amdgcn_readfirstlane(KSRC);                                             \
    plan.kp = PBSA_TILE_PTR(ksrc_, a.Kl, a.Kp) + wave * (TILE / 2);                                     \
    plan.klds = smem_s + (KENTRY) * TILE + wave * (TILE / 2);                                           \
  }
#define PBSA_PLAN_V(VSRC, VENTRY)                                                                       \
  {                                                                                                     \
    const int vsrc_ = __builtin_amdgcn_readfirstlane(VSRC);                                             \
    plan.vtile = PBSA_TILE_PTR(vsrc_, a.Vl, a.Vp);                                                      \
    plan.vp = plan.vtile + wave * (TILE / 2);                                                           \
    plan.vlds = smem_s + (2 + (VENTRY)) * TILE + wave * (TILE / 2);                                     \
  }
#define PBSA_PLAN_VRAGGED(VMETA)                                                                        \
  {                                                                                                     \
    const int vlast_ = (__builtin_amdgcn_readfirstlane(VMETA) & 0xFF) - 1;                              \
    plan.vragged = vlast_ < kTile - 1;                                                                  \
    if (plan.vragged) {                                                                                 \
      _Pragma("unroll") for (int i_ = 0; i_ < NIW; ++i_)                                                \
        plan.voff[i_] = min(32 * wave + RPI * i_ + rl, vlast_) * ROW + vchk;                            \
    }                                                                                                   \
  }
#define PBSA_PLAN_SHARED(KSRC, VSRC, VMETA, KENTRY, VENTRY)                                             \
  PBSA_PLAN_K(KSRC, KENTRY)                                                                             \
  PBSA_PLAN_V(VSRC, VENTRY)                                                                             \
  PBSA_PLAN_VRAGGED(VMETA)

  // One part of the shared list, tiles [TB, TE), as one pipelined run.  Tile t is sub-tiles 2t (buffers
  // A) and 2t+1 (buffers B):
  //   before   : QK(TB,0)
  //   step 2t  : softmax(t,0)  with  PV(t-1,1) (not for t = TB)  and  QK(t,1)
  //   step 2t+1: softmax(t,1)  with  PV(t,0)                     and  QK(t+1,0) (not for t = TE-1)
  //   after    : PV(TE-1,1)
  // Between the two steps of a tile the tiles K(t) and V(t-1) are dead: their ring entries are refilled
  // with K(t+2) and V(t+1), which have until the same point of the next tile to arrive.  Steps 2t+1 and
  // 2t+2 read the same two ring entries (V of t, K of t+1), so the loop body is that pair and takes one
  // set of addresses.  The ragged run masks, per tile, the keys that do not exist and the wave that does
  // not attend.
  // The addresses are computed once per tile and kept in registers (the empty asm stops the compiler from
  // recomputing them next to each use): an address made by a vector instruction right before the LDS read
  // that uses it stalls the wave for about ten cycles per read.
#define PBSA_ADDR_K(T_)                                                                                 \
  _Pragma("unroll") for (int ks = 0; ks < KS; ++ks) {                                                   \
    kx[ks] = ka0[ks] + ((T_) & 1) * TILE;                                                               \
    asm volatile("" : "+v"(kx[ks]));                                                                    \
  }
#define PBSA_ADDR_V(T_)                                                                                 \
  _Pragma("unroll") for (int dt = 0; dt < DT; ++dt) {                                                   \
    vx[dt] = va0[dt] + ((T_) & 1) * TILE;                                                               \
    asm volatile("" : "+v"(vx[dt]));                                                                    \
  }
#define PBSA_LIMITS(T_, RAGGED)                                                                         \
  if (RAGGED) {                                                                                         \
    const int meta_ = __builtin_amdgcn_readfirstlane(t_meta[T_]);                                       \
    const int len_ = meta_ & 0xFF;                                                                      \
    const bool on_ = (meta_ >> (8 + wave)) & 1;                                                         \
    lim0[0] = lim0[1] = (on_ ? min(len_, 32) : 0) - 4 * half;                                           \
    lim1[0] = lim1[1] = (on_ ? max(len_ - 32, 0) : 0) - 4 * half;                                       \
  }
  // The loads of K(T_+2) and V(T_+1) ride along the step that follows.  Past the end of the list the
  // last tile is fetched again: the ring entries it lands in are dead and never read.  The descriptors
  // of those tiles were read from LDS one tile earlier (d_ksrc, d_vsrc, d_vmeta), so that no LDS latency
  // sits between the barrier and the first load; the reads for the next turnover are issued here.
#define PBSA_FETCH_DESC(T_)                                                                             \
  {                                                                                                     \
    d_ksrc = t_src[min((T_) + 2, n_tiles - 1)];                                                         \
    d_vsrc = t_src[min((T_) + 1, n_tiles - 1)];                                                         \
    d_vmeta = t_meta[min((T_) + 1, n_tiles - 1)];                                                       \
  }
#define PBSA_NEXT_PLAN(T_)                                                                              \
  PBSA_PLAN_SHARED(d_ksrc, d_vsrc, d_vmeta, (T_) & 1, ((T_) + 1) & 1)                                   \
  PBSA_FETCH_DESC((T_) + 1)
#define PBSA_TURNOVER(T_)                                                                               \
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); /* K(T_+1), V(T_) have landed */                     \
  __syncthreads();
  /* the query fragments stay in the accumulator half of the register file (only MFMAs read them) */
#define PBSA_PIN_Q                                                                                      \
  _Pragma("unroll") for (int g_ = 0; g_ < 2; ++g_)                                                      \
    _Pragma("unroll") for (int ks_ = 0; ks_ < KS; ++ks_) asm volatile("" : "+a"(qf[g_][ks_]));
#define PBSA_RUN_SHARED(RAGGED, TB, TE)                                                                 \
  if ((TB) < (TE)) {                                                                                    \
    uint32_t kx[KS], vx[DT];                                                                            \
    int lim0[2] = {0, 0}, lim1[2] = {0, 0};                                                             \
    typedef StepKind<true, true, 0, 0> KindA;              /* the loop's first step of a tile */      \
    typedef StepKind<true, true, SUB1, SUB1> KindB;        /* and its second */                        \
    PBSA_ADDR_K(TB)                                                                                     \
    PBSA_ADDR_V(TB)                                                                                     \
    step<D, MASS, false, false, kNoLoads, StepKind<false, true, 0, 0>, false, kNextNone, void, NoMid>(  \
        vx, kx, qf, o, sB, sA, pB, pA, sr, lim0, plan, mo, frag, 0, 0, nomid);                          \
    if (!(RAGGED)) seed_reference(sA, sr);   /* (a ragged tile's scores are not masked yet) */          \
    PBSA_LIMITS(TB, RAGGED)                                                                             \
    PBSA_NEXT_PLAN(TB)                                                                                  \
    step<D, MASS, true, RAGGED, kNoLoads, StepKind<false, true, SUB1, 0>, false, kNextNone, void, NoMid>( \
        vx, kx, qf, o, sA, sB, pA, pB, sr, lim0, plan, mo, frag, 0, 0, nomid);                          \
    PBSA_TURNOVER(TB)                                                                                   \
    PBSA_ADDR_V(TB)                                                                                     \
    PBSA_ADDR_K((TB) + 1)                                                                               \
    /* (unconditional: fragments defined on one path only cost registers on all of them) */            \
    preload_frags<D, KindA>(frag, vx, kx);                                                              \
    for (int t = (TB); t < (TE) - 1; ++t) {                                                             \
      /* the tile's second step ends by moving the address registers to the other ring entries */       \
      const int dv_ = (t & 1) ? -TILE : TILE;                                                           \
      step<D, MASS, true, RAGGED, kLoads, KindA, true, kNextSame, KindB, NoMid>(                        \
          vx, kx, qf, o, sB, sA, pB, pA, sr, lim1, plan, mo, frag, 0, 0, nomid);                        \
      PBSA_LIMITS(t + 1, RAGGED)                                                                        \
      /* the plan of the next tile's loads is made inside the second step, which issues no loads */     \
      auto mid_ = [&](auto piece_) {                                                                    \
        constexpr int pc_ = decltype(piece_)::value;                                                    \
        if constexpr (pc_ == 0) PBSA_PLAN_K(d_ksrc, (t + 1) & 1)                                        \
        if constexpr (pc_ == 1) PBSA_PLAN_V(d_vsrc, (t + 2) & 1)                                        \
        if constexpr (pc_ == 2) PBSA_PLAN_VRAGGED(d_vmeta)                                              \
        if constexpr (pc_ == 3) d_ksrc = t_src[min(t + 4, n_tiles - 1)];                                \
        if constexpr (pc_ == 4) {                                                                       \
          d_vsrc = t_src[min(t + 3, n_tiles - 1)];                                                      \
          d_vmeta = t_meta[min(t + 3, n_tiles - 1)];                                                    \
        }                                                                                               \
      };                                                                                                \
      step<D, MASS, true, RAGGED, kNoLoads, KindB, true, kNextTile, KindA, decltype(mid_)>(             \
          vx, kx, qf, o, sA, sB, pA, pB, sr, lim0, plan, mo, frag, -dv_, dv_, mid_);                    \
    }                                                                                                   \
    /* the address registers now point at V(TE-1) */                                                    \
    step<D, MASS, true, RAGGED, kLoads, StepKind<true, false, 0, 0>, false, kNextSame,                  \
         StepKind<true, false, 0, SUB1>, NoMid>(vx, kx, qf, o, sB, sA, pB, pA, sr, lim1, plan, mo, frag, 0, 0, nomid); \
    step<D, MASS, false, false, kNoLoads, StepKind<true, false, 0, SUB1>, true, kNextNone, void, NoMid>( \
        vx, kx, qf, o, sA, sB, pA, pB, sr, lim0, plan, mo, frag, 0, 0, nomid);                          \
    /* between runs the compiler may copy the accumulators to other registers: let the matrix pipe drain first */ \
    acc_settle<DT>(o[0]);                                                                               \
    acc_settle<DT>(o[1]);                                                                               \
  }

  if (n_tiles > 0) {
    __syncthreads();                       // the setup scratch (aliasing the rings) is dead
    PBSA_PLAN_SHARED(t_src[0], t_src[0], t_meta[0], 0, 0)
    dma_all<D>(plan, true, true);
    if (n_tiles > 1) {
      PBSA_PLAN_SHARED(t_src[1], t_src[0], t_meta[0], 1, 0)
      dma_all<D>(plan, true, false);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    int d_ksrc, d_vsrc, d_vmeta;
    PBSA_FETCH_DESC(0)
    PBSA_RECORDS_AT(lo[0])
    PBSA_RUN_SHARED(false, 0, e0)
    PBSA_RECORDS_AT(tot[0] + lo[1])
    PBSA_RUN_SHARED(true, e0, n_tiles)
  }

  // ---- solo part ----------------------------------------------------------------------------------
  // Wave w streams its own full local tiles [solo_b, solo_e) through ring entry w of K and of V, which
  // it treats as two 32-key halves.  Sub-tile u = 2t + h lives in half h; in step u the wave computes
  // softmax(u), PV(u-1) from the other V half and QK(u+1) from the other K half, while the halves it
  // has finished with are refilled with K(u+2) and V(u), which must have landed when the step ends.
  //   before   : QK(2 TB)
  //   step 2t  : softmax(2t)    PV(2t-1) (not for t = TB)   QK(2t+1)        loads K(t+1, half 0), V(t, half 0)
  //   step 2t+1: softmax(2t+1)  PV(2t)                      QK(2t+2) (not for t = TE-1)   K(t+1, half 1), V(t, half 1)
  //   after    : PV(2 TE - 1)
  // These are the step instances of the shared loop with another load plan.  Past the end of the list
  // the last tile's K is fetched again into halves that are never read.
  if constexpr (G > 1) {
    // the other wave may still read the rings, and the shared part's trailing loads may still land in them
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (solo_b < solo_e) {
      PBSA_RECORDS_AT(tot[0] + tot[1] + (wave == 0 ? lo[2] : lo[3]))
      const unsigned char* kl_h = reinterpret_cast<const unsigned char*>(a.Kl) + head_l;
      const unsigned char* vl_h = reinterpret_cast<const unsigned char*>(a.Vl) + head_l;
      const uint32_t kring = smem_s + wave * TILE, vring = smem_s + (2 + wave) * TILE;
      plan.vragged = false;
      uint32_t kx[KS], vx[DT];
      const int lim0[2] = {0, 0};
#pragma unroll
      for (int ks = 0; ks < KS; ++ks) {
        kx[ks] = ka0[ks] + wave * TILE;
        asm volatile("" : "+v"(kx[ks]));
      }
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        vx[dt] = va0[dt] + wave * TILE;
        asm volatile("" : "+v"(vx[dt]));
      }
      int d_cur = t_src[solo_b], d_next, d_nn;
      // sources of the loads of the steps of tile t: K from tile t+1, V from tile t; HALF picks the rows
#define PBSA_SOLO_PLAN(HALF)                                                                            \
  plan.kp = kl_h + (size_t)(__builtin_amdgcn_readfirstlane(d_next) & 0x7FFFFFFF) * (kTile * D * 2) + (HALF) * SUB1; \
  plan.vp = vl_h + (size_t)(__builtin_amdgcn_readfirstlane(d_cur) & 0x7FFFFFFF) * (kTile * D * 2) + (HALF) * SUB1;  \
  plan.klds = kring + (HALF) * SUB1;                                                                    \
  plan.vlds = vring + (HALF) * SUB1;
#define PBSA_SOLO_LANDED asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      d_next = d_cur;                     // the whole K tile of the first solo tile, half by half
      PBSA_SOLO_PLAN(0)
      dma_all<D>(plan, true, false);
      PBSA_SOLO_PLAN(1)
      dma_all<D>(plan, true, false);
      d_next = t_src[min(solo_b + 1, solo_e - 1)];
      PBSA_SOLO_LANDED
      step<D, MASS, false, false, kNoLoads, StepKind<false, true, 0, 0>, false, kNextNone, void, NoMid>(vx, kx, qf, o, sB, sA, pB, pA, sr, lim0, plan, mo, frag, 0, 0, nomid);
      seed_reference(sA, sr);
      PBSA_SOLO_PLAN(0)
      step<D, MASS, true, false, kLoads, StepKind<false, true, SUB1, 0>, false, kNextNone, void, NoMid>(vx, kx, qf, o, sA, sB, pA, pB, sr, lim0, plan, mo, frag, 0, 0, nomid);
      PBSA_SOLO_LANDED
      for (int t = solo_b; t < solo_e - 1; ++t) {
        d_nn = t_src[min(t + 2, solo_e - 1)];
        PBSA_SOLO_PLAN(1)
        step<D, MASS, true, false, kLoads, StepKind<true, true, 0, 0>, false, kNextNone, void, NoMid>(vx, kx, qf, o, sB, sA, pB, pA, sr, lim0, plan, mo, frag, 0, 0, nomid);
        PBSA_SOLO_LANDED
        d_cur = d_next;
        d_next = d_nn;
        PBSA_SOLO_PLAN(0)
        step<D, MASS, true, false, kLoads, StepKind<true, true, SUB1, SUB1>, false, kNextNone, void, NoMid>(vx, kx, qf, o, sA, sB, pA, pB, sr, lim0, plan, mo, frag, 0, 0, nomid);
        PBSA_SOLO_LANDED
      }
      PBSA_SOLO_PLAN(1)
      step<D, MASS, true, false, kLoads, StepKind<true, false, 0, 0>, false, kNextNone, void, NoMid>(vx, kx, qf, o, sB, sA, pB, pA, sr, lim0, plan, mo, frag, 0, 0, nomid);
      PBSA_SOLO_LANDED
      step<D, MASS, false, false, kNoLoads, StepKind<true, false, 0, SUB1>, false, kNextNone, void, NoMid>(vx, kx, qf, o, sA, sB, pA, pB, sr, lim0, plan, mo, frag, 0, 0, nomid);
    }
  }

  // ---- epilogue ---------------------------------------------------------------------------------
  acc_settle<DT>(o[0]);
  acc_settle<DT>(o[1]);
  sum_settle(sr.l_run);
  if constexpr (SPLIT) {
    if (n_parts > 1) {
      // one of several: whole 1 KiB stores, in the accumulators' own order
      const size_t slot = (size_t)(logical - a.n_full) * n_parts + part;
      float* po = a.part_o + slot * (kRowsPerWg * D) + wave * (64 * D) + lane * 4;
#pragma unroll
      for (int g = 0; g < 2; ++g) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4)
            *reinterpret_cast<float4*>(po + ((g * DT + dt) * 4 + q4) * 256) =
                make_float4(o[g][dt][4 * q4], o[g][dt][4 * q4 + 1], o[g][dt][4 * q4 + 2], o[g][dt][4 * q4 + 3]);
        const float l_part = __shfl(sr.l_run[0], 32 * g + qn, 64);
        if (half == 0)
          *reinterpret_cast<float2*>(a.part_ml + (slot * kRowsPerWg + wave * 64 + g * 32 + qn) * 2) = make_float2(sr.m_ref[g], l_part);
      }
      return;
    }
  }
#pragma unroll
  for (int g = 0; g < 2; ++g) {
    // row r of the group: lane 32 g + r of the running sums
    const float l_tot = __shfl(sr.l_run[0], 32 * g + qn, 64);
    const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
    const int tok = tok0 + 32 * g;
    if (tok < a.Nq) {
      bf16_t* orow = a.O + (size_t)h * a.o_stride_h + (size_t)tok * a.o_stride_t;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          bf16x4 w;
#pragma unroll
          for (int e = 0; e < 4; ++e) w[e] = (__bf16)(o[g][dt][4 * q4 + e] * inv);
          *reinterpret_cast<bf16x4*>(orow + 32 * dt + 8 * q4 + 4 * half) = w;
        }
      if (a.lse && half == 0)
        a.lse[(size_t)h * a.Nq + tok] = l_tot > 0.0f ? sr.m_ref[g] * a.scale + __logf(l_tot) : -INFINITY;
    }
  }
}
#pragma clang diagnostic pop

// ------------------------------------------------------------------------------------------------
// Puts the parts of a split query tile together: O = sum_s w_s O_s / sum_s w_s l_s with w_s = 2^((m_s - max m) c2).  One
// wave instruction reads one of the 1 KiB pieces the attention wave stored (same lane, same elements); the row of a
// lane is lane % 32 of the piece's row group.  A part that met no key of a row has l_s = 0.
// ------------------------------------------------------------------------------------------------
constexpr int kCombineThreads = 256;
template <int D, int ROWS>                                 // rows of a split query tile: 128, or 64 of a team's
__global__ void __launch_bounds__(kCombineThreads) combine_kernel(AttnArgs a) {
  constexpr int DT = D / 32, PIECES = ROWS / 32 * DT * 4;  // per query tile: its row groups x DT x 4
  const int lane = threadIdx.x & 63, qn = lane & 31, half = lane >> 5;
  const int piece = blockIdx.x * (kCombineThreads / 64) + (threadIdx.x >> 6);
  static_assert(PIECES % (kCombineThreads / 64) == 0, "whole workgroups");
  const int wg = piece / (DT * 4), dt = piece / 4 % DT, q4 = piece % 4;      // row group, output tile, quarter
  const int n_qt = (a.Nq + ROWS - 1) / ROWS, tile = a.n_full + blockIdx.y;
  const int h = tile / n_qt, tok = (tile % n_qt) * ROWS + wg * 32 + qn;
  if (tok >= a.Nq) return;
  const size_t slot0 = (size_t)blockIdx.y * a.parts;
  const float2* ml = reinterpret_cast<const float2*>(a.part_ml) + slot0 * ROWS + wg * 32 + qn;
  const float* po = a.part_o + slot0 * (ROWS * D) + piece * 256 + lane * 4;
  const float c2 = a.scale * 1.4426950408889634f;
  float m[kMaxParts], l_tot = 0.0f, m_max = kInitMax;
  float4 acc = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
  float l[kMaxParts];
#pragma unroll
  for (int s = 0; s < kMaxParts; ++s) {
    const float2 v = s < a.parts ? ml[(size_t)s * ROWS] : make_float2(kInitMax, 0.0f);
    m[s] = v.x;
    l[s] = v.y;
    if (v.y > 0.0f) m_max = fmaxf(m_max, v.x);
  }
#pragma unroll
  for (int s = 0; s < kMaxParts; ++s) {
    if (s < a.parts) {
      const float4 v = *reinterpret_cast<const float4*>(po + (size_t)s * (ROWS * D));
      const float w = l[s] > 0.0f ? __builtin_amdgcn_exp2f((m[s] - m_max) * c2) : 0.0f;
      l_tot = __builtin_fmaf(w, l[s], l_tot);
      acc.x = __builtin_fmaf(w, v.x, acc.x);
      acc.y = __builtin_fmaf(w, v.y, acc.y);
      acc.z = __builtin_fmaf(w, v.z, acc.z);
      acc.w = __builtin_fmaf(w, v.w, acc.w);
    }
  }
  const float inv = l_tot > 0.0f ? 1.0f / l_tot : 0.0f;
  bf16x4 w4;
  w4[0] = (__bf16)(acc.x * inv);
  w4[1] = (__bf16)(acc.y * inv);
  w4[2] = (__bf16)(acc.z * inv);
  w4[3] = (__bf16)(acc.w * inv);
  *reinterpret_cast<bf16x4*>(a.O + (size_t)h * a.o_stride_h + (size_t)tok * a.o_stride_t + 32 * dt + 8 * q4 + 4 * half) = w4;
  if (a.lse && dt == 0 && q4 == 0 && half == 0)
    a.lse[(size_t)h * a.Nq + tok] = l_tot > 0.0f ? m_max * a.scale + __logf(l_tot) : -INFINITY;
}

}  // namespace

// How a launch is shared out (see SPLIT at attention_kernel).  The chip runs kPlaces workgroups at a time, so a launch
// of n query tiles lasts ceil(n / kPlaces) rounds and its last round may be nearly empty: a chunk of 5 heads x 1000 rows
// is 40 workgroups on 512 places.  The tiles of that last round are split over as many workgroups as it has places for,
// as long as a shorter walk gains more than the second launch and the partial results cost.  Depends on the shape
// alone, so that every call of a shape that is given the scratch -- with decisions, with mass, neither -- takes the same parts.
AttnSplit attn_split(const pbsa_params& p) {
  constexpr int kPlaces = 512;
  AttnSplit sp{0, 1, 0, 0, 0};
  const long n_wg = (long)p.H * ((p.Nq + kRowsPerWg - 1) / kRowsPerWg), n_full = n_wg / kPlaces * kPlaces, r = n_wg - n_full;
  const int tiles = (p.C + 1 + (p.k < p.n_loc_cap ? p.k : p.n_loc_cap)) * (p.B / kTile);
  if (r == 0 || r > kPlaces / 2) return sp;
  const float t_tile = p.d == 128 ? kTileUs128 : kTileUs64;
  const float part_us = (float)(2 * kRowsPerWg * p.d * 4) / kPartBytesPerUs;
  float best = tiles * t_tile - kSplitWorthUs;
  for (int s = 2; s <= kMaxParts && s <= tiles && s * r <= kPlaces; ++s) {
    const float us = (float)((tiles + s - 1) / s) * t_tile + kCombineUs + (float)(r * s) * part_us;
    if (us < best) {
      best = us;
      sp.parts = s;
    }
  }
  if (sp.parts == 1) return sp;
  sp.n_full = (int)n_full;
  sp.n_split = (int)r;
  sp.o_bytes = (size_t)r * sp.parts * kRowsPerWg * p.d * 4;
  sp.bytes = sp.o_bytes + (size_t)r * sp.parts * kRowsPerWg * 8;
  return sp;
}

// Microseconds that a wave takes for `tiles` tiles of its list while `waves` waves run, of 1024 that can: slower the fuller the
// chip is, which then holds a lower clock (measured, d = 128: 1.3-1.4 a tile with an eighth of the waves, 1.55 with 0.6 of
// them, 1.95 with all; d = 64: 1.0-1.2).
static float walk_us(int d, int tiles, int waves) {
  const float load = (float)waves / 1024.0f;
  return (float)tiles * (d == 128 ? 1.3f + 0.65f * load * load : 1.0f + 0.2f * load * load);
}

// By teams wherever they fit on the chip in one round -- 256 units of 64 rows in teams of four waves, 512 in teams of two, the
// workgroups that take decisions not counted -- and the list has a tile for more than one of them.  Against query tiles of 128 rows, whole or in the parts of attn_split
// and with their second launch (us): 2 x 256 rows of 64 with 7 tiles 13.4 in a step -> 11.4; 5 x 1000 x 64, 26 tiles
// 19.4 -> 12.5; 14 x 245 x 128, 16 tiles 20.8 -> 13.3; 11 x 1336 x 64, 54 tiles 31.1 -> 22.1; 8 x 2000 x 128, 92 tiles
// 58.1 -> 50.6; teams of two: 16 x 1100 x 64, 11 tiles 17.9 -> 12.2, 12 x 1800 x 128, 38 tiles 41.0 -> 35.9.  One tile
// alone: 5.7 -> 6.2, and nothing at all 6.8 -> 7.3, which stay as they are.  A team's waves stage their tiles by themselves
// and take 3 to 8 % longer for one (5 at d = 64), so long lists that the parts share out as well or better stay with them (6 x 4736 x 128, 202
// tiles 172.0 | 179.6; 4 x 5000 x 128, 74 tiles in three parts 58.4 | 63.0).  Few units with long lists take several teams
// each and the second launch: 1 x 1000 x 64, 82 tiles 21.0 -> 15.8 (one team 26.7); the parts of attn_split cost another
// 3 us beside theirs, for lists and runs of their own (4 x 210 x 128, 21 tiles: 20.5 by parts of two tiles, 17 by one
// team).  A call without scratch whose shape has use for it walks whole (one team to a unit would need none).
AttnTeam attn_team(const pbsa_params& p, bool scratch) {
  const long units = (long)p.H * ((p.Nq + 63) / 64), n_wg = (long)p.H * ((p.Nq + kRowsPerWg - 1) / kRowsPerWg);
  const int tiles = (p.C + 1 + (p.k < p.n_loc ? p.k : p.n_loc)) * (p.B / kTile);
  AttnTeam team{0, 1, 0};
  if (units > 512 || tiles < 3 || (long)p.n_loc_cap * (p.B / kTile) >= (1l << 24)) return team;     // (a list word has 24 bits for the tile)
  const AttnSplit sp = attn_split(p);
  if (sp.parts > 1 && !scratch) return team;
  team.units = (int)units;
  team.waves = units > 256 ? 2 : 4;
  constexpr float kPartsUs = 3.0f;
  const float own_tiles = p.d == 128 ? 1.09f : 1.05f;
  auto team_us = [&](int parts) {
    const int n = team.waves * parts;
    return own_tiles * walk_us(p.d, (tiles + n - 1) / n, (int)units * n) + (parts > 1 ? kCombineUs : 0.0f);
  };
  float best = team_us(1);
  // Not where the update's decisions, which ride as one more workgroup to a head and ahead of the units, leave as many of those
  // without a place, short walks end before short decisions have, and query tiles would find places beside them: with
  // decisions | attention alone, query tiles | teams: 28 x 539 x 64, 10 tiles 12.9 15.2 | 12.8 8.8; 130 x 170 x 64, 10 14.2 17.1 | 14.5
  // 11.2; 36 x 846 x 128, 10 18.8 23.7 | 19.2 16.4; 152 x 39 x 64, 5 9.9 13.0 | 9.8 7.4; 214 x 35 x 128, 3 9.4 15.6 | 9.3 8.9.  Longer
  // lists gain more than that costs (91 x 104 x 64, 22 tiles 19.6 -> 18.6 | 19.6 -> 12.1; 128 x 209 x 128, 28 42.2 -> 40.3 | 42.4 -> 35.1), and
  // decisions over more blocks end late by either way (5 x 3227 x 128, 8 tiles, 51 x 51 blocks 27.6 | 19.8).  All calls of a
  // shape go one way, whether they take decisions along or not: their outputs agree bit for bit.
  const int k = p.k < p.n_loc ? p.k : p.n_loc, decisions = p.nqb * (p.n_loc + p.C) <= 256 ? p.nqb * (p.n_loc + p.C) : 0;
  if (sp.parts == 1 && p.C <= PBSA_MAX_C && units + p.H > 1024 / team.waves && n_wg + p.H <= 512 && decisions > 0) {
    const float longer = (p.d == 128 ? 9.0f : 7.3f) + (float)decisions / (float)(64 * team.waves);    // by, beside the tiles
    // (a query tile over two blocks of 64 has some that only one of them selected)
    const float whole = (float)tiles + (p.B == 64 && p.Nq > 64 ? 0.5f * (float)std::min(k, p.n_loc - k) : 0.0f);
    if (best + longer > whole * walk_us(p.d, 1, (int)n_wg * 2)) return AttnTeam{0, 1, 0};
  }
  if (sp.parts == 1) return team;
  for (int s = 2; s <= sp.parts && s * units <= 256; ++s) {          // (what s parts leave fits in the scratch for sp.parts)
    const float us = team_us(s);
    if (us < best - (team.parts == 1 ? kSplitWorthUs : 0.0f)) {
      best = us;
      team.parts = s;
    }
  }
  if (walk_us(p.d, (tiles + sp.parts - 1) / sp.parts, (int)n_wg * 2 * sp.parts) + kCombineUs + kPartsUs < best) team.waves = 0;
  return team;
}

template <bool MASS, bool PLAN, bool SPLIT>
static void launch_attention_b(const pbsa_params& p, const AttnArgs& a, const PlanArgs<PLAN>& pl, dim3 grid,
                               hipStream_t stream) {
  const dim3 block(kThreads);
  if (p.d == 128 && p.B == 128) hipLaunchKernelGGL((attention_kernel<128, 128, MASS, PLAN, SPLIT>), grid, block, 0, stream, a, pl);
  else if (p.d == 128 && p.B == 64) hipLaunchKernelGGL((attention_kernel<128, 64, MASS, PLAN, SPLIT>), grid, block, 0, stream, a, pl);
  else if (p.d == 64 && p.B == 128) hipLaunchKernelGGL((attention_kernel<64, 128, MASS, PLAN, SPLIT>), grid, block, 0, stream, a, pl);
  else hipLaunchKernelGGL((attention_kernel<64, 64, MASS, PLAN, SPLIT>), grid, block, 0, stream, a, pl);
}

template <int ROWS>
static hipError_t launch_combine(const pbsa_params& p, const AttnArgs& a, int n_tiles, hipStream_t stream) {
  const dim3 grid(ROWS / 32 * (p.d / 32) * 4 / (kCombineThreads / 64), n_tiles);
  if (p.d == 128) hipLaunchKernelGGL((combine_kernel<128, ROWS>), grid, dim3(kCombineThreads), 0, stream, a);
  else hipLaunchKernelGGL((combine_kernel<64, ROWS>), grid, dim3(kCombineThreads), 0, stream, a);
  return hipGetLastError();
}

// split_ws: device scratch for attn_split(p).bytes, or nullptr: every query tile whole
template <bool MASS, bool PLAN>
static hipError_t launch_attention_t(const pbsa_params& p, AttnArgs a, const PlanArgs<PLAN>& pl, void* split_ws,
                                     hipStream_t stream) {
  const int n_wg = p.H * ((p.Nq + kRowsPerWg - 1) / kRowsPerWg);
  const int n_plan = PLAN ? 8 * ((p.H + 7) / 8) : 0;
  const AttnSplit sp = attn_split(p);
  if (const AttnTeam team = attn_team(p, split_ws != nullptr); team.waves > 0) {
    a.parts = team.parts;
    if (team.parts > 1) {
      a.part_o = static_cast<float*>(split_ws);
      a.part_ml = a.part_o + (size_t)team.units * team.parts * 64 * p.d;
    }
    const hipError_t e = launch_attention_team<MASS, PLAN>(p, a, pl, team.waves, n_plan, stream);
    return e != hipSuccess || team.parts == 1 ? e : launch_combine<64>(p, a, team.units, stream);
  }
  if (!split_ws || sp.parts == 1) {
    launch_attention_b<MASS, PLAN, false>(p, a, pl, dim3(n_plan + 8 * ((n_wg + 7) / 8)), stream);
    return hipGetLastError();
  }
  a.n_full = sp.n_full;
  a.parts = sp.parts;
  a.part_o = static_cast<float*>(split_ws);
  a.part_ml = reinterpret_cast<float*>(static_cast<char*>(split_ws) + sp.o_bytes);
  launch_attention_b<MASS, PLAN, true>(p, a, pl, dim3(n_plan + sp.n_full + 8 * ((sp.n_split * sp.parts + 7) / 8)), stream);
  hipError_t e = hipGetLastError();
  return e != hipSuccess ? e : launch_combine<kRowsPerWg>(p, a, sp.n_split, stream);
}

static AttnArgs attn_args(const pbsa_params& p, const bf16_t* Q, const bf16_t* Kp, const bf16_t* Vp, const int32_t* p_len,
                          const bf16_t* Kl, const bf16_t* Vl, const int32_t* l_len, const int32_t* l_map,
                          const int32_t* sel, bf16_t* O, float* lse, const MassRows* rows) {
  return AttnArgs{p.H, p.Nq, p.nqb, p.n_loc, p.n_loc_cap, p.C, p.k, p.scale, p.q_stride_h, p.q_stride_t,
                  p.o_stride_h, p.o_stride_t, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse,
                  rows ? rows->R : nullptr, rows ? rows->list : nullptr, rows ? rows->r_slots : 0,
                  rows ? rows->list_cap : 0, 0, 1, nullptr, nullptr, p.B};
}

hipError_t launch_attention(const pbsa_params& p, const bf16_t* Q, const bf16_t* Kp, const bf16_t* Vp,
                            const int32_t* p_len, const bf16_t* Kl, const bf16_t* Vl, const int32_t* l_len,
                            const int32_t* l_map, const int32_t* sel, bf16_t* O, float* lse, const MassRows* rows,
                            void* split_ws, hipStream_t stream) {
  const AttnArgs a = attn_args(p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse, rows);
  return rows ? launch_attention_t<true, false>(p, a, PlanArgs<false>{}, split_ws, stream)
              : launch_attention_t<false, false>(p, a, PlanArgs<false>{}, split_ws, stream);
}

hipError_t launch_attention_plan(const pbsa_params& p, const bf16_t* Q, const bf16_t* Kp, const bf16_t* Vp,
                                 const int32_t* p_len, const bf16_t* Kl, const bf16_t* Vl, const int32_t* l_len,
                                 const int32_t* l_map, const int32_t* sel, bf16_t* O, float* lse, const float* Qc,
                                 const float* Kc_l, const float* Zl, float* Kc_p, int64_t* p_id, int32_t* S_cnt, int fold,
                                 const int64_t* l_id, float* scores, int32_t* slot_src, const UpdateWs& ws, void* split_ws,
                                 hipStream_t stream) {
  const AttnArgs a = attn_args(p, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, lse, nullptr);
  PlanArgs<true> pl;
  pl.sa = plan_dev::make_score_args(p, Qc, Kc_l, Zl, Kc_p, p_len, l_map, ws);
  pl.ra = plan_dev::make_retain_args(p, ws.A, p.C + p.n_loc, 0, Kc_l, Kc_p, p_len, p_id, S_cnt, fold, l_len, l_map, l_id,
                                     scores, slot_src, ws);
  return launch_attention_t<false, true>(p, a, pl, split_ws, stream);
}

}  // namespace pbsa

// Backward of the PBSA fine stage for gfx950 (the gradient of Eq. 3-5; the paper's training kernel is
// the block-sparse attention backward).  With P the masked row softmax of Z = scale Q K^T and dO given:
//     dV = P^T dO        dP = dO V^T        dZ = P o (dP - D),  D[q] = dO[q] . O[q]
//     dQ = scale dZ K    dK = scale dZ^T Q
// P is recomputed from the forward's log-sum-exp: exp2(z c2 - lse log2 e); nothing of the forward's
// probabilities is stored.  A launch of prep, then one of dq and dkv together (bwd_walk_kernel; one of each at d = 64 where
// dq alone fills the chip), no atomics, every output element written by exactly one lane:
//   prep   per row -lse log2 e and -D (fp32, D from the bf16 tensors); per local block the query blocks that attend it
//   dq     one wave per 64 query rows: their Q and dO fragments stay in registers, the 64-key tiles they attend
//          (persistent slots, then the blocks of their row of sel) stream through LDS; where there are few such waves, two
//          or four share a walk
//   dkv    two waves per 64-key tile, or twice two where there are few, each pair with half of the walk: its K and V
//          fragments stay in registers, the 64-row tiles of the query blocks that attend it (all of them for a persistent
//          slot; those whose row of sel names the block otherwise, which prep has written down) stream through LDS
// Both have a fixed side in registers (MFMA B operands) and a streamed side in LDS (A operands):
//   A1 = T1 F1^T, A2 = T2 F2^T   32 streamed rows x 32 fixed rows per MFMA chain (v_mfma_f32_32x32x16_bf16)
//          dq:  T1 = K, T2 = V, F1 = Q, F2 = dO   ->  A1 = Z^T / scale, A2 = dP^T     (keys x queries)
//          dkv: T1 = Q, T2 = dO, F1 = K, F2 = V   ->  A1 = Z / scale,   A2 = dP       (queries x keys)
//   P and dZ, elementwise from A1, A2 and the per-query lse and D, rounded to bf16, are B operands as the
//   accumulators hold them (the contraction index enumerated in accumulator order), and the A operands of the
//   second products are transposing LDS reads of the streamed tiles with the same enumeration:
//          dq:  dQ^T += K^T dZ^T          dkv: dK^T += Q^T dZ,  dV^T += dO^T P
// Tiles go from global memory straight to LDS (global_load_lds), half a tile (32 streamed rows) per ring entry; the
// 16-byte chunks of a row are permuted by the row number (swz).  Rows past a tile's valid length are never loaded: their
// lanes fetch the last valid row, and a -inf in the place of its score or its lse makes their P an exact zero.  dq holds 64
// fixed rows per wave, so every fragment read from LDS feeds two MFMAs; dkv cannot at d = 128 (two outputs: 256
// accumulator registers for 64 keys) and holds 32 per wave: it reads one fragment per MFMA.
#include <algorithm>
#include <cmath>
#include <type_traits>
#include <utility>

#include "pbsa_internal.h"

namespace pbsa {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

constexpr int kTile = 64;
constexpr float kLog2e = 1.4426950408889634f;

struct BwdArgs {
  int H, Nq, nqb, n_loc, n_loc_cap, C, k, B;
  int dq_split;       // dq: the two waves of a workgroup share a row tile's walk, else each has a row tile
  float scale;
  long q_stride_h, q_stride_t, o_stride_h, o_stride_t;
  const bf16_t* Q;
  const bf16_t* Kp;
  const bf16_t* Vp;
  const int32_t* p_len;
  const bf16_t* Kl;
  const bf16_t* Vl;
  const int32_t* l_len;
  const int32_t* l_map;
  const int32_t* sel;
  const bf16_t* O;
  const bf16_t* dO;
  const float* lse;
  float* rows;        // [H][ceil(Nq / 64) * 2][64]: of 32 rows, -lse log2 e (-inf: no such row), then -rowsum(dO o O)
  uint32_t* att;      // [H][n_loc_cap][ceil(nqb / 32)] bit i: query block i attends local block l
  int4* order;        // [H][n_loc_cap] the local blocks, the most attended first: block, slot (-1: nowhere), tokens, attending blocks
  float* dQ;
  float* dKp;
  float* dVp;
  float* dKl;
  float* dVl;
};

__device__ __forceinline__ int lanes_below(unsigned long long mask) {
  return __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
}

// One wave-wide global -> LDS load of 16 bytes per lane: LDS bytes [lds_off + OFF, + 1024) receive lane i's 16 bytes, fetched
// from base + lane_off + OFF, at 16 i (the instruction's offset moves both addresses).  Completion is tracked by the issuing
// wave's vmcnt.
template <int OFF>
__device__ __forceinline__ void dma16_at(const void* base, uint32_t lane_off, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3"
               :
               : "s"(lds_off), "v"(lane_off), "s"(base), "n"(OFF)
               : "memory", "m0");
}

// the same with 4 bytes per lane: LDS bytes [lds_off, lds_off + 256)
__device__ __forceinline__ void dma4(const void* base, uint32_t lane_off, uint32_t lds_off) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, %2"
               :
               : "s"(lds_off), "v"(lane_off), "s"(base)
               : "memory", "m0");
}

// Where the 16-byte chunks of a tile row sit in LDS: logical chunk c of row r at chunk c ^ swz(r), the row number rotated
// left by one bit.  That is distinct over 16 consecutive rows (8 when a row has 8 chunks), which the row-wise operand reads
// need (16 consecutive rows, one logical chunk).  The transposing reads go through the banks 32 lanes at a time, four
// consecutive rows with four adjacent chunks each, and would need swz(r) >> 2 distinct over those rows; at d = 128 rows 0
// and 1 share theirs, and rows 2 and 3: two conflict cycles per read, by the counters the only ones (a permutation without
// them measured 0.998 to 1.004 of the time: not taken).  At d = 64, where a row is half a pass over the banks, the counters
// say 4.1 cycles per pair of a row-wise and a transposing read (3 heads x 1500 rows).
template <int CH>
__device__ __forceinline__ int swz(int r) {
  if constexpr (CH == 16) return ((r & 7) << 1) | ((r >> 3) & 1);
  else return ((r & 3) << 1) | ((r >> 2) & 1);
}

typedef __attribute__((address_space(3))) const bf16x8* lds_b128_t;
typedef __attribute__((address_space(3))) bf16x4* lds_tr_t;
typedef __attribute__((address_space(3))) const f32x4* lds_f4_t;
__device__ __forceinline__ bf16x8 lds_read_row(uint32_t addr) { return *(lds_b128_t)(uintptr_t)addr; }
// transposed fragment of 16 streamed rows: two transposing reads, of rows r and r + 8 of the 16
__device__ __forceinline__ bf16x8 lds_read_tr(uint32_t at_lo, uint32_t at_hi) {
  const bf16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_tr_t)(uintptr_t)at_lo);
  const bf16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_tr_t)(uintptr_t)at_hi);
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}
__device__ __forceinline__ void acc_mfma(f32x16& acc, const bf16x8& a, const bf16x8& b) {
  asm volatile("v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" : "+a"(acc) : "v"(a), "v"(b));
}
// f(0), f(1), .. with the number as a constant
template <typename F, int... I>
__device__ __forceinline__ void unroll(F f, std::integer_sequence<int, I...>) {
  (f(std::integral_constant<int, I>{}), ...);
}
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  bf16x2 pk;
  pk[0] = (__bf16)a;
  pk[1] = (__bf16)b;
  return __builtin_bit_cast(uint32_t, pk);
}
__device__ __forceinline__ bf16x8 as_bf16x8(const u32x4& w) { return __builtin_bit_cast(bf16x8, w); }

// Which item (row tile, rank) of which head a workgroup of a one-line grid works on.  Workgroups go to the 8 XCDs in
// turn.  The grid goes through the items of all heads eight at a time; of the 8 H items of such a step XCD x takes those
// numbered x H .. x H + H - 1 head by head, so that an XCD's workgroups belong to about H / 8 heads and share what they
// stream through its L2.  Items past a head's last are to be skipped.  (dq, 12 heads x 4680 x 128: every wave streams its
// 16 KB per turn, 2.4 GB in all, 9 TB/s with all heads on every XCD; 264 -> 211 us with 32 + 48 blocks of 64.)
__device__ __forceinline__ void head_item(int b, int H, int& h, int& item) {
  const int q = b >> 3, i = (b & 7) * H + q % H;
  h = i >> 3;
  item = (q / H) * 8 + (i & 7);
}
inline unsigned head_items(int n, int H) { return (unsigned)((n + 7) / 8 * 8) * (unsigned)H; }

// ------------------------------------------------------------------------------------------------
// Row scalars: -lse log2 e and -D, D = dO[q] . O[q]: 16 lanes per row, 8 elements each (d = 128) or 8 lanes (d = 64).
// Rows up to the next multiple of 64 are written too: -inf and 0, so that a copy of the last row that stands in for a
// missing one takes no part.
// ------------------------------------------------------------------------------------------------
__host__ __device__ inline long row_blocks(int Nq) { return (long)((Nq + kTile - 1) / kTile) * 2; }

// The first H workgroups of the launch turn a head's rows of sel around: which query blocks attend each local block, and
// the local blocks by how many do, most first (a counting sort; blocks that tie come in any order).  One scan of sel per
// head in the place of one per 64-key tile, and an order in which the long walks start first.
__device__ __forceinline__ void plan_head(const BwdArgs& a, int h, uint32_t* smem) {
  const int W = (a.nqb + 31) / 32, n_words = a.n_loc * W, tid = threadIdx.x;
  int* hist = reinterpret_cast<int*>(smem + n_words);       // bucket nqb - count
  for (int i = tid; i < n_words + a.nqb + 1; i += 256) smem[i] = 0;
  __syncthreads();
  const int32_t* sel_h = a.sel + (size_t)h * a.nqb * a.k;
  const int n_sel = a.nqb * a.k;
  for (int e0 = tid; e0 < n_sel; e0 += 8 * 256) {
    int v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = e0 + j * 256 < n_sel ? sel_h[e0 + j * 256] : -1;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      if (v[j] >= 0 && v[j] < a.n_loc) {
        const int i = (e0 + j * 256) / a.k;
        atomicOr(&smem[v[j] * W + (i >> 5)], 1u << (i & 31));
      }
  }
  __syncthreads();
  auto count = [&](int l) {
    int c = 0;
    for (int w = 0; w < W; ++w) c += __popc(smem[l * W + w]);
    return c;
  };
  for (int l = tid; l < a.n_loc; l += 256) atomicAdd(&hist[a.nqb - count(l)], 1);
  for (int i = tid; i < n_words; i += 256) a.att[(size_t)h * a.n_loc_cap * W + i] = smem[i];
  __syncthreads();
  if (tid < 64) {                          // counts -> first positions
    int before = 0;
    for (int b0 = 0; b0 <= a.nqb; b0 += 64) {
      const int mine = b0 + tid <= a.nqb ? hist[b0 + tid] : 0;
      int sum = mine;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int up = __shfl_up(sum, d, 64);
        if (tid >= d) sum += up;
      }
      if (b0 + tid <= a.nqb) hist[b0 + tid] = before + sum - mine;
      before += __shfl(sum, 63, 64);
    }
  }
  __syncthreads();
  for (int l = tid; l < a.n_loc; l += 256) {
    const int c = count(l), slot = a.l_map[l], len = min(max(a.l_len[l], 0), a.B);
    const bool ok = slot >= 0 && slot < a.n_loc_cap;
    a.order[(size_t)h * a.n_loc_cap + atomicAdd(&hist[a.nqb - c], 1)] = make_int4(l, ok ? slot : -1, len, c);
  }
}

template <int D>
__global__ void __launch_bounds__(256) bwd_prep_kernel(BwdArgs a) {
  extern __shared__ uint32_t plan_s[];
  constexpr int LPR = D / 8;               // lanes per row
  if ((int)blockIdx.x < a.H) {
    plan_head(a, (int)blockIdx.x, plan_s);
    return;
  }
  const long idx = (long)(blockIdx.x - a.H) * 256 + threadIdx.x;
  const long row = idx / LPR, per_head = row_blocks(a.Nq) * 32;
  const int part = (int)(idx % LPR);
  const int h = (int)(row / per_head), t = (int)(row % per_head);
  float acc = 0.0f;
  const bool ok = h < a.H && t < a.Nq;
  if (ok) {
    const size_t off = (size_t)h * a.o_stride_h + (size_t)t * a.o_stride_t + 8 * part;
    const bf16x8 o = *reinterpret_cast<const bf16x8*>(a.O + off);
    const bf16x8 g = *reinterpret_cast<const bf16x8*>(a.dO + off);
#pragma unroll
    for (int x = 0; x < 8; ++x) acc = __builtin_fmaf((float)o[x], (float)g[x], acc);
  }
#pragma unroll
  for (int s = 1; s < LPR; s <<= 1) acc += __shfl_xor(acc, s, 64);
  if (h < a.H && part == 0) {
    float* at = a.rows + (row / 32) * 64 + row % 32;
    at[0] = ok ? -a.lse[(size_t)h * a.Nq + t] * kLog2e : -INFINITY;
    at[32] = -acc;
  }
}

// 32 rows of an output, NT tiles of 32 dimensions each, whose transpose a wave holds in its accumulators (element v of tile
// dt is dim 32 dt + 8 (v / 4) + 4 (lane / 32) + v % 4 of row lane % 32), times `scale`, to memory, rows [0, n_rows) of them,
// through 4 NT KiB of LDS that nobody else uses: a lane's 16 bytes of a row go to LDS at chunk c ^ row and leave in
// instructions of 1 KiB.  Straight from the accumulators an instruction would write 32 bytes of each of 32 rows: 691.8 ->
// 685.5 us for select, forward and backward at 12 x 4680 x 128 with 32 + 48 blocks of 64, 430.4 -> 426.0 with 8 + 16 blocks of
// 128, 165.1 -> 162.7 at 16 x 2048 x 128.
template <int NT>
__device__ __forceinline__ void store_rows(float* dst, int pitch, const f32x16* o, float scale, int n_rows, unsigned char* scratch) {
  constexpr int CHUNKS = 8 * NT, RPS = 64 / CHUNKS;        // 16-byte chunks per row, rows per store instruction
  const int lane = threadIdx.x & 63, row = lane & 31, half = lane >> 5;
  float4* const lds = reinterpret_cast<float4*>(scratch);
#pragma unroll
  for (int dt = 0; dt < NT; ++dt)
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4)
      lds[row * CHUNKS + ((8 * dt + 2 * v4 + half) ^ (row & (CHUNKS - 1)))] =
          make_float4(o[dt][4 * v4] * scale, o[dt][4 * v4 + 1] * scale, o[dt][4 * v4 + 2] * scale, o[dt][4 * v4 + 3] * scale);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // other lanes' writes
#pragma unroll
  for (int i = 0; i < 32 / RPS; ++i) {
    const int r = RPS * i + lane / CHUNKS, c = lane % CHUNKS;
    const float4 v = lds[r * CHUNKS + (c ^ (r & (CHUNKS - 1)))];
    if (r < n_rows) *reinterpret_cast<float4*>(dst + (size_t)r * pitch + 4 * c) = v;
  }
}

// Partial sums change hands through LDS: a wave's accumulator tiles, one KiB per four elements and wave instruction.
template <int NT>
__device__ __forceinline__ void give_tiles(const f32x16* o, unsigned char* to) {
  float4* const lds = reinterpret_cast<float4*>(to) + (threadIdx.x & 63);
#pragma unroll
  for (int dt = 0; dt < NT; ++dt)
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4)
      lds[(4 * dt + v4) * 64] = make_float4(o[dt][4 * v4], o[dt][4 * v4 + 1], o[dt][4 * v4 + 2], o[dt][4 * v4 + 3]);
}
template <int NT>
__device__ __forceinline__ void add_tiles(f32x16* o, const unsigned char* from) {
  const float4* const lds = reinterpret_cast<const float4*>(from) + (threadIdx.x & 63);
#pragma unroll
  for (int dt = 0; dt < NT; ++dt)
#pragma unroll
    for (int v4 = 0; v4 < 4; ++v4) {
      const float4 x = lds[(4 * dt + v4) * 64];
      o[dt][4 * v4] += x.x;
      o[dt][4 * v4 + 1] += x.y;
      o[dt][4 * v4 + 2] += x.z;
      o[dt][4 * v4 + 3] += x.w;
    }
}

// ------------------------------------------------------------------------------------------------
// dkv: one workgroup per 64-key tile, NP pairs of waves with 1 / NP of its walk each; in a pair a wave has 32 keys
// ------------------------------------------------------------------------------------------------
template <int D, int NP>
__device__ __forceinline__ void dkv_body(const BwdArgs& a, const int block, unsigned char* smem_wg) {
  constexpr int kThreads = 128 * NP;
  constexpr int KS = D / 16, DT = D / 32, ROW = D * 2, TILE = kTile * ROW;
  constexpr int CH = D / 8, RPI = 64 / CH;          // 16-byte chunks per row, rows per load instruction
  constexpr int NI = 32 / RPI;                      // load instructions per wave per tile (its 32 rows)
  constexpr int HI_XOR = CH == 16 ? 16 : 0;         // row + 8 flips the lowest bit of the chunk permutation when it has 4 bits
  __shared__ int cnt_s[2 * 8];
  __shared__ __align__(256) float rows_wg[NP * 4 * 64];   // per ring entry, the scalars of the half tile's rows (BwdArgs::rows)
  // a ring for each pair of waves -- entry e holds a half of T1 at e TILE and of T2 behind it -- and, behind the rings, per
  // streamed tile: where it is
  int* lst_a = reinterpret_cast<int*>(smem_wg + NP * 4 * TILE);
  const int SUB = a.B / kTile;
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave_wg = __builtin_amdgcn_readfirstlane(tid >> 6), pair = wave_wg >> 1, wave = wave_wg & 1;
  unsigned char* const smem = smem_wg + pair * (4 * TILE);
  float* const rows_f = rows_wg + pair * 256;
  const int qn = lane & 31, half = lane >> 5;
  const float c2 = a.scale * kLog2e;

  // ---- what this workgroup is, and the list of streamed tiles ------------------------------------
  // The workgroup's 64-key tile: persistent (slot c) or local (logical block l).  A head's tiles have ranks, the
  // persistent ones first (every query block attends them: their walks are the longest), then the local ones from the
  // most attended to the least, and the grid goes through all heads rank by rank: a long walk that starts late ends the
  // launch late (with the local tiles in block order the last fifth of the launch ran less than half full).  12 heads x
  // 4680 x 128, with sel scanned once per head instead of once per tile: 32 + 48 blocks of 64 423 -> 355 us, 8 + 16 blocks of
  // 128 264 -> 225 us.
  const int n_pers = (a.C + 1) * SUB, n_ranks = n_pers + a.n_loc * SUB, n_cand = a.nqb * SUB;
  int h, rank;
  head_item(block, a.H, h, rank);
  if (rank >= n_ranks) return;             // the last eight ranks of a head need not be full
  const bool kv_local = rank >= n_pers;
  int fixed_len = 0, kv_slot_tile = 0;
  const uint32_t* att = a.att;             // the local block's row
  if (!kv_local) {
    const int c = rank / SUB, sub = rank % SUB;
    fixed_len = min(max(min(max(a.p_len[(size_t)h * (a.C + 1) + c], 0), a.B) - sub * kTile, 0), kTile);
    kv_slot_tile = rank;
  } else {
    const int4 o = a.order[(size_t)h * a.n_loc_cap + (rank - n_pers) / SUB];
    const int sub = (rank - n_pers) % SUB;
    if (o.y < 0) return;                   // a block that is nowhere: nothing to write either
    att += ((size_t)h * a.n_loc_cap + o.x) * ((a.nqb + 31) / 32);
    fixed_len = o.w > 0 ? min(max(o.z - sub * kTile, 0), kTile) : 0;
    kv_slot_tile = o.y * SUB + sub;
  }
  const size_t base = kv_local ? ((size_t)h * a.n_loc_cap * a.B + (size_t)kv_slot_tile * kTile) * D
                               : ((size_t)h * (a.C + 1) * a.B + (size_t)kv_slot_tile * kTile) * D;
  float* const dk = (kv_local ? a.dKl : a.dKp) + base;
  float* const dv = (kv_local ? a.dVl : a.dVp) + base;
  if (fixed_len == 0) {                    // no key, or nobody attends them
    for (int i = 4 * tid; i < kTile * D; i += 4 * kThreads) {
      *reinterpret_cast<float4*>(dk + i) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
      *reinterpret_cast<float4*>(dv + i) = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    }
    return;
  }

  // ---- fixed fragments (B operands): fixed row 32 w + lane % 32, dims 16 ks + 8 (lane / 32) .. + 8 ----
  // asked for before the list is built, so that they arrive meanwhile (with what prep leaves beside each block and the tiles
  // nobody attends written at once: select, forward and backward of 16 heads x 4000 x 64 with 4 + 8 blocks 164 -> 154 us)
  bf16x8 f1[KS], f2[KS];
  {
    const int row = min(32 * wave + qn, fixed_len - 1);
    const bf16_t* p1 = (kv_local ? a.Kl : a.Kp) + base + (size_t)row * D;
    const bf16_t* p2 = (kv_local ? a.Vl : a.Vp) + base + (size_t)row * D;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      f1[ks] = *reinterpret_cast<const bf16x8*>(p1 + 16 * ks + 8 * half);
      f2[ks] = *reinterpret_cast<const bf16x8*>(p2 + 16 * ks + 8 * half);
    }
  }

  // ---- the list of streamed tiles ----------------------------------------------------------------
  auto classify = [&](int i, int& where) -> bool {
    if (i >= n_cand) return false;
    const int ib = i / SUB;
    if (kv_local && !((att[ib >> 5] >> (ib & 31)) & 1u)) return false;
    where = i;                                      // row tile i covers tokens 64 i ..
    return a.Nq - i * kTile > 0;
  };
  constexpr int kMaxRounds = 8 / NP;       // 512 query blocks of two tiles / threads
  const int n_rounds = min((n_cand + kThreads - 1) / kThreads, kMaxRounds);
  // every candidate is looked at once (a look is a chain of dependent loads); what it found stays in registers
  // until the counts of all rounds are known
  int c_where[kMaxRounds];
  unsigned long long c_mask[kMaxRounds];
#pragma unroll
  for (int r = 0; r < kMaxRounds; ++r) {
    c_where[r] = 0;
    const bool on = r < n_rounds && classify(r * kThreads + tid, c_where[r]);
    c_mask[r] = __ballot(on);
    if (r < n_rounds && lane == 0) cnt_s[r * 2 * NP + wave_wg] = __popcll(c_mask[r]);
  }
  __syncthreads();
  int n_listed = 0;
  for (int q = 0; q < 2 * NP * n_rounds; ++q) n_listed += cnt_s[q];
#pragma unroll
  for (int r = 0; r < kMaxRounds; ++r) {
    if (r < n_rounds && ((c_mask[r] >> lane) & 1)) {
      int pos = lanes_below(c_mask[r]);
      for (int q = 0; q < r * 2 * NP + wave_wg; ++q) pos += cnt_s[q];
      lst_a[pos] = c_where[r];
    }
  }
  __syncthreads();
  // this pair's share of the list
  const int n_most = (n_listed + NP - 1) / NP, t_first = pair * n_most, n_tiles = min(n_most, n_listed - t_first);
  lst_a += t_first;

  // they have arrived before the walk starts: no wait for them inside it, where one would also wait for the tiles
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(f1[ks]), "+a"(f2[ks]));

  f32x16 out1[DT], out2[DT];               // dK^T and dV^T   (32 dims x 32 keys each)
#pragma unroll
  for (int dt = 0; dt < DT; ++dt)
#pragma unroll
    for (int v = 0; v < 16; ++v) out1[dt][v] = out2[dt][v] = 0.0f;
  // The output accumulators are only ever touched by the second products: they live in the accumulator half of the
  // register file for the whole walk (the products are issued as instructions with an accumulator destination), which
  // leaves the architectural half to the fragments, the first products' results and the elementwise stage.
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    asm volatile("" : "+a"(out1[dt]));
    asm volatile("" : "+a"(out2[dt]));
  }

  // ---- LDS addresses of this lane's operand reads ----------------------------------------------------
  // kept for one pair of ring entries each and moved to the other pair once per tile, so that everything else of an
  // address is a constant of the instruction: rd the row-wise reads, tl / th the transposing reads of rows r and r + 8,
  // sc_own / sc_next the row scalars of this tile's and of the next tile's pair
  const uint32_t smem_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const uint32_t ring_s = __builtin_amdgcn_readfirstlane(smem_lds);
  const uint32_t rows_s = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)rows_f);
  uint32_t rd[KS], tl[DT], th[DT];
  {
    const int kb = qn * ROW + ((half ^ swz<CH>(qn)) << 4);              // row lane % 32, logical chunk 2 ks + half
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rd[ks] = smem_lds + (uint32_t)(kb ^ (ks << 5));
    const int s16 = lane & 15, q16 = (lane >> 4) & 1;
    const int row0 = 4 * half + (s16 >> 2);                              // address row within 16 streamed rows
    const int sub = 2 * q16 + ((s16 & 3) >> 1), lo = (s16 & 1) * 8;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const uint32_t off = (uint32_t)(row0 * ROW + (((4 * dt + sub) ^ swz<CH>(row0)) << 4) + lo);
      tl[dt] = smem_lds + off;
      th[dt] = smem_lds + (off ^ HI_XOR) + 8 * ROW;
    }
  }
  uint32_t sc_own = rows_s + 16 * half, sc_next = sc_own + 512;

  // ---- staging -------------------------------------------------------------------------------------
  // The unit that travels is a half tile: 32 streamed rows of T1 and of T2 and the scalars of those rows, one ring
  // entry of four.  Wave w brings rows 16 w .. 16 w + 15 of the half.  Every wave issues the same number of loads per
  // half tile, so that one count serves the wait; past the end of the list the last half tile is fetched again into an
  // entry whose contents are never used.
  constexpr int HALF = TILE / 2, NH = NI / 2;    // NH: load instructions per wave, tensor and half tile
  constexpr int PER = 2 * NH + 1;               // loads per wave and half tile
  const int rl = lane / CH;
  const long st1 = a.q_stride_t * 2, st2 = a.o_stride_t * 2;     // row strides of the streamed tensors in bytes
  // A load's address: tile base + the lane's offset within the tile, and its instruction offset k 1024 on top, which the
  // lane's offset takes back; both are moved by 3 KiB against each other so that the offset is not below zero.
  constexpr int BIAS = 3072;
  const unsigned char* const b1 = reinterpret_cast<const unsigned char*>(a.Q + (size_t)h * a.q_stride_h) - BIAS;
  const unsigned char* const b2 = reinterpret_cast<const unsigned char*>(a.dO + (size_t)h * a.o_stride_h) - BIAS;
  const float* const rows_g = a.rows + (size_t)h * row_blocks(a.Nq) * 64;
  uint32_t so1[2][NH], so2[2][NH];         // [half][load]
  auto set_offsets = [&](int last) {       // rows past `last`: that row again
#pragma unroll
    for (int mg = 0; mg < 2; ++mg)
#pragma unroll
      for (int k = 0; k < NH; ++k) {
        const int r = 16 * wave + RPI * k + rl, src_row = min(32 * mg + r, last);
        const uint32_t chunk = (uint32_t)(((lane % CH) ^ swz<CH>(r)) << 4) + (uint32_t)(BIAS - k * 1024);
        so1[mg][k] = (uint32_t)(src_row * st1) + chunk;
        so2[mg][k] = (uint32_t)(src_row * st2) + chunk;
      }
  };
  set_offsets(kTile - 1);
  // a head's last row tile need not be full; it is the last of every list it is in, so the offsets change once
  const int ragged = a.Nq % kTile ? a.Nq / kTile : -1;
  const unsigned char* s1 = b1;            // the tile that is being fetched
  const unsigned char* s2 = b2;
  uint32_t rows_off = 0;
  auto stage_tile = [&](int where) {
    s1 = b1 + (size_t)where * kTile * st1;
    s2 = b2 + (size_t)where * kTile * st2;
    rows_off = (uint32_t)lane * 4u + (uint32_t)(where * 512);
  };
  // load i of a half: Q and dO in turn, then the scalars of the half's 32 rows (both waves bring the same)
  auto stage_one = [&](auto MG, auto I, uint32_t ring_at, uint32_t rows_at) {
    constexpr int mg = decltype(MG)::value, i = decltype(I)::value, k = i / 2;
    if constexpr (i < 2 * NH) {
      if constexpr (i % 2 == 0) dma16_at<k * 1024>(s1, so1[mg][k], ring_at + mg * TILE);
      else dma16_at<k * 1024>(s2, so2[mg][k], ring_at + mg * TILE + HALF);
    } else {
      dma4(rows_g + 64 * mg, rows_off, rows_at + mg * 256);
    }
  };
  auto stage_half = [&](auto MG, uint32_t ring_at, uint32_t rows_at) {
    unroll([&](auto I) { stage_one(MG, I, ring_at, rows_at); }, std::make_integer_sequence<int, PER>{});
  };
  uint32_t ring_at = ring_s + (uint32_t)(wave * (HALF / 2)), rows_at = rows_s;    // of the pair of entries of tile t

  // ---- the walk: a software pipeline over half tiles ---------------------------------------------------
  // Turn u, in two phases.  First: the first products of half tile u + 1 (2 KS MFMAs, their row fragments already in
  // registers), each with a slice of half tile u's elementwise stage behind it and, over the middle slices, the
  // transposing reads of half tile u.  Then a wait and the turn's one barrier: half tile u + 2 has landed, and nobody
  // reads half tile u any more.  Second: the second products of half tile u (4 DT MFMAs), each with a row fragment of
  // half tile u + 2 read behind it; half tile u + 4 is sent for, into the entry u has left, a load behind each product.
  // (The loads in bursts of four, their addresses computed there and then, held the wave up for some 150 cycles a turn: with
  // that, and addresses moved to the other ring entries where they were last used instead of behind the turn, 57.3 -> 53.1 us
  // at 3 x 1500 x 64, 133.7 -> 125.6 at 4 x 3000 x 128, 432.5 -> 425.5 at 12 x 4680 x 128 with 8 + 16 blocks of 128.  The large
  // ones are held by power: with zeros for data the same walks take 20 % less, at a higher clock.)
  // The compiler orders instructions without side effects as it likes: left alone it issued all the elementwise work
  // behind the last MFMA, and a turn took 2700 cycles for 1024 cycles of matrix work, on a compute unit of its own too
  // (12 heads x 4680 x 128 with 32 + 48 blocks of 64: select, forward and backward 969 -> 835 us; 8 + 16 blocks of 128: 640 ->
  // 552 us).  An empty asm with the value as its operand (pin) keeps each MFMA and each slice where it stands.
  // Per element: fma, exp2, multiply, half of two conversions.  The row's -D is what the accumulator starts from, and
  // rows that do not exist have -inf in the place of their -lse log2 e: their P is an exact zero without a mask.
  constexpr int NS = 2 * KS, EPS = 16 / NS;                // slices, accumulator elements per slice
  static_assert(EPS * NS == 16 && (EPS == 1 || EPS == 2), "slices cover the 16 elements");
  constexpr int NTF = 4 * DT;                              // transposed fragments of a half tile: [tensor][j][dt]
  static_assert(NTF == NS, "a row fragment behind every second product, two transposed ones per middle slice");
  const f32x16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  f32x16 c1 = zero, c2a = zero;            // A1, A2 - D of the half tile whose elementwise stage comes next
  bf16x8 x[NS];                            // row fragments: x[2 ks] of T1, x[2 ks + 1] of T2
  f32x16 dn;                               // -D of the rows those fragments hold, in accumulator order
  f32x4 nl0;                              // -lse log2 e of the first four rows of the next elementwise stage
  auto read_scalar4 = [&](uint32_t addr) { return *(lds_f4_t)(uintptr_t)addr; };
  auto read_dn4 = [&](uint32_t addr, int g) {
    const f32x4 v = read_scalar4(addr + 128 + 32 * g);
    dn[4 * g] = v.x; dn[4 * g + 1] = v.y; dn[4 * g + 2] = v.z; dn[4 * g + 3] = v.w;
  };
  auto read_dn = [&](uint32_t addr) {
#pragma unroll
    for (int g = 0; g < 4; ++g) read_dn4(addr, g);
  };
  int v_where = 0;                         // the tile after the one that is being fetched
  if (n_tiles > 0) {
    for (int j = 0; j < 2; ++j) {          // two tiles (the last one again where there is only one)
      const int where = __builtin_amdgcn_readfirstlane(lst_a[min(j, n_tiles - 1)]);
      if (where == ragged) set_offsets(a.Nq - where * kTile - 1);
      stage_tile(where);
      stage_half(std::integral_constant<int, 0>{}, ring_at + j * 2 * TILE, rows_at + j * 512);
      stage_half(std::integral_constant<int, 1>{}, ring_at + j * 2 * TILE, rows_at + j * 512);
    }
    v_where = lst_a[min(2, n_tiles - 1)];
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(2 * PER) : "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < NS; ++i) x[i] = lds_read_row(rd[i / 2] + (i % 2) * HALF);
    read_dn(sc_own);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      c1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[2 * ks], f1[ks], c1, 0, 0, 0);
      c2a = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[2 * ks + 1], f2[ks], ks == 0 ? dn : c2a, 0, 0, 0);
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < NS; ++i) x[i] = lds_read_row(rd[i / 2] + TILE + (i % 2) * HALF);
    read_dn(sc_own + 256);
    nl0 = read_scalar4(sc_own);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rd[ks] += 2 * TILE;     // the turns of tile t read the rows of tile t + 1
    // all here before the loop: inside it, only as much is waited for as the loop itself has outstanding
#pragma unroll
    for (int i = 0; i < NS; ++i) asm volatile("" : "+v"(x[i]));
    asm volatile("" : "+v"(dn), "+v"(nl0), "+v"(v_where));
  }
  uint32_t step = 2 * TILE, sc_step = 512;                  // to the other pair of ring entries and back
  // Two turns per tile, so that the accumulator sets trade places by name (no copies) and the half is a constant.
  auto turn = [&](auto MG, int t, f32x16& c1, f32x16& c2a, f32x16& n1, f32x16& n2) {
    constexpr int mg = decltype(MG)::value;
    int where = 0;
    if constexpr (mg == 0) {
      where = __builtin_amdgcn_readfirstlane(v_where);
      if (where == ragged) set_offsets(a.Nq - where * kTile - 1);
    }
    float nl[16], ex[16], zz[16];
    nl[0] = nl0.x; nl[1] = nl0.y; nl[2] = nl0.z; nl[3] = nl0.w;
    u32x4 eP[2], eZ[2];
    bf16x8 tf[NTF];
    auto finish = [&](int v) {             // the later half of an element, a slice behind its exponential
      zz[v] = ex[v] * c2a[v];
      if (v % 2 == 1) {
        eP[v / 8][(v % 8) / 2] = pack2(ex[v - 1], ex[v]);
        eZ[v / 8][(v % 8) / 2] = pack2(zz[v - 1], zz[v]);
        asm volatile("" : "+v"(eP[v / 8][(v % 8) / 2]), "+v"(eZ[v / 8][(v % 8) / 2]));
      }
    };
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) {
      const int ks = sl / 2;
      if (sl % 2 == 0) {
        n1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[sl], f1[ks], ks == 0 ? zero : n1, 0, 0, 0);
        asm volatile("" : "+v"(n1));
      } else {
        n2 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[sl], f2[ks], ks == 0 ? dn : n2, 0, 0, 0);
        asm volatile("" : "+v"(n2));
      }
      __builtin_amdgcn_sched_barrier(0);   // the MFMA first, then the slice
      // accumulator element v: streamed row 32 mg + 8 (v / 4) + 4 half + v % 4, fixed row 32 w + lane % 32
      if (sl * EPS % 4 == 0 && sl * EPS < 12) {              // the scalars of the next four rows
        const int g = sl * EPS / 4 + 1;
        const f32x4 v = read_scalar4(sc_own + 256 * mg + 32 * g);
        nl[4 * g] = v.x; nl[4 * g + 1] = v.y; nl[4 * g + 2] = v.z; nl[4 * g + 3] = v.w;
      }
      if (sl >= NS / 4 && sl < NS / 4 + NTF / 2) {
#pragma unroll
        for (int q = 0; q < 2; ++q) {
          const int i = 2 * (sl - NS / 4) + q, tensor = i / (2 * DT), j = (i / DT) % 2, dt = i % DT;
          const uint32_t at = (uint32_t)(mg * TILE + tensor * HALF + 16 * j * ROW);
          tf[i] = lds_read_tr(tl[dt] + at, th[dt] + at);
          if (mg == 1 && tensor == 1 && j == 1) {           // the last use this tile
            tl[dt] += step;
            th[dt] += step;
          }
        }
      }
      if (mg == 0 && sl == 1) stage_tile(where);
#pragma unroll
      for (int q = 0; q < EPS; ++q) {
        const int v = sl * EPS + q;
        ex[v] = __builtin_amdgcn_exp2f(__builtin_fmaf(c1[v], c2, nl[v]));
      }
#pragma unroll
      for (int q = 0; q < EPS; ++q)
        if (sl > 0) finish((sl - 1) * EPS + q);
#pragma unroll
      for (int q = 0; q < EPS; ++q) asm volatile("" : "+v"(ex[sl * EPS + q]));
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int q = 0; q < EPS; ++q) finish((NS - 1) * EPS + q);
    // this wave's rows of half tile u + 2 are in and its reads of half tile u done; then everybody's
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(PER) : "memory");
    __builtin_amdgcn_s_waitcnt(0xC07F);    // lgkmcnt(0), in the form the compiler counts
    __builtin_amdgcn_s_barrier();
    asm volatile("s_nop 4" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
    unroll([&](auto I) {
      constexpr int i = decltype(I)::value, tensor = i % 2, j = i / (2 * DT), dt = (i / 2) % DT;
      acc_mfma(tensor ? out2[dt] : out1[dt], tf[(2 * tensor + j) * DT + dt], as_bf16x8(tensor ? eP[j] : eZ[j]));
      __builtin_amdgcn_sched_barrier(0);
      x[i] = lds_read_row(rd[i / 2] + mg * TILE + (i % 2) * HALF);
      if constexpr (mg == 1 && i % 2 == 1) rd[i / 2] -= step;
      if constexpr (i >= 1 && i <= PER) stage_one(MG, std::integral_constant<int, i - 1>{}, ring_at, rows_at);
      if constexpr (i >= NTF / 2 - 2 && i < NTF / 2 + 2) read_dn4(sc_next + 256 * mg, i - (NTF / 2 - 2));
      if constexpr (i == NTF / 2 + 2) nl0 = read_scalar4(mg ? sc_next : sc_own + 256);
      if constexpr (mg == 1 && i == NTF / 2 + 3) {
        v_where = lst_a[min(t + 3, n_tiles - 1)];
        sc_own += sc_step;
        sc_next -= sc_step;
      }
      __builtin_amdgcn_sched_barrier(0);
    }, std::make_integer_sequence<int, NTF>{});
  };
  {
    f32x16 d1, d2;                         // the other accumulator set
    for (int t = 0; t < n_tiles; ++t) {
      turn(std::integral_constant<int, 0>{}, t, c1, c2a, d1, d2);
      turn(std::integral_constant<int, 1>{}, t, d1, d2, c1, c2a);
      ring_at += step;
      rows_at += sc_step;
      step = 0u - step;
      sc_step = 0u - sc_step;
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");         // the trailing loads land before the ring is used otherwise
  if constexpr (NP > 1)                    // a pair with a shorter share meets the other's barriers
    for (int i = 2 * max(n_tiles, 0) + (n_tiles > 0); i < 2 * n_most + (n_most > 0); ++i) __builtin_amdgcn_s_barrier();
  // the compiler does not see the matrix instructions that wrote the output accumulators: let the pipe drain
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    asm volatile("s_nop 15\n\ts_nop 15" : "+a"(out1[dt]));
    asm volatile("" : "+a"(out2[dt]));
  }

  // ---- outputs -------------------------------------------------------------------------------------
  // every row of the tile's slot is written: zeros past the valid length and for a block nobody attends
  __syncthreads();                         // the rings are dead: what any wave fetched last has landed
  const bool exists = 32 * wave + qn < fixed_len;
  unsigned char* const mine = smem + wave * (2 * TILE);
  const size_t row0 = (size_t)(32 * wave) * D;
  const float k_scale = exists ? a.scale : 0.0f, v_scale = exists ? 1.0f : 0.0f;
  if constexpr (NP == 1) {
    store_rows<DT>(dk + row0, D, out1, k_scale, 32, mine);
    store_rows<DT>(dv + row0, D, out2, v_scale, 32, mine + TILE);
  } else {
    // the first pair finishes dK, the second dV
    const unsigned char* const theirs = smem_wg + (pair ^ 1) * (4 * TILE) + wave * (2 * TILE);
    if (pair == 0) give_tiles<DT>(out2, mine);
    else give_tiles<DT>(out1, mine);
    __syncthreads();
    if (pair == 0) {
      add_tiles<DT>(out1, theirs);
      store_rows<DT>(dk + row0, D, out1, k_scale, 32, mine + TILE);
    } else {
      add_tiles<DT>(out2, theirs);
      store_rows<DT>(dv + row0, D, out2, v_scale, 32, mine + TILE);
    }
  }
}

// ------------------------------------------------------------------------------------------------
// dq with 64 query rows per wave (two MFMA column groups of 32), so that every K or V fragment read from LDS -- row-wise
// for the first products, transposed for the second -- feeds two MFMAs.  The wave stages its own half tiles (32 keys of K
// and of V per ring entry, two entries) and is the only one to read them: no barrier in the walk.  The two waves of a
// workgroup have a row tile each or, dq_split, half of one row tile's walk each, four a quarter of it: the sums meet in LDS
// at the end and are added in the order of the waves.  Q and dO fragments and the dQ^T accumulators fill the accumulator
// half of the register file (128 + 128 registers at d = 128).  Bound at 12 x 4680 x 128: matrix and vector work in one wave per SIMD at the clock the
// chip holds under it (222 GFLOP in 215 us, 1.03 PFLOP/s; a library product of 8192^3 reaches 1.19).  The elementwise stages
// are spread over 40 of a turn's 48 MFMAs; over 28 of them: 712.8 against 708.3 us for select, forward and backward, 89.8
// against 88.2 at 3 x 1500 x 64.  Two waves to a workgroup that share the tiles both attend (half the traffic with
// 128-token blocks, three half tiles on their way): 217 us, and 35.3 against 32.6 at 3 x 1500 x 64, where it lost.
// ------------------------------------------------------------------------------------------------
template <int D, int NWV>
__device__ __forceinline__ void dq_body(const BwdArgs& a, const int block, unsigned char* smem_wg) {
  constexpr int KS = D / 16, DT = D / 32, ROW = D * 2, TILE = kTile * ROW, HALF = TILE / 2;
  constexpr int CH = D / 8, RPI = 64 / CH;          // 16-byte chunks per row, rows per load instruction
  constexpr int NW = (32 / RPI) / 4;                // windows of four load instructions per tensor and half tile: 2 or 1
  constexpr int HI_XOR = CH == 16 ? 16 : 0;
  constexpr int NS = 2 * KS;                        // slices behind the first products
  const int SUB = a.B / kTile;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
  const int qn = lane & 31, half = lane >> 5;
  const int n_pers = (a.C + 1) * SUB, n_cand = n_pers + a.k * SUB;
  // each wave has a ring of its own -- entry e holds 32 rows of K at e * TILE and 32 rows of V behind them -- and, behind
  // the rings, a list
  unsigned char* const smem = smem_wg + wave * (2 * TILE);
  uint32_t* const lst = reinterpret_cast<uint32_t*>(smem_wg + NWV * 2 * TILE) + wave * n_cand;
  int h, r_tile;
  head_item(block, a.H, h, r_tile);
  const bool share = NWV == 4 || (NWV == 2 && a.dq_split);  // the waves share one row tile's walk
  if (!share) r_tile = NWV * r_tile + wave;
  if (r_tile * kTile >= a.Nq) return;
  const float c2 = a.scale * kLog2e;
  const int i_blk = r_tile * kTile / a.B;
  const int fixed_len = min(kTile, a.Nq - r_tile * kTile);

  // ---- the tiles these rows attend: persistent slots, then the blocks of their row of sel -----------------
  // the library takes rings of H * n_loc_cap * d * 4 < 2^32, with blocks of up to two tiles
  constexpr int kTileBits = 25;
  static_assert(2 * ((1ll << 32) / (64 * 4)) <= 1ll << kTileBits && kTile <= 1 << (31 - kTileBits), "one word per tile");
  int n_tiles = 0;
  for (int i0 = 0; i0 < n_cand; i0 += 64) {
    const int i = i0 + lane;
    uint32_t where = 0;                    // bit 31 local, bits 25 .. 30 rows - 1, the tile in the cache's tensor
    int rows = 0;
    if (i < n_pers) {
      const int c = i / SUB, sub = i % SUB;
      rows = min(max(min(max(a.p_len[(size_t)h * (a.C + 1) + c], 0), a.B) - sub * kTile, 0), kTile);
      where = (uint32_t)i;
    } else if (i < n_cand) {
      const int jj = (i - n_pers) / SUB, sub = (i - n_pers) % SUB;
      const int l = a.sel[((size_t)h * a.nqb + i_blk) * a.k + jj];
      if (l >= 0 && l < a.n_loc) {
        const int slot = a.l_map[l];
        if (slot >= 0 && slot < a.n_loc_cap) {
          rows = min(max(min(max(a.l_len[l], 0), a.B) - sub * kTile, 0), kTile);
          where = 0x80000000u | (uint32_t)(slot * SUB + sub);
        }
      }
    }
    const unsigned long long m = __ballot(rows > 0);
    if (rows > 0) lst[n_tiles + lanes_below(m)] = where | (uint32_t)(rows - 1) << kTileBits;
    n_tiles += __popcll(m);
  }
  n_tiles = __builtin_amdgcn_readfirstlane(n_tiles);
  int t_first = 0;                         // the wave's share of the list
  if (share) {
    const int n_most = (n_tiles + NWV - 1) / NWV;
    t_first = wave * n_most;
    n_tiles = min(n_tiles, t_first + n_most);
  }

  // ---- fixed fragments (B operands) of both column groups: row 32 n + lane % 32, dims 16 ks + 8 (lane / 32) .. + 8 ----
  bf16x8 f1[2][KS], f2[2][KS];
  float nl_fix[2], d_fix[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
    const int row = min(32 * n + qn, fixed_len - 1), tok = r_tile * kTile + row;
    const bf16_t* p1 = a.Q + (size_t)h * a.q_stride_h + (size_t)tok * a.q_stride_t;
    const bf16_t* p2 = a.dO + (size_t)h * a.o_stride_h + (size_t)tok * a.o_stride_t;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      f1[n][ks] = *reinterpret_cast<const bf16x8*>(p1 + 16 * ks + 8 * half);
      f2[n][ks] = *reinterpret_cast<const bf16x8*>(p2 + 16 * ks + 8 * half);
    }
    const float l = a.lse[(size_t)h * a.Nq + tok];
    nl_fix[n] = 32 * n + qn < fixed_len && l > -INFINITY ? -l * kLog2e : -INFINITY;
    d_fix[n] = a.rows[((size_t)h * row_blocks(a.Nq) + tok / 32) * 64 + 32 + tok % 32];
  }
  // only ever MFMA operands: they live in the accumulator half of the register file (and have arrived: no wait
  // for them inside the walk, where one would also wait for the tiles)
#pragma unroll
  for (int n = 0; n < 2; ++n) {
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) asm volatile("" : "+a"(f1[n][ks]), "+a"(f2[n][ks]));
    asm volatile("" : "+v"(nl_fix[n]));
  }
  // -D of the lane's query row of each group, sixteen times: what the dP accumulators start from
  f32x16 dn[2];
#pragma unroll
  for (int n = 0; n < 2; ++n) {
#pragma unroll
    for (int v = 0; v < 16; ++v) dn[n][v] = d_fix[n];
    asm volatile("" : "+v"(dn[n]));
  }
  f32x16 out[2][DT];                       // dQ^T: 32 dims x 32 rows per tile
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
#pragma unroll
      for (int v = 0; v < 16; ++v) out[n][dt][v] = 0.0f;
      asm volatile("" : "+a"(out[n][dt]));
    }

  // ---- LDS addresses of this lane's operand reads inside ring entry 0 ----------------------------------
  const uint32_t smem_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const uint32_t ring_s = __builtin_amdgcn_readfirstlane(smem_lds);
  uint32_t rd[KS], tl[DT], th[DT];         // row-wise reads; transposing reads of rows r and r + 8
  {
    const int kb = qn * ROW + ((half ^ swz<CH>(qn)) << 4);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) rd[ks] = smem_lds + (uint32_t)(kb ^ (ks << 5));
    const int s16 = lane & 15, q16 = (lane >> 4) & 1;
    const int row0 = 4 * half + (s16 >> 2);
    const int sub = 2 * q16 + ((s16 & 3) >> 1), lo = (s16 & 1) * 8;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      const uint32_t off = (uint32_t)(row0 * ROW + (((4 * dt + sub) ^ swz<CH>(row0)) << 4) + lo);
      tl[dt] = smem_lds + off;
      th[dt] = smem_lds + (off ^ HI_XOR) + 8 * ROW;
    }
  }

  // ---- staging: the wave brings whole half tiles (32 rows of K and of V, dense rows) ---------------------
  // in windows of 4 KiB (four loads of K, four of V).  A load's address: its window's base + the lane's offset in it + the
  // instruction's own offset, which the lane's offset takes back; the offsets are moved up by BIAS and the bases down, so
  // that a lane that fetches an earlier row than its own does not go below zero.
  constexpr int WROWS = 4 * RPI;           // rows of a window (the permutation repeats within them)
  constexpr uint32_t BIAS = 16384;
  static_assert((kTile - WROWS) * ROW + 3072 <= (int)BIAS, "no lane's offset is below zero");
  uint32_t so[4];
  auto set_offsets = [&](int first, int last) {             // rows first .. of the tile; past `last`: that row again
    int ln = lane;
    asm volatile("" : "+v"(ln));           // worked out here, not kept in registers throughout the walk
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int r = RPI * k + ln / CH;
      so[k] = (uint32_t)((min(first + r, last) - first) * ROW + (((ln % CH) ^ swz<CH>(r)) << 4) + (int)BIAS - k * 1024);
    }
  };
  set_offsets(0, kTile);
  const size_t hl = (size_t)h * a.n_loc_cap * a.B * D * 2 - BIAS, hp = (size_t)h * (a.C + 1) * a.B * D * 2 - BIAS;
  const unsigned char* const kl = reinterpret_cast<const unsigned char*>(a.Kl) + hl;
  const unsigned char* const vl = reinterpret_cast<const unsigned char*>(a.Vl) + hl;
  const unsigned char* const kp = reinterpret_cast<const unsigned char*>(a.Kp) + hp;
  const unsigned char* const vp = reinterpret_cast<const unsigned char*>(a.Vp) + hp;
  const unsigned char* s1 = kl;            // the tile that is being fetched
  const unsigned char* s2 = vl;
  int s_last = 0;                          // its last row
  auto stage_tile = [&](int word) {
    const size_t off = (size_t)(word & ((1 << kTileBits) - 1)) * TILE;
    s1 = (word < 0 ? kl : kp) + off;
    s2 = (word < 0 ? vl : vp) + off;
    s_last = (word >> kTileBits) & (kTile - 1);
  };
  // load i of half MG of that tile, into ring entry MG: window by window, K and V in turn.  A tile that is not full has
  // its offsets set before each window and set back behind the last.
  auto stage_one = [&](auto MG, auto I) {
    constexpr int mg = decltype(MG)::value, i = decltype(I)::value, w = i / 8, k = i % 8 / 2;
    constexpr int first = 32 * mg + WROWS * w;
    if constexpr (i % 8 == 0)
      if (s_last < first + WROWS - 1) set_offsets(first, s_last);
    dma16_at<k * 1024>((i % 2 ? s2 : s1) + first * ROW, so[k], ring_s + (uint32_t)(mg * TILE + (i % 2) * HALF + w * 4096));
    if constexpr (i == 8 * NW - 1)
      if (s_last < 32 * mg + 31) set_offsets(0, kTile);
  };

  // ---- the walk ------------------------------------------------------------------------------------------
  // A turn works on one half tile u, whose row fragments are in registers when it starts:
  //   1  the first products of column group 0            (2 KS MFMAs), behind them the elementwise stage of group 1, u - 1
  //   2  the second products of group 1, u - 1           (2 DT)
  //   3  the first products of group 1                   (2 KS), behind them the elementwise stage of group 0 and the
  //                                                      transposing reads of u
  //      then half tile u + 1 has landed (it was sent for a turn ago)
  //   4  the second products of group 0                  (2 DT), behind them the row reads of u + 1 and, two loads
  //                                                      behind each product, the fetching of u + 2
  // The last quarter of an elementwise stage runs behind the first DT of the second products that follow it: those need
  // its first half only.  Per element: fma, exp2, multiply, half of a conversion; -D is what the dP accumulators start
  // from, and in a tile that is not full a key past the end has -inf in the score accumulator's start (the scale is positive),
  // so its P is an exact zero; a full tile's accumulators start from the constant 0.  The empty asm statements keep MFMAs
  // and slices where they stand; without them the compiler issues all the elementwise work behind the last MFMA of its phase.
  // Select, forward and backward with the loads in bursts of four and the score accumulators' start kept in registers,
  // against this: 657.9 -> 653.3 us at 12 x 4680 x 128 with 32 + 48 blocks of 64, 409.5 -> 406.7 with 8 + 16 blocks of 128,
  // 389.4 -> 381.5 at 12 x 4680 x 64, 159.4 -> 157.8 at 16 x 2048 x 128.
  bf16x8 x[NS];                            // row fragments: x[2 ks] of K, x[2 ks + 1] of V
  // the list's words of the tile of the turn and of the tile that is fetched meanwhile, and, still on its way, the next one's
  int w_own = 0, w_next = 0, v_word = 0;
  if (t_first < n_tiles) {
    w_own = __builtin_amdgcn_readfirstlane((int)lst[t_first]);
    w_next = __builtin_amdgcn_readfirstlane((int)lst[min(t_first + 1, n_tiles - 1)]);
    stage_tile(w_own);
    unroll([&](auto I) { stage_one(std::integral_constant<int, 0>{}, I); }, std::make_integer_sequence<int, 8 * NW>{});
    unroll([&](auto I) { stage_one(std::integral_constant<int, 1>{}, I); }, std::make_integer_sequence<int, 8 * NW>{});
    asm volatile("s_waitcnt vmcnt(%0)" ::"n"(8 * NW) : "memory");
#pragma unroll
    for (int i = 0; i < NS; ++i) x[i] = lds_read_row(rd[i / 2] + (i % 2) * HALF);
#pragma unroll
    for (int i = 0; i < NS; ++i) asm volatile("" : "+v"(x[i]));
  }
  const f32x16 zero = {0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0, 0};
  f32x16 a1[2], a2[2];
  u32x4 eZ[2][2];
  bf16x8 tf[2 * DT];                       // transposed fragments: 16 keys j, 32 dims dt at j DT + dt
  float ex[2][16], zz[2][16];
  constexpr int E1 = 12;                   // elements of a stage that run behind the first products; E2 slots take the rest
  auto begin = [&](int n, int v) { ex[n][v] = __builtin_amdgcn_exp2f(__builtin_fmaf(a1[n][v], c2, nl_fix[n])); };
  auto finish = [&](int n, int v) {
    zz[n][v] = ex[n][v] * a2[n][v];
    if (v % 2 == 1) {
      eZ[n][v / 8][(v % 8) / 2] = pack2(zz[n][v - 1], zz[n][v]);
      asm volatile("" : "+v"(eZ[n][v / 8][(v % 8) / 2]));
    }
  };
  // elements [lo, hi) begun, [lo0, lo) finished
  auto slice = [&](int n, int lo0, int lo, int hi) {
#pragma unroll
    for (int v = lo; v < hi; ++v) begin(n, v);
#pragma unroll
    for (int v = lo0; v < lo; ++v) finish(n, v);
#pragma unroll
    for (int v = lo; v < hi; ++v) asm volatile("" : "+v"(ex[n][v]));
  };
  const auto nothing = [](auto) {};
  // the first products of group n and, behind them, elements 0 .. E1 - 1 of the other group's elementwise stage
  // accumulator element v: key 32 mg + 8 (v / 4) + 4 half + v % 4, query row 32 n + lane % 32.  Keys past the tile's
  // length hold a copy of its last row (`keys` of the half tile's exist); a query row that does not exist has nl = -inf.
  auto run_phase = [&](int n, auto PRODUCTS, int keys, auto behind) {
    const auto at = [](int sl) { return sl < 0 ? 0 : E1 * sl / NS; };
#pragma unroll
    for (int sl = 0; sl < NS; ++sl) {
      if constexpr (decltype(PRODUCTS)::value) {
        const int ks = sl / 2;
        if (sl == 0 && keys < 32) {
          f32x16 km;
          const int lim = keys - 4 * half;
#pragma unroll
          for (int v = 0; v < 16; ++v) km[v] = 8 * (v / 4) + (v % 4) < lim ? 0.0f : -INFINITY;
          a1[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[0], f1[n][0], km, 0, 0, 0);
          asm volatile("" : "+v"(a1[n]));
        } else if (sl % 2 == 0) {
          a1[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[sl], f1[n][ks], ks == 0 ? zero : a1[n], 0, 0, 0);
          asm volatile("" : "+v"(a1[n]));
        } else {
          a2[n] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x[sl], f2[n][ks], ks == 0 ? dn[n] : a2[n], 0, 0, 0);
          asm volatile("" : "+v"(a2[n]));
        }
        __builtin_amdgcn_sched_barrier(0);
      }
      behind(sl);
      slice(n ^ 1, at(sl - 1), at(sl), at(sl + 1));
      __builtin_amdgcn_sched_barrier(0);
    }
    // what the first DT of the second products need is finished before them
    static_assert(E1 * (NS - 1) / NS >= 8, "the first half of the elements is finished by the last slice");
    asm volatile("s_nop 4" ::: "memory");
  };
  // the second products of group n, the rest of its elementwise stage behind the first DT of them
  auto second_products = [&](auto N, auto behind) {
    constexpr int n = decltype(N)::value;
    constexpr int LAST = E1 * (NS - 1) / NS;                // begun in the last slice, not finished
    const auto at = [](int i) { return E1 + (16 - E1) * i / (DT - 1); };
    unroll([&](auto I) {
      constexpr int i = decltype(I)::value;
      if (i == DT) asm volatile("s_nop 4" ::: "memory");
      acc_mfma(out[n][i % DT], tf[i], as_bf16x8(eZ[n][i / DT]));
      __builtin_amdgcn_sched_barrier(0);
      behind(I);
      if (i < DT) slice(n, i == 0 ? LAST : at(i - 1), i < DT - 1 ? at(i) : 16, i < DT - 1 ? at(i + 1) : 16);
      __builtin_amdgcn_sched_barrier(0);
    }, std::make_integer_sequence<int, 2 * DT>{});
  };
  auto turn = [&](auto MG, int t) {
    constexpr int mg = decltype(MG)::value;                 // two turns per tile: the ring entry is the half
    if constexpr (mg == 0) {
      stage_tile(w_next);                  // past the end of the list the last tile again: nobody reads it
      v_word = (int)lst[min(t + 2, n_tiles - 1)];
    }
    const int keys = ((w_own >> kTileBits) & (kTile - 1)) + 1 - 32 * mg;
    __builtin_amdgcn_sched_barrier(0);
    run_phase(0, std::true_type{}, keys, nothing);
    second_products(std::integral_constant<int, 1>{}, nothing);
    {
      const uint32_t at0 = (uint32_t)(mg * TILE);
      run_phase(1, std::true_type{}, keys, [&](int sl) {
        if (sl >= NS / 4 && sl < NS / 4 + DT) {
#pragma unroll
          for (int r = 0; r < 2; ++r) {
            const int i = 2 * (sl - NS / 4) + r;
            const uint32_t at = at0 + (uint32_t)(16 * (i / DT) * ROW);
            tf[i] = lds_read_tr(tl[i % DT] + at, th[i % DT] + at);
          }
        }
      });
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // half tile u + 1 is in
    __builtin_amdgcn_s_waitcnt(0xC07F);                     // lgkmcnt(0): and u read (nobody else uses the ring)
    __builtin_amdgcn_sched_barrier(0);
    second_products(std::integral_constant<int, 0>{}, [&](auto I) {
      constexpr int i = decltype(I)::value;
      static_assert(8 * NW == 4 * DT, "two loads behind each product");
      stage_one(MG, std::integral_constant<int, 2 * i>{});
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        const int f = 2 * i + r;
        x[f] = lds_read_row(rd[f / 2] + (mg ^ 1) * TILE + (f % 2) * HALF);
      }
      stage_one(MG, std::integral_constant<int, 2 * i + 1>{});
    });
    if constexpr (mg == 1) {
      w_own = w_next;
      w_next = __builtin_amdgcn_readfirstlane(v_word);
    }
  };
  // before the first half tile: a stage of group 1 that adds nothing
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    a1[1][v] = -INFINITY;
    a2[1][v] = 0.0f;
  }
#pragma unroll
  for (int i = 0; i < 2 * DT; ++i) tf[i] = bf16x8{};
  if (t_first < n_tiles) {
    for (int t = t_first; t < n_tiles; ++t) {
      turn(std::integral_constant<int, 0>{}, t);
      turn(std::integral_constant<int, 1>{}, t);
    }
    run_phase(0, std::false_type{}, 32, nothing);               // group 1 of the last half tile
    second_products(std::integral_constant<int, 1>{}, nothing);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // the trailing loads land before the ring is used otherwise
  }
  // the compiler does not see the matrix instructions that wrote the output accumulators: let the pipe drain
#pragma unroll
  for (int n = 0; n < 2; ++n)
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) asm volatile("s_nop 15\n\ts_nop 15" : "+a"(out[n][dt]));
  if constexpr (NWV > 1) {
    if (share) {
      // every wave leaves its sums in its own ring, which nobody reads any more, and adds up its part of the tiles, in the
      // order of the waves: a column group (two waves), half of one (four)
      constexpr int NT = NWV == 4 ? DT / 2 : DT;
#pragma unroll
      for (int n = 0; n < 2; ++n) give_tiles<DT>(out[n], smem + n * TILE);
      __syncthreads();
      const int n = wave & 1, dt0 = (wave >> 1) * NT;
      const unsigned char* const from = smem_wg + n * TILE + dt0 * 4096;
      f32x16 sum[NT];
#pragma unroll
      for (int dt = 0; dt < NT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) sum[dt][v] = 0.0f;
#pragma unroll
      for (int w = 0; w < NWV; ++w) add_tiles<NT>(sum, from + w * (2 * TILE));
      __syncthreads();                     // everybody has taken theirs
      store_rows<NT>(a.dQ + ((size_t)h * a.Nq + (size_t)r_tile * kTile + 32 * n) * D + 32 * dt0, D, sum, a.scale,
                     fixed_len - 32 * n, smem);
      return;
    }
  }
#pragma unroll
  for (int n = 0; n < 2; ++n)
    store_rows<DT>(a.dQ + ((size_t)h * a.Nq + (size_t)r_tile * kTile + 32 * n) * D, D, out[n], a.scale, fixed_len - 32 * n,
                   smem + n * TILE);
}

// dq and dkv as one launch (neither needs what the other writes) or as a launch each.  A launch's time ends with its longest
// walks; as one launch the two kernels' ends and beginnings overlap, and the places dq leaves empty (888 waves on 1024
// places at 12 heads x 4680 rows) are dkv's from the start.  The dq workgroups, whose walks are the longest, come first.
// Select, forward and backward, two launches -> one (with dq_split where it applies): 712 -> 696 us at 12 x 4680 x 128 with
// 32 + 48 blocks of 64, 446 -> 433 with 8 + 16 blocks of 128, 227 -> 134 at 4 x 3000 x 128, 88 -> 57 at 3 x 1500 x 64.
constexpr int kDq = 1, kDkv = 2;
template <int D, int PARTS, int NWV>
__global__ void __launch_bounds__(64 * NWV) __attribute__((amdgpu_waves_per_eu(PARTS == kDkv ? 2 : 1)))
    bwd_walk_kernel(BwdArgs a, int n_dq) {
  extern __shared__ __align__(1024) unsigned char smem[];
  if constexpr (PARTS == kDq) {
    dq_body<D, NWV>(a, (int)blockIdx.x, smem);
  } else {
    if (PARTS != kDkv && (int)blockIdx.x < n_dq) dq_body<D, NWV>(a, (int)blockIdx.x, smem);
    else dkv_body<D, NWV / 2>(a, (int)blockIdx.x - n_dq, smem);
  }
}

template <int D, int PARTS, int NWV>
hipError_t launch_walk(const BwdArgs& a, unsigned n_dq, unsigned n_dkv, size_t lds, hipStream_t stream) {
  const auto kernel = bwd_walk_kernel<D, PARTS, NWV>;
  hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(kernel, dim3(n_dq + n_dkv), dim3(64 * NWV), lds, stream, a, (int)n_dq);
  return hipGetLastError();
}

}  // namespace

// row scalars, then the turned-around selection, then the order of the local blocks
struct BwdWorkspace {
  size_t att, order, bytes;
};
static BwdWorkspace bwd_workspace(const pbsa_params& p) {
  const auto up = [](size_t n) { return (n + 255) & ~(size_t)255; };
  BwdWorkspace w;
  w.att = (size_t)p.H * row_blocks(p.Nq) * 64 * 4;
  w.order = w.att + up((size_t)p.H * p.n_loc_cap * ((p.nqb + 31) / 32) * 4);
  w.bytes = w.order + up((size_t)p.H * p.n_loc_cap * 16);
  return w;
}
size_t bwd_workspace_bytes(const pbsa_params& p) { return bwd_workspace(p).bytes; }

// Whether four waves to a walk end a launch sooner than two.  It ends with its longest walk or when the places have taken all
// of them, and where the two are close a little later: microseconds of a workgroup beside its turns, of a turn (64 x 64) of dQ
// and of dK / dV, of the places for what their turns take, and of the launch beside that, fitted to 800 shapes (of two waves within
// 3 % at d = 64 and 5 % at 128, of four within 8 and 9).  Where the places set the end four waves are not only no better: the
// longest walks then depend on which blocks the rows select, where they are many (24 row tiles), and that is not known here, so
// past 1.2 times the longest walk it is two (all rows selecting the same blocks, 8 x 970 x 64 with 8 blocks 22 -> 30 us by four, 5 x 4729 x 64 with 15 + 36 87 -> 114).
static bool four_waves_end_sooner(const pbsa_params& p) {
  struct Fit {
    float own, dq, dkv, places, launch;
  };
  static constexpr Fit kFit[2][2] = {{{7.7f, 1.24f, 0.77f, 1.13f, 1.3f}, {4.4f, 1.26f, 0.85f, 1.29f, 5.8f}},      // d = 64: two, four
                                     {{5.8f, 1.87f, 1.11f, 1.55f, 6.3f}, {4.9f, 1.87f, 1.20f, 1.56f, 9.4f}}};     // 128
  const int sub = p.B / kTile, rows = (p.Nq + kTile - 1) / kTile, k = std::min(p.k, p.n_loc), tiles = p.H * rows;
  float us[2], walk = 0.0f, taken = 0.0f;
  for (int four = 0; four < 2; ++four) {
    const Fit& f = kFit[p.d == 128][four];
    const float waves = four ? 4.0f : 2.0f;
    const bool shared = four || tiles <= 256;              // dq: the waves of a workgroup share a walk
    const float dq = f.dq * (float)((p.C + 1 + k) * sub) / (shared ? waves : 1.0f), slot = f.dkv * (float)rows / (0.5f * waves);
    const float block = slot * (float)k / (float)p.n_loc;
    walk = f.own + std::max(dq, slot);
    taken = f.places * waves / 1024.0f * ((float)(shared ? tiles : (tiles + 1) / 2) * (f.own + dq) +
                                          (float)(p.H * sub) * ((float)(p.C + 1) * (f.own + slot) + (float)p.n_loc * (f.own + block)));
    const float w2 = walk * walk, t2 = taken * taken;
    us[four] = f.launch + std::sqrt(std::sqrt(w2 * w2 + t2 * t2));
  }
  return us[1] < 0.95f * us[0] && (rows < 24 || taken <= 1.2f * walk);
}

hipError_t launch_attention_bwd(const pbsa_params& p, const bf16_t* Q, const bf16_t* Kp, const bf16_t* Vp,
                                const int32_t* p_len, const bf16_t* Kl, const bf16_t* Vl, const int32_t* l_len,
                                const int32_t* l_map, const int32_t* sel, const bf16_t* O, const bf16_t* dO,
                                const float* lse, float* dQ, float* dKp, float* dVp, float* dKl, float* dVl, void* ws,
                                hipStream_t stream) {
  BwdArgs a{p.H, p.Nq, p.nqb, p.n_loc, p.n_loc_cap, p.C, p.k, p.B, 0, p.scale, p.q_stride_h, p.q_stride_t, p.o_stride_h,
            p.o_stride_t, Q, Kp, Vp, p_len, Kl, Vl, l_len, l_map, sel, O, dO, lse, static_cast<float*>(ws),
            reinterpret_cast<uint32_t*>(static_cast<char*>(ws) + bwd_workspace(p).att),
            reinterpret_cast<int4*>(static_cast<char*>(ws) + bwd_workspace(p).order), dQ, dKp, dVp, dKl, dVl};
  const int sub = p.B / kTile;
  const long n_lanes = p.H * row_blocks(p.Nq) * 32 * (p.d / 8);
  const dim3 pgrid((unsigned)((n_lanes + 255) / 256 + p.H));
  const size_t plan_lds = ((size_t)p.n_loc * ((p.nqb + 31) / 32) + p.nqb + 1) * 4;    // at most 35 KB (512 blocks)
  if (p.d == 128) hipLaunchKernelGGL(bwd_prep_kernel<128>, pgrid, dim3(256), plan_lds, stream, a);
  else hipLaunchKernelGGL(bwd_prep_kernel<64>, pgrid, dim3(256), plan_lds, stream, a);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int n_row_tiles = (p.Nq + kTile - 1) / kTile, n_tiles = p.H * n_row_tiles;
  const int n_cand = (p.C + 1 + p.k) * sub;                  // of a dq walk: its list
  const size_t tile = (size_t)kTile * p.d * 2;
  const unsigned n_dkv = head_items((p.C + 1 + p.n_loc) * sub, p.H);
  const size_t lds_dkv = 4 * tile + (size_t)4 * sub * p.nqb + 16;
  // Where the line lies between one launch and two: at d = 128 both bodies need a SIMD's whole register file per wave, and
  // one launch is never slower.  At d = 64 dkv by itself runs two waves per SIMD, beside dq one, which costs it more than
  // the shared launch saves where dq's walks are long and its waves fill the last round of 1024 places, the time dkv could
  // have had anyway: 12 x 4680 rows with 32 + 48 blocks of 64 (888 waves) 414 us as two launches and 422 as one, 13 x 4800 441
  // and 459; but 11 x 4680 (814 waves) 400 and 393, 16 x 4000 with 4 + 8 blocks 145 and 132, 12 x 4680 with 16 + 24 blocks 272
  // and 248, 8 x 2000 with 6 + 8 blocks 95 and 71.  Beyond one round, the backward by itself with the same 32 + 48 blocks:
  // 1036 waves 409 us as two launches and 350 as one, 1184 437 and 396, 1344 467 and 440, 1512 503 and 497, 1596 518 and 524,
  // 1680 (where it is two again) 540 and 542.
  const int rounds = (n_tiles + 1023) / 1024;
  if (p.d == 64 && n_cand >= 64 && 5 * n_tiles >= 4 * 1024 * rounds) {
    e = launch_walk<64, kDq, 1>(a, head_items(n_row_tiles, p.H), 0, 2 * tile + (size_t)4 * n_cand + 16, stream);
    if (e != hipSuccess) return e;
    return launch_walk<64, kDkv, 2>(a, 0, n_dkv, lds_dkv, stream);
  }
  // Four waves share a walk where the longest walks set the launch's end, which come first and then end half as late: a
  // workgroup of four has a compute unit to itself, so a launch that the places set takes as long or, with more workgroups
  // than units, longer.  The backward by itself, two waves -> four, us, where it is four:
  // 2 x 4866 x 128 with 8 + 2 blocks of 64 95 -> 64, 3 x 2582 x 64 with 2 + 6 of 128 41 -> 29, 4 x 125 x 128 with 57 + 1 of 128 117 -> 69,
  // 5 x 408 x 128 with 5 + 6 of 128 32 -> 26, 1 x 344 x 64 with 16 + 3 of 64 20 -> 16, 13 x 333 x 128 with 43 + 6 of 64 62 -> 57; where it is two:
  // 19 x 1424 x 64 with 15 + 8 of 128 96 | 125, 2 x 4258 x 128 with 22 + 23 of 128 104 to 113 | 112 to 123, 7 x 1899 x 64 with 2 + 9 of 64
  // 34 | 35, and for what selections it may meet 3 x 2105 x 64 with 44 + 2 of 128 66 | 52 to 61.
  // (Over 800 shapes, each with rows that select alike and not, one was slower by four, by 2 %; 12 % of the backward's
  // time, where the better way each time would give 16.)  Up to 448 workgroups, from eight row tiles on, four in any case (8 x 600 x 64: 22.4 -> 20.9,
  // which the model does not see).
  const size_t lds4 = 8 * tile + (size_t)4 * std::max(4 * n_cand, sub * p.nqb) + 16;
  const bool four = (n_tiles + p.H * (p.C + 1 + p.n_loc) * sub <= 448 && n_row_tiles >= 8) || four_waves_end_sooner(p);
  if (four && lds4 <= 156 * 1024) {
    const unsigned n_dq = head_items(n_row_tiles, p.H);
    return p.d == 128 ? launch_walk<128, kDq | kDkv, 4>(a, n_dq, n_dkv, lds4, stream)
                      : launch_walk<64, kDq | kDkv, 4>(a, n_dq, n_dkv, lds4, stream);
  }
  // Two waves share a walk where the row tiles are at most as many as the compute units: each walk has a unit to itself, and
  // half of it ends earlier (4 x 3000 x 128, 188 row tiles: 134 us split).  With 512 (16 x 2048 x 128) a row tile per wave
  // takes 165 us and the split, which loads the fixed fragments twice, 175; with 888 433 and 441.
  a.dq_split = n_tiles <= 256;
  const unsigned n_dq = head_items(a.dq_split ? n_row_tiles : (n_row_tiles + 1) / 2, p.H);
  const size_t lds = std::max(lds_dkv, 4 * tile + (size_t)8 * n_cand + 16);
  return p.d == 128 ? launch_walk<128, kDq | kDkv, 2>(a, n_dq, n_dkv, lds, stream)
                    : launch_walk<64, kDq | kDkv, 2>(a, n_dq, n_dkv, lds, stream);
}

}  // namespace pbsa

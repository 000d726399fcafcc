// Coarse stage and persistent-memory update kernels for gfx950 (HBM / latency bound; fp32 chains on matrix instructions).
//
//   pool_kernel         block representatives by average pooling, by threads (Eq. 6)
//   pool_tile_kernel    the same, a workgroup to a block
//   append_kernel       a chunk into the ring, pooled as it passes
//   select_kernel       coarse logits + row-wise top-k block selection      (Eq. 10-11)
//   select_small_kernel a small chunk's selection with its pooling, its append or the fold before it
//   score_rows_kernel   block-level softmax rows over persistent + local    (Eq. 7)
//   retain_kernel       column mean, Top-C retention, slot assignment       (Eq. 8-9)
//   fold_promote_kernel dropped blocks -> running-mean summary; kept newcomers -> slots
//
// This file is compiled with -ffp-contract=off: every fp32 operation below is exactly the one
// written (the arithmetic that decides block sets and slots is specified operation by operation
// in pbsa.h so that an independent implementation reproduces the integers bit for bit).
#include <type_traits>
#include <utility>

#include "pbsa_internal.h"
#include "pbsa_plan_device.h"

namespace pbsa {
namespace {

using namespace plan_dev;

constexpr int kThreads = 256;
// Of the fold's workgroups: with 256 threads there are 192 of them at 12 heads of 64 x 128 positions, and a quarter of the chip
// has none (128 -> 256 threads: fold 12.9 -> 14.1 us there, 4.8 -> 5.4 at two heads of 64 x 64; 64 threads: 14.0, 4.7).
constexpr int kFoldThreads = 128;
constexpr int kXC = 32;   // pooled-key dimensions staged through LDS per step

typedef __attribute__((ext_vector_type(4))) float f32x4;

__device__ __forceinline__ float bf_lo(uint32_t u) { return __uint_as_float(u << 16); }
__device__ __forceinline__ float bf_hi(uint32_t u) { return __uint_as_float(u & 0xFFFF0000u); }

__device__ __forceinline__ uint32_t f2bf_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return u >> 16;
}


// ------------------------------------------------------------------------------------------------
// Pooling.  One job = one block; D/2 threads per job, each owning 2 dimensions (one 4-byte load per
// token) and adding the tokens in ascending order.  The loads of a block are in flight together.
// ------------------------------------------------------------------------------------------------
// Adds min(N, len) tokens (two dimensions of them) to acc0 / acc1 in ascending order, all N loads in flight together.  The
// address walks from token to token: as a product of the token's number and the pitch, 64 bits wide, the addresses took
// longer than the sums.  Unless FULL, a load past the last token takes that one again and counts as zero (a sum that starts
// from +0 is never -0, so +0 leaves it as it is).
template <int N, bool FULL, typename PITCH>
__device__ __forceinline__ void pool_rows(const bf16_t* p, PITCH pitch, int len, float& acc0, float& acc1) {
  uint32_t v[N];
#pragma unroll
  for (int u = 0; u < N; ++u) {
    v[u] = *reinterpret_cast<const uint32_t*>(p);
    p += FULL || u + 1 < len ? (long)pitch : 0;
  }
#pragma unroll
  for (int u = 0; u < N; ++u) {
    const uint32_t w = FULL || u < len ? v[u] : 0u;
    acc0 = acc0 + bf_lo(w);
    acc1 = acc1 + bf_hi(w);
  }
}
// len tokens, at most 128 (none: nothing is read).  The wave takes one way through: its lanes may have two blocks.
template <typename PITCH>
__device__ __forceinline__ void pool_block(const bf16_t* p, PITCH pitch, int len, float& acc0, float& acc1) {
  if (len <= 0) return;
  if (__any(len > 64)) {
    if (__all(len == 128)) pool_rows<128, true>(p, pitch, len, acc0, acc1);
    else pool_rows<128, false>(p, pitch, len, acc0, acc1);
  } else {
    if (__all(len == 64)) pool_rows<64, true>(p, pitch, len, acc0, acc1);
    else pool_rows<64, false>(p, pitch, len, acc0, acc1);
  }
}

struct PoolArgs {
  int mode;                 // 0: generic blocks, 1: select (local key blocks, then query blocks)
  int n_jobs;
  int H, B, Nq, nqb, n_loc, n_loc_cap, pool_from, n_kjobs_per_head;   // n_kjobs_per_head: stale local key blocks
  long q_stride_h, q_stride_t;
  const bf16_t* X;          // mode 0: [n][B][D]; mode 1: Kl
  const bf16_t* Q;
  const int32_t* len;       // mode 0: [n]; mode 1: l_len
  const int32_t* l_map;
  float* out;               // mode 0: [n][D]; mode 1: Kc_l
  float* Qc;
};

// A job: where its block is, the elements from token to token, how many tokens (0 .. B), and the place of the result.
struct PoolJob {
  const bf16_t* src;
  long pitch;
  int len;
  float* dst;
};
// jobs [0, H*nk) of mode 1 pool local key blocks, the rest pool the chunk's query blocks
__device__ __forceinline__ bool pool_is_query(const PoolArgs& a, const int job) { return a.mode == 1 && job >= a.H * a.n_kjobs_per_head; }
template <int D>
__device__ __forceinline__ PoolJob pool_query_job(const PoolArgs& a, const int job) {
  const int jq = job - a.H * a.n_kjobs_per_head, h = jq / a.nqb, i = jq % a.nqb;
  return {a.Q + (size_t)h * a.q_stride_h + (size_t)i * a.B * a.q_stride_t, (long)a.q_stride_t, min(a.B, a.Nq - i * a.B),
          a.Qc + ((size_t)h * a.nqb + i) * D};
}
// false: there is no such block
template <int D>
__device__ __forceinline__ bool pool_key_job(const PoolArgs& a, const int job, PoolJob& j) {
  const int nk = a.n_kjobs_per_head;
  if (a.mode == 0) {
    j.src = a.X + (size_t)job * a.B * D;
    j.len = a.len[job];
    j.dst = a.out + (size_t)job * D;
  } else {
    const int h = job / nk, l = a.pool_from + job % nk;
    const int slot = a.l_map[l];
    if (slot < 0 || slot >= a.n_loc_cap) return false;
    j.src = a.X + ((size_t)h * a.n_loc_cap + slot) * a.B * D;
    j.len = a.len[l];
    j.dst = a.out + ((size_t)h * a.n_loc_cap + slot) * D;
  }
  j.len = max(0, min(j.len, a.B));
  j.pitch = D;
  return true;
}

template <int D, int NT>
__device__ __forceinline__ void pool_body(const PoolArgs& a, const int bx) {
  constexpr int TPJ = D / 2;
  const int job = bx * (NT / TPJ) + threadIdx.x / TPJ;
  const int c = threadIdx.x % TPJ;
  if (job >= a.n_jobs) return;
  PoolJob j;
  float acc0 = 0.0f, acc1 = 0.0f;
  if (pool_is_query(a, job)) {             // (a branch with all of its work in it: 2 to 4 % of the launch against one for the place, one for the sum)
    j = pool_query_job<D>(a, job);
    pool_block(j.src + 2 * c, j.pitch, j.len, acc0, acc1);
  } else {
    if (!pool_key_job<D>(a, job, j)) return;
    pool_block(j.src + 2 * c, std::integral_constant<long, D>{}, j.len, acc0, acc1);
  }
  const float fl = (float)j.len;
  float2 o;
  o.x = j.len > 0 ? acc0 / fl : 0.0f;
  o.y = j.len > 0 ? acc1 / fl : 0.0f;
  *reinterpret_cast<float2*>(j.dst + c * 2) = o;
}

// Adds the len rows of a block in LDS in ascending order, two dimensions per thread of the first D / 2: 64 consecutive words
// per row, free of bank conflicts.
template <int D>
__device__ __forceinline__ void pool_tile(const uint4* tile, int len, float* out) {
  const uint32_t* t32 = reinterpret_cast<const uint32_t*>(tile) + threadIdx.x;
  float acc0 = 0.0f, acc1 = 0.0f;
#pragma unroll 16
  for (int r = 0; r < len; ++r) {
    const uint32_t u = t32[r * (D / 2)];
    acc0 = acc0 + bf_lo(u);
    acc1 = acc1 + bf_hi(u);
  }
  const float fl = (float)len;
  *reinterpret_cast<float2*>(out + 2 * threadIdx.x) = len > 0 ? make_float2(acc0 / fl, acc1 / fl) : make_float2(0.0f, 0.0f);
}

template <int D>
__global__ void __launch_bounds__(kThreads) pool_kernel(PoolArgs a) {
  pool_body<D, kThreads>(a, blockIdx.x);
}

// A pooling launch by itself of blocks that all find a place on the chip: one workgroup to a block, 16 bytes a thread and load,
// all in flight, summed through LDS as the append does.  When: launch_pool.
template <int D, int BT>
__global__ void __launch_bounds__(kThreads) pool_tile_kernel(PoolArgs a) {
  constexpr int CPR = D / 8, RPS = kThreads / CPR, NS = BT / RPS;     // chunks per row, rows per sweep, sweeps
  __shared__ __align__(16) uint4 tile[BT * CPR];
  PoolJob j;
  if (pool_is_query(a, blockIdx.x)) j = pool_query_job<D>(a, blockIdx.x);
  else if (!pool_key_job<D>(a, blockIdx.x, j)) return;                // (all of the workgroup)
  if (j.len > 0) {
    const int r0 = threadIdx.x / CPR, c = threadIdx.x % CPR;
    f32x4 v[NS];                                                      // (as uint4 they go through scratch memory)
#pragma unroll
    for (int s = 0; s < NS; ++s) v[s] = *reinterpret_cast<const f32x4*>(j.src + (size_t)min(r0 + s * RPS, j.len - 1) * j.pitch + 8 * c);
#pragma unroll
    for (int s = 0; s < NS; ++s) *reinterpret_cast<f32x4*>(&tile[(r0 + s * RPS) * CPR + c]) = v[s];
  }
  __syncthreads();
  if (threadIdx.x < D / 2) pool_tile<D>(tile, j.len, j.dst);
}

// By tiles as long as the blocks find places side by side, four to a compute unit at most, and by threads beyond; sooner where
// all blocks are whole, whose loops over the rows have no test in them by threads, and at d = 128, where a wave of those is
// a block of its own.  Pooling and selection of a chunk, us, by threads -> by tiles, heads x blocks (as many older and newer):
//   not whole: 8 x 32 of 64 x 64 8.7 -> 8.4, 16 x 32 8.7 -> 8.4, 8 x 32 of 64 x 128 10.5 -> 8.9, 16 x 32 10.5 -> 9.2, 8 x 32 of 128 x 128
//   10.9 -> 9.9, 12 x 32 11.2 -> 10.5, 8 x 16 of 128 x 64 8.9 -> 8.9; 16 x 16 of 128 x 64 9.1 | 9.1, 28 x 16 9.1 | 9.5, 32 x 16 9.2 | 9.7;
//   whole: 8 x 32 of 64 x 64 8.1 -> 7.9, 12 x 32 8.2 -> 8.1, 16 x 32 8.3 | 8.3, 12 x 32 of 64 x 128 8.9 | 8.9, 16 x 32 9.0 | 9.2, 4 x 16 of
//   128 x 64 8.4 -> 8.3, 12 x 16 8.5 | 9.0, 24 x 16 8.8 | 9.4, 4 x 16 of 128 x 128 9.2 -> 9.0, 8 x 16 9.2 | 9.4, 20 x 16 9.6 | 10.3.
static int pool_tile_jobs(const PoolArgs& a, int d) {
  const bool whole = a.mode == 0 || a.Nq % a.B == 0;       // (mode 0 has its lengths on the device: whole as a rule)
  if (d == 64) return whole ? 768 : 1024;
  return whole ? 128 : a.B == 64 ? 512 : 1024;
}
template <int D>
static hipError_t launch_pool(const PoolArgs& a, hipStream_t stream) {
  const dim3 block(kThreads);
  if (a.n_jobs > pool_tile_jobs(a, D)) {
    constexpr int jpw = kThreads / (D / 2);
    hipLaunchKernelGGL(pool_kernel<D>, dim3((a.n_jobs + jpw - 1) / jpw), block, 0, stream, a);
  } else if (a.B == 128) {
    hipLaunchKernelGGL((pool_tile_kernel<D, 128>), dim3(a.n_jobs), block, 0, stream, a);
  } else {
    hipLaunchKernelGGL((pool_tile_kernel<D, 64>), dim3(a.n_jobs), block, 0, stream, a);
  }
  return hipGetLastError();
}

// ------------------------------------------------------------------------------------------------
// Cache append: a chunk's K and V (token-major per head) into nqb consecutive ring slots, and the pooled keys of those
// blocks (Eq. 6) from the rows as they pass.  One workgroup = one block of K or of V; a thread moves 16 bytes per
// sweep, all sweeps in flight together.  For K the rows also go to LDS, where D / 2 threads add them in ascending
// order (the pinned order of the pooling).
// Bound by HBM: each byte is read once and written once, and a selection that follows need not read K again: 11.1 us
// for a chunk of 12 x 4680 x 128 (57.5 MB moved, 5.2 TB/s), where four tensor copies took 27 us and the selection's
// own pooling launch another 8.7.  The chunk's queries can be pooled along (and are not copied): half as many workgroups
// again, which read a third of the bytes and write next to none, against the 1.3 to 2.8 us that the selection takes to pool
// them itself (a step of 5 x 1000 x 64 40.7 -> 38.2 us, of 8 x 2500 x 128 76.1 -> 72.8; up to which size: PbsaCache).
// ------------------------------------------------------------------------------------------------
struct AppendArgs {
  int B, Nq, nqb, n_loc_cap, slot0, zero_tail;
  long sh[3], st[3];        // element strides of K, of V and of Q
  const bf16_t* src[3];
  bf16_t* dst[2];
  float* Kc_l;
  float* Qc;
};

template <int D, int BT>
__global__ void __launch_bounds__(kThreads) append_kernel(AppendArgs a) {
  constexpr int CPR = D / 8, RPS = kThreads / CPR, NS = BT / RPS;     // chunks per row, rows per sweep, sweeps
  __shared__ __align__(16) uint4 tile[BT * CPR];
  const int i = blockIdx.x, h = blockIdx.y, kv = blockIdx.z;
  const bf16_t* src = a.src[kv];
  if (!src) return;
  const int len = min(BT, a.Nq - i * BT);
  const int r0 = threadIdx.x / CPR, c = threadIdx.x % CPR;
  src += (size_t)h * a.sh[kv] + (size_t)i * BT * a.st[kv] + 8 * c;
  const size_t slot = (size_t)h * a.n_loc_cap + a.slot0 + i;
  bf16_t* dst = kv == 2 ? nullptr : a.dst[kv] + slot * BT * D + 8 * c;
  uint4 v[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) v[s] = *reinterpret_cast<const uint4*>(src + (size_t)min(r0 + s * RPS, len - 1) * a.st[kv]);
  const bool pool = kv == 0 ? a.Kc_l != nullptr : kv == 2;
#pragma unroll
  for (int s = 0; s < NS; ++s) {
    const int r = r0 + s * RPS;
    if (pool) tile[r * CPR + c] = v[s];
    if (r >= len) v[s] = make_uint4(0u, 0u, 0u, 0u);
    if (dst && (r < len || a.zero_tail)) *reinterpret_cast<uint4*>(dst + (size_t)r * D) = v[s];
  }
  if (!pool) return;
  __syncthreads();
  if (threadIdx.x < D / 2) pool_tile<D>(tile, len, kv == 0 ? a.Kc_l + slot * D : a.Qc + ((size_t)h * a.nqb + i) * D);
}

// ------------------------------------------------------------------------------------------------
// Coarse logits.  A workgroup of 4 waves handles 4 query blocks (one per wave) of one head; lane
// `lane` of a wave owns columns j = lane + 64 m.  The pooled keys of all columns are staged through
// LDS kXC dimensions at a time, transposed ([x][j], pitch NM*64+2 keeps both the transposing stores
// and the per-column loads free of bank conflicts), so each accumulator runs the fixed chain
// acc = fma(q[x], k[x], acc), x ascending.
// ------------------------------------------------------------------------------------------------
template <int D, int NM>
__device__ __forceinline__ void coarse_dots(const float* const* cols, int n_cols, const float* qrow, float* kct,
                                            float (&acc)[NM]) {
  constexpr int NPAD = NM * 64 + 2;
  constexpr int P = NM * 64 * (kXC / 4) / kThreads;     // float4 loads per thread per round
  const int lane = threadIdx.x & 63;
#pragma unroll
  for (int m = 0; m < NM; ++m) acc[m] = 0.0f;
  __syncthreads();                                       // cols[] and qrow are visible
  // the global loads of round r+1 are in flight while round r is multiplied
  float4 pre[P];
#pragma unroll
  for (int u = 0; u < P; ++u) {
    const int idx = threadIdx.x + u * kThreads;
    if (idx < n_cols * (kXC / 4)) pre[u] = *reinterpret_cast<const float4*>(cols[idx / (kXC / 4)] + 4 * (idx % (kXC / 4)));
  }
  for (int x0 = 0; x0 < D; x0 += kXC) {
    if (x0 > 0) __syncthreads();                         // previous round's reads of kct are done
#pragma unroll
    for (int u = 0; u < P; ++u) {
      const int idx = threadIdx.x + u * kThreads;
      if (idx < n_cols * (kXC / 4)) {
        const int j = idx / (kXC / 4), xq = idx % (kXC / 4);
        kct[(4 * xq + 0) * NPAD + j] = pre[u].x;
        kct[(4 * xq + 1) * NPAD + j] = pre[u].y;
        kct[(4 * xq + 2) * NPAD + j] = pre[u].z;
        kct[(4 * xq + 3) * NPAD + j] = pre[u].w;
      }
    }
    __syncthreads();
    if (x0 + kXC < D) {
#pragma unroll
      for (int u = 0; u < P; ++u) {
        const int idx = threadIdx.x + u * kThreads;
        if (idx < n_cols * (kXC / 4))
          pre[u] = *reinterpret_cast<const float4*>(cols[idx / (kXC / 4)] + x0 + kXC + 4 * (idx % (kXC / 4)));
      }
    }
#pragma unroll 4
    for (int xx = 0; xx < kXC; ++xx) {
      const float q = qrow[x0 + xx];
#pragma unroll
      for (int m = 0; m < NM; ++m) acc[m] = __builtin_fmaf(q, kct[xx * NPAD + lane + 64 * m], acc[m]);
    }
  }
}


struct SelectArgs {
  int H, nqb, n_loc, n_loc_cap, k, causal;
  float scale;
  float* Kc_l;
  float* Qc;
  const int32_t* l_map;
  int32_t* sel;
  float* Zl;                // optional out: scaled logits of every local block, [H][nqb][n_loc]
  const bf16_t* Q;          // given: the query blocks are pooled here (into Qc), else Qc holds them
  int B, Nq;
  long q_stride_h, q_stride_t;
  const bf16_t* Kl;         // KEYS: blocks from pool_from on are pooled from here
  const int32_t* l_len;
  int pool_from;
  int chunk_slot;           // KEYS: -1, or they are those of a chunk that the same launch appends from this slot on, and Kl its
  long k_stride_h, k_stride_t;   // token-major rows
};

// One wave-wide global -> LDS load of 16 bytes per lane: LDS bytes [lds_off, lds_off + 1024) receive
// lane i's 16 bytes, fetched from base + voff, at lds_off + 16 i.  Completion is tracked by the issuing
// wave's vmcnt.  Earlier LDS reads of this wave are complete before the load is issued.
__device__ __forceinline__ void dma16(const void* base, uint32_t voff, uint32_t lds_off) {
  asm volatile("s_waitcnt lgkmcnt(0)\n\ts_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :
               : "s"(lds_off), "v"(voff), "s"(base)
               : "memory", "m0");
}

constexpr int kOwnKeys = 12;      // the most key blocks that the selection pools itself
template <int NM, bool KEYS>
constexpr int select_waves() { return KEYS ? 8 : NM < 4 ? 4 : NM; }

template <int D, int NM>
struct SelectGeo {
  static constexpr int DX = NM <= 8 ? 32 : 16;                                  // dimensions per round
  static constexpr int NR = D / DX, BUF = NM * 64 * DX * 4;                     // rounds, bytes of a round
  static constexpr int REST = 4 * D * 4 + 4 * NM * 64 * 4;                      // the queries and the logits
  static constexpr int FIT = (160 * 1024 - REST) / BUF;
  static constexpr int NBUF = FIT < NR ? FIT : NR;                              // rounds in LDS at a time
  static constexpr int LDS = NBUF * BUF + REST;
  static_assert(NBUF >= 2, "a round arrives while another one is multiplied");
};

// Selection (Eq. 10-11).  A workgroup handles 4 query blocks of one head; its NM waves split the local
// blocks: lane `lane` of wave w owns column j = 64 w + lane and runs the four chains
// acc_r = fma(q_r[x], k_j[x], acc_r), x ascending, as four rows of one matrix instruction per x: the instruction takes
// the queries from registers, where vector instructions had to read each of them from LDS for every 64 columns and the
// workgroup's LDS reads were what the chains waited for.  The pooled keys reach LDS by direct global -> LDS loads, DX
// dimensions (4 DX bytes per column) per round, as many rounds at a time as fit; a wave stages exactly the 64
// columns it consumes, so the rounds need no workgroup barrier.  Within a column's round the 16-byte
// chunks are permuted (logical chunk c of column j sits at c ^ ((j / 2) % (DX / 4))), which spreads the
// per-lane 16-byte reads of consecutive columns over the bank groups.  The logits then go to LDS and wave
// r ranks row r.  DX = 32 up to 8 waves; 16 beyond, where two rounds of 32 would not fit in LDS.  A query block is
// looked at by exactly one workgroup, so that one pools it (Eq. 6, D / 2 threads per block, tokens added in ascending
// order) while its pooled keys arrive; at least four waves, so that the four blocks are pooled and ranked side by side
// whatever NM is.  Latency bound, a chain of phases; inside a workgroup, by time stamps, against 64-bit products for the queries' addresses, chains of v_fma_f32 over two rounds in LDS
// and all 32 bits of the threshold: pooling 2.5 -> 1.3 us, logits 1.2 -> 0.5, threshold 1.2 -> 0.8 at 2 heads x 4 blocks of 64
// (16 columns of 64 dimensions); 3.7 -> 2.6, 2.7 -> 1.4, 2.6 -> 1.4 at 12 x 37 blocks of 128 (148 columns of 128).
//
// KEYS: the newest of the key blocks are pooled here too, by every workgroup of the head for itself (the first one also
// leaves them in Kc_l), beside its four query blocks: eight waves pool 16 blocks of 64 dimensions at a time, 8 of 128.
template <int D, int NM, bool KEYS = false>
__device__ __forceinline__ void select_body(const SelectArgs& a, const int bx, const int h, unsigned char* smem) {
  using G = SelectGeo<D, NM>;
  constexpr int NCP = NM * 64;                        // padded columns
  constexpr int DX = G::DX, BUF = G::BUF, NR = G::NR, NBUF = G::NBUF;
  constexpr int CPC = DX / 4;                         // 16-byte chunks per column and round
  constexpr int NI = 64 * CPC / 64;                   // load instructions per wave and round (64 columns)
  constexpr int CPI = 64 / CPC;                       // columns per instruction
  constexpr int NW = select_waves<NM, KEYS>(), NT = 64 * NW;   // waves, threads
  float* qs = reinterpret_cast<float*>(smem + NBUF * BUF);                      // [4][D]
  float* zs = qs + 4 * D;                                                       // [4][NCP]
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i0 = bx * 4;

  const bool has_cols = NM >= 4 || wave < NM;         // the waves that own columns

  int place[NM];                                      // KEYS: l_map of columns lane + 64 m
  if constexpr (KEYS)
#pragma unroll
    for (int m = 0; m < NM; ++m) place[m] = a.l_map[min(lane + 64 * m, a.n_loc - 1)];

  // this lane's share of the staging: instruction n fills columns 64 wave + CPI n + lane / CPC, physical chunk
  // lane % CPC
  uint32_t goff[NI];
#pragma unroll
  for (int n = 0; n < NI; ++n) {
    const int j = min(64 * wave, NCP - 64) + CPI * n + lane / CPC;
    int slot = a.l_map[min(j, a.n_loc - 1)];
    slot = min(max(slot, 0), a.n_loc_cap - 1);
    const int chunk = (lane % CPC) ^ ((j >> 1) % CPC);
    goff[n] = (uint32_t)(((size_t)h * a.n_loc_cap + slot) * D * 4 + chunk * 16);
  }
  const uint32_t smem_lds = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)smem;
  const uint32_t wave_lds = __builtin_amdgcn_readfirstlane(smem_lds + wave * (64 * DX * 4));
  const unsigned char* kbase = reinterpret_cast<const unsigned char*>(a.Kc_l);
#define PBSA_STAGE(R_)                                                                                 \
  _Pragma("unroll") for (int n_ = 0; n_ < NI; ++n_)                                                     \
      dma16(kbase + (R_) * (DX * 4), goff[n_], wave_lds + ((R_) % NBUF) * BUF + n_ * 1024);
  if (has_cols) {
#pragma unroll
    for (int r = 0; r < NBUF; ++r) PBSA_STAGE(r)
  }

  if constexpr (KEYS) {
    static_assert(NBUF == NR, "a column's place holds all of it");
    constexpr int JPS = NT / (D / 2), SW = (4 + kOwnKeys) / JPS;      // blocks at a time, times
    const int c = threadIdx.x % (D / 2), n_stale = a.n_loc - a.pool_from;
    float2 mean[SW];
    int slot[SW];                                     // of a key block (-1: it is nowhere)
    // an older block in the place of one of these has the new pooled keys too, and is staged with those from before
    bool twice = false;
#pragma unroll
    for (int m = 0; m < NM; ++m) place[m] = lane + 64 * m < a.pool_from ? min(max(place[m], 0), a.n_loc_cap - 1) : -2;
#pragma unroll
    for (int w = 0; w < SW; ++w) {
      const int job = w * JPS + (int)threadIdx.x / (D / 2), i = i0 + job, l = a.pool_from + job - 4;
      const bf16_t* p = nullptr;
      long pitch = 0;
      int len = 0;
      slot[w] = -1;
      if (job < 4) {
        if (i < a.nqb) {
          len = min(a.B, a.Nq - i * a.B);
          pitch = a.q_stride_t;
          p = a.Q + (size_t)h * a.q_stride_h + (size_t)i * a.B * pitch + 2 * c;
        }
      } else if (job < 4 + n_stale) {
        if (a.chunk_slot >= 0) {
          slot[w] = a.chunk_slot + job - 4;
          len = min(a.B, a.Nq - (job - 4) * a.B);
          pitch = a.k_stride_t;
          p = a.Kl + (size_t)h * a.k_stride_h + (size_t)(job - 4) * a.B * pitch + 2 * c;
        } else {
          const int at = a.l_map[l];
          if (at >= 0 && at < a.n_loc_cap) {
            len = max(0, min(a.l_len[l], a.B));
            pitch = D;
            p = a.Kl + ((size_t)h * a.n_loc_cap + at) * a.B * D + 2 * c;
            slot[w] = at;
          }
        }
      }
#pragma unroll
      for (int x = 0; x < 64; x += D / 2)
#pragma unroll
        for (int m = 0; m < NM; ++m) twice |= __any(place[m] == __builtin_amdgcn_readlane(slot[w], x));
      float acc0 = 0.0f, acc1 = 0.0f;
      pool_block(p, pitch, len, acc0, acc1);
      const float fl = (float)len;
      mean[w] = len > 0 ? make_float2(acc0 / fl, acc1 / fl) : make_float2(0.0f, 0.0f);
      if (job < 4) {
        if (i < a.nqb) *reinterpret_cast<float2*>(a.Qc + ((size_t)h * a.nqb + i) * D + 2 * c) = mean[w];
        *reinterpret_cast<float2*>(qs + job * D + 2 * c) = mean[w];
      }
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");  // what was staged for those columns has arrived: it is written over
    __syncthreads();
    auto put = [&](int w, int j) {
      const int r = 2 * c / DX, chunk = 2 * c % DX / 4;
      *reinterpret_cast<float2*>(smem + r * BUF + j * (DX * 4) + ((chunk ^ ((j >> 1) % CPC)) << 4) + (c % 2) * 8) = mean[w];
    };
#pragma unroll
    for (int w = 0; w < SW; ++w)
      if (slot[w] >= 0) {
        put(w, a.pool_from + w * JPS + (int)threadIdx.x / (D / 2) - 4);
        if (bx == 0) *reinterpret_cast<float2*>(a.Kc_l + ((size_t)h * a.n_loc_cap + slot[w]) * D + 2 * c) = mean[w];
      }
    if (__builtin_expect(twice, false)) {
#pragma unroll 1
      for (int j = 0; j < a.pool_from; ++j) {
        const int at = min(max(a.l_map[j], 0), a.n_loc_cap - 1);
#pragma unroll
        for (int w = 0; w < SW; ++w)
          if (slot[w] == at) put(w, j);
      }
    }
  } else if (a.Q) {
    const int r = threadIdx.x / (D / 2), c = threadIdx.x % (D / 2), i = i0 + r;
    if (r < 4) {
      float acc0 = 0.0f, acc1 = 0.0f;
      if (i < a.nqb) {
        const int len = min(a.B, a.Nq - i * a.B);
        const bf16_t* p = a.Q + (size_t)h * a.q_stride_h + (size_t)i * a.B * a.q_stride_t + 2 * c;
        if constexpr (NM <= 8) {
          pool_block(p, a.q_stride_t, len, acc0, acc1);
        } else {
          pool_rows<64, false>(p, a.q_stride_t, min(len, 64), acc0, acc1);
          if (len > 64) pool_rows<64, false>(p + 64 * a.q_stride_t, a.q_stride_t, len - 64, acc0, acc1);
        }
        const float fl = (float)len;
        acc0 = acc0 / fl;
        acc1 = acc1 / fl;
        *reinterpret_cast<float2*>(a.Qc + ((size_t)h * a.nqb + i) * D + 2 * c) = make_float2(acc0, acc1);
      }
      *reinterpret_cast<float2*>(qs + r * D + 2 * c) = make_float2(acc0, acc1);
    }
  } else {
    for (int idx = threadIdx.x; idx < 4 * D; idx += NT) {
      const int r = idx / D, x = idx % D;
      qs[idx] = i0 + r < a.nqb ? a.Qc[((size_t)h * a.nqb + i0 + r) * D + x] : 0.0f;
    }
  }
  __syncthreads();

  // The logits: lane = column; element r of acc runs the chain of query block r.  a_q[m] holds dimensions 16 m .. 16 m + 15 of
  // the four queries, as the instruction wants them.
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  const int jcol = 64 * wave + lane;
  const int sw = (jcol >> 1) % CPC;
  if (has_cols) {
    float a_q[D / 16];
#pragma unroll
    for (int m = 0; m < D / 16; ++m) a_q[m] = qs[(lane & 3) * D + 16 * m + (lane >> 2)];
    unroll([&](auto R) {
      constexpr int r0 = decltype(R)::value, later = (r0 + NBUF <= NR ? NBUF : NR - r0) - 1;   // rounds on their way behind r0
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(later * NI) : "memory");
      const unsigned char* kb = smem + (r0 % NBUF) * BUF + jcol * (DX * 4);
      float4 k4[CPC];
#pragma unroll
      for (int c = 0; c < CPC; ++c) k4[c] = *reinterpret_cast<const float4*>(kb + ((c ^ sw) << 4));
      unroll([&](auto C) {
        constexpr int c = decltype(C)::value, x = r0 * DX + 4 * c;
        acc = fma_4_rows<(x + 0) % 16>(a_q[x / 16], k4[c].x, acc);
        acc = fma_4_rows<(x + 1) % 16>(a_q[x / 16], k4[c].y, acc);
        acc = fma_4_rows<(x + 2) % 16>(a_q[x / 16], k4[c].z, acc);
        acc = fma_4_rows<(x + 3) % 16>(a_q[x / 16], k4[c].w, acc);
      }, std::make_integer_sequence<int, CPC>{});
      if constexpr (r0 + NBUF < NR) {
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");     // this round has been read: its place is free
        PBSA_STAGE(r0 + NBUF)
      }
    }, std::make_integer_sequence<int, NR>{});
  }
#undef PBSA_STAGE

  if (has_cols)
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const float z = acc[r] * a.scale;
    zs[r * NCP + jcol] = z;
    if (a.Zl && i0 + r < a.nqb && jcol < a.n_loc) a.Zl[((size_t)h * a.nqb + i0 + r) * a.n_loc + jcol] = z;
  }
  __syncthreads();

  {
    const int r = wave, i = i0 + r;
    if (r >= 4 || i >= a.nqb) return;
    // order-preserving integer keys; invisible columns get 0, below every real value
    const int nvis = a.causal ? a.n_loc - a.nqb + i + 1 : a.n_loc;
    uint32_t key[NM];
#pragma unroll
    for (int m = 0; m < NM; ++m) {
      float z = zs[r * NCP + lane + 64 * m];
      if (z == 0.0f) z = 0.0f;                    // -0 and +0 compare equal: give them one key
      const uint32_t b = __float_as_uint(z);
      const uint32_t ordered = (b & 0x80000000u) ? ~b : (b | 0x80000000u);
      key[m] = (lane + 64 * m < nvis) ? ordered : 0u;
    }
    const int kk = min(a.k, nvis);
    int32_t* out = a.sel + ((size_t)h * a.nqb + i) * a.k;
    if (kk > 0) {
      // T = kk-th largest key, found bit by bit: the largest T with #{key >= T} >= kk
      // (once exactly kk keys are at or above T, lower bits of it take none of them away)
      uint32_t T = 0;
      for (int bit = 31; bit >= 0; --bit) {
        const uint32_t cand = T | (1u << bit);
        int cnt = 0;
#pragma unroll
        for (int m = 0; m < NM; ++m) cnt += __popcll(__ballot(key[m] >= cand));
        if (cnt >= kk) T = cand;
        if (cnt == kk) break;
      }
      int n_gt = 0;
#pragma unroll
      for (int m = 0; m < NM; ++m) n_gt += __popcll(__ballot(key[m] > T));
      const int need_eq = kk - n_gt;              // ties at T taken in ascending block order
      int seen_eq = 0, pos = 0;
#pragma unroll
      for (int m = 0; m < NM; ++m) {
        const bool eq = key[m] == T;
        const uint64_t eq_mask = __ballot(eq);
        const bool take = key[m] > T || (eq && seen_eq + lanes_below(eq_mask) < need_eq);
        const uint64_t take_mask = __ballot(take);
        if (take) out[pos + lanes_below(take_mask)] = lane + 64 * m;
        seen_eq += __popcll(eq_mask);
        pos += __popcll(take_mask);
      }
    }
    for (int j = kk + lane; j < a.k; j += 64) out[j] = -1;
  }
}

template <int D, int NM>
__global__ void __launch_bounds__(64 * (NM < 4 ? 4 : NM)) select_kernel(SelectArgs a) {
  extern __shared__ __align__(1024) unsigned char smem[];
  select_body<D, NM>(a, blockIdx.x, blockIdx.y, smem);
}

// ------------------------------------------------------------------------------------------------
// Fold + promote.  One thread owns 4 dimensions of one position t of K or V of one head: it adds
// the dropped blocks' rows to the running sum in candidate order, rewrites the summary row, then
// copies row t of every kept newcomer into its slot.  A slot that is both dropped and refilled is
// read and written by the same thread, in that order.
// ------------------------------------------------------------------------------------------------
struct FoldArgs {
  int H, B, d, C, n_loc_cap, n_evict, fold;
  bf16_t* Kp;
  bf16_t* Vp;
  const bf16_t* Kl;
  const bf16_t* Vl;
  float* S_sum;
  const int32_t* S_cnt;
  const int32_t* fold_n;
  const int32_t* fold_src;
  const int32_t* fold_len;
  const int32_t* promo_slot;
  const int32_t* plen_new;  // the slots' lengths after the update ...
  int32_t* p_len;           // ... which this kernel commits
};

constexpr int kFoldBatch = 40, kFoldFew = 8;
constexpr int kPromoBatch = 8;

// FEW: up to so many dropped blocks take a batch of FEW instead of kFoldBatch
template <int NT, int FEW>
__device__ __forceinline__ void fold_promote_body(const FoldArgs& a, const int bx, const int h) {
  // per dropped candidate: its valid length and the address of its K and of its V block
  __shared__ const bf16_t* fptr_s[2][kMaxCand];
  __shared__ int flen_s[kMaxCand];
  __shared__ int promo_dst[PBSA_MAX_C], promo_src[PBSA_MAX_C], n_promo_s;   // refilled slots, compacted
  const int C = a.C, C1 = a.C + 1, ncand_max = a.C + a.n_evict;
  if (bx == 0)                             // nothing in this launch reads p_len: the lists carry the lengths they need
    for (int c = threadIdx.x; c < C1; c += NT) a.p_len[(size_t)h * C1 + c] = a.plen_new[(size_t)h * C1 + c];
  const int nf = a.fold && a.S_sum ? a.fold_n[h] : 0;
  const size_t blk = (size_t)a.B * a.d;
  for (int f = threadIdx.x; f < nf; f += NT) {
    const int src = a.fold_src[(size_t)h * ncand_max + f];
    flen_s[f] = a.fold_len[(size_t)h * ncand_max + f];
    fptr_s[0][f] = src < C ? a.Kp + ((size_t)h * C1 + src) * blk : a.Kl + ((size_t)h * a.n_loc_cap + (src - C)) * blk;
    fptr_s[1][f] = src < C ? a.Vp + ((size_t)h * C1 + src) * blk : a.Vl + ((size_t)h * a.n_loc_cap + (src - C)) * blk;
  }
  if (threadIdx.x < 64) {                  // wave 0 compacts the slots that are refilled (usually few or none)
    int n = 0;
    for (int c0 = 0; c0 < C; c0 += 64) {
      const int c = c0 + (int)threadIdx.x;
      const int ps = c < C ? a.promo_slot[(size_t)h * C + c] : -1;
      const uint64_t m = __ballot(ps >= 0);
      if (ps >= 0) {
        const int pos = n + lanes_below(m);
        promo_dst[pos] = c;
        promo_src[pos] = ps;
      }
      n += __popcll(m);
    }
    if (threadIdx.x == 0) n_promo_s = n;
  }
  __syncthreads();
  const int n_promo = n_promo_s;
  const int tpr = a.d / 4;                                     // threads per row: 4 dimensions each
  const int rows_per_wg = NT / tpr;
  const int row = bx * rows_per_wg + threadIdx.x / tpr;         // over [2][B]
  const int xc = (threadIdx.x % tpr) * 4;
  if (row >= 2 * a.B) return;
  const int kv = row / a.B, t = row % a.B;
  bf16_t* P = kv ? a.Vp : a.Kp;
  const bf16_t* L = kv ? a.Vl : a.Kl;
  const size_t rowoff = (size_t)t * a.d + xc;
  const bf16_t* Lh = L + (size_t)h * a.n_loc_cap * blk + rowoff;
  // promoted rows are independent of the fold: the first few are fetched before it starts
  uint2 pv[kPromoBatch];
#pragma unroll
  for (int u = 0; u < kPromoBatch; ++u)
    pv[u] = u < n_promo ? *reinterpret_cast<const uint2*>(Lh + (size_t)promo_src[u] * blk) : make_uint2(0u, 0u);
  if (nf > 0) {
    float* ssum = a.S_sum + ((size_t)h * 2 + kv) * blk + rowoff;
    float4 acc = *reinterpret_cast<float4*>(ssum);
    const int cnt = a.S_cnt[(size_t)h * a.B + t];     // already the new count (retain_kernel)
    // rows are loaded kFoldBatch at a time (row t exists in every block, valid or not) and added in
    // candidate order, the add predicated on t < len
    auto batch = [&](auto N, int f0) {
      uint2 v[decltype(N)::value];
#pragma unroll
      for (int u = 0; u < decltype(N)::value; ++u)
        v[u] = *reinterpret_cast<const uint2*>(fptr_s[kv][min(f0 + u, nf - 1)] + rowoff);
#pragma unroll
      for (int u = 0; u < decltype(N)::value; ++u) {
        if (f0 + u < nf && t < flen_s[f0 + u]) {
          acc.x = acc.x + bf_lo(v[u].x);
          acc.y = acc.y + bf_hi(v[u].x);
          acc.z = acc.z + bf_lo(v[u].y);
          acc.w = acc.w + bf_hi(v[u].y);
        }
      }
    };
    // (the code of a large batch takes longer to fetch than the few blocks of a small chunk to add)
    if (FEW > 0 && nf <= FEW) {
      batch(std::integral_constant<int, FEW ? FEW : 1>{}, 0);
    } else {
      for (int f0 = 0; f0 < nf; f0 += kFoldBatch) batch(std::integral_constant<int, kFoldBatch>{}, f0);
    }
    *reinterpret_cast<float4*>(ssum) = acc;
    if (cnt > 0) {
      const float fc = (float)cnt;
      uint2 w;
      w.x = f2bf_rne(acc.x / fc) | (f2bf_rne(acc.y / fc) << 16);
      w.y = f2bf_rne(acc.z / fc) | (f2bf_rne(acc.w / fc) << 16);
      *reinterpret_cast<uint2*>(P + ((size_t)h * C1 + C) * blk + rowoff) = w;
    }
  }
  // promoted rows: stores after the fold's loads (a refilled slot was read above by this thread)
#pragma unroll
  for (int u = 0; u < kPromoBatch; ++u)
    if (u < n_promo) *reinterpret_cast<uint2*>(P + ((size_t)h * C1 + promo_dst[u]) * blk + rowoff) = pv[u];
  for (int u0 = kPromoBatch; u0 < n_promo; u0 += kPromoBatch) {     // more than a few: the rest, batch by batch
#pragma unroll
    for (int u = 0; u < kPromoBatch; ++u)
      pv[u] = u0 + u < n_promo ? *reinterpret_cast<const uint2*>(Lh + (size_t)promo_src[u0 + u] * blk) : make_uint2(0u, 0u);
#pragma unroll
    for (int u = 0; u < kPromoBatch; ++u)
      if (u0 + u < n_promo) *reinterpret_cast<uint2*>(P + ((size_t)h * C1 + promo_dst[u0 + u]) * blk + rowoff) = pv[u];
  }
}

// The selection of a small chunk with everything that would be a launch before it: the pooling; the fold / promote of the
// update before it, in n_fold_x workgroups per head of their own; the copy of the chunk into the ring, one workgroup per
// block of K and of V.
template <int D>
__global__ void __launch_bounds__(512) select_small_kernel(SelectArgs a, FoldArgs fa, int n_fold_x, AppendArgs ap) {
  extern __shared__ __align__(1024) unsigned char smem[];
  const int h = blockIdx.y, n_sel_x = (a.nqb + 3) / 4;
  int bx = (int)blockIdx.x;
  if (bx < n_fold_x) {
    fold_promote_body<512, kFoldFew>(fa, bx, h);
    return;
  }
  bx -= n_fold_x;
  if (bx < n_sel_x) {
    select_body<D, 2, true>(a, bx, h, smem);
    return;
  }
  bx -= n_sel_x;
  constexpr int CPR = D / 8, RPS = 512 / CPR;              // 16-byte chunks per row, rows at a time
  const int kv = bx & 1, i = bx >> 1, c = threadIdx.x % CPR;
  const int len = min(ap.B, ap.Nq - i * ap.B), rows = ap.zero_tail ? ap.B : len;
  const bf16_t* const src = ap.src[kv] + (size_t)h * ap.sh[kv] + (size_t)i * ap.B * ap.st[kv] + 8 * c;
  bf16_t* const dst = ap.dst[kv] + ((size_t)h * ap.n_loc_cap + ap.slot0 + i) * ap.B * D + 8 * c;
#pragma unroll 4
  for (int r = threadIdx.x / CPR; r < rows; r += RPS) {
    uint4 v = *reinterpret_cast<const uint4*>(src + (size_t)min(r, len - 1) * ap.st[kv]);
    if (r >= len) v = make_uint4(0u, 0u, 0u, 0u);
    *reinterpret_cast<uint4*>(dst + (size_t)r * D) = v;
  }
}

// ------------------------------------------------------------------------------------------------
// Persistence scores, rows (Eq. 7): wave per query block; columns U = occupied persistent slots in
// slot order, then all local blocks.  Row softmax in the pinned order; the sum runs sequentially
// over the row in LDS.
// ------------------------------------------------------------------------------------------------

template <int D, int NM>
__global__ void __launch_bounds__(kThreads) score_rows_kernel(ScoreArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  constexpr int NPAD = NM * 64 + 2;
  float* kct = reinterpret_cast<float*>(smem);
  float* qs = kct + kXC * NPAD;
  const float** cols = reinterpret_cast<const float**>(qs + 4 * D);
  float* erow = reinterpret_cast<float*>(cols + NM * 64);                       // [4][NM*64]
  __shared__ int nP_s;
  __shared__ float sum_s[4];
  const int h = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + wave;
  const bool row_ok = i < a.nqb;
  if (threadIdx.x == 0) {
    int n = 0;
    for (int s = 0; s < a.C; ++s)
      if (a.p_len[(size_t)h * (a.C + 1) + s] > 0) cols[n++] = a.Kc_p + ((size_t)h * a.C + s) * D;
    nP_s = n;
  }
  __syncthreads();
  const int nP = nP_s, nU = nP + a.n_loc;
  for (int j = threadIdx.x; j < a.n_loc; j += kThreads) {
    int slot = a.l_map[j];
    slot = min(max(slot, 0), a.n_loc_cap - 1);
    cols[nP + j] = a.Kc_l + ((size_t)h * a.n_loc_cap + slot) * D;
  }
  for (int x = lane; x < D; x += 64) qs[wave * D + x] = row_ok ? a.Qc[((size_t)h * a.nqb + i) * D + x] : 0.0f;
  float acc[NM];
  coarse_dots<D, NM>(cols, nU, qs + wave * D, kct, acc);

  float mx = -INFINITY;
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    acc[m] = acc[m] * a.scale;
    if (lane + 64 * m < nU) mx = fmaxf(mx, acc[m]);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  float* er = erow + wave * (NM * 64);
#pragma unroll
  for (int m = 0; m < NM; ++m) {
    acc[m] = (lane + 64 * m < nU) ? pexp(acc[m] - mx) : 0.0f;
    er[lane + 64 * m] = acc[m];
  }
  __syncthreads();
  if (lane == 0) {
    float s = 0.0f;
#pragma unroll 16
    for (int j = 0; j < nU; ++j) s = s + er[j];
    sum_s[wave] = s;
  }
  __syncthreads();
  if (!row_ok) return;
  const float s = sum_s[wave];
  // stored column-major (A^T[h][j][i]) so the column means read contiguous rows
  // (only the columns that can be candidates are needed downstream: slots, then evicted blocks)
  float* acol = a.A + (size_t)h * a.nU_max * a.nqb_pad + i;
  const int n_need = nP + a.n_evict;
#pragma unroll
  for (int m = 0; m < NM; ++m)
    if (lane + 64 * m < n_need) acol[(size_t)(lane + 64 * m) * a.nqb_pad] = acc[m] / s;
}

// Same rows when the selection call has left the local logits in Zl: only the (at most 64) persistent
// columns are multiplied here; lane `lane` owns persistent column `lane` and local columns lane + 64 m.
template <int D, int NML>
__global__ void __launch_bounds__(kThreads) score_rows_z_kernel(ScoreArgs a) {
  extern __shared__ __align__(16) unsigned char smem[];
  float* kct = reinterpret_cast<float*>(smem);                                  // [64][D + 4]
  float* qs = kct + 64 * (D + 4);                                               // [4][D]
  const float** cols = reinterpret_cast<const float**>(qs + 4 * D);            // [64]
  float* erow = reinterpret_cast<float*>(cols + 64);                            // [4][64 + NML*64]
  __shared__ float sum_s[4];
  const int h = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int i = blockIdx.x * 4 + wave;
  const bool row_ok = i < a.nqb;
  const bool occ = lane < a.C && a.p_len[(size_t)h * (a.C + 1) + lane] > 0;
  const uint64_t occ_mask = __ballot(occ);
  const int nP = __popcll(occ_mask), nU = nP + a.n_loc;
  if (wave == 0 && occ) cols[lanes_below(occ_mask)] = a.Kc_p + ((size_t)h * a.C + lane) * D;
  for (int x = lane; x < D; x += 64) qs[wave * D + x] = row_ok ? a.Qc[((size_t)h * a.nqb + i) * D + x] : 0.0f;
  float zl[NML];
  const float* zrow = a.Zl + ((size_t)h * a.nqb + min(i, a.nqb - 1)) * a.n_loc;
#pragma unroll
  for (int m = 0; m < NML; ++m) zl[m] = lane + 64 * m < a.n_loc ? zrow[lane + 64 * m] : 0.0f;
  // the occupied slots' pooled keys, whole, [nP][D + 4] (the pitch spreads the 16-byte reads of 16
  // lanes over all banks); then lane c runs the chain of column c
  __syncthreads();                                       // cols[] and qs are visible
  constexpr int KP = D + 4;
  for (int idx = threadIdx.x; idx < nP * (D / 4); idx += kThreads) {
    const int u = idx / (D / 4), x4 = idx % (D / 4);
    *reinterpret_cast<float4*>(kct + u * KP + 4 * x4) = reinterpret_cast<const float4*>(cols[u])[x4];
  }
  __syncthreads();
  float accp = 0.0f;
  if (lane < nP) {
    const float4* q4p = reinterpret_cast<const float4*>(qs + wave * D);
    const float4* k4p = reinterpret_cast<const float4*>(kct + lane * KP);
#pragma unroll 8
    for (int x4 = 0; x4 < D / 4; ++x4) {
      const float4 q = q4p[x4], k = k4p[x4];
      accp = __builtin_fmaf(q.x, k.x, accp);
      accp = __builtin_fmaf(q.y, k.y, accp);
      accp = __builtin_fmaf(q.z, k.z, accp);
      accp = __builtin_fmaf(q.w, k.w, accp);
    }
  }
  const float zp = accp * a.scale;

  float mx = lane < nP ? zp : -INFINITY;
#pragma unroll
  for (int m = 0; m < NML; ++m)
    if (lane + 64 * m < a.n_loc) mx = fmaxf(mx, zl[m]);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off, 64));
  float* er = erow + wave * (64 + NML * 64);
  const float ep = lane < nP ? pexp(zp - mx) : 0.0f;
  if (lane < nP) er[lane] = ep;
#pragma unroll
  for (int m = 0; m < NML; ++m) {
    zl[m] = (lane + 64 * m < a.n_loc) ? pexp(zl[m] - mx) : 0.0f;
    if (lane + 64 * m < a.n_loc) er[nP + lane + 64 * m] = zl[m];
  }
  __syncthreads();
  if (lane == 0) {
    float s = 0.0f;
#pragma unroll 16
    for (int j = 0; j < nU; ++j) s = s + er[j];
    sum_s[wave] = s;
  }
  __syncthreads();
  if (!row_ok) return;
  const float s = sum_s[wave];
  float* acol = a.A + (size_t)h * a.nU_max * a.nqb_pad + i;
  if (lane < nP) acol[(size_t)lane * a.nqb_pad] = ep / s;
#pragma unroll
  for (int m = 0; m < NML; ++m)
    if (lane + 64 * m < a.n_evict) acol[(size_t)(nP + lane + 64 * m) * a.nqb_pad] = zl[m] / s;
}

// ------------------------------------------------------------------------------------------------
// Retention (Eq. 8-9): one workgroup per head (the body is shared with the attention launch that takes the
// decisions beside the attention: pbsa_plan_device.h).
// ------------------------------------------------------------------------------------------------
__global__ void __launch_bounds__(kThreads) retain_kernel(RetainArgs a) {
  __shared__ RetainLds L;
  const int h = blockIdx.x;
  retain_body<kThreads>(a, h, retain_prefetch<kThreads>(a, h), a.A + (size_t)h * a.nU_max * a.nqb_pad, false, L);
}

// The bf16 view of a summary given by its running sums and counts (slot C of every head): row t of K and of V is
// S_sum[t] / S_cnt[t], divided in fp32 and rounded to nearest even, where S_cnt[t] > 0; other rows stay as they are;
// the slot's length is the number of such rows.  One thread per 4 dimensions of a row, as in the fold.
__global__ void __launch_bounds__(kThreads) summary_view_kernel(int H, int B, int d, int C, const float* S_sum,
                                                                const int32_t* S_cnt, bf16_t* Kp, bf16_t* Vp,
                                                                int32_t* p_len) {
  const int h = blockIdx.y, C1 = C + 1;
  if (blockIdx.x == 0 && threadIdx.x < 64) {
    int n = 0;
    for (int t0 = 0; t0 < B; t0 += 64) {
      const int t = t0 + (int)threadIdx.x;
      n += __popcll(__ballot(t < B && S_cnt[(size_t)h * B + t] > 0));
    }
    if (threadIdx.x == 0) p_len[(size_t)h * C1 + C] = n;
  }
  const int tpr = d / 4, rows_per_wg = kThreads / tpr;
  const int row = blockIdx.x * rows_per_wg + threadIdx.x / tpr;
  if (row >= 2 * B) return;
  const int kv = row / B, t = row % B, xc = (threadIdx.x % tpr) * 4;
  const int cnt = S_cnt[(size_t)h * B + t];
  if (cnt <= 0) return;
  const size_t blk = (size_t)B * d, rowoff = (size_t)t * d + xc;
  const float4 acc = *reinterpret_cast<const float4*>(S_sum + ((size_t)h * 2 + kv) * blk + rowoff);
  const float fc = (float)cnt;
  uint2 w;
  w.x = f2bf_rne(acc.x / fc) | (f2bf_rne(acc.y / fc) << 16);
  w.y = f2bf_rne(acc.z / fc) | (f2bf_rne(acc.w / fc) << 16);
  *reinterpret_cast<uint2*>((kv ? Vp : Kp) + ((size_t)h * C1 + C) * blk + rowoff) = w;
}

template <int FEW>
__global__ void __launch_bounds__(kFoldThreads) fold_promote_kernel(FoldArgs a) {
  fold_promote_body<kFoldThreads, FEW>(a, blockIdx.x, blockIdx.y);
}

// The pooling of one chunk's selection call and the fold / promote of the update of the chunk before it, as one
// launch: the two touch disjoint data when the new chunk does not sit in the ring position whose blocks are being
// folded, and each is too short to fill the GPU for long.  The n_fold_x * H fold workgroups come first.
template <int D>
__global__ void __launch_bounds__(kFoldThreads) pool_fold_kernel(PoolArgs pa, FoldArgs fa, int n_fold_x) {
  const int n_fold = n_fold_x * fa.H, b = (int)blockIdx.x;      // the fold's workgroups run longest: they start first
  if (b >= n_fold) pool_body<D, kFoldThreads>(pa, b - n_fold);
  // (here the choice of a batch costs nothing: 15.0 us as for the large one alone, 15.2 where the host chooses, 12 heads x 37 blocks)
  else fold_promote_body<kFoldThreads, kFoldFew>(fa, b % n_fold_x, b / n_fold_x);
}

size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

template <typename K>
hipError_t allow_lds(K kernel, size_t bytes) {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize,
                             (int)bytes);
}

template <int NM>
size_t coarse_lds_bytes(int d, bool with_rows) {
  size_t b = (size_t)kXC * (NM * 64 + 2) * 4 + (size_t)4 * d * 4 + (size_t)NM * 64 * 8;
  if (with_rows) b += (size_t)4 * NM * 64 * 4;
  return b;
}

}  // namespace

UpdateWs carve_update_ws(const pbsa_params& p, void* base) {
  UpdateWs w;
  char* b = static_cast<char*>(base);
  size_t off = 0;
  const size_t nU_max = (size_t)p.C + p.n_loc, ncand = (size_t)p.C + p.n_evict;
  const size_t nqb_pad = ((size_t)p.nqb + 3) & ~(size_t)3;
  w.A = reinterpret_cast<float*>(b + off);          off += align256((size_t)p.H * nU_max * nqb_pad * 4);
  w.fold_n = reinterpret_cast<int32_t*>(b + off);   off += align256((size_t)p.H * 4);
  w.fold_src = reinterpret_cast<int32_t*>(b + off); off += align256((size_t)p.H * ncand * 4);
  w.fold_len = reinterpret_cast<int32_t*>(b + off); off += align256((size_t)p.H * ncand * 4);
  w.promo_slot = reinterpret_cast<int32_t*>(b + off); off += align256((size_t)p.H * (p.C + 1) * 4);
  w.plen_new = reinterpret_cast<int32_t*>(b + off); off += align256((size_t)p.H * (p.C + 1) * 4);
  w.bytes = off;
  return w;
}

hipError_t launch_pool_blocks(const pbsa_params& p, const bf16_t* X, const int32_t* len, int32_t n_blocks,
                              float* out, hipStream_t stream) {
  if (n_blocks == 0) return hipSuccess;
  PoolArgs a{};
  a.mode = 0; a.n_jobs = n_blocks; a.B = p.B; a.X = X; a.len = len; a.out = out;
  return p.d == 128 ? launch_pool<128>(a, stream) : launch_pool<64>(a, stream);
}

hipError_t launch_append(const pbsa_params& p, const bf16_t* K, const bf16_t* V, int64_t k_stride_h, int64_t k_stride_t,
                         int64_t v_stride_h, int64_t v_stride_t, int32_t slot0, int32_t zero_tail, bf16_t* Kl, bf16_t* Vl,
                         float* Kc_l, const bf16_t* Q, int64_t q_stride_h, int64_t q_stride_t, float* Qc, hipStream_t stream) {
  const AppendArgs a{p.B, p.Nq, p.nqb, p.n_loc_cap, slot0, zero_tail, {(long)k_stride_h, (long)v_stride_h, (long)q_stride_h},
                     {(long)k_stride_t, (long)v_stride_t, (long)q_stride_t}, {K, V, Q}, {Kl, Vl}, Kc_l, Qc};
  const dim3 grid(p.nqb, p.H, Q ? 3 : 2), block(kThreads);
  if (p.d == 128 && p.B == 128) hipLaunchKernelGGL((append_kernel<128, 128>), grid, block, 0, stream, a);
  else if (p.d == 128) hipLaunchKernelGGL((append_kernel<128, 64>), grid, block, 0, stream, a);
  else if (p.B == 128) hipLaunchKernelGGL((append_kernel<64, 128>), grid, block, 0, stream, a);
  else hipLaunchKernelGGL((append_kernel<64, 64>), grid, block, 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_summary_view(const pbsa_params& p, const float* S_sum, const int32_t* S_cnt, bf16_t* Kp, bf16_t* Vp,
                               int32_t* p_len, hipStream_t stream) {
  const int rows_per_wg = kThreads / (p.d / 4);
  hipLaunchKernelGGL(summary_view_kernel, dim3((2 * p.B + rows_per_wg - 1) / rows_per_wg, p.H), dim3(kThreads), 0, stream,
                     p.H, p.B, p.d, p.C, S_sum, S_cnt, Kp, Vp, p_len);
  return hipGetLastError();
}

template <int D, int NM>
static hipError_t launch_select_t(const SelectArgs& a, hipStream_t stream) {
  constexpr size_t lds = SelectGeo<D, NM>::LDS;
  hipError_t e = allow_lds(select_kernel<D, NM>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((select_kernel<D, NM>), dim3((a.nqb + 3) / 4, a.H), dim3(64 * (NM < 4 ? 4 : NM)), lds, stream, a);
  return hipGetLastError();
}

// Whether the selection launch pools the query blocks itself.  Not when nothing is selected and no logits are wanted
// (there is none), and not when key blocks are to be pooled first: that launch takes the queries along (a denoising pass
// of 12 x 4680 x 128: 511.7 -> 503.9 us for four; of 2 x 600 x 128: 151 -> 140 for four, of 3 x 1500 x 64 140 -> 130 for three).
// launch_select_apply leaves the queries in its pooling launch: the fold sets that launch's length
// and hides their 14 MB (186.3 us per chained step against 187.8 at H = 12, 4680 rows of 128, blocks of 64).
static bool select_pools_queries(const pbsa_params& p, const float* Zl) { return (p.k > 0 || Zl) && p.pool_from >= p.n_loc; }

static PoolArgs select_pool_args(const pbsa_params& p, const bf16_t* Q, const bf16_t* Kl, const int32_t* l_len,
                                 const int32_t* l_map, float* Kc_l, float* Qc, bool with_queries) {
  PoolArgs pa{};
  pa.mode = 1; pa.H = p.H; pa.B = p.B; pa.Nq = p.Nq; pa.nqb = p.nqb; pa.n_loc = p.n_loc; pa.n_loc_cap = p.n_loc_cap;
  pa.pool_from = p.pool_from; pa.n_kjobs_per_head = p.n_loc - p.pool_from;
  pa.n_jobs = p.H * (pa.n_kjobs_per_head + (with_queries ? p.nqb : 0));
  pa.q_stride_h = p.q_stride_h; pa.q_stride_t = p.q_stride_t;
  pa.X = Kl; pa.Q = Q; pa.len = l_len; pa.l_map = l_map; pa.out = Kc_l; pa.Qc = Qc;
  return pa;
}

static FoldArgs fold_args(const pbsa_params& p, bf16_t* Kp, bf16_t* Vp, int32_t* p_len, float* S_sum,
                          const int32_t* S_cnt, const bf16_t* Kl, const bf16_t* Vl, const UpdateWs& ws) {
  return FoldArgs{p.H, p.B, p.d, p.C, p.n_loc_cap, p.n_evict, S_sum != nullptr, Kp, Vp, Kl, Vl, S_sum, S_cnt, ws.fold_n,
                  ws.fold_src, ws.fold_len, ws.promo_slot, ws.plen_new, p_len};
}

static SelectArgs select_args(const pbsa_params& p, const bf16_t* Q, const int32_t* l_map, float* Kc_l, float* Qc, int32_t* sel,
                              float* Zl) {
  return SelectArgs{p.H, p.nqb, p.n_loc, p.n_loc_cap, p.k, p.causal, p.scale, Kc_l, Qc, l_map, sel, Zl,
                    Q, p.B, p.Nq, p.q_stride_h, p.q_stride_t, nullptr, nullptr, 0, -1, 0, 0};
}

// Workgroups per head that fold beside a small selection (each of 512 threads, four dimensions of a row to one).
static int small_fold_x(int B, int d) { return (2 * B + 512 / (d / 4) - 1) / (512 / (d / 4)); }

// Whether the selection pools the stale key blocks itself, and not a launch before it.  Every workgroup of a head then reads
// them all, beside its own four query blocks: at most 12 blocks, and a workgroup has a compute unit to itself, so no more
// than 256 of them.  Beyond 128 KiB a workgroup only chunks of whole blocks, whose loops over the rows are the shorter
// ones, and where the heads are few.  Two launches -> one, us, heads x blocks:
//   the selection by itself (a denoising pass): 12 x 4 of 64 x 64 7.9 -> 6.6, 256 x 4 8.9 -> 7.0, 64 x 12 8.9 -> 7.6, 12 x 4 of
//   64 x 128 8.8 -> 8.4, 12 x 4 of 128 x 64 8.6 -> 7.6, 256 x 1 7.3 -> 6.4; 96 x 12 of 64 x 64 9.8 | 13.8, 384 x 1 7.0 | 8.6, 192 x 8
//   9.9 | 13.7; beyond 128 KiB with whole blocks 16 x 12 of 64 x 128 8.5 -> 8.0, 16 x 8 of 128 x 64 8.5 -> 8.4, 16 x 4 of 128 x 128
//   8.9 -> 8.4, but 16 x 12 of 128 x 64 8.6 | 8.8, 64 x 12 of 64 x 128 9.0 | 13.1, 64 x 8 of 128 x 64 8.7 | 8.9; with a last block that is
//   not whole 12 x 6 of 64 x 128 8.8 | 9.7, 12 x 12 of 128 x 64 9.0 | 9.3, 12 x 4 of 128 x 128 9.4 | 10.6;
//   with the append, whose copies come behind (a step): 12 x 4 of 64 x 64 22.0 -> 20.7, 96 x 4 32.9 -> 32.1, 32 x 12 33.6 -> 32.4, 64 x 4 of
//   128 x 64 42.5 -> 40.5; 256 x 1 of 64 x 64 40.5 | 42.0, 64 x 12 45.4 | 45.6; beyond 128 KiB with whole blocks 16 x 12 of 64 x 128
//   36.8 -> 35.7, 16 x 12 of 128 x 64 33.4 -> 31.3, 32 x 4 of 128 x 128 45.6 -> 43.9, but 32 x 12 of 64 x 128 46.9 | 48.0, 64 x 4 of 128 x 128
//   59.5 | 60.3; with a last block that is not 12 x 6 of 64 x 128 26.9 | 27.4, 64 x 4 of 128 x 128 60.7 | 62.3;
//   with the fold of the update before, whose workgroups count as well (a chained step): 12 x 4 of 64 x 64
//   18.4 -> 15.9, 12 x 12 of 64 x 128 27.5 -> 26.5, 12 x 12 of 128 x 64 25.4 -> 23.2, 12 x 2 of 128 x 128 26.3 -> 25.1; 64 x 8 of
//   64 x 64 30.9 | 31.2, 32 x 12 of 128 x 64 32.1 | 33.5, 64 x 1 of 128 x 128 34.9 | 37.1, 256 x 1 75 | 89.
static bool select_is_small(const pbsa_params& p, int n_stale, const float* Zl, int fold_x, bool append) {
  if (!(p.k > 0 || Zl) || n_stale < 1 || n_stale > kOwnKeys || p.nqb > kOwnKeys || p.n_loc > 128) return false;
  const int bytes = (4 + n_stale) * p.B * p.d * 2;
  const long wgs = (long)p.H * ((p.nqb + 3) / 4 + fold_x);
  if (fold_x > 0) return bytes <= 256 * 1024 && wgs <= 256;
  if (bytes <= 128 * 1024) return wgs <= (append ? 128 : 256);
  return p.Nq % p.B == 0 && bytes <= 256 * 1024 && wgs <= 64 && (append || p.d * n_stale <= 1024);
}

template <int D>
static hipError_t launch_select_small(const SelectArgs& a, const FoldArgs* fa, const AppendArgs* ap, hipStream_t stream) {
  constexpr size_t lds = SelectGeo<D, 2>::LDS;
  const hipError_t e = allow_lds(select_small_kernel<D>, lds);
  if (e != hipSuccess) return e;
  const int n_fold_x = fa ? small_fold_x(fa->B, D) : 0;
  hipLaunchKernelGGL(select_small_kernel<D>, dim3(n_fold_x + (a.nqb + 3) / 4 + (ap ? 2 * a.nqb : 0), a.H), dim3(512), lds, stream, a,
                     fa ? *fa : FoldArgs{}, n_fold_x, ap ? *ap : AppendArgs{});
  return hipGetLastError();
}
static hipError_t launch_select_small(const pbsa_params& p, SelectArgs a, const bf16_t* Kl, const int32_t* l_len, const FoldArgs* fa,
                                      hipStream_t stream) {
  a.Kl = Kl;
  a.l_len = l_len;
  a.pool_from = p.pool_from;
  return p.d == 128 ? launch_select_small<128>(a, fa, nullptr, stream) : launch_select_small<64>(a, fa, nullptr, stream);
}

static hipError_t launch_select_logits(const pbsa_params& p, const bf16_t* Q, const int32_t* l_map, float* Kc_l, float* Qc,
                                       int32_t* sel, float* Zl, hipStream_t stream);

hipError_t launch_select(const pbsa_params& p, const bf16_t* Q, const bf16_t* Kl, const int32_t* l_len,
                         const int32_t* l_map, float* Kc_l, float* Qc, int32_t* sel, float* Zl, bool pooled,
                         hipStream_t stream) {
  if (pooled) return launch_select_logits(p, nullptr, l_map, Kc_l, Qc, sel, Zl, stream);
  if (select_is_small(p, p.n_loc - p.pool_from, Zl, 0, false))
    return launch_select_small(p, select_args(p, Q, l_map, Kc_l, Qc, sel, Zl), Kl, l_len, nullptr, stream);
  const bool in_select = select_pools_queries(p, Zl);
  const PoolArgs pa = select_pool_args(p, Q, Kl, l_len, l_map, Kc_l, Qc, !in_select);
  if (pa.n_jobs > 0) {
    const hipError_t e = p.d == 128 ? launch_pool<128>(pa, stream) : launch_pool<64>(pa, stream);
    if (e != hipSuccess) return e;
  }
  return launch_select_logits(p, in_select ? Q : nullptr, l_map, Kc_l, Qc, sel, Zl, stream);
}

hipError_t launch_append_select(const pbsa_params& p, const bf16_t* K, const bf16_t* V, int64_t k_stride_h, int64_t k_stride_t,
                                int64_t v_stride_h, int64_t v_stride_t, int32_t slot0, int32_t zero_tail, const bf16_t* Q, bf16_t* Kl,
                                bf16_t* Vl, const int32_t* l_map, float* Kc_l, float* Qc, int32_t* sel, float* Zl, hipStream_t stream) {
  if (!select_is_small(p, p.nqb, Zl, 0, true)) {
    const hipError_t e = launch_append(p, K, V, k_stride_h, k_stride_t, v_stride_h, v_stride_t, slot0, zero_tail, Kl, Vl, Kc_l, Q,
                                       p.q_stride_h, p.q_stride_t, Qc, stream);
    return e != hipSuccess ? e : launch_select_logits(p, nullptr, l_map, Kc_l, Qc, sel, Zl, stream);
  }
  SelectArgs a = select_args(p, Q, l_map, Kc_l, Qc, sel, Zl);
  a.Kl = K;
  a.pool_from = p.n_loc - p.nqb;
  a.chunk_slot = slot0;
  a.k_stride_h = (long)k_stride_h;
  a.k_stride_t = (long)k_stride_t;
  const AppendArgs ap{p.B, p.Nq, p.nqb, p.n_loc_cap, slot0, zero_tail, {(long)k_stride_h, (long)v_stride_h, 0},
                      {(long)k_stride_t, (long)v_stride_t, 0}, {K, V, nullptr}, {Kl, Vl}, nullptr, nullptr};
  return p.d == 128 ? launch_select_small<128>(a, nullptr, &ap, stream) : launch_select_small<64>(a, nullptr, &ap, stream);
}

hipError_t launch_select_apply(const pbsa_params& p, const bf16_t* Q, const bf16_t* Kl, const int32_t* l_len,
                               const int32_t* l_map, float* Kc_l, float* Qc, int32_t* sel, float* Zl,
                               const pbsa_params& pu, bf16_t* Kp, bf16_t* Vp, int32_t* p_len, float* S_sum,
                               const int32_t* S_cnt, const bf16_t* Vl, const UpdateWs& ws, hipStream_t stream) {
  const PoolArgs pa = select_pool_args(p, Q, Kl, l_len, l_map, Kc_l, Qc, true);
  const FoldArgs fa = fold_args(pu, Kp, Vp, p_len, S_sum, S_cnt, Kl, Vl, ws);
  if (select_is_small(p, p.n_loc - p.pool_from, Zl, small_fold_x(pu.B, pu.d), false))
    return launch_select_small(p, select_args(p, Q, l_map, Kc_l, Qc, sel, Zl), Kl, l_len, &fa, stream);
  // the fold / promote workgroups ride in the pooling launch, whose workgroups have the same size and no LDS (in the logits
  // launch, whose workgroups take 36 to 145 KiB each, they would wait for places: 33.0 us for the call against 30.1, measured
  // when those took 80)
  const int jpw = kFoldThreads / (p.d / 2), rows_per_wg = kFoldThreads / (pu.d / 4);
  const int n_fold_x = (2 * pu.B + rows_per_wg - 1) / rows_per_wg;
  const dim3 grid(n_fold_x * pu.H + (pa.n_jobs + jpw - 1) / jpw);
  if (p.d == 128) hipLaunchKernelGGL(pool_fold_kernel<128>, grid, dim3(kFoldThreads), 0, stream, pa, fa, n_fold_x);
  else hipLaunchKernelGGL(pool_fold_kernel<64>, grid, dim3(kFoldThreads), 0, stream, pa, fa, n_fold_x);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  return launch_select_logits(p, nullptr, l_map, Kc_l, Qc, sel, Zl, stream);
}

static hipError_t launch_select_logits(const pbsa_params& p, const bf16_t* Q, const int32_t* l_map, float* Kc_l, float* Qc,
                                       int32_t* sel, float* Zl, hipStream_t stream) {
  if (p.k == 0 && !Zl) return hipSuccess;

  const SelectArgs a = select_args(p, Q, l_map, Kc_l, Qc, sel, Zl);
  const int nm = (p.n_loc + 63) / 64;
  if (p.d == 128) {
    if (nm <= 2) return launch_select_t<128, 2>(a, stream);
    if (nm <= 5) return launch_select_t<128, 5>(a, stream);
    if (nm <= 8) return launch_select_t<128, 8>(a, stream);
    return launch_select_t<128, 11>(a, stream);
  }
  static_assert(PBSA_MAX_N_LOC <= 11 * 64, "one lane per local block");
  if (nm <= 2) return launch_select_t<64, 2>(a, stream);
  if (nm <= 5) return launch_select_t<64, 5>(a, stream);
  if (nm <= 8) return launch_select_t<64, 8>(a, stream);
  return launch_select_t<64, 11>(a, stream);
}

template <int D, int NM>
static hipError_t launch_rows_t(const ScoreArgs& a, hipStream_t stream) {
  const size_t lds = coarse_lds_bytes<NM>(D, true);
  hipError_t e = allow_lds(score_rows_kernel<D, NM>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((score_rows_kernel<D, NM>), dim3((a.nqb + 3) / 4, a.H), dim3(kThreads), lds, stream, a);
  return hipGetLastError();
}

template <int D, int NML>
static hipError_t launch_rows_z_t(const ScoreArgs& a, hipStream_t stream) {
  const size_t lds = (size_t)64 * (D + 4) * 4 + (size_t)4 * D * 4 + 64 * 8 + (size_t)4 * (64 + NML * 64) * 4;
  hipError_t e = allow_lds(score_rows_z_kernel<D, NML>, lds);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL((score_rows_z_kernel<D, NML>), dim3((a.nqb + 3) / 4, a.H), dim3(kThreads), lds, stream, a);
  return hipGetLastError();
}

static hipError_t launch_scores(const pbsa_params& p, const float* Qc, const float* Kc_l, const float* Zl,
                                const float* Kc_p, const int32_t* p_len, const int32_t* l_map, const UpdateWs& ws,
                                hipStream_t stream) {
  const int nU_max = p.C + p.n_loc;
  const ScoreArgs sa = make_score_args(p, Qc, Kc_l, Zl, Kc_p, p_len, l_map, ws);
  const int nm = (nU_max + 63) / 64;
  if (Zl) {
    const int nml = (p.n_loc + 63) / 64;
    if (p.d == 128)
      return nml <= 2 ? launch_rows_z_t<128, 2>(sa, stream) : nml <= 5 ? launch_rows_z_t<128, 5>(sa, stream)
                                                                      : launch_rows_z_t<128, 8>(sa, stream);
    return nml <= 2 ? launch_rows_z_t<64, 2>(sa, stream) : nml <= 5 ? launch_rows_z_t<64, 5>(sa, stream)
                                                                    : launch_rows_z_t<64, 8>(sa, stream);
  }
  if (p.d == 128)
    return nm <= 2 ? launch_rows_t<128, 2>(sa, stream) : nm <= 6 ? launch_rows_t<128, 6>(sa, stream)
                                                                : launch_rows_t<128, 9>(sa, stream);
  return nm <= 2 ? launch_rows_t<64, 2>(sa, stream) : nm <= 6 ? launch_rows_t<64, 6>(sa, stream)
                                                              : launch_rows_t<64, 9>(sa, stream);
}

// Retention given the matrix whose row sums are the scores (A: the coarse matrix in the workspace, or the mass matrix)
static hipError_t launch_retain(const pbsa_params& p, const float* A, int n_rows, int fine, const float* Kc_l,
                                float* Kc_p, const int32_t* p_len, int64_t* p_id, int32_t* S_cnt, int fold,
                                const int32_t* l_len, const int32_t* l_map, const int64_t* l_id, float* scores,
                                int32_t* slot_src, const UpdateWs& ws, hipStream_t stream) {
  const RetainArgs ra = make_retain_args(p, A, n_rows, fine, Kc_l, Kc_p, p_len, p_id, S_cnt, fold, l_len, l_map, l_id,
                                         scores, slot_src, ws);
  hipLaunchKernelGGL(retain_kernel, dim3(p.H), dim3(kThreads), 0, stream, ra);
  return hipGetLastError();
}

hipError_t launch_update_plan(const pbsa_params& p, const float* Qc, const float* Kc_l, const float* Zl, float* Kc_p,
                              const int32_t* p_len, int64_t* p_id, int32_t* S_cnt, int fold, const int32_t* l_len,
                              const int32_t* l_map, const int64_t* l_id, float* scores, int32_t* slot_src,
                              const UpdateWs& ws, hipStream_t stream) {
  hipError_t e = launch_scores(p, Qc, Kc_l, Zl, Kc_p, p_len, l_map, ws, stream);
  if (e != hipSuccess) return e;
  return launch_retain(p, ws.A, p.C + p.n_loc, 0, Kc_l, Kc_p, p_len, p_id, S_cnt, fold, l_len, l_map, l_id, scores,
                       slot_src, ws, stream);
}

hipError_t launch_update_apply(const pbsa_params& p, bf16_t* Kp, bf16_t* Vp, int32_t* p_len, float* S_sum,
                               const int32_t* S_cnt, const bf16_t* Kl, const bf16_t* Vl, const UpdateWs& ws,
                               hipStream_t stream) {
  const FoldArgs fa = fold_args(p, Kp, Vp, p_len, S_sum, S_cnt, Kl, Vl, ws);
  const int rows_per_wg = kFoldThreads / (p.d / 4);
  const dim3 grid((2 * p.B + rows_per_wg - 1) / rows_per_wg, p.H);
  // (the choice costs the large batch 0.8 us of 13 by itself, at 12 heads x 74 blocks: only where the update may drop so few)
  if (p.n_evict <= kFoldFew) hipLaunchKernelGGL(fold_promote_kernel<kFoldFew>, grid, dim3(kFoldThreads), 0, stream, fa);
  else hipLaunchKernelGGL(fold_promote_kernel<0>, grid, dim3(kFoldThreads), 0, stream, fa);
  return hipGetLastError();
}

hipError_t launch_update(const pbsa_params& p, const float* Qc, const float* Kc_l, const float* Zl, bf16_t* Kp,
                         bf16_t* Vp, float* Kc_p, int32_t* p_len, int64_t* p_id, float* S_sum, int32_t* S_cnt,
                         const bf16_t* Kl, const bf16_t* Vl, const int32_t* l_len, const int32_t* l_map,
                         const int64_t* l_id, float* scores, int32_t* slot_src, const UpdateWs& ws,
                         hipStream_t stream) {
  hipError_t e = launch_update_plan(p, Qc, Kc_l, Zl, Kc_p, p_len, p_id, S_cnt, S_sum != nullptr, l_len, l_map, l_id, scores,
                                    slot_src, ws, stream);
  if (e != hipSuccess) return e;
  return launch_update_apply(p, Kp, Vp, p_len, S_sum, S_cnt, Kl, Vl, ws, stream);
}

hipError_t launch_update_fine(const pbsa_params& p, const float* Mt, const float* Kc_l, bf16_t* Kp, bf16_t* Vp,
                              float* Kc_p, int32_t* p_len, int64_t* p_id, float* S_sum, int32_t* S_cnt,
                              const bf16_t* Kl, const bf16_t* Vl, const int32_t* l_len, const int32_t* l_map,
                              const int64_t* l_id, float* scores, int32_t* slot_src, const UpdateWs& ws,
                              hipStream_t stream) {
  hipError_t e = launch_retain(p, Mt, p.C + 1 + p.n_loc, 1, Kc_l, Kc_p, p_len, p_id, S_cnt, S_sum != nullptr, l_len, l_map,
                               l_id, scores, slot_src, ws, stream);
  if (e != hipSuccess) return e;
  return launch_update_apply(p, Kp, Vp, p_len, S_sum, S_cnt, Kl, Vl, ws, stream);
}

}  // namespace pbsa

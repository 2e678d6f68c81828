// Paged K/V append and prefix-cached paged prefill attention for gfx950.
//
// InferLog (arXiv 2507.08523) section 2.1.2: with prefix caching only the
// cache-missing suffix of a prompt is prefilled; its queries attend to the
// reused KV of the cached prefix plus their own freshly stored KV (section
// 3.2.2).  This file holds the two device steps of that path:
//
//  * kv_append: scatter new K/V rows into 16-token pool blocks.  K blocks are
//    token-major [16][D]; V blocks are stored dimension-major [D][16] so the
//    attention kernel can feed them to the matrix cores without a transpose.
//  * paged_attn: causal grouped-query attention of the suffix queries.  A
//    work item is 128 query columns of one (request, kv head); a column is a
//    (token, q head of the group) pair, so the G heads of a group share every
//    K/V tile.  The kernel is persistent: two 4-wave workgroups per CU (three
//    at head size 64) take items by position and, the uneven rest, from
//    per-XCD counters.  64-key tiles (4 pool blocks) stream through two K and
//    two V buffers in LDS, filled by direct global-to-LDS loads issued a tile
//    step ahead of use.  Per tile and wave:
//      S^T = K Q^T   on v_mfma_f32_32x32x16_bf16 (a lane owns one column),
//      causal mask, online softmax in fp32 on exp2 with the scale folded in:
//      the exponentials are taken against the running column max, and the
//      tile's column max is computed (and O rescaled) only when a lane's sum
//      of them leaves [0, 2^8] -- on an item's first tile, or when the max
//      has grown by several powers of two --,
//      O^T += V^T P^T on the same MFMA, P taken straight from the S^T
//      accumulators (K rows are staged in a permuted order that makes the
//      accumulator layout of S^T equal the operand layout P^T needs).
//    What bounds it: on large batches the power limit (zeros for inputs run
//    25-30% faster, at the same instructions), on small ones the latency of an
//    item's start and the number of items in flight.  Large batches at head size
//    128 take a wide layout: one 8-wave workgroup per CU on 256-column items, its
//    halves a phase apart, which loads every K/V tile into LDS half as often.
//    For all others it has half as many items and workgroups to fill the chip
//    with.  Attention launch, an 8-wave layout of two barriers a tile, with its
//    items fetched one by one from contended counters, -> now: 20 scheduler steps of 1024 tokens (32/8 heads, 604 keys)
//    538 -> 474 us with their appends; 64 prompts of 300 new tokens, half
//    cached 210 -> 180 us; 128 prompts of 48 new tokens after 976 shared ones
//    120 -> 107 us; 199 prompts of 118 tokens (16/2 heads, D 64) 76 -> 40 us.
//    The wide layout, that one -> narrow -> now, us: 512 prompts of 64 new tokens
//    after 2048 own ones (64/8 heads) 2272 -> 2297 -> 2252; 128 of 1024 (32/8)
//    1296 -> 1309 -> 1245; 128 of 1984 after 128 (64/8) 8621 -> 8621 -> 8363.
//  * the same attention split at a prefix every request of the batch shares
//    (modes kShared / kSuffix: two launches; kFused: one launch whose items
//    are 128 columns of the whole batch, over the shared tiles and then each
//    of their requests' own tiles).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <climits>
#include <cstdint>
#include <type_traits>

#include "../../include/ilpc.h"
#include "ilpc_internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBlock = 16;                    // tokens per pool block
constexpr int kWaves = 4;                     // waves per attention workgroup (two workgroups per CU); wide: 8 (one)
constexpr int kColsPerWave = 32;              // query columns per wave (MFMA N)
constexpr int kCols = kColsPerWave * kWaves;  // query columns per workgroup
constexpr int kKeys = 64;                     // keys per tile
constexpr int kTileBlocks = kKeys / kBlock;
constexpr int kMaxGroup = 64;                 // largest Hq / Hkv accepted
constexpr int kDecodeCols = 32;               // query columns the decode kernel takes per request

// LDS row that holds tile key k.  Inside every 16 keys the groups [4,8) and
// [8,12) trade places, so that MFMA row m of S^T carries key sigma(m) and the
// fp32 accumulator registers of S^T line up with the bf16 operand of P^T:
// lane half h then holds keys 16c + 8h + 0..7 in registers 8c..8c+7.
__device__ __forceinline__ int key_row(int k) {
  const int grp = (k >> 2) & 3;
  return k + (grp == 1 ? 4 : (grp == 2 ? -4 : 0));
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

// 16-byte slot of chunk c in LDS K row m: XOR-swizzled so that the 16 lanes an
// LDS cycle serves (16 consecutive rows, one chunk each) hit distinct banks.
template <int D>
__device__ __forceinline__ int k_slot(int m, int c) {
  return D == 128 ? (c ^ (m & 15)) : (c ^ ((m >> 1) & 7));
}

// 16-byte half (keys 0-7 or 8-15) of V row d of a [D][16] block in LDS.
__device__ __forceinline__ int v_slot(int d, int hf) { return hf ^ ((d >> 2) & 1) ^ ((d >> 3) & 1); }

// One (block, kv head) slab of a pool straight into LDS: instruction i moves
// 16 bytes per lane from base + off[i] + i KiB (base wave-uniform) to
// lds + i KiB + 16 * lane; the linear form uses one offset for every
// instruction.  Issued as inline assembly so that the compiler does not track
// it: tracked, every LDS read would first wait for all such loads in flight,
// which defeats the prefetch.  Callers wait with an explicit vmcnt.  M0
// carries the LDS address; no other code in these kernels uses M0, so it is
// clobbered without being restored.  The immediate offset moves both
// addresses, so a slab takes one M0 write, and the scalar base takes no
// vector address arithmetic.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void load_slab4(uint32_t o0, uint32_t o1, uint32_t o2, uint32_t o3, uint64_t base,
                                           uint32_t lds) {
  asm volatile("s_mov_b32 m0, %5\n\ts_nop 0\n\t"
               "global_load_lds_dwordx4 %0, %4\n\t"
               "global_load_lds_dwordx4 %1, %4 offset:1024\n\t"
               "global_load_lds_dwordx4 %2, %4 offset:2048\n\t"
               "global_load_lds_dwordx4 %3, %4 offset:3072"
               :
               : "v"(o0), "v"(o1), "v"(o2), "v"(o3), "s"(base), "s"(lds)
               : "memory", "m0");
}
__device__ __forceinline__ void load_slab2(uint32_t o0, uint32_t o1, uint64_t base, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\t"
               "global_load_lds_dwordx4 %0, %2\n\t"
               "global_load_lds_dwordx4 %1, %2 offset:1024"
               :
               : "v"(o0), "v"(o1), "s"(base), "s"(lds)
               : "memory", "m0");
}
// Kept out of the kernel templates: an LDS address-space cast instantiated in
// their host-side pass would drop the launch stubs.
__device__ __forceinline__ uint32_t lds_offset(uint8_t* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((__attribute__((address_space(3))) uint8_t*)p));
}
#pragma clang diagnostic pop
// Both are wave-uniform; where the compiler cannot tell, this makes them scalar.
__device__ __forceinline__ uint32_t scalar(uint32_t x) { return __builtin_amdgcn_readfirstlane(x); }
__device__ __forceinline__ uint64_t scalar(uint64_t x) {
  return uint64_t(scalar(uint32_t(x >> 32))) << 32 | scalar(uint32_t(x));
}
// A word of a table no kernel writes meanwhile, at a wave-uniform address,
// through the scalar cache (as a load from constant memory): a vector load
// would queue behind the tile loads in flight, and its wait would wait for them.
__device__ __forceinline__ int32_t scalar_load(const int32_t* p) {
  return *(const __attribute__((address_space(4))) int32_t*)scalar(reinterpret_cast<uint64_t>(p));
}
template <int N>
__device__ __forceinline__ void load_slab(const uint32_t* off, uint64_t base, uint32_t lds) {
  base = scalar(base);
  lds = scalar(lds);
  if constexpr (N == 4) load_slab4(off[0], off[1], off[2], off[3], base, lds);
  else load_slab2(off[0], off[1], base, lds);
}
template <int N>
__device__ __forceinline__ void load_slab_linear(uint32_t off, uint64_t base, uint32_t lds) {
  base = scalar(base);
  lds = scalar(lds);
  if constexpr (N == 4) load_slab4(off, off, off, off, base, lds);
  else load_slab2(off, off, base, lds);
}

// max(x, x of the lane 32 apart): v_permlane32_swap exchanges the two wave halves.
__device__ __forceinline__ float max_across_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// ---------------------------------------------------------------------------
// kv_append: one workgroup per (logical block touched, kv head, request).
template <int D>
__global__ __launch_bounds__(256) void kv_append_kernel(
    const uint16_t* __restrict__ k_new, const uint16_t* __restrict__ v_new,
    uint16_t* __restrict__ k_pool, uint16_t* __restrict__ v_pool, int num_blocks,
    const int32_t* __restrict__ block_tables, int max_blocks, const int32_t* __restrict__ cu_new,
    const int32_t* __restrict__ start_pos, int max_new, int Hkv) {
  constexpr int kChunks = D / 8;  // 16-byte chunks per row
  __shared__ __attribute__((aligned(16))) uint16_t sv[kBlock][D + 8];
  const int r = blockIdx.z, h = blockIdx.y;
  const int row0 = cu_new[r];
  int n = cu_new[r + 1] - row0;
  if (n > max_new) n = max_new;
  const int start = start_pos[r];
  if (n <= 0 || start < 0) return;
  const int lb = start / kBlock + int(blockIdx.x);
  const int p0 = max(start, lb * kBlock), p1 = min(start + n, (lb + 1) * kBlock);
  if (p0 >= p1 || lb >= max_blocks) return;
  const int phys = block_tables[size_t(r) * max_blocks + lb];
  if (phys < 0 || phys >= num_blocks) return;
  const int tid = threadIdx.x;
  const size_t kblk = (size_t(phys) * Hkv + h) * kBlock * D;  // same offset for K and V blocks

  for (int idx = tid; idx < kBlock * kChunks; idx += 256) {
    const int slot = idx / kChunks, c = idx % kChunks;
    const int p = lb * kBlock + slot;
    if (p >= p0 && p < p1) {
      const size_t src = (size_t(row0 + p - start) * Hkv + h) * D + c * 8;
      *(u32x4*)(k_pool + kblk + size_t(slot) * D + c * 8) = *(const u32x4*)(k_new + src);
      *(u32x4*)(&sv[slot][c * 8]) = *(const u32x4*)(v_new + src);
    }
  }
  __syncthreads();
  for (int idx = tid; idx < 2 * D; idx += 256) {
    const int d = idx >> 1, hf = idx & 1;
    const int pb = lb * kBlock + hf * 8;
    uint16_t* dst = v_pool + kblk + size_t(d) * kBlock + hf * 8;
    if (pb >= p0 && pb + 8 <= p1) {
      u32x4 w;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        w[e] = uint32_t(sv[hf * 8 + 2 * e][d]) | (uint32_t(sv[hf * 8 + 2 * e + 1][d]) << 16);
      *(u32x4*)dst = w;
    } else {
      for (int e = 0; e < 8; ++e) {
        const int p = pb + e;
        if (p >= p0 && p < p1) dst[e] = sv[hf * 8 + e][d];
      }
    }
  }
}

// ---------------------------------------------------------------------------
// paged attention.  Work items are (column tile, kv head, request) triples,
// numbered request-major with the heaviest column tile of a (request, kv head)
// first.  The kernel is persistent: two workgroups per CU take items from
// eight queues, one per XCD, each holding whole runs of item numbers
// so that the items sharing one (request, kv head) -- and so the same K/V
// blocks -- are worked on under one XCD's L2.  The queue counters live in the
// caller's workspace and are zero again when a launch ends (the hand-out is
// described in the kernel).
constexpr int kMaxTableBlocks = 1 << 24;  // block-table width accepted (keeps token positions in int)
// Largest per-lane sum of a tile's exponentials accepted without taking the
// tile's column max (each exponential is then at most this, 2^8).
constexpr float kSumLimit = 256.f;
constexpr int kQueueWords = 16;  // workspace: 8 queue counters, finished workgroups, drained queues
constexpr int kDoneWord = 8;
constexpr int kDrainedWord = 9;
constexpr unsigned kLongRounds = 16;
constexpr int kWideRounds = 8;  // items of the wide layout to a CU from which it runs
constexpr int kIndex = 2048;  // COUNTED: groups of requests, and one
constexpr unsigned kNoItem = ~0u, kAsk = ~0u - 1u;

// s_waitcnt vmcnt(n) with the other counters left free (n < 16).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  static_assert(N >= 0 && N < 16, "vmcnt immediate");
  __builtin_amdgcn_s_waitcnt(0x0F70 | N);
}

// s_waitcnt lgkmcnt(0) with the other counters left free.
__device__ __forceinline__ void wait_lgkmcnt0() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// Workgroup barrier without the memory fence of __syncthreads: the caller
// has already waited for exactly the loads it needs.  The empty asm keeps the
// compiler from moving memory accesses across it.
__device__ __forceinline__ void bare_barrier() {
  asm volatile("" ::: "memory");
  __builtin_amdgcn_s_barrier();
  asm volatile("" ::: "memory");
}

// What one launch of the attention kernel computes.
//   kFull:   each request's queries over all of its keys (causal).
//   kShared: first half of a split over a prefix of kv_split keys that every
//            request shares (same blocks, all before any query): every query
//            row of the batch over keys [0, kv_split) of request 0's table, no
//            mask; the unnormalised O, the running max and the sum go to
//            part_o / part_ml instead of out.
//   kSuffix: second half: each request's queries over keys [kv_split, L)
//            (causal), starting from the state kShared left, normalised into out.
// Splitting this way reads the shared K/V once per column tile of the whole
// batch instead of once per request (the log-sum-exp merge of the two halves
// is exact up to rounding).
//   kFused:  the same split in one launch: every item is 128 columns of the
//            whole batch's packed query rows (like kShared); it runs the
//            kv_split / 64 tiles every request shares, then, for each
//            request its rows belong to, that request's own tiles from
//            kv_split on, masked to that request's columns (a wave none of
//            whose columns belong to the request skips the tile).  No partial
//            state leaves the workgroup.
enum AttnMode { kFull = 0, kShared = 1, kSuffix = 2, kFused = 3 };

// kFused: per item, the request tiles after the shared ones, and the requests
// with rows in the item (at most 128 of them, one per column), in LDS.
constexpr int kFusedTiles = 2048;
constexpr int kFusedReqs = kCols + 4;

// Workgroups per CU: at D = 128 the registers hold two waves per SIMD, at
// D = 64 three.
constexpr int wgs_per_cu(int D) { return D == 64 ? 3 : 2; }

template <int D, int MODE, bool COUNTED, int WAVES>
__global__ __launch_bounds__(64 * WAVES, wgs_per_cu(D)) void paged_attn_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_pool,
    const uint16_t* __restrict__ v_pool, int num_blocks, const int32_t* __restrict__ block_tables,
    int max_blocks, const int32_t* __restrict__ cu_q, const int32_t* __restrict__ seq_lens, int n_req,
    int Hq, int Hkv, int n_col_tiles, unsigned n_items, unsigned chunk, int count_shift, float scale_log2,
    uint16_t* __restrict__ out, unsigned* __restrict__ queue, int kv_split, float* __restrict__ part_o,
    float* __restrict__ part_ml, int part_rows) {
  constexpr int kDch = D / 16;                    // 16-wide contraction chunks of Q.K^T
  constexpr int kDt = D / 32;                     // 32-row output tiles of O^T
  constexpr int kRowBytes = D * 2;                // one K row in LDS
  constexpr int kKch = D / 8;                     // 16-byte chunks per K row
  constexpr int kSlabBytes = kBlock * D * 2;      // one (block, kv head) slab: in a pool, and in LDS
  constexpr int kTileBytes = kTileBlocks * kSlabBytes;  // one K tile, or one V tile
  constexpr int kInsts = kSlabBytes / 1024;       // 1 KB direct loads of a slab
  constexpr int kThreads = 64 * WAVES, kCols = kColsPerWave * WAVES;
  constexpr bool kWide = WAVES == 2 * kTileBlocks;
  static_assert(kWide || WAVES == kTileBlocks, "a wave loads the K and the V of a pool block, or (kWide) one of them");
  // K tiles, then as many V tiles.
  constexpr int kBufs = kWide ? 3 : 2;
  __shared__ __attribute__((aligned(16))) uint8_t ring[2 * kBufs * kTileBytes];
  __shared__ unsigned s_item;
  // kFused: tile T_s + i of an item is tile f_tile[i] & 0xFFFFFF of the item's
  // request number f_tile[i] >> 24, which is request f_req[.], whose keys at
  // or past f_lim[.] no row of the item sees.
  constexpr bool kIsFused = MODE == kFused;
  __shared__ uint32_t f_tile[kIsFused ? kFusedTiles : 1];
  __shared__ int f_req[kIsFused ? kFusedReqs : 1], f_lim[kIsFused ? kFusedReqs : 1];
  __shared__ int f_count;
  constexpr bool kWholeBatch = MODE == kShared || MODE == kFused;  // items are columns of the whole batch
  // COUNTED: column tiles (of one kv head) before each group of 2^count_shift
  // requests, and behind the last one.
  static_assert(!(COUNTED && kWholeBatch), "those modes know their rows");
  __shared__ unsigned first_tile[COUNTED ? kIndex : 1];
  __shared__ unsigned s_sums[COUNTED ? WAVES : 1];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);  // wave-uniform
  const int n = lane & 31, hh = lane >> 5;
  const int blk = kWide ? wave & (kTileBlocks - 1) : wave;  // pool block of a tile this wave loads
  const bool lag = kWide && wave >= kTileBlocks;            // (kWide) the half that runs a phase behind, and loads V
  const int G = Hq / Hkv;
  const size_t slab_stride = size_t(Hkv) * kSlabBytes;

  // Two layouts, one of which runs: the wide one from part_rows rows on (kFull;
  // 0: only one is launched).
  if constexpr (MODE == kFull && COUNTED) {
    if (part_rows > 0 && (scalar_load(cu_q + n_req) >= part_rows) != kWide) return;
  }
  // The host sizes a launch by max_q_len.  With many numbers (count_shift >= 0)
  // the kernel first counts the column tiles there are, and numbers only those:
  // a batch with one long request among many short ones is nearly all empty
  // numbers otherwise, each of them an atomic on the shared counters.  us, one
  // by one (in the 8-wave layout, half as many) -> counted, 32/8 heads: 64
  // requests of 1 row but one of 4000 890 (546) -> 188, 256 and one of 2000 1537
  // (795) -> 102, 128 of 16 and one of 1000 445 (237) -> 59; where all hold work
  // the count costs 1 to 2 us (128 prompts of 1024 rows 1290 -> 1301).
  int n_groups = 0;
  auto tiles_of = [&](int r) -> unsigned {  // column tiles of request r
    int a = cu_q[r], b = cu_q[r + 1];
    if constexpr (MODE == kSuffix) b = min(b, part_rows);
    return b <= a ? 0u : unsigned(min((int64_t(b - a) * G + (kCols - 1)) / kCols, int64_t(n_col_tiles)));
  };
  if constexpr (COUNTED) {
    // every thread a run of groups; then a sum over the threads before it
    n_groups = (n_req + (1 << count_shift) - 1) >> count_shift;
    const int per = (n_groups + kThreads - 1) / kThreads;
    const int g0 = min(tid * per, n_groups), g1 = min(g0 + per, n_groups);
    unsigned mine = 0;
    for (int g = g0; g < g1; ++g) {
      unsigned t = 0;
      for (int r = g << count_shift; r < min((g + 1) << count_shift, n_req); ++r) t += tiles_of(r);
      first_tile[g] = t;
      mine += t;
    }
    unsigned sum = mine;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const unsigned v = __shfl_up(sum, off);
      sum += lane >= off ? v : 0u;
    }
    if (lane == 63) s_sums[wave] = sum;
    __syncthreads();
    unsigned before = sum - mine;
    for (int i = 0; i < wave; ++i) before += s_sums[i];
    for (int g = g0; g < g1; ++g) {
      const unsigned t = first_tile[g];
      first_tile[g] = before;
      before += t;
    }
    if (tid == kThreads - 1) first_tile[n_groups] = before;
    __syncthreads();
    n_items = __builtin_amdgcn_readfirstlane(first_tile[n_groups]) * unsigned(Hkv);
  } else if (kWholeBatch && count_shift >= 0) {
    int rows = scalar_load(cu_q + n_req);
    if constexpr (MODE == kShared) rows = min(rows, part_rows);
    n_col_tiles = int(min((int64_t(max(rows, 0)) * G + (kCols - 1)) / kCols, int64_t(n_col_tiles)));
    n_items = unsigned(n_col_tiles) * unsigned(Hkv);
  }
  if ((COUNTED || kWholeBatch) && count_shift >= 0) {
    if (n_items == 0) return;
    // (odd: a run of equal pairs must not put the same part of each into one queue)
    chunk = n_items >= kLongRounds * gridDim.x ? (n_items + 7u) / 8u : max(n_items / 256u, 1u) | 1u;
  }

  // Hand-out of the items.  Item numbers are cut into chunks of `chunk`; queue
  // x (one per XCD) holds the chunks x, x + 8, ..., and is worked by the
  // workgroups b = x (mod 8), which round-robin dispatch puts on XCD x.
  //   Short launches (under kLongRounds items a workgroup): the i-th of a
  // queue's W workgroups first takes items by position: i, 2W-1-i, 2W+i,
  // 4W-1-i, ... of the queue (turning round so that the heavy-first runs of a
  // (request, kv head) average out), for three quarters of the rounds; the
  // rest goes through the queue's counter, which levels uneven items.  The
  // eight counters share one cache line of the workspace, at 20-25 ns an
  // atomic for the whole chip: that is why only a quarter of the items pass
  // through them, and why no workgroup looks at another queue or counts itself
  // out: each asks its own counter once too often, and the one that gets the
  // last such number leaves the counter zero for the next call.
  //   Long launches: everything after the first round goes through the
  // counters (the XCDs do not run at one speed: leaving each its own eighth
  // cost 2-3% on 128 prompts of 1984 new tokens, 64/8 heads), and a workgroup
  // whose queue is drained helps the others.  The workgroup that takes the
  // last item of a queue counts it in queue[kDrainedWord]; that count (one
  // round trip) tells whether any queue still holds items, without a walk over
  // the drained queues.  The last workgroup to finish clears the counters.
  const unsigned s_x = blockIdx.x & 7u;
  const bool stealing = n_items >= kLongRounds * gridDim.x;
  auto queue_wgs = [&](unsigned x) { return (gridDim.x + 7u - x) >> 3; };
  auto queue_size = [&](unsigned x) {
    const unsigned nch = (n_items + chunk - 1u) / chunk, mine = (nch + 7u - x) >> 3;
    return mine * chunk - (((nch - 1u) & 7u) == x ? nch * chunk - n_items : 0u);
  };
  auto item_at = [&](unsigned x, unsigned p) { return ((p / chunk) * 8u + x) * chunk + p % chunk; };

  // This wave's direct loads of a tile: pool block `wave` of the tile, i.e.
  // its own quarter of a K tile and of a V tile.  LDS slot (row m, slot p) of
  // a K tile holds chunk k_slot(m, p) of key key_row(m); slot (d, p) of a V
  // block holds half v_slot(d, p) of row d.  Instruction i of a slab carries
  // an immediate offset of i KiB that moves its source and its destination
  // alike; koff takes the source's share back out (+1 KiB so that it stays
  // positive: the base passed is 1 KiB lower).  The V source moves by exactly
  // that, so one offset serves all its instructions.
  uint32_t koff[kInsts];
#pragma unroll
  for (int i = 0; i < kInsts; ++i) {
    const int m = i * (1024 / kRowBytes) + lane / kKch;
    koff[i] = uint32_t(key_row(m) * kRowBytes + k_slot<D>(m, lane % kKch) * 16 + 1024 - i * 1024);
  }
  const uint32_t voff = uint32_t((lane >> 1) * 32 + v_slot(lane >> 1, lane & 1) * 16);
  const uint32_t ring0 = lds_offset(ring) + blk * kSlabBytes;  // this wave's quarter of K tile 0

  // By position: this workgroup's next place in its queue, the end of that
  // part, the step to the place after; then what is left for the counter.
  const unsigned s_wgs = queue_wgs(s_x), s_size = queue_size(s_x);
  const unsigned s_rounds = s_size / s_wgs;
  const unsigned s_end =
      s_rounds <= 1u ? min(s_size, s_wgs) : stealing ? s_wgs : (s_rounds - s_rounds / 4u) * s_wgs;
  const unsigned s_left = s_size - s_end;
  unsigned s_next = blockIdx.x >> 3, s_step = 2u * s_wgs - 1u - 2u * (blockIdx.x >> 3);
  // The item to start next; kAsk: it is to be asked for.
  auto next_static = [&]() -> unsigned {
    const unsigned at = s_next;
    s_next += s_step;
    s_step = 2u * s_wgs - s_step;
    return at < s_end ? item_at(s_x, at) : (s_left ? kAsk : kNoItem);
  };
  // Lane 0 of wave 0 only: asks a counter; the item behind its answer.
  unsigned qsel = 0;  // (stealing) next queue to try, home first
  auto take = [&]() {
    return __hip_atomic_fetch_add(queue + ((s_x + qsel) & 7u), 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  };
  auto resolve = [&](unsigned i) -> unsigned {
    if (!stealing) {
      if (i < s_left) return item_at(s_x, s_end + i);
      if (i == s_left + s_wgs - 1u) __hip_atomic_store(queue + s_x, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      return kNoItem;
    }
    while (qsel < 8u) {
      const unsigned x = (s_x + qsel) & 7u, first = queue_wgs(x), left = queue_size(x) - first;
      if (i + 1 == left) __hip_atomic_fetch_add(queue + kDrainedWord, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (i < left) return item_at(x, first + i);
      ++qsel;
      if (qsel == 1u &&
          __hip_atomic_load(queue + kDrainedWord, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= 8u)
        qsel = 8u;
      if (qsel < 8u) i = take();
    }
    return kNoItem;
  };
  unsigned w = next_static();

  // Columns are split into (query row, head of the group) by a 16-bit
  // reciprocal of G: exact for the offsets met here, below G + kCols <= 320
  // (u * (65536 / G + 1 - 65536 / G exactly) < u * G / 65536 < 1 / G).
  const unsigned recip = 65536u / unsigned(G) + 1u;
  auto div_g = [&](int u) { return int((unsigned(u) * recip) >> 16); };

  // State of the item whose loads were last started ...
  int kvh = 0, row0 = 0, rem0 = 0;  // kv head; query row and head of its first column
  int n_valid = 0;                  // its query columns (up to kCols)
  int n_tiles = 0, key_lim = 0, n_blk_used = 0, wave_last = -1, wave_pos_min = 0, t0 = 0;
  int pos = 0, my_ord = 0, my_pos = 0;  // of this lane's column
  bool wave_active = false;
  const int32_t* bt = block_tables;
  int c_r = 0;                       // COUNTED: the item's request (the next one's, mostly),
  unsigned c_base = 0, c_tiles = 0;  // the column tiles before it, and its own
  int id_next = 0, raw_next = 0;  // block id of the next tile to issue V of, raw id of the one after
  const int T_s = kv_split / kKeys;  // kFused: tiles every request shares (at least 3)
  const uint64_t kbase0 = reinterpret_cast<uint64_t>(k_pool) - 1024, vbase0 = reinterpret_cast<uint64_t>(v_pool);
  // The two K and the two V buffers alternate by a tile count that runs on
  // across items, so that the first loads of an item never land in the V tile
  // a slower wave of the previous item still reads.
  int tbase = 0;
  bf16x8 qf[kDch];           // Q operand of this wave's 32 columns
  f32x16 o[kDt];             // unnormalised O^T
  float m_used = -INFINITY;  // max (log2 units) the exponentials of this column are taken against
  float l_run = 0.f;         // this lane half's share of the column's exponential sum
  bf16x8 pb[kTileBlocks];    // P of the tile whose V^T P^T is still due
  f32x16 sc0, sc1;           // scores of the tile whose softmax is next
  // Defined here, as whatever the registers hold (an undefined value would be
  // carried in registers of its own, 48 of them across the tile loop).
  asm volatile("" : "=v"(sc0), "=v"(sc1), "=v"(pb[0]), "=v"(pb[1]), "=v"(pb[2]), "=v"(pb[3]));
#pragma unroll
  for (int i = 0; i < kDch; ++i) asm volatile("" : "=v"(qf[i]));
#pragma unroll
  for (int i = 0; i < kDt; ++i) asm volatile("" : "=v"(o[i]));

  auto raw_id = [&](int tl) { return scalar_load(bt + min((t0 + tl) * kTileBlocks + blk, max_blocks - 1)); };
  // Pool block of this wave in tile tl, from the raw table entry; unusable
  // ids read block 0 instead (stray K rows only meet masked scores, stray V
  // rows past key_lim are zeroed below).
  auto usable = [&](int tl, int id) {
    if constexpr (kIsFused) return (id >= 0 && id < num_blocks) ? id : 0;
    return ((t0 + tl) * kTileBlocks + blk < n_blk_used && id >= 0 && id < num_blocks) ? id : 0;
  };
  auto buf = [&](int tl) { return (unsigned(tbase + tl) % unsigned(kBufs)) * kTileBytes; };
  auto slab_at = [&](int id) { return size_t(id) * slab_stride + size_t(kvh) * kSlabBytes; };
  auto issue_k = [&](int tl, int id) { load_slab<kInsts>(koff, kbase0 + slab_at(id), ring0 + buf(tl)); };
  auto issue_v = [&](int tl, int id) {
    load_slab_linear<kInsts>(voff, vbase0 + slab_at(id), ring0 + kBufs * kTileBytes + buf(tl));
  };
  auto k_at = [&](int tl) { return ring + buf(tl); };
  auto v_at = [&](int tl) { return ring + kBufs * kTileBytes + buf(tl); };
  // Element offset in q / out of the row of column offset co of an item.
  auto row_of = [&](int r0, int m0, int h, int co) {
    const int u = m0 + co, t = div_g(u);
    return (size_t(r0 + t) * Hq + size_t(h) * G + (u - t * G)) * D;
  };

  // Starts item w: reads its lengths and first block ids, issues the loads of
  // its K tiles 0 and 1, V tile 0 and Q.  False, with nothing issued, if the
  // item holds no query columns.
  auto start_item = [&]() -> bool {
    w = __builtin_amdgcn_readfirstlane(w);
    // kFused numbers items kv-head-major (the items of one kv head share the
    // prefix blocks, under one XCD's L2).
    int tile, r = 0;
    if constexpr (COUNTED) {
      // The last group that starts at or before tile w / Hkv: every 32nd first,
      // then the 32 behind it.
      const unsigned at = w / unsigned(Hkv);
      constexpr int kStride = kIndex / 64;
      if (at - c_base >= c_tiles) {
        const int blk = __popcll(__ballot(first_tile[min(lane * kStride, n_groups)] <= at)) - 1;
        const bool here = lane < kStride && first_tile[min(blk * kStride + lane, n_groups)] <= at;
        const int g = blk * kStride + __popcll(__ballot(here)) - 1;
        c_r = g << count_shift;
        c_base = __builtin_amdgcn_readfirstlane(first_tile[g]);
        c_tiles = __builtin_amdgcn_readfirstlane(first_tile[g + 1]) - c_base;
        if (count_shift > 0) {  // which of the group's requests (at most 64)
          const bool in = lane < (1 << count_shift) && c_r + lane < n_req;
          const unsigned t = in ? tiles_of(c_r + lane) : 0u;
          unsigned sum = t;
#pragma unroll
          for (int off = 1; off < 64; off <<= 1) {
            const unsigned v = __shfl_up(sum, off);
            sum += lane >= off ? v : 0u;
          }
          const int l = __popcll(__ballot(c_base + sum <= at));  // requests that end at or before it
          c_tiles = __builtin_amdgcn_readlane(t, l);
          c_base += __builtin_amdgcn_readlane(sum, l) - c_tiles;
          c_r += l;
        }
      }
      r = c_r;
      const unsigned in_r = w - c_base * unsigned(Hkv);
      kvh = int(in_r / c_tiles);
      tile = int(c_tiles - 1u - in_r % c_tiles);
    } else {
      tile = kIsFused ? int(w % unsigned(n_col_tiles)) : n_col_tiles - 1 - int(w % unsigned(n_col_tiles));
      const unsigned rest = w / unsigned(n_col_tiles);
      kvh = kIsFused ? int(rest) : int(rest % unsigned(Hkv));
      if (!kWholeBatch) r = int(rest / unsigned(Hkv));
    }
    // First key tile of this launch (the suffix half starts at kv_split).
    t0 = MODE == kSuffix ? kv_split / kKeys : 0;
    // This item's lengths and the block ids of its first three tiles are
    // loaded together: one round trip for all.  A block id is loaded
    // unconditionally (clamped into the table row) and checked where it is
    // used, so that no wait follows the scalar load.
    bt = block_tables + size_t(r) * max_blocks;
    // The shared half treats the whole batch as one request whose queries all
    // follow the kv_split shared keys.
    const int q0 = MODE == kShared || kIsFused ? 0 : scalar_load(cu_q + r);
    const int q_end = scalar_load(MODE == kShared || kIsFused ? cu_q + n_req : cu_q + r + 1);
    const int L_in = MODE == kShared || kIsFused ? kv_split + (q_end - q0) : scalar_load(seq_lens + r);
    const int raw_id0 = raw_id(0), raw_id1 = raw_id(1);
    raw_next = raw_id(2);
    // First use of all six values at once: the loads are issued together and
    // waited for once.
    asm volatile("" : : "s"(q0), "s"(q_end), "s"(L_in), "s"(raw_id0), "s"(raw_id1), "s"(raw_next));
    // In the split modes, rows past the partial-state buffer are not computed.
    const int q_len = MODE == kFull || kIsFused ? q_end - q0 : min(q_end, part_rows) - q0;
    const int n_cols = q_len * G;
    const int col0 = tile * kCols;
    const int L = MODE == kShared || kIsFused ? L_in : min(L_in, max_blocks * kBlock);
    if (q_len <= 0 || col0 >= n_cols || q_len > L) return false;
    const int qstart = L - q_len;  // position of the request's first query
    const int row_a = col0 / G;
    row0 = q0 + row_a;
    rem0 = col0 - row_a * G;
    n_valid = min(n_cols - col0, kCols);
    const int wave_first = wave * kColsPerWave;
    wave_active = wave_first < n_valid;
    // This lane's query column (padding columns repeat the last valid one).
    const int co = min(wave_first + n, n_valid - 1);
    const int pos0 = qstart + row_a;
    pos = MODE == kShared ? kv_split - 1 : pos0 + div_g(rem0 + co);
    wave_pos_min = MODE == kShared ? kv_split - 1 : pos0 + div_g(rem0 + min(wave_first, n_valid - 1));
    const int wg_pos_max = pos0 + div_g(rem0 + n_valid - 1);
    // Keys at or past key_lim are masked everywhere (and their V rows zeroed).
    key_lim = MODE == kShared ? kv_split : wg_pos_max + 1;
    // Tiles of this launch (kFused: the shared ones until the item's list is
    // read after the next barrier).
    // (at least one, also where the caller's shared_len breaks its contract)
    n_tiles = kIsFused ? T_s : max((key_lim - 1) / kKeys + 1 - t0, 1);
    n_blk_used = (key_lim + kBlock - 1) / kBlock;  // <= ceil(L / 16) <= max_blocks
    // Last tile (counted from t0) holding a key some column of this wave sees
    // (-1: no column).
    wave_last = !wave_active ? -1
                : MODE == kShared
                    ? n_tiles - 1
                    : (pos0 + div_g(rem0 + min(wave_first + kColsPerWave, n_valid) - 1)) / kKeys - t0;
    const int id0 = usable(0, raw_id0);
    id_next = usable(1, raw_id1);
    if (!lag) {
      issue_k(0, id0);
      issue_v(0, id0);
      if (1 < n_tiles) issue_k(1, id_next);
    }
    const size_t qrow = row_of(row0, rem0, kvh, co);
#pragma unroll
    for (int kc = 0; kc < kDch; ++kc) qf[kc] = as_bf16x8(*(const u32x4*)(q + qrow + kc * 16 + hh * 8));
    // kFused: with the first tiles and Q in flight, find the requests of the
    // item's rows, this lane's request and position, and (wave 0) the list of
    // request tiles; tiles 0-2 are shared, so request 0's table gave their ids.
    // Scalar loads only: they do not queue behind the tiles' vector loads.
    if constexpr (kIsFused) {
      const int row_b = row_a + div_g(rem0 + n_valid - 1);
      // lo: the largest request whose first row is at or before row_a; seven
      // probes a round trip
      int lo = 0, hi = n_req;  // cu_q[lo] <= row_a < cu_q[hi]
      while (hi - lo > 1) {
        const int st = (hi - lo + 7) >> 3;
        int c[7], next = lo;
#pragma unroll
        for (int k = 0; k < 7; ++k) c[k] = scalar_load(cu_q + min(lo + st * (k + 1), hi));
#pragma unroll
        for (int k = 0; k < 7; ++k)
          if (lo + st * (k + 1) < hi && c[k] <= row_a) next = lo + st * (k + 1);
        hi = min(next + st, hi);
        lo = next;
      }
      const int row_l = row_a + div_g(rem0 + co);
      int n_list = 0, ord = 0;
      my_ord = 0;
      my_pos = 0;
      // requests lo, lo + 1, ... while their rows start at or before row_b
      for (int rr = lo; rr < n_req && ord < kFusedReqs; ++rr) {
        const int b0 = scalar_load(cu_q + rr);
        if (b0 > row_b) break;
        const int b1 = scalar_load(cu_q + rr + 1);
        const int lo_row = max(b0, row_a), hi_row = min(b1 - 1, row_b);
        if (lo_row > hi_row) continue;  // no row of this item (or an empty request)
        const int Lr = min(scalar_load(seq_lens + rr), max_blocks * kBlock);
        if (row_l >= b0 && row_l < b1) {
          my_ord = ord;
          my_pos = Lr - (b1 - b0) + (row_l - b0);
        }
        // keys the item's rows of rr see end at lim; its tiles T_s .. go to the list
        const int lim = Lr - (b1 - b0) + (hi_row - b0) + 1;
        const int cnt = min(max(0, (lim + kKeys - 1) / kKeys - T_s), kFusedTiles - n_list);
        if (wave == 0) {
          for (int k = lane; k < cnt; k += 64) f_tile[n_list + k] = uint32_t(ord) << 24 | uint32_t(T_s + k);
          if (lane == 0) {
            f_req[ord] = rr;
            f_lim[ord] = lim;
          }
        }
        n_list += cnt;
        ++ord;
      }
      if (wave == 0) {
        if (lane == 0) f_count = n_list;
        wait_lgkmcnt0();  // the list is in LDS before the next barrier
      }
    }
    return true;
  };

  // Zero the V rows of keys >= lim in this wave's pool block of a V tile
  // starting at key j0 (the wave's own loads of it have landed; the other
  // waves read it only after the next barrier).
  auto zero_v_tail = [&](int tl, int j0, int lim) {
    const int nv_blk = lim - (j0 + blk * kBlock);
    if (nv_blk >= kBlock) return;
    uint8_t* sV = v_at(tl) + blk * kSlabBytes;
    const int nvalid = nv_blk - v_slot(lane >> 1, lane & 1) * 8;
#pragma unroll
    for (int i = 0; i < kInsts; ++i) {
      u32x4* ptr = (u32x4*)(sV + i * 1024 + lane * 16);
      u32x4 v = *ptr;
#pragma unroll
      for (int e = 0; e < 4; ++e)
        v[e] &= (2 * e < nvalid ? 0x0000FFFFu : 0u) | (2 * e + 1 < nvalid ? 0xFFFF0000u : 0u);
      *ptr = v;
    }
    wait_lgkmcnt0();
  };

  // Masks of the score tile starting at key j0 (scores of keys a column does
  // not see become -inf).  Lane half hh holds keys j0 + (e>>3)*16 + 8*hh +
  // (e&7) [+32] of the tile.
  auto mask = [&](int j0, int fused_thr) __attribute__((always_inline)) {
    auto keep_upto = [&](int rel) __attribute__((always_inline)) {  // key (e>>3)*16 + (e&7) [+32] is visible iff <= rel
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int k = (e >> 3) * 16 + (e & 7);
        sc0[e] = k > rel ? -INFINITY : sc0[e];
        sc1[e] = k + 32 > rel ? -INFINITY : sc1[e];
      }
    };
    if (kIsFused && fused_thr != INT_MAX) keep_upto(fused_thr);  // a request tile: its own rows, causal
    if (!kIsFused && j0 + kKeys - 1 > wave_pos_min) keep_upto(pos - j0 - hh * 8);  // causal (kShared: pos is its last key)
    if (MODE == kSuffix && j0 < kv_split) {  // keys of the shared prefix: done before
      int lo = kv_split - j0 - hh * 8;
      asm volatile("" : "+v"(lo));  // as above
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const int k = (e >> 3) * 16 + (e & 7);
        sc0[e] = k < lo ? -INFINITY : sc0[e];
        sc1[e] = k + 32 < lo ? -INFINITY : sc1[e];
      }
    }
  };

  // Softmax step of a masked score tile: P = exp2(S * scale_log2 - m_used),
  // rounded to bf16 for the V^T P^T product while the row sum adds the fp32
  // values.  m_used is the column max the exponentials were last rescaled to.
  // The step is accepted as long as every lane's sum of its exponentials lies
  // in [0, 2^8] (so no single one exceeds 2^8, the headroom the fp32
  // accumulators are given); otherwise -- on the first tile (`first`: m_used
  // is still -inf), or when the max has grown -- the tile's column max is
  // taken, O and the sum are rescaled to it and the exponentials recomputed.
  auto softmax = [&](bool first) __attribute__((always_inline)) {
    // Exponentials against the running max m_used, summed per lane half.
    auto exps = [&](float* ls) {
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        const float p0 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc0[e], scale_log2, -m_used));
        const float p1 = __builtin_amdgcn_exp2f(__builtin_fmaf(sc1[e], scale_log2, -m_used));
        pb[e >> 3][e & 7] = (__bf16)p0;
        pb[2 + (e >> 3)][e & 7] = (__bf16)p1;
        ls[e & 3] = e < 4 ? p0 + p1 : ls[e & 3] + (p0 + p1);
      }
      // The bf16 operands are formed here, not after the acceptance test:
      // sunk past it, all 32 fp32 exponentials would stay live across it.
      asm volatile("" : "+v"(pb[0]), "+v"(pb[1]), "+v"(pb[2]), "+v"(pb[3]));
    };
    float ls[4];
    float tsum = 0.f;
    bool slow = first;
    if (!first) {
      exps(ls);
      tsum = (ls[0] + ls[1]) + (ls[2] + ls[3]);
      // Accepted unless some lane's sum exceeds kSumLimit or is not a
      // number (an overflow, or -inf - -inf).
      slow = __ballot(!(tsum <= kSumLimit)) != 0;
    }
    if (slow) {
      float mx, mx2;
      asm("v_max3_f32 %0, %1, %2, %3\n\t"
          "v_max3_f32 %0, %0, %4, %5\n\t"
          "v_max3_f32 %0, %0, %6, %7\n\t"
          "v_max3_f32 %0, %0, %8, %9\n\t"
          "v_max3_f32 %0, %0, %10, %11\n\t"
          "v_max3_f32 %0, %0, %12, %13\n\t"
          "v_max3_f32 %0, %0, %14, %15\n\t"
          "v_max3_f32 %0, %0, %16, %17"
          : "=&v"(mx)
          : "v"(sc0[0]), "v"(sc1[0]), "v"(sc0[1]), "v"(sc1[1]), "v"(sc0[2]), "v"(sc1[2]), "v"(sc0[3]),
            "v"(sc1[3]), "v"(sc0[4]), "v"(sc1[4]), "v"(sc0[5]), "v"(sc1[5]), "v"(sc0[6]), "v"(sc1[6]),
            "v"(sc0[7]), "v"(sc1[7]), "v"(sc0[8]));
      asm("v_max3_f32 %0, %1, %2, %3\n\t"
          "v_max3_f32 %0, %0, %4, %5\n\t"
          "v_max3_f32 %0, %0, %6, %7\n\t"
          "v_max3_f32 %0, %0, %8, %9\n\t"
          "v_max3_f32 %0, %0, %10, %11\n\t"
          "v_max3_f32 %0, %0, %12, %13\n\t"
          "v_max3_f32 %0, %0, %14, %15\n\t"
          "v_max3_f32 %0, %0, %16, %0"
          : "=&v"(mx2)
          : "v"(mx), "v"(sc1[8]), "v"(sc0[9]), "v"(sc1[9]), "v"(sc0[10]), "v"(sc1[10]), "v"(sc0[11]),
            "v"(sc1[11]), "v"(sc0[12]), "v"(sc1[12]), "v"(sc0[13]), "v"(sc1[13]), "v"(sc0[14]),
            "v"(sc1[14]), "v"(sc0[15]), "v"(sc1[15]));
      mx = mx2;
      mx = max_across_halves(mx) * scale_log2;
      const float m_new = fmaxf(m_used, mx);
      const float alpha = __builtin_amdgcn_exp2f(m_used - m_new);
      m_used = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < kDt; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[dt][e] *= alpha;
      exps(ls);
      tsum = (ls[0] + ls[1]) + (ls[2] + ls[3]);
    }
    l_run += tsum;
  };

  // One matrix-core phase: O += V(sV) P over the tile's pool blocks
  // (kTileBlocks * kDt products), then S = K(sK) Q^T (2 * kDch products),
  // as one software-pipelined stream whose LDS operands are read kPrefetch
  // products ahead, so that a lone wave keeps the matrix core busy.
  constexpr int kPvSteps = kTileBlocks * kDt, kQkSteps = 2 * kDch, kPrefetch = 6;
  auto m_phase = [&](auto with_pv, auto with_qk, const uint8_t* sV, const uint8_t* sK) {
    constexpr int first = decltype(with_pv)::value ? 0 : kPvSteps;
    constexpr int last = decltype(with_qk)::value ? kPvSteps + kQkSteps : kPvSteps;
    auto operand = [&](int st) -> bf16x8 {
      if (st < kPvSteps) {
        const int b = st / kDt, d = (st % kDt) * 32 + n;
        return *(const bf16x8*)(sV + b * kSlabBytes + d * 32 + (v_slot(d, hh) << 4));
      }
      const int u = st - kPvSteps, m = (u & 1) * 32 + n;
      return *(const bf16x8*)(sK + m * kRowBytes + (k_slot<D>(m, (u >> 1) * 2 + hh) << 4));
    };
    // Raised issue priority for the phase: when another wave's softmax and
    // this wave's next product are both ready, the product goes first, so
    // the matrix core does not wait behind a run of vector instructions.
    // The scheduling barriers keep the phase's instructions between the two
    // priority changes.
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(1);
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(with_qk)::value) {
#pragma unroll
      for (int e = 0; e < 16; ++e) { sc0[e] = 0.f; sc1[e] = 0.f; }
    }
    bf16x8 buf[kPrefetch];
#pragma unroll
    for (int st = first; st < first + kPrefetch && st < last; ++st) buf[st % kPrefetch] = operand(st);
#pragma unroll
    for (int st = first; st < last; ++st) {
      const bf16x8 a = buf[st % kPrefetch];
      if (st + kPrefetch < last) buf[st % kPrefetch] = operand(st + kPrefetch);
      if (st < kPvSteps) {
        const int dt = st % kDt;
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, pb[st / kDt], o[dt], 0, 0, 0);
      } else {
        const int u = st - kPvSteps;
        if (u & 1) sc1 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[u >> 1], sc1, 0, 0, 0);
        else sc0 = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, qf[u >> 1], sc0, 0, 0, 0);
      }
    }
    // Pin the pipelined order for the scheduler (mask 0x100: LDS reads,
    // 0x008: matrix-core ops): kPrefetch reads, then one product per read,
    // then the last kPrefetch products.
    constexpr int steps = last - first, lead = steps < kPrefetch ? steps : kPrefetch;
    __builtin_amdgcn_sched_group_barrier(0x100, lead, 0);
#pragma unroll
    for (int st = 0; st < steps - lead; ++st) {
      __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
    __builtin_amdgcn_sched_group_barrier(0x008, lead, 0);
    __builtin_amdgcn_sched_barrier(0);
    __builtin_amdgcn_s_setprio(0);
    __builtin_amdgcn_sched_barrier(0);
  };
  using yes = std::true_type;
  using no = std::false_type;

  // Stores O of a finished item (its row0, rem0, kvh, n_valid as p_*), through
  // this wave's 4 KiB of LDS at tb.
  auto store_item = [&](int p_row0, int p_rem0, int p_kvh, int p_valid, uint8_t* tb) {
    if (wave * kColsPerWave >= p_valid) return;
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if constexpr (MODE == kShared) {  // unnormalised O, max and sum for the suffix half
      const int co = wave * kColsPerWave + n;
      if (co < p_valid) {
        const size_t prow = row_of(p_row0, p_rem0, p_kvh, co) / D;
        if (hh == 0) {
          part_ml[prow * 2] = m_used;
          part_ml[prow * 2 + 1] = l_tot;
        }
#pragma unroll
        for (int dt = 0; dt < kDt; ++dt)
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4) {
            const f32x4 v = {o[dt][g4 * 4], o[dt][g4 * 4 + 1], o[dt][g4 * 4 + 2], o[dt][g4 * 4 + 3]};
            *(f32x4*)(part_o + prow * D + dt * 32 + g4 * 8 + hh * 4) = v;
          }
      }
    } else if constexpr (D == 128) {
      // The normalised O leaves through LDS.  In the matrix-core layout a
      // lane holds 8-byte pieces of one output row, so direct stores put 16
      // bytes of 32 different rows into every instruction.  Each wave
      // writes its 32 rows, 64 dimensions at a time, then stores whole
      // 128-byte half rows, 8 lanes per half row.  16-byte chunks are
      // XOR-swizzled by row against bank conflicts.
      const float inv = 1.f / l_tot;
      static_assert(kSlabBytes >= kColsPerWave * 128, "transpose area");
      size_t orow4[4];  // output row of the 4 rows this lane stores
      bool ok4[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int co = wave * kColsPerWave + r * 8 + (lane >> 3);
        ok4[r] = co < p_valid;
        orow4[r] = row_of(p_row0, p_rem0, p_kvh, co);
      }
      const int ch_r = lane & 7;
#pragma unroll
      for (int p = 0; p < kDt / 2; ++p) {
#pragma unroll
        for (int dl = 0; dl < 2; ++dl)
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4) {
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (__bf16)(o[2 * p + dl][g4 * 4 + e] * inv);
            const int ch = dl * 4 + g4;
            *(bf16x4*)(tb + n * 128 + ((ch ^ (n & 7)) << 4) + hh * 8) = v;
          }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int row = r * 8 + (lane >> 3);
          const u32x4 val = *(const u32x4*)(tb + row * 128 + ((ch_r ^ (row & 7)) << 4));
          if (ok4[r]) *(u32x4*)(out + orow4[r] + p * 64 + ch_r * 8) = val;
        }
      }
    } else {
      const float inv = 1.f / l_tot;
      const int co = wave * kColsPerWave + n;
      if (co < p_valid) {
        uint16_t* orow = out + row_of(p_row0, p_rem0, p_kvh, co);
#pragma unroll
        for (int dt = 0; dt < kDt; ++dt)
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4) {
            bf16x4 v;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[e] = (__bf16)(o[dt][g4 * 4 + e] * inv);
            *(bf16x4*)(orow + dt * 32 + g4 * 8 + hh * 4) = v;
          }
      }
    }
  };

  // Schedule of an item; every wave runs
  //   start:  issue K(0), V(0), K(1) and Q
  //   wait for them; barrier S
  //   M_0 = [S(0) = K(0) Q^T]
  //   then for every tile j:
  //     wait for this wave's own loads (K(j+1), V(j)); barrier B_j;
  //     issue K(j+2) and V(j+1);
  //     V_j = [softmax S(j) -> P(j)]
  //     M_{j+1} = [O += V(j) P(j); S(j+1) = K(j+1) Q^T]   (no S after the last tile)
  // One barrier per tile.  Passing B_j, a wave knows that every wave has
  // ended M_j -- so the buffers of K(j) and V(j-1), which K(j+2) and V(j+1)
  // take, are free -- and that all of K(j+1) and V(j) has landed.  A load
  // has a whole tile step until the barrier that waits for it.  The waves of
  // a workgroup run the same phases together; what overlaps one's softmax
  // with matrix-core work is the other workgroup of the CU, one wave of each
  // on every SIMD.
  // Items overlap: the next item is started right after B_{n-1}, ahead of the
  // last tile's softmax and products, so that the round trips of an item's
  // start run behind the end of the one before.  At B_{n-1} the K buffers and
  // the V buffer of tile n-2 are free for the next item's K(0), K(1) and V(0)
  // (the tile count runs on).  The finished O is stored after the next item's
  // S, when nothing reads V(n-1) any more: that buffer is the transpose area
  // of the stores until the next item's B_0 (each wave its own quarter, which
  // only its own loads write).  The fused list is read only before B_{n-1},
  // the item word between B_{n-1} and the next S.
  //   kWide: both halves of the workgroup run the stream M_0, V_0, M_1, V_1, ...,
  // and meet in the same barriers, but waves 0-3 pass B_j before V_j and waves
  // 4-7 (lag) before M_j: between two barriers one half does V_j, M_{j+1}, the
  // other M_j, V_j, so that on every SIMD one wave's softmax meets the other's
  // products (at an item's end the lagging half's last products, and its store,
  // follow S).  A tile is read over two such intervals, so K and V have three
  // buffers each: behind B_j, K(j+2) takes the buffer of K(j-1), whose last
  // reader, the lagging half's M_{j-1}, ended before B_j, and V(j+1) that of
  // V(j-2), read with it; the next item's K(0), K(1) and V(0), issued after
  // B_{n-1}, those of K(n-3), K(n-2) and V(n-3).  Stores go through V(n-2)'s
  // buffer (waves 0-3) and K(n-1)'s (waves 4-7), free between S and B_0.  Waves
  // 0-3 issue all loads, in their softmax phase: issued by the lagging half in
  // front of its products, its share cost 8% of the launch.
  auto ask = [&]() {  // (nothing is in flight)
    __syncthreads();
    if (tid == 0) {
      s_item = qsel < 8u ? resolve(take()) : kNoItem;
      wait_lgkmcnt0();
    }
    __syncthreads();
    w = __builtin_amdgcn_readfirstlane(s_item);
    __syncthreads();
  };
  for (;;) {
  bool started = false;
  for (;;) {
    if (w == kAsk) ask();
    if (w == kNoItem) break;
    started = start_item();
    if (started) break;
    w = next_static();  // (an item without work)
  }
  if (!started) break;
  bool have_prev = false;  // a finished item's O is still to be stored
  int p_row0 = 0, p_rem0 = 0, p_kvh = 0, p_valid = 0;
  bool act = false;
  const uint8_t* v_last = ring;
  // Transpose area of the stores.
  auto store_area = [&]() { return (kWide && lag ? k_at(2) : v_at(1)) + blk * kSlabBytes; };
  for (;;) {
    if (!lag) wait_vmcnt<0>();
    bare_barrier();  // S
    if (lag && have_prev && act) m_phase(yes(), no(), v_last, ring);
    if constexpr (kIsFused) n_tiles = T_s + __builtin_amdgcn_readfirstlane(f_count);
    // The next item: a number is asked for here and read after B_{n-1}.
    w = next_static();
    unsigned ticket = 0;
    if (tid == 0 && w == kAsk && qsel < 8u) ticket = take();
    if (have_prev) store_item(p_row0, p_rem0, p_kvh, p_valid, store_area());
    if (w == kAsk && tid == 0) {
      s_item = resolve(ticket);
      wait_lgkmcnt0();
    }
#pragma unroll
    for (int dt = 0; dt < kDt; ++dt)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[dt][i] = 0.f;
#pragma unroll
    for (int dt = 0; dt < kDt; ++dt) asm volatile("" : "+v"(o[dt]));  // (no shared tuple of zeros)
    m_used = -INFINITY;
    l_run = 0.f;
    if constexpr (MODE == kSuffix) {
      // Continue from the shared half's state.  Lane half 0 carries the whole sum.
      const size_t prow = row_of(row0, rem0, kvh, min(wave * kColsPerWave + n, n_valid - 1)) / D;
      m_used = part_ml[prow * 2];
      l_run = hh == 0 ? part_ml[prow * 2 + 1] : 0.f;
#pragma unroll
      for (int dt = 0; dt < kDt; ++dt)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const f32x4 v = *(const f32x4*)(part_o + prow * D + dt * 32 + g4 * 8 + hh * 4);
#pragma unroll
          for (int e = 0; e < 4; ++e) o[dt][g4 * 4 + e] = v[e];
        }
    }
    // kFused: the item's request numbers this wave's columns belong to.
    const int ord_lo = kIsFused ? __builtin_amdgcn_readlane(my_ord, 0) : 0;
    const int ord_hi = kIsFused ? __builtin_amdgcn_readlane(my_ord, 31) : 0;
    // kFused: request number and tile of item tile tl (a request tile).
    auto fused_entry = [&](int tl, int& o_, int& tt) {
      const uint32_t e = __builtin_amdgcn_readfirstlane(f_tile[tl - T_s]);
      o_ = int(e >> 24);
      tt = int(e & 0xFFFFFFu);
    };
    // Whether some column of this wave meets tile tl of the item.
    auto active = [&](int tl, int ord) {
      if constexpr (kIsFused) return wave_active && (tl < T_s || (ord >= ord_lo && ord <= ord_hi));
      return tl <= wave_last;
    };
    act = wave_active;
    if constexpr (!kWide) {
      if (act) m_phase(no(), yes(), ring, k_at(0));
    }
    int cur_ord = 0, cur_tt = 0;  // kFused: request number and tile of item tile j (a shared one: itself)
    int j0 = t0 * kKeys, thr = INT_MAX, next_ord = 0, next_tt = 0;
    // First key and (kFused) mask threshold of tile j, and the zeroing of its V tail.
    auto before_barrier = [&](int j) {
      if constexpr (kIsFused) {
        j0 = cur_tt * kKeys;
        thr = INT_MAX;
        next_ord = 0;
        next_tt = j + 1;
        if (j >= T_s) {
          thr = cur_ord == my_ord ? my_pos - j0 - hh * 8 : -1;
          const int lim = __builtin_amdgcn_readfirstlane(f_lim[cur_ord]);
          if (j0 + kKeys > lim) zero_v_tail(j, j0, lim);
        }
        if (j + 1 >= T_s && j + 1 < n_tiles) fused_entry(j + 1, next_ord, next_tt);
      } else {
        j0 = (t0 + j) * kKeys;
        if (!lag && j0 + kKeys > key_lim) zero_v_tail(j, j0, key_lim);
      }
    };
    if constexpr (kWide) {
      auto barrier = [&](int j) {  // B_j, and the loads behind it
        if (!lag && j > 0) wait_vmcnt<0>();
        before_barrier(j);
        bare_barrier();
        if (!lag && j + 1 < n_tiles) {
          issue_v(j + 1, id_next);
          if (j + 2 < n_tiles) {
            id_next = usable(j + 2, raw_next);
            issue_k(j + 2, id_next);
          }
        }
      };
      if (lag) barrier(0);
      if (act) m_phase(no(), yes(), ring, k_at(0));
      if (!lag) barrier(0);
      for (int j = 0; j < n_tiles - 1; ++j) {
        if (!lag && j + 3 < n_tiles) raw_next = raw_id(j + 3);
        int jj = j;
        asm volatile("" : "+s"(jj));
        if (act) {
          mask(j0, thr);
          softmax(MODE != kSuffix && jj == 0);
        }
        asm volatile("" : "+s"(raw_next));
        if (lag) barrier(j + 1);
        if (act) m_phase(yes(), yes(), v_at(j), k_at(j + 1));
        if (!lag) barrier(j + 1);
        act = active(j + 1, 0);
      }
    }
    for (int j = 0; !kWide; ++j) {
      if (j > 0) wait_vmcnt<0>();  // (tile 0's were waited for before S; only stores follow them)
      before_barrier(j);
      bare_barrier();  // B_j
      if (j == n_tiles - 1) break;
      issue_v(j + 1, id_next);
      if (j + 2 < n_tiles) {
        id_next = usable(j + 2, raw_next);
        issue_k(j + 2, id_next);
      }
      // The block id of tile j+3, two steps ahead of its use.  Its scalar load
      // is waited for after the softmax (below), which reads no LDS, and not
      // by the first LDS read of the matrix-core phase, which would then wait
      // for all its operands in flight as well.
      if (j + 3 < n_tiles) {
        if constexpr (kIsFused) {
          int o_ = 0, tt = j + 3, rr = 0;
          if (j + 3 >= T_s) {
            fused_entry(j + 3, o_, tt);
            rr = __builtin_amdgcn_readfirstlane(f_req[o_]);
          }
          raw_next = scalar_load(block_tables + size_t(rr) * max_blocks + min(tt * kTileBlocks + wave, max_blocks - 1));
        } else {
          raw_next = raw_id(j + 3);
        }
      }
      int jj = j;
      asm volatile("" : "+s"(jj));  // keeps the first tile inside the loop (no second copy of its body)
      if (act) {
        mask(j0, thr);
        softmax(MODE != kSuffix && jj == 0);
      }
      asm volatile("" : "+s"(raw_next));
      // (S of a tile past the wave's last one is computed and ignored.)
      if (act) m_phase(yes(), yes(), v_at(j), k_at(j + 1));
      const bool act_next = active(j + 1, next_ord);
      if constexpr (kIsFused) {
        if (!act && act_next) m_phase(no(), yes(), ring, k_at(j + 1));
      }
      act = act_next;
      cur_ord = next_ord;
      cur_tt = next_tt;
    }
    if (act) mask(j0, thr);
    const bool first = MODE != kSuffix && n_tiles == 1;
    v_last = v_at(n_tiles - 1);
    tbase += n_tiles;
    p_row0 = row0;
    p_rem0 = rem0;
    p_kvh = kvh;
    p_valid = n_valid;
    if (w == kAsk) w = __builtin_amdgcn_readfirstlane(s_item);
    started = w != kNoItem && start_item();
    if (!started && w != kNoItem) w = next_static();  // (an item without work)
    if (act) {
      softmax(first);
      if (!lag) m_phase(yes(), no(), v_last, ring);
    }
    if (!started) break;
    have_prev = true;
  }
  if constexpr (kWide) {
    bare_barrier();  // (S)
    if (lag && act) m_phase(yes(), no(), v_last, ring);
  }
  store_item(p_row0, p_rem0, p_kvh, p_valid, kWide ? store_area() : ring + wave * kSlabBytes);
  }

  // (stealing) Every queue is drained.  The last workgroup out clears the
  // counters for the next call on this workspace (no workgroup asks any more by
  // then).  The exit count needs no fence.  Wave 0 (which made every queue
  // atomic of this workgroup) first waits until all its memory operations have
  // completed, so once the last workgroup sees the full count no queue atomic
  // of this launch is in flight.  The outputs are published by the end of the
  // kernel.
  if (stealing && tid == 0) {
    wait_vmcnt<0>();
    const unsigned done =
        __hip_atomic_fetch_add(queue + kDoneWord, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (done == gridDim.x - 1) {
      for (int i = 0; i <= kDrainedWord; ++i)
        __hip_atomic_store(queue + i, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
}

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

int launch_status(const char* what) {
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess)
    return ilpc::set_error(ILPC_EHIP, "%s: launch failed: %s", what, hipGetErrorString(e));
  return ILPC_OK;
}

}  // namespace

extern "C" int ilpc_kv_append(const uint16_t* k_new, const uint16_t* v_new, uint16_t* k_pool,
                              uint16_t* v_pool, int32_t num_blocks, const int32_t* block_tables,
                              int32_t max_blocks, const int32_t* cu_new, const int32_t* start_pos,
                              int32_t B, int32_t max_new, int32_t Hkv, int32_t D,
                              int32_t block_size, void* stream) {
  using ilpc::set_error;
  if (B < 0 || max_new < 0 || num_blocks < 0 || max_blocks < 1 || Hkv < 1)
    return set_error(ILPC_EINVAL, "ilpc_kv_append: negative or zero size");
  if (block_size != kBlock) return set_error(ILPC_EUNSUP, "ilpc_kv_append: block_size must be 16");
  if (D != 64 && D != 128) return set_error(ILPC_EUNSUP, "ilpc_kv_append: head_dim %d unsupported", D);
  if (B == 0 || max_new == 0) return ILPC_OK;
  if (!k_new || !v_new || !k_pool || !v_pool || !block_tables || !cu_new || !start_pos)
    return set_error(ILPC_EINVAL, "ilpc_kv_append: NULL pointer");
  if (!aligned16(k_new) || !aligned16(v_new) || !aligned16(k_pool) || !aligned16(v_pool))
    return set_error(ILPC_EINVAL, "ilpc_kv_append: K/V buffers must be 16-byte aligned");
  if (B > 65535 || Hkv > 65535) return set_error(ILPC_EUNSUP, "ilpc_kv_append: grid too large");
  const int slots = (max_new + kBlock - 2) / kBlock + 1;  // blocks a run of max_new can touch
  const dim3 grid(slots, Hkv, B);
  hipStream_t s = static_cast<hipStream_t>(stream);
  if (D == 128)
    hipLaunchKernelGGL(kv_append_kernel<128>, grid, dim3(256), 0, s, k_new, v_new, k_pool, v_pool,
                       num_blocks, block_tables, max_blocks, cu_new, start_pos, max_new, Hkv);
  else
    hipLaunchKernelGGL(kv_append_kernel<64>, grid, dim3(256), 0, s, k_new, v_new, k_pool, v_pool,
                       num_blocks, block_tables, max_blocks, cu_new, start_pos, max_new, Hkv);
  return launch_status("ilpc_kv_append");
}

namespace {

// The most workgroups a pair's keys are cut over, contexts up to 16 * max_blocks keys.
int decode_max_groups(int64_t B, int64_t Hkv, int64_t max_blocks) {
  return ilpc::decode_max_groups(B * Hkv, (max_blocks * kBlock + 31) / 32);
}

bool decode_shaped(int64_t max_q_len, int Hq, int Hkv) { return max_q_len * (Hq / Hkv) <= kDecodeCols; }

// Few query columns over long contexts.  The persistent kernel would put them
// on a few CUs, each running through all the keys; the decode kernel cuts the
// keys of a column tile of 32 over four or eight waves.  It is the faster one
// while its workgroups have a CU each (at D = 64 half of one).  us, decode ->
// persistent kernel, 8 kv heads and D 128 (4 and 64), 256 tiles (512) of 8
// requests: 1024 keys 16.9 -> 22.4 (14.0 -> 17.2), 4096 keys 43.6 -> 71.7
// (41.6 -> 54.6), 16384 keys 184 -> 278 (149 -> 203), 200 keys in a table of
// that width 8.6 -> 9.6; twice as many tiles, D 128: 25.6 -> 23.0, 78 -> 72, 327
// -> 276.  A shared prefix does not move the line (the split launch over 976
// shared keys is no faster with so few columns: 8 requests of 16 rows over 1936
// keys, G 4, 25.4 -> 42.3).
constexpr int64_t kFewMinKeys = 1024;  // context bound 16 * max_blocks

bool few_columns(int64_t B, int64_t max_q_len, int Hq, int Hkv, int D, int64_t max_blocks) {
  const int64_t tiles = B * Hkv * ((max_q_len * (Hq / Hkv) + kDecodeCols - 1) / kDecodeCols);
  return tiles <= int64_t(ilpc::device_cus()) * (D == 64 ? 2 : 1) && max_blocks * kBlock >= kFewMinKeys;
}

}  // namespace

extern "C" int ilpc_attn_workspace_bytes(int32_t B, int32_t max_q_len, int32_t Hq, int32_t Hkv,
                                         int32_t D, size_t* bytes) {
  if (!bytes || B < 0 || max_q_len < 0 || Hq < 1 || Hkv < 1 || D < 1)
    return ilpc::set_error(ILPC_EINVAL, "ilpc_attn_workspace_bytes: bad argument");
  *bytes = kQueueWords * sizeof(unsigned);
  // room for the partials of the decode kernel's workgroups, on batches of up to B requests
  if (B > 0 && max_q_len > 0 && decode_shaped(max_q_len, Hq, Hkv))
    *bytes += ilpc::decode_auto_bytes(int64_t(B) * Hkv, max_q_len, Hq, Hkv, D);
  return ILPC_OK;
}

namespace {

// Cascade workspace: two queue-counter blocks (one per launch), then the
// partial O [rows, Hq, D] and (max, sum) [rows, Hq, 2] in fp32, where
// rows = B * max_q_len; sections start on 256-byte boundaries.
constexpr size_t kCascadeHead = 256;
size_t align256(size_t x) { return (x + 255) & ~size_t(255); }
size_t cascade_part_o_bytes(int64_t rows, int Hq, int D) { return align256(size_t(rows) * Hq * D * 4); }
size_t cascade_bytes(int64_t rows, int Hq, int D) {
  return kCascadeHead + cascade_part_o_bytes(rows, Hq, D) + align256(size_t(rows) * Hq * 2 * 4);
}

// Argument checks shared by both attention entry points.
int check_attn_args(const char* fn, const uint16_t* q, const uint16_t* k_pool, const uint16_t* v_pool,
                    int32_t num_blocks, const int32_t* block_tables, int32_t max_blocks,
                    const int32_t* cu_q, const int32_t* seq_lens, int32_t B, int32_t max_q_len,
                    int32_t Hq, int32_t Hkv, int32_t D, int32_t block_size, float softmax_scale,
                    const uint16_t* out) {
  using ilpc::set_error;
  if (B < 0 || max_q_len < 0 || num_blocks < 1 || max_blocks < 1 || Hq < 1 || Hkv < 1)
    return set_error(ILPC_EINVAL, "%s: negative or zero size", fn);
  if (block_size != kBlock) return set_error(ILPC_EUNSUP, "%s: block_size must be 16", fn);
  if (D != 64 && D != 128) return set_error(ILPC_EUNSUP, "%s: head_dim %d unsupported", fn, D);
  if (Hq % Hkv != 0 || Hq / Hkv > kMaxGroup)
    return set_error(ILPC_EUNSUP, "%s: Hq %d / Hkv %d unsupported", fn, Hq, Hkv);
  if (!std::isfinite(softmax_scale)) return set_error(ILPC_EINVAL, "%s: softmax_scale is not finite", fn);
  if (max_blocks > kMaxTableBlocks)
    return set_error(ILPC_EUNSUP, "%s: max_blocks %d > %d", fn, max_blocks, kMaxTableBlocks);
  if (B == 0 || max_q_len == 0) return ILPC_OK;
  if (!q || !k_pool || !v_pool || !block_tables || !cu_q || !seq_lens || !out)
    return set_error(ILPC_EINVAL, "%s: NULL pointer", fn);
  if (!aligned16(q) || !aligned16(k_pool) || !aligned16(v_pool) || !aligned16(out))
    return set_error(ILPC_EINVAL, "%s: Q/K/V/out must be 16-byte aligned", fn);
  if (int64_t(B) * max_q_len * (Hq / Hkv) / kCols + 1 > (int64_t(1) << 31) / Hkv)
    return set_error(ILPC_EUNSUP, "%s: grid too large", fn);
  return ILPC_OK;
}

// One persistent launch of mode MODE over `items` work items.
template <int MODE>
int launch_attn(const char* fn, const uint16_t* q, const uint16_t* k_pool, const uint16_t* v_pool,
                int32_t num_blocks, const int32_t* block_tables, int32_t max_blocks, const int32_t* cu_q,
                const int32_t* seq_lens, int32_t B, int32_t Hq, int32_t Hkv, int32_t D, int64_t cols,
                float scale_log2, uint16_t* out, unsigned* queue, int kv_split, float* part_o,
                float* part_ml, int part_rows, hipStream_t s) {
  int64_t col_tiles = (cols + kCols - 1) / kCols;
  int64_t items = col_tiles * Hkv * (MODE == kShared || MODE == kFused ? 1 : B);
  if (items == 0) return ILPC_OK;
  if (items >= int64_t(kAsk)) return ilpc::set_error(ILPC_EUNSUP, "%s: grid too large", fn);
  const int cus = ilpc::device_cus();
  if (cus <= 0) return ilpc::set_error(ILPC_EHIP, "%s: cannot query the device", fn);
  const int64_t wgs = int64_t(wgs_per_cu(D)) * cus;
  unsigned grid = unsigned(items < wgs ? items : wgs);
  // Chunks of the item numbers dealt to the XCDs' queues in turn: whole
  // (request, kv head) pairs, whose items read the same K/V, when they deal out
  // evenly (or nearly so), else pieces that do.
  const int64_t pairs = items / col_tiles;
  // Whether the kernel counts the numbers that hold work: where there are many,
  // more than one to a pair (kWholeBatch: to a kv head); and from half as many
  // on where one request could hold most of the work and would put it on fewer
  // than eight queues, several rounds of it.  Below, taking the empty ones by
  // position costs less than the count does on a batch without any (8 rounds
  // of 64 rows over 200 keys 125 -> 128 us).
  const bool counted =
      col_tiles > 1 && B <= (kIndex - 1) * 64 &&
      (items >= int64_t(kLongRounds) * grid ||
       (MODE == kFull && Hkv < 8 && col_tiles * 16 >= 5 * int64_t(grid) && items >= int64_t(kLongRounds / 2) * grid));
  int shift = 0;
  while (((B - 1) >> shift) + 1 > kIndex - 1) ++shift;
  unsigned chunk = unsigned(
      items >= int64_t(kLongRounds) * grid ? (items + 7) / 8
      : pairs % 8 == 0 || pairs >= 256     ? col_tiles
                                           : std::max<int64_t>(items / 256, 1));
  unsigned threads = 64 * kWaves;
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, dim3(grid), dim3(threads), 0, s, q, k_pool, v_pool, num_blocks, block_tables, max_blocks,
                       cu_q, seq_lens, B, Hq, Hkv, int(col_tiles), unsigned(items), chunk, counted ? shift : -1,
                       scale_log2, out, queue, kv_split, part_o, part_ml, part_rows);
  };
  if constexpr (MODE == kFull || MODE == kSuffix) {
    if (counted) {
      if constexpr (MODE == kFull) {
        // Both layouts, of which the one that the batch's rows do not call for
        // returns at once (2 to 3 us; only the device knows how many rows
        // there are).  The wide one where the items fill its 256 columns -- 192
        // or 256 columns a pair 8-14% faster, 512 and from 1024 on 5-8%, 320,
        // 384 and 640 the same -- and give every CU eight of them: below, items
        // half as large level better (64 requests of 1 row but one of 600, 32/8
        // heads, 31 us narrow, 39 wide).
        constexpr int kWideCols = 2 * kCols;
        if (D == 128 && items >= int64_t(kLongRounds) * wgs && (cols >= 4 * kWideCols || (cols - 1) % kWideCols >= kCols)) {
          part_rows = int(std::max<int64_t>(1, int64_t(kWideRounds) * kWideCols * cus / Hq));
          const int64_t narrow_tiles = col_tiles, narrow_items = items;
          const unsigned narrow_grid = grid;
          col_tiles = (cols + kWideCols - 1) / kWideCols;
          items = col_tiles * Hkv * B;
          grid = unsigned(std::min<int64_t>(items, cus));
          threads = 128 * kWaves;
          launch(paged_attn_kernel<128, MODE, true, 2 * kWaves>);
          col_tiles = narrow_tiles, items = narrow_items, grid = narrow_grid, threads = 64 * kWaves;
        }
      }
      if (D == 128) launch(paged_attn_kernel<128, MODE, true, kWaves>);
      else launch(paged_attn_kernel<64, MODE, true, kWaves>);
      return launch_status(fn);
    }
  }
  if (D == 128) launch(paged_attn_kernel<128, MODE, false, kWaves>);
  else launch(paged_attn_kernel<64, MODE, false, kWaves>);
  return launch_status(fn);
}

}  // namespace

extern "C" int ilpc_paged_prefill_attn(const uint16_t* q, const uint16_t* k_pool,
                                       const uint16_t* v_pool, int32_t num_blocks,
                                       const int32_t* block_tables, int32_t max_blocks,
                                       const int32_t* cu_q, const int32_t* seq_lens, int32_t B,
                                       int32_t max_q_len, int32_t Hq, int32_t Hkv, int32_t D,
                                       int32_t block_size, float softmax_scale, uint16_t* out,
                                       void* workspace, size_t workspace_bytes, void* stream) {
  static const char* fn = "ilpc_paged_prefill_attn";
  int rc = check_attn_args(fn, q, k_pool, v_pool, num_blocks, block_tables, max_blocks, cu_q, seq_lens, B,
                           max_q_len, Hq, Hkv, D, block_size, softmax_scale, out);
  if (rc != ILPC_OK || B == 0 || max_q_len == 0) return rc;
  if (!workspace || workspace_bytes < kQueueWords * sizeof(unsigned) || !aligned16(workspace))
    return ilpc::set_error(ILPC_EINVAL, "%s: workspace must be %zu bytes, 16-byte aligned", fn,
                           kQueueWords * sizeof(unsigned));
  // Decode-shaped batches go to the decode kernel, a pair's keys over as many
  // workgroups as the workspace has room for partials (after the queue counters).
  // It needs none with one, and is faster than the persistent kernel (one
  // workgroup a pair, tile after tile) at that too: 4 requests, 8 kv heads, D 128,
  // 200 keys 8.3 -> 5.7 us, 1000 keys 20.2 -> 12.8, 2100 keys 38.0 -> 22.9.
  const float scale_log2 = softmax_scale * 1.4426950408889634f;
  if (decode_shaped(max_q_len, Hq, Hkv)) {
    const size_t head = kQueueWords * sizeof(unsigned);
    int n = decode_max_groups(B, Hkv, max_blocks);
    while (n > 1 && workspace_bytes < head + ilpc::decode_split_bytes(B, max_q_len, Hq, Hkv, D, n)) --n;
    return ilpc::launch_decode_attn(
        q, k_pool, v_pool, num_blocks, block_tables, max_blocks, cu_q, seq_lens, B, max_q_len, Hq, Hkv, D, scale_log2,
        out, n, true, n > 1 ? reinterpret_cast<float*>(static_cast<uint8_t*>(workspace) + head) : nullptr, stream);
  }
  if (few_columns(B, max_q_len, Hq, Hkv, D, max_blocks))
    return ilpc::launch_decode_attn(q, k_pool, v_pool, num_blocks, block_tables, max_blocks, cu_q, seq_lens, B,
                                    max_q_len, Hq, Hkv, D, scale_log2, out, 1, true, nullptr, stream);
  return launch_attn<kFull>(fn, q, k_pool, v_pool, num_blocks, block_tables, max_blocks, cu_q, seq_lens, B,
                            Hq, Hkv, D, int64_t(max_q_len) * (Hq / Hkv), scale_log2, out,
                            static_cast<unsigned*>(workspace), 0, nullptr, nullptr, 0,
                            static_cast<hipStream_t>(stream));
}


extern "C" int ilpc_decode_split(int32_t B, int32_t Hkv, int32_t max_blocks, int32_t* n_split) {
  if (!n_split || B < 0 || Hkv < 1 || max_blocks < 1)
    return ilpc::set_error(ILPC_EINVAL, "ilpc_decode_split: bad argument");
  *n_split = decode_max_groups(B, Hkv, max_blocks);
  return ILPC_OK;
}

extern "C" int ilpc_decode_workspace_bytes(int32_t B, int32_t max_q_len, int32_t Hq, int32_t Hkv, int32_t D,
                                           int32_t n_split, size_t* bytes) {
  if (!bytes || B < 0 || max_q_len < 0 || Hq < 1 || Hkv < 1 || D < 1 || n_split < 1 ||
      n_split > ilpc::kMaxSplit)
    return ilpc::set_error(ILPC_EINVAL, "ilpc_decode_workspace_bytes: bad argument");
  *bytes = ilpc::decode_split_bytes(B, max_q_len, Hq, Hkv, D, n_split);
  return ILPC_OK;
}

extern "C" int ilpc_paged_decode_attn(const uint16_t* q, const uint16_t* k_pool, const uint16_t* v_pool,
                                     int32_t num_blocks, const int32_t* block_tables, int32_t max_blocks,
                                     const int32_t* cu_q, const int32_t* seq_lens, int32_t B, int32_t max_q_len,
                                     int32_t Hq, int32_t Hkv, int32_t D, int32_t block_size,
                                     float softmax_scale, uint16_t* out, int32_t n_split, void* workspace,
                                     size_t workspace_bytes, void* stream) {
  static const char* fn = "ilpc_paged_decode_attn";
  int rc = check_attn_args(fn, q, k_pool, v_pool, num_blocks, block_tables, max_blocks, cu_q, seq_lens, B,
                           max_q_len, Hq, Hkv, D, block_size, softmax_scale, out);
  if (rc != ILPC_OK || B == 0 || max_q_len == 0) return rc;
  if (int64_t(max_q_len) * (Hq / Hkv) > kDecodeCols)
    return ilpc::set_error(ILPC_EUNSUP, "%s: max_q_len * Hq / Hkv = %lld > %d", fn,
                           (long long)max_q_len * (Hq / Hkv), kDecodeCols);
  if (n_split < 0 || n_split > ilpc::kMaxSplit)
    return ilpc::set_error(ILPC_EINVAL, "%s: n_split %d outside [0, %d]", fn, n_split, ilpc::kMaxSplit);
  const bool automatic = n_split == 0;
  if (automatic) n_split = decode_max_groups(B, Hkv, max_blocks);
  if (int64_t(B) * Hkv * n_split > INT32_MAX)
    return ilpc::set_error(ILPC_EUNSUP, "%s: B * Hkv * n_split too large", fn);
  const size_t need = ilpc::decode_split_bytes(B, max_q_len, Hq, Hkv, D, n_split);
  if (need && (!workspace || workspace_bytes < need || !aligned16(workspace)))
    return ilpc::set_error(ILPC_EINVAL, "%s: %d key ranges need a %zu-byte workspace, 16-byte aligned", fn,
                           n_split, need);
  return ilpc::launch_decode_attn(q, k_pool, v_pool, num_blocks, block_tables, max_blocks, cu_q, seq_lens, B,
                                  max_q_len, Hq, Hkv, D, softmax_scale * 1.4426950408889634f, out, n_split,
                                  automatic, static_cast<float*>(workspace), stream);
}

extern "C" int ilpc_attn_cascade_workspace_bytes(int32_t B, int32_t max_q_len, int32_t Hq, int32_t Hkv,
                                                 int32_t D, size_t* bytes) {
  if (!bytes || B < 0 || max_q_len < 0 || Hq < 1 || Hkv < 1 || D < 1)
    return ilpc::set_error(ILPC_EINVAL, "ilpc_attn_cascade_workspace_bytes: bad argument");
  *bytes = cascade_bytes(int64_t(B) * max_q_len, Hq, D);
  return ILPC_OK;
}

extern "C" int ilpc_paged_prefill_attn_cascade(
    const uint16_t* q, const uint16_t* k_pool, const uint16_t* v_pool, int32_t num_blocks,
    const int32_t* block_tables, int32_t max_blocks, const int32_t* cu_q, const int32_t* seq_lens,
    int32_t B, int32_t max_q_len, int32_t Hq, int32_t Hkv, int32_t D, int32_t block_size,
    int32_t shared_len, float softmax_scale, uint16_t* out, void* workspace, size_t workspace_bytes,
    void* stream) {
  static const char* fn = "ilpc_paged_prefill_attn_cascade";
  int rc = check_attn_args(fn, q, k_pool, v_pool, num_blocks, block_tables, max_blocks, cu_q, seq_lens, B,
                           max_q_len, Hq, Hkv, D, block_size, softmax_scale, out);
  if (rc != ILPC_OK) return rc;
  if (shared_len < 0 || shared_len % kBlock != 0 || shared_len > max_blocks * kBlock)
    return ilpc::set_error(ILPC_EINVAL, "%s: shared_len %d must be a multiple of 16 in [0, 16 * max_blocks]",
                           fn, shared_len);
  if (B == 0 || max_q_len == 0) return ILPC_OK;
  const int64_t rows = int64_t(B) * max_q_len;
  if (rows * Hq > (int64_t(1) << 31) - 1) return ilpc::set_error(ILPC_EUNSUP, "%s: batch too large", fn);
  const size_t need = cascade_bytes(rows, Hq, D);
  if (!workspace || workspace_bytes < need || !aligned16(workspace))
    return ilpc::set_error(ILPC_EINVAL, "%s: workspace must be %zu bytes, 16-byte aligned", fn, need);
  uint8_t* ws = static_cast<uint8_t*>(workspace);
  unsigned* queue_shared = reinterpret_cast<unsigned*>(ws);
  unsigned* queue_suffix = reinterpret_cast<unsigned*>(ws + kQueueWords * sizeof(unsigned));
  float* part_o = reinterpret_cast<float*>(ws + kCascadeHead);
  float* part_ml = reinterpret_cast<float*>(ws + kCascadeHead + cascade_part_o_bytes(rows, Hq, D));
  const float scale_log2 = softmax_scale * 1.4426950408889634f;
  hipStream_t s = static_cast<hipStream_t>(stream);
  const int G = Hq / Hkv;
  const int64_t cols = int64_t(max_q_len) * G;
  // (few_columns() as in ilpc_paged_prefill_attn, whose pass shared_len = 0 runs;
  // with so few columns the sharing saves less than the idle CUs cost)
  if (!decode_shaped(max_q_len, Hq, Hkv) && few_columns(B, max_q_len, Hq, Hkv, D, max_blocks))
    return ilpc::launch_decode_attn(q, k_pool, v_pool, num_blocks, block_tables, max_blocks, cu_q, seq_lens, B,
                                    max_q_len, Hq, Hkv, D, scale_log2, out, 1, true, nullptr, stream);
  if (shared_len == 0)
    return launch_attn<kFull>(fn, q, k_pool, v_pool, num_blocks, block_tables, max_blocks, cu_q, seq_lens,
                              B, Hq, Hkv, D, cols, scale_log2, out, queue_shared, 0, nullptr, nullptr,
                              0, s);
  // One launch (kFused) for prefill-shaped batches whose shared prefix holds
  // at least three 64-key tiles and whose per-item tile list fits: at most
  // 128 / G + 1 requests have rows in an item, each with at most
  // ceil(16 * max_blocks / 64) - T_s tiles of its own.
  const int64_t T_s = shared_len / kKeys;
  const int64_t own_tiles = std::max<int64_t>(0, (int64_t(max_blocks) * kBlock + kKeys - 1) / kKeys - T_s);
  if (T_s >= 3 && int64_t(max_q_len) * G >= 2 * kColsPerWave &&
      ((kCols + G - 1) / G + 1) * own_tiles <= kFusedTiles)
    return launch_attn<kFused>(fn, q, k_pool, v_pool, num_blocks, block_tables, max_blocks, cu_q, seq_lens, B,
                               Hq, Hkv, D, rows * G, scale_log2, out, queue_shared,
                               int(T_s * kKeys), nullptr, nullptr, int(rows), s);
  rc = launch_attn<kShared>(fn, q, k_pool, v_pool, num_blocks, block_tables, max_blocks, cu_q, seq_lens, B,
                            Hq, Hkv, D, rows * G, scale_log2, out, queue_shared,
                            shared_len, part_o, part_ml, int(rows), s);
  if (rc != ILPC_OK) return rc;
  return launch_attn<kSuffix>(fn, q, k_pool, v_pool, num_blocks, block_tables, max_blocks, cu_q, seq_lens, B,
                              Hq, Hkv, D, cols, scale_log2, out, queue_suffix, shared_len, part_o,
                              part_ml, int(rows), s);
}

// Paged attention for decode-shaped batches (a few query rows per request),
// for gfx950.
//
// InferLog section 2.1.2: after the prefill, each generated token attends to
// the cached KV of its whole context.  With one to a few query rows per
// request the work is bound by reading K and V from HBM, not by the matrix
// cores, so this kernel drops the workgroup-shared LDS ring of the prefill
// kernel: every wave owns one (request, kv head) -- or, where the batch has too
// few of these to fill the chip, a range of its keys -- and streams its K
// and V blocks straight from the pools into registers, two 16-token pool
// blocks (32 keys) per step, with the next step's loads in flight while the
// current one is computed.  The G query heads of the kv head times the
// request's q_len rows (at most 32 columns) form the N side of the same
// v_mfma_f32_32x32x16_bf16 products as the prefill kernel:
//   S^T = K Q^T  (K rows loaded in a permuted key order, so that the score
//                 accumulators are already laid out as the P^T operand),
//   O^T += V^T P^T  (V blocks are stored dimension-major, so each lane's
//                 operand is 16 contiguous bytes of one V row),
// with the online softmax in fp32 on exp2 (Q^T is kept in LDS, so that two
// steps of K/V fit in the registers).  Each XCD takes a contiguous range of
// requests, all kv heads of each: the (block, kv head) slabs of a pool block
// are adjacent in memory, and an XCD's reads stay within its requests' share
// of the pools.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>

#include "../../include/ilpc.h"
#include "ilpc_internal.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kBlock = 16;
constexpr int kStepKeys = 32;        // keys per step (two pool blocks)
constexpr int kMaxGroups = 16;       // most workgroups a pair's keys are cut over by the library's choice
constexpr float kLazyRescale = 8.f;  // log2 growth of a column max tolerated before rescaling O

// Key held by MFMA row m of a step: inside every 16 keys the groups [4,8)
// and [8,12) trade places, so that accumulator register e of lane half hh
// holds key (e >> 3) * 16 + 8 * hh + (e & 7), the layout of the P^T operand.
__device__ __forceinline__ int key_of_row(int m) {
  const int grp = (m >> 2) & 3;
  return m + (grp == 1 ? 4 : (grp == 2 ? -4 : 0));
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }

__device__ __forceinline__ float max_across_halves(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

template <int D>
struct StepRegs {
  u32x4 k[D / 16];      // K operand, one per 16-dimension chunk
  u32x4 v[2][D / 32];   // V^T operand, [pool block of the step][32-dimension tile]
};

// Waves of a workgroup whose waves work W to a (request, kv head) pair.
constexpr int group_waves(int W) { return W > 4 ? W : 4; }

// W waves of the workgroup (1, 2, 4 or 8) share a (request, kv head) pair's 32
// query columns: each takes its share of the steps, and their partial results
// are merged through LDS at the end.
template <int D, int W>
__global__ __launch_bounds__(64 * group_waves(W), 2) void decode_attn_kernel(
    const uint16_t* __restrict__ q, const uint16_t* __restrict__ k_pool,
    const uint16_t* __restrict__ v_pool, int num_blocks, const int32_t* __restrict__ block_tables,
    int max_blocks, const int32_t* __restrict__ cu_q, const int32_t* __restrict__ seq_lens, int n_req,
    int max_q_len, int Hq, int Hkv, float scale_log2, uint16_t* __restrict__ out, int n_ct, int n_split,
    int cols_cap, float* __restrict__ part_o, float* __restrict__ part_ml) {
  constexpr int kDch = D / 16, kDt = D / 32, kWavesPerGroup = group_waves(W);
  // Each wave's Q^T operand lives in LDS (read once per product), which keeps
  // two steps of K/V loads plus O within the registers of two waves per SIMD.
  // For the merge (W > 1) the same space then holds every wave's O, one row of
  // kRow floats per query column (4 more than D: rows start in other banks).
  constexpr int kRow = D + 4, kCols = 32;
  constexpr int kQBytes = kWavesPerGroup * kDch * 64 * 16, kOBytes = kWavesPerGroup * kCols * kRow * 4;
  __shared__ __attribute__((aligned(16))) uint8_t lds[W > 1 && kOBytes > kQBytes ? kOBytes : kQBytes];
  __shared__ float s_m[kWavesPerGroup][kCols], s_l[kWavesPerGroup][kCols];
  u32x4(*q_lds)[kDch][64] = reinterpret_cast<u32x4(*)[kDch][64]>(lds);
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 31, hh = lane >> 5;

  // Group b runs on XCD b % 8 (round-robin dispatch); XCD x takes a
  // contiguous range of groups, and items are numbered request-major (about
  // 5% more bandwidth on 512 distinct 2 K-token contexts than kv-head-major
  // numbering, which keeps one kv head's blocks in one XCD's L2 and is 2-3%
  // faster only when every request reads one shared prefix).
  const unsigned nb = gridDim.x, per = nb >> 3, extra = nb & 7u;
  const unsigned x = blockIdx.x & 7u, i = blockIdx.x >> 3;
  const unsigned group = x * per + min(x, extra) + i;
  const int item = int(group) * (kWavesPerGroup / W) + wave / W;
  const int n_items = n_req * Hkv * n_split * n_ct;
  if (W == 1 && item >= n_items) return;
  // The pair's steps are cut into n_split * W consecutive ranges, one per
  // wave.  With n_split > 1 each workgroup leaves its pair's unnormalised O,
  // max and sum in part_o / part_ml for decode_combine_kernel (cols_cap =
  // max_q_len * G columns per split).
  // Batches with more than 32 columns a pair (n_ct > 1 column tiles of 32) are
  // not split further.
  const bool in_grid = item < n_items;
  const int ct = in_grid ? item % n_ct : 0, rest = in_grid ? item / n_ct : 0;
  const int sp = rest % n_split, pair = rest / n_split;
  const int r = pair / Hkv, h = pair % Hkv;
  const int G = Hq / Hkv;

  const int q0 = cu_q[r], q_len = cu_q[r + 1] - q0;
  const int L = min(seq_lens[r], max_blocks * kBlock);
  // rows past max_q_len are not computed
  const int col0 = ct * kCols, n_cols = min(min(q_len, max_q_len) * G - col0, kCols);
  const bool valid = in_grid && q_len > 0 && q_len <= L && n_cols > 0;
  if (W == 1 && !valid) return;

  f32x16 o[kDt];
#pragma unroll
  for (int dt = 0; dt < kDt; ++dt)
#pragma unroll
    for (int e = 0; e < 16; ++e) o[dt][e] = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  bool col_valid = false;
  size_t qrow = 0;
  if (valid) {
  // This lane's query column (padding columns repeat the last valid one).
  col_valid = n < n_cols;
  const int colc = col0 + (col_valid ? n : n_cols - 1);
  const int t = colc / G;
  const int pos = L - q_len + t;  // keys 0 .. pos are visible to this column
  qrow = (size_t(q0 + t) * Hq + size_t(h) * G + (colc - t * G)) * D;
#pragma unroll
  for (int kc = 0; kc < kDch; ++kc) q_lds[wave][kc][lane] = *(const u32x4*)(q + qrow + kc * 16 + hh * 8);

  const int32_t* bt = block_tables + size_t(r) * max_blocks;
  const int n_blk = (L + kBlock - 1) / kBlock;
  // keys past the last column's position are not visited (and their V rows zeroed)
  const int key_end = L - q_len + (col0 + n_cols - 1) / G + 1;
  const int n_steps_all = (key_end + kStepKeys - 1) / kStepKeys;
  const int n_ranges = n_split * W, range = sp * W + wave % W;
  const int steps_per = (n_steps_all + n_ranges - 1) / n_ranges;
  const int s_begin = min(range * steps_per, n_steps_all);
  const int n_steps = min(s_begin + steps_per, n_steps_all);  // this wave runs steps s_begin .. n_steps-1
  const int krow = key_of_row(n);  // key of the step this lane's K operand row holds
  const size_t head_off = size_t(h) * kBlock * D;
  const size_t slab = size_t(Hkv) * kBlock * D;

  // Block ids come 64 at a time, one per lane, by vector loads issued a
  // window ahead of use (scalar loads would put a memory round trip, and a
  // wait shared with the LDS reads, in front of every step); a step picks its
  // two ids out with readlane.  Ids past the request's blocks or outside the
  // pool read block 0 (those keys are masked and their V rows zeroed).
  auto load_ids = [&](int window) {
    return bt[min(window * 64 + lane, max_blocks - 1)];
  };
  // Window w lives in ids[w & 1]; the other register receives window w + 1
  // (two named registers and a uniform branch: no copy that would wait for
  // the load in flight).
  int win = (2 * s_begin) >> 6;
  int ids0, ids1;
  if (win & 1) {
    ids1 = load_ids(win);
    ids0 = load_ids(win + 1);
  } else {
    ids0 = load_ids(win);
    ids1 = load_ids(win + 1);
  }
  auto block_id = [&](int lb) {
    const int id = (win & 1) ? __builtin_amdgcn_readlane(ids1, lb & 63) : __builtin_amdgcn_readlane(ids0, lb & 63);
    return (lb < n_blk && id >= 0 && id < num_blocks) ? id : 0;
  };
  auto load = [&](int s, StepRegs<D>& R) {
    if ((2 * s) >> 6 != win) {  // steps run in order: the next window
      if (win & 1) ids1 = load_ids(win + 2);
      else ids0 = load_ids(win + 2);
      ++win;
    }
    const int id0 = block_id(2 * s), id1 = block_id(2 * s + 1);
    const int idk = krow < kBlock ? id0 : id1;
    const uint16_t* ks = k_pool + size_t(idk) * slab + head_off + size_t(krow & 15) * D + hh * 8;
#pragma unroll
    for (int kc = 0; kc < kDch; ++kc) R.k[kc] = *(const u32x4*)(ks + kc * 16);
#pragma unroll
    for (int b = 0; b < 2; ++b) {
      const uint16_t* vs = v_pool + size_t(b ? id1 : id0) * slab + head_off + size_t(n) * kBlock + hh * 8;
#pragma unroll
      for (int dt = 0; dt < kDt; ++dt) R.v[b][dt] = *(const u32x4*)(vs + dt * 32 * kBlock);
    }
  };

  const int mask_from = L - q_len + col0 / G;  // steps reaching past this key need the causal mask

  auto compute = [&](int s, StepRegs<D>& R) {
    const int j0 = s * kStepKeys;
    f32x16 sc;
#pragma unroll
    for (int e = 0; e < 16; ++e) sc[e] = 0.f;
#pragma unroll
    for (int kc = 0; kc < kDch; ++kc)
      sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(R.k[kc]), as_bf16x8(q_lds[wave][kc][lane]), sc,
                                                  0, 0, 0);
    if (j0 + kStepKeys - 1 > mask_from) {
      // causal mask (keys past pos, which also covers keys >= L), and the V
      // rows of keys >= key_end zeroed: unwritten pool slots may hold any bits
      const int rel = pos - j0 - hh * 8;
#pragma unroll
      for (int e = 0; e < 16; ++e)
        if ((e >> 3) * 16 + (e & 7) > rel) sc[e] = -INFINITY;
      const int lim = key_end - j0 - hh * 8;  // keys b * 16 + e of this lane's V operand are valid iff < lim
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int dt = 0; dt < kDt; ++dt)
#pragma unroll
          for (int w = 0; w < 4; ++w) {
            const int k0 = b * 16 + 2 * w;
            R.v[b][dt][w] &= (k0 < lim ? 0x0000FFFFu : 0u) | (k0 + 1 < lim ? 0xFFFF0000u : 0u);
          }
    }
    float mx = sc[0];
#pragma unroll
    for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sc[e]);
    mx = max_across_halves(mx) * scale_log2;
    // Lazy rescale: O and the sum are rescaled only when a column max grows
    // by more than 2^8 over the one its exponentials are taken against (the
    // first step always sets it: key 0 is visible to every column).
    if (__ballot(mx > m_run + kLazyRescale)) {
      const float m_new = fmaxf(m_run, mx);
      // (a column with nothing visible yet keeps m = -inf and alpha = 1)
      const float alpha = m_new == m_run ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);
      m_run = m_new;
      l_run *= alpha;
#pragma unroll
      for (int dt = 0; dt < kDt; ++dt)
#pragma unroll
        for (int e = 0; e < 16; ++e) o[dt][e] *= alpha;
    }
    bf16x8 pb[2];
    float ls = 0.f;
    // until a column has seen a visible key (possible in a split that starts
    // past key 0) its scores and max are -inf: subtract 0 then, so that exp2
    // gives 0 rather than NaN
    const float m_sub = m_run == -INFINITY ? 0.f : m_run;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[e], scale_log2, -m_sub));
      pb[e >> 3][e & 7] = (__bf16)p;
      ls += p;
    }
    l_run += ls;
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int dt = 0; dt < kDt; ++dt)
        o[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(R.v[b][dt]), pb[b], o[dt], 0, 0, 0);
  };

  // Two register sets: the next step's loads fly while the current is computed.
  // The scheduling barriers keep each step's loads after the computation that
  // frees their registers: hoisted, they would need a third register set.
  StepRegs<D> ra, rb;
  int s = s_begin;
  if (s < n_steps) load(s, ra);
  for (; s + 1 < n_steps; s += 2) {
    load(s + 1, rb);
    __builtin_amdgcn_sched_barrier(0);
    compute(s, ra);
    __builtin_amdgcn_sched_barrier(0);
    if (s + 2 < n_steps) load(s + 2, ra);
    __builtin_amdgcn_sched_barrier(0);
    compute(s + 1, rb);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (s < n_steps) compute(s, ra);
  }

  const float l_tot = l_run + __shfl_xor(l_run, 32);
  if constexpr (W == 1) {
    if (n_split > 1) {
      // partial state of this (pair, split), valid columns only: O [cols_cap][D]
      // (unnormalised) in part_o, (max, sum) [cols_cap][2] in part_ml
      if (col_valid) {
        const size_t slot = (size_t(pair) * n_split + sp) * size_t(cols_cap) + n;
        float* po = part_o + slot * D;
#pragma unroll
        for (int dt = 0; dt < kDt; ++dt)
#pragma unroll
          for (int g4 = 0; g4 < 4; ++g4) {
            const f32x4 v = {o[dt][g4 * 4], o[dt][g4 * 4 + 1], o[dt][g4 * 4 + 2], o[dt][g4 * 4 + 3]};
            *(f32x4*)(po + dt * 32 + g4 * 8 + hh * 4) = v;
          }
        if (hh == 0) {
          part_ml[slot * 2] = m_run;
          part_ml[slot * 2 + 1] = l_tot;
        }
      }
      return;
    }
    if (col_valid) {
      const float inv = 1.f / l_tot;
      uint16_t* orow = out + qrow;
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
  } else {
    // Merge of the W ranges: every wave's O, max and sum to LDS (the first
    // barrier: no wave reads Q from there any more), then each thread of the
    // pair's waves sums pieces of 4 dimensions with weights 2^(m_k - M).
    float(*so)[kCols][kRow] = reinterpret_cast<float(*)[kCols][kRow]>(lds);
    __syncthreads();
    if (col_valid) {
#pragma unroll
      for (int dt = 0; dt < kDt; ++dt)
#pragma unroll
        for (int g4 = 0; g4 < 4; ++g4) {
          const f32x4 v = {o[dt][g4 * 4], o[dt][g4 * 4 + 1], o[dt][g4 * 4 + 2], o[dt][g4 * 4 + 3]};
          *(f32x4*)&so[wave][n][dt * 32 + g4 * 8 + hh * 4] = v;
        }
      if (hh == 0) {
        s_m[wave][n] = m_run;
        s_l[wave][n] = l_tot;
      }
    }
    __syncthreads();
    if (!valid) return;
    const int w0 = wave / W * W;  // first wave of the pair
    for (int u = (wave - w0) * 64 + lane; u < n_cols * (D / 4); u += W * 64) {
      const int c = u / (D / 4), d = u % (D / 4) * 4;
      float mx = s_m[w0][c];
#pragma unroll
      for (int k = 1; k < W; ++k) mx = fmaxf(mx, s_m[w0 + k][c]);
      f32x4 acc = {0.f, 0.f, 0.f, 0.f};
      float den = 0.f;
#pragma unroll
      for (int k = 0; k < W; ++k) {
        const float m = s_m[w0 + k][c];
        // (a range that saw no key of this column has m = -inf and weight 0)
        const float wgt = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mx);
        den += wgt * s_l[w0 + k][c];
        const f32x4 v = *(const f32x4*)&so[w0 + k][c][d];
#pragma unroll
        for (int e = 0; e < 4; ++e) acc[e] += wgt * v[e];
      }
      if (n_split > 1) {
        const size_t slot = (size_t(pair) * n_split + sp) * size_t(cols_cap) + c;
        *(f32x4*)(part_o + slot * D + d) = acc;
        if (d == 0) {
          part_ml[slot * 2] = mx;
          part_ml[slot * 2 + 1] = den;
        }
      } else {
        const int t = (col0 + c) / G;
        const float inv = 1.f / den;
        bf16x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = (__bf16)(acc[e] * inv);
        *(bf16x4*)(out + (size_t(q0 + t) * Hq + size_t(h) * G + (col0 + c - t * G)) * D + d) = v;
      }
    }
  }
}

// Merge of the n_split partial states of one (kv head, request, column):
// one wave each.  Lane k reads split k's (max, sum); with M = max_k m_k and
// w_k = 2^(m_k - M), O = sum_k w_k O_k / sum_k w_k l_k.  Lane l covers
// dimensions l * D/64 .. of O.  Split 0 holds key 0, visible to every
// column, so M is finite; a split that saw no visible key has m = -inf,
// O = 0 and weight 0.
constexpr int kCombineWaves = 4;  // per workgroup

template <int D>
__global__ __launch_bounds__(64 * kCombineWaves) void decode_combine_kernel(
    const float* __restrict__ part_o, const float* __restrict__ part_ml, const int32_t* __restrict__ cu_q,
    const int32_t* __restrict__ seq_lens,
    int max_blocks, int n_req, int max_q_len, int Hq, int Hkv, int n_split, int cols_cap,
    uint16_t* __restrict__ out) {
  constexpr int kPer = D / 64;  // dimensions per lane
  typedef float vec_t __attribute__((ext_vector_type(kPer)));
  const int lane = threadIdx.x & 63;
  const int64_t w = int64_t(blockIdx.x) * kCombineWaves + (threadIdx.x >> 6);
  const int c = int(w % cols_cap);
  const int pair = int(w / cols_cap);
  if (pair >= n_req * Hkv) return;
  const int r = pair / Hkv, h = pair % Hkv;
  const int G = Hq / Hkv;
  const int q0 = cu_q[r], q_len = cu_q[r + 1] - q0;
  const int L = min(seq_lens[r], max_blocks * kBlock);
  const int n_cols = min(q_len, max_q_len) * G;
  if (q_len <= 0 || q_len > L || n_cols > 32 || c >= n_cols) return;

  // slot of (pair, split k, column c) = (pair * n_split + k) * cols_cap + c
  const size_t slot0 = size_t(pair) * n_split * cols_cap + c;
  float m = -INFINITY, l = 0.f;
  if (lane < n_split) {
    m = part_ml[(slot0 + size_t(lane) * cols_cap) * 2];
    l = part_ml[(slot0 + size_t(lane) * cols_cap) * 2 + 1];
  }
  float mx = m;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mx = fmaxf(mx, __shfl_xor(mx, off));
  const float wgt = m == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m - mx);
  float den = wgt * l;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) den += __shfl_xor(den, off);

  const float* po = part_o + slot0 * D + lane * kPer;
  const size_t chunk = size_t(cols_cap) * D;  // stride between splits
  vec_t acc = {};
  int k = 0;
  for (; k + 4 <= n_split; k += 4) {
    vec_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) v[u] = *(const vec_t*)(po + (k + u) * chunk);
#pragma unroll
    for (int u = 0; u < 4; ++u)
      acc += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wgt), k + u)) * v[u];
  }
  for (; k < n_split; ++k)
    acc += __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wgt), k)) * *(const vec_t*)(po + k * chunk);

  const int t = c / G;
  uint16_t* orow = out + (size_t(q0 + t) * Hq + size_t(h) * G + (c - t * G)) * D + lane * kPer;
  const float inv = 1.f / den;
#pragma unroll
  for (int e = 0; e < kPer; ++e) orow[e] = __builtin_bit_cast(uint16_t, (__bf16)(acc[e] * inv));
}

}  // namespace

namespace ilpc {

int device_cus() {
  static int cached[64] = {};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) return 0;
  if (dev < 64 && cached[dev] > 0) return cached[dev];
  int cus = 0;
  if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
  if (dev < 64) cached[dev] = cus;
  return cus;
}

size_t decode_split_bytes(int B, int max_q_len, int Hq, int Hkv, int D, int n_split) {
  const int64_t cols = std::min<int64_t>(int64_t(max_q_len) * (Hq / Hkv), 32);
  return n_split > 1 ? size_t(B) * Hkv * n_split * cols * (D + 2) * sizeof(float) : 0;
}

// How a launch cuts its pairs: waves of a workgroup to a pair (column tile of
// a pair), and workgroups to a pair (with more than one, a second launch merges
// their partials).  steps: 32-key steps of the longest context; n_max: room for
// partials; least: ranges, one per wave, there have to be.
//
// A CU takes in about 58 GB/s whatever runs on it (8000 keys, D 128, us: one
// workgroup of four waves 71.7, of eight 72.3), so what shortens a long context
// is CUs, and what the launch waits for is the CUs with most to do.  Four waves
// to a pair, a workgroup of its own, as long as each has a CU to itself (at
// D = 64, whose steps and merge are shorter, two pairs to a CU).  Then two, up to
// four pairs to a CU, where all workgroups run at once; and four again, quarters
// of the load, where twos or whole pairs leave some CUs twice the work of others:
// up to half as many pairs again as two (four) to a CU, from 8 (32) steps on,
// where the merges pay.  8 kv heads, D 128, contexts of 0.85 to 1 of these
// lengths, unshared and (60% of the keys shared by all requests), us by one, two,
// four:
//   320 pairs of 2400 keys   118, 70.7, 80.1 (86.0, 46.0, 50.1)
//   512 of 1056              42.2, 40.9, 41.0 (41.3, 24.7, 24.8)
//   576 of 300               16.9, 21.0, 18.8 (15.6, 16.4, 14.9)
//   576 of 1000              47.4, 57.3, 48.8 (40.4, 39.9, 31.9)
//   768 of 800               46.1, 50.8, 45.9 (35.9, 33.1, 27.9)
//   800 of 1056              75.8, 80.9, 81.5 (46.7, 42.6, 42.3)
//   1024 of 1056             95.4, 95.1, 95.6 (53.6, 43.7, 45.0)
//   1248 of 2000             277, 242, 226  (of 2400: 211, 163, 146)
//   1536 of 2000             302, 274, 277  (of 2400: 215, 177, 177)
// D 64, 4 kv heads: 264 of 300 9.3, 6.9, 6.5; 320 of 1056 27.0, 17.0, 17.6 (25.9,
// 15.4, 13.5); 600 of 500 16.0, 16.9, 15.1 (14.0, 13.0, 11.0).  Eight gain only
// at D = 64 where a pair has one workgroup (4 requests, 2 kv heads, 16 K keys
// 86.5 -> 73.8; 64 of 800 8.9 -> 8.2; not on few pairs of that many: 20 of 830
// keys 7.5 -> 7.8).
//
// A wave's steps follow each other at about 1 us (D = 64: 0.55) and the second
// launch costs 3 to 3.5 us, so workgroups are added -- one to a CU, at most 16 --
// where they take kGain steps off every wave, and no more of them than keep that
// step count; at D = 64 from 32 steps on (26 steps: 7.5 -> 7.7, and 10.9 -> 12.7
// for a step issued with its append, where the host's third launch shows); below
// three to a pair (over 85 pairs) the reads are the bound and two pay only past
// 128 steps.  us, one workgroup -> this rule, 8 kv heads, D 128
// (D 64 with 2 kv heads): 1 request of 604 keys 9.2 -> 8.5, of 8000 71.7 -> 13.2;
// 4 of 1000 12.8 -> 8.7 (8.2 -> 7.2), of 2100 22.9 -> 12.4, of 4000 38.5 -> 16.9
// (22.1 -> 8.3); 8 of 2100 23.4 -> 17.2; 16 of 8000 110.8 -> 95.3; left at one
// because it loses: 4 of 400 (7.5 -> 8.0), 16 of 2100 (24.5 -> 26.8).
struct Plan {
  int waves, groups;
};

static Plan decode_plan(int64_t pairs, int64_t steps, int D, int64_t n_max, int64_t least) {
  const int64_t cus = device_cus();
  const bool four = pairs <= (D == 64 ? 2 : 1) * cus || (pairs > 2 * cus && pairs <= 3 * cus && steps >= 8) ||
                    (pairs > 4 * cus && pairs <= 6 * cus && steps >= 32);
  int64_t w = four ? 4 : pairs <= 4 * cus ? 2 : 1, n = 1;
  while (w > steps) w /= 2;
  if (w == 4 && cus / pairs >= 3) {
    const int64_t room = std::min<int64_t>({cus / pairs, n_max, kMaxGroups});
    const int64_t alone = (steps + 3) / 4, each = (alone + room - 1) / room;  // steps a wave
    const int64_t kGain = D == 64 ? 6 : 4;
    if (alone - each >= kGain && (D == 128 || steps >= 32)) n = (steps + 4 * each - 1) / (4 * each);
  } else if (w == 4 && cus / pairs == 2 && n_max >= 2 && steps > 128) {
    n = 2;
  }
  if (D == 64 && w == 4 && n == 1 && pairs <= cus && steps >= (cus / pairs >= 3 ? 32 : 24)) w = 8;
  // More ranges asked for (up to one a step): one workgroup of eight waves if
  // that is enough, else of four while they have a CU each (us, 1 request of 400
  // keys, 8 kv heads: 8 ranges as 1 x 8 8.4, 2 x 4 9.1; 16 as 2 x 8 9.8, 4 x 4
  // 7.9), else of eight, which leaves fewer partials.
  least = std::min(least, steps);
  if (n * w < least) {
    if (pairs * ((least + 7) / 8) <= cus && (least <= 8 || pairs * ((least + 3) / 4) > cus)) w = 8;
    n = std::max(n, (least + w - 1) / w);
  }
  return {int(w), int(n)};
}

int decode_max_groups(int64_t pairs, int64_t steps) {
  if (pairs <= 0) return 1;
  const int64_t n = std::min<int64_t>(device_cus() / pairs, kMaxGroups);
  return int(std::max<int64_t>(1, steps > 0 ? std::min(n, (steps + 3) / 4) : n));
}

size_t decode_auto_bytes(int64_t pairs, int max_q_len, int Hq, int Hkv, int D) {
  const int64_t sets = std::min<int64_t>(pairs * kMaxGroups, device_cus());
  const int64_t cols = std::min<int64_t>(int64_t(max_q_len) * (Hq / Hkv), 32);
  return size_t(sets) * cols * (D + 2) * sizeof(float);
}

int launch_decode_attn(const uint16_t* q, const uint16_t* k_pool, const uint16_t* v_pool, int num_blocks,
                       const int32_t* block_tables, int max_blocks, const int32_t* cu_q,
                       const int32_t* seq_lens, int B, int max_q_len, int Hq, int Hkv, int D,
                       float scale_log2, uint16_t* out, int n_split, bool automatic, float* part,
                       void* stream_ptr) {
  hipStream_t stream = static_cast<hipStream_t>(stream_ptr);
  const int64_t all_cols = int64_t(max_q_len) * (Hq / Hkv);
  const int64_t n_ct = (all_cols + 31) / 32;
  if (n_split < 1 || n_split > kMaxSplit || (n_split > 1 && n_ct > 1))
    return set_error(ILPC_EINVAL, "decode attention: bad split");
  if (device_cus() <= 0) return set_error(ILPC_EHIP, "decode attention: cannot query the device");
  const int cols_cap = int(std::min<int64_t>(all_cols, 32));
  const int64_t pairs = int64_t(B) * Hkv * n_ct;
  const int64_t steps = (int64_t(max_blocks) * kBlock + kStepKeys - 1) / kStepKeys;
  const Plan plan = decode_plan(pairs, steps, D, n_split, automatic ? 1 : n_split);
  const int w = plan.waves;
  n_split = plan.groups;
  if (n_split > 1 && !part) return set_error(ILPC_EINVAL, "decode attention: no room for partial results");
  float* part_ml = part ? part + size_t(B) * Hkv * n_split * cols_cap * D : nullptr;
  const int64_t items = pairs * n_split, per_group = group_waves(w) / w;
  const int64_t groups = (items + per_group - 1) / per_group;
  if (items > INT32_MAX) return set_error(ILPC_EUNSUP, "decode attention: batch too large");
  const dim3 grid{unsigned(groups)}, block{unsigned(64 * group_waves(w))};
  auto launch = [&](auto kernel) {
    hipLaunchKernelGGL(kernel, grid, block, 0, stream, q, k_pool, v_pool, num_blocks, block_tables, max_blocks,
                       cu_q, seq_lens, B, max_q_len, Hq, Hkv, scale_log2, out, int(n_ct), n_split, cols_cap, part,
                       part_ml);
  };
  if (D == 128) {
    if (w == 1) launch(decode_attn_kernel<128, 1>);
    else if (w == 2) launch(decode_attn_kernel<128, 2>);
    else if (w == 4) launch(decode_attn_kernel<128, 4>);
    else launch(decode_attn_kernel<128, 8>);
  } else {
    if (w == 1) launch(decode_attn_kernel<64, 1>);
    else if (w == 2) launch(decode_attn_kernel<64, 2>);
    else if (w == 4) launch(decode_attn_kernel<64, 4>);
    else launch(decode_attn_kernel<64, 8>);
  }
  hipError_t e = hipGetLastError();
  if (e == hipSuccess && n_split > 1) {
    const dim3 cgrid{unsigned((int64_t(B) * Hkv * cols_cap + kCombineWaves - 1) / kCombineWaves)};
    const dim3 cblock{64 * kCombineWaves};
    if (D == 128)
      hipLaunchKernelGGL(decode_combine_kernel<128>, cgrid, cblock, 0, stream, part, part_ml, cu_q, seq_lens,
                         max_blocks, B, max_q_len, Hq, Hkv, n_split, cols_cap, out);
    else
      hipLaunchKernelGGL(decode_combine_kernel<64>, cgrid, cblock, 0, stream, part, part_ml, cu_q, seq_lens,
                         max_blocks, B, max_q_len, Hq, Hkv, n_split, cols_cap, out);
    e = hipGetLastError();
  }
  if (e != hipSuccess)
    return set_error(ILPC_EHIP, "decode attention: launch failed: %s", hipGetErrorString(e));
  return ILPC_OK;
}

}  // namespace ilpc

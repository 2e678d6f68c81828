// Internal helpers shared by the library's translation units (not part of the ABI).
#pragma once

#include <cstdarg>
#include <cstddef>
#include <cstdint>

namespace ilpc {

// Records a message for ilpc_last_error() on the calling thread and returns `code`.
int set_error(int code, const char* fmt, ...) __attribute__((format(printf, 2, 3)));

// Paged attention for few query columns (q_len * Hq / Hkv per request), 32 to
// a wave: one wave per (request, kv head) and column tile, more (each a range
// of the keys) where these are too few to fill the chip.  Arguments as for
// ilpc_paged_prefill_attn, already checked; scale_log2 = softmax scale *
// log2(e); stream is a hipStream_t.
// With 1 < n_split <= kMaxSplit (at most 32 columns a request) each pair's
// keys are cut into at least n_split ranges, one per wave; the waves of a
// workgroup merge theirs, and the partial states of a pair's workgroups go to
// `part` (decode_split_bytes() bytes, 16-byte aligned) and are merged by a
// second launch.  With `automatic` n_split only bounds the workgroups a pair
// may take (the room in `part`).
int launch_decode_attn(const uint16_t* q, const uint16_t* k_pool, const uint16_t* v_pool, int num_blocks,
                       const int32_t* block_tables, int max_blocks, const int32_t* cu_q,
                       const int32_t* seq_lens, int B, int max_q_len, int Hq, int Hkv, int D,
                       float scale_log2, uint16_t* out, int n_split, bool automatic, float* part, void* stream);
size_t decode_split_bytes(int B, int max_q_len, int Hq, int Hkv, int D, int n_split);
constexpr int kMaxSplit = 64;

// The most workgroups to a (request, kv head) pair an automatic launch takes
// (steps: 32-key steps of the longest context; 0: any), and the bytes of
// partial states with which no batch of at most `pairs` pairs takes fewer.
int decode_max_groups(int64_t pairs, int64_t steps);
size_t decode_auto_bytes(int64_t pairs, int max_q_len, int Hq, int Hkv, int D);

// Compute units of the current device, looked up once per device (0: unknown).
int device_cus();

}  // namespace ilpc

// Internal declarations shared by the translation units of libdfa (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dfa.h"

namespace dfa {

// Launch wrappers: every one validates nothing (the ABI layer did) and returns a dfa_status.
int launch_merge(const dfa_merge_desc& md, const dfa_merge_pair* pairs, int n, hipStream_t st);
// Several partials (o_b, lse_b) into one (o, lse) each.  What becomes of that, `accumulate`: it is only written; it takes part as
// the state that a forward continues from (lse = -inf or no number: empty, whatever its o); or as an operand of a merge
// (lse = -inf: weight zero, its o counts and is zero).
enum { MERGE_WRITE, MERGE_CONTINUE, MERGE_ALL };
struct MergeShape { int heads, rows, d; bool b_bf16; int64_t b_sh, b_ss, lb_sh; };
struct MergeGroup { void* o; float* lse; int64_t o_sh, o_ss, l_sh; int first, n, accumulate, o_bf16; };
struct MergePart { const void* o; const float* lse; };
int launch_merge_parts(const MergeShape& sh, const MergeGroup* groups, int n, const MergePart* parts, hipStream_t st);
int launch_delta(const dfa_shape& sh, const void* o, const void* dO, float* delta, hipStream_t st);
int launch_fill_zero_rows(float* p, int heads, int rows, int d, int64_t stride_h, int64_t stride_s,
                          hipStream_t st);
int launch_fill_empty_fwd(const dfa_shape& sh, void* o, float* lse, hipStream_t st);

// The pairs of a launch share the shape and write disjoint outputs (backward: all select the same ones).
// ws: scratch of bwd_*_workspace() bytes (0: none is used), or null; with less the work is divided into fewer parts.
int launch_fwd_f32(const dfa_shape& sh, const dfa_fwd_pair* pairs, int n, hipStream_t st);
// sequence: one causal call of all chunks, which stands for their pairs.
int launch_bwd_f32(const dfa_shape& sh, const dfa_bwd_pair* pairs, int n, bool sequence, void* ws, int64_t ws_bytes,
                   hipStream_t st);
int64_t bwd_f32_workspace(const dfa_shape& sh, int n, bool dq, bool dk, bool sequence);

int launch_fwd_bf16(const dfa_shape& sh, const dfa_fwd_pair* pairs, int n, hipStream_t st);

// Spans.  Their keys are cut in parts where that pays; the parts' results take ws (part_floats() each) and are merged.
int launch_span_bf16(const dfa_shape& sh, const dfa_fwd_span* spans, int n, void* ws, int64_t ws_bytes, hipStream_t st);
int launch_span_f32(const dfa_shape& sh, const dfa_fwd_span* spans, int n, void* ws, int64_t ws_bytes, hipStream_t st);
int64_t span_bf16_workspace(const dfa_shape& sh, const dfa_fwd_span* spans, int n);
int64_t span_f32_workspace(const dfa_shape& sh, const dfa_fwd_span* spans, int n);
int launch_bwd_bf16(const dfa_shape& sh, const dfa_bwd_pair* pairs, int n, void* ws, int64_t ws_bytes,
                    hipStream_t st);
int64_t bwd_bf16_workspace(const dfa_shape& sh, int n, bool dq, bool dk);

// The forms that these calls take (dfa_form).
dfa_form fwd_bf16_form(const dfa_shape& sh, int n);
dfa_form fwd_f32_form(const dfa_shape& sh, int n);
dfa_form bwd_bf16_form(const dfa_shape& sh, int n, bool dq, bool dk, int64_t ws_bytes);
dfa_form bwd_f32_form(const dfa_shape& sh, int n, bool dq, bool dk, int64_t ws_bytes, bool sequence);
dfa_form span_bf16_form(const dfa_shape& sh, const dfa_fwd_span* spans, int n, int64_t ws_bytes);
dfa_form span_f32_form(const dfa_shape& sh, const dfa_fwd_span* spans, int n, int64_t ws_bytes);

// Which item a workgroup takes.  Workgroup ids go round-robin over the 8 XCDs, and in order: a workgroup waits for
// its XCD even if another is free.  Every XCD gets a contiguous range of (head, tile) items, so that the tiles of a
// head share its operands in one L2 - and, where the tiles of a causal chunk are of different length, every
// XCD whole heads.  (Plain ids put every eighth tile on the same XCD: a causal call then took as long as a full
// one: fp32 backward of 32 heads x 4096, d = 128, 7.2 ms against 4.8.)
// snake: causal calls of one or two heads, where a range would hold long or short tiles only: ids in rows of
// eight, every second row backwards, give each XCD the same mix (fp32 backward of one head x 4096 495 -> 387 us,
// 2 over 1 heads 743 -> 675; from four heads on ranges are the better ones: 4 heads 938 against 1162).  bf16, ranges
// against this: forward of one head x 16384 221 / 215 us, x 32768 800 / 515, of two heads x 4096 54 / 58, x 16384 383 / 282, x
// 32768 956 / 704; backward of one head x 16384 348 / 354, x 32768 1225 / 927, of two x 16384 553 / 592, x 32768 2270 / 1890;
// no difference below 4096 rows.
struct XcdMap { int total, per_xcd, snake; };
inline XcdMap xcd_map(int64_t total, int causal, int64_t groups) {
  return XcdMap{static_cast<int>(total), static_cast<int>((total + 7) / 8), causal && groups <= 2};
}
inline int64_t xcd_blocks(const XcdMap& m) { return static_cast<int64_t>(m.per_xcd) * 8; }
__device__ __forceinline__ int xcd_item(const XcdMap& m, int bid) {      // >= total: none
  const int x = bid & 7, i = bid >> 3;
  return m.snake ? i * 8 + (i & 1 ? 7 - x : x) : x * m.per_xcd + i;
}

inline int hip_status(hipError_t e) { return e == hipSuccess ? DFA_OK : DFA_ERR_HIP; }
inline int last_launch_status() { return hip_status(hipGetLastError()); }

}  // namespace dfa

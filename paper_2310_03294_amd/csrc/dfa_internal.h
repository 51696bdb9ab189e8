// Internal declarations shared by the translation units of libdfa (not part of the ABI).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "dfa.h"

namespace dfa {

// Launch wrappers: every one validates nothing (the ABI layer did) and returns a dfa_status.
int launch_merge(const dfa_merge_desc& md, const dfa_merge_pair* pairs, int n, hipStream_t st);
int launch_delta(const dfa_shape& sh, const void* o, const void* dO, float* delta, hipStream_t st);
int launch_fill_zero_rows(float* p, int heads, int rows, int d, int64_t stride_h, int64_t stride_s,
                          hipStream_t st);
int launch_fill_empty_fwd(const dfa_shape& sh, void* o, float* lse, hipStream_t st);

// The pairs of a launch share the shape and write disjoint outputs (backward: all select the same ones).
// ws: scratch of bwd_bf16_workspace() bytes (0: none is used), or null; with less the work is divided into fewer parts.
int launch_fwd_f32(const dfa_shape& sh, const dfa_fwd_pair* pairs, int n, hipStream_t st);
int launch_bwd_f32(const dfa_shape& sh, const dfa_bwd_pair* pairs, int n, hipStream_t st);

int launch_fwd_bf16(const dfa_shape& sh, const dfa_fwd_pair* pairs, int n, hipStream_t st);
int launch_bwd_bf16(const dfa_shape& sh, const dfa_bwd_pair* pairs, int n, void* ws, int64_t ws_bytes,
                    hipStream_t st);
int64_t bwd_bf16_workspace(const dfa_shape& sh, int n, bool dq, bool dk);

inline int hip_status(hipError_t e) { return e == hipSuccess ? DFA_OK : DFA_ERR_HIP; }
inline int last_launch_status() { return hip_status(hipGetLastError()); }

}  // namespace dfa

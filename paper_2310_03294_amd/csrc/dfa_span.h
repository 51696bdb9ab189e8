// Spans of keys (dfa_span_fwd): how they are cut in parts, and the launches of the parts and of the merges that follow.
#pragma once

#include <algorithm>

#include "dfa_internal.h"

namespace dfa {

constexpr int MAX_SPAN_PARTS = 16;
constexpr int64_t MAX_SPAN_BYTES = int64_t{128} << 20;      // of the parts' results

// A part of a span as the kernels take it.  off: key kv of the part is visible to query row i if kv <= i + off.
struct SpanPart {
  const void *q, *k, *v;
  void* o;
  float* lse;
  int64_t o_sh, o_ss, l_sh;
  int n_keys, off, accumulate, o_bf16;
};

// One chunk and its own keys alone: a sequence, which stands for the pairs of several workers' chunks.
inline bool is_sequence(const dfa_shape& sh, const dfa_fwd_span* spans, int n) {
  return n == 1 && spans[0].own && spans[0].n_keys == sh.s_q;
}

// Keys of a span before the query chunk's own.
inline int64_t keys_before(const dfa_shape& sh, const dfa_fwd_span& x) { return x.own ? x.n_keys - sh.s_q : x.n_keys; }
// Parts that a span is cut in, at most `parts`: of 128 keys at least, and none begins among the chunk's own keys (a workgroup
// always has keys that its first row sees).
inline int span_parts(const dfa_shape& sh, const dfa_fwd_span& x, int parts) {
  const int64_t most = keys_before(sh, x) / 128 + (x.own ? 1 : 0);
  return static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(parts, most)));
}
// Where part i of `parts` begins: at a multiple of 128 keys, equal shares of the visible ones (the chunk's own count half).
inline int span_cut(const dfa_shape& sh, const dfa_fwd_span& x, int parts, int i) {
  const int64_t before = keys_before(sh, x), visible = before + (x.own ? sh.s_q / 2 : 0);
  const int64_t tiles = before / 128;
  if (i == 0) return 0;
  if (i == parts) return x.n_keys;
  // (never an empty part: part i begins at tile i or later, and leaves the parts after it a tile each)
  return static_cast<int>(std::min<int64_t>(std::max<int64_t>(visible * i / parts / 128, i), tiles - (parts - 1 - i) + (x.own ? 0 : -1)) * 128);
}

inline int64_t part_floats(const dfa_shape& sh) {
  const int64_t o = static_cast<int64_t>(sh.h_q) * sh.s_q * sh.d, lse = static_cast<int64_t>(sh.h_q) * sh.s_q;
  return o + (lse + 3) / 4 * 4;      // keeps the next part's o on 16 bytes
}
// Bytes of the parts' results of a cut in at most `parts`.
inline int64_t parts_bytes(const dfa_shape& sh, const dfa_fwd_span* spans, int n, int parts) {
  int64_t results = 0;
  for (int i = 0; i < n; ++i) {
    const int np = span_parts(sh, spans[i], parts);
    results += np > 1 ? np : 0;
  }
  return results * part_floats(sh) * 4;
}

// What a launch does: workgroups, their keys in whole tiles, the longest walk, bytes of the parts' results; cut: whether any of its
// spans is in more than one part.
struct LaunchWork { int64_t workgroups; double keys, longest; int64_t part_bytes; bool cut; };
// The launches that run_spans makes of a cut in at most `parts`, up to `per` parts to a launch, with `blocks` workgroups per part:
// us_of(LaunchWork) summed up.
template <class F>
double sum_of_launches(const dfa_shape& sh, const dfa_fwd_span* spans, int n, int parts, int per, int64_t blocks, int tile, F us_of) {
  LaunchWork w{0, 0., 0., 0, false};
  double us = 0;
  int count = 0;
  for (int i = 0; i < n; ++i) {
    const int np = span_parts(sh, spans[i], parts);
    if (count + np > per) {
      us += us_of(w);
      w = LaunchWork{0, 0., 0., 0, false};
      count = 0;
    }
    for (int j = 0, k0 = 0; j < np; ++j) {
      const int k1 = span_cut(sh, spans[i], np, j + 1);
      const double keys = static_cast<double>((k1 - k0 + tile - 1) / tile * tile);
      w.longest = std::max(w.longest, keys);
      w.keys += blocks * (keys - (j + 1 == np && spans[i].own ? sh.s_q / 2 / tile * tile : 0));
      k0 = k1;
    }
    w.workgroups += blocks * np;
    if (np > 1) { w.part_bytes += np * part_floats(sh) * 4; w.cut = true; }
    count += np;
  }
  return us + us_of(w);
}
constexpr int SPAN_CUTS[] = {1, 2, 3, 4, 6, 8, 12, MAX_SPAN_PARTS};      // numbers of parts that are tried

// The spans' parts, up to PER to a launch (launch(parts, count)), each launch followed by the merge of the spans that were
// cut, through ws.
template <int PER, class Launch>
int run_spans(const dfa_shape& sh, const dfa_fwd_span* spans, int n, int parts, void* ws, hipStream_t st, Launch launch) {
  static_assert(PER >= MAX_SPAN_PARTS);
  const int64_t kv_row = sh.kv_stride_s * (sh.dtype == DFA_BF16 ? 2 : 4);
  const int64_t heads_rows = static_cast<int64_t>(sh.h_q) * sh.s_q;
  SpanPart todo[PER];
  MergeGroup groups[PER];
  MergePart results[PER];
  int count = 0, n_groups = 0, n_results = 0;
  float* next = static_cast<float*>(ws);
  auto flush = [&] {
    int rc = launch(todo, count);
    if (rc == DFA_OK && n_groups)
      rc = launch_merge_parts({sh.h_q, sh.s_q, sh.d, false, static_cast<int64_t>(sh.s_q) * sh.d, sh.d, sh.s_q}, groups, n_groups,
                              results, st);
    count = n_groups = n_results = 0;
    next = static_cast<float*>(ws);
    return rc;
  };
  for (int i = 0; i < n; ++i) {
    const dfa_fwd_span& x = spans[i];
    const int np = span_parts(sh, x, parts), own_off = x.own ? x.n_keys - sh.s_q : 1 << 30;
    if (count + np > PER) {
      const int rc = flush();
      if (rc) return rc;
    }
    if (np > 1)
      groups[n_groups++] = {x.o, x.lse, x.o_stride_h, x.o_stride_s, x.lse_stride_h, n_results, np,
                            x.accumulate ? MERGE_CONTINUE : MERGE_WRITE, sh.o_dtype == DFA_BF16};
    for (int j = 0; j < np; ++j) {
      const int k0 = span_cut(sh, x, np, j);
      SpanPart& y = todo[count++];
      y = {x.q, static_cast<const char*>(x.k) + k0 * kv_row, static_cast<const char*>(x.v) + k0 * kv_row, x.o, x.lse,
           x.o_stride_h, x.o_stride_s, x.lse_stride_h, span_cut(sh, x, np, j + 1) - k0, x.own ? own_off - k0 : own_off,
           x.accumulate != 0, sh.o_dtype == DFA_BF16};
      if (np > 1) {
        y.o = next; y.lse = next + heads_rows * sh.d;
        y.o_sh = static_cast<int64_t>(sh.s_q) * sh.d; y.o_ss = sh.d; y.l_sh = sh.s_q; y.accumulate = y.o_bf16 = 0;
        results[n_results++] = {y.o, y.lse};
        next += part_floats(sh);
      }
    }
  }
  return count ? flush() : DFA_OK;
}

}  // namespace dfa

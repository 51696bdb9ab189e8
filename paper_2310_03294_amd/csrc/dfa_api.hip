// C-ABI layer: argument validation on the host, then dispatch to the kernel launchers.
#include "dfa_internal.h"

namespace {

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }
bool mult8(int64_t x) { return (x & 7) == 0; }

// spans: a query chunk's own keys may have others before them
int check_common(const dfa_shape* sh, bool spans = false) {
  if (!sh) return DFA_ERR_NULL;
  if (sh->reserved != 0) return DFA_ERR_ARG;
  if (sh->dtype != DFA_BF16 && sh->dtype != DFA_F32) return DFA_ERR_DTYPE;
  if (sh->o_dtype != DFA_BF16 && sh->o_dtype != DFA_F32) return DFA_ERR_DTYPE;
  if (sh->h_q < 1 || sh->h_kv < 1 || sh->h_q % sh->h_kv != 0) return DFA_ERR_SHAPE;
  if (sh->h_q > 65535) return DFA_ERR_SHAPE;
  if (sh->s_q < 0 || sh->s_k < 0) return DFA_ERR_SHAPE;
  if (sh->d != 64 && sh->d != 128) return DFA_ERR_SHAPE;
  if (sh->dtype == DFA_BF16 && sh->d != 128) return DFA_ERR_SHAPE;
  if (sh->causal != 0 && sh->causal != 1) return DFA_ERR_ARG;
  if (sh->causal && (spans ? sh->s_k < sh->s_q : sh->s_q != sh->s_k)) return DFA_ERR_ARG;
  if (!(sh->scale == sh->scale) || sh->scale <= 0.f) return DFA_ERR_ARG;
  return DFA_OK;
}

bool stride_ok(int64_t sh_, int64_t ss, int d, int rows) {
  if (ss < d || !mult8(ss) || !mult8(sh_)) return false;
  // head offsets are formed in 64 bits from at most 65535 heads: keep them far from overflow
  if (sh_ < 0 || sh_ > (int64_t{1} << 40)) return false;
  // the kernels address one head's slice of a chunk with 32-bit byte offsets (fp32 at most):
  // rows * ss * 4 < 2^31, compared without forming a product that could overflow
  if (rows > 0 && ss > ((int64_t{1} << 29) - 1) / rows) return false;
  return true;
}

// head stride of an [heads, rows] fp32 vector (lse, D)
bool row_stride_ok(int64_t sh_, int rows) { return sh_ >= rows && sh_ <= (int64_t{1} << 40); }

}  // namespace

extern "C" const char* dfa_status_str(int s) {
  switch (s) {
    case DFA_OK: return "DFA_OK";
    case DFA_ERR_NULL: return "DFA_ERR_NULL: required pointer is NULL";
    case DFA_ERR_SHAPE: return "DFA_ERR_SHAPE: unsupported size, stride or alignment";
    case DFA_ERR_DTYPE: return "DFA_ERR_DTYPE: unsupported dtype";
    case DFA_ERR_ARG: return "DFA_ERR_ARG: inconsistent arguments";
    case DFA_ERR_HIP: return "DFA_ERR_HIP: HIP runtime error";
    default: return "unknown dfa_status";
  }
}

extern "C" int dfa_version(void) { return 100; }

extern "C" int dfa_chunk_fwd_batch(const dfa_shape* sh, const dfa_fwd_pair* pairs, int32_t n_pairs, void* stream) {
  int rc = check_common(sh);
  if (rc != DFA_OK) return rc;
  if (n_pairs < 0) return DFA_ERR_ARG;
  if (n_pairs == 0) return DFA_OK;
  if (!pairs) return DFA_ERR_NULL;
  const bool have_kv = sh->s_k > 0;   // an empty key/value chunk may come with NULL k, v
  for (int i = 0; i < n_pairs; ++i) {
    const dfa_fwd_pair& p = pairs[i];
    if (!p.q || !p.o || !p.lse || (have_kv && (!p.k || !p.v))) return DFA_ERR_NULL;
    if (!aligned16(p.q) || !aligned16(p.o) || (have_kv && (!aligned16(p.k) || !aligned16(p.v)))) return DFA_ERR_SHAPE;
    if (!stride_ok(p.o_stride_h, p.o_stride_s, sh->d, sh->s_q) || !row_stride_ok(p.lse_stride_h, sh->s_q))
      return DFA_ERR_SHAPE;
  }
  if (!stride_ok(sh->q_stride_h, sh->q_stride_s, sh->d, sh->s_q) ||
      !stride_ok(sh->kv_stride_h, sh->kv_stride_s, sh->d, sh->s_k))
    return DFA_ERR_SHAPE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (sh->s_q == 0) return DFA_OK;
  if (sh->s_k == 0) {
    for (int i = 0; i < n_pairs; ++i) {
      if (pairs[i].accumulate) continue;
      dfa_shape one = *sh;
      one.o_stride_h = pairs[i].o_stride_h; one.o_stride_s = pairs[i].o_stride_s;
      one.lse_stride_h = pairs[i].lse_stride_h;
      rc = dfa::launch_fill_empty_fwd(one, pairs[i].o, pairs[i].lse, st);
      if (rc) return rc;
    }
    return DFA_OK;
  }
  return sh->dtype == DFA_F32 ? dfa::launch_fwd_f32(*sh, pairs, n_pairs, st) : dfa::launch_fwd_bf16(*sh, pairs, n_pairs, st);
}

namespace {
int check_spans(const dfa_shape* sh, const dfa_fwd_span* spans, int32_t n) {
  dfa_shape s = *sh;
  s.causal = 0; s.s_k = 0;
  int rc = check_common(&s);
  if (rc != DFA_OK) return rc;
  if (n < 0) return DFA_ERR_ARG;
  if (n > 0 && !spans) return DFA_ERR_NULL;
  for (int i = 0; i < n; ++i) {
    const dfa_fwd_span& x = spans[i];
    if (x.n_keys < 1) return DFA_ERR_SHAPE;
    if (x.reserved != 0 || (x.own && x.n_keys < sh->s_q)) return DFA_ERR_ARG;
    if (!stride_ok(sh->kv_stride_h, sh->kv_stride_s, sh->d, x.n_keys)) return DFA_ERR_SHAPE;
  }
  return DFA_OK;
}
}  // namespace

extern "C" int dfa_span_fwd(const dfa_shape* sh, const dfa_fwd_span* spans, int32_t n_spans, void* workspace,
                            int64_t workspace_bytes, void* stream) {
  if (!sh) return DFA_ERR_NULL;
  const int rc = check_spans(sh, spans, n_spans);
  if (rc != DFA_OK) return rc;
  for (int i = 0; i < n_spans; ++i) {
    const dfa_fwd_span& p = spans[i];
    if (!p.q || !p.k || !p.v || !p.o || !p.lse) return DFA_ERR_NULL;
    if (!aligned16(p.q) || !aligned16(p.k) || !aligned16(p.v) || !aligned16(p.o)) return DFA_ERR_SHAPE;
    if (!stride_ok(p.o_stride_h, p.o_stride_s, sh->d, sh->s_q) || !row_stride_ok(p.lse_stride_h, sh->s_q)) return DFA_ERR_SHAPE;
  }
  if (!stride_ok(sh->q_stride_h, sh->q_stride_s, sh->d, sh->s_q)) return DFA_ERR_SHAPE;
  if (workspace_bytes < 0) return DFA_ERR_ARG;
  if (!aligned16(workspace)) return DFA_ERR_SHAPE;
  if (sh->s_q == 0 || n_spans == 0) return DFA_OK;
  hipStream_t st = static_cast<hipStream_t>(stream);
  return sh->dtype == DFA_F32 ? dfa::launch_span_f32(*sh, spans, n_spans, workspace, workspace_bytes, st)
                              : dfa::launch_span_bf16(*sh, spans, n_spans, workspace, workspace_bytes, st);
}

extern "C" int64_t dfa_span_fwd_workspace(const dfa_shape* sh, const dfa_fwd_span* spans, int32_t n_spans) {
  if (!sh) return DFA_ERR_NULL;
  const int rc = check_spans(sh, spans, n_spans);
  if (rc != DFA_OK) return rc;
  if (sh->s_q == 0 || n_spans == 0) return 0;
  return sh->dtype == DFA_F32 ? dfa::span_f32_workspace(*sh, spans, n_spans) : dfa::span_bf16_workspace(*sh, spans, n_spans);
}

extern "C" int dfa_chunk_fwd_form(const dfa_shape* sh, int32_t n_pairs, dfa_form* form) {
  const int rc = check_common(sh);
  if (rc != DFA_OK) return rc;
  if (!form) return DFA_ERR_NULL;
  if (n_pairs < 1) return DFA_ERR_ARG;
  if (sh->s_q == 0 || sh->s_k == 0) return DFA_ERR_SHAPE;
  *form = sh->dtype == DFA_F32 ? dfa::fwd_f32_form(*sh, n_pairs) : dfa::fwd_bf16_form(*sh, n_pairs);
  return DFA_OK;
}

extern "C" int dfa_span_fwd_form(const dfa_shape* sh, const dfa_fwd_span* spans, int32_t n_spans, int64_t workspace_bytes,
                                 dfa_form* form) {
  if (!sh || !form) return DFA_ERR_NULL;
  const int rc = check_spans(sh, spans, n_spans);
  if (rc != DFA_OK) return rc;
  if (n_spans < 1 || workspace_bytes < 0) return DFA_ERR_ARG;
  if (sh->s_q == 0) return DFA_ERR_SHAPE;
  *form = sh->dtype == DFA_F32 ? dfa::span_f32_form(*sh, spans, n_spans, workspace_bytes)
                               : dfa::span_bf16_form(*sh, spans, n_spans, workspace_bytes);
  return DFA_OK;
}

namespace {
int chunk_fwd(const dfa_shape* sh, const void* q, const void* k, const void* v,
              void* o, float* lse, int accumulate, void* stream) {
  if (!sh) return DFA_ERR_NULL;
  const dfa_fwd_pair p{q, k, v, o, lse, sh->o_stride_h, sh->o_stride_s, sh->lse_stride_h, accumulate, 0};
  return dfa_chunk_fwd_batch(sh, &p, 1, stream);
}
}  // namespace

extern "C" int dfa_chunk_fwd(const dfa_shape* sh, const void* q, const void* k, const void* v,
                             void* o, float* lse, void* stream) {
  return chunk_fwd(sh, q, k, v, o, lse, 0, stream);
}

extern "C" int dfa_chunk_fwd_acc(const dfa_shape* sh, const void* q, const void* k, const void* v,
                                 void* o, float* lse, void* stream) {
  return chunk_fwd(sh, q, k, v, o, lse, 1, stream);
}

extern "C" int dfa_merge_batch(const dfa_merge_desc* md, const dfa_merge_pair* pairs, int32_t n_pairs, void* stream) {
  if (!md) return DFA_ERR_NULL;
  if (md->heads < 0 || md->rows < 0 || md->heads > 65535) return DFA_ERR_SHAPE;
  if (md->d != 64 && md->d != 128) return DFA_ERR_SHAPE;
  if (md->o_dtype != DFA_BF16 && md->o_dtype != DFA_F32) return DFA_ERR_DTYPE;
  if (n_pairs < 0) return DFA_ERR_ARG;
  if (n_pairs > 0 && !pairs) return DFA_ERR_NULL;
  for (int i = 0; i < n_pairs; ++i) {
    const dfa_merge_pair& p = pairs[i];
    if (!p.o_a || !p.lse_a || !p.o_b || !p.lse_b) return DFA_ERR_NULL;
    if (!aligned16(p.o_a) || !aligned16(p.o_b)) return DFA_ERR_SHAPE;
  }
  if (!stride_ok(md->a_stride_h, md->a_stride_s, md->d, md->rows) ||
      !stride_ok(md->b_stride_h, md->b_stride_s, md->d, md->rows))
    return DFA_ERR_SHAPE;
  if (!row_stride_ok(md->lse_a_stride_h, md->rows) || !row_stride_ok(md->lse_b_stride_h, md->rows)) return DFA_ERR_SHAPE;
  for (int i = 0; i < n_pairs; ++i)
    if (pairs[i].o_a == pairs[i].o_b || pairs[i].lse_a == pairs[i].lse_b) return DFA_ERR_ARG;
  if (md->rows == 0 || md->heads == 0 || n_pairs == 0) return DFA_OK;
  return dfa::launch_merge(*md, pairs, n_pairs, static_cast<hipStream_t>(stream));
}

extern "C" int dfa_merge(const dfa_merge_desc* md, void* o_a, float* lse_a,
                         const void* o_b, const float* lse_b, void* stream) {
  const dfa_merge_pair p{o_a, lse_a, o_b, lse_b};
  return dfa_merge_batch(md, &p, 1, stream);
}

extern "C" int dfa_delta(const dfa_shape* sh, const void* o, const void* dO, float* delta, void* stream) {
  int rc = check_common(sh);
  if (rc != DFA_OK) return rc;
  if (!o || !dO || !delta) return DFA_ERR_NULL;
  if (!aligned16(o) || !aligned16(dO)) return DFA_ERR_SHAPE;
  if (!stride_ok(sh->q_stride_h, sh->q_stride_s, sh->d, sh->s_q) ||
      !stride_ok(sh->o_stride_h, sh->o_stride_s, sh->d, sh->s_q))
    return DFA_ERR_SHAPE;
  if (!row_stride_ok(sh->lse_stride_h, sh->s_q)) return DFA_ERR_SHAPE;
  if (sh->s_q == 0) return DFA_OK;
  return dfa::launch_delta(*sh, o, dO, delta, static_cast<hipStream_t>(stream));
}

namespace {
int bwd_batch(const dfa_shape* sh, const dfa_bwd_pair* pairs, int32_t n_pairs, void* workspace, int64_t workspace_bytes,
              void* stream, bool spans) {
  int rc = check_common(sh, spans);
  if (rc != DFA_OK) return rc;
  if (n_pairs < 0) return DFA_ERR_ARG;
  if (n_pairs == 0) return DFA_OK;
  if (!pairs) return DFA_ERR_NULL;
  for (int i = 0; i < n_pairs; ++i) {
    const dfa_bwd_pair& p = pairs[i];
    if (!p.q || !p.k || !p.v || !p.lse || !p.delta || !p.dO) return DFA_ERR_NULL;
    // dq alone, (dk, dv) alone, or all three: a NULL output selects which gradients are computed
    if ((p.dk == nullptr) != (p.dv == nullptr)) return DFA_ERR_NULL;
    if (!p.dq && !p.dk) return DFA_ERR_NULL;
    if ((p.dq == nullptr) != (pairs[0].dq == nullptr) || (p.dk == nullptr) != (pairs[0].dk == nullptr)) return DFA_ERR_ARG;
    if (!aligned16(p.q) || !aligned16(p.k) || !aligned16(p.v) || !aligned16(p.dO) || !aligned16(p.dq) ||
        !aligned16(p.dk) || !aligned16(p.dv))
      return DFA_ERR_SHAPE;
  }
  if (!stride_ok(sh->q_stride_h, sh->q_stride_s, sh->d, sh->s_q) ||
      !stride_ok(sh->kv_stride_h, sh->kv_stride_s, sh->d, sh->s_k) ||
      !stride_ok(sh->dq_stride_h, sh->dq_stride_s, sh->d, sh->s_q) ||
      !stride_ok(sh->dkv_stride_h, sh->dkv_stride_s, sh->d, sh->s_k))
    return DFA_ERR_SHAPE;
  if (!row_stride_ok(sh->lse_stride_h, sh->s_q)) return DFA_ERR_SHAPE;
  if (workspace_bytes < 0) return DFA_ERR_ARG;
  if (!aligned16(workspace)) return DFA_ERR_SHAPE;
  hipStream_t st = static_cast<hipStream_t>(stream);
  if (sh->s_q == 0 || sh->s_k == 0) {
    // nothing flows through an empty pair; honour "overwrite" semantics
    for (int i = 0; i < n_pairs; ++i) {
      const dfa_bwd_pair& p = pairs[i];
      if (sh->s_q > 0 && p.dq && !p.accumulate_dq) {
        rc = dfa::launch_fill_zero_rows(p.dq, sh->h_q, sh->s_q, sh->d, sh->dq_stride_h, sh->dq_stride_s, st); if (rc) return rc;
      }
      if (sh->s_k > 0 && p.dk && !p.accumulate_dkv) {
        rc = dfa::launch_fill_zero_rows(p.dk, sh->h_kv, sh->s_k, sh->d, sh->dkv_stride_h, sh->dkv_stride_s, st); if (rc) return rc;
        rc = dfa::launch_fill_zero_rows(p.dv, sh->h_kv, sh->s_k, sh->d, sh->dkv_stride_h, sh->dkv_stride_s, st); if (rc) return rc;
      }
    }
    return DFA_OK;
  }
  const bool sequence = spans && sh->causal && sh->s_q == sh->s_k;
  return sh->dtype == DFA_F32 ? dfa::launch_bwd_f32(*sh, pairs, n_pairs, sequence, workspace, workspace_bytes, st)
                              : dfa::launch_bwd_bf16(*sh, pairs, n_pairs, workspace, workspace_bytes, st);
}

int64_t bwd_workspace(const dfa_shape* sh, int32_t n_pairs, int32_t want_dq, int32_t want_dkv, bool spans) {
  const int rc = check_common(sh, spans);
  if (rc != DFA_OK) return rc;
  if (n_pairs < 0) return DFA_ERR_ARG;
  if (n_pairs == 0 || sh->s_q == 0 || sh->s_k == 0) return 0;
  const bool sequence = spans && sh->causal && sh->s_q == sh->s_k;
  return sh->dtype == DFA_F32 ? dfa::bwd_f32_workspace(*sh, n_pairs, want_dq != 0, want_dkv != 0, sequence)
                              : dfa::bwd_bf16_workspace(*sh, n_pairs, want_dq != 0, want_dkv != 0);
}

int bwd_form(const dfa_shape* sh, int32_t n_pairs, int32_t want_dq, int32_t want_dkv, int64_t workspace_bytes, dfa_form* form,
             bool spans) {
  const int rc = check_common(sh, spans);
  if (rc != DFA_OK) return rc;
  if (!form) return DFA_ERR_NULL;
  if (n_pairs < 1 || workspace_bytes < 0 || (!want_dq && !want_dkv)) return DFA_ERR_ARG;
  if (sh->s_q == 0 || sh->s_k == 0) return DFA_ERR_SHAPE;
  const bool sequence = spans && sh->causal && sh->s_q == sh->s_k;
  *form = sh->dtype == DFA_F32 ? dfa::bwd_f32_form(*sh, n_pairs, want_dq != 0, want_dkv != 0, workspace_bytes, sequence)
                               : dfa::bwd_bf16_form(*sh, n_pairs, want_dq != 0, want_dkv != 0, workspace_bytes);
  return DFA_OK;
}

}  // namespace

extern "C" int dfa_chunk_bwd_form(const dfa_shape* sh, int32_t n_pairs, int32_t want_dq, int32_t want_dkv, int64_t workspace_bytes,
                                  dfa_form* form) {
  return bwd_form(sh, n_pairs, want_dq, want_dkv, workspace_bytes, form, false);
}
extern "C" int dfa_span_bwd_form(const dfa_shape* sh, int32_t want_dq, int32_t want_dkv, int64_t workspace_bytes, dfa_form* form) {
  return bwd_form(sh, 1, want_dq, want_dkv, workspace_bytes, form, true);
}

extern "C" int dfa_chunk_bwd_batch(const dfa_shape* sh, const dfa_bwd_pair* pairs, int32_t n_pairs, void* workspace,
                                   int64_t workspace_bytes, void* stream) {
  return bwd_batch(sh, pairs, n_pairs, workspace, workspace_bytes, stream, false);
}
extern "C" int64_t dfa_chunk_bwd_workspace(const dfa_shape* sh, int32_t n_pairs, int32_t want_dq, int32_t want_dkv) {
  return bwd_workspace(sh, n_pairs, want_dq, want_dkv, false);
}

extern "C" int dfa_span_bwd(const dfa_shape* sh, const dfa_bwd_pair* span, void* workspace, int64_t workspace_bytes, void* stream) {
  return bwd_batch(sh, span, 1, workspace, workspace_bytes, stream, true);
}
extern "C" int64_t dfa_span_bwd_workspace(const dfa_shape* sh, int32_t want_dq, int32_t want_dkv) {
  return bwd_workspace(sh, 1, want_dq, want_dkv, true);
}

extern "C" int dfa_chunk_bwd(const dfa_shape* sh, const void* q, const void* k, const void* v,
                             const float* lse, const float* delta, const void* dO,
                             float* dq, float* dk, float* dv, int accumulate, void* stream) {
  const dfa_bwd_pair p{q, k, v, lse, delta, dO, dq, dk, dv, accumulate != 0, accumulate != 0};
  return dfa_chunk_bwd_batch(sh, &p, 1, nullptr, 0, stream);
}

// HBM-bound row kernels: the merge (rescale) of two partial results, the D = rowsum(dO o O)
// pre-pass of the backward, and small fill kernels.  One query row is d values wide; a row is
// handled by adjacent lanes, so every global access of a wavefront is a run of full cache lines.
// Operands that are not needed again soon are read past the caches (nontemporal loads), which leaves
// them to what is: 32 heads x 16384, fp32, merge and then D 157 + 67 -> 115 + 57 us in the kernels (7.0 TB/s in both;
// a plain copy of the same tensor runs at 5.4), 231 -> 188 us for the two calls.
#include "dfa_internal.h"

namespace dfa {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct Vec8 { float v[8]; };

// STREAM: past the caches
template <bool BF16, bool STREAM = false>
__device__ inline Vec8 load8(const void* base, int64_t elem_off) {
  Vec8 r;
  if constexpr (BF16) {
    const u32x4* p = reinterpret_cast<const u32x4*>(static_cast<const __bf16*>(base) + elem_off);
    const u32x4 raw = STREAM ? __builtin_nontemporal_load(p) : *p;
    bf16x8 b = __builtin_bit_cast(bf16x8, raw);
#pragma unroll
    for (int i = 0; i < 8; ++i) r.v[i] = static_cast<float>(b[i]);
  } else {
    const f32x4* p = reinterpret_cast<const f32x4*>(static_cast<const float*>(base) + elem_off);
    const f32x4 a = STREAM ? __builtin_nontemporal_load(p) : p[0], b = STREAM ? __builtin_nontemporal_load(p + 1) : p[1];
#pragma unroll
    for (int i = 0; i < 4; ++i) { r.v[i] = a[i]; r.v[4 + i] = b[i]; }
  }
  return r;
}

template <bool BF16>
__device__ inline void store8(void* base, int64_t elem_off, const Vec8& r) {
  if constexpr (BF16) {
    bf16x8 b;
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = static_cast<__bf16>(r.v[i]);
    *reinterpret_cast<uint4*>(static_cast<__bf16*>(base) + elem_off) = __builtin_bit_cast(uint4, b);
  } else {
    float4* p = reinterpret_cast<float4*>(static_cast<float*>(base) + elem_off);
    p[0] = make_float4(r.v[0], r.v[1], r.v[2], r.v[3]);
    p[1] = make_float4(r.v[4], r.v[5], r.v[6], r.v[7]);
  }
}

constexpr int MAX_PAIRS = 16;          // per launch (blockIdx.z): the pairs travel in the kernel arguments
template <int NP> struct MergePairs { dfa_merge_pair pair[NP]; };

// 16 bytes of a row as fp32 values
template <bool BF16> struct Vec16 { static constexpr int N = BF16 ? 8 : 4; float v[N]; };
template <bool BF16, bool STREAM>
__device__ inline Vec16<BF16> load16(const void* base, int64_t elem_off) {
  const u32x4* p = reinterpret_cast<const u32x4*>(static_cast<const char*>(base) + elem_off * (BF16 ? 2 : 4));
  const u32x4 raw = STREAM ? __builtin_nontemporal_load(p) : *p;
  Vec16<BF16> r;
  if constexpr (BF16) {
    const bf16x8 b = __builtin_bit_cast(bf16x8, raw);
#pragma unroll
    for (int i = 0; i < 8; ++i) r.v[i] = static_cast<float>(b[i]);
  } else {
    const f32x4 f = __builtin_bit_cast(f32x4, raw);
#pragma unroll
    for (int i = 0; i < 4; ++i) r.v[i] = f[i];
  }
  return r;
}
template <bool BF16>
__device__ inline void store16(void* base, int64_t elem_off, const Vec16<BF16>& r) {
  if constexpr (BF16) {
    bf16x8 b;
#pragma unroll
    for (int i = 0; i < 8; ++i) b[i] = static_cast<__bf16>(r.v[i]);
    *reinterpret_cast<bf16x8*>(static_cast<__bf16*>(base) + elem_off) = b;
  } else {
    *reinterpret_cast<f32x4*>(static_cast<float*>(base) + elem_off) = f32x4{r.v[0], r.v[1], r.v[2], r.v[3]};
  }
}

// (o_a, lse_a) <- merge((o_a, lse_a), (o_b, lse_b)), Section 3.2 rescale(.)
// 16 bytes per lane and row, ROWS rows in flight per lane; (o_b, lse_b) is read for the last time, (o_a, lse_a)
// is what the next step continues from.  32 heads x 16384, fp32: 157 us with 32 bytes per lane and cached
// loads, 147 with this division, 115 with o_b past the caches (7.0 TB/s; four rows in flight: 116).
template <int D, bool BF16> constexpr int kMergeLanes = D / (BF16 ? 8 : 4);       // lanes per row
template <int D, bool BF16, int NP, int ROWS>
__global__ void __launch_bounds__(256) k_merge(dfa_merge_desc md, MergePairs<NP> pairs) {
  const dfa_merge_pair& pr = pairs.pair[NP == 1 ? 0 : blockIdx.z];
  constexpr int LPR = kMergeLanes<D, BF16>, RPB = 256 / LPR, VN = Vec16<BF16>::N;
  const int lane = threadIdx.x % LPR, h = blockIdx.y;
  const int row0 = blockIdx.x * RPB * ROWS + threadIdx.x / LPR;
  float* la_p = pr.lse_a + h * md.lse_a_stride_h;
  const float* lb_p = pr.lse_b + h * md.lse_b_stride_h;
  Vec16<BF16> a[ROWS], b[ROWS];
  float la[ROWS], lb[ROWS];
  auto off_a = [&](int row) { return h * md.a_stride_h + static_cast<int64_t>(row) * md.a_stride_s + lane * VN; };
#pragma unroll
  for (int u = 0; u < ROWS; ++u) {
    const int row = min(row0 + u * RPB, md.rows - 1);
    a[u] = load16<BF16, false>(pr.o_a, off_a(row));
    b[u] = load16<BF16, true>(pr.o_b, h * md.b_stride_h + static_cast<int64_t>(row) * md.b_stride_s + lane * VN);
    la[u] = la_p[row];
    lb[u] = lb_p[row];
  }
#pragma unroll
  for (int u = 0; u < ROWS; ++u) {
    const int row = row0 + u * RPB;
    if (row >= md.rows) break;
    const float m = fmaxf(la[u], lb[u]);
    float wa = 0.f, wb = 0.f, l = -INFINITY;
    if (m > -INFINITY) {
      const float ea = expf(la[u] - m), eb = expf(lb[u] - m);   // one of them is exactly 1
      const float s = ea + eb;
      l = m + logf(s);
      const float inv = 1.f / s;
      wa = ea * inv; wb = eb * inv;
    }
#pragma unroll
    for (int i = 0; i < VN; ++i) a[u].v[i] = wa * a[u].v[i] + wb * b[u].v[i];
    store16<BF16>(pr.o_a, off_a(row), a[u]);
    if (lane == 0) la_p[row] = l;
  }
}

// (o_a, lse_a) <- merge of (o_a, lse_a), unless it is only written, and several (o_b, lse_b), in one pass: three partials of 32
// heads x 4096, fp32, as three merges 91 us, in one 58.
constexpr int MAX_GROUPS = 16, MAX_PARTS = 32, GROUP_PARTS = 8;      // per launch, and of a group
struct MergeParts {
  int rows;
  int64_t b_sh, b_ss, lb_sh;
  MergeGroup group[MAX_GROUPS];
  MergePart part[MAX_PARTS];
};
template <int N, bool BF16>
__device__ inline void load_row(float (&v)[N], const void* base, int64_t off) {
#pragma unroll
  for (int i = 0; i < N; i += 4) {
    if constexpr (BF16) {
      typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
      const bf16x4 b = *reinterpret_cast<const bf16x4*>(static_cast<const __bf16*>(base) + off + i);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[i + e] = static_cast<float>(b[e]);
    } else {
      const f32x4 f = *reinterpret_cast<const f32x4*>(static_cast<const float*>(base) + off + i);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[i + e] = f[e];
    }
  }
}
template <int D, bool BF16>
__global__ void __launch_bounds__(256) k_merge_parts(MergeParts p) {
  constexpr int LPR = kMergeLanes<D, BF16>, RPB = 256 / LPR, VN = Vec16<BF16>::N;
  const MergeGroup& g = p.group[blockIdx.z];
  const MergePart* part = p.part + g.first;
  const int lane = threadIdx.x % LPR, h = blockIdx.y;
  const int row = blockIdx.x * RPB + threadIdx.x / LPR;
  if (row >= p.rows) return;
  Vec16<BF16> b[GROUP_PARTS];
  float lb[GROUP_PARTS];
#pragma unroll
  for (int i = 0; i < GROUP_PARTS; ++i) {
    if (i >= g.n) break;
    b[i] = load16<BF16, true>(part[i].o, h * p.b_sh + static_cast<int64_t>(row) * p.b_ss + lane * VN);
    lb[i] = part[i].lse[h * p.lb_sh + row];
  }
  const int64_t off_a = h * g.o_sh + static_cast<int64_t>(row) * g.o_ss + lane * VN;
  float* la_p = g.lse + h * g.l_sh + row;
  float a[VN];
#pragma unroll
  for (int i = 0; i < VN; ++i) a[i] = 0.f;
  float la = g.accumulate ? *la_p : -INFINITY;
  if (g.accumulate == MERGE_CONTINUE && !(la > -INFINITY)) la = -INFINITY;
  if (la > -INFINITY || g.accumulate == MERGE_ALL) {
    if (g.o_bf16) load_row<VN, true>(a, g.o, off_a); else load_row<VN, false>(a, g.o, off_a);
  }
  float m = la;
#pragma unroll
  for (int i = 0; i < GROUP_PARTS; ++i) m = i < g.n ? fmaxf(m, lb[i]) : m;
  // Nothing to weigh against: all weights are zero, and what is no number stays that, as in k_merge.
  const bool any = m > -INFINITY;
  const float wa = any ? expf(la - m) : 0.f;
  float s = wa;
#pragma unroll
  for (int e = 0; e < VN; ++e) a[e] *= wa;
#pragma unroll
  for (int i = 0; i < GROUP_PARTS; ++i) {
    if (i >= g.n) break;
    const float w = any ? expf(lb[i] - m) : 0.f;
    s += w;
#pragma unroll
    for (int e = 0; e < VN; ++e) a[e] = fmaf(w, b[i].v[e], a[e]);
  }
  const float l = any ? m + logf(s) : -INFINITY, inv = any ? 1.f / s : 0.f;
#pragma unroll
  for (int e = 0; e < VN; ++e) a[e] *= inv;
#pragma unroll
  for (int e = 0; e < VN; e += 4) {
    if (g.o_bf16) {
      typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
      bf16x4 x;
#pragma unroll
      for (int i = 0; i < 4; ++i) x[i] = static_cast<__bf16>(a[e + i]);
      *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(g.o) + off_a + e) = x;
    } else {
      *reinterpret_cast<f32x4*>(static_cast<float*>(g.o) + off_a + e) = f32x4{a[e], a[e + 1], a[e + 2], a[e + 3]};
    }
  }
  if (lane == 0) *la_p = l;
}

// D_i = sum_c dO_ic * O_ic  (Section 3.3: the saved output feeds the backward).  STREAM: dO past the caches.
template <int D, bool DO_BF16, bool O_BF16, bool STREAM>
__global__ void __launch_bounds__(256) k_delta(int s_q, const void* __restrict__ o, int64_t o_sh, int64_t o_ss,
                                               const void* __restrict__ dO, int64_t q_sh, int64_t q_ss,
                                               float* __restrict__ delta, int64_t l_sh) {
  constexpr int LPR = D / 8;
  constexpr int RPB = 256 / LPR;
  const int lane = threadIdx.x % LPR;
  const int h = blockIdx.y;
  const int row = blockIdx.x * RPB + threadIdx.x / LPR;
  float acc = 0.f;
  if (row < s_q) {
    const Vec8 a = load8<O_BF16>(o, h * o_sh + static_cast<int64_t>(row) * o_ss + lane * 8);
    const Vec8 b = load8<DO_BF16, STREAM>(dO, h * q_sh + static_cast<int64_t>(row) * q_ss + lane * 8);
#pragma unroll
    for (int i = 0; i < 8; ++i) acc = fmaf(a.v[i], b.v[i], acc);
  }
#pragma unroll
  for (int off = LPR / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
  if (row < s_q && lane == 0) delta[h * l_sh + row] = acc;
}

__global__ void __launch_bounds__(256) k_zero_rows(float* __restrict__ p, int rows, int d4, int64_t sh, int64_t ss) {
  const int h = blockIdx.y;
  const int per_row = d4;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < static_cast<int64_t>(rows) * per_row;
       i += static_cast<int64_t>(gridDim.x) * 256) {
    const int64_t r = i / per_row; const int c = static_cast<int>(i % per_row);
    reinterpret_cast<float4*>(p + h * sh + r * ss)[c] = make_float4(0.f, 0.f, 0.f, 0.f);
  }
}

template <bool BF16>
__global__ void __launch_bounds__(256) k_empty_fwd(int s_q, int d8, void* __restrict__ o, int64_t o_sh, int64_t o_ss,
                                                   float* __restrict__ lse, int64_t l_sh) {
  const int h = blockIdx.y;
  Vec8 z; for (int i = 0; i < 8; ++i) z.v[i] = 0.f;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < static_cast<int64_t>(s_q) * d8;
       i += static_cast<int64_t>(gridDim.x) * 256) {
    const int64_t r = i / d8; const int c = static_cast<int>(i % d8);
    store8<BF16>(o, h * o_sh + r * o_ss + c * 8, z);
    if (c == 0) lse[h * l_sh + r] = -INFINITY;
  }
}

int grid_for(int64_t items, int per_block) {
  int64_t g = (items + per_block - 1) / per_block;
  const int64_t cap = 256 * 16;   // 256 CUs, a few blocks each; kernels are grid-stride
  return static_cast<int>(g < 1 ? 1 : (g > cap ? cap : g));
}

}  // namespace

template <int D, bool BF16, int ROWS>
static void merge_rows(const dfa_merge_desc& md, const MergePairs<MAX_PAIRS>& all, int n, hipStream_t st) {
  constexpr int rows = 256 / kMergeLanes<D, BF16> * ROWS;
  const dim3 grid((md.rows - 1) / rows + 1, md.heads, n);
  if (n > 1) k_merge<D, BF16, MAX_PAIRS, ROWS><<<grid, 256, 0, st>>>(md, all);
  else k_merge<D, BF16, 1, ROWS><<<grid, 256, 0, st>>>(md, MergePairs<1>{{all.pair[0]}});
}

template <int D, bool BF16>
static void merge_form(const dfa_merge_desc& md, const MergePairs<MAX_PAIRS>& all, int n, hipStream_t st) {
  // One row per lane while all workgroups are resident at once (eight per CU) that way: 8 heads x 112, fp32, 2.87 -> 2.65 us,
  // 32 x 300 3.95 -> 3.65; two rows beyond (32 x 1024, o_b just written, 10.4 against 11.0).
  const int64_t blocks = (static_cast<int64_t>(md.rows) * kMergeLanes<D, BF16> + 255) / 256 * md.heads * n;
  if (blocks <= 2048) merge_rows<D, BF16, 1>(md, all, n, st);
  else merge_rows<D, BF16, 2>(md, all, n, st);
}

// Groups of any number and length: as many launches as they take.
class MergeQueue {
 public:
  MergeQueue(const MergeShape& sh, hipStream_t st) : sh_(sh), st_(st) {
    p_.rows = sh.rows; p_.b_sh = sh.b_sh; p_.b_ss = sh.b_ss; p_.lb_sh = sh.lb_sh;
  }
  // n parts into a group; more: its parts go on from here (the ones before come first).
  int add(const MergeGroup& g, const MergePart* parts, int n, bool more) {
    for (int done = 0; done < n; done += GROUP_PARTS) {
      const int take = n - done < GROUP_PARTS ? n - done : GROUP_PARTS;
      more |= done > 0;
      if (more || ng_ == MAX_GROUPS || np_ + take > MAX_PARTS) {      // a group that goes on continues from what it has written
        const int rc = flush();
        if (rc) return rc;
      }
      MergeGroup& x = p_.group[ng_++];
      x = g;
      x.first = np_; x.n = take;
      if (more) x.accumulate = MERGE_ALL;
      for (int i = 0; i < take; ++i) p_.part[np_++] = parts[done + i];
    }
    return DFA_OK;
  }
  int flush() {
    if (!ng_) return DFA_OK;
    if (sh_.d == 128) sh_.b_bf16 ? go<128, true>() : go<128, false>();
    else sh_.b_bf16 ? go<64, true>() : go<64, false>();
    ng_ = np_ = 0;
    return last_launch_status();
  }

 private:
  template <int D, bool BF16>
  void go() {
    constexpr int per = 256 / kMergeLanes<D, BF16>;
    k_merge_parts<D, BF16><<<dim3((sh_.rows - 1) / per + 1, sh_.heads, ng_), 256, 0, st_>>>(p_);
  }
  MergeShape sh_;
  hipStream_t st_;
  MergeParts p_{};
  int ng_ = 0, np_ = 0;
};

int launch_merge_parts(const MergeShape& sh, const MergeGroup* groups, int n, const MergePart* parts, hipStream_t st) {
  MergeQueue queue(sh, st);
  for (int i = 0; i < n; ++i) {
    const int rc = queue.add(groups[i], parts + groups[i].first, groups[i].n, false);
    if (rc) return rc;
  }
  return queue.flush();
}

int launch_merge(const dfa_merge_desc& md, const dfa_merge_pair* pairs, int n, hipStream_t st) {
  auto same = [&](int i) { return i > 0 && pairs[i].o_a == pairs[i - 1].o_a && pairs[i].lse_a == pairs[i - 1].lse_a; };
  bool several = false;
  for (int i = 1; i < n; ++i) several |= same(i);
  if (several) {      // into one destination, one after the other
    MergeQueue queue({md.heads, md.rows, md.d, md.o_dtype == DFA_BF16, md.b_stride_h, md.b_stride_s, md.lse_b_stride_h}, st);
    MergePart parts[GROUP_PARTS];
    int count = 0;
    bool more = false;
    for (int i = 0; i < n; ++i) {
      parts[count++] = {pairs[i].o_b, pairs[i].lse_b};
      const bool last = i + 1 == n || !same(i + 1);
      if (!last && count < GROUP_PARTS) continue;
      const int rc = queue.add({pairs[i].o_a, pairs[i].lse_a, md.a_stride_h, md.a_stride_s, md.lse_a_stride_h, 0, 0, MERGE_ALL,
                                md.o_dtype == DFA_BF16}, parts, count, more);
      if (rc) return rc;
      count = 0;
      more = !last;
    }
    return queue.flush();
  }
  for (; n > MAX_PAIRS; pairs += MAX_PAIRS, n -= MAX_PAIRS) {
    const int rc = launch_merge(md, pairs, MAX_PAIRS, st);
    if (rc) return rc;
  }
  MergePairs<MAX_PAIRS> all{};
  for (int i = 0; i < n; ++i) all.pair[i] = pairs[i];
  const bool b = md.o_dtype == DFA_BF16;
  if (md.d == 128) b ? merge_form<128, true>(md, all, n, st) : merge_form<128, false>(md, all, n, st);
  else b ? merge_form<64, true>(md, all, n, st) : merge_form<64, false>(md, all, n, st);
  return last_launch_status();
}

int launch_delta(const dfa_shape& sh, const void* o, const void* dO, float* delta, hipStream_t st) {
  const int rpb = 256 / (sh.d / 8);
  dim3 grid((sh.s_q + rpb - 1) / rpb, sh.h_q);
  const bool dob = sh.dtype == DFA_BF16, ob = sh.o_dtype == DFA_BF16;
  // The backward that follows reads dO again, from the caches as long as it and o fit the 256 MB that all
  // XCDs share; a larger dO only pushes out the o that the last merge has left there (o and dO of 32 heads x
  // 16384: 67 -> 56 us).
  const int64_t bytes = static_cast<int64_t>(sh.h_q) * sh.s_q * sh.d * ((dob ? 2 : 4) + (ob ? 2 : 4));
  const bool stream = bytes > (int64_t{256} << 20);
#define DFA_DELTA(DD, A, B) (stream ? k_delta<DD, A, B, true> : k_delta<DD, A, B, false>)<<<grid, 256, 0, st>>>( \
      sh.s_q, o, sh.o_stride_h, sh.o_stride_s, dO, sh.q_stride_h, sh.q_stride_s, delta, sh.lse_stride_h)
  if (sh.d == 128) {
    if (dob && ob) DFA_DELTA(128, true, true); else if (dob) DFA_DELTA(128, true, false);
    else if (ob) DFA_DELTA(128, false, true); else DFA_DELTA(128, false, false);
  } else {
    if (dob && ob) DFA_DELTA(64, true, true); else if (dob) DFA_DELTA(64, true, false);
    else if (ob) DFA_DELTA(64, false, true); else DFA_DELTA(64, false, false);
  }
#undef DFA_DELTA
  return last_launch_status();
}

int launch_fill_zero_rows(float* p, int heads, int rows, int d, int64_t stride_h, int64_t stride_s, hipStream_t st) {
  dim3 grid(grid_for(static_cast<int64_t>(rows) * (d / 4), 256), heads);
  k_zero_rows<<<grid, 256, 0, st>>>(p, rows, d / 4, stride_h, stride_s);
  return last_launch_status();
}

int launch_fill_empty_fwd(const dfa_shape& sh, void* o, float* lse, hipStream_t st) {
  dim3 grid(grid_for(static_cast<int64_t>(sh.s_q) * (sh.d / 8), 256), sh.h_q);
  if (sh.o_dtype == DFA_BF16) k_empty_fwd<true><<<grid, 256, 0, st>>>(sh.s_q, sh.d / 8, o, sh.o_stride_h, sh.o_stride_s, lse, sh.lse_stride_h);
  else k_empty_fwd<false><<<grid, 256, 0, st>>>(sh.s_q, sh.d / 8, o, sh.o_stride_h, sh.o_stride_s, lse, sh.lse_stride_h);
  return last_launch_status();
}

}  // namespace dfa

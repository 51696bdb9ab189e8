// fp32 mode of the chunk kernels: fp32 operands, results and sums, products of all 24 bits (backward: of values from 2^-110 on), any s_q / s_k.
// This is the precision-reference mode of the library (1e-5 agreement with fp64); the bf16 kernels
// are the fast path.
//
// Products of the backward.  An fp32 value is the exact sum of three bf16 ones: its upper 16 bits, the rounded rest, what that leaves (a
// value below 2^-110 in magnitude but for what lies below 2^-133, the smallest bf16 number: with dO of 2^-112 dv is 2.5e-7 off, dq and dk,
// whose factors P (dP - D) are smaller, 2.7e-6; with dO of 2^-118 9e-6 and 1.7e-4).  The split is a published one: Henry, Tang, Heinecke,
// "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", 2019.  Of the nine
// products of two such sums the six largest (the others are below 2^-23 of the product, of either sign) run on
// v_mfma_f32_32x32x16_bf16, the largest as one chain and the five small ones as another, added at the end.  That is 192 cycles per
// 32x32x16 against 512 of v_mfma_f32_32x32x2_f32, and closer to the exact sum: relative error of a product over 128 / 1024
// N(0,1) values 6.5e-8 / 1.9e-7 against 2.0e-7 / 5.7e-7 (a chain is rounded once per 16 terms instead of every two).
// Infinities and NaN: the largest product has them as the fp32 one would (signalling NaN are made quiet first), the chain of the small
// ones is bounded before it is added.  us, fp32 products / these: 32 heads x 4096 8785 / 5779, 32 over 8 x 2048 2200 / 1467, 8 over 2 x 1024 diagonal 141 / 109,
// one head x 256 diagonal at d = 64 19.4 / 16.5; the gradients are half as far from the exact ones.
// fp32 products (v_mfma_f32_32x32x2_f32) are left in the backward with 128-row tiles at d = 128, for which three values per
// element do not fit the LDS, and in the forward: there the split tiles leave room for one workgroup per CU, whose exponentials
// nobody's products cover (walks of 8 over 2 heads x 4096 359 us, 440 split).
//
// Layout of either, lane l, r = l % 32, h = l / 32: C/D (16 fp32): C[(i/4)*8 + 4h + i%4][r].  The contraction index only has to
// match between A and B, so a C tile is fed back as B operand: its registers 8u .. 8u+7 hold rows 16u + (e/4)*8 + 4h + e%4, and
// the A operand (of the bf16 product) is gathered in that order by the transposing LDS read.
// fp32 product: A operand A[r][h], B operand B[h][r];
//  * a product over d takes d = 8t + 4h + e in step 4t + e: one 16-byte read of a row serves four steps;
//  * column block j of a d-wide result holds d = NB m + j (NB = d / 32), so the A operands of all NB blocks come from
//    ONE read of NB consecutive floats.
// A wavefront owns 32 rows of the stationary operand and walks over 32-row blocks of the other,
// which four wavefronts share through LDS (rows padded by 4 floats: both kinds of reads are free of
// bank conflicts).  The four wavefronts of a workgroup are NR row blocks x NS = 4 / NR parts of every
// tile; with NS > 1 the partial results of the parts are combined through LDS at the end.  NS = 4 is
// for calls with few rows: it gives four times the workgroups, each with a quarter of the serial work.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "dfa_internal.h"
#include "dfa_mfma.h"
#include "dfa_place.h"
#include "dfa_span.h"

namespace dfa {
namespace {

constexpr int NT = 256;        // threads per workgroup: 4 wavefronts

// Products of split values (see above); else fp32 products.
template <int D, int NS> constexpr bool kSplit = !(D == 128 && NS == 4);
typedef float f32x2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// The operands of one (query chunk, key/value chunk) pair of the backward.
struct Pair {
  const float *q, *k, *v, *dO, *lse, *delta;
  float *dq, *dk, *dv;
  int acc_q, acc_kv;           // add to what dq / dk, dv hold
};
constexpr int MAX_PAIRS = 16;  // per launch: the pairs travel in the kernel arguments

struct F32Params {
  const float *q, *k, *v;
  void* o; float* lse;
  int s_q, s_k, h_q, h_kv, group, causal, o_bf16, accumulate;
  int nx_kv, n_kv;             // dk/dv: row blocks per key/value head, workgroups of a pair
  int nx_q, n_q;               // forward, dq: row blocks per query head, workgroups of a pair
  int pairs;
  XcdMap map_kv, map_q;        // workgroups of all pairs; the forward's are map_q
  int shares;                  // dk, dv: workgroups that share the query tiles of a row block
  float* partial;              // shares > 1: their sums, 2 D floats per key row
  int q_shares;                // dq: workgroups that share the key tiles of a row block
  float* q_partial;            // q_shares > 1: their sums, D floats per query row
  float scale;
  int64_t q_sh, q_ss, kv_sh, kv_ss, o_sh, o_ss, l_sh, dq_sh, dq_ss, dkv_sh, dkv_ss;
};
struct F32BwdParams : F32Params { Pair pair[MAX_PAIRS]; };

struct FwdPair {
  const float *q, *k, *v;
  void* o; float* lse;
  int accumulate;
  int64_t o_sh, o_ss, l_sh;
};
struct F32FwdBatch : F32Params { FwdPair fpair[MAX_PAIRS]; };
// Query chunks against spans of keys, each with its own number of them; off: key kv is visible to query row i if kv <= i + off.
struct Span : FwdPair { int s_k, off, o_bf16; };
struct F32FwdSpans : F32Params { int heads; Span span[MAX_PAIRS]; };
struct F32SpanParams : F32Params { int off; };
template <class P> __device__ __forceinline__ int off_of(const P&) { return 0; }
__device__ __forceinline__ int off_of(const F32SpanParams& p) { return p.off; }

// The operands of an item's pair; item becomes its number within the pair.
__device__ __forceinline__ const F32Params& pair_of(const F32Params& a, int&) { return a; }
__device__ __forceinline__ F32Params pair_of(const F32FwdBatch& a, int& item) {
  F32Params p = a;
  const FwdPair& x = a.fpair[item / a.n_q];
  item %= a.n_q;
  p.q = x.q; p.k = x.k; p.v = x.v; p.o = x.o; p.lse = x.lse; p.accumulate = x.accumulate;
  p.o_sh = x.o_sh; p.o_ss = x.o_ss; p.l_sh = x.l_sh;
  return p;
}

// (as in the bf16 forward: an XCD takes its heads of all spans, span by span, the longest first)
__device__ __forceinline__ F32SpanParams pair_of(const F32FwdSpans& a, int& item) {
  int i = item / a.n_q, r = item % a.n_q;
  if (a.heads) {
    const int x = item / a.map_q.per_xcd, y = item % a.map_q.per_xcd, run = a.heads * a.nx_q;
    i = y / run; r = x * run + y % run;
  }
  item = r;
  F32SpanParams p;
  static_cast<F32Params&>(p) = a;
  const Span& s = a.span[i];
  p.q = s.q; p.k = s.k; p.v = s.v; p.o = s.o; p.lse = s.lse; p.accumulate = s.accumulate;
  p.o_sh = s.o_sh; p.o_ss = s.o_ss; p.l_sh = s.l_sh; p.s_k = s.s_k; p.o_bf16 = s.o_bf16; p.off = s.off;
  return p;
}

template <int NB> struct Run;      // NB consecutive floats
template <> struct Run<4> { typedef f32x4 type; };
template <> struct Run<2> { typedef f32x2 type; };

template <int NB>
__device__ __forceinline__ void zero(f32x16 (&c)[NB]) {
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) c[j][i] = 0.f;
}

// One 32-row block as a B operand over d, straight from global memory: lane holds row `row`,
// d = 8t + 4h .. +3; rows past the end are zero.
template <int D>
__device__ __forceinline__ void load_rows(f32x4 (&b)[D / 8], const float* src, int64_t ss, int row, bool ok, int hh) {
  const float* p = src + static_cast<int64_t>(ok ? row : 0) * ss + 4 * hh;
#pragma unroll
  for (int t = 0; t < D / 8; ++t) {
    b[t] = *reinterpret_cast<const f32x4*>(p + 8 * t);
    if (!ok) b[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
}

template <int D, int ROWS> struct Planes;

// A pair of ROWS x D tiles on their way from global memory to LDS.  load() issues the reads of a tile
// while the tile before it is computed on; store() writes what has arrived.  Rows past the end are zero.
template <int D, int ROWS>
struct TilePair {
  static constexpr int LD = D + 4, C4 = D / 4, N = ROWS * C4 / NT;
  f32x4 a[N], b[N];
  __device__ __forceinline__ void load(const float* A, const float* B, int64_t ss, int row0, int nrows) {
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int i = threadIdx.x + n * NT, r = row0 + i / C4, c = (i % C4) * 4;
      const int64_t off = static_cast<int64_t>(min(r, nrows - 1)) * ss + c;
      a[n] = *reinterpret_cast<const f32x4*>(A + off);
      b[n] = *reinterpret_cast<const f32x4*>(B + off);
    }
  }
  // (Whole tiles apart: the selections would be an instruction per value.)
  __device__ __forceinline__ void store_split(char* As, char* Bs, int row0, int nrows) const {
    auto put = [&](auto whole) DFA_INLINE {
#pragma unroll
      for (int n = 0; n < N; ++n) {
        const int i = threadIdx.x + n * NT, r = i / C4, c = (i % C4) * 4;
        const bool ok = decltype(whole)::value || row0 + r < nrows;
        const f32x4 z = {0.f, 0.f, 0.f, 0.f};
        Planes<D, ROWS>::put(As, r, c, ok ? a[n] : z);
        Planes<D, ROWS>::put(Bs, r, c, ok ? b[n] : z);
      }
    };
    if (row0 + ROWS <= nrows) put(std::true_type{});
    else put(std::false_type{});
  }
  __device__ __forceinline__ void store(float* As, float* Bs, int row0, int nrows) const {
#pragma unroll
    for (int n = 0; n < N; ++n) {
      const int i = threadIdx.x + n * NT, r = i / C4, c = (i % C4) * 4;
      const bool ok = row0 + r < nrows;
      const f32x4 z = {0.f, 0.f, 0.f, 0.f};
      *reinterpret_cast<f32x4*>(As + r * LD + c) = ok ? a[n] : z;
      *reinterpret_cast<f32x4*>(Bs + r * LD + c) = ok ? b[n] : z;
    }
  }
};

// ---- split values ----
struct Split8 { bf16x8 h, m, l; };
// Two values: upper halves, rounded rests, what is left.  (A NaN is made a quiet one, whose upper half is one too; of a signalling one
// with its payload in the lower half that would be an infinity.)
__device__ __forceinline__ void split2(float a, float b, uint32_t& h, uint32_t& m, uint32_t& l) {
  a = __builtin_canonicalizef(a);
  b = __builtin_canonicalizef(b);
  const uint32_t ua = __builtin_bit_cast(uint32_t, a), ub = __builtin_bit_cast(uint32_t, b);
  h = __builtin_amdgcn_perm(ub, ua, 0x07060302);
  const float ra = a - __builtin_bit_cast(float, ua & 0xffff0000u), rb = b - __builtin_bit_cast(float, ub & 0xffff0000u);
  bf16x2 t;
  t[0] = static_cast<__bf16>(ra); t[1] = static_cast<__bf16>(rb);
  m = __builtin_bit_cast(uint32_t, t);
  t[0] = static_cast<__bf16>(ra - __builtin_bit_cast(float, m << 16));
  t[1] = static_cast<__bf16>(rb - __builtin_bit_cast(float, m & 0xffff0000u));
  l = __builtin_bit_cast(uint32_t, t);
}
template <class F>
__device__ __forceinline__ Split8 split8(F value) {      // value(e), e = 0 .. 7
  u32x4 h, m, l;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    uint32_t x, y, z;
    split2(value(2 * e), value(2 * e + 1), x, y, z);
    h[e] = x; m[e] = y; l[e] = z;
  }
  return {__builtin_bit_cast(bf16x8, h), __builtin_bit_cast(bf16x8, m), __builtin_bit_cast(bf16x8, l)};
}
// main += the largest product, rest += the five small ones, the smallest first
__device__ __forceinline__ void mfma_split(const Split8& a, const Split8& b, f32x16& main, f32x16& rest) {
  rest = mfma32(a.l, b.h, rest);
  rest = mfma32(a.h, b.l, rest);
  rest = mfma32(a.m, b.m, rest);
  rest = mfma32(a.m, b.h, rest);
  rest = mfma32(a.h, b.m, rest);
  main = mfma32(a.h, b.h, main);
}
__device__ __forceinline__ float bounded(float x) { return __builtin_amdgcn_fmed3f(x, -3.402823466e38f, 3.402823466e38f); }

// A ROWS x D tile in LDS as three bf16 tiles of 272-byte rows (at d = 64 the first two share theirs).
template <int D, int ROWS> struct Planes {
  static constexpr int BYTES = (D == 128 ? 3 : 2) * ROWS * kRowBytes;
  static constexpr int at(int plane) { return D == 128 ? plane * ROWS * kRowBytes : plane == 2 ? ROWS * kRowBytes : plane * 128; }
  __device__ static __forceinline__ Split8 rows(const char* t, int off) {      // off: tile_off(row, h) + 32 ks
    return {lds_read_b128(t, off + at(0)), lds_read_b128(t, off + at(1)), lds_read_b128(t, off + at(2))};
  }
  __device__ static __forceinline__ Split8 cols(const char* t, int off) {      // off: gather_base + row0 * kRowBytes + 64 db
    return {lds_gather(t, off + at(0)), lds_gather(t, off + at(1)), lds_gather(t, off + at(2))};
  }
  // four consecutive values of a row, from column c
  __device__ static __forceinline__ void put(char* t, int r, int c, f32x4 x) {
    uint32_t h[2], m[2], l[2];
    split2(x[0], x[1], h[0], m[0], l[0]);
    split2(x[2], x[3], h[1], m[1], l[1]);
    char* p = t + prow(r) * kRowBytes + 2 * c;
    *reinterpret_cast<u32x2*>(p + at(0)) = u32x2{h[0], h[1]};
    *reinterpret_cast<u32x2*>(p + at(1)) = u32x2{m[0], m[1]};
    *reinterpret_cast<u32x2*>(p + at(2)) = u32x2{l[0], l[1]};
  }
};

// One 32-row block as a split B operand over d, straight from global memory: lane holds row `row`, d = 16 ks + 8h .. +7.
template <int D>
__device__ __forceinline__ void load_rows(Split8 (&b)[D / 16], const float* src, int64_t ss, int row, bool ok, int hh) {
  const float* p = src + static_cast<int64_t>(ok ? row : 0) * ss + 8 * hh;
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) {
    f32x4 x = *reinterpret_cast<const f32x4*>(p + 16 * ks), y = *reinterpret_cast<const f32x4*>(p + 16 * ks + 4);
    if (!ok) x = y = f32x4{0.f, 0.f, 0.f, 0.f};
    b[ks] = split8([&](int e) { return e < 4 ? x[e] : y[e - 4]; });
  }
}

// The columns of 32 rows' W as a B operand: w[u] of rows 16u + (e/4)*8 + 4h + e%4.
__device__ __forceinline__ void split_tile(Split8 (&b)[2], const f32x16& w) {
#pragma unroll
  for (int u = 0; u < 2; ++u) b[u] = split8([&](int e) { return w[8 * u + e]; });
}
__device__ __forceinline__ f32x16 zero16() {
  f32x16 z;
#pragma unroll
  for (int i = 0; i < 16; ++i) z[i] = 0.f;
  return z;
}

// A operands in the order of their use, each read from LDS AHEAD steps (of six products, 192 cycles) before it is used: with one
// wavefront per SIMD nobody else's work covers a read that is waited for.
template <int N, int AHEAD, class Read, class Use>
__device__ __forceinline__ void stream(Read read, Use use) {
  Split8 z[AHEAD + 1];
#pragma unroll
  for (int i = 0; i < AHEAD; ++i) z[i] = read(i);
  DFA_SCHED_FENCE();
#pragma unroll
  for (int i = 0; i < N; ++i) {
    if (i + AHEAD < N) z[(i + AHEAD) % (AHEAD + 1)] = read(i + AHEAD);
    use(i, z[i % (AHEAD + 1)]);
    DFA_SCHED_FENCE();
  }
}

// acc^T += X^T W, one 32-column block after the other, two steps of 16 rows each: the sums of a block's 32 rows (SUM: the largest
// products' too) are added while the next block's products run.
template <int D, bool SUM> struct ColSums {
  f32x16 main[2], rest[2];
  __device__ __forceinline__ void add(f32x16 (&acc)[D / 32], int db) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const float x = main[db & 1][i] + bounded(rest[db & 1][i]);
      acc[db][i] = SUM ? acc[db][i] + x : x;
    }
  }
  // step c = 2 db + u
  __device__ __forceinline__ void step(f32x16 (&acc)[D / 32], int c, const Split8& x, const Split8 (&w)[2]) {
    const int db = c >> 1, u = c & 1;
    if (u == 0) {
      rest[db & 1] = zero16();
      if constexpr (SUM) main[db & 1] = zero16();
      else main[db & 1] = acc[db];
    }
    mfma_split(x, w[u], main[db & 1], rest[db & 1]);
    if (u == 0 && db > 0) add(acc, db - 1);
    if (c == D / 16 - 1) add(acc, db);
  }
};

// ---- runs: a d-wide result leaves in D / 8 runs of four consecutive floats per lane ----
template <int D, bool SPLIT>
__device__ __forceinline__ f32x4 run_of(const f32x16 (&c)[D / 32], int k) {
  if constexpr (SPLIT) return f32x4{c[k >> 2][4 * (k & 3)], c[k >> 2][4 * (k & 3) + 1], c[k >> 2][4 * (k & 3) + 2], c[k >> 2][4 * (k & 3) + 3]};
  else return f32x4{c[0][k], c[1][k], c[2][k], c[3][k]};
}
template <bool SPLIT> __device__ __forceinline__ int run_col(int k, int hh) {
  return SPLIT ? (k >> 2) * 32 + (k & 3) * 8 + 4 * hh : 4 * ((k >> 2) * 8 + 4 * hh + (k & 3));
}

// C += X Y^T over d: X is a 32-row block in LDS (row r of it for lane r), Y a register operand.
template <int D>
__device__ __forceinline__ void row_product(f32x16& c, const float* Xs, const f32x4 (&y)[D / 8], int r32, int hh) {
  const float* x = Xs + r32 * (D + 4) + 4 * hh;
#pragma unroll
  for (int t = 0; t < D / 8; ++t) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(x + 8 * t);
    c = mfma_f32(a.x, y[t].x, c);
    c = mfma_f32(a.y, y[t].y, c);
    c = mfma_f32(a.z, y[t].z, c);
    c = mfma_f32(a.w, y[t].w, c);
  }
}

// The same with Y (32 rows too) in LDS.
template <int D>
__device__ __forceinline__ void row_product(f32x16& c, const float* Xs, const float* Ys, int r32, int hh) {
  const float* x = Xs + r32 * (D + 4) + 4 * hh;
  const float* y = Ys + r32 * (D + 4) + 4 * hh;
#pragma unroll
  for (int t = 0; t < D / 8; ++t) {
    const f32x4 a = *reinterpret_cast<const f32x4*>(x + 8 * t), b = *reinterpret_cast<const f32x4*>(y + 8 * t);
    c = mfma_f32(a.x, b.x, c);
    c = mfma_f32(a.y, b.y, c);
    c = mfma_f32(a.z, b.z, c);
    c = mfma_f32(a.w, b.w, c);
  }
}

// acc^T += X^T W: X is a 32-row block in LDS, W a C tile (its rows are X's rows).
template <int D>
__device__ __forceinline__ void col_product(f32x16 (&acc)[D / 32], const float* Xs, const f32x16& w, int r32, int hh) {
  constexpr int NB = D / 32;
  typedef typename Run<NB>::type run_t;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const run_t a = *reinterpret_cast<const run_t*>(Xs + ((i >> 2) * 8 + 4 * hh + (i & 3)) * (D + 4) + NB * r32);
#pragma unroll
    for (int j = 0; j < NB; ++j) acc[j] = mfma_f32(a[j], w[i], acc[j]);
  }
}

// Sum of a result over the NS parts of a row block, left in part 0: `x` is LDS space for
// 4 * NV * 64 floats (NV registers of the result per lane).
template <int NB>
__device__ __forceinline__ void put_result(float* x, const f32x16 (&c)[NB], int lane) {
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) x[(j * 16 + i) * 64 + lane] = c[j][i];
}
template <int NB>
__device__ __forceinline__ void add_result(const float* x, f32x16 (&c)[NB], int lane, float f) {
#pragma unroll
  for (int j = 0; j < NB; ++j)
#pragma unroll
    for (int i = 0; i < 16; ++i) c[j][i] = fmaf(x[(j * 16 + i) * 64 + lane], f, c[j][i]);
}

// Row `dst` (+)= f * result
template <int D, bool SPLIT>
__device__ __forceinline__ void write_grad(float* dst, const f32x16 (&c)[D / 32], float f, int accumulate, int hh) {
#pragma unroll
  for (int k = 0; k < D / 8; ++k) {
    f32x4* p = reinterpret_cast<f32x4*>(dst + run_col<SPLIT>(k, hh));
    f32x4 x = run_of<D, SPLIT>(c, k) * f;
    if (accumulate) x += *p;
    *p = x;
  }
}

// Keys per LDS tile of the forward: 32 per part, and at least 64 (a single part then takes two blocks in
// turn).  The backward holds more in registers and takes 32 rows per part throughout.
template <int NS> constexpr int kTile = NS == 4 ? 128 : 64;

template <int D, int ROWS>
constexpr size_t fwd_smem() { return sizeof(float) * 2 * ROWS * (D + 4); }
// The backward: two tiles of 32 NS rows and two floats per row.
template <int D, int NS>
constexpr size_t smem_bytes() {
  constexpr int ROWS = 32 * NS;
  return (kSplit<D, NS> ? 2 * Planes<D, ROWS>::BYTES : sizeof(float) * 2 * ROWS * (D + 4)) + sizeof(float) * 2 * ROWS;
}

// Forward.  Online softmax as in the pseudo-code of Appendix A (running row maximum m and row sum l,
// old terms multiplied by exp(m_old - m_new)); a lane holds the scores of ONE query.
template <int D, int NS, class Args>
__global__ void __launch_bounds__(NT, NS == 4 ? 1 : 2) k_fwd_f32(Args a) {
  constexpr int NR = 4 / NS, NB = D / 32, LD = D + 4, BK = kTile<NS>;
  typedef typename Run<NB>::type run_t;
  extern __shared__ __align__(16) float smem[];
  float* Ks = smem;
  float* Vs = Ks + BK * LD;
  const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), rb = wave % NR, part = wave / NR;
  int item = xcd_item(a.map_q, blockIdx.x);
  if (item >= a.map_q.total) return;
  const auto& p = pair_of(a, item);
  const int off = off_of(p);
  const int h = item / p.nx_q, kh = h / p.group;
  int xq = item % p.nx_q;
  if (p.causal) xq = p.nx_q - 1 - xq;       // longest rows first
  const int q0 = xq * NR * 32, q0w = q0 + rb * 32, qrow = q0w + r32;
  const bool qvalid = qrow < p.s_q;
  const float* kg = p.k + kh * p.kv_sh;
  const float* vg = p.v + kh * p.kv_sh;
  const int k_end = p.causal ? min(p.s_k, q0 + NR * 32 + off) : p.s_k;

  TilePair<D, BK> tile;
  tile.load(kg, vg, p.kv_ss, 0, p.s_k);
  f32x4 q[D / 8];
  load_rows<D>(q, p.q + h * p.q_sh, p.q_ss, qrow, qvalid, hh);

  // Empty state, or (accumulate, first part) the state of the earlier key/value chunks: the normalised
  // output with its logsumexp is the running (o, m, l) with m = lse and l = 1.
  f32x16 o[NB];
  zero(o);
  float m_run = -INFINITY, l_run = 0.f;      // l_run: this lane's half of the row sum
  const int64_t obase = h * p.o_sh + static_cast<int64_t>(qvalid ? qrow : 0) * p.o_ss;
  if (p.accumulate && part == 0 && qvalid) {
    const float L = p.lse[h * p.l_sh + qrow];
    if (L > -INFINITY) {
      m_run = L;
      l_run = hh == 0 ? 1.f : 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i)
#pragma unroll
        for (int j = 0; j < NB; ++j) {
          const int64_t off = obase + NB * ((i >> 2) * 8 + 4 * hh + (i & 3)) + j;
          o[j][i] = p.o_bf16 ? static_cast<float>(static_cast<const __bf16*>(p.o)[off]) : static_cast<const float*>(p.o)[off];
        }
    }
  }

  for (int k0 = 0; k0 < k_end; k0 += BK) {
    if (k0) __syncthreads();                 // the tile before has been read
    tile.store(Ks, Vs, k0, p.s_k);
    __syncthreads();
    if (k0 + BK < k_end) tile.load(kg, vg, p.kv_ss, k0 + BK, p.s_k);
#pragma unroll
    for (int kb = part * 32; kb < BK; kb += NS * 32) {
      const int kb0 = k0 + kb;
      if (kb0 >= p.s_k || (p.causal && kb0 > q0w + 31 + off)) break;
      f32x16 s;
#pragma unroll
      for (int i = 0; i < 16; ++i) s[i] = 0.f;
      row_product<D>(s, Ks + kb * LD, q, r32, hh);
      float mx = -INFINITY;
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int kvi = kb0 + (i >> 2) * 8 + 4 * hh + (i & 3);
        s[i] = kvi < p.s_k && !(p.causal && kvi > qrow + off) ? s[i] * p.scale : -INFINITY;
        mx = fmaxf(mx, s[i]);
      }
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m_run, mx);
      const float m_safe = m_new == -INFINITY ? 0.f : m_new;
      const float alpha = expf(m_run - m_safe);   // exp(-inf) = 0 on the first block
      float sum = 0.f;
#pragma unroll
      for (int i = 0; i < 16; ++i) { s[i] = expf(s[i] - m_safe); sum += s[i]; }
      m_run = m_new;
      l_run = l_run * alpha + sum;
      if (__any(alpha != 1.f)) {
#pragma unroll
        for (int j = 0; j < NB; ++j)
#pragma unroll
          for (int i = 0; i < 16; ++i) o[j][i] *= alpha;
      }
      col_product<D>(o, Vs + kb * LD, s, r32, hh);
    }
  }

  float l_tot = l_run + __shfl_xor(l_run, 32);
  if constexpr (NS > 1) {       // combine the parts: exact, against the largest of their maxima
    constexpr int NV = NB * 16;
    float* st = smem + 4 * NV * 64;          // m, l of every wavefront's 32 rows
    __syncthreads();
    if (part > 0) put_result<NB>(smem + wave * NV * 64, o, lane);
    if (hh == 0) { st[wave * 64 + r32] = m_run; st[wave * 64 + 32 + r32] = l_tot; }
    __syncthreads();
    if (part > 0) return;
    float m = m_run;
#pragma unroll
    for (int s = 1; s < NS; ++s) m = fmaxf(m, st[(s * NR + rb) * 64 + r32]);
    const float m_safe = m == -INFINITY ? 0.f : m;
    const float f0 = expf(m_run - m_safe);
    l_tot *= f0;
#pragma unroll
    for (int j = 0; j < NB; ++j)
#pragma unroll
      for (int i = 0; i < 16; ++i) o[j][i] *= f0;
#pragma unroll
    for (int s = 1; s < NS; ++s) {
      const int w = s * NR + rb;
      const float f = expf(st[w * 64 + r32] - m_safe);
      l_tot = fmaf(st[w * 64 + 32 + r32], f, l_tot);
      add_result<NB>(smem + w * NV * 64, o, lane, f);
    }
    m_run = m;
  }
  if (!qvalid) return;
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  if (hh == 0) p.lse[h * p.l_sh + qrow] = l_tot > 0.f ? m_run + logf(l_tot) : -INFINITY;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int64_t off = obase + NB * ((i >> 2) * 8 + 4 * hh + (i & 3));
    if (p.o_bf16) {
#pragma unroll
      for (int j = 0; j < NB; ++j) static_cast<__bf16*>(p.o)[off + j] = static_cast<__bf16>(o[j][i] * inv);
    } else {
      run_t x;
#pragma unroll
      for (int j = 0; j < NB; ++j) x[j] = o[j][i] * inv;
      *reinterpret_cast<run_t*>(static_cast<float*>(p.o) + off) = x;
    }
  }
}

// dk, dv of one workgroup's key rows: K and V rows in registers, Q / dO tiles (with lse and D) in LDS,
// summed over the query heads of the group.
// V_LDS: at d = 128 K, V (of three values each), dK, dV and the tile on its way are more registers than
// there are; V then stays in LDS (with split values, of all of the workgroup's rows).
template <int D, int NS> constexpr bool kVLds = D == 128;
template <int D, int NS> constexpr size_t v_bytes() {
  return !kVLds<D, NS> ? 0 : kSplit<D, NS> ? Planes<D, 128 / NS>::BYTES : sizeof(float) * 32 * (D + 4);
}
// SHARED: p.shares workgroups share the query tiles of a row block.
// SUMS (a sequence that stands for the pairs of several chunks): dk, dv as sums of 32 query rows each, added up.  The rounding
// errors of one chain over all rows grow with its length.  Relative error of dk, dv in a schedule of 4 heads x 8000, d = 128, with
// fp32 products: one chain 1.6e-6, sums 5.8e-7 and 5.1e-7 (pair by pair, 1000 rows each in one chain, 7.0e-7 and 6.6e-7).  They
// took 7 to 8 % of a backward at d = 128 and 1 to 2 % at d = 64, so a pair, whose chain is no longer than it ever was, goes without.
template <int D, int NS, bool SHARED, bool SUMS>
__device__ __forceinline__ void bwd_dkdv(const F32Params& p, const Pair& pr, int item, float* partial, float* smem) {
  constexpr int NR = 4 / NS, NB = D / 32, LD = D + 4, BQ = 32 * NS;
  constexpr bool V_LDS = kVLds<D, NS>, SPLIT = kSplit<D, NS>;
  char* Qp = reinterpret_cast<char*>(smem);
  char* Gp = Qp + (SPLIT ? Planes<D, BQ>::BYTES : 0);
  float* Qs = smem;
  float* Gs = Qs + BQ * LD;
  float* Ls = SPLIT ? reinterpret_cast<float*>(Gp + Planes<D, BQ>::BYTES) : Gs + BQ * LD;
  float* Vs = Ls + 2 * BQ;                   // after lse and D
  const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), rb = wave % NR, part = wave / NR;
  const int share = SHARED ? item / p.nx_kv % p.shares : 0, kh = SHARED ? item / p.nx_kv / p.shares : item / p.nx_kv;
  const int k0 = (item % p.nx_kv) * NR * 32, k0w = k0 + rb * 32, kvrow = k0w + r32;
  const bool kvalid = kvrow < p.s_k;
  const int off = p.s_k - p.s_q;             // causal: key kv is visible to query row i if kv <= i + off
  const int q_begin = p.causal ? max(0, k0 - off) : 0;

  TilePair<D, BQ> tile;
  float ld = 0.f;                            // lse (first BQ threads) or D (next BQ) of the tile on its way
  auto load = [&](int hq, int q0) {
    tile.load(pr.q + hq * p.q_sh, pr.dO + hq * p.q_sh, p.q_ss, q0, p.s_q);
    if (tid < 2 * BQ) {
      const int r = q0 + tid % BQ;
      const float* src = (tid < BQ ? pr.lse : pr.delta) + hq * p.l_sh;
      ld = r < p.s_q ? src[r] : tid < BQ ? -INFINITY : 0.f;
    }
  };
  int hq = kh * p.group, q0 = q_begin;
  const int h_end = hq + p.group;
  int left = 0;                              // SHARED: query tiles of this workgroup's share
  if constexpr (SHARED) {
    const int ntq = (p.s_q - q_begin + BQ - 1) / BQ;
    const int64_t walk = static_cast<int64_t>(ntq) * p.group;
    const int it0 = static_cast<int>(walk * share / p.shares);
    left = static_cast<int>(walk * (share + 1) / p.shares) - it0;
    if (left > 0) { hq += it0 / ntq; q0 += it0 % ntq * BQ; }       // (else a tile is loaded, and not used)
  }
  load(hq, q0);
  const int a_base = tile_off(r32, hh), g_base = gather_base(lane);
  std::conditional_t<SPLIT, Split8[D / 16], f32x4[D / 8]> k;
  std::conditional_t<SPLIT, Split8[V_LDS ? 1 : D / 16], f32x4[V_LDS ? 1 : D / 8]> v;
  char* Vp = reinterpret_cast<char*>(Vs);
  load_rows<D>(k, pr.k + kh * p.kv_sh, p.kv_ss, kvrow, kvalid, hh);
  if constexpr (V_LDS) {
    for (int i = tid; i < NR * 32 * (D / 4); i += NT) {
      const int r = k0 + i / (D / 4), c = (i % (D / 4)) * 4;
      f32x4 x = {0.f, 0.f, 0.f, 0.f};
      if (r < p.s_k) x = *reinterpret_cast<const f32x4*>(pr.v + kh * p.kv_sh + static_cast<int64_t>(r) * p.kv_ss + c);
      if constexpr (SPLIT) Planes<D, NR * 32>::put(Vp, r - k0, c, x);
      else *reinterpret_cast<f32x4*>(Vs + (r - k0) * LD + c) = x;
    }
  } else {
    load_rows<D>(v, pr.v + kh * p.kv_sh, p.kv_ss, kvrow, kvalid, hh);
  }
  f32x16 dk[NB], dv[NB];
  zero(dk);
  zero(dv);
  for (bool first = true; SHARED ? left > 0 : hq < h_end; first = false) {
    if (!first) __syncthreads();
    if constexpr (SPLIT) tile.store_split(Qp, Gp, q0, p.s_q);
    else tile.store(Qs, Gs, q0, p.s_q);
    if (tid < 2 * BQ) Ls[tid] = ld;          // lse, then D
    __syncthreads();
    const int q0t = q0 + part * 32;          // this wavefront's 32 rows of the tile
    q0 += BQ;
    if (q0 >= p.s_q) { q0 = q_begin; ++hq; }
    if (SHARED ? --left > 0 : hq < h_end) load(hq, q0);
    if (q0t >= p.s_q || (p.causal && k0w > q0t + 31 + off)) continue;
    const float* Qw = Qs + part * 32 * LD;
    const float* Gw = Gs + part * 32 * LD;
    f32x16 s, dp;
    auto weights = [&]() DFA_INLINE {          // s: P, dp: dS
      // (the rows' L and D four at a time, hidden scores as -inf: a branch and a read of their own for each of the 16 took
      // longer than the products)
      const float* row = Ls + part * 32 + 4 * hh;
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 L = *reinterpret_cast<const f32x4*>(row + 8 * j);      // -inf for rows past the end and empty rows
#pragma unroll
        for (int e = 0; e < 4; ++e) s[4 * j + e] = L[e] > -INFINITY ? s[4 * j + e] * p.scale - L[e] : -INFINITY;
      }
      if (p.causal && k0w + 31 > q0t + off) {
#pragma unroll
        for (int i = 0; i < 16; ++i)
          if (kvrow > q0t + (i >> 2) * 8 + 4 * hh + (i & 3) + off) s[i] = -INFINITY;
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const f32x4 D4 = *reinterpret_cast<const f32x4*>(row + BQ + 8 * j);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          s[4 * j + e] = expf(s[4 * j + e]);
          dp[4 * j + e] = s[4 * j + e] * (dp[4 * j + e] - D4[e]);
        }
      }
    };
    if constexpr (SPLIT) {
      constexpr int KS = D / 16;
      constexpr int AHEAD = D == 128 && NS == 2 ? 1 : 2;      // (no registers left for two)
      typedef Planes<D, BQ> Tile;
      f32x16 sr = zero16(), dpr = zero16();
      Split8 vz, w[2], x[2];
      ColSums<D, SUMS> cs;
      s = zero16(); dp = zero16();
      const int row0 = part * 32 * kRowBytes;
      stream<2 * KS + 4 * NB, AHEAD>([&](int i) DFA_INLINE {
        if (i < 2 * KS) return Tile::rows(i & 1 ? Gp : Qp, a_base + row0 + (i >> 1) * 32);
        const int c = i - 2 * KS, db = (c >> 1) % NB;
        return Tile::cols(c < 2 * NB ? Gp : Qp, g_base + row0 + 16 * (c & 1) * kRowBytes + db * 64);
      }, [&](int i, const Split8& a) DFA_INLINE {
        if (i < 2 * KS) {
          if (!(i & 1)) {
            if constexpr (V_LDS) vz = Planes<D, NR * 32>::rows(Vp, a_base + rb * 32 * kRowBytes + (i >> 1) * 32);
            mfma_split(a, k[i >> 1], s, sr);
          } else if constexpr (V_LDS) {
            mfma_split(a, vz, dp, dpr);
          } else {
            mfma_split(a, v[i >> 1], dp, dpr);
          }
          return;
        }
        const int c = i - 2 * KS;
        if (c == 0) {
#pragma unroll
          for (int e = 0; e < 16; ++e) { s[e] += bounded(sr[e]); dp[e] += bounded(dpr[e]); }
          weights();
          split_tile(w, s);
        }
        if (c < 2 * NB) cs.step(dv, c, a, w);
        else cs.step(dk, c - 2 * NB, a, x);
        if (c == 0) split_tile(x, dp);
      });
    } else {
      static_assert(SPLIT || !SUMS, "no registers left for the sums");
#pragma unroll
      for (int i = 0; i < 16; ++i) { s[i] = 0.f; dp[i] = 0.f; }
      row_product<D>(s, Qw, k, r32, hh);
      if constexpr (V_LDS) row_product<D>(dp, Gw, Vs, r32, hh);
      else row_product<D>(dp, Gw, v, r32, hh);
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const int r = (i >> 2) * 8 + 4 * hh + (i & 3);
        const float L = Ls[part * 32 + r];
        const bool vis = L > -INFINITY && !(p.causal && kvrow > q0t + r + off);
        s[i] = vis ? expf(s[i] * p.scale - L) : 0.f;
        dp[i] = s[i] * (dp[i] - Ls[BQ + part * 32 + r]);
      }
      col_product<D>(dv, Gw, s, r32, hh);
      col_product<D>(dk, Qw, dp, r32, hh);
    }
  }
  if constexpr (NS > 1) {
    constexpr int NV = NB * 16;
    __syncthreads();
    if (part > 0) {
      float* x = smem + (wave - NR) * 2 * NV * 64;
      put_result<NB>(x, dk, lane);
      put_result<NB>(x + NV * 64, dv, lane);
    }
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int s = 1; s < NS; ++s) {
      const float* x = smem + (s * NR + rb - NR) * 2 * NV * 64;
      add_result<NB>(x, dk, lane, 1.f);
      add_result<NB>(x + NV * 64, dv, lane, 1.f);
    }
  }
  if constexpr (SHARED) {       // k_reduce_f32 adds the shares up
    constexpr int RUNS = D / 8;
    f32x4* x = reinterpret_cast<f32x4*>(partial) + rb * 2 * RUNS * 64 + lane;
#pragma unroll
    for (int i = 0; i < RUNS; ++i) {
      x[i * 64] = run_of<D, SPLIT>(dk, i);
      x[(RUNS + i) * 64] = run_of<D, SPLIT>(dv, i);
    }
    return;
  }
  if (!kvalid) return;
  const int64_t dst = kh * p.dkv_sh + static_cast<int64_t>(kvrow) * p.dkv_ss;
  write_grad<D, SPLIT>(pr.dk + dst, dk, p.scale, pr.acc_kv, hh);
  write_grad<D, SPLIT>(pr.dv + dst, dv, 1.f, pr.acc_kv, hh);
}

// dq of one workgroup's query rows: Q and dO rows in registers, K / V tiles in LDS.
// q_shares > 1: its share of the key tiles only, k_reduce_f32 adds the shares up.
template <int D, int NS>
__device__ __forceinline__ void bwd_dq(const F32Params& p, const Pair& pr, int item, float* partial, float* smem) {
  constexpr int NR = 4 / NS, NB = D / 32, LD = D + 4, BK = 32 * NS;
  constexpr bool SPLIT = kSplit<D, NS>;
  char* Kp = reinterpret_cast<char*>(smem);
  char* Vp = Kp + (SPLIT ? Planes<D, BK>::BYTES : 0);
  float* Ks = smem;
  float* Vs = Ks + BK * LD;
  const int tid = threadIdx.x, lane = tid & 63, r32 = lane & 31, hh = lane >> 5;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), rb = wave % NR, part = wave / NR;
  const int share = item / p.nx_q % p.q_shares, h = item / p.nx_q / p.q_shares, kh = h / p.group;
  int xq = item % p.nx_q;
  if (p.causal) xq = p.nx_q - 1 - xq;
  const int q0 = xq * NR * 32, q0w = q0 + rb * 32, qrow = q0w + r32;
  const bool qvalid = qrow < p.s_q;
  const float* kg = pr.k + kh * p.kv_sh;
  const float* vg = pr.v + kh * p.kv_sh;
  const int off = p.s_k - p.s_q;
  int k_end = p.causal ? min(p.s_k, q0 + NR * 32 + off) : p.s_k, k_begin = 0;
  if (p.q_shares > 1) {
    const int64_t ntk = (k_end + BK - 1) / BK;
    k_begin = static_cast<int>(ntk * share / p.q_shares) * BK;
    k_end = min(k_end, static_cast<int>(ntk * (share + 1) / p.q_shares) * BK);
  }

  TilePair<D, BK> tile;
  tile.load(kg, vg, p.kv_ss, k_begin, p.s_k);
  const int a_base = tile_off(r32, hh), g_base = gather_base(lane);
  std::conditional_t<SPLIT, Split8[D / 16], f32x4[D / 8]> q, g;
  load_rows<D>(q, pr.q + h * p.q_sh, p.q_ss, qrow, qvalid, hh);
  load_rows<D>(g, pr.dO + h * p.q_sh, p.q_ss, qrow, qvalid, hh);
  const float L = qvalid ? pr.lse[h * p.l_sh + qrow] : -INFINITY;
  const float Dr = qvalid ? pr.delta[h * p.l_sh + qrow] : 0.f;
  // fp32 products: sums of two tiles (64 keys of a part) each, added up, since the rounding errors of one chain over all keys grow
  // with its length.  Relative error of dq from exact lse and D, one chain / this: 2 over 1 heads, 300 x 16384 1.31e-6 / 6.3e-7, 8
  // heads x 4096 9.9e-7 / 5.9e-7 (with sums of eight tiles 6.4e-7, of four 6.1e-7).  Split products: sums of one tile.
  constexpr int RUN = SPLIT ? 1 : 2;
  f32x16 dq[NB], run[SPLIT ? 1 : NB];
  zero(dq);
  for (int k0 = k_begin; k0 < k_end;) {
    if constexpr (!SPLIT) zero(run);
    for (int n = 0; n < RUN && k0 < k_end; ++n, k0 += BK) {
      if (k0 > k_begin) __syncthreads();
      if constexpr (SPLIT) tile.store_split(Kp, Vp, k0, p.s_k);
      else tile.store(Ks, Vs, k0, p.s_k);
      __syncthreads();
      if (k0 + BK < k_end) tile.load(kg, vg, p.kv_ss, k0 + BK, p.s_k);
      const int kb0 = k0 + part * 32;
      if (kb0 >= p.s_k || (p.causal && kb0 > q0w + 31 + off)) continue;
      const float* Kw = Ks + part * 32 * LD;
      f32x16 s, dp;
      auto weights = [&]() DFA_INLINE {        // dp: dS
#pragma unroll
        for (int i = 0; i < 16; ++i) s[i] = L > -INFINITY ? s[i] * p.scale - L : -INFINITY;
        if (kb0 + 32 > p.s_k || (p.causal && kb0 + 31 > q0w + off)) {
#pragma unroll
          for (int i = 0; i < 16; ++i) {
            const int kvi = kb0 + (i >> 2) * 8 + 4 * hh + (i & 3);
            if (kvi >= p.s_k || (p.causal && kvi > qrow + off)) s[i] = -INFINITY;
          }
        }
#pragma unroll
        for (int i = 0; i < 16; ++i) dp[i] = expf(s[i]) * (dp[i] - Dr);
      };
      if constexpr (SPLIT) {
        constexpr int KS = D / 16;
        constexpr int AHEAD = D == 128 && NS == 2 ? 1 : 2;
        typedef Planes<D, BK> Tile;
        f32x16 sr = zero16(), dpr = zero16();
        Split8 w[2];
        ColSums<D, true> cs;
        s = zero16(); dp = zero16();
        const int row0 = part * 32 * kRowBytes;
        stream<2 * KS + 2 * NB, AHEAD>([&](int i) DFA_INLINE {
          if (i < 2 * KS) return Tile::rows(i & 1 ? Vp : Kp, a_base + row0 + (i >> 1) * 32);
          const int c = i - 2 * KS;
          return Tile::cols(Kp, g_base + row0 + 16 * (c & 1) * kRowBytes + (c >> 1) * 64);
        }, [&](int i, const Split8& a) DFA_INLINE {
          if (i < 2 * KS) {
            if (i & 1) mfma_split(a, g[i >> 1], dp, dpr);
            else mfma_split(a, q[i >> 1], s, sr);
            return;
          }
          if (i == 2 * KS) {
#pragma unroll
            for (int e = 0; e < 16; ++e) { s[e] += bounded(sr[e]); dp[e] += bounded(dpr[e]); }
            weights();
            split_tile(w, dp);
          }
          cs.step(dq, i - 2 * KS, a, w);
        });
      } else {
#pragma unroll
        for (int i = 0; i < 16; ++i) { s[i] = 0.f; dp[i] = 0.f; }
        row_product<D>(s, Kw, q, r32, hh);
        row_product<D>(dp, Vs + part * 32 * LD, g, r32, hh);
        weights();
        col_product<D>(run, Kw, dp, r32, hh);
      }
    }
    if constexpr (!SPLIT) {
#pragma unroll
      for (int j = 0; j < NB; ++j)
#pragma unroll
        for (int i = 0; i < 16; ++i) dq[j][i] += run[j][i];
    }
  }
  if constexpr (NS > 1) {
    constexpr int NV = NB * 16;
    __syncthreads();
    if (part > 0) put_result<NB>(smem + wave * NV * 64, dq, lane);
    __syncthreads();
    if (part > 0) return;
#pragma unroll
    for (int s = 1; s < NS; ++s) add_result<NB>(smem + (s * NR + rb) * NV * 64, dq, lane, 1.f);
  }
  if (p.q_shares > 1) {
    constexpr int RUNS = D / 8;
    f32x4* x = reinterpret_cast<f32x4*>(partial) + rb * RUNS * 64 + lane;
#pragma unroll
    for (int i = 0; i < RUNS; ++i) x[i * 64] = run_of<D, SPLIT>(dq, i);
    return;
  }
  if (!qvalid) return;
  write_grad<D, SPLIT>(pr.dq + h * p.dq_sh + static_cast<int64_t>(qrow) * p.dq_ss, dq, p.scale, pr.acc_q, hh);
}

// Backward: 7 products in two kinds of workgroups of ONE launch (dk/dv first, they are the longer
// ones), no atomics, no zero fill, a fixed order of summation.  The fused
// form (5 products, dq added with fp32 atomics) left a short chunk with as few workgroups as it has key
// tiles.
template <int D, int NS, bool SHARED, bool SUMS>
__global__ void __launch_bounds__(NT, 1) k_bwd_f32(F32BwdParams p) {
  extern __shared__ __align__(16) float smem[];
  const int grid_kv = p.map_kv.per_xcd * 8, bid = blockIdx.x;
  if (bid < grid_kv) {
    const int item = xcd_item(p.map_kv, bid);
    if (item < p.map_kv.total)
      bwd_dkdv<D, NS, SHARED, SUMS>(p, p.pair[item / p.n_kv], item % p.n_kv,
                              p.partial + static_cast<int64_t>(item) * (4 / NS * 64 * D), smem);
  } else {
    const int item = xcd_item(p.map_q, bid - grid_kv);
    if (item < p.map_q.total)
      bwd_dq<D, NS>(p, p.pair[item / p.n_q], item % p.n_q, p.q_partial + static_cast<int64_t>(item) * (4 / NS * 32 * D), smem);
  }
}

// dk, dv (KV: blockIdx.y = 2 * 32-row block + dv) or dq (blockIdx.y = 32-row block) of a block of NR * 32 rows from the sums of
// its shares: blockIdx.x = row block, 256 threads, each a quarter of a lane's runs.  The order of the sum is that of the shares.
template <int D, int NR, bool KV>
__global__ void __launch_bounds__(NT) k_reduce_f32(F32BwdParams p) {
  constexpr int RUNS = D / 8, MINE = RUNS / 4;
  constexpr bool SPLIT = kSplit<D, 4 / NR>;
  const int nx = KV ? p.nx_kv : p.nx_q, heads = KV ? p.h_kv : p.h_q, shares = KV ? p.shares : p.q_shares;
  const int xr = blockIdx.x % nx, ph = blockIdx.x / nx;                // ph: pair * heads + head
  const Pair& pr = p.pair[ph / heads];
  const int rb = KV ? blockIdx.y >> 1 : blockIdx.y, is_dv = KV ? blockIdx.y & 1 : 0;
  const int lane = threadIdx.x & 63, i0 = (threadIdx.x >> 6) * MINE;
  const int xrow = !KV && p.causal ? nx - 1 - xr : xr;      // (dq: the longest rows come first)
  const int row = (xrow * NR + rb) * 32 + (lane & 31);
  if (row >= (KV ? p.s_k : p.s_q)) return;
  const int64_t block = NR * (KV ? 2 : 1) * RUNS * 64, step = static_cast<int64_t>(nx) * block;      // in runs
  const f32x4* src = reinterpret_cast<const f32x4*>(KV ? p.partial : p.q_partial) +
                     (static_cast<int64_t>(ph) * shares * nx + xr) * block + (blockIdx.y * RUNS + i0) * 64 + lane;
  f32x4 a[MINE];
#pragma unroll
  for (int i = 0; i < MINE; ++i) a[i] = src[i * 64];
#pragma unroll 4      // (the reads of four shares on their way)
  for (int s = 1; s < shares; ++s) {
    src += step;
#pragma unroll
    for (int i = 0; i < MINE; ++i) a[i] += src[i * 64];
  }
  float* out = KV ? (is_dv ? pr.dv : pr.dk) : pr.dq;
  float* dst = out + (ph % heads) * (KV ? p.dkv_sh : p.dq_sh) + static_cast<int64_t>(row) * (KV ? p.dkv_ss : p.dq_ss);
  const float f = is_dv ? 1.f : p.scale;
  const int add = KV ? pr.acc_kv : pr.acc_q;
#pragma unroll
  for (int i = 0; i < MINE; ++i) {
    f32x4* d = reinterpret_cast<f32x4*>(dst + run_col<SPLIT>(i0 + i, lane >> 5));
    f32x4 x = a[i] * f;
    if (add) x += *d;
    *d = x;
  }
}

F32Params make_params(const dfa_shape& sh) {
  F32Params p{};
  p.s_q = sh.s_q; p.s_k = sh.s_k; p.h_q = sh.h_q; p.h_kv = sh.h_kv; p.group = sh.h_q / sh.h_kv; p.causal = sh.causal;
  p.o_bf16 = sh.o_dtype == DFA_BF16; p.scale = sh.scale;
  p.q_sh = sh.q_stride_h; p.q_ss = sh.q_stride_s; p.kv_sh = sh.kv_stride_h; p.kv_ss = sh.kv_stride_s;
  p.o_sh = sh.o_stride_h; p.o_ss = sh.o_stride_s; p.l_sh = sh.lse_stride_h;
  p.dq_sh = sh.dq_stride_h; p.dq_ss = sh.dq_stride_s; p.dkv_sh = sh.dkv_stride_h; p.dkv_ss = sh.dkv_stride_s;
  return p;
}

// More than 64 KB of dynamic LDS needs the opt-in, once per kernel and process (thread-safe).
template <class P, void (*KERNEL)(P)>
int launch(const P& p, int64_t blocks, size_t smem, hipStream_t st) {
  static std::once_flag once;
  static int attr_rc = DFA_OK;
  std::call_once(once, [smem] {
    attr_rc = hip_status(hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(smem)));
  });
  if (attr_rc) return attr_rc;
  if (blocks > (1 << 30)) return DFA_ERR_SHAPE;
  KERNEL<<<static_cast<int>(blocks), NT, smem, st>>>(p);
  return last_launch_status();
}

int64_t blocks_of(int rows, int per) { return (static_cast<int64_t>(rows) + per - 1) / per; }

template <int D, int NS, class Args>
int fwd(Args& p, hipStream_t st) {
  const int rows = 32 * (4 / NS);
  // tiles; the combination of the parts takes 4 results and 256 floats of row statistics
  const size_t comb = NS > 1 ? sizeof(float) * (4 * (D / 32) * 16 * 64 + 256) : 0;
  const size_t tiles = fwd_smem<D, kTile<NS>>();
  p.nx_q = static_cast<int>(blocks_of(p.s_q, rows));
  const int64_t n_q = static_cast<int64_t>(p.nx_q) * p.h_q;
  if (n_q * p.pairs > (1 << 30)) return DFA_ERR_SHAPE;
  p.n_q = static_cast<int>(n_q);
  p.map_q = xcd_map(n_q * p.pairs, p.causal, static_cast<int64_t>(p.h_q) * p.pairs);
  return launch<Args, k_fwd_f32<D, NS, Args>>(p, xcd_blocks(p.map_q), tiles > comb ? tiles : comb, st);
}

int fwd_parts(const dfa_shape& sh, int pairs) {
  // Parts per tile.  A workgroup with more parts is done sooner, but stages every tile for fewer rows and
  // runs fewer wavefronts per SIMD.  us per full pair, d = 128, with 1 / 2 / 4 parts:
  //   8 heads x 256 rows 47 / 29 / 22, 32 x 256 49 / 31 / 28, 8 x 1024 174 / 103 / 71 (<= 256 workgroups of
  //   4 parts: one round),  32 x 1024 190 / 183 / 271,  32 x 4096 2361 / 2501 / 3920 (116 TFLOP/s with 1);
  //   causal, 32 x 4096, 2 parts: 1402 (2043 with every eighth row block on the same XCD).
  // The vector-FMA kernel this one replaced took 610 us at 8 x 1024.
  const int64_t wg2 = blocks_of(sh.s_q, 64) * sh.h_q * pairs, wg4 = blocks_of(sh.s_q, 32) * sh.h_q * pairs;
  return wg4 <= 256 ? 4 : wg2 <= 512 || sh.causal ? 2 : 1;
}

template <class Args>
int fwd_form(Args& p, const dfa_shape& sh, hipStream_t st) {
  const int parts = fwd_parts(sh, p.pairs);
  if (sh.d == 128) return parts == 4 ? fwd<128, 4, Args>(p, st) : parts == 2 ? fwd<128, 2, Args>(p, st) : fwd<128, 1, Args>(p, st);
  return parts == 4 ? fwd<64, 4, Args>(p, st) : parts == 2 ? fwd<64, 2, Args>(p, st) : fwd<64, 1, Args>(p, st);
}

// Spans.  Parts per tile (NS) and parts that the keys of a span are cut in, by an estimate launch by launch, fitted to 130 forwards of
// shares and of all workers, every division timed (chosen / best 1.02 in the mean): 6 us per workgroup and, per tile of a walk at d =
// 128, 9 us with 4 parts of 32 keys, 6.1 with 2 (9.8 where two workgroups share a CU); a launch that runs in one round takes its
// longest walk, a longer one the device's even share and a third of a walk; the merge 5 us and 3 TB/s.  (Taking all spans as
// one launch and keys as they are made tiny and many-launch calls slower than their pairs: 64 over 8 heads x 8 x 94, window 1,
// forward 99 pairs, 113 so; one head x 8 x 445, ring 179 / 188.)  One part of each tile (128 rows) was timed too: within
// 3 % either way of two parts on the longest shares, slower elsewhere.
struct SpanPlan { int ns, parts; double us; };
SpanPlan span_plan(const dfa_shape& sh, const dfa_fwd_span* spans, int n, int64_t ws_bytes) {
  SpanPlan best{0, 1, 0.};
  const double width = sh.d == 128 ? 1.0 : 0.55;
  for (int ns : {4, 2}) {
    const int64_t blocks = blocks_of(sh.s_q, 128 / ns) * sh.h_q;
    const int keys_of_tile = ns == 4 ? 128 : 64;
    for (int parts : SPAN_CUTS) {
      const int64_t bytes = parts_bytes(sh, spans, n, parts);
      if (parts > 1 && (!bytes || bytes > ws_bytes)) break;
      const double us = sum_of_launches(sh, spans, n, parts, MAX_PAIRS, blocks, keys_of_tile, [&](const LaunchWork& w) {
        const bool shared = ns == 2 && w.workgroups > 256;
        const double tile = width * (ns == 4 ? 9.0 : shared ? 9.8 : 6.1) / keys_of_tile;      // per key
        double x = 6 + w.longest * tile;
        if (w.workgroups > (ns == 4 ? 256 : 512)) x = std::max(x, 6 + w.keys * tile / (shared ? 512 : 256) + 0.3 * w.longest * tile);
        return x + (w.cut ? 5 + 2 * w.part_bytes / 3e6 : 0);
      });
      if (!best.ns || us < best.us) best = {ns, parts, us};
    }
  }
  return best;
}

template <int D, int NS>
int fwd_spans(F32FwdSpans& p, int n, hipStream_t st) {
  const int rows = 32 * (4 / NS);
  const size_t comb = sizeof(float) * (4 * (D / 32) * 16 * 64 + 256), tiles = fwd_smem<D, kTile<NS>>();
  p.nx_q = static_cast<int>(blocks_of(p.s_q, rows));
  const int64_t n_q = static_cast<int64_t>(p.nx_q) * p.h_q;
  if (n_q * n > (1 << 30)) return DFA_ERR_SHAPE;
  p.n_q = static_cast<int>(n_q);
  p.heads = p.h_q % 8 == 0 ? p.h_q / 8 : 0;
  p.map_q = xcd_map(n_q * n, 1, p.heads ? 8 : 1);
  std::stable_sort(p.span, p.span + n, [](const Span& x, const Span& y) { return x.s_k > y.s_k; });
  return launch<F32FwdSpans, k_fwd_f32<D, NS, F32FwdSpans>>(p, xcd_blocks(p.map_q), tiles > comb ? tiles : comb, st);
}

template <int D, int NS, bool SUMS>
int bwd(F32BwdParams p, hipStream_t st) {
  const int rows = 32 * (4 / NS);
  const size_t comb = NS > 1 ? sizeof(float) * (4 - 4 / NS) * 2 * (D / 32) * 16 * 64 : 0;
  const size_t tiles = smem_bytes<D, NS>() + v_bytes<D, NS>();
  p.nx_kv = static_cast<int>(blocks_of(p.s_k, rows));
  p.nx_q = static_cast<int>(blocks_of(p.s_q, rows));
  const int64_t n_kv = p.pair[0].dk ? static_cast<int64_t>(p.nx_kv) * p.h_kv * p.shares : 0;
  const int64_t n_q = p.pair[0].dq ? static_cast<int64_t>(p.nx_q) * p.h_q * p.q_shares : 0;
  if ((n_kv + n_q) * p.pairs > (1 << 30)) return DFA_ERR_SHAPE;
  p.n_kv = static_cast<int>(n_kv);
  p.n_q = static_cast<int>(n_q);
  p.map_kv = xcd_map(n_kv * p.pairs, p.causal, static_cast<int64_t>(p.h_kv) * p.shares * p.pairs);
  p.map_q = xcd_map(n_q * p.pairs, p.causal, static_cast<int64_t>(p.h_q) * p.q_shares * p.pairs);
  if (p.shares > 1) p.q_partial += n_kv * p.pairs * (rows * 2 * D);      // after the sums of dk, dv
  const int64_t blocks = xcd_blocks(p.map_kv) + xcd_blocks(p.map_q);
  const size_t smem = tiles > comb ? tiles : comb;
  const int rc = p.shares > 1 ? launch<F32BwdParams, k_bwd_f32<D, NS, true, SUMS>>(p, blocks, smem, st)
                              : launch<F32BwdParams, k_bwd_f32<D, NS, false, SUMS>>(p, blocks, smem, st);
  if (rc) return rc;
  if (p.shares > 1)
    k_reduce_f32<D, 4 / NS, true><<<dim3(static_cast<unsigned>(n_kv * p.pairs / p.shares), 2 * (4 / NS)), NT, 0, st>>>(p);
  if (p.q_shares > 1)
    k_reduce_f32<D, 4 / NS, false><<<dim3(static_cast<unsigned>(n_q * p.pairs / p.q_shares), 4 / NS), NT, 0, st>>>(p);
  return last_launch_status();
}

// How a backward is divided: parts of every tile inside a workgroup, and workgroups that share the query tiles of
// a block of key rows or the keys of a row block of dq.  A dk/dv workgroup walks over all query heads of its group, so with grouped
// heads a few workgroups would run long after the others, and the walk of a row block of dq over many keys, or of a diagonal's last
// rows, may be the whole call; sharing a walk sends its sums (2 D floats per key row, D per query row) through memory and a further
// launch.  The estimate places the workgroups (dfa_place.h), with constants fitted to 322 calls at d = 128 and 253 at d = 64 (pairs,
// diagonals, sequences, spans, few rows against many keys), every division timed: chosen / best 1.010 and 1.013 in the mean; of 110
// other calls 1.028 (an estimate by even shares, fitted to fp32 products in every form: 1.087, 1.041 and 1.067).  The 4-part form, on
// fp32 products at d = 128, is the best one there of calls that are short and whose walks cannot be shared: without scratch 8 heads x
// 512 diagonal 60.7 us, 71.5 with 2 parts.  us, as the even shares chose / so: 8 heads x 512 diagonal 60.7 / 51.1, 4 x 1024 104.7 / 64.2,
// 4 x 1536 198.6 / 108.7, 32 over 8 x 333 107.5 / 68.5, 8 over 2 x 768 95.2 / 75.7, x 2048 at d = 64 182 / 163, full pair
// of 32 over 8 x 1024 459 / 389.
struct Plan { int parts, shares, q_shares; double us; int64_t bytes; };

// us: of a workgroup, of a tile of the walks of dk, dv and of dq, with 1, 2 and 4 parts; `tail` and `late` of dfa_place.h; of the
// sums' launches, per share, and their GB/ms.
struct Terms { double start[3], kv[3], q[3], tail, late, sums, per_share, per_q_share, rate; };
constexpr Terms D128{{11.77, 11.49, 10.2}, {6.5, 7.38, 11.71}, {4.37, 5.32, 9.71}, 0.36, 0.24, 1.54, 0.16, 0.17, 8.21};
constexpr Terms D64{{6.63, 6.61, 6.08}, {3.53, 4.24, 5.58}, {2.87, 3.11, 3.98}, 0.16, 0.35, 3.92, 0.04, 0.04, 10.26};

// A call with `parts` parts of every tile, undivided: what the divisions of a plan have in common.
struct Undivided {
  int parts, form, d, group, causal;
  int64_t kv_heads, q_heads;              // of all pairs
  int64_t n_kv, n_q, q_blocks, q_tiles, bytes;      // workgroups of dk, dv and of dq (and per head); key tiles; a dk/dv workgroup's sums (dq: half)
  double walk_kv, walk_q, mean;           // tiles; mean: of a walk, the query chunk's own keys are half visible
  int64_t ws_bytes;
};
Undivided undivided(const dfa_shape& sh, int pairs, bool dq, bool dk, int64_t ws_bytes, int parts) {
  const int rows = 128 / parts, tile = 32 * parts, group = sh.h_q / sh.h_kv;
  const int64_t q_tiles = blocks_of(sh.s_k, tile);
  return {parts, parts / 2, sh.d, group, sh.causal, static_cast<int64_t>(sh.h_kv) * pairs, static_cast<int64_t>(sh.h_q) * pairs,
          dk ? blocks_of(sh.s_k, rows) * sh.h_kv * pairs : 0, dq ? blocks_of(sh.s_q, rows) * sh.h_q * pairs : 0, blocks_of(sh.s_q, rows),
          q_tiles, static_cast<int64_t>(rows) * 2 * sh.d * 4, static_cast<double>(group * blocks_of(sh.s_q, tile)), static_cast<double>(q_tiles),
          sh.causal ? 1 - 0.5 * sh.s_q / sh.s_k : 1.0, ws_bytes};
}
// The walks of one kind of workgroup in `shares`: its workgroups, their sums' bytes and the us that these take.
struct Shared { Kind kind; int shares; int64_t bytes; double us; };
Shared shared(const Undivided& c, bool kv, int shares) {
  const Terms& k = c.d == 128 ? D128 : D64;
  const int64_t n = (kv ? c.n_kv : c.n_q) * shares;
  const double start = k.start[c.form], walk = (kv ? k.kv[c.form] * c.walk_kv : k.q[c.form] * c.walk_q) / shares;
  const double mean = (start + walk * c.mean) * (c.causal ? uneven((kv ? c.kv_heads : c.q_heads) * shares) : 1.0);
  const int64_t bytes = shares > 1 ? n * (kv ? c.bytes : c.bytes / 2) : 0;
  return {{(n + XCDS - 1) / XCDS, start + walk, mean, kv ? 0 : c.q_blocks}, shares, bytes,
          shares > 1 ? k.sums + (kv ? k.per_share : k.per_q_share) * shares + 2 * bytes / (k.rate * 1e6) : 0.};
}
// The same by even shares, without a look at rounds: 6 us per workgroup, us per tile for 1, 2 and 4 parts (at d = 64 0.55 of them),
// half a workgroup beyond the device's share.  For calls whose forms still stand in the old proportions, as all take split products:
// sequences, and walks of several chunks at d = 64.  Placed, 70 sequences at d = 128 took 0.98 of the time in the mean, but some far
// more (4 heads x 926 59 -> 73 us, 4 over 1 x 922 61 -> 75), and 82 walks at d = 64 1.005 (one head x 922 x 4610 55 -> 72).
double even_shares(const Undivided& c, const Shared& kv, const Shared& q, bool diagonal) {
  constexpr double per_kv[3] = {9.3, 10.3, 12.2}, per_q[3] = {7, 7.7, 9.7};
  const double width = c.d == 128 ? 1.0 : 0.55;
  const int64_t n_kv = c.n_kv * kv.shares, n_q = c.n_q * q.shares, sums = kv.bytes + q.bytes;
  const double w_kv = width * per_kv[c.form] * c.walk_kv / kv.shares, w_q = width * per_q[c.form] * c.walk_q / q.shares;
  const double t_kv = n_kv ? 6 + w_kv : 0., t_q = n_q ? 6 + w_q : 0.;
  double us = std::max(t_kv, t_q);
  if (n_kv + n_q > XCDS * CUS) {
    const double even_kv = n_kv * (6 + w_kv * c.mean) / (XCDS * CUS), even_q = n_q * (6 + w_q * c.mean) / (XCDS * CUS);
    us = std::max(us, diagonal ? even_kv * uneven(c.kv_heads * kv.shares) + std::max(t_q, even_q * uneven(c.q_heads * q.shares) + 0.3 * t_q)
                               : even_kv + even_q + 0.45 * us);
  }
  return sums > 0 ? (us + 4 * ((kv.shares > 1) + (q.shares > 1)) + 2 * sums / 2.5e6) / 0.92 : us;
}
Plan best_of(const Undivided* calls, int n, int most_q, bool even, bool diagonal) {
  Plan best{0, 0, 0, 0., 0};
  for (const Undivided* c = calls; c < calls + n; ++c) {
    const Terms& k = c->d == 128 ? D128 : D64;
    // Of a causal call whose walks are about equally long (many keys before the chunk's own) whole rounds count too.
    const double equal = c->causal ? std::max(0., 2 * c->mean - 1) * std::max(0., 2 * c->mean - 1) : 0.;
    Shared kv[10];
    int n_kv = 0;
    for (int shares : {1, 2, 3, 4, 6, 8, 12, 16, 24, 32}) {
      if (shares > 1 && (!c->n_kv || shares > 4 * c->group || c->n_kv * shares > 1024)) break;
      kv[n_kv++] = shared(*c, true, shares);
    }
    for (int q_shares = 1; q_shares <= most_q; q_shares *= 2) {
      if (q_shares > 1 && (c->n_q * q_shares > 1024 || q_shares > c->q_tiles)) break;
      const Shared q = shared(*c, false, q_shares);
      double low = 1e30;
      for (int i = 0; i < n_kv && kv[i].bytes + q.bytes <= c->ws_bytes; ++i) {
        if (even) {
          const double us = even_shares(*c, kv[i], q, diagonal);
          if (!best.parts || us < best.us) best = {c->parts, kv[i].shares, q_shares, us, kv[i].bytes + q.bytes};
          continue;
        }
        double us = makespan(kv[i].kind, q.kind, c->causal, k.start[c->form] + 2 * k.kv[c->form], k.tail, k.late);
        if (equal > 0) us += equal * std::max(0., placed(kv[i].kind.n, kv[i].kind.longest, q.kind.n, q.kind.longest) - us);
        us += kv[i].us + q.us;
        if (!best.parts || us < best.us) best = {c->parts, kv[i].shares, q_shares, us, kv[i].bytes + q.bytes};
        low = std::min(low, us);
        if (us > 1.5 * low) break;      // (nor with more)
      }
    }
  }
  return best;
}

// sequence: a causal call that stands for the pairs of several chunks; dk, dv as sums (no 4 parts at d = 128).  dq's walks may be shared
// with a few rows against many keys, and of a causal call of all gradients.
Plan plan(const dfa_shape& sh, int pairs, bool dq, bool dk, int64_t ws_bytes, bool sequence) {
  ws_bytes = std::min(ws_bytes, int64_t{128} << 20);
  const Undivided calls[] = {undivided(sh, pairs, dq, dk, ws_bytes, 1), undivided(sh, pairs, dq, dk, ws_bytes, 2),
                             undivided(sh, pairs, dq, dk, ws_bytes, 4)};
  const bool few = dq && sh.s_k / 8 >= sh.s_q, diagonal = sh.causal && dq && dk && pairs == 1;
  const bool even = sequence || (sh.d == 64 && sh.causal && sh.s_k > sh.s_q);
  return best_of(calls, sequence && sh.d == 128 ? 2 : 3, few ? 64 : diagonal ? 8 : 1, even, diagonal && !few);
}

}  // namespace

int launch_fwd_f32(const dfa_shape& sh, const dfa_fwd_pair* pairs, int n, hipStream_t st) {
  for (; n > MAX_PAIRS; pairs += MAX_PAIRS, n -= MAX_PAIRS) {
    const int rc = launch_fwd_f32(sh, pairs, MAX_PAIRS, st);
    if (rc) return rc;
  }
  auto operand = [](const void* x) { return static_cast<const float*>(x); };
  F32FwdBatch p{};
  static_cast<F32Params&>(p) = make_params(sh);
  const dfa_fwd_pair& x = pairs[0];
  p.q = operand(x.q); p.k = operand(x.k); p.v = operand(x.v); p.o = x.o; p.lse = x.lse; p.accumulate = x.accumulate;
  p.o_sh = x.o_stride_h; p.o_ss = x.o_stride_s; p.l_sh = x.lse_stride_h;
  p.pairs = n;
  if (n == 1) return fwd_form<F32Params>(p, sh, st);
  for (int i = 0; i < n; ++i) {
    const dfa_fwd_pair& y = pairs[i];
    p.fpair[i] = FwdPair{operand(y.q), operand(y.k), operand(y.v), y.o, y.lse, y.accumulate, y.o_stride_h, y.o_stride_s,
                         y.lse_stride_h};
  }
  return fwd_form<F32FwdBatch>(p, sh, st);
}

int launch_bwd_f32(const dfa_shape& sh, const dfa_bwd_pair* pairs, int n, bool sequence, void* ws, int64_t ws_bytes, hipStream_t st) {
  for (; n > MAX_PAIRS; pairs += MAX_PAIRS, n -= MAX_PAIRS) {
    const int rc = launch_bwd_f32(sh, pairs, MAX_PAIRS, sequence, ws, ws_bytes, st);
    if (rc) return rc;
  }
  F32BwdParams p{};
  static_cast<F32Params&>(p) = make_params(sh);
  p.pairs = n;
  for (int i = 0; i < n; ++i) {
    const dfa_bwd_pair& x = pairs[i];
    p.pair[i] = Pair{static_cast<const float*>(x.q), static_cast<const float*>(x.k), static_cast<const float*>(x.v),
                     static_cast<const float*>(x.dO), x.lse, x.delta, x.dq, x.dk, x.dv, x.accumulate_dq,
                     x.accumulate_dkv};
  }
  const Plan pl = plan(sh, n, pairs[0].dq, pairs[0].dk, ws ? ws_bytes : 0, sequence);
  p.shares = pl.shares;
  p.q_shares = pl.q_shares;
  p.partial = p.q_partial = static_cast<float*>(ws);
  if (sequence) {
    if (sh.d == 128) return pl.parts == 2 ? bwd<128, 2, true>(p, st) : bwd<128, 1, true>(p, st);
    return pl.parts == 4 ? bwd<64, 4, true>(p, st) : pl.parts == 2 ? bwd<64, 2, true>(p, st) : bwd<64, 1, true>(p, st);
  }
  if (sh.d == 128)
    return pl.parts == 4 ? bwd<128, 4, false>(p, st) : pl.parts == 2 ? bwd<128, 2, false>(p, st) : bwd<128, 1, false>(p, st);
  return pl.parts == 4 ? bwd<64, 4, false>(p, st) : pl.parts == 2 ? bwd<64, 2, false>(p, st) : bwd<64, 1, false>(p, st);
}

dfa_form bwd_f32_form(const dfa_shape& sh, int n, bool dq, bool dk, int64_t ws_bytes, bool sequence) {
  const Plan x = plan(sh, (n - 1) % MAX_PAIRS + 1, dq, dk, ws_bytes, sequence);
  return {128 / x.parts, x.parts, x.shares, x.q_shares};
}

int64_t bwd_f32_workspace(const dfa_shape& sh, int n, bool dq, bool dk, bool sequence) {
  return plan(sh, std::min(n, MAX_PAIRS), dq, dk, INT64_MAX, sequence).bytes;
}

int launch_span_f32(const dfa_shape& sh, const dfa_fwd_span* spans, int n, void* ws, int64_t ws_bytes, hipStream_t st) {
  const SpanPlan pl = span_plan(sh, spans, n, ws ? ws_bytes : 0);
  F32FwdSpans p{};
  static_cast<F32Params&>(p) = make_params(sh);
  p.causal = 1; p.pairs = 1;
  return run_spans<MAX_PAIRS>(sh, spans, n, pl.parts, ws, st, [&](const SpanPart* part, int count) {
    for (int i = 0; i < count; ++i) {
      const SpanPart& x = part[i];
      Span& y = p.span[i];
      y.q = static_cast<const float*>(x.q); y.k = static_cast<const float*>(x.k); y.v = static_cast<const float*>(x.v);
      y.o = x.o; y.lse = x.lse; y.accumulate = x.accumulate; y.o_sh = x.o_sh; y.o_ss = x.o_ss; y.l_sh = x.l_sh;
      y.s_k = x.n_keys; y.off = x.off; y.o_bf16 = x.o_bf16;
    }
    if (sh.d == 128) return pl.ns == 4 ? fwd_spans<128, 4>(p, count, st) : fwd_spans<128, 2>(p, count, st);
    return pl.ns == 4 ? fwd_spans<64, 4>(p, count, st) : fwd_spans<64, 2>(p, count, st);
  });
}

int64_t span_f32_workspace(const dfa_shape& sh, const dfa_fwd_span* spans, int n) {
  return parts_bytes(sh, spans, n, span_plan(sh, spans, n, MAX_SPAN_BYTES).parts);
}

dfa_form fwd_f32_form(const dfa_shape& sh, int n) {
  const int parts = fwd_parts(sh, (n - 1) % MAX_PAIRS + 1);
  return {128 / parts, parts, 1, 0};
}

dfa_form span_f32_form(const dfa_shape& sh, const dfa_fwd_span* spans, int n, int64_t ws_bytes) {
  const SpanPlan pl = span_plan(sh, spans, n, ws_bytes);
  return {128 / pl.ns, pl.ns, pl.parts, 0};
}

}  // namespace dfa

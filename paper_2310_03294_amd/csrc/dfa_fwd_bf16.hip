// bf16 forward chunk kernel for gfx950: attn(q_p, k_r, v_r) of one chunk pair from the empty
// state (forward pseudo-code of Appendix A; Eq. 1 restricted to one key/value chunk).
//
// Work decomposition.  A workgroup of 4 wavefronts owns 128 query rows of one head, each
// wavefront 32 of them, and walks over the key/value chunk in tiles of 64 rows staged in LDS.
// Per tile a wavefront computes S^T = K Q^T (keys x queries) so that every lane holds 32
// scores of ONE query: the running row maximum / row sum of the online softmax are then
// per-lane scalars plus one exchange between lane l and l+32.  The exponentiated tile is fed
// straight back, from registers, as the B operand of O^T += V^T P^T.
// Q stays in registers for the whole kernel; K/V tiles are copied from global memory straight
// into LDS (double-buffered); K is read from LDS with ds_read_b128, V with the transposing
// ds_read_b64_tr_b16.  The causal mask is applied only on tiles that straddle the
// diagonal; tiles above it are skipped.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "dfa_internal.h"
#include "dfa_mfma.h"
#include "dfa_span.h"

namespace dfa {
namespace {

constexpr int D = 128;
constexpr int BM = 128;     // query rows per workgroup
constexpr int BN = 64;      // key rows per LDS tile
constexpr int NTHREADS = 256;
constexpr int TILE_BYTES = BN * kRowBytes;   // rows padded to 272 B
constexpr float LOG2E = 1.4426950408889634f;

struct FwdParams {
  const __bf16 *q, *k, *v;
  void* o; float* lse;
  int s_q, s_k, h_q, group, causal, o_bf16, accumulate, ntq;
  XcdMap map;
  float scale;
  int64_t q_sh, q_ss, kv_sh, kv_ss, o_sh, o_ss, l_sh;
};

// Several pairs of one shape in a launch; the operands above are then not used.
struct Pair {
  const __bf16 *q, *k, *v;
  void* o; float* lse;
  int accumulate;
  int64_t o_sh, o_ss, l_sh;
};
constexpr int MAX_PAIRS = 16;       // per launch: the pairs travel in the kernel arguments
struct FwdBatch : FwdParams {
  int per_pair;                     // (head, query tile) items of a pair
  Pair pair[MAX_PAIRS];
};

// Spans: query chunks against consecutive keys, each span with a number of keys of its own, the last of which may be the
// chunk's own.  The longest walks come first: an XCD takes its heads of all spans, span by span (`heads` of them; 0: the
// heads do not divide into XCDs, and the items of a span go over all XCDs in turn).
struct Span : Pair { int s_k, off, o_bf16; };       // off: key kv is visible to query row i if kv <= i + off
struct FwdSpans : FwdParams {
  int per_pair, heads;
  Span span[MAX_PAIRS];
};
struct SpanParams : FwdParams { int off; };
template <class Args> constexpr bool kSpans = std::is_same_v<Args, FwdSpans>;

// Keys up to which query row 0 sees (a single pair or a list of pairs of equal chunks: its own).
template <class P> __device__ __forceinline__ int off_of(const P&) { return 0; }
__device__ __forceinline__ int off_of(const SpanParams& p) { return p.off; }

// The operands of an item's pair; item becomes its number within the pair.  (One pair alone is no list:
// picking it costs every workgroup another round trip to the argument memory.)
__device__ __forceinline__ const FwdParams& pair_of(const FwdParams& a, int&) { return a; }
__device__ __forceinline__ SpanParams pair_of(const FwdSpans& a, int& item) {
  int i = item / a.per_pair, r = item % a.per_pair;
  if (a.heads) {
    const int x = item / a.map.per_xcd, y = item % a.map.per_xcd, run = a.heads * a.ntq;      // items of a span on an XCD
    i = y / run; r = x * run + y % run;
  }
  item = r;
  SpanParams p;
  static_cast<FwdParams&>(p) = a;
  const Span& s = a.span[i];
  p.q = s.q; p.k = s.k; p.v = s.v; p.o = s.o; p.lse = s.lse; p.accumulate = s.accumulate;
  p.o_sh = s.o_sh; p.o_ss = s.o_ss; p.l_sh = s.l_sh; p.s_k = s.s_k; p.o_bf16 = s.o_bf16; p.off = s.off;
  return p;
}
__device__ __forceinline__ FwdParams pair_of(const FwdBatch& a, int& item) {
  FwdParams p = a;
  const Pair& x = a.pair[item / a.per_pair];
  item %= a.per_pair;
  p.q = x.q; p.k = x.k; p.v = x.v; p.o = x.o; p.lse = x.lse; p.accumulate = x.accumulate;
  p.o_sh = x.o_sh; p.o_ss = x.o_ss; p.l_sh = x.l_sh;
  return p;
}

// O^T tile of one query row per lane, read from (the state of earlier chunks) and written to memory
__device__ __forceinline__ void load_o(f32x16 (&o)[4], const FwdParams& p, int head, int qrow, int hh) {
  const int64_t obase = head * p.o_sh + static_cast<int64_t>(qrow) * p.o_ss;
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const int col = db * 32 + g4 * 8 + hh * 4;
      if (p.o_bf16) {
        const bf16x4 b = *reinterpret_cast<const bf16x4*>(static_cast<const __bf16*>(p.o) + obase + col);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[db][g4 * 4 + e] = static_cast<float>(b[e]);
      } else {
        const float4 x = *reinterpret_cast<const float4*>(static_cast<const float*>(p.o) + obase + col);
        o[db][g4 * 4] = x.x; o[db][g4 * 4 + 1] = x.y; o[db][g4 * 4 + 2] = x.z; o[db][g4 * 4 + 3] = x.w;
      }
    }
}
__device__ __forceinline__ void store_o(const f32x16 (&o)[4], const FwdParams& p, int head, int qrow, int hh, float inv) {
  const int64_t obase = head * p.o_sh + static_cast<int64_t>(qrow) * p.o_ss;
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const int col = db * 32 + g4 * 8 + hh * 4;
      const float x0 = o[db][g4 * 4 + 0] * inv, x1 = o[db][g4 * 4 + 1] * inv;
      const float x2 = o[db][g4 * 4 + 2] * inv, x3 = o[db][g4 * 4 + 3] * inv;
      if (p.o_bf16) {
        bf16x4 b; b[0] = static_cast<__bf16>(x0); b[1] = static_cast<__bf16>(x1);
        b[2] = static_cast<__bf16>(x2); b[3] = static_cast<__bf16>(x3);
        *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.o) + obase + col) = b;
      } else {
        *reinterpret_cast<float4*>(static_cast<float*>(p.o) + obase + col) = make_float4(x0, x1, x2, x3);
      }
    }
}

// FULL: a full pair.  Its row sums are taken over the bf16-rounded weights that multiply V, those of the diagonal pair
// over the fp32 weights (the same in the other forms of 128 and 256 rows).
template <bool FULL, class Args>
__global__ void __launch_bounds__(NTHREADS, 2) k_fwd_bf16(Args a) {
  extern __shared__ __align__(16) char smem[];   // two (K tile, V tile) buffers

  const int bid = blockIdx.x;
  int item = xcd_item(a.map, bid);
  if (item >= a.map.total) return;
  const FwdParams& p = pair_of(a, item);
  const int head = item / p.ntq;
  int tq = item % p.ntq;
  if (p.causal) tq = p.ntq - 1 - tq;      // longest rows first
  const int kh = head / p.group;
  const int q0 = tq * BM;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keeps tile branches scalar
  const int r32 = lane & 31, hh = lane >> 5;
  const int q0w = q0 + wave * 32;
  const int qrow = q0w + r32;
  const bool qvalid = qrow < p.s_q;
  const int a_base = tile_off(r32, hh);     // per-lane LDS bases; the rest of every address is constant
  const int g_base = gather_base(lane);

  const char* kg = reinterpret_cast<const char*>(p.k + kh * p.kv_sh);
  const char* vg = reinterpret_cast<const char*>(p.v + kh * p.kv_sh);
  const uint32_t kv_rowbytes = static_cast<uint32_t>(p.kv_ss) * 2;
  const TileLane tl = tile_lane(wave, lane, kv_rowbytes);

  // Q^T operand: lane holds Q[qrow][16 ks + 8 hh .. +7]
  bf16x8 qreg[8];
  {
    const __bf16* qp = p.q + head * p.q_sh + static_cast<int64_t>(qrow) * p.q_ss + 8 * hh;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      uint4 raw = make_uint4(0, 0, 0, 0);
      if (qvalid) raw = *reinterpret_cast<const uint4*>(qp + 16 * ks);
      qreg[ks] = __builtin_bit_cast(bf16x8, raw);
    }
  }

  f32x16 o[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) o[i][j] = 0.f;
  float m_run = -INFINITY;     // running maximum of the raw scores q.k
  float l_run = 0.f;           // this lane's half of the running row sum
  const float c2 = p.scale * LOG2E;
  if (p.accumulate && qvalid) {
    // State of the earlier key/value chunks: the normalised output with its logsumexp is the
    // running (o, m, l) with m = lse (in raw-score units: lse / scale) and l = 1.
    const float L = p.lse[head * p.l_sh + qrow];
    if (L > -INFINITY) {
      m_run = L / p.scale;
      l_run = hh == 0 ? 1.f : 0.f;
      load_o(o, p, head, qrow, hh);
    }
  }

  const int k_end = p.causal ? min(p.s_k, q0 + BM) : p.s_k;
  const int ntiles = (k_end + BN - 1) / BN;

  // K/V tiles go from global memory straight into LDS; key rows past s_k are clamped to the last
  // row and masked below.  Tile t + 1 is on its way while tile t is computed on.
  tile_dma(kg, kv_rowbytes, 0, p.s_k - 1, tl, smem, wave, lane);
  tile_dma(vg, kv_rowbytes, 0, p.s_k - 1, tl, smem + TILE_BYTES, wave, lane);
  lds_dma_wait();
  __syncthreads();

  // Online softmax of one 32-key block (exp2 domain, scores scaled by scale*log2 e), with a lazy
  // running maximum: the reference maximum m_run only moves when some row's block maximum exceeds
  // it by more than 2^8 in the exp2 domain (or on the first block).  Until then exponentials are
  // taken against the stale maximum - they stay below 2^8, harmless in fp32 / bf16 - and O needs
  // no rescaling; the final division by the row sum makes the result independent of the reference.
  // Returns the factor O has to be multiplied by (1 when the reference did not move).
  auto softmax_block = [&](f32x16& s, bf16x8 (&pb)[2]) {
    float mx = fmaxf(fmaxf(s[0], s[1]), s[2]);
#pragma unroll
    for (int j = 3; j < 15; j += 2) mx = fmaxf(fmaxf(mx, s[j]), s[j + 1]);
    mx = fmaxf(mx, s[15]);
    float alpha = 1.f;
    if (__any((mx - m_run) * c2 > 8.f)) {          // -inf reference (first block) also lands here
      mx = fmaxf(mx, __shfl_xor(mx, 32));
      const float m_new = fmaxf(m_run, mx);
      const float mc_new = (m_new == -INFINITY) ? 0.f : m_new * c2;
      alpha = __builtin_amdgcn_exp2f(m_run * c2 - mc_new);
      m_run = m_new;
      l_run *= alpha;
    }
    const float mc = (m_run == -INFINITY) ? 0.f : m_run * c2;
    float sum = 0.f;
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const float e = __builtin_amdgcn_exp2f(fmaf(s[j], c2, -mc));
      s[j] = e;
      if (!FULL) sum += e;
    }
    pb[0] = pack8(s, 0); pb[1] = pack8(s, 8);
    l_run += FULL ? sum8(pb[0], 0.f) + sum8(pb[1], 0.f) : sum;
    return alpha;
  };
  auto rescale_o = [&](float alpha) {
    if (__any(alpha != 1.f)) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) o[i][j] *= alpha;
    }
  };
  auto mask_block = [&](f32x16& s, int kbase) {
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      const int kvi = kbase + (j >> 2) * 8 + hh * 4 + (j & 3);
      if (kvi >= p.s_k || (p.causal && kvi > qrow)) s[j] = -INFINITY;
    }
  };

  for (int it = 0; it < ntiles; ++it) {
    const int k0 = it * BN;
    const bool more = it + 1 < ntiles;
    const int boff = (it & 1) * 2 * TILE_BYTES;
    const char* Ks = smem + boff;
    const char* Vs = Ks + TILE_BYTES;
    // The next K and V tiles into the other buffer, their pieces issued one at a time between the
    // MFMAs of stages 1 and 4 (in a burst they stall the wavefront while the memory pipe takes them
    // in).  After the last tile the same tile goes once more into the idle buffer: no branch
    // around the copies.
    const char* Kn = smem + (2 * TILE_BYTES - boff);
    const int kn0 = more ? k0 + BN : k0;
    const TileCopy ck = tile_copy_plan(kg, kv_rowbytes, kn0, p.s_k - 1, tl, Kn, wave, lane);
    const TileCopy cv = tile_copy_plan(vg, kv_rowbytes, kn0, p.s_k - 1, tl, Kn + TILE_BYTES, wave, lane);

    const bool active = !(p.causal && k0 > q0w + 31);
    if (!active) {      // nothing to compute for this wavefront's rows: only its share of the copies
      tile_copy_piece<0>(ck); tile_copy_piece<1>(ck); tile_copy_piece<2>(ck); tile_copy_piece<3>(ck);
      tile_copy_piece<0>(cv); tile_copy_piece<1>(cv); tile_copy_piece<2>(cv); tile_copy_piece<3>(cv);
      if (wave == 0) { tile_copy_piece<4>(ck); tile_copy_piece<4>(cv); }
    }
    if (active) {
      const bool need_mask = (k0 + BN > p.s_k) || (p.causal && k0 + BN - 1 > q0w);
      // Software pipeline over the two 32-key blocks of the tile: the MFMAs of one block run
      // under the softmax arithmetic of the other; LDS operand reads run ahead of their MFMAs.
      bf16x8 ka[4], gv[2], pb0[2], pb1[2];
      f32x16 s0, s1;
#pragma unroll
      for (int j = 0; j < 16; ++j) { s0[j] = 0.f; s1[j] = 0.f; }
#pragma unroll
      for (int ks = 0; ks < 4; ++ks) ka[ks] = lds_read_b128(Ks, a_base + ks * 32);
      DFA_SCHED_FENCE();
      // stage 1: S0^T = K0 Q^T
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        s0 = mfma32(ka[ks & 3], qreg[ks], s0);
        ka[ks & 3] = lds_read_b128(Ks, ks < 4 ? a_base + (ks + 4) * 32 : a_base + 32 * kRowBytes + (ks - 4) * 32);
        if (ks == 0) tile_copy_piece<0>(ck);
        if (ks == 2) tile_copy_piece<1>(ck);
        if (ks == 4) tile_copy_piece<2>(ck);
        if (ks == 6) tile_copy_piece<3>(ck);
        DFA_SCHED_FENCE();
      }
      if (wave == 0) { tile_copy_piece<4>(ck); tile_copy_piece<4>(cv); }
      if (need_mask) mask_block(s0, k0);
      DFA_SCHED_FENCE();
      // stage 2: S1^T = K1 Q^T  ||  softmax of block 0
      float alpha0;
      {
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {
          s1 = mfma32(ka[ks & 3], qreg[ks], s1);
          if (ks < 4) ka[ks & 3] = lds_read_b128(Ks, a_base + 32 * kRowBytes + (ks + 4) * 32);
        }
        gv[0] = lds_gather(Vs, g_base);
        gv[1] = lds_gather(Vs, g_base + 64);
        alpha0 = softmax_block(s0, pb0);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // 1 MFMA
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);   // 1 LDS read
          __builtin_amdgcn_sched_group_barrier(0x002, 9, 0);   // 9 VALU
        }
      }
      DFA_SCHED_FENCE();
      rescale_o(alpha0);
      if (need_mask) mask_block(s1, k0 + 32);
      DFA_SCHED_FENCE();
      // stage 3: O^T += V0^T P0^T  ||  softmax of block 1
      float alpha1;
      {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
          o[i & 3] = mfma32(gv[i & 1], pb0[i >> 2], o[i & 3]);
          const int n = i + 2;    // next gather: block 0 second half, then block 1
          gv[i & 1] = lds_gather(Vs, g_base + (n >> 2) * 16 * kRowBytes + (n & 3) * 64);
        }
        alpha1 = softmax_block(s1, pb1);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x002, 9, 0);
        }
      }
      DFA_SCHED_FENCE();
      rescale_o(alpha1);
      DFA_SCHED_FENCE();
      // stage 4: O^T += V1^T P1^T
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        o[i & 3] = mfma32(gv[i & 1], pb1[i >> 2], o[i & 3]);
        if (i + 2 < 8) {
          const int n = i + 10;
          gv[i & 1] = lds_gather(Vs, g_base + (n >> 2) * 16 * kRowBytes + (n & 3) * 64);
        }
        if (i == 0) tile_copy_piece<0>(cv);
        if (i == 2) tile_copy_piece<1>(cv);
        if (i == 4) tile_copy_piece<2>(cv);
        if (i == 6) tile_copy_piece<3>(cv);
        DFA_SCHED_FENCE();
      }
    }
    lds_dma_wait();
    __syncthreads();
  }

  // epilogue: combine the two half-sums, normalise, write O and the logsumexp
  const float l_tot = l_run + __shfl_xor(l_run, 32);
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  if (qvalid) {
    if (hh == 0) p.lse[head * p.l_sh + qrow] = l_tot > 0.f ? m_run * p.scale + logf(l_tot) : -INFINITY;
    store_o(o, p, head, qrow, hh, inv);
  }
}

// ============================================================================================
// Wavefront-specialised forward for full (unmasked) pairs: 16 wavefronts on 256 query rows, four
// per SIMD.
//   8 "S" wavefronts (32 query rows each, Q^T in registers): S^T = K Q^T, online softmax (one
//     reference update per 64-key tile), and the exponentiated tile P^T handed over through LDS as
//     bf16 together with the factor by which the running maximum moved; wavefronts 0-3 also issue
//     the global -> LDS copies of the K tiles, 4-7 those of the V tiles;
//   8 "PV" wavefronts (the same 32 rows each): O^T = O^T * factor + V^T P^T, one tile behind their
//     S wavefront, so one barrier per tile suffices; with only O^T to hold they read V^T six steps
//     ahead of their MFMAs.
// A wavefront overlaps nothing with itself (measured), different wavefronts of a SIMD do: here the
// exponentials of two S wavefronts run under the MFMAs of all four.  Measured against the
// 4-wavefront kernel above: 10 % faster on a 4096 x 4096 pair in spite of a lower clock under
// load (1.8 GHz).  On the causal diagonal pair its 256-row granularity costs half a row block per row
// of tiles: slower than the kernel above up to about 6000 rows, 8 % faster at 16384.
// ============================================================================================
namespace full_pair {

constexpr int NT = 1024;
constexpr int BMW = 256;                       // query rows per workgroup
constexpr int PX_BYTES = 8 * 4096;             // P^T hand-over: 8 query blocks x (64 keys x 32 queries bf16)
constexpr int AL_BYTES = 8 * 32 * 4;           // rescale factor per query row
// LDS map.  Tile t: K slot t % 2, V slot t % 3, P^T / factor slot t % 2; row statistics at the end.
constexpr int OFF_K = 0;
constexpr int OFF_V = OFF_K + 2 * TILE_BYTES;
constexpr int OFF_PX = OFF_V + 3 * TILE_BYTES;
constexpr int OFF_AL = OFF_PX + 2 * PX_BYTES;
constexpr int OFF_ST = OFF_AL + 2 * AL_BYTES;  // 1 / row sum, written once by the S wavefronts
constexpr int SMEM_BYTES = OFF_ST + AL_BYTES;

// RAGGED: s_k is no multiple of the 64-row tile, so the last K/V tile has rows past the end.
// CAUSAL: the diagonal pair; its row sums are taken over the fp32 weights, as in the other causal forms (of a span: where a tile
// has keys of the chunk's own; before them over the rounded weights, as for full pairs).
template <bool RAGGED, bool CAUSAL, class Args>
__global__ void __launch_bounds__(NT, 1) k_fwd_bf16(Args a) {
  extern __shared__ __align__(16) char smem[];

  const int bid = blockIdx.x;
  int item = xcd_item(a.map, bid);
  if (item >= a.map.total) return;
  const auto& p = pair_of(a, item);
  const int head = item / p.ntq;
  int tq = item % p.ntq;
  if (CAUSAL) tq = p.ntq - 1 - tq;      // longest rows first
  const int kh = head / p.group;
  const int q0 = tq * BMW;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: role branches stay scalar
  const bool pv_wave = wave >= 8;
  const int r32 = lane & 31, hh = lane >> 5;
  const float c2 = p.scale * LOG2E;

  const int off = off_of(p);
  const int k_end = CAUSAL ? min(p.s_k, q0 + BMW + off) : p.s_k;
  const int ntiles = (k_end + BN - 1) / BN;

  if (!pv_wave) {
    // ------------------------------------------------------------------ S wavefront
    const int q0w = q0 + wave * 32;
    const int qrow = q0w + r32;
    const bool qvalid = qrow < p.s_q;
    const int a_base = tile_off(r32, hh);
    bf16x8 qreg[8];      // Q^T operand: lane holds Q[qrow][16 ks + 8 hh .. +7]
    {
      const __bf16* qp = p.q + head * p.q_sh + static_cast<int64_t>(qvalid ? qrow : 0) * p.q_ss + 8 * hh;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        uint4 raw = *reinterpret_cast<const uint4*>(qp + 16 * ks);
        if (!qvalid) raw = make_uint4(0, 0, 0, 0);
        qreg[ks] = __builtin_bit_cast(bf16x8, raw);
      }
    }
    float m_run = -INFINITY;     // running maximum of the raw scores q.k
    float l_run = 0.f;           // this lane's half of the running row sum
    if (p.accumulate && qvalid) {
      // state of the earlier key/value chunks: running (o, m, l) with m = lse (raw-score units), l = 1
      const float L = p.lse[head * p.l_sh + qrow];
      if (L > -INFINITY) { m_run = L / p.scale; l_run = hh == 0 ? 1.f : 0.f; }
    }
    float* al = reinterpret_cast<float*>(smem + OFF_AL) + wave * 32 + r32;
    // the S wavefronts (registers to spare) issue the global -> LDS copies of the K/V tiles
    const char* kg = reinterpret_cast<const char*>(p.k + kh * p.kv_sh);
    const char* vg = reinterpret_cast<const char*>(p.v + kh * p.kv_sh);
    const uint32_t kv_rowbytes = static_cast<uint32_t>(p.kv_ss) * 2;
    const TileLane tl = tile_lane(wave & 3, lane, kv_rowbytes);
    const char* cg = wave < 4 ? kg : vg;      // wavefronts 0-3 copy K tiles, 4-7 V tiles
    const int last = p.s_k - 1;
    tile_dma(cg, kv_rowbytes, 0, last, tl, wave < 4 ? smem + OFF_K : smem + OFF_V, wave & 3, lane);
    lds_dma_wait();
    __syncthreads();                         // tile 0 is in LDS
    for (int it = 0; it < ntiles; ++it) {
      const int k0 = it * BN;
      const char* Ks = smem + OFF_K + (it & 1) * TILE_BYTES;
      // This wavefront's pieces of the next K (or V) tile, issued one at a time between the MFMAs
      // below: in a burst they would stall it while the memory pipe takes them in.  After the last
      // tile the same tile goes once more into a ring slot nobody reads (no branch around the copies).
      const TileCopy cn = tile_copy_plan<RAGGED>(cg, kv_rowbytes, it + 1 < ntiles ? k0 + BN : k0, last, tl,
                                         wave < 4 ? smem + OFF_K + ((it + 1) & 1) * TILE_BYTES
                                                  : smem + OFF_V + ((it + 1) % 3) * TILE_BYTES,
                                         wave & 3, lane);
      const bool active = !(CAUSAL && k0 > q0w + 31 + off);   // else: the whole tile lies above this block's diagonal
      if (!active) {
        tile_copy_piece<0>(cn); tile_copy_piece<1>(cn); tile_copy_piece<2>(cn); tile_copy_piece<3>(cn);
        if ((wave & 3) == 0) tile_copy_piece<4>(cn);
      }
      if (active) {
        f32x16 s0, s1;
        // S^T = K Q^T of the tile's two 32-key blocks.  COPIES: this wavefront's pieces of the next
        // tile's copy go out between the MFMAs (false when the products are done a second time).
        auto s_products = [&](auto copies) {
          constexpr bool COPIES = decltype(copies)::value;
          bf16x8 x0[4], x1[4];
          f32x16 zero;
#pragma unroll
          for (int j = 0; j < 16; ++j) zero[j] = 0.f;
#pragma unroll
          for (int ks = 0; ks < 3; ++ks) {
            x0[ks] = lds_read_b128(Ks, a_base + ks * 32);
            x1[ks] = lds_read_b128(Ks, a_base + 32 * kRowBytes + ks * 32);
          }
          DFA_SCHED_FENCE();
          __builtin_amdgcn_s_setprio(3);         // MFMAs first: the other wavefronts' VALU work fills the gaps
#pragma unroll
          for (int ks = 0; ks < 8; ++ks) {
            if (ks + 3 < 8) {
              x0[(ks + 3) & 3] = lds_read_b128(Ks, a_base + (ks + 3) * 32);
              x1[(ks + 3) & 3] = lds_read_b128(Ks, a_base + 32 * kRowBytes + (ks + 3) * 32);
            }
            s0 = mfma32(x0[ks & 3], qreg[ks], ks == 0 ? zero : s0);
            s1 = mfma32(x1[ks & 3], qreg[ks], ks == 0 ? zero : s1);
            if (COPIES) {
              if (ks == 0) tile_copy_piece<0>(cn);
              if (ks == 2) tile_copy_piece<1>(cn);
              if (ks == 4) tile_copy_piece<2>(cn);
              if (ks == 6) tile_copy_piece<3>(cn);
            }
            DFA_SCHED_FENCE();
          }
          __builtin_amdgcn_s_setprio(0);
          if (COPIES && (wave & 3) == 0) tile_copy_piece<4>(cn);
          if ((k0 + BN > p.s_k) || (CAUSAL && k0 + BN - 1 > q0w + off)) {
#pragma unroll
            for (int j = 0; j < 16; ++j) {
              const int kvi = k0 + (j >> 2) * 8 + hh * 4 + (j & 3);
              if (kvi >= p.s_k || (CAUSAL && kvi > qrow + off)) s0[j] = -INFINITY;
              if (kvi + 32 >= p.s_k || (CAUSAL && kvi + 32 > qrow + off)) s1[j] = -INFINITY;
            }
          }
        };
        // Moves the reference maximum up to the tile's row maxima; returns the factor by which what
        // has been accumulated against the old reference shrinks.
        auto new_reference = [&]() {
          float mx = fmaxf(s0[0], s1[0]);
#pragma unroll
          for (int j = 1; j < 16; ++j) mx = fmaxf(fmaxf(mx, s0[j]), s1[j]);
          mx = fmaxf(mx, __shfl_xor(mx, 32));
          const float m_new = fmaxf(m_run, mx);
          const float mc_new = (m_new == -INFINITY) ? 0.f : m_new * c2;
          const float a = __builtin_amdgcn_exp2f(m_run * c2 - mc_new);
          m_run = m_new;
          l_run *= a;
          return a;
        };
        // P^T = exp2(S^T c - reference) rounded to bf16, and this lane's half of the tile's row sum, taken
        // over the ROUNDED values (v_dot2c_f32_bf16 against a pair of ones: one instruction per two
        // scores), so that the sum that normalises O is the sum of exactly the weights that multiply V.
        bf16x8 p0, p1, p2, p3;
        const bool rounded = kSpans<Args> ? k0 + BN <= off : !CAUSAL;
        auto exponentials = [&]() {
          const float mc = (m_run == -INFINITY) ? 0.f : m_run * c2;
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            s0[j] = __builtin_amdgcn_exp2f(fmaf(s0[j], c2, -mc));
            s1[j] = __builtin_amdgcn_exp2f(fmaf(s1[j], c2, -mc));
          }
          p0 = pack8(s0, 0); p1 = pack8(s0, 8); p2 = pack8(s1, 0); p3 = pack8(s1, 8);
          // independent chains, so that the adds do not wait for one another
          if (!rounded) {
            float a[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int j = 0; j < 16; ++j) { a[j & 1] += s0[j]; a[2 + (j & 1)] += s1[j]; }
            return (a[0] + a[1]) + (a[2] + a[3]);
          }
          const float sa = sum8(p2, sum8(p0, 0.f)), sb = sum8(p3, sum8(p1, 0.f));
          return sa + sb;
        };
        // Online softmax of the 64-key tile (exp2 domain) against a reference maximum that is only
        // moved when it has to be.  A tile is first exponentiated against the reference as it stands,
        // without looking for its maximum: as long as no score lies more than 2^14 above the
        // reference, the exponentials are harmless in fp32 / bf16, O needs no rescaling, and the final
        // division by the row sum removes the reference.  The reference is derived from the scores
        // themselves (row maximum, one exchange between the two half rows) on a row's first tile -
        // so the largest weight seen is at least 1 and later tiles cannot underflow the row sum - and
        // again when a tile's half-row sum shows a score far above it (or is no number): that tile's
        // products are then done once more and the tile is redone with the moved reference.
        float alpha = 1.f;
        s_products(std::true_type{});
        const bool fresh = __any(m_run == -INFINITY);
        if (fresh) alpha = new_reference();
        float sum = exponentials();
        if (!fresh && __any(!(sum <= 16384.f))) {
          s_products(std::false_type{});
          alpha = new_reference();
          sum = exponentials();
        }
        l_run += sum;
        // hand P^T and the factor to the PV wavefront: lane-private, any layout will do
        char* px = smem + OFF_PX + (it & 1) * PX_BYTES + wave * 4096 + lane * 16;
        *reinterpret_cast<bf16x8*>(px) = p0;
        *reinterpret_cast<bf16x8*>(px + 1024) = p1;
        *reinterpret_cast<bf16x8*>(px + 2048) = p2;
        *reinterpret_cast<bf16x8*>(px + 3072) = p3;
        if (hh == 0) al[(it & 1) * (AL_BYTES / 4)] = alpha;
      }
      lds_dma_wait();
      __syncthreads();
    }
    // row statistics: logsumexp to memory, 1 / row sum to the PV wavefront
    const float l_tot = l_run + __shfl_xor(l_run, 32);
    if (hh == 0) {
      reinterpret_cast<float*>(smem + OFF_ST)[wave * 32 + r32] = l_tot > 0.f ? 1.f / l_tot : 0.f;
      if (qvalid) p.lse[head * p.l_sh + qrow] = l_tot > 0.f ? m_run * p.scale + logf(l_tot) : -INFINITY;
    }
    __syncthreads();                         // the PV wavefronts' last slot
  } else {
    // ------------------------------------------------------------------ PV wavefront
    const int sw = wave - 8;                 // serves S wavefront sw: the same 32 query rows
    const int q0w = q0 + sw * 32;
    const int qrow = q0w + r32;
    const bool qvalid = qrow < p.s_q;
    const int g_base = gather_base(lane);

    f32x16 o[4];         // O^T: [d block][d within block][query]
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) o[i][j] = 0.f;
    if (p.accumulate && qvalid && p.lse[head * p.l_sh + qrow] > -INFINITY) load_o(o, p, head, qrow, hh);
    // O^T = O^T * factor + V^T P^T for tile t (skipped when the tile lies above the block's diagonal)
    auto pv_tile = [&](int t) {
      const int k0 = t * BN;
      if (CAUSAL && k0 > q0w + 31 + off) return;
      const char* Vs = smem + OFF_V + (t % 3) * TILE_BYTES;
      const char* px = smem + OFF_PX + (t & 1) * PX_BYTES + sw * 4096 + lane * 16;
      const float a = reinterpret_cast<const float*>(smem + OFF_AL)[(t & 1) * (AL_BYTES / 4) + sw * 32 + r32];
      constexpr int AHEAD = 6;               // V^T gathers run this many steps ahead of their MFMAs
      const uint32_t vb = lds_pin(lds_addr(Vs) + g_base);
      auto voff = [&](int n) {               // n = key block * 8 + half * 4 + d block
        return ((n >> 3) * 32 + ((n >> 2) & 1) * 16) * kRowBytes + (n & 3) * 64;
      };
      bf16x8 y[AHEAD + 1], pa[4];
#pragma unroll
      for (int j = 0; j < 4; ++j) pa[j] = *reinterpret_cast<const bf16x8*>(px + j * 1024);
#pragma unroll
      for (int n = 0; n < AHEAD; ++n) y[n] = lds_gather_at(vb, voff(n));
      if (__any(a != 1.f)) {
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int j = 0; j < 16; ++j) o[i][j] *= a;
      }
      DFA_SCHED_FENCE();
      __builtin_amdgcn_s_setprio(3);
#pragma unroll
      for (int n = 0; n < 16; ++n) {
        if (n + AHEAD < 16) y[(n + AHEAD) % (AHEAD + 1)] = lds_gather_at(vb, voff(n + AHEAD));
        o[n & 3] = mfma32(y[n % (AHEAD + 1)], pa[n >> 2], o[n & 3]);
        DFA_SCHED_FENCE();
      }
      __builtin_amdgcn_s_setprio(0);
    };

    __syncthreads();                         // tile 0 is in LDS
    for (int it = 0; it < ntiles; ++it) {    // slot it: finish tile it - 1
      if (it > 0) pv_tile(it - 1);
      __syncthreads();
    }
    pv_tile(ntiles - 1);
    __syncthreads();                         // row statistics are in LDS

    if (qvalid) {
      const float inv = reinterpret_cast<const float*>(smem + OFF_ST)[sw * 32 + r32];
      store_o(o, p, head, qrow, hh, inv);
    }
  }
}

}  // namespace full_pair

// ============================================================================================
// Forward for calls that do not fill the device, full or causal: a workgroup owns RB blocks of 32 rows and its
// wavefronts divide the KEYS as well, NS parts of 32 keys per tile (RB = 2, NS = 2: 64 rows, 4 wavefronts,
// 64-key tiles, two workgroups per CU; RB = 2, NS = 4: 8 wavefronts, 128-key tiles, one workgroup per CU;
// RB = 4, NS = 2: 128 rows, 8 wavefronts, 64-key tiles, one workgroup per CU, two wavefronts per SIMD).  Every wavefront runs its
// own online softmax over its keys; the parts of a row block are combined through LDS at the end.
// Such a call is bound by the serial walk over the key tiles with most CUs idle: this form has 2-4
// times the workgroups and each wavefront 1/NS of the walk (8 heads x 2048 x 2048: 52 us with 256-row
// workgroups, 43 with 128-row ones, 34 here).  Where the device is full it is the slowest form: one
// 32-key block per wavefront and tile leaves its exponentials uncovered.
// LO (64 rows): the matrix pipes have room, so the weights enter the second product as two bf16 values, the
// rounded weight and its remainder (o is then off by 2^-17 of a weight instead of 2^-9, for 1 us of 18 at 8 heads x 1024), and the row sums
// are fp32 sums of the fp32 weights.  With 128 rows rounding and sums are those of the 128-row kernel.
// A remainder is zero or negative as often as not: against an infinite value of V the two products give NaN, where the
// rounded weight alone gives that infinity.  A workgroup that ends with a value that is not finite therefore walks over
// its keys once more without the remainders.  (Looking for one takes 0.15 to 0.3 us of a call: 8 heads x 256 8.7 -> 9.0 us, x 1024
// 18.4 -> 18.55; with both walks as one loop body the causal form spilled.)
// ============================================================================================
namespace split {

template <int NS> constexpr int kKeys = 32 * NS;                          // keys per tile
template <int NS> constexpr int kTilesBytes = 2 * (kKeys<NS> / BN) * TILE_BYTES;      // K and V of one tile
template <int NS> constexpr int kSmem = 2 * kTilesBytes<NS>;
constexpr int RES_BYTES = 64 * 64 * 4;         // a wavefront's O^T, 64 registers per lane

template <int RB, int NS, bool CAUSAL, class Args>
__global__ void __launch_bounds__(RB * NS * 64, RB * NS == 4 ? 2 : 1) k_fwd_bf16(Args a) {
  constexpr int BMS = RB * 32;                 // query rows per workgroup
  constexpr bool LO = RB == 2;
  constexpr int SUB = kKeys<NS> / BN;          // 64-row sub-tiles of a K (or V) tile
  extern __shared__ __align__(16) char smem[]; // two buffers of (SUB K sub-tiles, SUB V sub-tiles)

  const int bid = blockIdx.x;
  int item = xcd_item(a.map, bid);
  if (item >= a.map.total) return;
  const auto& p = pair_of(a, item);
  const int head = item / p.ntq;
  int tq = item % p.ntq;
  if (CAUSAL) tq = p.ntq - 1 - tq;           // longest rows first
  const int kh = head / p.group;
  const int q0 = tq * BMS;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int rb = wave % RB, part = wave / RB;
  const int q0w = q0 + rb * 32;
  const float c2 = p.scale * LOG2E;

  const char* kg = reinterpret_cast<const char*>(p.k + kh * p.kv_sh);
  const char* vg = reinterpret_cast<const char*>(p.v + kh * p.kv_sh);
  const uint32_t kv_rowbytes = static_cast<uint32_t>(p.kv_ss) * 2;
  const int off = off_of(p);
  const int k_end = CAUSAL ? min(p.s_k, q0 + BMS + off) : p.s_k;
  const int ntiles = (k_end + kKeys<NS> - 1) / kKeys<NS>;
  // wavefronts 4s .. 4s + 3 copy sub-tile s of K and of V
  // (8 wavefronts and one sub-tile: 0-3 copy K, 4-7 copy V)
  constexpr bool ONE = RB * NS == 8 && SUB == 1;
  const int cw = wave & 3, sub = ONE ? 0 : wave >> 2;
  const bool v_copy = ONE && wave >= 4;
  const int last = p.s_k - 1;
  const int koff = sub * TILE_BYTES, voff = (SUB + sub) * TILE_BYTES;

  f32x16 o[4];
  float m_run, l_run;                          // raw-score units; l_run: this lane's half of the row sum
  int lane = threadIdx.x & 63;

  // The walk over the keys.  REM: the weights' remainders too.
  auto walk = [&](auto rem) {
    constexpr bool REM = decltype(rem)::value;
    if constexpr (LO) lane = static_cast<int>(lds_pin(lane));      // opaque: no walk keeps registers for the other
    const int r32 = lane & 31, hh = lane >> 5;
    const int qrow = q0w + r32;
    const bool qvalid = qrow < p.s_q;
    const int a_base = tile_off(r32, hh);
    const int g_base = gather_base(lane);
    const TileLane tl = tile_lane(cw, lane, kv_rowbytes);
    // rows past the end are clamped to the last row (and masked); a sub-tile wholly past it likewise
    tile_dma(v_copy ? vg : kg, kv_rowbytes, sub * BN, last, tl, smem + (v_copy ? voff : koff), cw, lane);
    if (!ONE) tile_dma(vg, kv_rowbytes, sub * BN, last, tl, smem + voff, cw, lane);

    bf16x8 qreg[8];
    {
      const __bf16* qp = p.q + head * p.q_sh + static_cast<int64_t>(qvalid ? qrow : 0) * p.q_ss + 8 * hh;
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) {
        uint4 raw = *reinterpret_cast<const uint4*>(qp + 16 * ks);
        if (!qvalid) raw = make_uint4(0, 0, 0, 0);
        qreg[ks] = __builtin_bit_cast(bf16x8, raw);
      }
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) o[i][j] = 0.f;
    m_run = -INFINITY; l_run = 0.f;
    if (p.accumulate && part == 0 && qvalid) {   // the state of the earlier chunks goes into the first part
      const float L = p.lse[head * p.l_sh + qrow];
      if (L > -INFINITY) {
        m_run = L / p.scale;
        l_run = hh == 0 ? 1.f : 0.f;
        load_o(o, p, head, qrow, hh);
      }
    }
    lds_dma_wait();
    __syncthreads();

    for (int it = 0; it < ntiles; ++it) {
      const int k0 = it * kKeys<NS>;
      const char* buf = smem + (it & 1) * kTilesBytes<NS>;
      char* nbuf = smem + ((it & 1) ^ 1) * kTilesBytes<NS>;
      const int kn = (it + 1 < ntiles ? k0 + kKeys<NS> : k0) + sub * BN;
      const TileCopy ck = tile_copy_plan(v_copy ? vg : kg, kv_rowbytes, kn, last, tl, nbuf + (v_copy ? voff : koff), cw, lane);
      const TileCopy cv = tile_copy_plan(vg, kv_rowbytes, kn, last, tl, nbuf + voff, cw, lane);
      const int kb0 = k0 + part * 32;            // this wavefront's 32 keys
      const char* Ks = buf + (part >> 1) * TILE_BYTES;
      const char* Vs = Ks + SUB * TILE_BYTES;
      const int row = (part & 1) * 32 * kRowBytes;
      if (kb0 < p.s_k && !(CAUSAL && kb0 > q0w + 31 + off)) {
        bf16x8 ka[4], gv[4];
        f32x16 s;
#pragma unroll
        for (int j = 0; j < 16; ++j) s[j] = 0.f;
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) ka[ks] = lds_read_b128(Ks, a_base + row + ks * 32);
        DFA_SCHED_FENCE();
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) {         // S^T = K Q^T
          s = mfma32(ka[ks & 3], qreg[ks], s);
          if (ks < 4) ka[ks & 3] = lds_read_b128(Ks, a_base + row + (ks + 4) * 32);
          if (ks == 0) tile_copy_piece<0>(ck);
          if (ks == 2) tile_copy_piece<1>(ck);
          if (ks == 4) tile_copy_piece<2>(ck);
          if (ks == 6) tile_copy_piece<3>(ck);
          DFA_SCHED_FENCE();
        }
        if (cw == 0) { tile_copy_piece<4>(ck); if (!ONE) tile_copy_piece<4>(cv); }
#pragma unroll
        for (int i = 0; i < 4; ++i) gv[i] = lds_gather(Vs, g_base + row + i * 64);
        if (kb0 + 32 > p.s_k || (CAUSAL && kb0 + 31 > q0w + off)) {
#pragma unroll
          for (int j = 0; j < 16; ++j) {
            const int kvi = kb0 + (j >> 2) * 8 + hh * 4 + (j & 3);
            if (kvi >= p.s_k || (CAUSAL && kvi > qrow + off)) s[j] = -INFINITY;
          }
        }
        // online softmax with the lazy running maximum of the 128-row kernel
        float mx = fmaxf(fmaxf(s[0], s[1]), s[2]);
#pragma unroll
        for (int j = 3; j < 15; j += 2) mx = fmaxf(fmaxf(mx, s[j]), s[j + 1]);
        mx = fmaxf(mx, s[15]);
        float alpha = 1.f;
        if (__any((mx - m_run) * c2 > 8.f)) {
          mx = fmaxf(mx, __shfl_xor(mx, 32));
          const float m_new = fmaxf(m_run, mx);
          const float mc_new = (m_new == -INFINITY) ? 0.f : m_new * c2;
          alpha = __builtin_amdgcn_exp2f(m_run * c2 - mc_new);
          m_run = m_new;
          l_run *= alpha;
        }
        const float mc = (m_run == -INFINITY) ? 0.f : m_run * c2;
        const bool rounded = !LO && (kSpans<Args> ? kb0 + 32 <= off : !CAUSAL);
        float sum = 0.f;
#pragma unroll
        for (int j = 0; j < 16; ++j) s[j] = __builtin_amdgcn_exp2f(fmaf(s[j], c2, -mc));
        if (!rounded) {
#pragma unroll
          for (int j = 0; j < 16; ++j) sum += s[j];
        }
        if (__any(alpha != 1.f)) {
#pragma unroll
          for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int j = 0; j < 16; ++j) o[i][j] *= alpha;
        }
        bf16x8 pb[2], pl[2];                     // the weights, and what rounding them to bf16 left over
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          pb[u] = pack8(s, 8 * u);
          if constexpr (REM) {
#pragma unroll
            for (int e = 0; e < 8; ++e) s[8 * u + e] -= static_cast<float>(pb[u][e]);
            pl[u] = pack8(s, 8 * u);
          }
          if (rounded) sum = sum8(pb[u], sum);
        }
        l_run += sum;
        DFA_SCHED_FENCE();
#pragma unroll
        for (int i = 0; i < 8; ++i) {            // O^T += V^T P^T
          o[i & 3] = mfma32(gv[i & 3], pb[i >> 2], o[i & 3]);
          if constexpr (REM) o[i & 3] = mfma32(gv[i & 3], pl[i >> 2], o[i & 3]);
          if (i < 4) gv[i & 3] = lds_gather(Vs, g_base + row + 16 * kRowBytes + i * 64);
          if (!ONE && i == 0) tile_copy_piece<0>(cv);
          if (!ONE && i == 2) tile_copy_piece<1>(cv);
          if (!ONE && i == 4) tile_copy_piece<2>(cv);
          if (!ONE && i == 6) tile_copy_piece<3>(cv);
          DFA_SCHED_FENCE();
        }
      } else {                                   // nothing for this wavefront: only its share of the copies
        tile_copy_piece<0>(ck); tile_copy_piece<1>(ck); tile_copy_piece<2>(ck); tile_copy_piece<3>(ck);
        if (cw == 0) tile_copy_piece<4>(ck);
        if (!ONE) {
          tile_copy_piece<0>(cv); tile_copy_piece<1>(cv); tile_copy_piece<2>(cv); tile_copy_piece<3>(cv);
          if (cw == 0) tile_copy_piece<4>(cv);
        }
      }
      lds_dma_wait();
      __syncthreads();
    }
  };
  // combine the parts of a row block in part 0, against the largest of their reference maxima
  float* st = reinterpret_cast<float*>(smem + RB * (NS - 1) * RES_BYTES);      // (m, l) per part and row
  float l_tot;
  auto leave = [&] {
    l_tot = l_run + __shfl_xor(l_run, 32);
    if (part > 0) {
      float* x = reinterpret_cast<float*>(smem + (wave - RB) * RES_BYTES) + lane;
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 16; ++j) x[(i * 16 + j) * 64] = o[i][j];
      if (lane < 32) { st[wave * 64 + lane] = m_run; st[wave * 64 + 32 + lane] = l_tot; }
    }
  };
  float m;                                     // the largest reference
  auto largest = [&] {
    m = m_run;
#pragma unroll
    for (int s = 1; s < NS; ++s) m = fmaxf(m, st[(s * RB + rb) * 64 + (lane & 31)]);
  };
  walk(std::bool_constant<LO>{});
  leave();
  if constexpr (LO) {
    int* odd = reinterpret_cast<int*>(st + RB * NS * 64);          // per wavefront: a value is not finite
    float top[4] = {0.f, 0.f, 0.f, 0.f};       // of the magnitudes; maximum() hands on what is no number
#pragma unroll
    for (int j = 0; j < 16; j += 2)
#pragma unroll
      for (int i = 0; i < 4; ++i)
        top[i] = __builtin_elementwise_maximum(__builtin_elementwise_maximum(top[i], fabsf(o[i][j])), fabsf(o[i][j + 1]));
    odd[wave] = __any(!(__builtin_elementwise_maximum(__builtin_elementwise_maximum(top[0], top[1]),
                                                      __builtin_elementwise_maximum(top[2], top[3])) < INFINITY));
    __syncthreads();
    int any = 0;
#pragma unroll
    for (int w = 0; w < RB * NS; ++w) any |= odd[w];
    largest();
    if (__builtin_expect(__builtin_amdgcn_readfirstlane(any), 0)) {
      __syncthreads();                         // the tiles go where the results are
      walk(std::false_type{});
      leave();
      __syncthreads();
      largest();
    }
  } else {
    __syncthreads();
    largest();
  }
  if (part > 0) return;
  const int r32 = lane & 31, hh = lane >> 5;
  const int qrow = q0w + r32;
  const bool qvalid = qrow < p.s_q;
  const float mc = (m == -INFINITY) ? 0.f : m * c2;
  const float f0 = __builtin_amdgcn_exp2f(m_run * c2 - mc);
  l_tot *= f0;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 16; ++j) o[i][j] *= f0;
#pragma unroll 1      // (unrolled, the reads of all parts are hoisted and spill)
  for (int s = 1; s < NS; ++s) {
    const int w = s * RB + rb;
    const float f = __builtin_amdgcn_exp2f(st[w * 64 + r32] * c2 - mc);
    l_tot = fmaf(st[w * 64 + 32 + r32], f, l_tot);
    const float* x = reinterpret_cast<const float*>(smem + (w - RB) * RES_BYTES) + lane;
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < 16; ++j) o[i][j] = fmaf(x[(i * 16 + j) * 64], f, o[i][j]);
  }
  if (!qvalid) return;
  if (hh == 0) p.lse[head * p.l_sh + qrow] = l_tot > 0.f ? m * p.scale + logf(l_tot) : -INFINITY;
  store_o(o, p, head, qrow, hh, l_tot > 0.f ? 1.f / l_tot : 0.f);
}

}  // namespace split

// > 64 KB of dynamic LDS needs the opt-in, once per kernel and process (thread-safe)
template <class Args, void (*KERNEL)(Args)>
int launch(const Args& p, int threads, int smem, hipStream_t st) {
  static std::once_flag once;
  static int attr_rc = DFA_OK;
  std::call_once(once, [smem] {
    attr_rc = hip_status(hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, smem));
  });
  if (attr_rc) return attr_rc;
  KERNEL<<<static_cast<int>(xcd_blocks(p.map)), threads, smem, st>>>(p);
  return last_launch_status();
}

// Diagonal pairs in the 64-row form, by the rows of a pair and the number of 64-row workgroups of all.
bool causal_with_remainders(int64_t s_q, int64_t n64) { return n64 <= 256 || (n64 <= 512 && s_q >= 2048); }

// The form of n pairs of one shape.  sequence: a causal call that stands for the pairs of several workers' chunks.
struct FwdForm { int rows, parts; };      // query rows of a workgroup, parts that it divides the keys of a tile in
FwdForm form_of(const dfa_shape& sh, int n, bool sequence) {
  // Which form.  us per call on one box, d = 128, 256-row / 128-row / 64-row NS = 2 / 64-row NS = 4 workgroups:
  //   full pairs    8 heads x 256 rows 13.5 / 9.6 / 8.6 / 9.5    x 1024 30.5 / 24.2 / 22 / 18.4
  //                 x 2048 52.5 / 42.7 / 40 / 34.2 (256 64-row workgroups)   x 4096 97 / 82 / 100 / 105
  //                 x 8192 242 / 270 / 344 / 382    32 heads x 1024 32.8 / 27.2 / 29.6 / 34.5
  //                 x 2777 162 / 147 / 184 / 205 (352 256-row workgroups)      x 4096 250 / 273 / 356 / 381
  //   causal        8 heads x 1024 29.9 / 24.8 / 21.5 / 19.4   x 4096 95 / 85 / 78 / 69
  //                 x 16384 492 / 564 / 720 / 800
  //                 32 heads x 1024 31.5 / 26.4 / 27.1 / 30.9   x 4096 179 / 174 / 195 / 221
  //                 x 8192 515 / 563 / 715 / 791   x 16384 1950 / 2112 / 2748 / 2985
  auto count = [&](int rows) { return (static_cast<int64_t>(sh.s_q) + rows - 1) / rows * sh.h_q * n; };
  const int64_t n256 = count(256), n128 = count(128), n64 = count(64);
  bool wide;          // 256 rows
  int parts = 0;      // 64 rows with this many parts
  bool two = false;   // 128 rows with two parts
  if (sh.causal) {
    // The diagonal's longest row block sets the time of a call that does not fill the device, so long
    // chunks are split further; the 256-row form needs chunks long enough that its masked half tiles do
    // not count, and whole tiles (ragged chunks, 32 heads x 14197: 1664 us against 1608 with 128 rows).
    if (causal_with_remainders(sh.s_q, n64)) parts = 4;
    // A sequence of several chunks, whose shortest lists of pairs have half as many workgroups at least.  us with 2 / 4 parts: 32
    // heads x 600 20.2 / 23.1, x 1024 32.7 / 35.4, 24 x 800 21.4 / 22.2, 16 x 1200 28.4 / 23.0, x 1400 31.9 / 26.3, x 2000 56 / 43.
    else if (sequence && n64 <= 512) parts = sh.s_q <= 1024 ? 2 : 4;
    wide = n256 >= 512 && sh.s_q >= 6144 && sh.s_k % BN == 0;
    // Two parts per tile where the 128-row form's longest walk decides: 16 heads x 2500 59 -> 51 us, x 4096
    // 117 -> 96, 8 x 6000 131 -> 112; not where short walks share the CUs anyway (32 x 1500 45 -> 49).  It is one workgroup
    // per CU, so more than 256 of them need the longer walks: 24 x 1500 (288) 37.5 -> 33.7, 32 x 1300 (352) 43 -> 41, but
    // 40 x 1024 (320) 36.8 -> 40.4, 64 x 566 (320) 21.2 -> 25.8; and fewer than that gain nothing below 1024 rows: 32 x 1024
    // 26.3 -> 26.2, x 700 18.8 -> 19.3, 64 x 384 14.8 -> 15.5.
    two = sh.s_q >= 1024 && n128 <= (sh.s_q > 2048 ? 512 : sh.s_q >= 1280 ? 352 : 256);
  } else {
    // (Calls whose rows are whole rounds of 256-row workgroups and a small rest come here as two: rows_of_whole_rounds.)
    // One round of 64-row workgroups at most: split the keys.  The 128-row form (10 % slower per row, two
    // workgroups per CU) where it needs one workgroup per CU at most, or where the last round of 256-row
    // workgroups would be half empty or worse.
    if (n64 <= 256) parts = 4;
    // Two parts per tile where the 128-row form would have one wavefront per SIMD (8 heads x 2777 57 -> 46 us, x
    // 4096 82 -> 72; 32 x 1024 27.4 -> 25.1), and for long walks up to two rounds of 256-row workgroups where that form is
    // no better (16 x 5500 282 -> 265, 24 x 3300 171 -> 165, 32 x 2777 156.5 -> 155.5; 32 x 5120, three rounds, 419 -> 434).  Up to
    // 2048 keys one part is the better: 64 x 1300 76 against 80 (256 rows: 81.5), 32 x 2700 x 2000 109 against 111 (116),
    // 128 x 700 x 500 41 against 46 (43).
    const int64_t last_round = n256 % 256;
    wide = n128 > 256 && !(n256 > 256 && n256 < 768 && last_round > 0 && last_round <= 128);
    two = n128 <= 256 || (n256 < 512 && sh.s_k > 2048);
  }
  if (parts) return {64, sh.s_k <= 384 ? 2 : parts};      // (three 128-key tiles at most: the smaller tiles start sooner)
  return wide ? FwdForm{256, 1} : FwdForm{128, two ? 2 : 1};
}

// n pairs of one shape (n > 1: in FwdBatch)
template <class Args>
int launch_form(Args& p, const dfa_shape& sh, int n, bool sequence, hipStream_t st) {
  const FwdForm form = form_of(sh, n, sequence);
  const int64_t heads = static_cast<int64_t>(sh.h_q) * n;
  if ((static_cast<int64_t>(sh.s_q) + 127) / 128 * heads > (1 << 30) && (sh.causal || n > 1)) return DFA_ERR_SHAPE;
  p.ntq = (sh.s_q + form.rows - 1) / form.rows;
  p.map = xcd_map(p.ntq * heads, sh.causal, heads);
  if constexpr (std::is_same_v<Args, FwdBatch>) p.per_pair = p.ntq * sh.h_q;
  if (form.rows == 64) {
    if (form.parts == 2) return sh.causal ? launch<Args, split::k_fwd_bf16<2, 2, true, Args>>(p, 256, split::kSmem<2>, st)
                                     : launch<Args, split::k_fwd_bf16<2, 2, false, Args>>(p, 256, split::kSmem<2>, st);
    return sh.causal ? launch<Args, split::k_fwd_bf16<2, 4, true, Args>>(p, 512, split::kSmem<4>, st)
                     : launch<Args, split::k_fwd_bf16<2, 4, false, Args>>(p, 512, split::kSmem<4>, st);
  }
  if (form.rows == 128 && form.parts == 2) {
    return sh.causal ? launch<Args, split::k_fwd_bf16<4, 2, true, Args>>(p, 512, split::kSmem<2>, st)
                     : launch<Args, split::k_fwd_bf16<4, 2, false, Args>>(p, 512, split::kSmem<2>, st);
  }
  if (form.rows == 128) {
    return sh.causal ? launch<Args, k_fwd_bf16<false, Args>>(p, NTHREADS, 4 * TILE_BYTES, st)
                     : launch<Args, k_fwd_bf16<true, Args>>(p, NTHREADS, 4 * TILE_BYTES, st);
  }
  constexpr int nt = full_pair::NT, smem = full_pair::SMEM_BYTES;
  const bool ragged = sh.s_k % BN != 0;
  if (sh.causal) return launch<Args, full_pair::k_fwd_bf16<false, true, Args>>(p, nt, smem, st);
  return ragged ? launch<Args, full_pair::k_fwd_bf16<true, false, Args>>(p, nt, smem, st)
                : launch<Args, full_pair::k_fwd_bf16<false, false, Args>>(p, nt, smem, st);
}

// Of which keys of a list of spans the weights enter with their remainders (64-row form): no fewer than in the pairs that the spans
// stand for, where launch_form takes each as a call of its own, or, with several owners, the pairs of a time step as one list.
//   ALL   (The form with 128 rows and remainders was tried: walk of 3 chunks of 8 heads x 1000 38.5 -> 43.4 us, of 5 x 2048 143.5 ->
//         145, of 9 x 2048 258 -> 245.  Without the remainders the latter two are 15 % faster, and o 200 times as far off.)
//   OWN   of the chunks' own: those go out as diagonal pairs, the keys before them as a walk that continues from there
//   NONE
enum class Remainders { ALL, OWN, NONE };

int64_t last_launch(int64_t pairs) { return (pairs - 1) % MAX_PAIRS + 1; }      // pairs of a list's last launch

Remainders remainders(const dfa_shape& sh, const dfa_fwd_span* spans, int n) {
  int64_t owners = 0, full = MAX_PAIRS;      // full: pairs of the smallest list of full pairs
  for (int i = 0; i < n; ++i) owners += spans[i].own != 0;
  if (owners < 2 || owners < n) full = 1;
  for (int i = 0; i < n && full > 1; ++i) {
    const int64_t step = (spans[i].n_keys - 1) / sh.s_q;      // the last one that this walk has a pair in
    int64_t list = 0;
    for (int j = 0; j < n; ++j) list += spans[j].n_keys > step * sh.s_q;
    if (step > 0) full = std::min(full, last_launch(list));
  }
  const int64_t n64 = (static_cast<int64_t>(sh.s_q) + 63) / 64 * sh.h_q;
  if (n64 * full <= 256) return Remainders::ALL;
  return owners && causal_with_remainders(sh.s_q, n64 * last_launch(owners)) ? Remainders::OWN : Remainders::NONE;
}

// Which form, and in how many parts the keys of a span are cut (the parts are merged afterwards): by an estimate launch by launch,
// fitted to 154 forwards of shares and windows of 64 to 5000 rows, every division timed (chosen / best 1.004 in the mean, none
// slower than the pairs one by one): 8 us and, per tile of 64 keys, 1.0 us with 64-row workgroups (four key parts), 1.3 with
// 128-row ones (two) and 1.7 with 256-row ones; a launch that runs in one round takes its longest walk, a longer one the device's
// even share and about half a walk; the merge 8 us and 3 TB/s.  (With 1.1 and 1.9, as measured on walks that fill the device less,
// 128 rows were taken too often: us, pairs / so / now: 32 over 8 heads, 3 chunks of 3200 476 / 550 / 431, 64 over 8, 2 of 704
// 53 / 59 / 40, 16 over 4, 3 of 4158 493 / 551 / 402.)
struct SpanPlan { int rows, parts; double us; };

SpanPlan span_plan(const dfa_shape& sh, const dfa_fwd_span* spans, int n, bool all_remainders, int64_t ws_bytes) {
  SpanPlan best{};
  for (int rows : {64, 128, 256}) {
    if (rows > 64 && all_remainders) break;
    const double tile = (rows == 64 ? 1.0 : rows == 128 ? 1.3 : 1.7) / BN;      // per key
    const int64_t blocks = (static_cast<int64_t>(sh.s_q) + rows - 1) / rows * sh.h_q;
    for (int parts : SPAN_CUTS) {
      const int64_t bytes = parts_bytes(sh, spans, n, parts);
      if (parts > 1 && (!bytes || bytes > ws_bytes)) break;
      const double us = sum_of_launches(sh, spans, n, parts, MAX_PAIRS, blocks, BN, [&](const LaunchWork& w) {
        double x = 8 + w.longest * tile;
        if (w.workgroups > 256) x = std::max(x, 8 + w.keys * tile / 256 + 0.45 * w.longest * tile);
        return x + (w.cut ? 8 + 2 * w.part_bytes / 3e6 : 0);
      });
      if (!best.rows || us < best.us) best = {rows, parts, us};
    }
  }
  return best;
}

int launch_spans(FwdSpans& p, const dfa_shape& sh, int n, int rows, hipStream_t st) {
  p.ntq = (sh.s_q + rows - 1) / rows;
  p.per_pair = p.ntq * sh.h_q;
  p.heads = sh.h_q % 8 == 0 ? sh.h_q / 8 : 0;
  if (static_cast<int64_t>(p.per_pair) * n > (1 << 30)) return DFA_ERR_SHAPE;
  p.map = xcd_map(static_cast<int64_t>(p.per_pair) * n, 1, p.heads ? 8 : 1);      // (1: every second row of items backwards)
  std::stable_sort(p.span, p.span + n, [](const Span& x, const Span& y) { return x.s_k > y.s_k; });
  if (rows == 64) return launch<FwdSpans, split::k_fwd_bf16<2, 4, true, FwdSpans>>(p, 512, split::kSmem<4>, st);
  if (rows == 128) return launch<FwdSpans, split::k_fwd_bf16<4, 2, true, FwdSpans>>(p, 512, split::kSmem<2>, st);
  constexpr int nt = full_pair::NT, smem = full_pair::SMEM_BYTES;
  bool whole = true;
  for (int i = 0; i < n; ++i) whole &= p.span[i].s_k % BN == 0;
  return whole ? launch<FwdSpans, full_pair::k_fwd_bf16<false, true, FwdSpans>>(p, nt, smem, st)
               : launch<FwdSpans, full_pair::k_fwd_bf16<true, true, FwdSpans>>(p, nt, smem, st);
}

// Spans without the keys of the chunks' own, which are diagonal pairs, of MAX_PAIRS spans at a time.
struct WithoutOwn {
  dfa_fwd_pair pair[MAX_PAIRS];
  dfa_fwd_span rest[MAX_PAIRS];
  int pairs = 0, spans = 0;
  bool chunks = true;      // what is left are single chunks: full pairs
  WithoutOwn(const dfa_shape& sh, const dfa_fwd_span* spans_, int n) {
    for (int i = 0; i < n; ++i) {
      dfa_fwd_span x = spans_[i];
      if (x.own) {
        x.n_keys -= sh.s_q;
        const int64_t own = x.n_keys * sh.kv_stride_s * 2;
        pair[pairs++] = {x.q, static_cast<const char*>(x.k) + own, static_cast<const char*>(x.v) + own, x.o, x.lse, x.o_stride_h,
                         x.o_stride_s, x.lse_stride_h, x.accumulate, 0};
        x.own = 0;
        x.accumulate = 1;
      }
      if (x.n_keys > 0) rest[spans++] = x;
      chunks &= x.n_keys == 0 || x.n_keys == sh.s_q;
    }
  }
};

}  // namespace

// Query rows of full pairs that are whole rounds of 256-row workgroups, where the rows after them are better taken by a launch of
// their own; 0: all in one launch.  All workgroups of a full pair are equally long, so a round that is not full costs as
// much as one that is; in 128-row workgroups, one per CU at most, the rest takes 0.6 of that.  us per call, one launch /
// two: 32 heads x 2777 x 3001 keys 156 / 146, x 3072 186 / 169, x 5120 429 / 401, x 10300 1712 / 1648, x 18500 5301 / 5051, 8 x 10000
// 461 / 423, 16 x 5000 x 4000 196 / 181, 64 x 1300 90 / 81, 96 x 700 x 2000 125 / 99.  Not with fewer keys, where the second launch
// and its prologue count: 32 x 2777 x 1200 keys and more gain 3 to 6 %, x 1024 60.7 / 61.0, x 512 37 / 41, 8 x 16896 x 700 78 / 81;
// nor where 128-row workgroups alone have no more rounds (160 x 400).
int64_t rows_of_whole_rounds(const dfa_shape& sh, int n) {
  const int64_t heads = static_cast<int64_t>(sh.h_q) * n, n256 = (static_cast<int64_t>(sh.s_q) + 255) / 256 * heads;
  const int64_t n128 = (static_cast<int64_t>(sh.s_q) + 127) / 128 * heads, rounds = n256 / 256;
  if (sh.causal || sh.s_k <= 1024 || !rounds || n128 <= rounds * 512) return 0;
  const int64_t rows = rounds * 256 / heads * 256, rest = sh.s_q - rows;
  return rows > 0 && rest > 0 && (rest + 127) / 128 * heads <= 256 ? rows : 0;
}

namespace {
int launch_pairs(const dfa_shape& sh, const dfa_fwd_pair* pairs, int n, bool sequence, hipStream_t st) {
  for (; n > MAX_PAIRS; pairs += MAX_PAIRS, n -= MAX_PAIRS) {
    const int rc = launch_pairs(sh, pairs, MAX_PAIRS, sequence, st);
    if (rc) return rc;
  }
  if (const int64_t rows = rows_of_whole_rounds(sh, n)) {
    dfa_shape part = sh;
    part.s_q = static_cast<int32_t>(rows);
    int rc = launch_pairs(part, pairs, n, sequence, st);
    if (rc) return rc;
    part.s_q = static_cast<int32_t>(sh.s_q - rows);
    dfa_fwd_pair rest[MAX_PAIRS];
    for (int i = 0; i < n; ++i) {
      rest[i] = pairs[i];
      rest[i].q = static_cast<const char*>(pairs[i].q) + rows * sh.q_stride_s * 2;
      rest[i].o = static_cast<char*>(pairs[i].o) + rows * pairs[i].o_stride_s * (sh.o_dtype == DFA_BF16 ? 2 : 4);
      rest[i].lse = pairs[i].lse + rows;
    }
    return launch_pairs(part, rest, n, sequence, st);
  }
  auto operand = [](const void* x) { return static_cast<const __bf16*>(x); };
  FwdBatch p{};
  const dfa_fwd_pair& x = pairs[0];
  p.q = operand(x.q); p.k = operand(x.k); p.v = operand(x.v); p.o = x.o; p.lse = x.lse; p.accumulate = x.accumulate;
  p.o_sh = x.o_stride_h; p.o_ss = x.o_stride_s; p.l_sh = x.lse_stride_h;
  p.s_q = sh.s_q; p.s_k = sh.s_k; p.h_q = sh.h_q; p.group = sh.h_q / sh.h_kv; p.causal = sh.causal;
  p.o_bf16 = sh.o_dtype == DFA_BF16; p.scale = sh.scale;
  p.q_sh = sh.q_stride_h; p.q_ss = sh.q_stride_s; p.kv_sh = sh.kv_stride_h; p.kv_ss = sh.kv_stride_s;
  if (n == 1) return launch_form<FwdParams>(p, sh, 1, sequence, st);
  for (int i = 0; i < n; ++i) {
    const dfa_fwd_pair& y = pairs[i];
    p.pair[i] = Pair{operand(y.q), operand(y.k), operand(y.v), y.o, y.lse, y.accumulate, y.o_stride_h, y.o_stride_s,
                     y.lse_stride_h};
  }
  return launch_form<FwdBatch>(p, sh, n, sequence, st);
}

int run_spans_bf16(const dfa_shape& sh, const dfa_fwd_span* spans, int n, bool all_remainders, void* ws, int64_t ws_bytes,
                   hipStream_t st) {
  const SpanPlan pl = span_plan(sh, spans, n, all_remainders, ws ? ws_bytes : 0);
  FwdSpans p{};
  p.s_q = sh.s_q; p.s_k = sh.s_k; p.h_q = sh.h_q; p.group = sh.h_q / sh.h_kv; p.causal = 1; p.scale = sh.scale;
  p.q_sh = sh.q_stride_h; p.q_ss = sh.q_stride_s; p.kv_sh = sh.kv_stride_h; p.kv_ss = sh.kv_stride_s;
  return run_spans<MAX_PAIRS>(sh, spans, n, pl.parts, ws, st, [&](const SpanPart* part, int count) {
    for (int i = 0; i < count; ++i) {
      const SpanPart& x = part[i];
      Span& y = p.span[i];
      y.q = static_cast<const __bf16*>(x.q); y.k = static_cast<const __bf16*>(x.k); y.v = static_cast<const __bf16*>(x.v);
      y.o = x.o; y.lse = x.lse; y.accumulate = x.accumulate; y.o_sh = x.o_sh; y.o_ss = x.o_ss; y.l_sh = x.l_sh;
      y.s_k = x.n_keys; y.off = x.off; y.o_bf16 = x.o_bf16;
    }
    return launch_spans(p, sh, count, pl.rows, st);
  });
}

int64_t span_bytes(const dfa_shape& sh, const dfa_fwd_span* spans, int n, bool all_remainders) {
  return parts_bytes(sh, spans, n, span_plan(sh, spans, n, all_remainders, MAX_SPAN_BYTES).parts);
}

dfa_shape own_pair(dfa_shape sh) {
  sh.s_k = sh.s_q; sh.causal = 1;
  return sh;
}
}  // namespace

int launch_fwd_bf16(const dfa_shape& sh, const dfa_fwd_pair* pairs, int n, hipStream_t st) {
  return launch_pairs(sh, pairs, n, false, st);
}

int launch_span_bf16(const dfa_shape& sh, const dfa_fwd_span* spans, int n, void* ws, int64_t ws_bytes, hipStream_t st) {
  const dfa_shape own = own_pair(sh);
  if (is_sequence(sh, spans, n)) return launch_pairs(own, WithoutOwn(sh, spans, 1).pair, 1, true, st);
  const Remainders rem = remainders(sh, spans, n);
  if (rem != Remainders::OWN) return run_spans_bf16(sh, spans, n, rem == Remainders::ALL, ws, ws_bytes, st);
  for (int i = 0; i < n; i += MAX_PAIRS) {
    const WithoutOwn x(sh, spans + i, std::min(MAX_PAIRS, n - i));
    int rc = x.pairs ? launch_pairs(own, x.pair, x.pairs, false, st) : DFA_OK;
    if (rc == DFA_OK && x.spans) {
      if (x.chunks) {      // (8 heads x 2048, four helpers' pairs 125 us as walks, 91 as a list with the diagonal)
        dfa_shape full = own;
        full.causal = 0;
        dfa_fwd_pair pairs[MAX_PAIRS];
        for (int j = 0; j < x.spans; ++j) {
          const dfa_fwd_span& y = x.rest[j];
          pairs[j] = {y.q, y.k, y.v, y.o, y.lse, y.o_stride_h, y.o_stride_s, y.lse_stride_h, y.accumulate, 0};
        }
        rc = launch_pairs(full, pairs, x.spans, false, st);
      } else {
        rc = run_spans_bf16(sh, x.rest, x.spans, false, ws, ws_bytes, st);
      }
    }
    if (rc) return rc;
  }
  return DFA_OK;
}

int64_t span_bf16_workspace(const dfa_shape& sh, const dfa_fwd_span* spans, int n) {
  if (is_sequence(sh, spans, n)) return 0;
  const Remainders rem = remainders(sh, spans, n);
  if (rem != Remainders::OWN) return span_bytes(sh, spans, n, rem == Remainders::ALL);
  int64_t most = 0;
  for (int i = 0; i < n; i += MAX_PAIRS) {
    const WithoutOwn x(sh, spans + i, std::min(MAX_PAIRS, n - i));
    if (x.spans && !x.chunks) most = std::max(most, span_bytes(sh, x.rest, x.spans, false));
  }
  return most;
}

dfa_form fwd_bf16_form(const dfa_shape& sh, int n) {
  n = static_cast<int>(last_launch(n));
  if (rows_of_whole_rounds(sh, n)) return {256, 1, 1, 0};
  const FwdForm f = form_of(sh, n, false);
  return {f.rows, f.parts, 1, 0};
}

dfa_form span_bf16_form(const dfa_shape& sh, const dfa_fwd_span* spans, int n, int64_t ws_bytes) {
  if (is_sequence(sh, spans, n)) {
    const FwdForm f = form_of(own_pair(sh), 1, true);
    return {f.rows, f.parts, 1, 0};
  }
  const Remainders rem = remainders(sh, spans, n);
  auto of = [&](const dfa_fwd_span* x, int count) {
    const SpanPlan pl = span_plan(sh, x, count, rem == Remainders::ALL, ws_bytes);
    return dfa_form{pl.rows, 256 / pl.rows, pl.parts, 0};
  };
  if (rem != Remainders::OWN) return of(spans, n);
  const WithoutOwn x(sh, spans, std::min(MAX_PAIRS, n));
  dfa_shape pair = own_pair(sh);
  if (!x.spans) return fwd_bf16_form(pair, x.pairs);
  pair.causal = 0;
  return x.chunks ? fwd_bf16_form(pair, x.spans) : of(x.rest, x.spans);
}

}  // namespace dfa

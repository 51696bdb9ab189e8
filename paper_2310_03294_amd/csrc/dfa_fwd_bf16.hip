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

// The same for 16x16 tiles of O^T, o[16 columns of d][16 rows] of the rows qrow + 16 nb (those that there are; load_o: that
// have a state).
template <int RB>
__device__ __forceinline__ void load_o(f32x4 (&o)[8][RB], const FwdParams& p, int head, int qrow, int g, const bool (&has)[RB]) {
#pragma unroll
  for (int nb = 0; nb < RB; ++nb) {
    if (!has[nb]) continue;
    const int64_t at = head * p.o_sh + static_cast<int64_t>(qrow + 16 * nb) * p.o_ss + 4 * g;
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      if (p.o_bf16) {
        const bf16x4 b = *reinterpret_cast<const bf16x4*>(static_cast<const __bf16*>(p.o) + at + 16 * db);
#pragma unroll
        for (int e = 0; e < 4; ++e) o[db][nb][e] = static_cast<float>(b[e]);
      } else {
        o[db][nb] = *reinterpret_cast<const f32x4*>(static_cast<const float*>(p.o) + at + 16 * db);
      }
    }
  }
}
template <int RB>
__device__ __forceinline__ void store_o(const f32x4 (&o)[8][RB], const FwdParams& p, int head, int qrow, int g, const float (&inv)[RB]) {
#pragma unroll
  for (int nb = 0; nb < RB; ++nb) {
    if (qrow + 16 * nb >= p.s_q) break;
    const int64_t at = head * p.o_sh + static_cast<int64_t>(qrow + 16 * nb) * p.o_ss + 4 * g;
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      const f32x4 x = o[db][nb] * inv[nb];
      if (p.o_bf16) {
        bf16x4 b;
#pragma unroll
        for (int e = 0; e < 4; ++e) b[e] = static_cast<__bf16>(x[e]);
        *reinterpret_cast<bf16x4*>(static_cast<__bf16*>(p.o) + at + 16 * db) = b;
      } else {
        *reinterpret_cast<f32x4*>(static_cast<float*>(p.o) + at + 16 * db) = x;
      }
    }
  }
}

// FULL: a full pair.  Its row sums are taken over the bf16-rounded weights that multiply V, those of the diagonal pair
// over the fp32 weights (the same in the other forms of 128 and 256 rows).
template <bool FULL, class Args>
__global__ void __launch_bounds__(NTHREADS, 2) k_fwd_bf16(Args a) {
  extern __shared__ __align__(128) char smem[];   // two (K tile, V tile) buffers

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
// Wavefront-specialised forward for full (unmasked) pairs: 8 wavefronts on 256 query rows, two per SIMD.
//   4 "S" wavefronts (64 query rows each, Q^T in registers): S^T = K Q^T and the exponentials, 32 keys of one between
//     32 keys of the other (each pipe waits for the other otherwise: one wavefront overlaps its own vector instructions with
//     its own MFMAs only where they stand between them and do not depend on one another); the exponentiated tile P^T goes
//     to the PV wavefront through LDS as bf16.  They also issue the global -> LDS copies of the K tiles;
//   4 "PV" wavefronts (the same 64 rows each): O^T = O^T * factor + V^T P^T and the row sums, one tile behind, so one
//     barrier per tile suffices; they copy the V tiles.
// 64 rows per wavefront: a row of K or V that is read from LDS serves four products.  With 32 rows (16 wavefronts, twice the
// LDS reads, no interleaving) a full pair of 32 heads x 65536 takes 58.2 ms, 56.2 so; all products of a tile before its
// exponentials 58.7; one kind of wavefront that does both (one per SIMD, 512 registers, no hand-over) 64.8; 32x32x16
// products, 16 wavefronts 59.2.  The matrix pipes are 66 % busy at 1.9 GHz.
// On the causal diagonal pair the 256-row granularity costs half a row block per row
// of tiles: slower than the kernel above up to about 6000 rows, faster at 16384.
// ============================================================================================
namespace full_pair {

constexpr int NT = 512;
constexpr int TILE_BYTES = kTile64;
constexpr int BMW = 256;                       // query rows per workgroup
constexpr int WROWS = 64;                      // of a wavefront
constexpr int RB = WROWS / 16;                 // its 16-row blocks
constexpr int PX_WAVE = BN * WROWS * 2;        // P^T hand-over of a wavefront
constexpr int PX_BYTES = BMW / WROWS * PX_WAVE;
constexpr int AL_BYTES = BMW * 4;              // rescale factor per query row
// LDS map.  Tile t: K slot t % 3, V slot t % 2, P^T / factor slot t % 2; row statistics at the end.
constexpr int OFF_K = 0;
constexpr int OFF_V = OFF_K + 3 * TILE_BYTES;
constexpr int OFF_PX = OFF_V + 2 * TILE_BYTES;
constexpr int OFF_AL = OFF_PX + 2 * PX_BYTES;
constexpr int OFF_ST = OFF_AL + 2 * AL_BYTES;  // (reference, row sum) as the S wavefronts have them, written once
constexpr int OFF_MV = OFF_ST + 2 * AL_BYTES;  // per tile slot and wavefront: a factor is not 1
constexpr int SMEM_BYTES = OFF_MV + 2 * 4 * 4;

// RAGGED: s_k is no multiple of the 64-row tile, so the last K/V tile has rows past the end.
// CAUSAL: the diagonal pair; its row sums are taken over the fp32 weights, as in the other causal forms (of a span: where a tile
// has keys of the chunk's own; before them over the rounded weights, as for full pairs).
template <bool RAGGED, bool CAUSAL, class Args>
__global__ void __launch_bounds__(NT, 2) k_fwd_bf16(Args a) {
  extern __shared__ __align__(128) char smem[];

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
  const bool pv_wave = wave >= 4;
  const int sw = wave & 3;                                     // row block of the wavefront
  const int r16 = lane & 15, g = lane >> 4;
  const float c2 = p.scale * LOG2E;
  const int q0w = q0 + sw * WROWS;
  const int qrow = q0w + r16;                                  // and qrow + 16, + 32, + 48

  const int off = off_of(p);
  const int k_end = CAUSAL ? min(p.s_k, q0 + BMW + off) : p.s_k;
  const int ntiles = (k_end + BN - 1) / BN;
  const uint32_t kv_rowbytes = static_cast<uint32_t>(p.kv_ss) * 2;
  const TileLane16 tl = tile16_lane(sw, lane, kv_rowbytes);
  const int last = p.s_k - 1;
  // tiles that have keys which the wavefront's rows see: the first ones
  const int seen = CAUSAL ? min(ntiles, (q0w + WROWS - 1 + off) / BN + 1) : ntiles;

  if (!pv_wave) {
    // ------------------------------------------------------------------ S wavefront
    const uint32_t a_base = row16_base(lane);
    bf16x8 qreg[4][RB];                      // Q^T operand of the lane's rows
    float m_run[RB];                         // running maxima of the raw scores q.k
    float l_run[RB];                         // this lane's quarter of the running sums of unrounded weights
#pragma unroll
    for (int nb = 0; nb < RB; ++nb) {
      const int row = qrow + 16 * nb;
      const bool ok = row < p.s_q;
      const __bf16* qp = p.q + head * p.q_sh + static_cast<int64_t>(ok ? row : 0) * p.q_ss;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        uint4 raw = *reinterpret_cast<const uint4*>(qp + step16_col(s, g));
        if (!ok) raw = make_uint4(0, 0, 0, 0);
        qreg[s][nb] = __builtin_bit_cast(bf16x8, raw);
      }
      m_run[nb] = -INFINITY;
      l_run[nb] = 0.f;
      if (p.accumulate && ok) {
        // state of the earlier key/value chunks: running (o, m, l) with m = lse (raw-score units), l = 1
        const float L = p.lse[head * p.l_sh + row];
        if (L > -INFINITY) { m_run[nb] = L / p.scale; l_run[nb] = g == 0 ? 1.f : 0.f; }
      }
    }
    float* al = reinterpret_cast<float*>(smem + OFF_AL) + sw * WROWS + r16;      // factors by which what was accumulated so far shrinks
    int* mv = reinterpret_cast<int*>(smem + OFF_MV) + sw;
    const char* kg = uniform_ptr(p.k + kh * p.kv_sh);
    auto k_plan = [&](int t, int slot) {     // (past the last tile the same once more, into a slot that is not read again)
      return tile16_copy_plan<RAGGED>(kg, kv_rowbytes, min(t, ntiles - 1) * BN, last, tl, smem + OFF_K + slot * TILE_BYTES, sw, lane);
    };
    tile16_copy(k_plan(0, 0));
    tile16_copy(k_plan(1, 1));
    lds_dma_wait();
    __syncthreads();                         // K tiles 0 and 1 are in LDS

    // A tile goes in two halves of 32 keys: the products of one are issued between the exponentials of the other, a
    // product and a score at a time, so that both pipes and the LDS are busy all along.  (All products of a tile first,
    // its exponentials after them: the matrix pipes are 52 % busy, at 2.2 GHz.)
    typedef f32x4 Half[2][RB];               // [16-key block][16-row block]
    constexpr int AHEAD = 3;                 // row reads run this many steps (of RB products) ahead, into the next half
    u32x4 x[AHEAD + 1];
    auto read_ahead = [&](const Rows16& rows, int half, int n) DFA_INLINE {
      x[n & AHEAD] = __builtin_bit_cast(u32x4, rows.read(2 * half + (n & 1), n >> 1));
    };
    // step n of S^T = K Q^T of a half: 16-key block n % 2, 32 elements of d from n / 2
    auto product = [&](Half& s, bf16x8 k, int n, int nb) DFA_INLINE {
      s[n & 1][nb] = mfma16(k, qreg[n >> 1][nb], n < 2 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[n & 1][nb]);
    };
    auto products = [&](Half& s, const char* Ks, int half) DFA_INLINE {
      const Rows16 rows(Ks, a_base);
#pragma unroll
      for (int n = 0; n < 8; ++n) {
        const bf16x8 k = rows.read(2 * half + (n & 1), n >> 1);
#pragma unroll
        for (int nb = 0; nb < RB; ++nb) product(s, k, n, nb);
      }
    };
    auto mask = [&](Half& s, int k0) DFA_INLINE {
      if ((k0 + 32 > p.s_k) || (CAUSAL && k0 + 31 > q0w + off)) {
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int kvi = k0 + mb * 16 + g * 4 + i;
#pragma unroll
            for (int nb = 0; nb < RB; ++nb)
              if (kvi >= p.s_k || (CAUSAL && kvi > qrow + 16 * nb + off)) s[mb][nb][i] = -INFINITY;
          }
      }
    };
    auto row_max = [&](const Half& s, int nb) DFA_INLINE {
      float mx = s[0][nb][0];
#pragma unroll
      for (int j = 1; j < 8; ++j) mx = fmaxf(mx, s[j >> 2][nb][j & 3]);
      mx = fmaxf(mx, __shfl_xor(mx, 16));
      return fmaxf(mx, __shfl_xor(mx, 32));
    };
    float mc[RB];                            // the references in the exponents' units
#pragma unroll
    for (int nb = 0; nb < RB; ++nb) mc[nb] = m_run[nb] == -INFINITY ? 0.f : m_run[nb] * c2;
    // Rows without a reference take the maximum of the tile's scores for one, so that its largest weight is exactly 1 (of the first
    // 32 keys' scores only, the largest weight and all others relative to it are rounded: 1 % more error in short rows).  The
    // second half's products are done here and, as always, between the exponentials of the first: half a tile per walk.
    int open = 1;                            // there are such rows
    auto first_reference = [&](const Half& s, Half& t, const char* Ks, int k0) DFA_INLINE {
      products(t, Ks, 1);
      mask(t, k0 + 32);
      bool none = false;
#pragma unroll
      for (int nb = 0; nb < RB; ++nb) {
        const float mx = fmaxf(row_max(s, nb), row_max(t, nb));
        if (m_run[nb] == -INFINITY) m_run[nb] = mx;
        mc[nb] = m_run[nb] == -INFINITY ? 0.f : m_run[nb] * c2;
        none |= m_run[nb] == -INFINITY;
      }
      open = __builtin_amdgcn_readfirstlane(__any(none));
    };
    // P^T = exp2(S^T c - reference) rounded to bf16, score j of the lane's 8 RB (a row's 8 keys one after the other) between
    // the products of the other half, handed to the PV wavefront through LDS (lane-private, any layout will do).  The row
    // sum that normalises O is the sum of exactly the weights that multiply V: the PV wavefront, which has vector
    // instructions to spare, adds up the ROUNDED weights; on a diagonal it is the sum of the fp32 values, here.
    // (v_dot2c_f32_bf16, which adds two of them at once, waits until the matrix pipe of the SIMD is empty: with 32 of them
    // per tile in here a full pair of 32 heads x 65536 takes 71 ms instead of 59.)
    // Step j takes the exponential of score j, the exponent of the next and the rounding of the two before: what depends on
    // an instruction comes a product later, or the wavefront would wait for it.
    float ready, top;                        // the exponent of the next score; the largest weight, unrounded: sum of eight
    u32x4 word;
    auto begin = [&](const Half& s) DFA_INLINE { ready = fmaf(s[0][0][0], c2, -mc[0]); };
    auto pair = [&](auto rounded, Half& s, int j, char* px) DFA_INLINE {      // weights j - 2 and j - 1
      const int nb = (j - 2) >> 3, e = (j - 2) & 7;
      const float w0 = s[e >> 2][nb][e & 3], w1 = s[e >> 2][nb][(e & 3) + 1];
      bf16x2 two;
      two[0] = static_cast<__bf16>(w0);
      two[1] = static_cast<__bf16>(w1);
      if (decltype(rounded)::value) top = fmaxf(fmaxf(top, w0), w1);
      word[e >> 1] = __builtin_bit_cast(uint32_t, two);
      if (e == 6) *reinterpret_cast<u32x4*>(px + nb * 1024) = word;
    };
    auto score = [&](auto rounded, Half& s, float (&sum)[RB], int j, char* px) DFA_INLINE {
      const int nb = j >> 3, e = j & 7;
      const float w = __builtin_amdgcn_exp2f(ready);
      if (j + 1 < 8 * RB) ready = fmaf(s[((j + 1) >> 2) & 1][(j + 1) >> 3][(j + 1) & 3], c2, -mc[(j + 1) >> 3]);
      if (j >= 2 && !(j & 1)) pair(rounded, s, j, px);
      if (!decltype(rounded)::value && j > 0) {      // the weight before
        const int b = (j - 1) >> 3, i = (j - 1) & 7;
        sum[b] = i ? sum[b] + s[i >> 2][b][i & 3] : s[0][b][0];
      }
      s[e >> 2][nb][e & 3] = w;
    };
    auto end = [&](auto rounded, Half& s, float (&sum)[RB], char* px) DFA_INLINE {
      pair(rounded, s, 8 * RB, px);
      if (!decltype(rounded)::value) {       // (32 comparisons fewer: diagonal of 32 heads x 16384 1912 -> 1879 us)
        sum[RB - 1] += s[1][RB - 1][3];
#pragma unroll
        for (int nb = 0; nb < RB; ++nb) top = fmaxf(top, sum[nb]);
      }
    };

    // Online softmax (exp2 domain) against a reference maximum that is only
    // moved when it has to be.  A half is first exponentiated against the reference as it stands,
    // without looking for its maximum: as long as no score lies more than 2^14 above the
    // reference, the exponentials are harmless in fp32 / bf16, O needs no rescaling, and the final
    // division by the row sum removes the reference.  The reference is derived from the scores
    // themselves (row maximum, exchanged between the lanes of a row) on a row's first tile -
    // so the largest weight seen is at least 1 and later keys cannot underflow the row sum - and
    // again when the largest weight of a tile shows a score far above it: the tile's
    // products are then done once more and taken against the moved reference.  (A weight that is no number moves
    // nothing: its row is none either way.)
    Half sa, sb;                             // the scores of keys 0 .. 31 and 32 .. 63 of a tile
    products(sa, smem + OFF_K, 0);
    {
      const Rows16 rows(smem + OFF_K, a_base);
#pragma unroll
      for (int n = 0; n < AHEAD; ++n) read_ahead(rows, 1, n);
    }
    int it = 0, k_slot = 0;
    auto tile = [&](auto rounded) {
      const int k0 = it * BN, next = k_slot == 2 ? 0 : k_slot + 1;
      const char* Ks = smem + OFF_K + k_slot * TILE_BYTES;
      const char* Kn = smem + OFF_K + next * TILE_BYTES;
      // This wavefront's pieces of the K tile after the next, issued one at a time between the products: in a burst they
      // would stall it while the memory pipe takes them in.
      const TileCopy16 cn = k_plan(it + 2, next == 2 ? 0 : next + 1);
      const Rows16 rows(Ks, a_base), rows_next(Kn, a_base);
      char* px = smem + OFF_PX + (it & 1) * PX_BYTES + sw * PX_WAVE + lane * 16;
      float sum0[RB], sum1[RB];
      top = 0.f;

      mask(sa, k0);
      if (open) first_reference(sa, sb, Ks, k0);
      begin(sa);
#pragma unroll
      for (int n = 0; n < 8; ++n) {
        // The slot's barrier: not at its end, where the last weights are still on their way into LDS, but behind
        // the first products of the next.  (No row reads are in flight here.)
        if (n == 1) {
          lds_dma_wait();
          __syncthreads();
          read_ahead(rows, 1, AHEAD);
        }
        if (n > 0) {
          if (n + AHEAD < 8) read_ahead(rows, 1, n + AHEAD);
          else read_ahead(rows_next, 0, n + AHEAD - 8);
        }
#pragma unroll
        for (int nb = 0; nb < RB; ++nb) {
          product(sb, __builtin_bit_cast(bf16x8, x[n & AHEAD]), n, nb);
          score(rounded, sa, sum0, RB * n + nb, px);
          DFA_SCHED_FENCE();
        }
        if (n == 1) tile16_copy_piece<0>(cn);
        if (n == 3) tile16_copy_piece<1>(cn);
        if (n == 5) tile16_copy_piece<2>(cn);
        if (n == 7) tile16_copy_piece<3>(cn);
      }
      end(rounded, sa, sum0, px);
      mask(sb, k0 + 32);
      begin(sb);
#pragma unroll
      for (int n = 0; n < 8; ++n) {
        if (n + AHEAD < 8) read_ahead(rows_next, 0, n + AHEAD);
        else read_ahead(rows_next, 1, n + AHEAD - 8);
#pragma unroll
        for (int nb = 0; nb < RB; ++nb) {
          product(sa, __builtin_bit_cast(bf16x8, x[n & AHEAD]), n, nb);
          score(rounded, sb, sum1, RB * n + nb, px + RB * 1024);
          DFA_SCHED_FENCE();
        }
      }
      end(rounded, sb, sum1, px + RB * 1024);
      const bool moved = __any(top > 16384.f);
      if (moved) {
        float mx[RB];
        products(sb, Ks, 0);
        mask(sb, k0);
#pragma unroll
        for (int nb = 0; nb < RB; ++nb) mx[nb] = row_max(sb, nb);
        products(sb, Ks, 1);
        mask(sb, k0 + 32);
#pragma unroll
        for (int nb = 0; nb < RB; ++nb) {
          const float m_new = fmaxf(fmaxf(m_run[nb], mx[nb]), row_max(sb, nb));
          const float mc_new = (m_new == -INFINITY) ? 0.f : m_new * c2;
          const float alpha = __builtin_amdgcn_exp2f(m_run[nb] * c2 - mc_new);
          m_run[nb] = m_new;
          mc[nb] = mc_new;
          l_run[nb] *= alpha;
          if (g == 0) al[(it & 1) * (AL_BYTES / 4) + nb * 16] = alpha;
        }
        begin(sb);
#pragma unroll
        for (int j = 0; j < 8 * RB; ++j) score(rounded, sb, sum1, j, px + RB * 1024);
        end(rounded, sb, sum1, px + RB * 1024);
        products(sb, Ks, 0);
        mask(sb, k0);
        begin(sb);
#pragma unroll
        for (int j = 0; j < 8 * RB; ++j) score(rounded, sb, sum0, j, px);
        end(rounded, sb, sum0, px);
      }
      if (!decltype(rounded)::value)
#pragma unroll
        for (int nb = 0; nb < RB; ++nb) l_run[nb] += sum0[nb] + sum1[nb];
      if (lane == 0) mv[(it & 1) * 4] = moved;
      k_slot = next;
    };
    __builtin_amdgcn_s_setprio(3);           // before the PV wavefront, which fills the gaps
    if constexpr (kSpans<Args>) {
      const int before = min(seen, off / BN);      // tiles before the chunk's own keys
      for (; it < before; ++it) tile(std::true_type{});
    }
    for (; it < seen; ++it) tile(std::bool_constant<!CAUSAL>{});
    for (; CAUSAL && it < ntiles; ++it) {    // tiles above this block's diagonal: only the copies
      const int next = k_slot == 2 ? 0 : k_slot + 1;
      lds_dma_wait();
      __syncthreads();
      tile16_copy(k_plan(it + 2, next == 2 ? 0 : next + 1));
      k_slot = next;
    }
    // references and row sums to the PV wavefront
#pragma unroll
    for (int nb = 0; nb < RB; ++nb) {
      float l_tot = l_run[nb] + __shfl_xor(l_run[nb], 16);
      l_tot += __shfl_xor(l_tot, 32);
      float* st = reinterpret_cast<float*>(smem + OFF_ST) + sw * WROWS + nb * 16 + r16;
      if (g == 0) { st[0] = m_run[nb]; st[BMW] = l_tot; }
    }
    lds_dma_wait();
    __syncthreads();                         // the PV wavefronts' last slot
  } else {
    // ------------------------------------------------------------------ PV wavefront: the rows of S wavefront sw
    const uint32_t g_base = gather16_base(lane);
    const char* vg = uniform_ptr(p.v + kh * p.kv_sh);

    f32x4 o[8][RB];      // O^T: [16 columns of d][16 rows]
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int nb = 0; nb < RB; ++nb) o[i][nb] = f32x4{0.f, 0.f, 0.f, 0.f};
    if (p.accumulate) {
      bool has[RB];
#pragma unroll
      for (int nb = 0; nb < RB; ++nb) has[nb] = qrow + 16 * nb < p.s_q && p.lse[head * p.l_sh + qrow + 16 * nb] > -INFINITY;
      load_o(o, p, head, qrow, g, has);
    }
    auto v_plan = [&](int it) {
      return tile16_copy_plan<RAGGED>(vg, kv_rowbytes, min(it, ntiles - 1) * BN, last, tl, smem + OFF_V + (it & 1) * TILE_BYTES, sw, lane);
    };
    __syncthreads();                         // K tiles 0 and 1 are in LDS
    tile16_copy(v_plan(0));
    lds_dma_wait();
    __syncthreads();
    // Slot it, from the barrier at which P of tile it - 1 is there: V tile `it` on its way (after the last the same once more,
    // into the slot that nobody reads), O^T = O^T * factor + V^T P^T for tile it - 1, and the row sums of its rounded weights.
    // Sums: v_mfma_f32_4x4x4_16b_bf16 against ones adds up a lane's four weights, in each of four registers (in 8 cycles of a
    // pipe that has 2048 to do; taking the weights apart for v_add_f32 takes 128 vector instructions a tile).  A tile's weights
    // make a sum of their own: the running sum is rounded once per tile, not four times.
    float l_run[RB];                         // this lane's quarter of the rows' sums
#pragma unroll
    for (int nb = 0; nb < RB; ++nb) l_run[nb] = 0.f;
    int it = 1;
    auto slot = [&](auto rounded) {
      lds_dma_wait();
      __syncthreads();
      __builtin_amdgcn_s_setprio(3);         // up to the products, or the S wavefront leaves it no room to get there
      const TileCopy16 cn = v_plan(it);
      const int t = it - 1;
      const char* Vs = smem + OFF_V + (t & 1) * TILE_BYTES;
      const char* px = smem + OFF_PX + (t & 1) * PX_BYTES + sw * PX_WAVE + lane * 16;
      const float* al = reinterpret_cast<const float*>(smem + OFF_AL) + (t & 1) * (AL_BYTES / 4) + sw * WROWS + r16;
      constexpr int AHEAD = 3;               // V^T gathers run this many steps ahead of their MFMAs
      const Gather16 cols(Vs, g_base);       // step n = 8 * (32-key block) + d block
      auto gather = [&](int n) { return cols.read(2 * (n >> 3), n & 7); };
      bf16x8 y[AHEAD + 1];
      u32x4 pa[2][RB];
      f32x4 sum[RB];                         // of the tile, in each register
      const int moved = *(reinterpret_cast<const int*>(smem + OFF_MV) + (t & 1) * 4 + sw);
#pragma unroll
      for (int n = 0; n < AHEAD; ++n) y[n] = gather(n);
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int nb = 0; nb < RB; ++nb) pa[u][nb] = *reinterpret_cast<const u32x4*>(px + (u * RB + nb) * 1024);
      if (__builtin_amdgcn_readfirstlane(moved)) {
#pragma unroll
        for (int nb = 0; nb < RB; ++nb) {
          const float a = al[nb * 16];
#pragma unroll
          for (int i = 0; i < 8; ++i) o[i][nb] *= a;
          l_run[nb] *= a;
        }
      }
      __builtin_amdgcn_s_setprio(0);
      DFA_SCHED_FENCE();
#pragma unroll
      for (int n = 0; n < 16; ++n) {
        if (n + AHEAD < 16) y[(n + AHEAD) % (AHEAD + 1)] = gather(n + AHEAD);
#pragma unroll
        for (int nb = 0; nb < RB; ++nb) {
          o[n & 7][nb] = mfma16(y[n % (AHEAD + 1)], __builtin_bit_cast(bf16x8, pa[n >> 3][nb]), o[n & 7][nb]);
          if (decltype(rounded)::value && !(n & 3)) {      // half of the row's weights of 32 keys
            const u32x4 w = pa[n >> 3][nb];
            sum[nb] = mfma_sum4(n & 4 ? u32x2{w[2], w[3]} : u32x2{w[0], w[1]}, n == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sum[nb]);
          }
          DFA_SCHED_FENCE();
        }
        if (n == 0) tile16_copy_piece<0>(cn);
        if (n == 2) tile16_copy_piece<1>(cn);
        if (n == 4) tile16_copy_piece<2>(cn);
        if (n == 6) tile16_copy_piece<3>(cn);
      }
      if (decltype(rounded)::value) {
#pragma unroll
        for (int nb = 0; nb < RB; ++nb) l_run[nb] += sum[nb][0];
      }
    };
    if constexpr (kSpans<Args>) {
      const int before = min(seen, off / BN);
      for (; it <= before; ++it) slot(std::true_type{});
    }
    for (; it <= seen; ++it) slot(std::bool_constant<!CAUSAL>{});
    for (; CAUSAL && it <= ntiles; ++it) {
      lds_dma_wait();
      __syncthreads();
      tile16_copy(v_plan(it));
    }
    lds_dma_wait();                          // nothing is left on its way into LDS
    // logsumexp and 1 / row sum
    float inv[RB];
#pragma unroll
    for (int nb = 0; nb < RB; ++nb) {
      float l_tot = l_run[nb];
      l_tot += __shfl_xor(l_tot, 16);
      l_tot += __shfl_xor(l_tot, 32);
      const float* st = reinterpret_cast<const float*>(smem + OFF_ST) + sw * WROWS + nb * 16 + r16;
      l_tot += st[BMW];
      inv[nb] = l_tot > 0.f ? 1.f / l_tot : 0.f;
      const int row = qrow + 16 * nb;
      if (g == 0 && row < p.s_q) p.lse[head * p.l_sh + row] = l_tot > 0.f ? st[0] * p.scale + logf(l_tot) : -INFINITY;
    }
    store_o(o, p, head, qrow, g, inv);
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
  extern __shared__ __align__(128) char smem[]; // two buffers of (SUB K sub-tiles, SUB V sub-tiles)

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
  // (256-row figures of an earlier form of that kernel, since 5 % faster; where the crossovers lie with it: below, at each line.)
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
    // not count, and whole tiles (ragged chunks, 32 heads x 14197: 1664 us against 1608 with 128 rows).  With the present 256-row
    // kernel, us, 128 rows / 256: 14 heads x 5376 164 / 185, 20 x 5120 190 / 208, 24 x 5120 196 / 210, 36 x 4864 264 / 271, 10 x 11264
    // 449 / 443; behind the line 20 x 6912 312 / 324, 24 x 7168 345 / 354, 22 x 6400 299 / 286, 10 x 14336 685 / 655, 40 x 6144 447 / 418,
    // 20 x 9216 533 / 505, 24 x 9216 569 / 520.  Before it the wider form is ahead where every XCD has whole pairs of heads:
    // 16 heads x 4608 130 / 119, x 6144 173 / 156, x 7680 253 / 214, 32 x 5376 263 / 244, 64 x 5120 483 / 453.
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
// 53 / 59 / 40, 16 over 4, 3 of 4158 493 / 551 / 402.)  The 256-row kernel is 5 % faster since; every division of 217 random
// spans timed with it: chosen / best 1.011 in the mean, 1.005 with constants fitted to them, so these stay.
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
// nor where 128-row workgroups alone have no more rounds (160 x 400).  With the present 256-row kernel 60 random full pairs of 8 to 64
// heads x 500 to 10000 rows took as long as the best of one launch, two, and 128 rows (within 1 %), but for rests of rounds with fewer
// than 750 keys (32 x 8794 x 508 114, 106 with 128 rows).
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

// bf16 backward chunk kernels for gfx950: dq, dk, dv contributions of one chunk pair from the
// saved logsumexp and D = rowsum(dO o O), without re-running the forward (Section 3.3).
//
// Two kinds of workgroups, no atomics, deterministic; a call that wants all gradients launches both kinds
// at once (k_bwd_bf16), a call that wants one side launches that kind alone:
//
//  k_bwd_dkdv_bf16 (key-stationary).  A workgroup of 8 wavefronts owns 128 key rows of one kv
//  head and walks over the query heads of the group and their query tiles of 64 rows, staged
//  (Q, dO, lse, D) through LDS rings.  The wavefronts are specialised in pairs per 32-key block,
//  one of each kind per SIMD, so that the exponentials of one overlap the MFMAs of the other:
//    "S" wavefront  (K^T in registers):  S = Q K^T, P = exp2(S c - lse log2e), hands P (bf16)
//                                        to its partner through LDS, dV^T += dO^T P
//    "dP" wavefront (V^T in registers):  dP - D = dO V^T - D (the MFMA chains start from -D),
//                                        dS = P o (dP - D), dK^T += Q^T dS
//  (queries x keys tiles on v_mfma_f32_16x16x32_bf16: each lane holds 16 queries of TWO keys; P
//  and dS are fed back from registers as B operands; dO^T, Q^T are gathered from LDS with the
//  transposing read; with 32x32x16 products a full pair of 32 heads x 16384 took 6 % longer).  The dP wavefronts run one tile behind, so one barrier per tile suffices.
//  Wavefronts raise their priority while they issue MFMAs, so that the other kind's VALU work
//  fills the gaps instead of delaying them.
//  dv / dk are written once per workgroup (summed over the group's query heads in registers).
//
//  k_bwd_dq_bf16 (query-stationary).  A workgroup owns 128 or 256 query rows of one head (Q^T, dO^T,
//  lse, D in registers) and walks over the key/value chunk in tiles of 64 rows in LDS: S^T = K Q^T,
//  dP^T = V dO^T (keys x queries: each lane holds 8 keys of TWO queries, so lse and D are per-lane
//  scalars), dS^T from registers as the B operand of dQ^T += K^T dS^T.
//
// The fused alternative (one kernel, dq by fp32 atomics) was measured first: the L2 atomic units
// retire about one fp32 atomic per clock and channel (~3.1e11 per second on the whole chip),
// which caps a 128-key workgroup tile at ~400 TFLOP/s no matter how the rest is scheduled.
// Recomputing S and dP in a second kernel costs 7 products instead of 5 but has no such cap.
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "dfa_internal.h"
#include "dfa_mfma.h"
#include "dfa_place.h"

namespace dfa {
namespace {

constexpr float LOG2E = 1.4426950408889634f;

// Workgroups of one kind: tiles per head, (head, tile) items of one pair, and those of all pairs.
struct Items { int ntile, per_pair; XcdMap map; };

// The operands of one (query chunk, key/value chunk) pair.
struct Pair {
  const __bf16 *q, *k, *v, *dO;
  const float *lse, *delta;
  float *dq, *dk, *dv;
  int acc_q, acc_kv;         // add to what dq / dk, dv hold
};
constexpr int MAX_PAIRS = 16;       // per launch: the pairs travel in the kernel arguments

struct BwdParams {
  int s_q, s_k, h_q, h_kv, group, causal, q_first;
  int off;                   // causal: key kv is visible to query row i if kv <= i + off (keys before the chunk's own)
  int parts;                 // dk, dv: workgroups that share the query tiles of a key tile
  f32x4* partial;            // parts > 1: their sums, PART_F4 per workgroup
  int q_parts;               // dq: workgroups that share the key tiles of a row block
  f32x4* q_partial;          // q_parts > 1: their sums
  Items kv_items, q_items;
  float scale;
  int64_t q_sh, q_ss, kv_sh, kv_ss, l_sh, dq_sh, dq_ss, dkv_sh, dkv_ss;
};

// One pair's operands are read together with everything else; picking them from a list first costs every
// workgroup another round trip to the argument memory (1 % of a call of 4096 workgroups).
template <int NP> struct BwdPairs : BwdParams { Pair pair[NP]; };
template <int NP>
__device__ __forceinline__ const Pair& pair_of(const BwdPairs<NP>& p, const Items& it, int item) {
  return p.pair[NP == 1 ? 0 : item / it.per_pair];
}
template <int NP>
__device__ __forceinline__ int item_in_pair(const Items& it, int item) { return NP == 1 ? item : item % it.per_pair; }

// ============================================================================================
// dK, dV
// ============================================================================================
namespace kv {

constexpr int NT = 512;     // 8 wavefronts: 4 "S" wavefronts (dV) and 4 "dP" wavefronts (dK)
constexpr int BN = 128;     // key rows per workgroup, 32 per wavefront pair
constexpr int BM = 64;      // query rows per LDS tile
constexpr int QTILE_BYTES = kTile64;
constexpr int LD_BYTES = 1024;                // lse'[64], -D[64], 128 spare floats
constexpr int PX_BYTES = 4 * 4096;            // P hand-over: 4 key blocks x (64 x 32 bf16)
// LDS map.  Tile t lives in Q slot t % 4, dO slot t % 2, lse/D slot t % 3, P slot t % 2.
constexpr int OFF_Q = 0;
constexpr int OFF_G = OFF_Q + 4 * QTILE_BYTES;
constexpr int OFF_LD = OFF_G + 2 * QTILE_BYTES;
constexpr int OFF_PX = OFF_LD + 3 * LD_BYTES;
constexpr int SMEM_BYTES = OFF_PX + 2 * PX_BYTES;
// dk and dv of a workgroup in its own order: (wavefront, four registers, lane), 128 KB
constexpr int PART_F4 = 8 * 16 * 64;

// The Q and dO tiles go from global memory straight into LDS (global_load_lds_dwordx4: every
// lane supplies its own global address, the wavefront's 64 x 16 bytes land contiguously at the
// LDS address in M0).  A tile is 16 such 1 KB pieces; of the four wavefronts that copy a
// tile, wavefront w moves the four of its rows 16w .. 16w + 15.  Only lse / D pass through a register.  The S wavefronts copy the Q tiles, the dP wavefronts the dO
// tiles, each piece issued from inline assembly between two MFMAs of a product (the memory pipe
// takes ~17 cycles per piece and CU: issued in a burst, the pieces stall the wavefront) and waited
// for just before the slot's barrier.  Measured with time stamps per phase: all staging at the top
// of the slot cost the S wavefronts, which are the critical path, 600-900 of ~3500 cycles per tile.
struct QTileRegs { float ld; bool ld_ok; };

// Where the next (Q, dO, lse, D) tile comes from: wave-uniform head bases, advanced tile by
// tile (no division in the loop), plus per-thread 32-bit byte offsets inside the head.
struct QTileCursor {
  const char *qh, *gh;       // Q and dO of the head
  const float* ldh;          // lse (even wavefronts) or D (odd wavefronts) of the head
  int q0;                    // first query row of the tile
};

// Cursor to the next tile: the next rows, or the next query head of the group.
__device__ __forceinline__ void qtile_advance(QTileCursor& cur, const BwdParams& p, int q_begin, int q_end) {
  cur.q0 += 64;
  if (cur.q0 >= q_end) {
    cur.q0 = q_begin;
    cur.qh += p.q_sh * 2; cur.gh += p.q_sh * 2; cur.ldh += p.l_sh;
  }
}
// The same as selects only (adv false: the cursor stays), for use inside the straight-line loops.
__device__ __forceinline__ void qtile_advance_if(QTileCursor& cur, bool adv, const BwdParams& p, int q_begin,
                                                 int q_end) {
  const int nq = cur.q0 + 64;
  const bool wrap = nq >= q_end;
  const int64_t hs = (adv && wrap) ? p.q_sh * 2 : 0;
  const int64_t ls = (adv && wrap) ? p.l_sh : 0;
  cur.q0 = adv ? (wrap ? q_begin : nq) : cur.q0;
  cur.qh += hs; cur.gh += hs; cur.ldh += ls;
}

// Rows past s_q are clamped to the last row instead of zero-filled: their lse' is +inf, so P and
// dS vanish for them whatever (finite) Q and dO the tile holds.  head: Q or dO of the cursor's head.
__device__ __forceinline__ void qtile_copy(const char* head, const QTileCursor& cur, const TileLane16& m, const BwdParams& p,
                                           char* tile, int w, int lane) {
  tile16_copy(tile16_copy_plan(head, static_cast<uint32_t>(p.q_ss) * 2, cur.q0, p.s_q - 1, m, tile, w, lane));
}

// lse (S wavefronts 0, 2, 3) or D (S wavefront 1) of the tile's 64 rows, one per lane, into a
// register.  Wavefronts 2 and 3 only go through the motions (their values land in a spare part
// of the slot), which keeps the staging free of branches.
__device__ __forceinline__ void qtile_load_ld(QTileRegs& t, const QTileCursor& cur, const BwdParams& p, int tid) {
  const int last = p.s_q - 1;
  const int r = cur.q0 + (tid & 63);
  t.ld_ok = r <= last;
  t.ld = cur.ldh[static_cast<uint32_t>(min(r, last))];
}

// LDs: the slot's 256 floats: lse'[64], -D[64], 128 spare.
__device__ __forceinline__ void qtile_store(const QTileRegs& t, float* LDs, int tid, bool is_d) {
  // lse pre-multiplied by log2 e; +inf makes P exactly 0 for an absent or empty row
  const float l = (t.ld_ok && t.ld > -INFINITY) ? t.ld * LOG2E : INFINITY;
  const float d = t.ld_ok ? -t.ld : 0.f;      // -D: the value the dP accumulators start from
  LDs[tid] = is_d ? d : l;
}

// A wavefront's stream of A operands: per slot 16 row reads (of a product over d) and 16 gathers (of a product over the
// tile's rows), each for two products, in the order in which they are used.  An LDS read that was asked for LEAD operands
// ago has arrived even with all wavefronts reading (about 330 cycles; the LDS itself is busy a third of the time): with
// 6 row reads and 4 gathers ahead every product waited for its operand.  With this and the same in dq a full pair of 32 heads
// x 16384 takes 11150 us instead of 11300, a diagonal of 32 over 8 heads x 1500 98.0 instead of 101.4; the matrix pipes
// are 64 (dk, dv) and 68 % (dq) busy at 1.95 GHz.
// (Kept as raw 32-bit vectors: carried around a loop as bf16 vectors they would be taken apart into 16-bit halves and put
// together again.)
constexpr int RING = 16, LEAD = 14;
typedef u32x4 Ring[RING];
struct NoHook { __device__ __forceinline__ void operator()(int) const {} };

// c[mb][nb] += X[16-row block mb] * B^T[16-key block nb] over d for the tile's 64 rows: X rows are read from LDS
// (A operand), B is the wavefront's K^T or V^T held in registers; the caller sets what the
// chains start from (zero, or -D for the dP products).  Step n = 4 s + mb.
__device__ __forceinline__ u32x4 row_operand(const Rows16& rows, int n) { return __builtin_bit_cast(u32x4, rows.read(n & 3, n >> 2)); }
// read(i): operand i of the stream, counted from the step's own slot; hook(n) runs after the MFMAs of step n (the callers issue
// their tile-copy pieces there)
template <int AT, class Read, class Hook = NoHook>
__device__ __forceinline__ void row_products(f32x4 (&c)[4][2], Ring& z, const bf16x8 (&bT)[4][2], Read read, Hook hook = Hook()) {
#pragma unroll
  for (int n = 0; n < 16; ++n) {
    z[(n + LEAD) % RING] = read(AT + n + LEAD);
    const bf16x8 a = __builtin_bit_cast(bf16x8, z[n]);
    c[n & 3][0] = mfma16(a, bT[n >> 2][0], c[n & 3][0]);
    c[n & 3][1] = mfma16(a, bT[n >> 2][1], c[n & 3][1]);
    hook(n);
    DFA_SCHED_FENCE();
  }
}

// acc[db][nb] += Y^T[16 columns db of d][64 queries] * W[64 queries][16 keys nb]: Y^T is gathered from the
// row-major LDS tile with the transposing read, W (P or dS) comes from registers in the order
// two MFMA result tiles have (w[u][nb] = query blocks 2u and 2u + 1).  Step n = 8 u + db.
__device__ __forceinline__ u32x4 col_operand(const Gather16& cols, int n) { return __builtin_bit_cast(u32x4, cols.read(2 * (n >> 3), n & 7)); }
template <int AT, class Read, class Hook = NoHook>
__device__ __forceinline__ void col_products(f32x4 (&acc)[8][2], Ring& z, const bf16x8 (&w)[2][2], Read read, Hook hook = Hook()) {
#pragma unroll
  for (int n = 0; n < 16; ++n) {
    z[(n + LEAD) % RING] = read(AT + n + LEAD);
    const bf16x8 a = __builtin_bit_cast(bf16x8, z[n]);
    acc[n & 7][0] = mfma16(a, w[n >> 3][0], acc[n & 7][0]);
    acc[n & 7][1] = mfma16(a, w[n >> 3][1], acc[n & 7][1]);
    hook(n);
    DFA_SCHED_FENCE();
  }
}

// RAGGED: s_q is no multiple of the 64-row tile, so a head's last tile has rows past the end.
// PARTS: several workgroups share the query tiles of a key tile.
template <bool RAGGED, bool PARTS>
__device__ __forceinline__ void dkdv(const BwdParams& p, const Pair& pr, int item, f32x4* partial, char* smem) {
  const int tk = item % p.kv_items.ntile;  // causal: low key tiles meet the most query tiles and come first
  const int part = PARTS ? item / p.kv_items.ntile % p.parts : 0;
  const int kh = PARTS ? item / p.kv_items.ntile / p.parts : item / p.kv_items.ntile;
  const int k0 = tk * BN;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: role branches stay scalar
  const int kb = wave & 3;            // 32-key block of this wavefront
  const bool dp_wave = wave >= 4;     // false: S, P, dV;  true: dP, dS, dK
  const int r16 = lane & 15, g = lane >> 4;
  const int kvrow = k0 + kb * 32 + r16;                       // and kvrow + 16
  // per-lane LDS bases; everything else in an LDS address is a compile-time constant
  const uint32_t a_base = row16_base(lane);                   // row reads (A operand of S, dP)
  const uint32_t g_base = gather16_base(lane);                // transposed gathers of Q, dO

  // B operands over d of this wavefront's 32 keys: K^T for an S wavefront, V^T for a dP wavefront
  bf16x8 bT[4][2];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) {
    const int row = kvrow + 16 * nb;
    const bool ok = row < p.s_k;
    const __bf16* src = (dp_wave ? pr.v : pr.k) + kh * p.kv_sh + static_cast<int64_t>(ok ? row : 0) * p.kv_ss;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      uint4 a = *reinterpret_cast<const uint4*>(src + step16_col(s, g));
      if (!ok) a = make_uint4(0, 0, 0, 0);
      bT[s][nb] = __builtin_bit_cast(bf16x8, a);
    }
  }

  // dV^T (S wavefront) or dK^T (dP wavefront): [d block][key block]
  f32x4 acc[8][2];
#pragma unroll
  for (int i = 0; i < 8; ++i) acc[i][0] = acc[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};

  const float c2 = p.scale * LOG2E;
  const int off = p.off;
  const int q_begin = p.causal ? max(0, k0 - off) & ~(BM - 1) : 0;
  const int ntq = (p.s_q - q_begin + BM - 1) / BM;  // query tiles per head for this key tile
  // this workgroup's share of the group's ntq * group query tiles
  const int walk = ntq * p.group;
  const int it0 = PARTS ? static_cast<int>(static_cast<int64_t>(walk) * part / p.parts) : 0;
  const int niter = PARTS ? static_cast<int>(static_cast<int64_t>(walk) * (part + 1) / p.parts) - it0 : walk;
  if (PARTS && niter == 0) {          // more parts than tiles (the last key tiles of a diagonal chunk)
#pragma unroll
    for (int i = 0; i < 16; ++i) partial[(wave * 16 + i) * 64 + lane] = f32x4{0.f, 0.f, 0.f, 0.f};
    return;
  }

  // Tile staging.  Two cursors: `cur` for the tile copies (during slot t Q tile t + 2 by the S wavefronts, which read a
  // tile's first operands before its slot begins, and dO tile t + 1 by the dP wavefronts), `curl` for lse / D (S wavefronts), which pass through a
  // register and run one tile further ahead.  Order inside a slot: store the held lse / D, load
  // the next ones, THEN issue the copies - the compiler knows nothing of the copies, so any wait
  // it places for its own loads must come before them or it would wait for them too.
  QTileRegs tr;
  QTileCursor cur, curl;
  {
    const int hq0 = kh * p.group + it0 / ntq;
    cur.qh = reinterpret_cast<const char*>(pr.q + hq0 * p.q_sh);
    cur.gh = reinterpret_cast<const char*>(pr.dO + hq0 * p.q_sh);
    cur.ldh = (kb == 1 ? pr.delta : pr.lse) + hq0 * p.l_sh;
    cur.q0 = q_begin + it0 % ntq * BM;
    curl = cur;
  }
  const int q_end = q_begin + ntq * BM;
  const uint32_t q_rowbytes = static_cast<uint32_t>(p.q_ss) * 2;
  const TileLane16 tl = tile16_lane(kb, lane, q_rowbytes);
  if (!dp_wave) {
    qtile_load_ld(tr, curl, p, tid);
    qtile_store(tr, reinterpret_cast<float*>(smem + OFF_LD), tid, kb == 1);
    if (niter > 1) {
      qtile_advance(curl, p, q_begin, q_end);
      qtile_load_ld(tr, curl, p, tid);           // lse / D of tile 1, stored in slot 0
    }
    qtile_copy(cur.qh, cur, tl, p, smem + OFF_Q, kb, lane);
    qtile_copy(cur.gh, cur, tl, p, smem + OFF_G, kb, lane);
    if (niter > 1) qtile_advance(cur, p, q_begin, q_end);
    qtile_copy(cur.qh, cur, tl, p, smem + OFF_Q + QTILE_BYTES, kb, lane);
    lds_dma_wait();                                // this wavefront's copies into LDS have landed
  }
  __syncthreads();

  // One barrier per tile.  Between two barriers ("slot" t) the S wavefronts take tile t all the
  // way (S, P, hand P over through LDS, dV) while the dP wavefronts finish tile t-1 (dS, dK) and
  // then start tile t (dP).  The two kinds share each SIMD, so the exponentials of one overlap
  // the MFMAs of the other.  Both kinds run niter + 1 slots (the S wavefronts idle in the last,
  // the dP wavefronts have no dS/dK in the first); each kind has its own straight-line loop.
  int slot = 0;            // t % 3
  auto q_tile = [&](int t) { return smem + OFF_Q + (t & 3) * QTILE_BYTES; };
  Ring z;
  if (!dp_wave) {
    int q0 = q_begin + it0 % ntq * BM;      // first query row of tile `it`
    {
      const Rows16 rows(q_tile(0), a_base);
#pragma unroll
      for (int n = 0; n < LEAD; ++n) z[n] = row_operand(rows, n);
    }
    for (int it = 0; it < niter; ++it) {
      const int next = slot == 2 ? 0 : slot + 1;
      const Rows16 rows(q_tile(it), a_base), rows_next(q_tile(it + 1), a_base);
      const Gather16 cols(smem + OFF_G + (it & 1) * QTILE_BYTES, g_base);
      const float* Ls = reinterpret_cast<const float*>(smem + OFF_LD + slot * LD_BYTES);
      // Staging, all of it inside the S products so that it costs no time of its own, and without
      // branches (past the last tile the cursors stay: the same tile, lse and D go once more into
      // ring slots nobody reads).  First (step 0) lse / D: tile it + 1 from the register into
      // LDS, tile it + 2 into the register - before the first copy of the slot, because the
      // compiler's wait for that register would otherwise wait for the copies too.  Then the Q
      // tile it + 2, one piece every fourth step.
      qtile_advance_if(cur, it + 2 < niter, p, q_begin, q_end);
      const TileCopy16 cq = tile16_copy_plan<RAGGED>(cur.qh, q_rowbytes, cur.q0, p.s_q - 1, tl, q_tile(it + 2), kb, lane);
      f32x4 c[4][2];
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) c[mb][0] = c[mb][1] = f32x4{0.f, 0.f, 0.f, 0.f};
      // lse' of the lane's rows, read under the last products; with the reads of P of the dP wavefronts all on their way at once,
      // one head x 4096 94.0 -> 92.6 us, 32 heads x 4096 787 -> 776.
      f32x4 l4[4];
      __builtin_amdgcn_s_setprio(3);
      row_products<0>(c, z, bT, [&](int i) DFA_INLINE { return i < 16 ? row_operand(rows, i) : col_operand(cols, i - 16); }, [&](int n) {          // S = Q K^T
        if (n == 1) {
          qtile_store(tr, reinterpret_cast<float*>(smem + OFF_LD + next * LD_BYTES), tid, kb == 1);
          qtile_advance_if(curl, it + 2 < niter, p, q_begin, q_end);
          qtile_load_ld(tr, curl, p, tid);
        }
        if (n == 3) tile16_copy_piece<0>(cq);
        if (n == 7) tile16_copy_piece<1>(cq);
        if (n == 11) tile16_copy_piece<2>(cq);
        if (n == 15) tile16_copy_piece<3>(cq);
        if (n >= 10 && n < 14) l4[n - 10] = *reinterpret_cast<const f32x4*>(Ls + (n - 10) * 16 + g * 4);
      });
      __builtin_amdgcn_s_setprio(0);
      // Only the causal diagonal needs a mask: query rows past s_q carry lse' = +inf (P = 0)
      // and key rows past s_k only feed dk/dv rows that are never written.
      if (p.causal && q0 + off < k0 + BN - 1) {
#pragma unroll
        for (int mb = 0; mb < 4; ++mb)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int qrow = q0 + off + mb * 16 + g * 4 + i;
            if (kvrow > qrow) c[mb][0][i] = -INFINITY;
            if (kvrow + 16 > qrow) c[mb][1][i] = -INFINITY;
          }
      }
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) {
        const f32x4 l = l4[mb];
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
          for (int i = 0; i < 4; ++i) c[mb][nb][i] = __builtin_amdgcn_exp2f(fmaf(c[mb][nb][i], c2, -l[i]));
      }
      bf16x8 w[2][2];
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) w[u][nb] = pack16(c[2 * u][nb], c[2 * u + 1][nb]);
      {  // hand P to the dP wavefront of the same key block: lane-private, any layout will do
        char* px = smem + OFF_PX + (it & 1) * PX_BYTES + kb * 4096 + lane * 16;
#pragma unroll
        for (int j = 0; j < 4; ++j) *reinterpret_cast<bf16x8*>(px + j * 1024) = w[j >> 1][j & 1];
      }
      __builtin_amdgcn_s_setprio(3);
      col_products<16>(acc, z, w, [&](int i) DFA_INLINE { return i < 32 ? col_operand(cols, i - 16) : row_operand(rows_next, i - 32); });    // dV^T += dO^T P
      __builtin_amdgcn_s_setprio(0);
      lds_dma_wait();                                // this wavefront's copies into LDS have landed
      // P and lse / D are in LDS: operands read after they were written have been used (a wavefront's LDS operations
      // are done in order); what is still on its way is the next tile's.
      DFA_BARRIER_NO_DRAIN();
      slot = next;
      q0 = q0 + BM >= q_end ? q_begin : q0 + BM;
    }
    __syncthreads();      // the dP wavefronts' last slot
  } else {
    f32x4 c[4][2];        // dP of the tile in flight, carried over the barrier
    bf16x8 w[2][2];
    // -D of a tile's 64 query rows in the accumulator layout: the dP chains start from it, so what
    // they end with is dP - D
    auto neg_d = [&](int ld_slot) {
      // One base register: OFF_LD is beyond the reach of the instruction's offset, and the compiler would add it to each of
      // the addresses (32 over 8 heads x 12000 6902 -> 6835 us, 64 over 8 x 3800 x 22659 8395 -> 8327).
      const uint32_t Ds = lds_pin(lds_addr(smem + OFF_LD + ld_slot * LD_BYTES) + 256 + g * 16);
#pragma unroll
      for (int mb = 0; mb < 4; ++mb) c[mb][0] = c[mb][1] = *(DFA_LDS const f32x4*)(Ds + mb * 64);
    };
    auto dS_prev = [&](int it) {                     // dS of tile it - 1 from P (LDS) and dP - D (registers)
      const char* px = smem + OFF_PX + ((it & 1) ^ 1) * PX_BYTES + kb * 4096 + lane * 16;
#pragma unroll
      for (int j = 0; j < 4; ++j) w[j >> 1][j & 1] = *reinterpret_cast<const bf16x8*>(px + j * 1024);
      DFA_SCHED_FENCE();       // (else two at a time are read and waited for)
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
#pragma unroll
          for (int e = 0; e < 8; ++e) c[2 * u + (e >> 2)][nb][e & 3] *= static_cast<float>(w[u][nb][e]);
          w[u][nb] = pack16(c[2 * u][nb], c[2 * u + 1][nb]);
        }
    };
    // The dP wavefronts copy the dO tiles: tile t + 1 during slot t, its pieces spread over the
    // products (past the last tile the cursor stays: the same tile goes into the unused slot).
    {  // slot 0: dP of tile 0 only
      qtile_advance_if(cur, niter > 1, p, q_begin, q_end);
      const TileCopy16 cg = tile16_copy_plan<RAGGED>(cur.gh, q_rowbytes, cur.q0, p.s_q - 1, tl,
                                                     smem + OFF_G + QTILE_BYTES, kb, lane);
      neg_d(0);
      const Rows16 rows(smem + OFF_G, a_base);
      const Gather16 cols(q_tile(0), g_base);
#pragma unroll
      for (int n = 0; n < LEAD; ++n) z[n] = row_operand(rows, n);
      row_products<16>(c, z, bT, [&](int i) DFA_INLINE { return i < 32 ? row_operand(rows, i - 16) : col_operand(cols, i - 32); }, [&](int n) {
        if (n == 1) tile16_copy_piece<0>(cg);
        if (n == 5) tile16_copy_piece<1>(cg);
        if (n == 9) tile16_copy_piece<2>(cg);
        if (n == 13) tile16_copy_piece<3>(cg);
      });
      lds_dma_wait();
      DFA_BARRIER_NO_DRAIN();
      slot = 1;
    }
    for (int it = 1; it < niter; ++it) {
      const int next = slot == 2 ? 0 : slot + 1;
      const Rows16 rows(smem + OFF_G + (it & 1) * QTILE_BYTES, a_base);
      const Gather16 cols(q_tile(it - 1), g_base), cols_next(q_tile(it), g_base);
      qtile_advance_if(cur, it + 1 < niter, p, q_begin, q_end);
      const TileCopy16 cg = tile16_copy_plan<RAGGED>(cur.gh, q_rowbytes, cur.q0, p.s_q - 1, tl,
                                                     smem + OFF_G + ((it + 1) & 1) * QTILE_BYTES, kb, lane);
      __builtin_amdgcn_s_setprio(3);
      dS_prev(it);
      neg_d(slot);                               // read straight into the accumulators, under the dK products
      col_products<0>(acc, z, w, [&](int i) DFA_INLINE { return i < 16 ? col_operand(cols, i) : row_operand(rows, i - 16); }, [&](int n) {  // dK^T += Q^T dS
        if (n == 1) tile16_copy_piece<0>(cg);
        if (n == 5) tile16_copy_piece<1>(cg);
        if (n == 9) tile16_copy_piece<2>(cg);
        if (n == 13) tile16_copy_piece<3>(cg);
      });
      row_products<16>(c, z, bT, [&](int i) DFA_INLINE { return i < 32 ? row_operand(rows, i - 16) : col_operand(cols_next, i - 32); });   // dP - D = dO V^T - D
      __builtin_amdgcn_s_setprio(0);
      lds_dma_wait();                            // this wavefront's copies into LDS have landed
      DFA_BARRIER_NO_DRAIN();                    // nothing else it wrote has to be seen by the others
      slot = next;
    }
    dS_prev(niter);
    const Gather16 cols(q_tile(niter - 1), g_base);
    col_products<0>(acc, z, w, [&](int i) DFA_INLINE { return col_operand(cols, i & 15); });
    __syncthreads();
  }

  if constexpr (PARTS) {     // k_reduce_dkdv adds the parts up
#pragma unroll
    for (int i = 0; i < 16; ++i) partial[(wave * 16 + i) * 64 + lane] = acc[i >> 1][i & 1];
  } else {
    const float f = dp_wave ? p.scale : 1.f;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb) {
      const int row = kvrow + 16 * nb;
      if (row >= p.s_k) break;
      float* dst = (dp_wave ? pr.dk : pr.dv) + kh * p.dkv_sh + static_cast<int64_t>(row) * p.dkv_ss + g * 4;
#pragma unroll
      for (int db = 0; db < 8; ++db) {
        f32x4 a = acc[db][nb] * f;
        if (pr.acc_kv) a += *reinterpret_cast<const f32x4*>(dst + db * 16);
        *reinterpret_cast<f32x4*>(dst + db * 16) = a;
      }
    }
  }
}

}  // namespace kv

// ============================================================================================
// dQ
// ============================================================================================
namespace qs {

constexpr int BN = 64;      // key rows per LDS tile
constexpr int TILE_BYTES = kTile64;

// NW wavefronts, NW / NS row blocks of 32 query rows each times NS parts of every key tile; two wavefronts
// per SIMD either way: NW = 4 (128 rows, two workgroups per CU, scheduled independently of each other) or
// NW = 8, NS = 1 (256 rows, one workgroup per CU: every K/V tile copy and every barrier serve twice the
// rows; measured 2-3 % faster on long chunks, where the copies are what the second independent workgroup
// used to hide, and no faster on short ones and on the causal diagonal pair, which keep the 128-row form).
// NW = 8, NS = 2 (128 rows, one workgroup per CU, half the serial walk each) is for calls that do not fill
// the device; the sums of the two parts are added through LDS at the end.
// PARTS: q_parts workgroups share the key tiles of a row block; k_reduce_dq adds their sums up.
template <int NW, int NS, bool PARTS>
__device__ __forceinline__ void dq(const BwdParams& p, const Pair& pr, int item, f32x4* partial, char* smem) {   // smem: (K tile, V tile) buffers, three with 8 wavefronts, two with 4
  constexpr int BM = NW / NS * 32;     // query rows per workgroup
  const int share = PARTS ? item / p.q_items.ntile % p.q_parts : 0;
  const int head = PARTS ? item / p.q_items.ntile / p.q_parts : item / p.q_items.ntile;
  int tq = item % p.q_items.ntile;
  if (p.causal) tq = p.q_items.ntile - 1 - tq;      // longest rows first
  const int kh = head / p.group;
  const int q0 = tq * BM;

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: keeps tile branches scalar
  const int r16 = lane & 15, g = lane >> 4;
  const int rb = wave % (NW / NS), part = wave / (NW / NS);    // row block, part of every key tile
  const int q0w = q0 + rb * 32;
  const int qrow = q0w + r16;                                  // and qrow + 16
  // (with two parts the part's rows come in here, once: as a block index they would be added to every address of every tile)
  const uint32_t of_part = NS == 2 ? part * 2 * kBlock16 : 0;
  const uint32_t a_base = row16_base(lane) + of_part, g_base = gather16_base(lane) + of_part;

  const char* kg = reinterpret_cast<const char*>(pr.k + kh * p.kv_sh);
  const char* vg = reinterpret_cast<const char*>(pr.v + kh * p.kv_sh);
  const uint32_t kv_rowbytes = static_cast<uint32_t>(p.kv_ss) * 2;
  // Tile copies: with 4 wavefronts each moves its quarter of the K tile and of the V tile; with 8,
  // wavefronts 0-3 move the K tile and 4-7 the V tile.
  const int cw = wave & 3;

  // Q^T and dO^T operands of the lane's two rows; lse' and -D of them (-D in every element: the accumulator the dP^T
  // products start from, which saves the subtraction per score)
  bf16x8 qB[4][2], gB[4][2];
  float Lr[2];
  f32x4 negD[2];
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) {
    const int row = qrow + 16 * nb;
    const bool ok = row < p.s_q;
    const int64_t off = head * p.q_sh + static_cast<int64_t>(ok ? row : 0) * p.q_ss;
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      uint4 a = *reinterpret_cast<const uint4*>(pr.q + off + step16_col(s, g));
      uint4 b = *reinterpret_cast<const uint4*>(pr.dO + off + step16_col(s, g));
      if (!ok) { a = make_uint4(0, 0, 0, 0); b = make_uint4(0, 0, 0, 0); }
      qB[s][nb] = __builtin_bit_cast(bf16x8, a);
      gB[s][nb] = __builtin_bit_cast(bf16x8, b);
    }
    Lr[nb] = INFINITY;                    // +inf makes P exactly 0 for rows past the end
    float d = 0.f;
    if (ok) {
      const float L = pr.lse[head * p.l_sh + row];
      Lr[nb] = L > -INFINITY ? L * LOG2E : INFINITY;
      d = pr.delta[head * p.l_sh + row];
    }
    negD[nb] = f32x4{-d, -d, -d, -d};
  }
  f32x4 dqT[8][2];
#pragma unroll
  for (int i = 0; i < 8; ++i) dqT[i][0] = dqT[i][1] = f32x4{0.f, 0.f, 0.f, 0.f};
  const float c2 = p.scale * LOG2E;

  const int off = p.off;
  const int k_end = p.causal ? min(p.s_k, q0 + BM + off) : p.s_k;
  const int all = (k_end + BN - 1) / BN;
  const int it0 = PARTS ? all * share / p.q_parts : 0, ntiles = PARTS ? all * (share + 1) / p.q_parts : all;

  // K/V tiles go from global memory straight into LDS; key rows past s_k are clamped to the last
  // row and masked below.  With one workgroup per CU three tiles are there: the one that is computed on, the next, whose
  // first operands are read ahead, and the one after it on its way; one barrier per tile, in the middle of its work.  With two
  // workgroups per CU there is room for two, and the barrier stands at the end of a tile.
  constexpr bool WIDE = NW == 8;
  constexpr int SLOTS = WIDE ? 3 : 2;
  const int end = max(ntiles - 1, it0);            // (a share may have no tile)
  const uint32_t lane_row = sat32(static_cast<uint64_t>(16 * cw + (lane >> 4)) * kv_rowbytes);
  auto at = [&](int slot, bool v) DFA_INLINE { return smem + (2 * slot + v) * TILE_BYTES; };
  auto plan = [&](int it, int slot, bool v) DFA_INLINE {
    return TileRows16(v ? vg : kg, kv_rowbytes, min(it, end) * BN, p.s_k - 1, at(slot, v), cw, lane, lane_row);
  };
  const bool v_wave = WIDE && wave >= 4;           // with 8 wavefronts: this wavefront's tile
#pragma unroll
  for (int i = 0; i < SLOTS - 1; ++i) {
    plan(it0 + i, i, v_wave).all();
    if (!WIDE) plan(it0 + i, i, true).all();
  }
  lds_dma_wait();
  __syncthreads();

  // Tiles that have keys which the wavefront's rows see, counted once: compared with the offset in every tile, the form with two
  // parts spilled 6 registers (8 heads x 1000 x 1900 47.2 us, 39.7 so).
  const int seen = p.causal ? min(ntiles, (q0w + 31 + off - (NS == 2 ? part * 32 : 0) + BN) / BN) : ntiles;
  // The stream of A operands, 24 per 32 keys: K and V rows in turn (S^T = K Q^T, dP^T = V dO^T: step t = 2 s + mb takes
  // two) and 8 gathers of K (dQ^T += K^T dS^T), each read LEAD operands before it is used.
  constexpr int RING = WIDE ? 12 : 8, LEAD = RING - 2;
  u32x4 z[RING];
  // (rows of the slot's K tile, its V tile behind it)
  auto operand = [&](const Rows16& rows, const Gather16& kc, int nk, int e) DFA_INLINE {
    const bf16x8 x = e >= 16 ? kc.read(2 * nk, e - 16) : rows.read(2 * nk + ((e >> 1) & 1), e >> 2, e & 1);
    return __builtin_bit_cast(u32x4, x);
  };
  int slot = 0, it = it0;
  auto read_first = [&](int slot) DFA_INLINE {
    const Rows16 rows(at(slot, false), a_base);
    const Gather16 kc(at(slot, false), g_base);
#pragma unroll
    for (int e = 0; e < LEAD; ++e) z[e] = operand(rows, kc, 0, e);
  };
  if (WIDE) read_first(0);
  for (; it < seen; ++it) {
    const int k0 = it * BN;
    const int next = slot + 1 == SLOTS ? 0 : slot + 1, free = next + 1 == SLOTS ? 0 : next + 1;
    const Rows16 rows(at(slot, false), a_base), rows_next(at(next, false), a_base);
    const Gather16 kc(at(slot, false), g_base);
    // The pieces of a tile on its way are spread between the MFMAs (issued in a burst they stall the wavefront while the
    // memory pipe takes them in).  After the last tile the same tile goes once more into a slot that is not read
    // again, which keeps the loop free of branches around the copies.
    const TileRows16 ck = WIDE ? plan(it + 2, free, v_wave) : plan(it + 1, next, false);
    const TileRows16 cv = plan(it + 1, next, true);      // (two workgroups per CU)
    if (!WIDE) read_first(slot);
    const bool need_mask = (k0 + BN > p.s_k) || (p.causal && k0 + BN - 1 > q0w + off);
#pragma unroll
    for (int n = 0; n < 2 / NS; ++n) {
      const int key0 = k0 + (NS == 2 ? part : n) * 32;      // of this 32-key block
      const bool last_half = n == 2 / NS - 1;
      auto read_ahead = [&](int e) DFA_INLINE {
        if (e < 24) z[e % RING] = operand(rows, kc, n, e);
        else if (!last_half) z[e % RING] = operand(rows, kc, n + 1, e - 24);
        else if (WIDE) z[e % RING] = operand(rows_next, kc, 0, e - 24);
      };
      f32x4 s[2][2], dp[2][2];                   // [key block][row block]
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        if (WIDE && last_half && t == 6) {       // the next tile is there, nobody reads the one before any more
          lds_dma_wait();
          DFA_BARRIER_NO_DRAIN();
        }
        const int mb = t & 1;
        read_ahead(2 * t + LEAD);
        read_ahead(2 * t + 1 + LEAD);
        const bf16x8 ka = __builtin_bit_cast(bf16x8, z[2 * t % RING]), va = __builtin_bit_cast(bf16x8, z[(2 * t + 1) % RING]);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) s[mb][nb] = mfma16(ka, qB[t >> 1][nb], t < 2 ? f32x4{0.f, 0.f, 0.f, 0.f} : s[mb][nb]);
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) dp[mb][nb] = mfma16(va, gB[t >> 1][nb], t < 2 ? negD[nb] : dp[mb][nb]);      // from -D
        if (!WIDE) {                             // one piece of the next tiles every other step
          const TileRows16& c = n == 0 ? ck : cv;
          if (t == 0) c.piece<0>();
          if (t == 2) c.piece<1>();
          if (t == 4) c.piece<2>();
          if (t == 6) c.piece<3>();
        }
        DFA_SCHED_FENCE();
      }
      // dS^T = P^T o (dP^T - D): lse' is a per-lane scalar here, -D came in through the accumulator
#pragma unroll
      for (int mb = 0; mb < 2; ++mb)
#pragma unroll
        for (int nb = 0; nb < 2; ++nb)
#pragma unroll
          for (int i = 0; i < 4; ++i) dp[mb][nb][i] *= __builtin_amdgcn_exp2f(fmaf(s[mb][nb][i], c2, -Lr[nb]));
      if (need_mask) {
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int kvi = key0 + mb * 16 + g * 4 + i;
#pragma unroll
            for (int nb = 0; nb < 2; ++nb)
              if (kvi >= p.s_k || (p.causal && kvi > qrow + 16 * nb + off)) dp[mb][nb][i] = 0.f;
          }
      }
      // dQ^T += K^T dS^T over the 32 keys, 8 blocks of 16 columns
      const bf16x8 sb[2] = {pack16(dp[0][0], dp[1][0]), pack16(dp[0][1], dp[1][1])};
      DFA_SCHED_FENCE();
#pragma unroll
      for (int db = 0; db < 8; ++db) {
        read_ahead(16 + db + LEAD);
        const bf16x8 gk = __builtin_bit_cast(bf16x8, z[(16 + db) % RING]);
        dqT[db][0] = mfma16(gk, sb[0], dqT[db][0]);
        dqT[db][1] = mfma16(gk, sb[1], dqT[db][1]);
        if (WIDE && last_half) {
          if (db == 0) ck.piece<0>();
          if (db == 2) ck.piece<1>();
          if (db == 4) ck.piece<2>();
          if (db == 6) ck.piece<3>();
        }
        DFA_SCHED_FENCE();
      }
    }
    slot = next;
    if (!WIDE) {
      lds_dma_wait();
      __syncthreads();
    }
  }
  for (; it < ntiles; ++it) {                      // nothing to compute for this wavefront's rows: only its share of the copies
    const int next = slot + 1 == SLOTS ? 0 : slot + 1, free = next + 1 == SLOTS ? 0 : next + 1;
    if (WIDE) {
      lds_dma_wait();
      DFA_BARRIER_NO_DRAIN();
      plan(it + 2, free, v_wave).all();
    } else {
      plan(it + 1, next, false).all();
      plan(it + 1, next, true).all();
      lds_dma_wait();
      __syncthreads();
    }
    slot = next;
  }
  if (WIDE) lds_dma_wait();                        // nothing is left on its way into LDS
  if (NS == 2) __syncthreads();

  if constexpr (NS == 2) {      // the second part's sums through LDS (the tiles are no longer needed)
    f32x4* x = reinterpret_cast<f32x4*>(smem) + rb * 1024 + lane;
    if (part == 1) {
#pragma unroll
      for (int i = 0; i < 16; ++i) x[i * 64] = dqT[i >> 1][i & 1];
    }
    __syncthreads();
    if (part == 1) return;
#pragma unroll
    for (int i = 0; i < 16; ++i) dqT[i >> 1][i & 1] += x[i * 64];
  }
  if constexpr (PARTS) {
#pragma unroll
    for (int i = 0; i < 16; ++i) partial[(rb * 16 + i) * 64 + lane] = dqT[i >> 1][i & 1];
    return;
  }
#pragma unroll
  for (int nb = 0; nb < 2; ++nb) {
    const int row = qrow + 16 * nb;
    if (row >= p.s_q) break;
    float* dst = pr.dq + head * p.dq_sh + static_cast<int64_t>(row) * p.dq_ss + g * 4;
#pragma unroll
    for (int db = 0; db < 8; ++db) {
      f32x4 a = dqT[db][nb] * p.scale;
      if (pr.acc_q) a += *reinterpret_cast<const f32x4*>(dst + db * 16);
      *reinterpret_cast<f32x4*>(dst + db * 16) = a;
    }
  }
}

}  // namespace qs

// dk, dv of a key tile from the sums of its parts: grid (4 column blocks, key tiles), 512 threads in the
// order of the workgroups that wrote them.  The order of the sum is that of the parts.
__global__ void __launch_bounds__(kv::NT) k_reduce_dkdv(BwdPairs<MAX_PAIRS> p) {
  const int tile = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tk = tile % p.kv_items.ntile, pk = tile / p.kv_items.ntile;      // pk: pair * h_kv + kv head
  const Pair& pr = p.pair[pk / p.h_kv];
  const bool is_dk = wave >= 4;
  const int row = tk * kv::BN + (wave & 3) * 32 + (lane & 15);       // and row + 16
  if (row >= p.s_k) return;
  const int64_t step = static_cast<int64_t>(p.kv_items.ntile) * kv::PART_F4;
  const f32x4* src = p.partial + (static_cast<int64_t>(pk) * p.parts * p.kv_items.ntile + tk) * kv::PART_F4 +
                     (wave * 16 + blockIdx.x * 4) * 64 + lane;
  f32x4 a[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = src[i * 64];
  for (int s = 1; s < p.parts; ++s) {
    src += step;
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] += src[i * 64];
  }
  float* dst = (is_dk ? pr.dk : pr.dv) + (pk % p.h_kv) * p.dkv_sh + static_cast<int64_t>(row) * p.dkv_ss +
               blockIdx.x * 32 + (lane >> 4) * 4;
  const float f = is_dk ? p.scale : 1.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {      // column block 2 blockIdx.x + i / 2, row block i % 2
    if (row + 16 * (i & 1) >= p.s_k) continue;
    f32x4* d = reinterpret_cast<f32x4*>(dst + (i & 1) * 16 * p.dkv_ss + (i >> 1) * 16);
    f32x4 x = a[i] * f;
    if (pr.acc_kv) x += *d;
    *d = x;
  }
}

// dq of a row block of 128 rows from the sums of its parts: grid (4 column blocks, row blocks of all heads), 256 threads.
constexpr int QPART_F4 = 4 * 16 * 64;
__global__ void __launch_bounds__(256) k_reduce_dq(BwdPairs<1> p) {
  const int ntile = p.q_items.ntile, tid = threadIdx.x, lane = tid & 63, rb = tid >> 6;
  const int head = blockIdx.y / ntile, slot = blockIdx.y % ntile, tq = p.causal ? ntile - 1 - slot : slot;
  const int row = tq * 128 + rb * 32 + (lane & 15);      // and row + 16
  if (row >= p.s_q) return;
  const f32x4* src = p.q_partial + (static_cast<int64_t>(head) * p.q_parts * ntile + slot) * QPART_F4 + (rb * 16 + blockIdx.x * 4) * 64 + lane;
  f32x4 a[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) a[i] = src[i * 64];
#pragma unroll 4      // (the reads of four parts on their way)
  for (int s = 1; s < p.q_parts; ++s) {
    src += static_cast<int64_t>(ntile) * QPART_F4;
#pragma unroll
    for (int i = 0; i < 4; ++i) a[i] += src[i * 64];
  }
  float* dst = p.pair[0].dq + head * p.dq_sh + static_cast<int64_t>(row) * p.dq_ss + blockIdx.x * 32 + (lane >> 4) * 4;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    if (row + 16 * (i & 1) >= p.s_q) continue;
    f32x4* d = reinterpret_cast<f32x4*>(dst + (i & 1) * 16 * p.dq_ss + (i >> 1) * 16);
    f32x4 x = a[i] * p.scale;
    if (p.pair[0].acc_q) x += *d;
    *d = x;
  }
}

// The kernels: dk, dv alone, dq alone, and both kinds of workgroups in one launch; of NP pairs at most.
template <bool RAGGED, bool PARTS, int NP>
__device__ __forceinline__ void run_dkdv(const BwdPairs<NP>& p, int bid, char* smem) {
  const int item = xcd_item(p.kv_items.map, bid);
  if (item < p.kv_items.map.total)
    kv::dkdv<RAGGED, PARTS>(p, pair_of(p, p.kv_items, item), item_in_pair<NP>(p.kv_items, item),
                            p.partial + static_cast<int64_t>(item) * kv::PART_F4, smem);
}
template <int NW, int NS, bool PARTS, int NP>
__device__ __forceinline__ void run_dq(const BwdPairs<NP>& p, int bid, char* smem) {
  const int item = xcd_item(p.q_items.map, bid);
  if (item < p.q_items.map.total)
    qs::dq<NW, NS, PARTS>(p, pair_of(p, p.q_items, item), item_in_pair<NP>(p.q_items, item),
                          p.q_partial + static_cast<int64_t>(item) * QPART_F4, smem);
}

template <bool RAGGED, bool PARTS, int NP>
__global__ void __launch_bounds__(kv::NT, 2) k_bwd_dkdv_bf16(BwdPairs<NP> p) {
  extern __shared__ __align__(128) char smem[];
  run_dkdv<RAGGED, PARTS, NP>(p, blockIdx.x, smem);
}

template <int NW, int NP>
__global__ void __launch_bounds__(NW * 64, NW == 4 ? 2 : 1) k_bwd_dq_bf16(BwdPairs<NP> p) {
  extern __shared__ __align__(128) char smem[];
  run_dq<NW, 1, false, NP>(p, blockIdx.x, smem);
}

template <bool RAGGED, int NS, bool PARTS, int NP, bool Q_PARTS = false>
__global__ void __launch_bounds__(kv::NT, 2) k_bwd_bf16(BwdPairs<NP> p) {
  extern __shared__ __align__(128) char smem[];
  const int n_kv = p.kv_items.map.per_xcd * 8, n_q = p.q_items.map.per_xcd * 8;
  const int bid = blockIdx.x;
  if (p.q_first ? bid >= n_q : bid < n_kv) run_dkdv<RAGGED, PARTS, NP>(p, p.q_first ? bid - n_q : bid, smem);
  else run_dq<8, NS, Q_PARTS, NP>(p, p.q_first ? bid : bid - n_kv, smem);
}

// > 64 KB of dynamic LDS needs the opt-in, once per kernel and process (thread-safe)
template <int NP, void (*KERNEL)(BwdPairs<NP>)>
int launch(const BwdPairs<MAX_PAIRS>& all, int64_t blocks, int threads, int smem, hipStream_t st) {
  static std::once_flag once;
  static int attr_rc = DFA_OK;
  std::call_once(once, [smem] {
    attr_rc = hip_status(hipFuncSetAttribute(reinterpret_cast<const void*>(KERNEL),
                                             hipFuncAttributeMaxDynamicSharedMemorySize, smem));
  });
  if (attr_rc) return attr_rc;
  BwdPairs<NP> p;
  static_cast<BwdParams&>(p) = all;
  for (int i = 0; i < NP; ++i) p.pair[i] = all.pair[i];
  KERNEL<<<static_cast<int>(blocks), threads, smem, st>>>(p);
  return last_launch_status();
}

// f(true) or f(false), as a compile-time constant
template <class F>
int with(bool b, F f) { return b ? f(std::true_type{}) : f(std::false_type{}); }

// Items of `rows` rows each of `heads` heads (or heads x parts) and `pairs` pairs; false: more than a launch takes.
bool make_items(Items& it, int s, int rows, int heads, int pairs, int causal) {
  const int64_t n = (static_cast<int64_t>(s) + rows - 1) / rows, total = n * heads * pairs;
  if (total > (1 << 29)) return false;
  it.ntile = static_cast<int>(n);
  it.per_pair = static_cast<int>(n * heads);
  it.map = xcd_map(total, causal, static_cast<int64_t>(heads) * pairs);
  return true;
}

int64_t blocks_of(int rows, int per) { return (static_cast<int64_t>(rows) + per - 1) / per; }

constexpr int64_t PART_BYTES = kv::PART_F4 * 16;

// How a call's work is divided: dq by 128-row workgroups with two key parts (split) or by 256-row ones, `parts` workgroups per
// key tile for dk, dv, `q_parts` per row block for dq; which kind's workgroups come first.
struct Plan { bool split; int parts; double us; int q_parts; int64_t bytes; bool q_first; };

// A dk/dv workgroup walks over the query tiles of its whole group of heads, and with grouped heads there are few of them; the walk
// of a row block of dq over many keys may be the whole call.  Several workgroups share such a walk, and their sums (128 KB, 64 KB
// each) go through memory and a further launch.  What a division takes is estimated by placing its workgroups as the hardware does:
// in order, one per CU, each XCD its range of them.  The constants are fitted to 262 calls of 1 to 32 heads (own or grouped) x 200 to
// 9000 rows and 56 spans of 2 to 9 chunks, every division timed: chosen / best 1.003 in the mean for full pairs, 1.005 for
// diagonals, 1.03 for spans (an estimate by even shares, fitted to kernels on 32x32x16 products, 1.03, 1.03 and 1.045).
// us, as it chose / so: one head x 3000 72.3 / 59.4, 32 over 8 heads x 640 diagonal 39.2 / 32.9, x 1280 118.6 / 102.0, 16 over 4 x 2304
// 182 / 143, x 1500 diagonal 65.7 / 57.2, 8 over 2 x 4352 x 5322 381 / 300; span of 4 x 237 33.2 / 25.1.
struct Call {
  int group, s_q, s_k, causal, kv_heads, q_heads;      // heads: of all pairs
  int64_t kv1, n256, n128;      // workgroups of dk, dv undivided, of dq by 256 and by 128 rows
  int64_t q_tiles, k_tiles;     // that an undivided dk/dv workgroup and one of dq walk over
  double mean;                  // of a walk: the query chunk's own keys are half visible
  int64_t ws_bytes;
  bool longest_first;           // (else the kind of which there are fewer per head)
};

bool feasible(const Call& c, int parts, int q_parts) {
  return (parts == 1 || (c.kv1 && parts <= 4 * c.group && c.kv1 * parts <= 1024)) && (q_parts == 1 || c.n128 * q_parts <= 1024) &&
         (q_parts > 1 ? c.n128 * q_parts * QPART_F4 * 16 : 0) + (parts > 1 ? c.kv1 * parts * PART_BYTES : 0) <= c.ws_bytes;
}
// 256-row workgroups of dq where there are many of them or all workgroups run at once.  (In between they are few and long, and
// the estimate has them too short: 32 heads x 900 diagonal 62.2 us, 57.8 split, x 1024 63.0, 60.0.)
bool wide_dq(const Call& c, int parts) { return c.n256 > 128 || c.kv1 * parts + c.n256 <= XCDS * CUS; }

// us: of a workgroup, and per tile of its walk (slower by `slow` with 256 workgroups and more, dq's 128 rows by `many` with four
// rounds of them); `tail`, `late`: see below; of the sums' launches, per part, and their GB/ms; what divisions have to gain.
struct Terms { double f_kv, tile_kv, f_wide, tile_wide, f_split, tile_split, f_slow, slow, many, tail, late, sums_kv, part_kv, sums_q, part_q, rate, gain; };
constexpr Terms PAIR{7.8, 1.356, 14.6, 1.90, 13.7, 0.894, 0.11, 0.01, 0.21, 0.32, 0.32, 1.7, 0.10, 0, 0, 12.8, 0.98};
constexpr Terms SPAN{7.3, 1.343, 6.9, 1.88, 6.7, 1.126, 0.04, 0.02, 0.083, 0.47, 0.66, 2.7, 0.64, 3.2, 0.22, 12.5, 1.0};

Plan estimate(const Call& c, int parts, int q_parts, bool split) {
  const Terms& k = c.longest_first ? SPAN : PAIR;
  const int64_t n_kv = c.kv1 * parts, n_q = split ? c.n128 * q_parts : c.n256;
  const int64_t q_bytes = q_parts > 1 ? n_q * QPART_F4 * 16 : 0, kv_bytes = parts > 1 ? n_kv * PART_BYTES : 0;
  Plan x{split, parts, 0., q_parts, kv_bytes + q_bytes, false};
  const double rounds = static_cast<double>(n_kv + n_q) / (XCDS * CUS), busy = std::min(1., std::max(0., 2 * rounds - 1));
  const double slow = 1 + k.slow * busy, f_slow = 1 + k.f_slow * busy;
  const double f_kv = k.f_kv * f_slow, tile_kv = k.tile_kv * slow, f_q = (split ? k.f_split : k.f_wide) * f_slow;
  const double tile_q = (split ? k.tile_split * (1 + k.many * std::min(1., std::max(0., (rounds - 1) / 3))) : k.tile_wide) * slow;
  const double w_kv = tile_kv * c.q_tiles / parts, w_q = tile_q * c.k_tiles / q_parts;
  x.q_first = c.longest_first ? f_q + w_q > f_kv + w_kv : c.group <= parts;
  const Kind kv{(n_kv + XCDS - 1) / XCDS, f_kv + w_kv, (f_kv + w_kv * c.mean) * (c.causal ? uneven(static_cast<int64_t>(c.kv_heads) * parts) : 1.0),
                blocks_of(c.s_k, kv::BN)};
  const Kind q{(n_q + XCDS - 1) / XCDS, f_q + w_q, (f_q + w_q * c.mean) * (c.causal ? uneven(static_cast<int64_t>(c.q_heads) * q_parts) : 1.0),
               blocks_of(c.s_q, split ? 128 : 256)};
  x.us = makespan(x.q_first ? q : kv, x.q_first ? kv : q, c.causal, f_kv + 2 * k.tile_kv, k.tail, k.late);
  if (parts > 1 || q_parts > 1) x.us /= k.gain;
  if (parts > 1) x.us += k.sums_kv + k.part_kv * parts + 2 * kv_bytes / (k.rate * 1e6);
  if (q_parts > 1) x.us += k.sums_q + k.part_q * q_parts + 2 * q_bytes / (k.rate * 1e6);
  return x;
}
constexpr int PARTS[] = {1, 2, 3, 4, 6, 8, 12, 16, 24, 32};
constexpr int Q_PARTS[] = {1, 2, 3, 4, 6, 8, 12, 16};

Plan best_of(const Call& c, bool dq, int most_q) {
  Plan best{};
  for (int q_parts : Q_PARTS) {
    if (q_parts > most_q || !feasible(c, 1, q_parts)) break;
    double low = 1e30;
    for (int parts : PARTS) {
      if (!feasible(c, parts, q_parts)) break;
      double least = 1e30;
      for (bool split : {false, true}) {
        if (split ? !dq : q_parts > 1 || (dq && !wide_dq(c, parts))) continue;
        const Plan x = estimate(c, parts, q_parts, split);
        if (!best.parts || x.us < best.us) best = x;
        least = std::min(least, x.us);
      }
      low = std::min(low, least);
      if (least > 1.5 * low) break;      // (nor with more)
    }
  }
  return best;
}

// dq alone: 256-row workgroups for walks of 128 key tiles and more, not on a diagonal, where they fill whole rounds of the device
// (a last round of few of them takes as long as any other; two 128-row workgroups per CU share it better).  256 / 128 rows, 32 heads and
// lists of them: 256 workgroups x 8192 keys 0.96, 512 and 768 0.98, 1024 to 2560 0.98 to 1.00, x 16384 and more 0.95 to 0.99; but 320
// 1.22, 384 1.16, 640 1.10; x 6000 0.98 to 1.015, x 4096 0.98 to 1.02, x 2048 1.02 to 1.08, 32 heads x 16 pairs of 128 rows 1.7.
bool wide_alone(const dfa_shape& sh, int pairs) {
  const int64_t rows = static_cast<int64_t>(sh.s_q) * sh.h_q * pairs, rounds = (blocks_of(sh.s_q, 256) * sh.h_q * pairs + 255) / 256;
  return (!sh.causal || sh.s_k / 2 >= sh.s_q) && sh.s_k >= 8192 && rounds * (256 * 256) <= rows + rows / 32;
}

Plan plan(const dfa_shape& sh, int pairs, bool dq, bool dk, int64_t ws_bytes) {
  const int group = sh.h_q / sh.h_kv;
  Call c{group, sh.s_q, sh.s_k, sh.causal, sh.h_kv * pairs, sh.h_q * pairs,
         dk ? blocks_of(sh.s_k, kv::BN) * sh.h_kv * pairs : 0, dq ? blocks_of(sh.s_q, 256) * sh.h_q * pairs : 0,
         dq ? blocks_of(sh.s_q, 128) * sh.h_q * pairs : 0, group * blocks_of(sh.s_q, kv::BM), blocks_of(sh.s_k, qs::BN),
         sh.causal ? 1 - 0.5 * sh.s_q / sh.s_k : 1.0, std::min(ws_bytes, int64_t{128} << 20), false};
  const Plan best = best_of(c, dq, 1);
  // From two keys per row on (a span of chunks) dq's walks may be shared
  if (!dq || !dk || pairs > 1 || sh.s_k / 2 < sh.s_q) return best;
  c.longest_first = true;
  const Plan span = best_of(c, dq, 16);
  // A pair of chunks: only where the gain is beyond what the estimate errs.
  return sh.causal || span.us < 0.88 * best.us ? span : best;
}

}  // namespace

int launch_bwd_bf16(const dfa_shape& sh, const dfa_bwd_pair* pairs, int n, void* ws, int64_t ws_bytes,
                    hipStream_t st) {
  for (; n > MAX_PAIRS; pairs += MAX_PAIRS, n -= MAX_PAIRS) {
    const int rc = launch_bwd_bf16(sh, pairs, MAX_PAIRS, ws, ws_bytes, st);
    if (rc) return rc;
  }
  BwdPairs<MAX_PAIRS> p{};
  for (int i = 0; i < n; ++i) {
    const dfa_bwd_pair& x = pairs[i];
    p.pair[i] = Pair{static_cast<const __bf16*>(x.q), static_cast<const __bf16*>(x.k), static_cast<const __bf16*>(x.v),
                     static_cast<const __bf16*>(x.dO), x.lse, x.delta, x.dq, x.dk, x.dv, x.accumulate_dq,
                     x.accumulate_dkv};
  }
  p.s_q = sh.s_q; p.s_k = sh.s_k; p.h_q = sh.h_q; p.h_kv = sh.h_kv; p.group = sh.h_q / sh.h_kv;
  p.causal = sh.causal; p.off = sh.s_k - sh.s_q; p.scale = sh.scale;
  p.q_sh = sh.q_stride_h; p.q_ss = sh.q_stride_s; p.kv_sh = sh.kv_stride_h; p.kv_ss = sh.kv_stride_s;
  p.l_sh = sh.lse_stride_h; p.dq_sh = sh.dq_stride_h; p.dq_ss = sh.dq_stride_s;
  p.dkv_sh = sh.dkv_stride_h; p.dkv_ss = sh.dkv_stride_s;

  const bool ragged = sh.s_q % kv::BM != 0, dq = pairs[0].dq, dk = pairs[0].dk;
  const Plan pl = plan(sh, n, dq, dk, ws ? ws_bytes : 0);
  p.parts = pl.parts;
  p.q_parts = pl.q_parts;
  p.partial = p.q_partial = static_cast<f32x4*>(ws);
  if (p.parts > 1) p.q_partial += p.parts * blocks_of(sh.s_k, kv::BN) * sh.h_kv * n * kv::PART_F4;
  if (dk && !make_items(p.kv_items, sh.s_k, kv::BN, sh.h_kv * p.parts, n, sh.causal)) return DFA_ERR_SHAPE;
  auto reduce = [&] {
    if (p.parts > 1) k_reduce_dkdv<<<dim3(4, p.kv_items.map.total / p.parts), kv::NT, 0, st>>>(p);
    if (p.q_parts > 1) {
      BwdPairs<1> one;
      static_cast<BwdParams&>(one) = p;
      one.pair[0] = p.pair[0];
      k_reduce_dq<<<dim3(4, p.q_items.map.total / p.q_parts), 256, 0, st>>>(one);
    }
    return last_launch_status();
  };
  if (dk && dq) {
    // Both kinds in one launch: the second kind's workgroups fill the CUs that the first leaves idle.  us per
    // call, two launches / here:  8 heads x 512 rows 35 / 19, x 2048 98 / 60, x 4096 225 / 212;  32 x 4096
    // 823 / 804, x 16384 12364 / 12350;  32 over 8 heads x 1024 119 / 91, x 4096 802 / 783, causal 560 / 475.
    // (Within 2 % either way where the last round of workgroups decides, e.g. 32 x 2777 426 / 435.)
    // The longer workgroups first: a dk/dv workgroup walks over its part of the query heads of a group.
    p.q_first = pl.q_first;
    if (!make_items(p.q_items, sh.s_q, pl.split ? 128 : 256, sh.h_q * p.q_parts, n, sh.causal)) return DFA_ERR_SHAPE;
    const int64_t blocks = xcd_blocks(p.kv_items.map) + xcd_blocks(p.q_items.map);
    // Ten rounds of workgroups and more: nothing is left to fill, and each kind alone has the better use of
    // the L2 (32 heads x 12000 6775 against 6808 us).  (Nor would a grid take more than 2^23 of them.)  A list stays
    // a list: eight diagonal pairs of 32 heads x 2048 take 1374 us as sixteen launches, 1171 as two, 1205 as one; sixteen of
    // 8 heads x 4096 3066 / 1881 / 1933, full pairs 3585 / 3341 / 3338.
    if (p.kv_items.map.total >= 2560) {
      dfa_bwd_pair side[MAX_PAIRS];
      for (int i = 0; i < n; ++i) { side[i] = pairs[i]; side[i].dq = nullptr; }
      const int rc = launch_bwd_bf16(sh, side, n, nullptr, 0, st);
      if (rc) return rc;
      for (int i = 0; i < n; ++i) { side[i] = pairs[i]; side[i].dk = side[i].dv = nullptr; }
      return launch_bwd_bf16(sh, side, n, nullptr, 0, st);
    }
    const int rc = with(n > 1, [&](auto m) {
      constexpr int NP = m() ? MAX_PAIRS : 1;
      return with(ragged, [&](auto r) {
        return with(p.parts > 1, [&](auto s) {
          if constexpr (NP == 1)
            if (p.q_parts > 1) return launch<1, k_bwd_bf16<r(), 2, s(), 1, true>>(p, blocks, kv::NT, kv::SMEM_BYTES, st);
          return pl.split ? launch<NP, k_bwd_bf16<r(), 2, s(), NP>>(p, blocks, kv::NT, kv::SMEM_BYTES, st)
                          : launch<NP, k_bwd_bf16<r(), 1, s(), NP>>(p, blocks, kv::NT, kv::SMEM_BYTES, st);
        });
      });
    });
    return rc ? rc : reduce();
  }
  return with(n > 1, [&](auto m) {
    constexpr int NP = m() ? MAX_PAIRS : 1;
    if (dk) {
      const int64_t blocks = xcd_blocks(p.kv_items.map);
      const int rc = with(ragged, [&](auto r) {
        return with(p.parts > 1, [&](auto s) {
          return launch<NP, k_bwd_dkdv_bf16<r(), s(), NP>>(p, blocks, kv::NT, kv::SMEM_BYTES, st);
        });
      });
      return rc ? rc : reduce();
    }
    const bool wide = wide_alone(sh, n);
    if (!make_items(p.q_items, sh.s_q, wide ? 256 : 128, sh.h_q, n, sh.causal)) return static_cast<int>(DFA_ERR_SHAPE);
    const int64_t blocks = xcd_blocks(p.q_items.map);
    return wide ? launch<NP, k_bwd_dq_bf16<8, NP>>(p, blocks, 512, 6 * qs::TILE_BYTES, st)
                : launch<NP, k_bwd_dq_bf16<4, NP>>(p, blocks, 256, 4 * qs::TILE_BYTES, st);
  });
}

dfa_form bwd_bf16_form(const dfa_shape& sh, int n, bool dq, bool dk, int64_t ws_bytes) {
  n = (n - 1) % MAX_PAIRS + 1;
  if (!dk) return {wide_alone(sh, n) ? 256 : 128, 1, 1, 1};
  const Plan x = plan(sh, n, dq, dk, ws_bytes);
  return {x.split ? 128 : 256, x.split ? 2 : 1, x.parts, x.q_parts};
}

int64_t bwd_bf16_workspace(const dfa_shape& sh, int n, bool dq, bool dk) {
  return plan(sh, std::min(n, MAX_PAIRS), dq, dk, INT64_MAX).bytes;
}

}  // namespace dfa

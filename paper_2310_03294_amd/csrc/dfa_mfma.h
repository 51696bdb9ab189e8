// Building blocks for the bf16 MFMA kernels on gfx950 (CDNA4): vector types, the
// v_mfma_f32_32x32x16_bf16 wrapper with its register layouts, and the LDS tile layout.
//
// v_mfma_f32_32x32x16_bf16 computes C[32x32] += A[32x16] B[16x32] per wavefront.  With
// lane l, r = l % 32, h = l / 32:
//   A operand (8 bf16): A[r][8h .. 8h+7]         B operand (8 bf16): B[8h .. 8h+7][r]
//   C/D (16 fp32):      C[(i/4)*8 + 4h + i%4][r] for i = 0..15
// Because the contraction index only has to match between A and B, a C tile can be fed
// back as the B operand of the next product without any data movement: the 8 values
// C[.][r] with i in [8u, 8u+8) become B[8h+e][r], provided the A operand of that product is
// gathered with the same row order, rows (e/4)*8 + 4h + e%4 of the 16-row block u.
//
// LDS tiles hold rows of 128 bf16 padded to 272 bytes, and logical row r is stored at physical
// row prow(r) (a 4x4 transpose of the low four row bits).  With that, both access patterns
// used here are bank-conflict free AND every address is a per-lane base plus a compile-time
// constant: ds_read_b128 of one 16-byte chunk column from 16 consecutive logical rows (their
// physical rows are 16 distinct values mod 16, and 272 = 256 + 16), and ds_read_b64_tr_b16 of
// 4 consecutive logical rows x 64 B (their physical rows are 4 apart: 4 * 272 = 64 mod 256).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dfa {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));   // an operand piece as raw bits (for values carried around a loop)

#define DFA_LDS __attribute__((address_space(3)))

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// (Inline-assembly forms of the MFMA with operand register files fixed by hand were tried and
// dropped: hipcc places accumulator copies next to such statements without the wait states the
// hardware needs there, which gave wrong results; the builtin above is the only form used.)

// for lambdas that work on register arrays
#define DFA_INLINE __attribute__((always_inline))

#define DFA_SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)
// Workgroup barrier without the wait for this wavefront's outstanding memory operations that
// __syncthreads() puts in front of it.  For a wavefront that only READS shared tiles and whose
// reads still in flight target registers it consumes later (the compiler's own counters cover
// those): nothing it wrote has to be visible to the others.  The "memory" clobber keeps the
// compiler from moving memory accesses across it.
#define DFA_BARRIER_NO_DRAIN() asm volatile("s_barrier" ::: "memory")

constexpr int kRowBytes = 272;

__device__ __forceinline__ int prow(int r) { return (r & ~15) | ((r & 3) << 2) | ((r >> 2) & 3); }

// byte offset of 16-byte chunk c of logical row r
__device__ __forceinline__ int tile_off(int r, int c) { return prow(r) * kRowBytes + (c << 4); }

__device__ __forceinline__ uint32_t lds_addr(const char* p) {
  return static_cast<uint32_t>(reinterpret_cast<uintptr_t>((DFA_LDS const char*)p));
}

__device__ __forceinline__ bf16x8 lds_read_b128(const char* base, int off) {
  return *reinterpret_cast<const bf16x8*>(base + off);
}

// Transposing LDS read (ds_read_b64_tr_b16).  Within each group of 16 lanes, lane j supplies
// the address of 4 consecutive bf16; lane i receives, for t = 0..3, element (i % 4) of the
// 4 that lane (4t + i/4) of its group addressed.
__device__ __forceinline__ bf16x4 lds_read_tr(const char* base, int off) {
  s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16(
      (DFA_LDS s16x4*)(base + off));
  return __builtin_bit_cast(bf16x4, v);
}

// Gather for an operand whose contraction runs over tile ROWS (the tile is stored row-major, so
// this is a transposed read).  gather_base(lane) is the per-lane part; lds_gather(base, off)
// with off = row0 * kRowBytes + col0 * 2 (row0 a multiple of 16, col0 a multiple of 32) returns
// the 8 values  tile[row0 + (e/4)*8 + 4h + e%4][col0 + lane%32],  e = 0..7,  h = lane/32,
// which is the row order in which an MFMA result tile is fed back as a B operand.
__device__ __forceinline__ int gather_base(int lane) {
  const int g = lane >> 4, j = lane & 15;
  return tile_off(4 * (g >> 1) + (j >> 2), 2 * (g & 1) + ((j & 3) >> 1)) + ((j & 1) << 3);
}

// The same from a 32-bit LDS address held in a register that the compiler must take as it is
// (see lds_pin): the constant part of every read then goes into the instruction's offset field.
__device__ __forceinline__ bf16x4 lds_read_tr_at(uint32_t addr, int off) {
  s16x4 v = __builtin_amdgcn_ds_read_tr16_b64_v4i16((DFA_LDS s16x4*)(addr + off));
  return __builtin_bit_cast(bf16x4, v);
}
// Makes `addr` opaque to the compiler, so that it stays THE base register of the reads that
// follow.  Left alone, the compiler may pick a base above them and spend one v_add per read on
// the (negative, not encodable) differences.
__device__ __forceinline__ uint32_t lds_pin(uint32_t addr) {
  asm volatile("" : "+v"(addr));
  return addr;
}

__device__ __forceinline__ bf16x8 lds_gather(const char* base, int off) {
  const bf16x4 lo = lds_read_tr(base, off);
  const bf16x4 hi = lds_read_tr(base, off + 2 * kRowBytes);   // logical rows +8 = physical rows +2
  return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
}

// ---- global memory -> LDS tile copy without a register stop-over --------------------------
// global_load_lds_dwordx4: every lane supplies its own global address and the wavefront's
// 64 x 16 bytes land contiguously at the LDS byte address M0 + the instruction's offset.  A
// padded 64-row tile (64 x kRowBytes = 17 KB) is 17 such 1 KB pieces; of 4 copying wavefronts,
// wavefront w moves pieces 4w .. 4w+3 with ONE write of M0 (the immediate offsets 0, 1024, 2048,
// 3072 step through them; measured: 21 instead of 40 cycles of issue per copy) and wavefront 0
// also piece 16.  Byte 16 s of the tile is chunk s % 17 of physical row s / 17; chunk 16 is the
// row's pad and receives a copy of chunk 15.
//
// The copy is issued from inline assembly, so the compiler neither sees it nor waits for it:
// lds_dma_wait() before the barrier that publishes the tile is the caller's duty.  (Compiler-
// tracked loads stay correct next to it: extra loads in flight only make its waits stricter, so
// keep them before the copies in program order.)
//
// The immediate offset also moves the global address, so piece j's lane offset carries
// 3072 - 1024 j and the scalar base is taken 3072 bytes early: voff holds, per lane and piece,
// that adjusted byte offset from the tile's first row for a tile wholly inside the matrix.
struct TileLane { uint32_t voff[5]; };

__device__ __forceinline__ void tile_lane_rc(int w, int lane, int j, int& row, uint32_t& cb) {
  const int s = (j < 4 ? 4 * w + j : 16) * 64 + lane;
  row = prow(s / 17);                              // prow is its own inverse
  const int c = s % 17;
  cb = static_cast<uint32_t>(c < 15 ? c : 15) * 16;
}

__device__ __forceinline__ TileLane tile_lane(int w, int lane, uint32_t rowbytes) {
  TileLane m;
#pragma unroll
  for (int j = 0; j < 5; ++j) {
    int row; uint32_t cb;
    tile_lane_rc(w, lane, j, row, cb);
    m.voff[j] = static_cast<uint32_t>(row) * rowbytes + cb + (j < 4 ? 3072 - 1024 * j : 3072);
  }
  return m;
}

// gbase and lds must be wave-uniform; v* are this lane's byte offsets from gbase.
__device__ __forceinline__ void lds_dma16(const char* gbase, uint32_t voff, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
               :: "s"(lds), "v"(voff), "s"(gbase) : "memory", "m0");
}
// four consecutive 1 KB pieces at lds; piece j reads from gbase + vj + 1024 j
__device__ __forceinline__ void lds_dma16x4(const char* gbase, uint32_t v0, uint32_t v1, uint32_t v2,
                                            uint32_t v3, uint32_t lds) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\t"
               "global_load_lds_dwordx4 %1, %5\n\t"
               "global_load_lds_dwordx4 %2, %5 offset:1024\n\t"
               "global_load_lds_dwordx4 %3, %5 offset:2048\n\t"
               "global_load_lds_dwordx4 %4, %5 offset:3072"
               :: "s"(lds), "v"(v0), "v"(v1), "v"(v2), "v"(v3), "s"(gbase) : "memory", "m0");
}

// Rows row0 .. row0 + 63 of a [rows, d = 128] bf16 matrix at gbase (row pitch rowbytes) into the
// padded LDS tile at `tile`; rows past `last` are clamped to it (callers mask them).  A tile
// inside the matrix costs no vector arithmetic: the tile's position goes into the scalar base.
__device__ __forceinline__ void tile_dma(const char* gbase, uint32_t rowbytes, int row0, int last,
                                         const TileLane& m, const char* tile, int w, int lane) {
  const uint32_t base = lds_addr(tile);
  const char* g3 = gbase - 3072;                   // see TileLane
  if (row0 + 63 <= last) {
    const char* g = g3 + static_cast<uint64_t>(static_cast<uint32_t>(row0)) * rowbytes;
    lds_dma16x4(g, m.voff[0], m.voff[1], m.voff[2], m.voff[3], base + w * 4096);
    if (w == 0) lds_dma16(g, m.voff[4], base + 16 * 1024);
  } else {
    uint32_t v[5];
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      int row; uint32_t cb;
      tile_lane_rc(w, lane, j, row, cb);
      const int r = row0 + row;
      v[j] = static_cast<uint32_t>(r < last ? r : last) * rowbytes + cb + (j < 4 ? 3072 - 1024 * j : 3072);
    }
    lds_dma16x4(g3, v[0], v[1], v[2], v[3], base + w * 4096);
    if (w == 0) lds_dma16(g3, v[4], base + 16 * 1024);
  }
}

// One wavefront's share of a tile copy (pieces 4w .. 4w + 3, and piece 16 for w == 0), resolved
// to a scalar base and per-lane offsets, so that the pieces can be issued one at a time between
// other instructions: the memory pipe takes about 17 cycles per 1 KB piece and CU, and a
// wavefront that issues its pieces in a burst stalls until the pipe has taken them all.
struct TileCopy {
  const char* g;        // scalar base (taken 3072 bytes early, see TileLane)
  uint32_t v[5];        // per-lane byte offsets of the five pieces
  uint32_t lds, lds16;  // LDS addresses of piece 4w and of piece 16
};

// RAGGED false: the caller guarantees that every tile lies wholly inside the matrix.
template <bool RAGGED = true>
__device__ __forceinline__ TileCopy tile_copy_plan(const char* gbase, uint32_t rowbytes, int row0, int last,
                                                   const TileLane& m, const char* tile, int w, int lane) {
  TileCopy c;
  const uint32_t base = lds_addr(tile);
  c.lds = base + w * 4096;
  c.lds16 = base + 16 * 1024;
  const char* g3 = gbase - 3072;
  if (!RAGGED || row0 + 63 <= last) {              // tile inside the matrix: its position goes into the scalar base
    c.g = g3 + static_cast<uint64_t>(static_cast<uint32_t>(row0)) * rowbytes;
#pragma unroll
    for (int j = 0; j < 5; ++j) c.v[j] = m.voff[j];
  } else {                                         // rows past `last` are clamped to it
    c.g = g3;
#pragma unroll
    for (int j = 0; j < 5; ++j) {
      int row; uint32_t cb;
      tile_lane_rc(w, lane, j, row, cb);
      const int r = row0 + row;
      c.v[j] = static_cast<uint32_t>(r < last ? r : last) * rowbytes + cb + (j < 4 ? 3072 - 1024 * j : 3072);
    }
  }
  return c;
}

// Piece J of the plan: J = 0..3 are pieces 4w + J, J = 4 is piece 16 (issue it from one wavefront only).
template <int J>
__device__ __forceinline__ void tile_copy_piece(const TileCopy& c) {
  if constexpr (J == 0)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(c.lds), "v"(c.v[0]), "s"(c.g) : "memory", "m0");
  else if constexpr (J == 1)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:1024"
                 :: "s"(c.lds), "v"(c.v[1]), "s"(c.g) : "memory", "m0");
  else if constexpr (J == 2)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:2048"
                 :: "s"(c.lds), "v"(c.v[2]), "s"(c.g) : "memory", "m0");
  else if constexpr (J == 3)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:3072"
                 :: "s"(c.lds), "v"(c.v[3]), "s"(c.g) : "memory", "m0");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                 :: "s"(c.lds16), "v"(c.v[4]), "s"(c.g) : "memory", "m0");
}

// A pointer that is the same in all lanes, in scalar registers whatever the compiler can prove of it.
__device__ __forceinline__ const char* uniform_ptr(const void* p) {
  const uint64_t x = reinterpret_cast<uintptr_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x)), hi = __builtin_amdgcn_readfirstlane(static_cast<uint32_t>(x >> 32));
  return reinterpret_cast<const char*>(static_cast<uint64_t>(hi) << 32 | lo);
}

// ---- 16x16x32 tiles -------------------------------------------------------------------------
// v_mfma_f32_16x16x32_bf16 computes C[16x16] += A[16x32] B[32x16]; with lane l, r = l % 16, g = l / 16:
//   A operand (8 bf16): A[r][8g .. 8g+7]     B operand (8 bf16): B[8g .. 8g+7][r]
//   C/D (4 fp32):       C[4g + i][r]
// Why two of these rather than one 32x32x16 of the same work: the device holds its power limit by lowering the
// clock, and a product of this shape costs less energy (half as many accumulator reads and writes per
// multiplication).  On N(0,1) operands the matrix pipes sustain 1.95-2.06 PFLOP/s with it, 1.68-1.80 with the
// larger shape (register-resident stream, 36 ms launches, one device).
// Two C tiles of 16 rows each, one below the other, are fed back as a B operand: the eight values of lane
// group g are rows 4g .. 4g+3 of the first and of the second tile, and the A operand is gathered in that order.
//
// LDS tile: blocks of 16 rows of 128 bf16.  Row r of a block lies at row16_off(r / 4) + 256 (r % 4), its 16-byte
// chunk c at c ^ 2 (r % 4) ^ (r / 8); a row read takes step s of a product over d from chunk 8 (s / 2) + 2g + s % 2.  With
// that a row read (16 rows x 4 chunks, ds_read_b128) and a gather (16 rows x 32 bytes, ds_read_b64_tr_b16) meet every bank
// once per pass, every address is one of two (row reads) or four (gathers) per-lane bases, an exclusive or apart, plus a
// constant, and the four rows of a 1 KB piece of a copy lie together: a tile of 64 rows is 16 pieces, no padding is
// copied.  Tiles start at multiples of 128 bytes.
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// c[i] + the sum of the lane's four bf16 values, for each i (a product against ones).
__device__ __forceinline__ f32x4 mfma_sum4(u32x2 w, f32x4 c) {
  const s16x4 ones = {0x3f80, 0x3f80, 0x3f80, 0x3f80};
  return __builtin_amdgcn_mfma_f32_4x4x4bf16_1k(ones, __builtin_bit_cast(s16x4, w), c, 0, 0, 0);
}

constexpr int kBlock16 = 4608;                        // bytes of a 16-row block
constexpr int kTile64 = 4 * kBlock16;                 // of a 64-row tile
__host__ __device__ constexpr int row16_off(int k) { return 1152 * k; }

// element that step s of a product over d takes first in lane group g (8 from there on)
__device__ __forceinline__ int step16_col(int s, int g) { return 64 * (s >> 1) + 16 * g + 8 * (s & 1); }

// Row reads: rows[r] = X[16 block + lane % 16][step16_col(s, g) ..  + 7].  row16_base: the per-lane part of an address.
__device__ __forceinline__ uint32_t row16_base(int lane) {
  const int r = lane & 15, g = lane >> 4;
  return row16_off(r >> 2) + 256 * (r & 3) + 32 * (g ^ (r & 3)) + 16 * (r >> 3);
}
// (The exclusive or stands at the read, between products: with all of a tile's bases made first, ten dependent instructions at the
// start of a slot kept the matrix pipes waiting: backward of one head x 4096 96.0 -> 94.0 us, 32 heads x 4096 794 -> 787.)
struct Rows16 {
  uint32_t a;
  __device__ __forceinline__ Rows16(const char* tile, uint32_t base) : a(lds_addr(tile) + base) {}
  // tile: of several that lie one after the other (the constant goes into the instruction's offset); two addresses, by s % 2
  __device__ __forceinline__ bf16x8 read(int block, int s, int tile = 0) const {
    return *(DFA_LDS const bf16x8*)((a ^ 16 * (s & 1)) + tile * kTile64 + block * kBlock16 + 128 * (s >> 1));
  }
};

// Gathers: the 8 values  X[16 block + 16 (e/4) + 4g + e%4][16 db + lane%16],  e = 0..7, of two 16-row blocks.
__device__ __forceinline__ uint32_t gather16_base(int lane) {
  const int g = lane >> 4, q = (lane >> 2) & 3, j = lane & 3;
  return row16_off(g) + 256 * q + 32 * q + 16 * ((j >> 1) ^ (g >> 1)) + 8 * (j & 1);
}
struct Gather16 {
  uint32_t a;
  __device__ __forceinline__ Gather16(const char* tile, uint32_t base) : a(lds_addr(tile) + base) {}
  __device__ __forceinline__ bf16x8 read(int block, int db) const {
    const int at = block * kBlock16 + 128 * (db >> 2);
    const uint32_t x = a ^ 32 * (db & 3);             // four addresses, by db % 4
    const bf16x4 lo = lds_read_tr_at(x, at), hi = lds_read_tr_at(x, at + kBlock16);
    return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  }
};

__device__ __forceinline__ bf16x8 pack16(f32x4 a, f32x4 b) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 4; ++e) { r[e] = static_cast<__bf16>(a[e]); r[4 + e] = static_cast<__bf16>(b[e]); }
  return r;
}

// Copies of such tiles: of 4 copying wavefronts, wavefront w moves block w in four pieces.  (As above, the immediate
// offset moves the global address too, so piece j's lane offset carries the difference and the scalar base is early.)
struct TileLane16 { uint32_t voff[4]; };
constexpr int kEarly16 = row16_off(3);

__device__ __forceinline__ void tile16_lane_rc(int w, int lane, int j, int& row, uint32_t& cb) {
  const int q = lane >> 4;
  row = 16 * w + 4 * j + q;
  cb = static_cast<uint32_t>((lane & 15) ^ (2 * q) ^ (j >> 1)) * 16 + (kEarly16 - row16_off(j));
}
__device__ __forceinline__ TileLane16 tile16_lane(int w, int lane, uint32_t rowbytes) {
  TileLane16 m;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    int row; uint32_t cb;
    tile16_lane_rc(w, lane, j, row, cb);
    m.voff[j] = static_cast<uint32_t>(row) * rowbytes + cb;
  }
  return m;
}

struct TileCopy16 {
  const char* g;        // scalar base, kEarly16 bytes early
  uint32_t v[4];        // per-lane byte offsets of the four pieces
  uint32_t lds;         // LDS address of block w
};
// Rows row0 .. row0 + 63 of a [rows, 128] bf16 matrix at gbase; rows past `last` are clamped to it (RAGGED false: there are none).
template <bool RAGGED = true>
__device__ __forceinline__ TileCopy16 tile16_copy_plan(const char* gbase, uint32_t rowbytes, int row0, int last,
                                                       const TileLane16& m, const char* tile, int w, int lane) {
  TileCopy16 c;
  c.lds = lds_addr(tile) + w * kBlock16;
  const char* g = gbase - kEarly16;
  if (!RAGGED || row0 + 63 <= last) {
    c.g = g + static_cast<uint64_t>(static_cast<uint32_t>(row0)) * rowbytes;
#pragma unroll
    for (int j = 0; j < 4; ++j) c.v[j] = m.voff[j];
  } else {
    c.g = g;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int row; uint32_t cb;
      tile16_lane_rc(w, lane, j, row, cb);
      const int r = row0 + row;
      c.v[j] = static_cast<uint32_t>(r < last ? r : last) * rowbytes + cb;
    }
  }
  return c;
}
template <int J>
__device__ __forceinline__ void tile16_copy_piece(const TileCopy16& c) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3"
               :: "s"(c.lds), "v"(c.v[J]), "s"(c.g), "n"(row16_off(J)) : "memory", "m0");
}
// The same without per-lane offsets kept for each piece (seven registers fewer): a row's offset from the first one's, clamped to the
// last row's, as bytes (what passes 2^32 stays there: a few rows far apart).
__device__ __forceinline__ uint32_t sat32(uint64_t x) { return x < 0xffffffffu ? static_cast<uint32_t>(x) : 0xffffffffu; }
struct TileRows16 {
  const char* g;        // scalar base, kEarly16 bytes early
  uint32_t rowbytes, last, row, cb, lds;      // row: of the lane's first piece
  // lane_row: sat32 of (16 w + lane / 16) * rowbytes
  __device__ __forceinline__ TileRows16(const char* gbase, uint32_t rowbytes, int row0, int last_row, const char* tile, int w, int lane,
                                        uint32_t lane_row)
      : g(gbase - kEarly16), rowbytes(rowbytes), last(static_cast<uint32_t>(last_row) * rowbytes),
        row(__builtin_elementwise_add_sat(static_cast<uint32_t>(row0 < last_row ? row0 : last_row) * rowbytes, lane_row)),
        cb(16 * ((lane & 15) ^ (2 * (lane >> 4)))), lds(lds_addr(tile) + w * kBlock16) {}
  template <int J> __device__ __forceinline__ void piece() const {
    const uint32_t r = __builtin_elementwise_add_sat(row, sat32(static_cast<uint64_t>(4 * J) * rowbytes));
    const uint32_t v = (r < last ? r : last) + (cb ^ (16 * (J >> 1))) + (kEarly16 - row16_off(J));
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 offset:%3"
                 :: "s"(lds), "v"(v), "s"(g), "n"(row16_off(J)) : "memory", "m0");
  }
  __device__ __forceinline__ void all() const { piece<0>(); piece<1>(); piece<2>(); piece<3>(); }
};
__device__ __forceinline__ void tile16_copy(const TileCopy16& c) {
  tile16_copy_piece<0>(c); tile16_copy_piece<1>(c); tile16_copy_piece<2>(c); tile16_copy_piece<3>(c);
}

__device__ __forceinline__ void lds_dma_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// acc + the sum of the eight bf16 values of v, in fp32: v_dot2c_f32_bf16 against a pair of ones adds
// two of them per instruction.
__device__ __forceinline__ float sum8(bf16x8 v, float acc) {
  bf16x2 ones;
  ones[0] = static_cast<__bf16>(1.f); ones[1] = ones[0];
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(v, v, 0, 1), ones, acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(v, v, 2, 3), ones, acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(v, v, 4, 5), ones, acc, false);
  acc = __builtin_amdgcn_fdot2_f32_bf16(__builtin_shufflevector(v, v, 6, 7), ones, acc, false);
  return acc;
}

__device__ __forceinline__ bf16x8 pack8(const f32x16& v, int first) {
  bf16x8 r;
#pragma unroll
  for (int e = 0; e < 8; ++e) r[e] = static_cast<__bf16>(v[first + e]);
  return r;
}

}  // namespace dfa

// Measurement aid for the MFMA roofline: a register-resident stream of
// v_mfma_f32_16x16x32_bf16, the product of the kernels that dominate a share, on every SIMD of the device (2 wavefronts per
// SIMD, eight independent accumulator tiles each, no memory traffic inside the loop).  Timed by the caller, it gives what
// the matrix pipes deliver at the clock the device sustains under this load, which sits below the
// published peak (that one assumes the maximum clock).
#include <hip/hip_runtime.h>
#include "dfa.h"
#include "dfa_mfma.h"

namespace dfa {
namespace {
constexpr int PROBE_GRID = 512;      // 2 workgroups of 4 wavefronts per CU on 256 CUs
constexpr int PROBE_BLOCK = 256;

__global__ void __launch_bounds__(PROBE_BLOCK, 2) k_mfma_probe(float* out, int iters) {
  const int lane = threadIdx.x & 63;
  bf16x8 a, b;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    a[i] = static_cast<__bf16>(1.0f / 1024.0f * static_cast<float>((lane + i) & 7));
    b[i] = static_cast<__bf16>(1.0f / 1024.0f * static_cast<float>((lane * 3 + i) & 7));
  }
  f32x4 c[8] = {};
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 8; ++i) c[i] = mfma16(a, b, c[i]);
  }
  float x = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) x += c[i][i & 3];
  out[blockIdx.x * PROBE_BLOCK + threadIdx.x] = x;
}

// The same stream fed with caller-supplied operand values: every wavefront loads eight A and eight B
// operands (16 bytes per lane each) from `ops` once and rotates through them, so that consecutive
// MFMAs see different operands, as they do in the attention kernels.  What the matrix pipes sustain
// depends on the operand VALUES: the device holds a power limit by lowering its clock, and operands
// with many toggling bits draw more power per MFMA than the near-constant ones of the plain probe.
__global__ void __launch_bounds__(PROBE_BLOCK, 2) k_mfma_probe_data(const uint4* __restrict__ ops, uint32_t mask,
                                                                    float* out, int iters) {
  const uint32_t t = blockIdx.x * PROBE_BLOCK + threadIdx.x;
  bf16x8 a[8], b[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    a[i] = __builtin_bit_cast(bf16x8, ops[(t + i * 4099u) & mask]);
    b[i] = __builtin_bit_cast(bf16x8, ops[(t + i * 4099u + 31337u) & mask]);
  }
  f32x4 c[8] = {};
  for (int it = 0; it < iters; ++it) {
#pragma unroll
    for (int i = 0; i < 8; ++i) {      // one A operand for two of B, as the kernels have it
      c[i] = mfma16(a[i], b[i], c[i]);
      c[(i + 4) & 7] = mfma16(a[i], b[(i + 1) & 7], c[(i + 4) & 7]);
    }
    if ((it & 255) == 255) {      // keep the accumulators in range, whatever the operands are
#pragma unroll
      for (int i = 0; i < 8; ++i) c[i] *= 0.001f;
    }
  }
  float x = 0.f;
#pragma unroll
  for (int i = 0; i < 8; ++i) x += c[i][i & 3];
  out[t] = x;
}
}  // namespace
}  // namespace dfa

extern "C" int dfa_mfma_probe(float* out, int64_t n_out, int32_t iters, double* flop, void* stream) {
  using namespace dfa;
  if (out == nullptr) return DFA_ERR_NULL;
  if (iters < 1 || n_out < static_cast<int64_t>(PROBE_GRID) * PROBE_BLOCK) return DFA_ERR_ARG;
  hipStream_t st = static_cast<hipStream_t>(stream);
  k_mfma_probe<<<PROBE_GRID, PROBE_BLOCK, 0, st>>>(out, iters);
  if (hipGetLastError() != hipSuccess) return DFA_ERR_HIP;
  if (flop != nullptr)
    *flop = 2.0 * 16 * 16 * 32 * 8.0 * iters * (PROBE_GRID * (PROBE_BLOCK / 64));   // 8 MFMAs per iteration and wavefront
  return DFA_OK;
}

extern "C" int dfa_mfma_probe_data(const void* operands, int64_t operand_bytes, float* out, int64_t n_out,
                                   int32_t iters, double* flop, void* stream) {
  using namespace dfa;
  if (out == nullptr || operands == nullptr) return DFA_ERR_NULL;
  if (iters < 1 || n_out < static_cast<int64_t>(PROBE_GRID) * PROBE_BLOCK) return DFA_ERR_ARG;
  if ((reinterpret_cast<uintptr_t>(operands) & 15u) != 0) return DFA_ERR_SHAPE;
  // the largest power of two of 16-byte pieces that fits, at least 64 K of them (1 MiB)
  int64_t pieces = 65536;
  if (operand_bytes < pieces * 16) return DFA_ERR_ARG;
  while (pieces * 2 * 16 <= operand_bytes && pieces < (int64_t{1} << 30)) pieces *= 2;
  hipStream_t st = static_cast<hipStream_t>(stream);
  k_mfma_probe_data<<<PROBE_GRID, PROBE_BLOCK, 0, st>>>(static_cast<const uint4*>(operands),
                                                        static_cast<uint32_t>(pieces - 1), out, iters);
  if (hipGetLastError() != hipSuccess) return DFA_ERR_HIP;
  if (flop != nullptr)
    *flop = 2.0 * 16 * 16 * 32 * 16.0 * iters * (PROBE_GRID * (PROBE_BLOCK / 64));   // 16 MFMAs per iteration and wavefront
  return DFA_OK;
}

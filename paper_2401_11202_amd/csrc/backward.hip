// HBM-bound helpers of the MLP backward pass: the activation backward (dZ
// and H from Z and dH, with the block column sums of dZ for db1 fused) and
// deterministic column sums for the bias gradients.
#include "kernels.h"
#include "device_math.h"

namespace partir {
namespace {

typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

constexpr int TR = 64;   // rows of an act_backward tile

__device__ __forceinline__ float bf2f(uint16_t u) { return __uint_as_float((uint32_t)u << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) { return __builtin_bit_cast(uint16_t, (__bf16)f); }

// 256 threads per 64 x TC tile; a thread handles 16-byte chunks (8 elements) of
// Z and dH.  Bound by memory (8 bytes per element).  TC = 128 issues the loads
// of its four chunks before the first store (which the compiler must assume to
// alias them); TC = 64 takes its two chunks one after the other and has more
// workgroups to cover the latency.  The launch says which is taken when.
template <int TC>
__global__ __launch_bounds__(256) void act_backward_kernel(ActBwdParams p) {
  constexpr int TP = TC + 2;               // LDS row pitch in elements (spreads rows over banks)
  constexpr int NCH = TR * TC / 8 / 256;   // 16-byte chunks per thread
  constexpr int FLY = TC == 128 ? NCH : 1; // of them loaded at once
  __shared__ uint16_t tdz[TR][TP];
  const int ntc = (p.cols + TC - 1) / TC;      // 1-D grid: tile (row block, col block)
  const int r0 = (int)(blockIdx.x / ntc) * TR, c0 = (int)(blockIdx.x % ntc) * TC;
  const int tid = threadIdx.x;
  const int c = (tid % (TC / 8)) * 8, rt = tid / (TC / 8);   // chunk k: row rt + k TR / NCH
  i32x4 zv[NCH], gv[NCH];
  auto load = [&](int k) {
    const int r = rt + k * (TR / NCH);
    if (r0 + r < p.rows && c0 + c < p.cols) {
      const int64_t off = (int64_t)(r0 + r) * p.ld + c0 + c;
      zv[k] = *(const i32x4*)(p.Z + off);
      gv[k] = *(const i32x4*)(p.dH + off);
    }
  };
#pragma unroll
  for (int k = 0; k < NCH; ++k) {
    if (k % FLY == 0)
#pragma unroll
      for (int j = 0; j < FLY; ++j) load(k + j);
    const int r = rt + k * (TR / NCH);
    if (r0 + r < p.rows && c0 + c < p.cols) {
      const int64_t off = (int64_t)(r0 + r) * p.ld + c0 + c;
      const uint16_t* z = (const uint16_t*)&zv[k];
      const uint16_t* g = (const uint16_t*)&gv[k];
      i32x4 dzv, hv;
      uint16_t* dz = (uint16_t*)&dzv;
      uint16_t* hh = (uint16_t*)&hv;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float x = bf2f(z[j]);
        float y = x, d = 1.0f;
        if (p.act) gelu_erf_and_grad(x, y, d);
        dz[j] = f2bf(bf2f(g[j]) * d);
        hh[j] = f2bf(y);
        if (p.colpart) tdz[r][c + j] = dz[j];
      }
      *(i32x4*)(p.dZ + off) = dzv;
      *(i32x4*)(p.H + off) = hv;
    }
  }
  if (p.colpart) {
    // column sums of the stored dZ over this tile's rows: four quarters of 16
    // rows, then the quarters in order (a fixed order: deterministic)
    __shared__ float qs[4][TC];
    __syncthreads();
    const int nr = min(TR, p.rows - r0);
#pragma unroll
    for (int e = 0; e < 4 * TC / 256; ++e) {
      const int cc = (tid + 256 * e) % TC, q = (tid + 256 * e) / TC;
      float s = 0.0f;
      if (c0 + cc < p.cols)
        for (int r = q * 16; r < min(nr, q * 16 + 16); ++r) s += bf2f(tdz[r][cc]);
      qs[q][cc] = s;
    }
    __syncthreads();
    if (tid < TC && c0 + tid < p.cols)
      p.colpart[(int64_t)(r0 / TR) * p.cols + c0 + tid] = ((qs[0][tid] + qs[1][tid]) + qs[2][tid]) + qs[3][tid];
  }
}

// stage 1: partial[b][c] = sum_{r in block b} in[r][c] over blocks of 64
// rows, as four quarters of 16 rows added in order.  Wave q of a workgroup
// sums quarter q of 512 columns (8 a lane, its 16 row loads all in flight);
// a bias gradient is a few MB, so the time is the latency of one such round
// (one thread for all 64 rows: 1536 x 2560 22 us, 48 workgroups; now 5.0).
__global__ __launch_bounds__(256) void colsum_partial_kernel(ColSumParams p) {
  __shared__ float qs[4][512];
  const int lane = threadIdx.x & 63, q = threadIdx.x >> 6;
  const int c = blockIdx.y * 512 + lane * 8;
  const int b = blockIdx.x;
  const int q0 = b * kColSumChunk + 16 * q, qe = min(p.rows, q0 + 16);
  i32x4 v[16];
#pragma unroll
  for (int r = 0; r < 16; ++r)
    v[r] = (c < p.cols && q0 + r < qe) ? *(const i32x4*)(p.in + (int64_t)(q0 + r) * p.ld + c) : i32x4{0, 0, 0, 0};
  float s[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int r = 0; r < 16; ++r) {
    const uint16_t* e = (const uint16_t*)&v[r];
#pragma unroll
    for (int j = 0; j < 8; ++j) s[j] += bf2f(e[j]);
  }
#pragma unroll
  for (int j = 0; j < 8; ++j) qs[q][lane * 8 + j] = s[j];
  __syncthreads();
#pragma unroll
  for (int e = 0; e < 2; ++e) {
    const int i = threadIdx.x + 256 * e, col = blockIdx.y * 512 + i;
    if (col < p.cols) p.partial[(int64_t)b * p.cols + col] = ((qs[0][i] + qs[1][i]) + qs[2][i]) + qs[3][i];
  }
}

// stage 2: out[c] = sum_b partial[b][c], blocks ascending
__global__ __launch_bounds__(64) void colsum_final_kernel(ColSumParams p) {
  const int c = blockIdx.x * 64 + threadIdx.x;
  if (c >= p.cols) return;
  const int nb = (p.rows + kColSumChunk - 1) / kColSumChunk;
  float s = 0.0f;
  int b = 0;
  for (; b + 32 <= nb; b += 32) {   // 32 loads in flight, added in block order
    float v[32];
#pragma unroll
    for (int j = 0; j < 32; ++j) v[j] = p.partial[(int64_t)(b + j) * p.cols + c];
#pragma unroll
    for (int j = 0; j < 32; ++j) s += v[j];
  }
  for (; b + 8 <= nb; b += 8) {
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = p.partial[(int64_t)(b + j) * p.cols + c];
#pragma unroll
    for (int j = 0; j < 8; ++j) s += v[j];
  }
  for (; b < nb; ++b) s += p.partial[(int64_t)b * p.cols + c];
  p.out[c] = s;
}

// From here on the four arrays (8 bytes per element) are well past the 256 MB
// of the last-level cache and HBM's latency has to be covered by loads in
// flight.  64- against 128-wide tiles, us: 1536 x 10240 33.6 / 33.7,
// 4096 x 8192 52.1 / 52.6, 8192 x 8192 97.8 / 92.2,
// 8192 x 12288 167 / 150, 8192 x 16384 222 / 196.
constexpr int64_t kWideAct = (int64_t)1 << 26;   // elements

}  // namespace

static unsigned tile_grid(int rows, int cols, int TC) {
  const int64_t n = (int64_t)((rows + TR - 1) / TR) * ((cols + TC - 1) / TC);
  return n < (int64_t)1 << 31 ? (unsigned)n : 0u;
}

hipError_t launch_act_backward(const ActBwdParams& p, hipStream_t s) {
  if (p.rows == 0 || p.cols == 0) return hipSuccess;
  const int tc = (int64_t)p.rows * p.cols >= kWideAct ? 128 : 64;
  const unsigned grid = tile_grid(p.rows, p.cols, tc);
  if (p.rows % 8 || p.cols % 8 || !grid) return hipErrorInvalidValue;
  if (tc == 128) hipLaunchKernelGGL((act_backward_kernel<128>), dim3(grid), dim3(256), 0, s, p);
  else hipLaunchKernelGGL((act_backward_kernel<64>), dim3(grid), dim3(256), 0, s, p);
  return hipGetLastError();
}

hipError_t launch_colsum(const ColSumParams& p, hipStream_t s) {
  if (p.cols == 0) return hipSuccess;
  if (p.cols % 8) return hipErrorInvalidValue;
  const int nb = (p.rows + kColSumChunk - 1) / kColSumChunk;
  const unsigned gy = (unsigned)((p.cols + 511) / 512);
  if (gy > 65535) return hipErrorInvalidValue;
  if (nb > 0 && !p.partial_ready)
    hipLaunchKernelGGL(colsum_partial_kernel, dim3((unsigned)nb, gy), dim3(256), 0, s, p);
  hipLaunchKernelGGL(colsum_final_kernel, dim3((unsigned)((p.cols + 63) / 64)), dim3(64), 0, s, p);
  return hipGetLastError();
}

}  // namespace partir

// A bf16 Linear with a residual on few rows and a long K: its tiles are too few for the chip, so K is cut as well (the EPI_PART form of
// tile_kernel, k_tile.hip) and the kernel here adds the parts, the bias and the residual and takes the norm that follows.  What bounded
// it: 333 x 4096 x 11008 in 64 x 128 tiles is 192 workgroups that multiply 172 K-tiles one after the other at one workgroup a CU, 81 us;
// in four runs of 192 x 128 tiles, 256 workgroups of 43 K-tiles, 48 with the sum.  us, uncut / cut: 700 x 4096 x 11008 95 / 75,
// 70 x 4096 x 11008 44 / 29, 700 x 2048 x 5632 42 / 31, with the norm 333 x 4096 x 4096 37 / 28.
#include <algorithm>
#include "device_common.h"
#include "kernels.h"
#include "split.h"
#include "tile.h"

namespace sm {

typedef unsigned int sp_u32x4 __attribute__((ext_vector_type(4)));
typedef float sp_f32x4 __attribute__((ext_vector_type(4)));

namespace {
constexpr int kSumCols = 2048;      // columns per step of sum_parts_kernel

__device__ __forceinline__ float sp_block_sum(float v, float* red) {
  v = wave_sum(v);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
  __syncthreads();
  v = (red[0] + red[1]) + (red[2] + red[3]);
  __syncthreads();
  return v;
}

// y = sum of the parts + bias + residual (one rounding) and, if a.n, n = norm(y) of the stored values: a workgroup per row, the row
// in registers.  Bound by the parts' bytes, which are in the memory-side cache; everything a row needs is requested before anything
// is summed.
template <int MAXP>
__global__ __launch_bounds__(256) void sum_parts_kernel(SumPartsArgs a) {
  __shared__ float red[4];
  const int nch = a.N / 8;
  const int64_t row = blockIdx.x, base = row * a.N, step = a.M * a.N;
  sp_u32x4 res[MAXP], bias[MAXP], gam[MAXP], bet[MAXP];
  float v[MAXP][8];
#pragma unroll
  for (int j = 0; j < MAXP; ++j) {      // past the row's end: its last chunk again, never stored
    const int c = min((int)threadIdx.x + 256 * j, nch - 1) * 8;
    res[j] = *(const sp_u32x4*)(a.res + base + c);
    bias[j] = *(const sp_u32x4*)((a.bias ? a.bias : a.res) + c);
    gam[j] = *(const sp_u32x4*)((a.n ? a.gamma : a.res) + c);
    bet[j] = *(const sp_u32x4*)((a.n && a.beta ? a.beta : a.res) + c);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[j][e] = 0.f;
  }
  for (int s0 = 0; s0 < a.splits; s0 += 4) {
    sp_f32x4 p[4][MAXP][2];
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int j = 0; j < MAXP; ++j) {
        const float* src = a.part + (int64_t)min(s0 + i, a.splits - 1) * step + base + min((int)threadIdx.x + 256 * j, nch - 1) * 8;
        p[i][j][0] = *(const sp_f32x4*)src;
        p[i][j][1] = *(const sp_f32x4*)(src + 4);
      }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const bool on = s0 + i < a.splits;
#pragma unroll
      for (int j = 0; j < MAXP; ++j)
#pragma unroll
        for (int e = 0; e < 8; ++e) v[j][e] += on ? p[i][j][e >> 2][e & 3] : 0.f;
    }
  }
  float sum = 0.f;
#pragma unroll
  for (int j = 0; j < MAXP; ++j) {
    const int c = threadIdx.x + 256 * j;
    float r[8], b[8];
    unpack8(res[j], r); unpack8(bias[j], b);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[j][e] = (v[j][e] + (a.bias ? b[e] : 0.f)) + r[e];
    const sp_u32x4 o = pack8(v[j]);
    if (c < nch) *(sp_u32x4*)(a.y + base + 8 * c) = o;
    unpack8(o, v[j]);
#pragma unroll
    for (int e = 0; e < 8; ++e) sum += c < nch ? v[j][e] : 0.f;
  }
  if (!a.n) return;
  const float mean = a.rms ? 0.f : sp_block_sum(sum, red) / (float)a.N;
  sum = 0.f;
#pragma unroll
  for (int j = 0; j < MAXP; ++j)
#pragma unroll
    for (int e = 0; e < 8; ++e) { const float d = v[j][e] - mean; sum += (int)threadIdx.x + 256 * j < nch ? d * d : 0.f; }
  const float rstd = rsqrtf(sp_block_sum(sum, red) / (float)a.N + a.eps);
#pragma unroll
  for (int j = 0; j < MAXP; ++j) {
    const int c = threadIdx.x + 256 * j;
    float g[8], b[8];
    unpack8(gam[j], g); unpack8(bet[j], b);
#pragma unroll
    for (int e = 0; e < 8; ++e) v[j][e] = fmaf((v[j][e] - mean) * rstd, g[e], a.beta ? b[e] : 0.f);
    if (c < nch) *(sp_u32x4*)(a.n + base + 8 * c) = pack8(v[j]);
  }
}
}  // namespace

// uncut costs, us: the column-split kernel is bound by its stream of weights, measured at 2 TB/s with 64-row tiles (70 x 4096 x 11008 44,
// 128 x 4096 x 4096 21); with 32-row tiles, in one round, it is the better form (50 x 4096 x 4096 12.0, cut 15.3; 33 x 4096 x 11008
// 25.7, cut 27.5; 100 x 2048 x 5632 13.0, cut 18.5).  gemm_kernel's own estimate is 5 to 30 % low at K >= 4096 on these shapes (333 x 4096 x 4096 31,
// estimated 25); the sum kernel saves 3 to 4 us of the norm's launch
bool splitk_plan(const GemmArgs& g, bool norm_after, SplitKPlan* p) {
  p->splits = 0;
  if (g.M < 1) return false;
  const bool narrow = split_linear_use(g);
  if (narrow && ((g.M + 31) / 32) * ((g.N + 31) / 32) <= 256) return false;
  const double us = narrow ? 3. + 1e-6 * g.N * (double)g.K : 1.1 * gemm_kernel_cost(g);
  return tile_parts_plan(g, .97 * (us + (norm_after ? 3. : 0.)), p);
}

int launch_sum_parts(const SumPartsArgs& sum, void* stream) {
  if (sum.N > 2 * kSumCols || sum.N % 8 || sum.M > INT32_MAX) return (int)hipErrorInvalidValue;
  hipStream_t s = (hipStream_t)stream;
  const dim3 grid((unsigned)sum.M);
  if (sum.N <= kSumCols) sum_parts_kernel<1><<<grid, dim3(256), 0, s>>>(sum);
  else sum_parts_kernel<2><<<grid, dim3(256), 0, s>>>(sum);
  return (int)hipGetLastError();
}

}  // namespace sm

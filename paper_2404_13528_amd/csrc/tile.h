// Large-tile Linears (k_tile.hip).
#pragma once
#include <cstdint>

namespace sm {

struct GemmArgs;
bool tile_linear_use(const GemmArgs& g, int* mi, int* ni);      // whether launch_gemm runs g in large tiles, if it gets past the column-split kernel, and in which (64 mi x 64 ni)
int launch_tile_linear(const GemmArgs& g, int mi, int ni, void* stream);
double gemm_kernel_cost(const GemmArgs& g);                             // what gemm_kernel (k_gemm.hip) takes for g, us

// Strips of the tile grid: xn of them, 8 / xn XCDs per strip; an XCD then reads M / (8 / xn) rows of A and N / xn rows of W, in total
// xn M + (8 / xn) N rows of K elements: the xn that makes that smallest
inline int xcd_strips(int64_t M, int N, int tiles_n) {
  int xn = 1;
  double best = 1e300;
  for (int c = 1; c <= 8; c *= 2) {
    const double rows = (double)c * (double)M + (8.0 / c) * (double)N;
    if (rows < best && c <= tiles_n) { best = rows; xn = c; }
  }
  return xn;
}

// A bf16 Linear with a residual on few rows, cut over K: parts in fp32, summed by a second kernel that also takes the norm behind it
struct SplitKPlan { int mi, ni, splits; };
struct SumPartsArgs {
  const float* part; int splits; int64_t M; int N;      // [splits][M][N]
  const unsigned short *bias, *res; unsigned short* y;  // bias may be null; y may be res
  const unsigned short *gamma, *beta; unsigned short* n; float eps; int rms;      // n != null: the norm of y's rows goes there; beta may be null
};
bool splitk_plan(const GemmArgs& g, bool norm_after, SplitKPlan* p);      // whether that is the better form; by shape alone (a caller who has picked a tile of gemm_kernel, gemm_tile_chosen, gets that)
int launch_sum_parts(const SumPartsArgs& sum, void* stream);
bool tile_parts_plan(const GemmArgs& g, double unsplit, SplitKPlan* p);      // (k_tile.hip) the best tile and number of parts, if better than `unsplit` us
int launch_tile_parts(const GemmArgs& g, int mi, int ni, int splits, float* part, void* stream);
bool gemm_tile_chosen(const GemmArgs& g);                                   // (k_gemm.hip) the caller or the tuner has picked a tile of gemm_kernel for g

}  // namespace sm

// Large-tile Linears (k_tile.hip).
#pragma once

namespace sm {

struct GemmArgs;
bool launch_tile_linear(const GemmArgs& g, void* stream, int* rc);      // runs g in large tiles where that is the better form; false: not
double gemm_kernel_cost(const GemmArgs& g);                             // what gemm_kernel (k_gemm.hip) takes for g, us

}  // namespace sm

// Launchers of the column-split Linears (k_split.hip).
#pragma once
#include <cstdint>
#include "index_map.h"
#include "split_order.h"

namespace sm {

// Linears on few rows (k_split.hip), cut over output columns.  All offsets in elements.
struct LinPhase {
  const void *A, *W, *bias, *res; void* out;      // W row-major [N, K]; bias, res may be null
  const void *ln_g, *ln_b; float eps;             // ln_g != null: LayerNorm of A's rows over K first
  int act;                                        // SM_ACT_NONE or SM_ACT_GELU, before the residual
  const int32_t *a_tab, *o_tab, *r_tab;           // row r of A at a_tab[r] * a_mul (null: r * a_ld), of out at o_tab[r] * o_mul (r * o_ld), of res at r_tab[r] (r * r_ld)
  int a_ld, a_mul, o_ld, o_mul, r_ld;
  int N, K;                                       // multiples of 8 and of 16
  int ring;                                       // 1: K-tiles through a ring of LDS stages (no LayerNorm), 0: whole panels resident
};
struct SplitArgs {
  LinPhase ph[4]; int n_ph, M;
  int tiles_m, tiles_n[4], first[5];              // set by the launchers, as the rest
  unsigned lds_w, lds_g, lds_slot;
  int group_rows, n_groups, group_words, group_tasks;      // chained form: row tiles, groups, counters and tasks of a group
  int* counters;
};
int launch_split_single(SplitArgs& a, int dtype, int mi, int wn, void* stream);      // tile 32 mi x 32 wn: (1, 1), (1, 2), (2, 2)
struct GemmArgs;
bool split_linear_use(const GemmArgs& g);                                       // whether launch_gemm runs g in this form
bool launch_split_linear(const GemmArgs& g, void* stream, int* rc);      // runs g as a single split Linear where that is the better form; false: not
size_t split_counter_ints(int64_t M);             // counters of one chained launch, zero on entry
int launch_split_chain(SplitArgs& a, int* counters, int mi, void* stream);           // bf16; rows in tiles of 32 mi

}  // namespace sm

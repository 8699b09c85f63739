// Subset-table ("cube") engine of whole-order reductions: see nplets_cube.hip.
#pragma once

#include "nplets_fwd_common.hpp"

namespace thoi {

constexpr int kCubeSuffix = 10;                       // variables of a table row
constexpr int kCubeRow = 1 << kCubeSuffix;
constexpr int kCubeMinN = 21, kCubeMaxN = 30;

// Whether the library's choice for this reduction is the cube engine, workspace permitting.
bool cube_wanted(int32_t N, int64_t D, const thoi_nplets* sel, const thoi_eval_opts* opts);
// Datasets whose tables are held at a time, and the bytes of those tables.
int64_t cube_group(int32_t N, int64_t D);
size_t cube_table_bytes(int32_t N, int64_t D);
// Segments the reduction of one dataset leaves (an upper bound).
int64_t cube_segments(int32_t N, int kmin, int kmax);
void cube_launch(const EvalArgs& a, const RedArgs& red, int kmin, int kmax, double* table, hipStream_t s);

}  // namespace thoi

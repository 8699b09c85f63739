// Subset-table ("cube") engine of whole-order reductions: see nplets_cube.hip (the table and the
// filter) and nplets_cube_verify.hip (the n-plets the filter leaves open).
#pragma once

#include <functional>

#include "nplets_fwd_common.hpp"

namespace thoi {

constexpr int kCubeSuffix = 10;                       // variables of a table row
constexpr int kCubeRow = 1 << kCubeSuffix;
constexpr int kCubeMinN = 21, kCubeMaxN = 30;
constexpr int kCubeMinN32 = 26;                       // FP32 + refinement (a factorisation per n-plet / the table, ms, all
                                                      // orders: N = 22 0.51 / 0.45, 23 0.72 / 0.54, 24 1.16 / 0.75, 25
                                                      // 2.06 / 1.12, 26 3.76 / 1.92: the line could lie lower)

// The orders of a call and the rows of one launch: block (chunk c, order i) takes order p[i].k of the
// rows [row0 + c * per, row0 + (c + 1) * per).
struct CubePiece {
    int32_t k, pad;
    int64_t pos0;                                      // position of the order's first n-plet
};
struct CubeTable {
    int32_t n, per, chunks, row0;
    CubePiece p[kCubeMaxN + 1];
};

// N-plets whose result the filter cannot tell (row of the table << 10 | subset of the last ten),
// by order: cnt[k] of them at list + off[k].
struct CubeOpen {
    uint32_t* list;
    uint32_t* cnt;                                     // [32]
    int64_t off[kCubeMaxN + 2];
};
constexpr int kVerifyBlocks = 256;                     // workgroups per order and launch

// Estimated times (ns) of one dataset in FP32: by order, a factorisation of every n-plet and the evaluation of all of
// them as open ones; and the table with none open.
struct CubeCost {
    float factor[kCubeMaxN + 1], open[kCubeMaxN + 1], table;
};

// FP32, by dataset, cleared before the call: whether the table is taken for it, the orders that have reported, and
// their open shares in 2^-16.  FP64: null, the table is taken.
struct CubeGate {
    uint32_t* take;                                    // [D]
    uint32_t* done;                                    // [D]
    uint32_t* share;                                   // [D][32]
};
constexpr size_t kCubeGateBytes = 34 * 4;              // per dataset

// Whether the library's choice for this reduction is the cube engine, workspace permitting.
bool cube_wanted(int32_t N, int64_t D, const thoi_nplets* sel, const thoi_eval_opts* opts);
// Largest order the cube engine takes (FP32: the lane engine's; orders above go to the pair engine).
int cube_kmax(bool f32, int kmax);
// Bytes behind the segments and the queue: tables, sample keys and open lists.
size_t cube_bytes(int32_t N, int64_t D, int kmin, int kmax, bool f32);
// Segments the reduction of a dataset leaves (an upper bound).
int64_t cube_segments(int32_t N, int kmin, int kmax, bool f32);
// beside (or empty): launches of the call that do not touch the table, put on a stream beside the first
// table's build.  rest (or empty): a factorisation of every n-plet of kmin..kmax for the datasets that gate.take
// leaves out.  serial: everything on s.
void cube_launch(const EvalArgs& a, const RedArgs& red, int kmin, int kmax, bool f32, bool serial, const CubeGate& gate,
                 void* mem, const std::function<void(hipStream_t)>& beside,
                 const std::function<void(const FanScope&)>& rest, hipStream_t s);
// Decides gate.take from a sample of each dataset's n-plets (FP32).
void cube_gate_launch(const EvalArgs& a, const CubeTable& tab, const RedArgs& red, const CubeGate& gate, const CubeCost& cost,
                      hipStream_t s);
// The open n-plets of dataset d, evaluated as the lane and pair engines do, on branches `from` to
// `from` + 4 of the scope (modulo what it has).
void cube_verify_launch(const EvalArgs& a, const CubeTable& tab, const CubeOpen& open, const RedArgs& red, int64_t d,
                        bool f32, const FanScope& fan, int from);

}  // namespace thoi

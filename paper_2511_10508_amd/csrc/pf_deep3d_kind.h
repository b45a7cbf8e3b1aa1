// Shapes and launchers of the 3D deep-tile kernels: one (precision, kind) pair
// each, instantiated in kernels_d3d_<kind>_<precision>.hip; kernels_deep3d.hip
// plans and dispatches.
#pragma once

#include "pf_dispatch.h"
#include "pf_internal.h"

namespace pf {

using Deep3Radii = RList<1, 2>;

// W values per lane, LZ planes, EU waves per SIMD that the registers must allow.
template <int W_, int LZ_, int EU_>
struct Deep3Tile {
    static constexpr int W = W_, LZ = LZ_, EU = EU_;
};
// Eight planes, two values per lane (four measured slower at either precision:
// Gray-Scott FP32 96^3 8.8 against 5.4 us a step).  FP32 without reductions
// keeps four waves per SIMD, which costs it at most a few spilled registers
// (192^3 Gray-Scott p4 38 against 42 us); with reductions or in FP64 that spills
// hundreds of bytes (96^3 Allen-Cahn FP64 p4 with reductions 66 against 15 us).
template <typename T, int KIND, int R, bool RED>
using Deep3Flat = Deep3Tile<2, 8, (sizeof(T) == 4 && !RED) ? 4 : 2>;
// Twelve planes: more steps per launch for r = 1, and the least that a
// Cahn-Hilliard step with r = 2 (halo 4) can do with; sixteen for FP32 there
// (96^3 12.5 against 16.5 us).
template <typename T, int KIND, int R, bool RED>
using Deep3Tall = Deep3Tile<2, (KIND == kCH && R == 2 && sizeof(T) == 4 && !RED) ? 16 : 12, 2>;
// FP64 two-field kernels with r = 2 and reductions spill a kilobyte a lane
// (96^3 66 us a step against 30 us marching): not built.
template <typename T, int KIND, int R, bool RED>
constexpr bool deep3d_built()
{
    return !(sizeof(T) == 8 && R == 2 && RED && KIND != kAC);
}

template <typename T, int KIND>
hipError_t launch_deep3d_kind(const Launch &L, const StepArgs<T> &a, const DeepPlan &plan, bool red, hipStream_t s);

}  // namespace pf

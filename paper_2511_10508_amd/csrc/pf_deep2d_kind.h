// Shapes and launchers of the 2D deep-tile kernels: one (precision, kind) pair
// each, instantiated in kernels_d2d_<kind>_<precision>.hip so that the pairs
// compile in parallel; kernels_deep2d.hip plans and dispatches.
#pragma once

#include "pf_dispatch.h"
#include "pf_internal.h"

namespace pf {

using DeepRadii = RList<1, 2>;

// W values per lane, LR rows per wave, at most NWM waves per workgroup (16:
// up to 128 registers a lane; 8: up to 256).
template <int W_, int LR_, int NWM_>
struct DeepTile {
    static constexpr int W = W_, LR = LR_, NWM = NWM_;
};
// The narrow shape (64 columns) fills the chip on small grids.  Two fields
// with reductions take at most eight waves: with 128 registers they spill
// (12-588 B a lane).
template <typename T, int KIND, int R, bool RED>
using DeepNarrow = DeepTile<1, 8, ((KIND == kGS || KIND == kMC) && RED) ? 8 : 16>;
// The wide shape has the smaller halo share.  Two-field FP64 kernels with
// r = 2 or reductions stay narrow (8192^2: Model C r = 2 160 us a step against
// 186 us on 128 columns, Gray-Scott with reductions 166 against 172 us), and what spills at 128 registers takes eight waves.
template <typename T, int KIND, int R, bool RED>
struct DeepWideOf {
    using type = DeepTile<2, 8, 16>;
};
template <int KIND, int R, bool RED>
struct DeepWideOf<float, KIND, R, RED> {
    using type = std::conditional_t<
        KIND == kAC || (KIND == kCH && R == 1), DeepTile<4, 4, 16>,
        std::conditional_t<KIND == kCH && !RED, DeepTile<4, 8, 16>,
                           std::conditional_t<KIND != kCH && RED, DeepTile<2, 8, 8>, DeepTile<2, 8, 16>>>>;
};
template <int KIND, int R, bool RED>
struct DeepWideOf<double, KIND, R, RED> {
    using type = std::conditional_t<
        (KIND == kGS || KIND == kMC) && (R == 2 || RED), DeepNarrow<double, KIND, R, RED>,
        std::conditional_t<RED || KIND == kMC, DeepTile<2, 8, 8>,
                           std::conditional_t<KIND == kCH && R == 1, DeepTile<2, 4, 16>, DeepTile<2, 8, 16>>>>;
};
template <typename T, int KIND, int R, bool RED>
using DeepWide = typename DeepWideOf<T, KIND, R, RED>::type;

// The batched launches: narrow tiles of eight waves (64 x 64 sites), as many
// steps as leave 48 x 48 of them written.
template <typename T, int KIND, int R>
using DeepServed = DeepTile<1, 8, 8>;
constexpr int deep_served_steps(int kind, int r) { return 8 / (kind == kCH ? 2 * r : r); }

template <typename T, int KIND>
hipError_t launch_deep2d_batched_kind(const Launch &L, const BatchTable<T> &t, int32_t k, int32_t S, int32_t blocks,
                                      hipStream_t s);
template <typename T, int KIND>
hipError_t launch_deep2d_kind(const Launch &L, const StepArgs<T> &a, const DeepPlan &plan, bool red, hipStream_t s);

}  // namespace pf

// Runtime -> compile-time dispatch helpers for the kernel families.
#pragma once

#include <type_traits>

#include "pf_internal.h"

namespace pf {

template <int... Rs> struct RList {};

// Calls f(std::integral_constant<int, R>) for the R of the list equal to r.
template <typename F, int R0, int... Rs>
bool dispatch_r(int r, RList<R0, Rs...>, F &&f)
{
    if (r == R0) {
        f(std::integral_constant<int, R0>{});
        return true;
    }
    if constexpr (sizeof...(Rs) > 0)
        return dispatch_r(r, RList<Rs...>{}, f);
    else
        return false;
}

template <typename F>
bool dispatch_kind(int kind, F &&f)
{
    switch (kind) {
    case kAC: f(std::integral_constant<int, kAC>{}); return true;
    case kCH: f(std::integral_constant<int, kCH>{}); return true;
    case kGS: f(std::integral_constant<int, kGS>{}); return true;
    case kMC: f(std::integral_constant<int, kMC>{}); return true;
    default: return false;
    }
}

// dispatch_kind plus the direct-biharmonic Cahn-Hilliard kernels (the
// families that have them: 1D, 2D fused, generic, reductions).
template <typename F>
bool dispatch_kind_all(int kind, F &&f)
{
    if (kind == kCHD) {
        f(std::integral_constant<int, kCHD>{});
        return true;
    }
    return dispatch_kind(kind, f);
}

// dispatch_kind_all plus Model H (the per-site generic kernels only).
template <typename F>
bool dispatch_kind_generic(int kind, F &&f)
{
    if (kind == kMH) {
        f(std::integral_constant<int, kMH>{});
        return true;
    }
    return dispatch_kind_all(kind, f);
}

template <typename F>
void dispatch_prec(int fp32, F &&f)
{
    if (fp32)
        f(float(0));
    else
        f(double(0));
}

inline int64_t cdiv(int64_t a, int64_t b) { return (a + b - 1) / b; }

// Chunks along the marching axis (extent n, `halo` rows or planes computed beyond
// each end of a chunk) of `tiles` tiles: the count with the least rounds of
// workgroups times steps of a workgroup, `slots` of them running at once.  (A
// nearly empty last round costs as much as a full one, and a short chunk is mostly
// halo: Model H p4 FP64 on 256 x 192 x 160 took ten chunks of 16 planes, 880
// workgroups in four rounds of 24 planes; five of 32 make two rounds of 40.)
// `usual` (short chunks, whose planes stay in the last-level cache) stands unless
// the estimate gains 8 %: 512^3 FP32 p4 in ten chunks 1.70 ms, in the eight that
// the estimate finds 7 % better 1.83 ms.
inline int64_t best_chunks(int64_t tiles, int64_t n, int64_t halo, int64_t slots, int64_t usual)
{
    auto cost = [&](int64_t c) {
        const int64_t len = cdiv(n, c), items = tiles * cdiv(n, len);
        // beyond a dozen rounds workgroups no longer start and end together
        const double r = (double)items / (double)slots, rounds = r > 12 ? r + 0.5 : (double)cdiv(items, slots);
        // one round leaves no workgroup to follow an early one
        return rounds * (double)(len + 2 * halo + 2) * (items <= slots ? 1.05 : 1.0);
    };
    int64_t best = usual;
    double least = 0.92 * cost(usual);
    for (int64_t c = 1; c <= 1024 && (c == 1 || cdiv(n, c) >= 4); ++c)
        if (cost(c) < least) {
            least = cost(c);
            best = c;
        }
    return best;
}

}  // namespace pf

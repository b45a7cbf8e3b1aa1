// Launchers of the spectral step's own transforms, per precision; included by
// the kernels_fft_*.hip files and declared to kernels_spectral.hip.
#pragma once

#include "pf_dispatch.h"
#include "pf_fft.h"

namespace pf {

template <typename F, int N0, int... Ns>
bool dispatch_len(int64_t n, RList<N0, Ns...>, F &&f)
{
    return dispatch_r((int)n, RList<N0, Ns...>{}, f);
}

template <typename T>
hipError_t launch_fft_rows_t(const StepArgs<T> &a, const FftArgs &f, bool inverse, hipStream_t s)
{
    hipError_t err = hipErrorInvalidValue;
    dispatch_len(a.nx / 2, RList<32, 64, 128, 256, 512, 1024, 2048, 4096>{}, [&](auto mc) {
        constexpr int M = decltype(mc)::value;
        using S = RowShape<M>;
        const dim3 grid((unsigned)cdiv(a.ny * a.nz, S::ROWS));
        if (inverse)
            hipLaunchKernelGGL((k_fft_rows_inv<T, M>), grid, dim3(S::THREADS), 0, s, a, f);
        else
            hipLaunchKernelGGL((k_fft_rows<T, M>), grid, dim3(S::THREADS), 0, s, a, f);
        err = hipGetLastError();
    });
    return err;
}

template <typename T>
hipError_t launch_fft_cols_t(const SpecArgs &p, const FftArgs &f, int64_t n, bool along_z, int64_t batches,
                             int mode, hipStream_t s)
{
    hipError_t err = hipErrorInvalidValue;
    dispatch_len(n, RList<32, 64, 128, 256, 512, 1024, 2048, 4096>{}, [&](auto nc) {
        constexpr int N = decltype(nc)::value;
        auto go = [&](auto modec, auto zc) {
            constexpr int MODE = decltype(modec)::value;
            constexpr bool Z = decltype(zc)::value;
            using S = ColShape<T, N, Z>;
            const dim3 grid((unsigned)cdiv(f.cols, S::COLS), (unsigned)batches);
            hipLaunchKernelGGL((k_fft_cols<T, N, MODE, Z>), grid, dim3(S::THREADS), 0, s, p, f);
        };
        auto axis = [&](auto zc) {
            if (mode == kFftForward)
                go(std::integral_constant<int, kFftForward>{}, zc);
            else if (mode == kFftUpdate)
                go(std::integral_constant<int, kFftUpdate>{}, zc);
            else if constexpr (!decltype(zc)::value)  // the last axis goes back by the update
                go(std::integral_constant<int, kFftInverse>{}, zc);
        };
        if (along_z)
            axis(std::true_type{});
        else
            axis(std::false_type{});
        err = hipGetLastError();
    });
    return err;
}

}  // namespace pf

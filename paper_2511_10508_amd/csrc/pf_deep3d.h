// 3D deep-tile kernels of libpfmi (gfx950, wave64): bricks in registers, one or
// a few time steps per launch, for grids that the marching kernels' tall tiles
// leave most of the chip idle on.
//
// A workgroup of NW waves owns a brick of LZ planes by 4 NW rows by 16 W
// columns, halo included: a wave holds four rows of 16 lanes, W values per lane
// and every plane, in registers.  z-neighbours are registers, x-neighbours
// rotations within 16 lanes (DPP), y-neighbours come from the brick's copy in
// LDS, two barriers a step.  As in 2D (pf_deep2d.h) the brick is loaded once, S steps
// compute all of it, the halo of S steps keeps the written interior clear of
// what is wrong at its faces, and planes are updated in place by moving R
// slots up and down; a brick as wide (high) as the grid is periodic by itself.
// Same per-site functions and neighbour order as everywhere.
//
// What bounds it: the launch (5.4 us with the loads of a brick) up to 64^3, then the
// VALU times the halo share ((TX TY TZ) / (ow oh od): 2-3), against tall marching
// tiles that keep 48 of 256 compute units busy on 96^3 and take a barrier per
// plane.  Microseconds per step against the autotuned marching kernels (default
// chunk for the first): 96^3 Cahn-Hilliard FP32 p2 with reductions 10.4 (34), 64^3
// Gray-Scott FP32 p2 4.2 (26), 100^3 FP64 10 (18), 128^3 Allen-Cahn FP32 p4 10 (25).
#pragma once

#include "pf_deep2d.h"

namespace pf {

// Value of lane (lane + D) mod 16 of the row of 16 lanes.
template <int D>
__device__ __forceinline__ float row_rot(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, x), 0x120 + (16 - D) % 16, 0xF,
                                                              0xF, false));
}
template <int D>
__device__ __forceinline__ double row_rot(double x)
{
    return row_ror<(16 - D) % 16>(x);
}
template <typename T, int W, int R>
__device__ __forceinline__ void gather_row(const T (&c)[W], T (&e)[W + 2 * R])
{
    static_for<0, W + 2 * R>([&](auto kc) {
        constexpr int k = decltype(kc)::value - R;
        constexpr int d = k >= 0 ? k / W : -((-k + W - 1) / W);
        constexpr int el = k - d * W;
        if constexpr (d == 0)
            e[k + R] = c[el];
        else
            e[k + R] = row_rot<d>(c[el]);
    });
}

template <typename T, int KIND, int R, int W, int LZ>
struct Deep3Shape {
    static constexpr int HS = KIND == kCH ? 2 * R : R;
    static constexpr int NF = nfields_kind(KIND);
    static constexpr int TX = 16 * W;
    static constexpr int NX = KIND == kCH ? 2 : NF;                            // streams in LDS
    static constexpr int LDS_PER_WAVE = NX * LZ * 4 * TX * (int)sizeof(T);
    static_assert(R <= W, "x-neighbours within the next lane");
};

template <typename T, int KIND, int R, int W, int LZ, bool RED>
__device__ __forceinline__ void deep3d_brick(const StepArgs<T> &a, const Deep3Args &p, int par, int32_t tile)
{
    using D = Deep3Shape<T, KIND, R, W, LZ>;
    constexpr int TX = D::TX, NF = D::NF, SL = LZ + R;
    extern __shared__ __align__(16) unsigned char deep_lds[];
    const int l = threadIdx.x & 63, lx = l & 15;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int NW = __builtin_amdgcn_readfirstlane((int)(blockDim.x >> 6));
    const int TY = 4 * NW;
    const int ry = 4 * w + (l >> 4);  // row of the brick
    const int32_t tx = tile % p.tilesx, tyz = tile / p.tilesx, ty = tyz % p.tilesy, tz = tyz / p.tilesy;
    const int32_t nx = (int32_t)a.nx, ny = (int32_t)a.ny, nz = (int32_t)a.nz;
    const int32_t x0 = tx * p.ow - p.hx, y0 = ty * p.oh - p.hy, z0 = tz * p.od - p.hz;
    const int32_t xl = x0 + lx * W;
    const int opar = par ^ 1;
    const int plane = TY * TX;
    T *lds = reinterpret_cast<T *>(deep_lds);
    // this lane's place in plane 0 of stream f, and its y-neighbours' rows
    auto at = [&](int f) { return lds + (size_t)f * LZ * plane + ry * TX + lx * W; };
    int dp[R], dm[R];
#pragma unroll
    for (int j = 1; j <= R; ++j) {
        dp[j - 1] = ((ry + j >= TY ? ry + j - TY : ry + j) - ry) * TX;
        dm[j - 1] = ((ry - j < 0 ? ry - j + TY : ry - j) - ry) * TX;
    }
    bool ov[W], all = true;
    const bool own_row = ry >= p.hy && ry < p.hy + p.oh && y0 + ry < ny;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const int c = lx * W + i;
        ov[i] = own_row && c >= p.hx && c < p.hx + p.ow && xl + i < nx;
        all = all && ov[i];
    }
    auto own_plane = [&](int k) { return k >= p.hz && k < p.hz + p.od && z0 + k < nz; };
    const bool vec = x0 >= 0 && x0 + TX <= nx;
    const int64_t rowoff = (int64_t)wrap32(y0 + ry, ny) * a.pitch;

    T u[KIND == kCH ? LZ : SL][W];
    T v1[NF == 1 ? 1 : KIND == kMC ? LZ : SL][W];
    T aux[(KIND == kCH || KIND == kMC) ? LZ : 1][W];
    constexpr int U0 = KIND == kCH ? 0 : R, V0 = KIND == kMC ? 0 : R;
    {
        int32_t col[W];
#pragma unroll
        for (int i = 0; i < W; ++i) col[i] = wrap32(xl + i, nx);
        const T *in0 = a.buf[0][par], *in1 = a.buf[NF - 1][par];
#pragma unroll
        for (int k = 0; k < LZ; ++k) {
            const int64_t off = (int64_t)wrap32(z0 + k, nz) * a.plane + rowoff;
            if (vec) {
                row_load<W>(in0 + off + xl, u[k + U0]);
                if constexpr (NF == 2) row_load<W>(in1 + off + xl, v1[k + V0]);
            } else {
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    u[k + U0][i] = in0[off + col[i]];
                    if constexpr (NF == 2) v1[k + V0][i] = in1[off + col[i]];
                }
            }
        }
    }
    const T six = T(6);

    // pair sums of every element of plane k: x from e, y from LDS stream f, z from the planes
    auto pairs = [&](auto kc, int f, const T (&e)[W + 2 * R], auto &&row, T (&S)[W][R], T (&yp)[R][W]) {
        constexpr int k = decltype(kc)::value;
        const T *q = at(f) + k * plane;
        static_for<1, R + 1>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            // planes beyond the brick: any value will do
            constexpr int kp = k + j < LZ ? k + j : k, km = k - j >= 0 ? k - j : k;
            T ym[W];
            row_load<W>(q + dp[j - 1], yp[j - 1]);
            row_load<W>(q + dm[j - 1], ym);
#pragma unroll
            for (int i = 0; i < W; ++i)
                S[i][j - 1] = ((e[R + i + j] + e[R + i - j]) + (yp[j - 1][i] + ym[i])) +
                              (row(std::integral_constant<int, kp>{}, i) + row(std::integral_constant<int, km>{}, i));
        });
    };
    auto fwd = [&](auto kc, int i, const T (&e)[W + 2 * R], auto &&row, const T (&yp)[R][W], double (&P)[R]) {
        constexpr int k = decltype(kc)::value;
        static_for<1, R + 1>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            constexpr int kp = k + j < LZ ? k + j : k;
            P[j - 1] = ((double)e[R + i + j] + (double)yp[j - 1][i]) + (double)row(std::integral_constant<int, kp>{}, i);
        });
    };
    // stream f of every plane to LDS
    auto put = [&](int f, auto &&row) {
        T *q = at(f);
        static_for<0, LZ>([&](auto kc) {
            T v[W];
            row(kc, v);
            row_store<W>(q + decltype(kc)::value * plane, v);
        });
    };

    auto step = [&](auto oddc, int32_t s) {
        constexpr bool ODD = decltype(oddc)::value;
        constexpr int U = ODD ? 0 : R, UN = ODD ? R : 0;
        RedState red;
        constexpr int G = Vec<T>::V > W ? Vec<T>::V / W : 1;
        double s0 = 0.0, s1 = 0.0;
        auto add_site = [&](int k, int i, double x, double y) {
            const bool own = ov[i] && own_plane(k);
            s0 += own ? x : 0.0;
            s1 += own ? y : 0.0;
            red.bad += own && !finite_val(x) ? 1u : 0u;
            if constexpr (NF == 2) red.bad += own && !finite_val(y) ? 1u : 0u;
        };
        auto plane_end = [&](int n) {
            if (n % G == 0) {
                acc_add(red.q0, s0);
                acc_add(red.q1, s1);
                s0 = s1 = 0.0;
            }
        };
        if constexpr (KIND == kCH) {
            auto crow = [&](auto kc, int i) { return u[decltype(kc)::value][i]; };
            auto mrow = [&](auto kc, int i) { return aux[decltype(kc)::value][i]; };
            static_for<0, LZ>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                T e[W + 2 * R], S[W][R], yp[R][W];
                gather_row<T, W, R>(u[k], e);
                pairs(kc, 0, e, crow, S, yp);
                static_for<0, W>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    const T c0 = u[k][i];
                    aux[k][i] = ch_mu<T, R>(a, c0, S[i], c0 * six);
                    if constexpr (RED) {
                        const double x = (double)c0;
                        if constexpr (std::is_same<T, double>::value) {
                            add_site(k, i, x, energy_from_mu(a.c2, x, aux[k][i]));
                        } else {
                            double P[R];
                            fwd(kc, i, e, crow, yp, P);
                            add_site(k, i, x, energy_by_parts<R>(a.c1, a.c2, a.w64, 3.0 * a.w64sum, x, P));
                        }
                    }
                });
                if constexpr (RED) plane_end(k + 1);
            });
            put(1, [&](auto kc, T (&q)[W]) {
                for (int i = 0; i < W; ++i) q[i] = aux[decltype(kc)::value][i];
            });
            __syncthreads();
            static_for<0, LZ>([&](auto kc) {
                constexpr int k = decltype(kc)::value;
                T e[W + 2 * R], S[W][R], yp[R][W];
                gather_row<T, W, R>(aux[k], e);
                pairs(kc, 1, e, mrow, S, yp);
                static_for<0, W>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    u[k][i] = ch_update<T, R>(a, u[k][i], S[i], aux[k][i] * six);
                });
            });
            put(0, [&](auto kc, T (&q)[W]) {
                for (int i = 0; i < W; ++i) q[i] = u[decltype(kc)::value][i];
            });
        } else {
            auto urow = [&](auto kc, int i) { return u[decltype(kc)::value + U][i]; };
            auto vrow = [&](auto kc, int i) {
                if constexpr (KIND == kMC)
                    return aux[decltype(kc)::value][i];  // g
                else
                    return v1[(NF == 2 ? decltype(kc)::value + U : 0)][i];
            };
            if constexpr (KIND == kMC) {
                static_for<0, LZ>([&](auto kc) {
                    constexpr int k = decltype(kc)::value;
#pragma unroll
                    for (int i = 0; i < W; ++i) aux[k][i] = mc_g(a, u[k + U][i], v1[k][i]);
                });
            }
            static_for<0, LZ>([&](auto qc) {
                constexpr int k = ODD ? LZ - 1 - decltype(qc)::value : decltype(qc)::value;
                constexpr std::integral_constant<int, k> kc{};
                T e[NF][W + 2 * R], S[NF][W][R], yp[R][W], yq[R][W], res[NF][W];
                gather_row<T, W, R>(u[k + U], e[0]);
                if constexpr (KIND == kMC)
                    gather_row<T, W, R>(aux[k], e[NF - 1]);
                else if constexpr (NF == 2)
                    gather_row<T, W, R>(v1[k + U], e[NF - 1]);
                pairs(kc, 0, e[0], urow, S[0], yp);
                if constexpr (NF == 2) pairs(kc, 1, e[NF - 1], vrow, S[NF - 1], yq);
                static_for<0, W>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    const T u0 = u[k + U][i];
                    if constexpr (KIND == kAC) {
                        res[0][i] = ac_update<T, R>(a, u0, S[0][i], u0 * six);
                    } else if constexpr (KIND == kMC) {
                        mc_update<T, R>(a, u0, v1[k][i], S[0][i], S[NF - 1][i], u0 * six, aux[k][i] * six, res[0][i],
                                        res[NF - 1][i]);
                    } else {
                        const T w0 = v1[(NF == 2 ? k + U : 0)][i];
                        gs_update<T, R>(a, u0, w0, S[0][i], S[NF - 1][i], u0 * six, w0 * six, res[0][i],
                                        res[NF - 1][i]);
                    }
                    if constexpr (RED) {
                        const double x = (double)u0;
                        if constexpr (KIND == kAC) {
                            if constexpr (std::is_same<T, double>::value) {
                                add_site(k, i, x, energy_density<R>(a.c1, a.c2, a.w64, x, S[0][i], x * 6.0));
                            } else {
                                double P[R];
                                fwd(kc, i, e[0], urow, yp, P);
                                add_site(k, i, x, energy_by_parts<R>(a.c1, a.c2, a.w64, 3.0 * a.w64sum, x, P));
                            }
                        } else {
                            add_site(k, i, x, (double)v1[(KIND == kMC ? k : NF == 2 ? k + U : 0)][i]);
                        }
                    }
                });
                if constexpr (RED) plane_end(decltype(qc)::value + 1);
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    u[k + UN][i] = res[0][i];
                    if constexpr (NF == 2) v1[KIND == kMC ? k : k + UN][i] = res[NF - 1][i];
                }
            });
            if (s + 1 < p.steps) {  // uniform: the last step leaves nothing for LDS
                __syncthreads();  // every wave has read the old planes
                put(0, [&](auto kc, T (&q)[W]) {
                    for (int i = 0; i < W; ++i) q[i] = u[decltype(kc)::value + UN][i];
                });
                if constexpr (KIND == kMC)
                    put(1, [&](auto kc, T (&q)[W]) {
                        constexpr int k = decltype(kc)::value;
                        for (int i = 0; i < W; ++i) q[i] = mc_g(a, u[k + UN][i], v1[k][i]);
                    });
                else if constexpr (NF == 2)
                    put(1, [&](auto kc, T (&q)[W]) {
                        for (int i = 0; i < W; ++i) q[i] = v1[decltype(kc)::value + UN][i];
                    });
            }
        }
        if constexpr (RED)
            red_flush_pair(red, a.part + (int64_t)s * kNumQ * a.pstride, a.pstride, (int64_t)tile * NW + w, l);
        __syncthreads();
    };

    put(0, [&](auto kc, T (&q)[W]) {
        for (int i = 0; i < W; ++i) q[i] = u[decltype(kc)::value + U0][i];
    });
    if constexpr (KIND == kMC)
        put(1, [&](auto kc, T (&q)[W]) {
            constexpr int k = decltype(kc)::value;
            for (int i = 0; i < W; ++i) q[i] = mc_g(a, u[k + U0][i], v1[k][i]);
        });
    else if constexpr (NF == 2)
        put(1, [&](auto kc, T (&q)[W]) {
            for (int i = 0; i < W; ++i) q[i] = v1[decltype(kc)::value + V0][i];
        });
    __syncthreads();

    auto write = [&](auto oddc) {
        constexpr bool ODD = decltype(oddc)::value;
        constexpr int U = KIND == kCH ? 0 : ODD ? 0 : R, V = KIND == kMC ? 0 : ODD ? 0 : R;
        T *out0 = a.buf[0][opar], *out1 = a.buf[NF - 1][opar];
        static_for<0, LZ>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            if (!own_plane(k)) return;
            const int64_t off = (int64_t)(z0 + k) * a.plane + rowoff + xl;
            if (vec && all) {
                row_store<W>(out0 + off, u[k + U]);
                if constexpr (NF == 2) row_store<W>(out1 + off, v1[k + V]);
            } else {
#pragma unroll
                for (int i = 0; i < W; ++i)
                    if (ov[i]) {
                        out0[off + i] = u[k + U][i];
                        if constexpr (NF == 2) out1[off + i] = v1[k + V][i];
                    }
            }
        });
    };
    int32_t s = 0;
    for (; s + 2 <= p.steps; s += 2) {
        step(std::false_type{}, s);
        step(std::true_type{}, s + 1);
    }
    if (s < p.steps) {
        step(std::false_type{}, s);
        write(std::true_type{});
    } else {
        write(std::false_type{});
    }
}

template <typename T, int KIND, int R, int W, int LZ, int EU, bool RED>
__global__ void __launch_bounds__(64 * kDeep3Waves) __attribute__((amdgpu_waves_per_eu(EU)))
    k_deep3d(StepArgs<T> a, Deep3Args p)
{
    deep3d_brick<T, KIND, R, W, LZ, RED>(a, p, a.parity, xcd_item(blockIdx.x, gridDim.x));
}

// Persistent batched form, as k_deep2d_batched.
template <typename T, int KIND, int R, int W, int LZ, int EU>
__global__ void __launch_bounds__(64 * kDeep3Waves) __attribute__((amdgpu_waves_per_eu(EU)))
    k_deep3d_batched(BatchTable<T> tb, int32_t k, int32_t S)
{
    const int32_t n = *tb.count;
    const int32_t total = tb.item_start[n];
    for (int32_t b = blockIdx.x; b < total; b += gridDim.x) {
        const int32_t g = xcd_item(b, total);
        const int i = __builtin_amdgcn_readfirstlane(batch_request(tb, n, g));
        const int32_t left = tb.steps[i] - k;
        if (left <= 0) continue;
        const StepArgs<T> a = batch_args(tb, i, k / S);
        Deep3Args p = a.deep;
        p.steps = left < S ? left : S;
        deep3d_brick<T, KIND, R, W, LZ, false>(a, p, 0, g - tb.item_start[i]);
        __syncthreads();  // the next brick reuses the LDS
    }
}

}  // namespace pf

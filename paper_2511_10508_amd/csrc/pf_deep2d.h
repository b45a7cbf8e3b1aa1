// 2D deep-tile kernels of libpfmi (gfx950, wave64): several time steps per
// launch, the tile in registers.
//
// A workgroup of NW waves owns a tile of NW LR rows by 64 W columns, halo
// included: wave w holds rows [w LR, (w + 1) LR), lane l columns
// [l W, (l + 1) W).  It loads the tile once, takes S steps and writes the
// interior once.  Every step computes the whole tile; what depends on values
// beyond it is wrong from the edge inwards, one stencil radius a stage, and
// the halo of S steps keeps the written interior clear of it, so no site is
// masked.  x-neighbours are lane rotations (DPP), y-neighbours are
// registers, and only the first and last r rows of every wave cross waves
// through LDS.  Rotations and the ring of waves wrap round, so a tile as
// wide (high) as the grid needs no halo in x (y): it is periodic by itself.
//
// The state is updated in place: Allen-Cahn, Gray-Scott and the phi of Model C
// keep LR + r row slots and a step moves every row r slots (up on even, down
// on odd steps), so the new row overwrites the row that no later row reads
// and no register is copied; Cahn-Hilliard holds c and mu, Model C rho and
// g = rho + c3 phi^2 besides.  Every site is evaluated with the per-site
// functions and neighbour order of the other kernels, so fields are bitwise
// those of single steps.
//
// What bounds it: small grids the launch (4.1 us with the loads and stores of a
// tile, shared by S steps) and the barrier of a step (0.2 us); from about 1024^2
// the VALU, times the halo share of the tile ((TX TY) / (ow oh): 1.3-1.5), for
// which S is chosen against the 1 / S share of the HBM traffic.  Microseconds
// per step against one or two steps per launch of the marching kernels: 128^2
// Allen-Cahn FP64 p2 0.63 (1.24 with the whole grid in one workgroup), 256^2
// Cahn-Hilliard FP32 p2 0.99 (7.3), 1024^2 Cahn-Hilliard FP64 p4 with
// reductions 7.6 (21.3), 2048^2 Model C FP32 p4 10.4 (22.4), 12000^2
// Allen-Cahn FP64 p2 96 (228), Gray-Scott 236 (468).
#pragma once

#include "pf_device.h"

namespace pf {

// Whole-wave lane rotations by DPP: lane i receives lane i + 1 (wave_rol:1)
// or lane i - 1 (wave_ror:1), lane 63 and lane 0 wrapping round.
__device__ __forceinline__ int rot_from_next(int v) { return __builtin_amdgcn_mov_dpp(v, 0x134, 0xF, 0xF, false); }
__device__ __forceinline__ int rot_from_prev(int v) { return __builtin_amdgcn_mov_dpp(v, 0x13C, 0xF, 0xF, false); }
// Value of lane (lane + D) mod 64.
template <int D>
__device__ __forceinline__ float lane_rot(float x)
{
    int v = __builtin_bit_cast(int, x);
#pragma unroll
    for (int i = 0; i < (D > 0 ? D : -D); ++i) v = D > 0 ? rot_from_next(v) : rot_from_prev(v);
    return __builtin_bit_cast(float, v);
}
template <int D>
__device__ __forceinline__ double lane_rot(double x)
{
    const long long b = __builtin_bit_cast(long long, x);
    int lo = (int)b, hi = (int)(b >> 32);
#pragma unroll
    for (int i = 0; i < (D > 0 ? D : -D); ++i) {
        lo = D > 0 ? rot_from_next(lo) : rot_from_prev(lo);
        hi = D > 0 ? rot_from_next(hi) : rot_from_prev(hi);
    }
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned int)lo);
}

// gather_x by rotations: e[k + R] is the value k columns from the lane's first.
template <typename T, int W, int R>
__device__ __forceinline__ void gather_rot(const T (&c)[W], T (&e)[W + 2 * R])
{
    static_for<0, W + 2 * R>([&](auto kc) {
        constexpr int k = decltype(kc)::value - R;
        constexpr int d = k >= 0 ? k / W : -((-k + W - 1) / W);
        constexpr int el = k - d * W;
        if constexpr (d == 0)
            e[k + R] = c[el];
        else
            e[k + R] = lane_rot<d>(c[el]);
    });
}

template <int W, typename T>
__device__ __forceinline__ void row_load(const T *__restrict__ p, T (&o)[W])
{
    if constexpr (W == 1) {
        o[0] = p[0];
    } else {
        typedef T vec __attribute__((ext_vector_type(W)));
        const vec v = *reinterpret_cast<const vec *>(p);
#pragma unroll
        for (int i = 0; i < W; ++i) o[i] = v[i];
    }
}
template <int W, typename T>
__device__ __forceinline__ void row_store(T *__restrict__ p, const T (&o)[W])
{
    if constexpr (W == 1) {
        p[0] = o[0];
    } else {
        typedef T vec __attribute__((ext_vector_type(W)));
        vec v;
#pragma unroll
        for (int i = 0; i < W; ++i) v[i] = o[i];
        *reinterpret_cast<vec *>(p) = v;
    }
}

// Lane moves of the per-step reductions, all on the VALU (an LDS permute per
// level would stand in the way of a step of a microsecond).
__device__ __forceinline__ void half_swap(double &x, double &y)
{
    // upper half of x with the lower half of y
    long long a = __builtin_bit_cast(long long, x), b = __builtin_bit_cast(long long, y);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)a, (unsigned)b, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(a >> 32), (unsigned)(b >> 32), false, false);
    x = __builtin_bit_cast(double, ((long long)hi[0] << 32) | lo[0]);
    y = __builtin_bit_cast(double, ((long long)hi[1] << 32) | lo[1]);
}
// The value of the other 16-lane row of the pair, beside one's own: x becomes
// that of the even row, the result that of the odd row.
__device__ __forceinline__ double row_pair(double &x)
{
    const long long a = __builtin_bit_cast(long long, x);
    const auto lo = __builtin_amdgcn_permlane16_swap((unsigned)a, (unsigned)a, false, false);
    const auto hi = __builtin_amdgcn_permlane16_swap((unsigned)(a >> 32), (unsigned)(a >> 32), false, false);
    x = __builtin_bit_cast(double, ((long long)hi[0] << 32) | lo[0]);
    return __builtin_bit_cast(double, ((long long)hi[1] << 32) | lo[1]);
}
// row_ror:N within each row of 16 lanes
template <int N>
__device__ __forceinline__ double row_ror(double x)
{
    const long long a = __builtin_bit_cast(long long, x);
    const int lo = __builtin_amdgcn_mov_dpp((int)a, 0x120 + N, 0xF, 0xF, false);
    const int hi = __builtin_amdgcn_mov_dpp((int)(a >> 32), 0x120 + N, 0xF, 0xF, false);
    return __builtin_bit_cast(double, ((long long)hi << 32) | (unsigned)lo);
}

// One step's reductions of a wave: one swap of halves leaves q0 to the lower
// 32 lanes and q1 to the upper, so every level merges one pair for both; the
// count is zero almost always and then costs a ballot.
__device__ __forceinline__ void red_flush_pair(const RedState &r, double2 *part, int64_t pstride, int64_t slot,
                                               int lane)
{
    Acc m = r.q0, o = r.q1;
    half_swap(m.hi, o.hi);
    half_swap(m.lo, o.lo);
    acc_merge(m, o);
    o.hi = row_pair(m.hi);
    o.lo = row_pair(m.lo);
    acc_merge(m, o);
    static_for<0, 4>([&](auto nc) {
        constexpr int N = 8 >> decltype(nc)::value;
        const Acc q{row_ror<N>(m.hi), row_ror<N>(m.lo)};
        acc_merge(m, q);
    });
    double c = 0.0;
    if (__any(r.bad != 0)) c = wave_sum_exact((double)r.bad);
    if (lane == 0) {
        part[slot] = make_double2(m.hi, m.lo);
        part[2 * pstride + slot] = make_double2(c, 0.0);
    }
    if (lane == 32) part[pstride + slot] = make_double2(m.hi, m.lo);
}

// Shape of one kernel: HS rows and columns of halo per step, NX streams of
// edge rows in LDS, double-buffered by step parity (DB) except for
// Cahn-Hilliard, whose two streams (c, mu) alternate between two barriers.
template <typename T, int KIND, int R, int W, int LR>
struct DeepShape {
    static constexpr int HS = KIND == kCH ? 2 * R : R;
    static constexpr int NF = nfields_kind(KIND);
    static constexpr int TX = 64 * W;
    static constexpr int NX = KIND == kCH ? 2 : NF;
    static constexpr int DB = KIND == kCH ? 1 : 2;
    static constexpr int EDGE = 2 * R * TX;                     // values per wave, stream and buffer
    static constexpr int LDS_PER_WAVE = NX * DB * EDGE * (int)sizeof(T);
    static_assert(R <= LR, "a wave's neighbours are the next waves");
};

template <typename T, int KIND, int R, int W, int LR, bool RED>
__device__ __forceinline__ void deep2d_tile(const StepArgs<T> &a, const DeepArgs &p, int par, int32_t tile)
{
    using D = DeepShape<T, KIND, R, W, LR>;
    constexpr int TX = D::TX, NF = D::NF, SL = LR + R;
    extern __shared__ __align__(16) unsigned char deep_lds[];
    const int l = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int NW = __builtin_amdgcn_readfirstlane((int)(blockDim.x >> 6));
    const int wu = w == 0 ? NW - 1 : w - 1, wd = w + 1 == NW ? 0 : w + 1;
    const int32_t ty = tile / p.tilesx, tx = tile - ty * p.tilesx;
    const int32_t nx = (int32_t)a.nx, ny = (int32_t)a.ny;
    const int32_t x0 = tx * p.ow - p.hx, y0 = ty * p.oh - p.hy + w * LR;  // first column, this wave's first row
    const int32_t xl = x0 + l * W;
    const int opar = par ^ 1;

    // edge rows of wave v, stream f, buffer b: first R rows, then last R rows
    auto edge = [&](int b, int f, int v) {
        return reinterpret_cast<T *>(deep_lds) + ((size_t)((b * D::NX + f) * NW + v)) * D::EDGE + l * W;
    };
    // the written columns of this lane and rows of this wave
    bool ov[W], all = true;
#pragma unroll
    for (int i = 0; i < W; ++i) {
        const int c = l * W + i;
        ov[i] = c >= p.hx && c < p.hx + p.ow && xl + i < nx;
        all = all && ov[i];
    }
    unsigned rows = 0;  // bit k: row y0 + k is written
#pragma unroll
    for (int k = 0; k < LR; ++k) {
        const int t = w * LR + k;
        if (t >= p.hy && t < p.hy + p.oh && y0 + k < ny) rows |= 1u << k;
    }
    // whole rows inside the grid: vector accesses (tiles start at multiples of W, rows at multiples of 16 bytes)
    const bool vec = x0 >= 0 && x0 + TX <= nx;

    T u[KIND == kCH ? LR : SL][W];                         // c, phi, u
    T v1[NF == 1 ? 1 : KIND == kMC ? LR : SL][W];          // rho, v
    T aux[(KIND == kCH || KIND == kMC) ? LR : 1][W];       // mu, g
    constexpr int U0 = KIND == kCH ? 0 : R, V0 = KIND == kMC ? 0 : R;  // slot of row 0 at even steps
    {
        int32_t col[W];
#pragma unroll
        for (int i = 0; i < W; ++i) col[i] = wrap32(xl + i, nx);
        const T *in0 = a.buf[0][par], *in1 = a.buf[NF - 1][par];
#pragma unroll
        for (int k = 0; k < LR; ++k) {
            const int64_t off = (int64_t)wrap32(y0 + k, ny) * a.pitch;
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
    const T four = T(4);

    // write the edge rows of one stream: row(k) gives row k's W values
    auto put = [&](int b, int f, auto &&row) {
        T *e = edge(b, f, w);
        static_for<0, R>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            T q[W];
            row(std::integral_constant<int, t>{}, q);
            row_store<W>(e + t * TX, q);
            row(std::integral_constant<int, LR - R + t>{}, q);
            row_store<W>(e + (R + t) * TX, q);
        });
    };
    // the R rows before row 0 (up[m]: row -1 - m) and after the last (dn[m]: row LR + m)
    auto take = [&](int b, int f, T (&up)[R][W], T (&dn)[R][W]) {
        const T *eu = edge(b, f, wu), *ed = edge(b, f, wd);
#pragma unroll
        for (int m = 0; m < R; ++m) {
            row_load<W>(eu + (2 * R - 1 - m) * TX, up[m]);
            row_load<W>(ed + m * TX, dn[m]);
        }
    };
    // neighbour pair sums of element i of row k: x from e, y from the rows
    auto pairs = [&](auto kc, int i, const T (&e)[W + 2 * R], auto &&row, const T (&up)[R][W], const T (&dn)[R][W],
                     T (&S)[R]) {
        constexpr int k = decltype(kc)::value;
        static_for<1, R + 1>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            T yp, ym;
            if constexpr (k + j < LR)
                yp = row(std::integral_constant<int, k + j>{}, i);
            else
                yp = dn[k + j - LR][i];
            if constexpr (k - j >= 0)
                ym = row(std::integral_constant<int, k - j>{}, i);
            else
                ym = up[j - k - 1][i];
            S[j - 1] = (e[R + i + j] + e[R + i - j]) + (yp + ym);
        });
    };
    // forward-neighbour sums in FP64 (energy by parts, FP32 storage)
    auto fwd = [&](auto kc, int i, const T (&e)[W + 2 * R], auto &&row, const T (&dn)[R][W], double (&P)[R]) {
        constexpr int k = decltype(kc)::value;
        static_for<1, R + 1>([&](auto jc) {
            constexpr int j = decltype(jc)::value;
            double yp;
            if constexpr (k + j < LR)
                yp = (double)row(std::integral_constant<int, k + j>{}, i);
            else
                yp = (double)dn[k + j - LR][i];
            P[j - 1] = (double)e[R + i + j] + yp;
        });
    };

    // One step.  ODD: the rows of u (and Gray-Scott's v) are in slots k
    // instead of k + R and move back up.
    auto step = [&](auto oddc, int32_t s) {
        constexpr bool ODD = decltype(oddc)::value;
        constexpr int U = ODD ? 0 : R, UN = ODD ? R : 0;  // slot of row 0: before, after
        const int b = D::DB == 2 ? (ODD ? 1 : 0) : 0;
        RedState red;
        // Reductions: the masked values of G rows (V values, as a row of the
        // marching kernels has) are summed and join the lane's compensated sums.
        constexpr int G = Vec<T>::V > W ? Vec<T>::V / W : 1;
        static_assert(LR % G == 0, "whole groups of rows");
        double s0 = 0.0, s1 = 0.0;
        // value x of field 0 and y (energy density or field 1) of a site of row k
        auto add_site = [&](int k, int i, double x, double y) {
            const bool own = ov[i] && ((rows >> k) & 1u);
            s0 += own ? x : 0.0;
            s1 += own ? y : 0.0;
            red.bad += own && !finite_val(x) ? 1u : 0u;
            if constexpr (NF == 2) red.bad += own && !finite_val(y) ? 1u : 0u;
        };
        auto row_end = [&](int n) {  // n: rows done
            if (n % G == 0) {
                acc_add(red.q0, s0);
                acc_add(red.q1, s1);
                s0 = s1 = 0.0;
            }
        };
        if constexpr (KIND == kCH) {
            auto crow = [&](auto kc, int i) { return u[decltype(kc)::value][i]; };
            auto mrow = [&](auto kc, int i) { return aux[decltype(kc)::value][i]; };
            {
                T up[R][W], dn[R][W];
                take(0, 0, up, dn);
                static_for<0, LR>([&](auto kc) {
                    constexpr int k = decltype(kc)::value;
                    T e[W + 2 * R];
                    gather_rot<T, W, R>(u[k], e);
                    static_for<0, W>([&](auto ic) {
                        constexpr int i = decltype(ic)::value;
                        T S[R];
                        pairs(kc, i, e, crow, up, dn, S);
                        const T c0 = u[k][i];
                        aux[k][i] = ch_mu<T, R>(a, c0, S, c0 * four);
                        if constexpr (RED) {
                            const double x = (double)c0;
                            if constexpr (std::is_same<T, double>::value) {
                                add_site(k, i, x, energy_from_mu(a.c2, x, aux[k][i]));
                            } else {
                                double P[R];
                                fwd(kc, i, e, crow, dn, P);
                                add_site(k, i, x, energy_by_parts<R>(a.c1, a.c2, a.w64, 2.0 * a.w64sum, x, P));
                            }
                        }
                    });
                    if constexpr (RED) row_end(k + 1);
                });
            }
            put(0, 1, [&](auto kc, T (&q)[W]) {
                for (int i = 0; i < W; ++i) q[i] = aux[decltype(kc)::value][i];
            });
            __syncthreads();
            {
                T up[R][W], dn[R][W];
                take(0, 1, up, dn);
                static_for<0, LR>([&](auto kc) {
                    constexpr int k = decltype(kc)::value;
                    T e[W + 2 * R];
                    gather_rot<T, W, R>(aux[k], e);
                    static_for<0, W>([&](auto ic) {
                        constexpr int i = decltype(ic)::value;
                        T S[R];
                        pairs(kc, i, e, mrow, up, dn, S);
                        u[k][i] = ch_update<T, R>(a, u[k][i], S, aux[k][i] * four);
                    });
                });
            }
            put(0, 0, [&](auto kc, T (&q)[W]) {
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
                static_for<0, LR>([&](auto kc) {
                    constexpr int k = decltype(kc)::value;
#pragma unroll
                    for (int i = 0; i < W; ++i) aux[k][i] = mc_g(a, u[k + U][i], v1[k][i]);
                });
            }
            T up[NF][R][W], dn[NF][R][W];
#pragma unroll
            for (int f = 0; f < NF; ++f) take(b, f, up[f], dn[f]);
            static_for<0, LR>([&](auto qc) {
                constexpr int k = ODD ? LR - 1 - decltype(qc)::value : decltype(qc)::value;
                constexpr std::integral_constant<int, k> kc{};
                T e[NF][W + 2 * R], res[NF][W];
                gather_rot<T, W, R>(u[k + U], e[0]);
                if constexpr (KIND == kMC)
                    gather_rot<T, W, R>(aux[k], e[NF - 1]);
                else if constexpr (NF == 2)
                    gather_rot<T, W, R>(v1[k + U], e[NF - 1]);
                static_for<0, W>([&](auto ic) {
                    constexpr int i = decltype(ic)::value;
                    T S[NF][R];
                    pairs(kc, i, e[0], urow, up[0], dn[0], S[0]);
                    if constexpr (NF == 2) pairs(kc, i, e[NF - 1], vrow, up[NF - 1], dn[NF - 1], S[NF - 1]);
                    const T u0 = u[k + U][i];
                    if constexpr (KIND == kAC) {
                        res[0][i] = ac_update<T, R>(a, u0, S[0], u0 * four);
                    } else if constexpr (KIND == kMC) {
                        mc_update<T, R>(a, u0, v1[k][i], S[0], S[NF - 1], u0 * four, aux[k][i] * four, res[0][i],
                                        res[NF - 1][i]);
                    } else {
                        const T w0 = v1[(NF == 2 ? k + U : 0)][i];
                        gs_update<T, R>(a, u0, w0, S[0], S[NF - 1], u0 * four, w0 * four, res[0][i], res[NF - 1][i]);
                    }
                    if constexpr (RED) {
                        const double x = (double)u0;
                        if constexpr (KIND == kAC) {
                            if constexpr (std::is_same<T, double>::value) {
                                add_site(k, i, x, energy_density<R>(a.c1, a.c2, a.w64, x, S[0], x * 4.0));
                            } else {
                                double P[R];
                                fwd(kc, i, e[0], urow, dn[0], P);
                                add_site(k, i, x, energy_by_parts<R>(a.c1, a.c2, a.w64, 2.0 * a.w64sum, x, P));
                            }
                        } else {
                            add_site(k, i, x, (double)v1[(KIND == kMC ? k : NF == 2 ? k + U : 0)][i]);
                        }
                    }
                });
                if constexpr (RED) row_end(decltype(qc)::value + 1);
#pragma unroll
                for (int i = 0; i < W; ++i) {
                    u[k + UN][i] = res[0][i];
                    if constexpr (NF == 2) v1[KIND == kMC ? k : k + UN][i] = res[NF - 1][i];
                }
            });
            put(b ^ 1, 0, [&](auto kc, T (&q)[W]) {
                for (int i = 0; i < W; ++i) q[i] = u[decltype(kc)::value + UN][i];
            });
            if constexpr (KIND == kMC)
                put(b ^ 1, NF - 1, [&](auto kc, T (&q)[W]) {
                    constexpr int k = decltype(kc)::value;
                    for (int i = 0; i < W; ++i) q[i] = mc_g(a, u[k + UN][i], v1[k][i]);
                });
            else if constexpr (NF == 2)
                put(b ^ 1, NF - 1, [&](auto kc, T (&q)[W]) {
                    for (int i = 0; i < W; ++i) q[i] = v1[decltype(kc)::value + UN][i];
                });
        }
        if constexpr (RED)
            red_flush_pair(red, a.part + (int64_t)s * kNumQ * a.pstride, a.pstride,
                           (int64_t)tile * NW + w, l);
        __syncthreads();
    };

    // the edges of the loaded state
    put(0, 0, [&](auto kc, T (&q)[W]) {
        for (int i = 0; i < W; ++i) q[i] = u[decltype(kc)::value + U0][i];
    });
    if constexpr (KIND == kMC)
        put(0, NF - 1, [&](auto kc, T (&q)[W]) {
            constexpr int k = decltype(kc)::value;
            for (int i = 0; i < W; ++i) q[i] = mc_g(a, u[k + U0][i], v1[k][i]);
        });
    else if constexpr (NF == 2)
        put(0, NF - 1, [&](auto kc, T (&q)[W]) {
            for (int i = 0; i < W; ++i) q[i] = v1[decltype(kc)::value + V0][i];
        });
    __syncthreads();

    // write the interior; ODD: after an odd number of steps
    auto write = [&](auto oddc) {
        constexpr bool ODD = decltype(oddc)::value;
        constexpr int U = KIND == kCH ? 0 : ODD ? 0 : R, V = KIND == kMC ? 0 : ODD ? 0 : R;
        T *out0 = a.buf[0][opar], *out1 = a.buf[NF - 1][opar];
        static_for<0, LR>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            if (!((rows >> k) & 1u)) return;
            const int64_t off = (int64_t)(y0 + k) * a.pitch + xl;
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

template <typename T, int KIND, int R, int W, int LR, int NWM, bool RED>
__global__ void __launch_bounds__(64 * NWM) k_deep2d(StepArgs<T> a, DeepArgs p)
{
    deep2d_tile<T, KIND, R, W, LR, RED>(a, p, a.parity, xcd_item(blockIdx.x, gridDim.x));
}

// Persistent batched form (see k_step2d_batched): S steps per launch of every
// request that has steps left at step k of the tick, on tiles of one shape.  The
// loop is uniform over the workgroup.
template <typename T, int KIND, int R, int W, int LR, int NWM>
__global__ void __launch_bounds__(64 * NWM) k_deep2d_batched(BatchTable<T> tb, int32_t k, int32_t S)
{
    const int32_t n = *tb.count;
    const int32_t total = tb.item_start[n];
    for (int32_t b = blockIdx.x; b < total; b += gridDim.x) {
        const int32_t g = xcd_item(b, total);
        const int i = __builtin_amdgcn_readfirstlane(batch_request(tb, n, g));
        const int32_t left = tb.steps[i] - k;
        if (left <= 0) continue;
        const StepArgs<T> a = batch_args(tb, i, k / S);
        const DeepArgs p{left < S ? left : S, a.deep.hx, a.deep.hy, a.deep.ow, a.deep.oh, a.deep.tilesx};
        deep2d_tile<T, KIND, R, W, LR, false>(a, p, 0, g - tb.item_start[i]);
        __syncthreads();  // the next tile reuses the LDS
    }
}

}  // namespace pf

// Planning and dispatch of the 3D deep-tile kernels (their launchers are
// instantiated per precision and kind in kernels_d3d_*.hip).
#include <algorithm>
#include <cmath>

#include "pf_deep3d.h"
#include "pf_deep3d_kind.h"

namespace pf {

namespace {

constexpr int kCUs = 256;
constexpr int kLdsPerCU = 160 * 1024;

// VALU instructions per site and step, fitted to the measured times (32^3 to
// 192^3) of every kernel, spills included: [flat, tall] per (kind, r), FP32 then
// FP64, without and with reductions.
constexpr double kOps[4][2][2][2][2] = {
    // [kind][r - 1][fp64][red][tall]
    {{{{4, 4}, {31, 42}}, {{4, 10}, {39, 53}}}, {{{7, 9}, {61, 68}}, {{6, 17}, {69, 157}}}},        // AC
    {{{{12, 20}, {54, 120}}, {{20, 41}, {65, 100}}}, {{{60, 60}, {110, 110}}, {{70, 70}, {300, 300}}}},  // CH
    {{{{14, 22}, {49, 63}}, {{24, 43}, {73, 73}}}, {{{17, 45}, {85, 133}}, {{29, 68}, {400, 400}}}},   // GS
    {{{{15, 32}, {48, 64}}, {{26, 61}, {90, 90}}}, {{{17, 50}, {89, 146}}, {{36, 121}, {400, 400}}}},  // MC
};

}  // namespace

// Estimated as in 2D (plan_deep2d): a fixed part per launch, the steps of the
// waves that share a SIMD, a fixed part per round of bricks, and the traffic at
// 9 TB/s (these grids stay in the last-level cache).  Stencils with a halo of
// one plane a step take at least two steps a launch (96^3 Gray-Scott with
// reductions 11 against 17 us).  On 32^3 to 192^3 the plan it picks was within 5 %
// (mean) of the best of 25 (steps, waves) pairs of either shape.
bool plan_deep3d(const Launch &L, int64_t nx, int64_t ny, int64_t nz, int64_t steps, bool red, DeepPlan *plan)
{
    if (L.ndim != 3 || steps < 1 || nx > (1 << 30) || ny > (1 << 30) || nz > (1 << 30)) return false;
    bool ok = false;
    dispatch_prec(L.fp32, [&](auto tz) {
        using T = decltype(tz);
        dispatch_kind(L.kind, [&](auto kc) {
            constexpr int KIND = decltype(kc)::value;
            dispatch_r(L.r, Deep3Radii{}, [&](auto rc) {
                constexpr int R = decltype(rc)::value;
                if (red && !deep3d_built<T, KIND, R, true>()) return;
                double best = 1e30;
                auto consider = [&](auto tile, int tall) {
                    using Tile = decltype(tile);
                    constexpr int W = Tile::W, LZ = Tile::LZ;
                    using D = Deep3Shape<T, KIND, R, W, LZ>;
                    const int stages = KIND == kCH ? 2 : 1;
                    const double wave_ops = LZ * W * kOps[KIND - 1][R - 1][sizeof(T) == 8][red][tall];
                    for (int waves : {2, 3, 4, 6, 8}) {
                        const int lds = waves * D::LDS_PER_WAVE;
                        if (lds > kLdsPerCU) continue;
                        const int res = std::max(1, std::min(Tile::EU * 4 / waves, kLdsPerCU / lds));
                        for (int S : {1, 2, 3, 4}) {
                            const int h = S * D::HS;
                            if (S > steps || 2 * h + 2 > LZ || (S == 1 && steps > 1 && D::HS == 1)) continue;
                            const int TX = D::TX, TY = 4 * waves;
                            const int hx = nx == TX ? 0 : (h + W - 1) / W * W, hy = ny == TY ? 0 : h;
                            if (TX - 2 * hx < 4 || TY - 2 * hy < 2) continue;
                            const int64_t tx = cdiv(nx, TX - 2 * hx), ty = cdiv(ny, TY - 2 * hy);
                            const int64_t tzs = cdiv(nz, LZ - 2 * h), tiles = tx * ty * tzs;
                            if (tiles * waves >= kDeepMaxWaves) continue;
                            const double b = (double)tiles / kCUs;
                            auto step_us = [&](double blocks) {
                                return blocks * waves / 4 * wave_ops * 4 / 2400.0 + (blocks <= 1 ? 0.48 * stages : 0.0);
                            };
                            double t = 5.4 + ((double)tiles * TX * TY * LZ + (double)nx * ny * nz) * sizeof(T) *
                                                 D::NF / 9e6;
                            if (b <= res) {
                                t += S * step_us(std::ceil(b));
                            } else {
                                double rounds = b / res;
                                if (rounds < 4) rounds = 0.43 * rounds + 0.57 * std::ceil(rounds);
                                t += rounds * (S * step_us(res) + 0.43) * (waves > 4 ? 1.16 : 1.0);
                            }
                            const double us = t / S;
                            if (us < best) {
                                best = us;
                                plan->wide = tall;
                                plan->waves = waves;
                                plan->tiles = (int32_t)tiles;
                                plan->lds = lds;
                                plan->us = us;
                                plan->steps = S;
                                plan->args3 = Deep3Args{S, hx, hy, h, (int32_t)(cdiv(cdiv(nx, tx), W) * W),
                                                        (int32_t)cdiv(ny, ty), (int32_t)cdiv(nz, tzs), (int32_t)tx,
                                                        (int32_t)ty};
                            }
                        }
                    }
                };
                if (red) {
                    consider(Deep3Flat<T, KIND, R, true>{}, 0);
                    consider(Deep3Tall<T, KIND, R, true>{}, 1);
                } else {
                    consider(Deep3Flat<T, KIND, R, false>{}, 0);
                    consider(Deep3Tall<T, KIND, R, false>{}, 1);
                }
                ok = best < 1e30;
            });
        });
    });
    return ok;
}

bool plan_deep2d_served(const Launch &L, int64_t nx, int64_t ny, Deep3Args *a, int32_t *tiles, double *work_us);

bool plan_deep_served(const Launch &L, int64_t nx, int64_t ny, int64_t nz, Deep3Args *a, int32_t *tiles, double *work_us)
{
    if (L.ndim == 2) return plan_deep2d_served(L, nx, ny, a, tiles, work_us);
    if (L.ndim != 3) return false;
    bool ok = false;
    dispatch_prec(L.fp32, [&](auto tz) {
        using T = decltype(tz);
        dispatch_kind(L.kind, [&](auto kc) {
            constexpr int KIND = decltype(kc)::value;
            dispatch_r(L.r, Deep3Radii{}, [&](auto rc) {
                constexpr int R = decltype(rc)::value;
                using V = Deep3Served<T, KIND, R>;
                using Tile = typename V::tile;
                constexpr int W = Tile::W, LZ = Tile::LZ;
                using D = Deep3Shape<T, KIND, R, W, LZ>;
                const int h = V::steps * D::HS, TX = D::TX, TY = 4 * V::waves;
                const int hx = nx == TX ? 0 : (h + W - 1) / W * W, hy = ny == TY ? 0 : h;
                const int64_t tx = cdiv(nx, TX - 2 * hx), ty = cdiv(ny, TY - 2 * hy), tzs = cdiv(nz, LZ - 2 * h);
                if (tx * ty * tzs > (1 << 24)) return;
                *a = Deep3Args{V::steps, hx, hy, h, (int32_t)(cdiv(cdiv(nx, tx), W) * W), (int32_t)cdiv(ny, ty),
                               (int32_t)cdiv(nz, tzs), (int32_t)tx, (int32_t)ty};
                *tiles = (int32_t)(tx * ty * tzs);
                const bool tall = KIND == kCH && R == 2;
                // instructions over 1024 SIMDs, and the bricks' loads at 2.4 TB/s (six requests
                // of 200^3, estimated / measured us per step: Allen-Cahn p2 FP32 155 / 149,
                // Gray-Scott p2 FP32 335 / 339, Gray-Scott p2 FP64 660 / 562)
                *work_us = (double)*tiles * (V::waves * LZ * W * kOps[KIND - 1][R - 1][sizeof(T) == 8][0][tall] * 4 /
                                                 2400.0 / (4 * kCUs) +
                                             (double)TX * TY * LZ * sizeof(T) * D::NF / 2.4e6 / V::steps);
                ok = true;
            });
        });
    });
    return ok;
}

// Thousands of sites up to which the bricks beat the (autotuned) marching
// kernels, from both measured on 40^3 to 256^3: the marching kernels take about the
// same time from 40^3 to 128^3 (FP32 Gray-Scott p2 24-26 us a step, bricks 3.6, 7.0,
// 10.5 at 40^3, 100^3, 128^3 and 49 against 56 at 256^3; FP64 Cahn-Hilliard p4 16-20
// us, bricks 8, 11, 36 at 40^3, 64^3, 100^3), so they win from where the halo share
// of a brick outweighs the compute units that their tall tiles leave idle.
int64_t deep3d_most_sites(const Launch &L, bool red)
{
    constexpr int64_t k[4][2][2][2] = {
        // [kind][r - 1][fp64][red]
        {{{17000, 6000}, {4000, 2500}}, {{17000, 4000}, {2200, 1200}}},  // AC
        {{{2000, 1800}, {500, 700}}, {{900, 700}, {400, 0}}},            // CH
        {{{17000, 5000}, {2100, 2100}}, {{4000, 1800}, {1200, 0}}},      // GS
        {{{4000, 2800}, {1200, 1000}}, {{4000, 1800}, {1200, 0}}},       // MC
    };
    if (L.kind < kAC || L.kind > kMC || L.r < 1 || L.r > 2) return 0;
    return 1000 * k[L.kind - 1][L.r - 1][!L.fp32][red];
}

hipError_t launch_deep3d(const Launch &L, const void *args, const DeepPlan &plan, int32_t steps, bool red,
                         hipStream_t s)
{
    hipError_t err = hipErrorInvalidValue;
    if (steps < 1 || steps > plan.steps || plan.tiles < 1) return err;
    DeepPlan p = plan;
    p.args3.steps = steps;
    dispatch_prec(L.fp32, [&](auto tz) {
        using T = decltype(tz);
        dispatch_kind(L.kind, [&](auto kc) {
            err = launch_deep3d_kind<T, decltype(kc)::value>(L, *static_cast<const StepArgs<T> *>(args), p, red, s);
        });
    });
    return err;
}

}  // namespace pf

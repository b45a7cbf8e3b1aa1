// Planning and dispatch of the 2D deep-tile kernels (their launchers are
// instantiated per precision and kind in kernels_d2d_*.hip).
#include <algorithm>
#include <cmath>

#include "pf_deep2d.h"
#include "pf_deep2d_kind.h"

namespace pf {

namespace {

constexpr int kCUs = 256;
constexpr int kLdsPerCU = 160 * 1024;

// VALU instructions per site and step, fitted (with the other constants of
// plan_deep2d) to the measured times of 31 kernels on 128^2 to 8192^2 grids.
double ops_per_site(int kind, int r, bool fp32, bool red)
{
    double o = kind == kAC ? (r == 1 ? 9.7 : 20.0) : kind == kCH ? (r == 1 ? 13.5 : 36.7) : (r == 1 ? 27.0 : 47.5);
    if (fp32) o *= 0.8;
    if (red) o += fp32 ? 24.0 : kind == kAC ? 27.0 : kind == kCH ? 31.0 : 23.0;
    return o;
}

}  // namespace

// Estimated time of one launch of S steps: a fixed part (launch to launch
// 2.4 us, the first loads and last stores of a tile), S steps of the waves a
// SIMD holds (a wave's instruction takes four clocks at 2.4 GHz) with the
// barriers' latency where few workgroups share a CU, and the HBM traffic
// (5.65 TB/s) where the chip turns over more than one round of tiles; there
// tiles of more than 64 rows measured slower (one workgroup per CU, whose
// loads and stores nothing covers).  On 128^2 to 8192^2 the plan it picks was
// within 5 % (mean) of the best of up to 45 (steps, waves) pairs per shape.
bool plan_deep2d(const Launch &L, int64_t nx, int64_t ny, int64_t steps, bool red, DeepPlan *plan)
{
    if (L.ndim != 2 || steps < 1 || nx > (1 << 30) || ny > (1 << 30)) return false;
    bool ok = false;
    dispatch_prec(L.fp32, [&](auto tz) {
        using T = decltype(tz);
        dispatch_kind(L.kind, [&](auto kc) {
            constexpr int KIND = decltype(kc)::value;
            dispatch_r(L.r, DeepRadii{}, [&](auto rc) {
                constexpr int R = decltype(rc)::value;
                double best = 1e30;
                const double ops = ops_per_site(KIND, R, L.fp32, red);
                auto consider = [&](auto tile, int wide) {
                    using Tile = decltype(tile);
                    using D = DeepShape<T, KIND, R, Tile::W, Tile::LR>;
                    constexpr int W = Tile::W, LR = Tile::LR;
                    const int stages = KIND == kCH ? 2 : 1;
                    const double wave_ops = LR * W * ops + (red ? 65.0 : 0.0);
                    for (int waves : {4, 6, 8, 12, 16}) {
                        if (waves > Tile::NWM) continue;
                        const int lds = waves * D::LDS_PER_WAVE;
                        if (lds > kLdsPerCU) continue;
                        const int res = std::max(1, std::min(Tile::NWM / waves, kLdsPerCU / lds));
                        for (int S : {1, 2, 3, 4, 6, 8, 12, 16, kDeepMaxSteps}) {
                            if (S > steps || (S > 1 && S * D::HS > 24)) continue;
                            const int h = S * D::HS;
                            const int TX = D::TX, TY = waves * LR;
                            const int hx = nx == TX ? 0 : (h + W - 1) / W * W, hy = ny == TY ? 0 : h;
                            if (TX - 2 * hx < 8 || TY - 2 * hy < 4) continue;
                            const int64_t tx = cdiv(nx, TX - 2 * hx), ty = cdiv(ny, TY - 2 * hy);
                            const int64_t tiles = tx * ty;
                            if (tiles * waves >= kDeepMaxWaves) continue;
                            const double b = (double)tiles / kCUs;
                            auto step_us = [&](double blocks) {
                                return blocks * waves / 4 * wave_ops * 4 / 2400.0 +
                                       0.2 * stages * (blocks <= 1 ? 1.0 : blocks <= 2 ? 0.65 : 0.07);
                            };
                            const double bytes = ((double)tiles * TX * TY + (double)nx * ny) * sizeof(T) * D::NF;
                            double t = 4.1;
                            if (b <= res) {
                                t += S * step_us(std::ceil(b)) + bytes / 8e6;
                            } else {
                                double rounds = b / res;
                                if (rounds < 4) rounds = 0.6 * rounds + 0.4 * std::ceil(rounds);
                                const double high = TY > 96 ? 1.25 : TY > 64 ? 1.12 : 1.0;
                                t += std::max(high * rounds * S * step_us(res) + bytes / 13.5e6, bytes / 5.65e6);
                            }
                            const double us = t / S;
                            if (us < best) {
                                best = us;
                                plan->wide = wide;
                                plan->waves = waves;
                                plan->tiles = (int32_t)tiles;
                                plan->lds = lds;
                                plan->us = us;
                                plan->steps = S;
                                plan->args = DeepArgs{S, hx, hy, (int32_t)(cdiv(cdiv(nx, tx), W) * W),
                                                      (int32_t)cdiv(ny, ty), (int32_t)tx};
                            }
                        }
                    }
                };
                if (red) {
                    consider(DeepNarrow<T, KIND, R, true>{}, 0);
                    consider(DeepWide<T, KIND, R, true>{}, 1);
                } else {
                    consider(DeepNarrow<T, KIND, R, false>{}, 0);
                    consider(DeepWide<T, KIND, R, false>{}, 1);
                }
                ok = best < 1e30;
            });
        });
    });
    return ok;
}

// Where the two-step marching kernels overtake (march / deep times measured on
// 512^2 to 20000^2 grids, FP64 / FP32): they compute no halo rows within a
// strip, so they win where the halo is wide (r = 2) or the reductions make
// every computed site dear.
//   r = 1: never (1.2-2.5 times at 20000^2);  r = 2: Allen-Cahn never / 3000^2
//   (0.97), Cahn-Hilliard 1500^2 (1.4) to 3000^2 (0.74), Gray-Scott and
//   Model C 6000^2 (1.03-1.1) to 12000^2 (0.8)
//   reductions, r = 1: Gray-Scott FP64 never (1.26), the others at 3000^2 (0.9-1.2;
//   1500^2 2.0-2.9);  r = 2: 1500^2 (1.0-2.0) to 3000^2 (0.8-1.0)
// A call of one step has no second step to share a tile's loads: marching / deep
// times of such calls were 0.88-0.92 for two fields in FP64 with reductions at 1024^2
// to 3000^2 (1.15 at 515 x 389); 0.91 for Allen-Cahn r = 2 and Cahn-Hilliard r = 1 in
// FP32 and Cahn-Hilliard r = 2 in FP64 at 1700^2 (1.2-1.4 at 1024^2); 0.91 for two
// fields in FP32 with r = 2 at 6000^2 (1.03 at 3000^2); 0.98 or more elsewhere.
int64_t deep2d_most_sites(const Launch &L, bool red, int64_t steps)
{
    constexpr int64_t M = 1000000, all = INT64_MAX;
    const bool two = L.kind == kGS || L.kind == kMC;
    if (steps == 1) {
        if (red && two && !L.fp32) return M / 2;
        if (!red && two && L.fp32 && L.r == 2) return 9 * M;
        if (!red && (L.fp32 ? (L.kind == kAC && L.r == 2) || (L.kind == kCH && L.r == 1) : L.kind == kCH && L.r == 2))
            return 3 * M / 2;
    }
    if (!red) {
        if (L.r == 1) return all;
        if (L.kind == kAC) return L.fp32 ? 6 * M : all;
        return two ? 36 * M : 3 * M;
    }
    if (L.r == 1) return L.fp32 ? 7 * M : L.kind == kGS ? all : 9 * M;
    return two && !L.fp32 ? 2 * M : 7 * M / 2;
}

// Whole-chip time of a step: its waves' instructions over 1024 SIMDs, half as much
// again for the barriers, and the tiles' loads at 2.4 TB/s (six requests of 3000^2,
// estimated / measured us per step: Allen-Cahn p2 FP32 49 / 50, Gray-Scott p2 FP64
// 181 / 184, Allen-Cahn p4 FP64 156 / 184).
bool plan_deep2d_served(const Launch &L, int64_t nx, int64_t ny, Deep3Args *a, int32_t *tiles, double *work_us)
{
    bool ok = false;
    dispatch_prec(L.fp32, [&](auto tz) {
        using T = decltype(tz);
        dispatch_kind(L.kind, [&](auto kc) {
            constexpr int KIND = decltype(kc)::value;
            dispatch_r(L.r, DeepRadii{}, [&](auto rc) {
                constexpr int R = decltype(rc)::value;
                using Tile = DeepServed<T, KIND, R>;
                using D = DeepShape<T, KIND, R, Tile::W, Tile::LR>;
                const int S = deep_served_steps(KIND, R), h = S * D::HS, TY = Tile::NWM * Tile::LR;
                const int hx = nx == D::TX ? 0 : h, hy = ny == TY ? 0 : h;
                const int64_t tx = cdiv(nx, D::TX - 2 * hx), ty = cdiv(ny, TY - 2 * hy);
                if (tx * ty > (1 << 24)) return;
                *a = Deep3Args{S, hx, hy, 0, (int32_t)cdiv(nx, tx), (int32_t)cdiv(ny, ty), 1, (int32_t)tx, (int32_t)ty};
                *tiles = (int32_t)(tx * ty);
                *work_us = (double)*tiles * (1.5 * Tile::NWM * Tile::LR * Tile::W * ops_per_site(KIND, R, L.fp32, false) *
                                                 4 / 2400.0 / (4 * kCUs) +
                                             (double)D::TX * TY * sizeof(T) * D::NF / 2.4e6 / S);
                ok = true;
            });
        });
    });
    return ok;
}

hipError_t launch_deep2d(const Launch &L, const void *args, const DeepPlan &plan, int32_t steps, bool red,
                         hipStream_t s)
{
    hipError_t err = hipErrorInvalidValue;
    if (steps < 1 || steps > plan.steps || plan.tiles < 1) return err;
    DeepPlan p = plan;
    p.args.steps = steps;
    dispatch_prec(L.fp32, [&](auto tz) {
        using T = decltype(tz);
        dispatch_kind(L.kind, [&](auto kc) {
            err = launch_deep2d_kind<T, decltype(kc)::value>(L, *static_cast<const StepArgs<T> *>(args), p, red, s);
        });
    });
    return err;
}

}  // namespace pf

// Fourier transforms of the spectral step on grids whose extents are powers of
// two, fused with the step's element-wise work:
//   rows:    the explicit term of a row and its real-to-complex transform
//   columns: transform along an axis; along the last one the implicit update of
//            the kept spectrum and the inverse transform follow in registers
//   rows:    complex-to-real transform into the next state
// so a 2D step moves 8 P bytes per site (P: bytes per value) in three launches
// where the library transforms and the element-wise kernels took ten launches
// and 21-27 P.
//
// A transform of length N runs on N / 16 threads of 16 values each, by Stockham
// passes of radix 16 and one of what is left, exchanged through LDS (padded by
// one value in 17: the first pass's stride of 16 values would hit one bank).  The
// inverse takes the radices in the opposite order, so the values that a forward
// transform leaves in a thread are those that the inverse starts from.
// Twiddle factors come from an FP64 table, rounded once from long double; those of
// a radix-16 pass are at most one product of two.
//
// What bounds it: on 2048^2 FP64 a kernel's values fill the registers of the chip
// once, so its loads, transforms and stores follow one another: 64 MB in 19 us
// (rows), 134 MB in 40 us (columns with the update), of which the VALU takes 5 and
// 8 us; larger grids approach the traffic (4096^2 FP64 341 us a step, 195 us of
// HBM traffic at 5.5 TB/s).  us per step before (hipFFT) / now: 512^2 30 / 21,
// 2048^2 152 / 78, 4096^2 563 / 340, 256^3 588 / 291, FP32 116 / 60, 331 / 177,
// 384 / 154.  Error against 80-bit transforms over 20 steps, now / hipFFT: 0.9 in
// FP64, 0.4-0.7 in FP32.  Spectra of whole rows, one (nx / 2 + 1) apart, made the columns
// kernel fetch every line twice (69 us on 2048^2).
#pragma once

#include "pf_device.h"

namespace pf {

template <typename T>
struct Cx {
    T x, y;
};
template <typename T>
__device__ __forceinline__ Cx<T> operator+(Cx<T> a, Cx<T> b) { return {a.x + b.x, a.y + b.y}; }
template <typename T>
__device__ __forceinline__ Cx<T> operator-(Cx<T> a, Cx<T> b) { return {a.x - b.x, a.y - b.y}; }
template <typename T>
__device__ __forceinline__ Cx<T> cmul(Cx<T> a, Cx<T> b)
{
    return {fma(a.x, b.x, -(a.y * b.y)), fma(a.x, b.y, a.y * b.x)};
}
// FP32 value times an FP64 factor, rounded once (FP64 multiply-adds issue at the
// FP32 rate): with FP32 factors and products the error against 80-bit transforms
// was 1.1-1.4 of hipFFT's.
__device__ __forceinline__ Cx<float> cmul(Cx<float> a, Cx<double> b)
{
    const double x = (double)a.x, y = (double)a.y;
    return {(float)fma(x, b.x, -(y * b.y)), (float)fma(x, b.y, y * b.x)};
}
// a times -i (forward) or +i (inverse)
template <bool INV, typename T>
__device__ __forceinline__ Cx<T> rot90(Cx<T> a)
{
    return INV ? Cx<T>{-a.y, a.x} : Cx<T>{a.y, -a.x};
}
// a times exp(-+ 2 pi i k / 16)
template <bool INV, int K, typename T>
__device__ __forceinline__ Cx<T> mul16(Cx<T> a)
{
    constexpr double c[5] = {1.0, 0.92387953251128675613, 0.70710678118654752440, 0.38268343236508977173, 0.0};
    if constexpr (K == 0) return a;
    else if constexpr (K == 4) return rot90<INV>(a);
    else if constexpr (K > 4) return rot90<INV>(mul16<INV, K - 4>(a));
    else if constexpr (K == 2) {
        const T h = (T)c[2];
        return INV ? Cx<T>{(a.x - a.y) * h, (a.x + a.y) * h} : Cx<T>{(a.x + a.y) * h, (a.y - a.x) * h};
    } else {
        return cmul(a, Cx<double>{c[K], INV ? c[4 - K] : -c[4 - K]});
    }
}
template <bool INV, typename T>
__device__ __forceinline__ void dft2(Cx<T> &a, Cx<T> &b)
{
    const Cx<T> t = a - b;
    a = a + b;
    b = t;
}
template <bool INV, typename T>
__device__ __forceinline__ void dft4(Cx<T> &a, Cx<T> &b, Cx<T> &c, Cx<T> &d)
{
    const Cx<T> p = a + c, q = a - c, r = b + d, s = rot90<INV>(b - d);
    a = p + r;
    b = q + s;
    c = p - r;
    d = q - s;
}
// Transform of R consecutive values in place (natural order in and out).
template <bool INV, int R, typename T>
__device__ __forceinline__ void dft(Cx<T> *v)
{
    if constexpr (R == 2) {
        dft2<INV>(v[0], v[1]);
    } else if constexpr (R == 4) {
        dft4<INV>(v[0], v[1], v[2], v[3]);
    } else {
        // R = 4 A: transforms of length 4 over the residues mod A, twiddles, then of length A
        constexpr int A = R / 4;
        static_for<0, A>([&](auto ac) {
            constexpr int a = decltype(ac)::value;
            dft4<INV>(v[a], v[a + A], v[a + 2 * A], v[a + 3 * A]);
            v[a + A] = mul16<INV, a * 16 / R>(v[a + A]);
            v[a + 2 * A] = mul16<INV, 2 * a * 16 / R>(v[a + 2 * A]);
            v[a + 3 * A] = mul16<INV, 3 * a * 16 / R>(v[a + 3 * A]);
        });
        Cx<T> o[R];
        static_for<0, 4>([&](auto kc) {
            constexpr int k = decltype(kc)::value;
            Cx<T> w[A];
            static_for<0, A>([&](auto ac) { w[decltype(ac)::value] = v[decltype(ac)::value + k * A]; });
            dft<INV, A>(w);
            static_for<0, A>([&](auto ac) { o[k + 4 * decltype(ac)::value] = w[decltype(ac)::value]; });
        });
        static_for<0, R>([&](auto ic) { v[decltype(ic)::value] = o[decltype(ic)::value]; });
    }
}

constexpr int kE = 16;  // values per thread

// Passes of a length-N transform: radix 16 as often as it goes, then the rest;
// REV: the rest first.
template <int N, bool REV>
struct Passes {
    static constexpr int full = N >= 4096 ? 3 : N >= 256 ? 2 : 1;
    static constexpr int rest = N / (full == 3 ? 4096 : full == 2 ? 256 : 16);
    static constexpr int count = full + (rest > 1 ? 1 : 0);
    template <int P>
    static constexpr int radix()
    {
        if (rest == 1) return 16;
        return REV ? (P == 0 ? rest : 16) : (P < full ? 16 : rest);
    }
    template <int P>
    static constexpr int before()  // product of the radices of the passes before P
    {
        if constexpr (P == 0)
            return 1;
        else
            return before<P - 1>() * radix<P - 1>();
    }
    static_assert(rest == 1 || rest == 2 || rest == 4 || rest == 8, "a power of two from 32 to 4096");
};

__device__ __forceinline__ constexpr int fft_pad(int i) { return i + (i >> 4); }

// Twiddle factors of a pass, loaded ahead of the exchange before it, of each of
// the thread's transforms (tw[k tws] = exp(-2 pi i k / N)): w, w^2, w^3, then w^4,
// w^8, w^12; the others are products of two.
template <int N, bool REV, int P>
struct PassTw {
    using Ps = Passes<N, REV>;
    static constexpr int R = Ps::template radix<P>(), NS = Ps::template before<P>(), Q = kE / R;
    static constexpr int NW = NS == 1 ? 0 : R == 2 ? 1 : R == 4 ? 3 : R == 8 ? 4 : 6;
    Cx<double> w[Q][NW > 0 ? NW : 1];
    __device__ __forceinline__ void load(int t, const Cx<double> *__restrict__ tw, int tws)
    {
        static_for<0, Q>([&](auto qc) {
            constexpr int q = decltype(qc)::value;
            const int k = ((t + q * (N / kE)) % NS) * (N / (NS * R)) * tws;
            static_for<0, NW>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                w[q][i] = tw[k * (i < 3 ? i + 1 : 4 * (i - 2))];
            });
        });
    }
};
// One pass: twiddles and radix-R transforms.
template <int N, bool INV, bool REV, int P, typename T>
__device__ __forceinline__ void fft_pass(Cx<T> (&v)[kE], const PassTw<N, REV, P> &pt)
{
    using Pt = PassTw<N, REV, P>;
    constexpr int R = Pt::R;
    static_for<0, kE / R>([&](auto qc) {
        constexpr int q = decltype(qc)::value;
        Cx<T> *x = v + q * R;
        if constexpr (Pt::NS > 1) {
            auto get = [&](int i) {
                Cx<double> w = pt.w[q][i];
                if (INV) w.y = -w.y;
                return w;
            };
            const Cx<double> w1 = get(0);
            x[1] = cmul(x[1], w1);
            if constexpr (R >= 4) {
                const Cx<double> w2 = get(1), w3 = get(2);
                x[2] = cmul(x[2], w2);
                x[3] = cmul(x[3], w3);
                static_for<1, R / 4>([&](auto mc) {
                    constexpr int m = decltype(mc)::value;
                    const Cx<double> w = get(m + 2);
                    x[4 * m] = cmul(x[4 * m], w);
                    x[4 * m + 1] = cmul(x[4 * m + 1], cmul(w, w1));
                    x[4 * m + 2] = cmul(x[4 * m + 2], cmul(w, w2));
                    x[4 * m + 3] = cmul(x[4 * m + 3], cmul(w, w3));
                });
            }
        }
        dft<INV, R>(x);
    });
}
// Index of value e of thread t: what pass P reads, and where it leaves it.
template <int N, bool REV, int P>
__device__ __forceinline__ int fft_in(int t, int e)
{
    constexpr int R = Passes<N, REV>::template radix<P>();
    return t + (e / R) * (N / kE) + (e % R) * (N / R);
}
template <int N, bool REV, int P>
__device__ __forceinline__ int fft_out(int t, int e)
{
    constexpr int R = Passes<N, REV>::template radix<P>(), NS = Passes<N, REV>::template before<P>();
    const int j = t + (e / R) * (N / kE);
    return (j / NS) * (NS * R) + j % NS + (e % R) * NS;
}
// All passes, the values loaded by fft_in of pass 0 and left by fft_out of the
// last.  at(i): place of value i in lds (one component at a time).  Every thread
// of the workgroup calls it.
template <int N, bool INV, bool REV, int P, typename T, typename F>
__device__ __forceinline__ void fft_from(Cx<T> (&v)[kE], int t, const Cx<double> *__restrict__ tw, int tws, T *lds, F &&at,
                                         const PassTw<N, REV, P> &pt)
{
    using Ps = Passes<N, REV>;
    fft_pass<N, INV, REV, P>(v, pt);
    if constexpr (P + 1 < Ps::count) {
        PassTw<N, REV, P + 1> next;
        next.load(t, tw, tws);
        __syncthreads();
        static_for<0, kE>([&](auto ec) { lds[at(fft_out<N, REV, P>(t, decltype(ec)::value))] = v[decltype(ec)::value].x; });
        __syncthreads();
        static_for<0, kE>([&](auto ec) { v[decltype(ec)::value].x = lds[at(fft_in<N, REV, P + 1>(t, decltype(ec)::value))]; });
        __syncthreads();
        static_for<0, kE>([&](auto ec) { lds[at(fft_out<N, REV, P>(t, decltype(ec)::value))] = v[decltype(ec)::value].y; });
        __syncthreads();
        static_for<0, kE>([&](auto ec) { v[decltype(ec)::value].y = lds[at(fft_in<N, REV, P + 1>(t, decltype(ec)::value))]; });
        fft_from<N, INV, REV, P + 1>(v, t, tw, tws, lds, at, next);
    }
}
template <int N, bool INV, bool REV, typename T, typename F>
__device__ __forceinline__ void fft_all(Cx<T> (&v)[kE], int t, const Cx<double> *__restrict__ tw, int tws, T *lds, F &&at)
{
    PassTw<N, REV, 0> none;  // the first pass has no twiddles
    fft_from<N, INV, REV, 0>(v, t, tw, tws, lds, at, none);
}

// Half spectra lie in groups of kCw columns (64 bytes): value (kx, y) of a plane at
// ((kx / cw) ny + y) cw + kx % cw, the columns padded to whole groups.  A group's
// columns are one contiguous block, and the rows of a rows workgroup fill whole
// lines of it.
template <typename T>
constexpr int kCw = 32 / (int)sizeof(T);

// ---------------------------------------------------------------------------
// Rows.  nx = 2 M real values as M complex ones (even + i odd): Z their
// transform, X[k] = (Z[k] + Z*[M-k]) / 2 - i w^k (Z[k] - Z*[M-k]) / 2, w =
// exp(-2 pi i / nx), and back Z[k] = (X[k] + X*[M-k]) + i w^-k (X[k] - X*[M-k]).
// A workgroup takes kRowThreads / (M / 16) rows.
template <int M>
struct RowShape {
    static constexpr int TH = M / kE;
    // four rows (two of the longest), at least a wave
    static constexpr int THREADS = TH >= 256 ? 2 * TH : TH >= 16 ? 4 * TH : 64;
    static constexpr int ROWS = THREADS / TH;
    static constexpr int LDS = M + M / 16;  // values per row
};

// op: 0 the values themselves, kAC / kCH the explicit term.
template <typename T, int M>
__global__ void __launch_bounds__((RowShape<M>::THREADS)) k_fft_rows(StepArgs<T> a, FftArgs f)
{
    using S = RowShape<M>;
    __shared__ T lds[S::ROWS * S::LDS];
    const int t = threadIdx.x % S::TH, r = threadIdx.x / S::TH;
    const int32_t ny = (int32_t)a.ny, rows = ny * (int32_t)a.nz, row = blockIdx.x * S::ROWS + r;
    const bool live = row < rows;
    const Cx<double> *tw = static_cast<const Cx<double> *>(f.twx);
    T *L = lds + r * S::LDS;
    auto at = [](int i) { return fft_pad(i); };
    Cx<T> v[kE];
    const int32_t rr = live ? row : 0;
    const T *u = a.buf[0][a.parity] + (int64_t)(rr / ny) * a.plane + (int64_t)(rr % ny) * a.pitch;
    const T c1 = (T)a.c1, c2 = (T)a.c2;
    static_for<0, kE>([&](auto ec) {
        constexpr int e = decltype(ec)::value;
        v[e] = *reinterpret_cast<const Cx<T> *>(u + 2 * fft_in<M, false, 0>(t, e));
    });
    if (f.op) {
        const bool ac = f.op == kAC;
        static_for<0, kE>([&](auto ec) {
            constexpr int e = decltype(ec)::value;
            auto g = [&](T x) {
                const T x3 = (x * x) * x;
                return ac ? c1 * x - c2 * x3 : c2 * x3 - c1 * x;
            };
            v[e] = {g(v[e].x), g(v[e].y)};
        });
    }
    fft_all<M, false, false>(v, t, tw, 2, L, at);
    // pairs k, M - k through LDS, one component at a time
    constexpr int LP = Passes<M, false>::count - 1;
    T px[kE], py[kE];  // Z[M - k] of the thread's k = t + e M / 16
    Cx<T> z[kE];
    static_for<0, 2>([&](auto cc) {
        constexpr int c = decltype(cc)::value;
        __syncthreads();
        static_for<0, kE>([&](auto ec) {
            constexpr int e = decltype(ec)::value;
            L[fft_pad(fft_out<M, false, LP>(t, e))] = c ? v[e].y : v[e].x;
        });
        __syncthreads();
        static_for<0, kE>([&](auto ec) {
            constexpr int e = decltype(ec)::value;
            const int k = t + e * S::TH;
            (c ? z[e].y : z[e].x) = L[fft_pad(k)];
            (c ? py[e] : px[e]) = L[fft_pad(k ? M - k : 0)];
        });
    });
    if (!live) return;
    Cx<T> *out = static_cast<Cx<T> *>(f.out) + (int64_t)(row / ny) * f.batch;
    const int32_t y = row % ny;
    auto place = [&](int k) { return (int64_t)((k / kCw<T>) * (int64_t)ny + y) * kCw<T> + k % kCw<T>; };
    const T half = T(0.5);
    static_for<0, kE>([&](auto ec) {
        constexpr int e = decltype(ec)::value;
        const int k = t + e * S::TH;
        const Cx<T> q{px[e], -py[e]}, s = z[e] + q, d = z[e] - q;
        const Cx<T> o = cmul(Cx<T>{d.y, -d.x}, tw[k]);  // -i w d
        out[place(k)] = {half * (s.x + o.x), half * (s.y + o.y)};
        if (k == 0) out[place(M)] = {z[e].x - z[e].y, T(0)};
    });
}

// Inverse rows: half spectra f.in into the rows of buf[0][parity ^ 1], unnormalised.
template <typename T, int M>
__global__ void __launch_bounds__((RowShape<M>::THREADS)) k_fft_rows_inv(StepArgs<T> a, FftArgs f)
{
    using S = RowShape<M>;
    __shared__ T lds[S::ROWS * S::LDS];
    const int t = threadIdx.x % S::TH, r = threadIdx.x / S::TH;
    const int32_t ny = (int32_t)a.ny, rows = ny * (int32_t)a.nz, row = blockIdx.x * S::ROWS + r;
    const bool live = row < rows;
    const Cx<double> *tw = static_cast<const Cx<double> *>(f.twx);
    const int32_t rr = live ? row : 0;
    const Cx<T> *in = static_cast<const Cx<T> *>(f.in) + (int64_t)(rr / ny) * f.batch;
    const int32_t y = rr % ny;
    auto place = [&](int k) { return (int64_t)((k / kCw<T>) * (int64_t)ny + y) * kCw<T> + k % kCw<T>; };
    Cx<T> v[kE];
    static_for<0, kE>([&](auto ec) {
        constexpr int e = decltype(ec)::value;
        const int k = fft_in<M, true, 0>(t, e);
        const Cx<T> x = in[place(k)], m = in[place(M - k)], q{m.x, -m.y}, s = x + q, d = x - q;
        Cx<double> w = tw[k];
        w.y = -w.y;
        const Cx<T> o = cmul(Cx<T>{-d.y, d.x}, w);  // i w^-k d
        v[e] = s + o;
    });
    fft_all<M, true, true>(v, t, tw, 2, lds + r * S::LDS, [](int i) { return fft_pad(i); });
    if (!live) return;
    T *o = a.buf[0][a.parity ^ 1] + (int64_t)(row / ny) * a.plane + (int64_t)(row % ny) * a.pitch;
    constexpr int LP = Passes<M, true>::count - 1;
    static_for<0, kE>([&](auto ec) {
        constexpr int e = decltype(ec)::value;
        *reinterpret_cast<Cx<T> *>(o + 2 * fft_out<M, true, LP>(t, e)) = v[e];
    });
}

// ---------------------------------------------------------------------------
// Columns: transforms of length N.  Along y (Z = false) a workgroup takes whole
// column groups, each a contiguous block, blockIdx.y the plane; along z it takes
// adjacent values of a plane, f.stride apart from plane to plane.
enum { kFftForward = 0, kFftInverse = 1, kFftUpdate = 2 };

template <typename T, int N, bool Z>
struct ColShape {
    static constexpr int TH = N / kE, CW = kCw<T>;
    // columns that lanes run over first: y a group (part of one where its threads
    // would pass 512), z as many as make 256 threads, 64 at most
    static constexpr int CL = !Z ? (CW * TH <= 512 ? CW : 512 / TH)
                                 : TH >= 128 ? 512 / TH : (256 / TH) < 64 ? (256 / TH) : 64;
    static constexpr int GROUPS = CL * TH >= 64 ? 1 : 64 / (CL * TH);  // at least a wave
    static constexpr int COLS = GROUPS * CL;
    static constexpr int THREADS = COLS * TH;
    static constexpr int LDS = (N + N / 16) * COLS;
};

template <typename T, int N, int MODE, bool Z>
__global__ void __launch_bounds__((ColShape<T, N, Z>::THREADS)) k_fft_cols(SpecArgs p, FftArgs f)
{
    using S = ColShape<T, N, Z>;
    constexpr int CL = S::CL;
    __shared__ T lds[S::LDS];
    const int c = threadIdx.x % CL, t = (threadIdx.x / CL) % S::TH, g = threadIdx.x / (CL * S::TH);
    const int64_t col = (int64_t)xcd_item(blockIdx.x, gridDim.x) * S::COLS + g * CL + c;
    const bool live = col < f.cols;
    const int64_t cc = live ? col : 0;
    const int64_t base = Z ? cc : (cc / S::CW) * ((int64_t)N * S::CW) + cc % S::CW;
    const int64_t vs = Z ? f.stride : S::CW;
    Cx<T> *x = static_cast<Cx<T> *>(f.out) + (int64_t)blockIdx.y * f.batch + base;
    const Cx<double> *tw = static_cast<const Cx<double> *>(f.tw);
    T *L = lds + g * ((N + N / 16) * CL);
    auto at = [&](int i) { return fft_pad(i) * CL + c; };
    constexpr bool REV = MODE == kFftInverse;
    constexpr int LP = Passes<N, REV>::count - 1;
    Cx<T> v[kE], u[MODE == kFftUpdate ? (N <= 1024 ? kE : 8) : 1];
    static_for<0, kE>([&](auto ec) {
        constexpr int e = decltype(ec)::value;
        v[e] = x[(int64_t)fft_in<N, REV, 0>(t, e) * vs];
    });
    Cx<T> *uh = static_cast<Cx<T> *>(p.uh) + base;
    // the kept spectrum, ahead of the transform where the registers hold both
    constexpr bool AHEAD = N <= 1024;
    if constexpr (MODE == kFftUpdate && AHEAD)
        static_for<0, kE>([&](auto ec) {
            constexpr int e = decltype(ec)::value;
            u[e] = uh[(int64_t)fft_out<N, false, LP>(t, e) * vs];
        });
    fft_all<N, MODE == kFftInverse, REV>(v, t, tw, 1, L, at);
    if constexpr (MODE == kFftUpdate) {
        // the implicit update of the kept spectrum (see SpecArgs), FP64 factors
        const int32_t ny = (int32_t)p.ny;
        const int32_t kxi = (int32_t)(Z ? (col / ((int64_t)ny * S::CW)) * S::CW + col % S::CW : col);
        const int32_t mid = Z ? (int32_t)((col / S::CW) % ny) : 0;
        const double kx = (double)kxi * p.sx;
        const double km = (double)(2 * mid <= ny ? mid : mid - ny) * p.sy;
        const double sl = Z ? p.sz : p.sy;
        const bool ac = f.op == kAC;
        static_for<0, kE>([&](auto ec) {
            constexpr int e = decltype(ec)::value;
            const int i = fft_out<N, false, LP>(t, e);
            const double kl = (double)(2 * i <= N ? i : i - N) * sl;
            const double K2 = Z ? kx * kx + km * km + kl * kl : kx * kx + kl * kl;
            // else in two parts, so that at most eight of its values are held beside v
            if constexpr (!AHEAD && e % 8 == 0)
                static_for<e, e + 8>([&](auto uc) {
                    constexpr int b = decltype(uc)::value;
                    u[b % 8] = uh[(int64_t)fft_out<N, false, LP>(t, b) * vs];
                });
            const Cx<T> us = u[AHEAD ? e : e % 8];
            Cx<T> o;
            if (ac) {
                const double q = 1.0 / (1.0 + p.dt * K2), d = p.dt * p.inv_n;
                o.x = (T)((p.u_scale * (double)us.x + d * (double)v[e].x) * q);
                o.y = (T)((p.u_scale * (double)us.y + d * (double)v[e].y) * q);
            } else {
                const double q = 1.0 / (1.0 + p.dt * K2 * K2), d = p.dt * K2 * p.inv_n;
                o.x = (T)((p.u_scale * (double)us.x - d * (double)v[e].x) * q);
                o.y = (T)((p.u_scale * (double)us.y - d * (double)v[e].y) * q);
            }
            if (live) uh[(int64_t)i * vs] = o;
            v[e] = o;
        });
        fft_all<N, true, true>(v, t, tw, 1, L, at);
        constexpr int LI = Passes<N, true>::count - 1;
        if (!live) return;
        static_for<0, kE>([&](auto ec) {
            constexpr int e = decltype(ec)::value;
            x[(int64_t)fft_out<N, true, LI>(t, e) * vs] = v[e];
        });
    } else {
        if (!live) return;
        static_for<0, kE>([&](auto ec) {
            constexpr int e = decltype(ec)::value;
            x[(int64_t)fft_out<N, REV, LP>(t, e) * vs] = v[e];
        });
    }
}

}  // namespace pf

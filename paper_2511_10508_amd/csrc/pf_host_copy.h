// Copies between caller memory (FP64, dense) and device fields through a
// small pinned buffer.  A copy straight to or from pageable memory costs 6.8 us
// a row here (2.7 ms for a 515 x 389 field, 3.5 ms for 512^2); pinned halves of
// 4 MiB, filled by one linear copy while the host converts the other, move the
// same fields in 0.2 ms.  The row padding is copied out and skipped, and is
// never written.
#pragma once

#include <algorithm>
#include <cstring>
#include <mutex>

#include <hip/hip_runtime.h>

namespace pf {

// Two pinned halves, allocated on first use (as much as a transfer needs, at
// most kHalf bytes each) and kept by their owner until release().  A transfer
// holds `mu` from ensure() to its last use of the halves: its owner's other
// threads would overwrite them, or free them to get larger ones.
struct PinnedStage {
    static constexpr size_t kHalf = 4u << 20;
    std::mutex mu;
    void *half[2] = {nullptr, nullptr};
    hipEvent_t ev[2] = {nullptr, nullptr};
    size_t bytes = 0;

    hipError_t ensure(size_t want)
    {
        want = std::min(kHalf, (want + 4095) / 4096 * 4096);
        if (want <= bytes) return hipSuccess;
        release();
        for (int i = 0; i < 2; ++i) {
            hipError_t e = hipHostMalloc(&half[i], want, hipHostMallocDefault);
            if (e == hipSuccess) e = hipEventCreateWithFlags(&ev[i], hipEventDisableTiming);
            if (e != hipSuccess) {
                release();
                return e;
            }
        }
        bytes = want;
        return hipSuccess;
    }
    void release()
    {
        for (int i = 0; i < 2; ++i) {
            if (half[i]) (void)hipHostFree(half[i]);
            if (ev[i]) (void)hipEventDestroy(ev[i]);
            half[i] = nullptr;
            ev[i] = nullptr;
        }
        bytes = 0;
    }
};

// Elements [e0, e1) of a pitched array, as runs of one row each:
// f(first element, its place among the nx columns of every row, length).
template <typename F>
inline void pitched_runs(int64_t e0, int64_t e1, int64_t nx, int64_t pitch, F &&f)
{
    if (nx == pitch) {
        f(e0, e0, e1 - e0);
        return;
    }
    for (int64_t row = e0 / pitch; row * pitch < e1; ++row) {
        const int64_t lo = std::max(e0, row * pitch), hi = std::min(e1, row * pitch + nx);
        if (lo < hi) f(lo, row * nx + (lo - row * pitch), hi - lo);
    }
}

// Device field (rows of `pitch` elements of ts = 4 or 8 bytes) to host; waits
// for `stream`.
inline hipError_t copy_field_out(PinnedStage &st, const void *dev, size_t ts, int64_t nx, int64_t rows, int64_t pitch,
                                 double *host, hipStream_t stream)
{
    std::lock_guard<std::mutex> lk(st.mu);
    const int64_t total = rows * pitch;
    hipError_t e = st.ensure((size_t)total * ts);
    const int64_t step = (int64_t)(st.bytes / ts);
    auto fetch = [&](int64_t k) {  // chunk k into half k & 1
        const int64_t at = k * step, n = std::min(step, total - at);
        e = hipMemcpyAsync(st.half[k & 1], static_cast<const char *>(dev) + (size_t)at * ts, (size_t)n * ts,
                           hipMemcpyDeviceToHost, stream);
        if (e == hipSuccess) e = hipEventRecord(st.ev[k & 1], stream);
    };
    const int64_t chunks = step > 0 ? (total + step - 1) / step : 0;
    if (e == hipSuccess) fetch(0);
    for (int64_t k = 0; k < chunks && e == hipSuccess; ++k) {
        if (k + 1 < chunks) fetch(k + 1);
        if (e == hipSuccess) e = hipEventSynchronize(st.ev[k & 1]);
        if (e != hipSuccess) break;
        const int64_t at = k * step;
        const void *src = st.half[k & 1];
        pitched_runs(at, std::min(at + step, total), nx, pitch, [&](int64_t from, int64_t to, int64_t n) {
            if (ts == 8) {
                std::memcpy(host + to, static_cast<const double *>(src) + (from - at), (size_t)n * 8);
            } else {
                const float *s = static_cast<const float *>(src) + (from - at);
                for (int64_t i = 0; i < n; ++i) host[to + i] = (double)s[i];
            }
        });
    }
    if (e != hipSuccess) (void)hipStreamSynchronize(stream);  // nothing may still write the halves
    return e;
}

// Host to device field (FP32 storage rounds to nearest); waits for `stream`.
inline hipError_t copy_field_in(PinnedStage &st, void *dev, size_t ts, int64_t nx, int64_t rows, int64_t pitch,
                                const double *host, hipStream_t stream)
{
    std::lock_guard<std::mutex> lk(st.mu);
    const int64_t total = nx * rows;  // dense elements
    hipError_t e = st.ensure((size_t)total * ts);
    if (e != hipSuccess) return e;
    // padded rows go by whole rows where a half holds one, else by parts of a row
    int64_t step = (int64_t)(st.bytes / ts);
    if (nx != pitch && step > nx) step = step / nx * nx;
    int64_t at = 0;
    for (int64_t k = 0; at < total && e == hipSuccess; ++k) {
        int64_t n = std::min(step, total - at);
        if (nx != pitch && step < nx) n = std::min(n, nx - at % nx);
        void *half = st.half[k & 1];
        if (k >= 2) e = hipEventSynchronize(st.ev[k & 1]);
        if (e != hipSuccess) break;
        if (ts == 8) {
            std::memcpy(half, host + at, (size_t)n * 8);
        } else {
            float *d = static_cast<float *>(half);
            for (int64_t i = 0; i < n; ++i) d[i] = (float)host[at + i];
        }
        char *to = static_cast<char *>(dev) + (size_t)(at / nx * pitch + at % nx) * ts;
        if (nx == pitch || n < nx)
            e = hipMemcpyAsync(to, half, (size_t)n * ts, hipMemcpyHostToDevice, stream);
        else
            e = hipMemcpy2DAsync(to, ts * (size_t)pitch, half, ts * (size_t)nx, ts * (size_t)nx, (size_t)(n / nx),
                                 hipMemcpyHostToDevice, stream);
        if (e == hipSuccess) e = hipEventRecord(st.ev[k & 1], stream);
        at += n;
    }
    const hipError_t s = hipStreamSynchronize(stream);
    return e != hipSuccess ? e : s;
}

}  // namespace pf

// Two threads per direction through one pinned stage (csrc/pf_host_copy.h) on
// the fake executor (fake_device.cpp): fields of different sizes, so that one
// transfer makes the halves grow while another uses them.  Every value is
// checked; the process exits non-zero on any mismatch.
#include <cstdio>
#include <thread>
#include <vector>

#include "../../paper_2511_10508_amd/csrc/pf_host_copy.h"

namespace {

struct Field {
    int64_t nx, rows, pitch;
    std::vector<double> dev, host;

    Field(int64_t nx_, int64_t rows_, int64_t pitch_, double base)
        : nx(nx_), rows(rows_), pitch(pitch_), dev((size_t)(rows_ * pitch_), -1.0), host((size_t)(nx_ * rows_))
    {
        for (int64_t i = 0; i < nx * rows; ++i) host[i] = base + (double)i;
        for (int64_t y = 0; y < rows; ++y)
            for (int64_t x = 0; x < nx; ++x) dev[y * pitch + x] = host[y * nx + x];
    }
};

}  // namespace

int main()
{
    pf::PinnedStage st;
    hipStream_t stream = nullptr;
    if (hipStreamCreateWithFlags(&stream, hipStreamNonBlocking) != hipSuccess) return 2;
    int bad[3] = {0, 0, 0};
    auto reader = [&](int id, Field f) {
        std::vector<double> out(f.host.size());
        for (int rep = 0; rep < 20; ++rep) {
            std::fill(out.begin(), out.end(), 0.0);
            if (pf::copy_field_out(st, f.dev.data(), 8, f.nx, f.rows, f.pitch, out.data(), stream) != hipSuccess) bad[id]++;
            if (out != f.host) bad[id]++;
        }
    };
    auto writer = [&](int id, Field f) {
        for (int rep = 0; rep < 20; ++rep) {
            std::vector<double> to(f.dev.size(), -1.0);
            if (pf::copy_field_in(st, to.data(), 8, f.nx, f.rows, f.pitch, f.host.data(), stream) != hipSuccess) bad[id]++;
            if (to != f.dev) bad[id]++;
        }
    };
    std::thread a(reader, 0, Field(61, 40, 64, 1e6)), b(reader, 1, Field(1000, 1100, 1000, 2e6)),
        c(writer, 2, Field(333, 700, 336, 3e6));
    a.join();
    b.join();
    c.join();
    st.release();
    (void)hipStreamDestroy(stream);
    if (bad[0] + bad[1] + bad[2]) {
        std::fprintf(stderr, "wrong transfers: %d %d %d\n", bad[0], bad[1], bad[2]);
        return 1;
    }
    std::printf("host_copy_threads: ok\n");
    return 0;
}

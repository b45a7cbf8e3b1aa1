// Allocation failures of the serving scheduler's tables (csrc/serve.cpp) on the
// fake executor (fake_device.cpp), by the linker's --wrap: whichever allocation of
// a class or of its tuning table fails, nothing is left allocated and a later
// attempt succeeds.  Exits non-zero on a mismatch.
#include "../../paper_2511_10508_amd/csrc/serve.cpp"

#include <cstdio>

static int g_fail_at = 0, g_calls = 0, g_live = 0;

extern "C" {
hipError_t __real_hipMalloc(void **p, size_t n);
hipError_t __real_hipFree(void *p);
hipError_t __real_hipHostMalloc(void **p, size_t n, unsigned int f);
hipError_t __real_hipHostFree(void *p);
static bool failing() { return g_fail_at && ++g_calls == g_fail_at; }
hipError_t __wrap_hipMalloc(void **p, size_t n)
{
    if (failing()) return hipErrorOutOfMemory;
    g_live++;
    return __real_hipMalloc(p, n);
}
hipError_t __wrap_hipFree(void *p)
{
    g_live -= p != nullptr;
    return __real_hipFree(p);
}
hipError_t __wrap_hipHostMalloc(void **p, size_t n, unsigned int f)
{
    if (failing()) return hipErrorOutOfMemory;
    g_live++;
    return __real_hipHostMalloc(p, n, f);
}
hipError_t __wrap_hipHostFree(void *p)
{
    g_live -= p != nullptr;
    return __real_hipHostFree(p);
}
}

namespace pf {

static int run()
{
    Server s;
    s.max_slots = 4;
    (void)hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking);
    (void)hipEventCreate(&s.tev[0]);
    (void)hipEventCreate(&s.tev[1]);
    pf_desc d;
    std::memset(&d, 0, sizeof d);
    d.struct_size = sizeof(pf_desc);
    d.kind = PF_AC;
    d.nfields = 1;
    d.ndim = 2;
    d.n[0] = d.n[1] = 100;
    d.n[2] = 1;
    d.dx = 1.0;
    d.dt = 0.01;
    d.order = 4;
    Req r;
    r.desc = d;
    if (model_create(&d, s.stream, nullptr, 0, &r.m, true) != PF_OK) return 2;
    int bad = 0;
    auto expect = [&](bool ok, const char *what, int k) {
        if (!ok) {
            std::fprintf(stderr, "%s, allocation %d: %d live\n", what, k, g_live);
            bad = 1;
        }
    };
    for (int k = 1; k <= 4; ++k) {
        g_fail_at = k, g_calls = 0;
        expect(class_of(&s, r.m) == -1 && g_live == 0, "class", k);
    }
    g_fail_at = 0;
    r.cls = class_of(&s, r.m);
    expect(r.cls == 0 && g_live == 4, "class", 0);
    for (int k = 1; k <= 2; ++k) {
        g_fail_at = k, g_calls = 0;
        s.tuned.clear();
        tune_served(&s, &r);
        expect(g_live == 4, "tuning table", k);
    }
    g_fail_at = 0;
    s.tuned.clear();
    tune_served(&s, &r);
    expect(g_live == 6 && r.march_us > 0.0, "tuning table", 0);
    (void)hipStreamSynchronize(s.stream);
    return bad;
}

}  // namespace pf

int main()
{
    if (pf::run()) return 1;
    std::printf("serve_nomem: ok\n");
    return 0;
}

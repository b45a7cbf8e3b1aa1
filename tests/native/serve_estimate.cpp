// Estimated times of the serving scheduler (csrc/serve.cpp) on the fake executor
// (fake_device.cpp), whose launches all take the same time: a request of a tuned
// size bucket gets the time measured on another grid of the bucket in proportion
// to its own work, one that was never tuned a time that grows with its bytes.
// Exits non-zero on a mismatch.
#include "../../paper_2511_10508_amd/csrc/serve.cpp"

#include <cmath>
#include <cstdio>

namespace pf {

static Req *request(Server *s, int64_t nx, int64_t ny)
{
    Req *r = new Req();
    std::memset(&r->desc, 0, sizeof r->desc);
    r->desc.struct_size = sizeof(pf_desc);
    r->desc.kind = PF_AC;
    r->desc.nfields = 1;
    r->desc.ndim = 2;
    r->desc.n[0] = nx;
    r->desc.n[1] = ny;
    r->desc.n[2] = 1;
    r->desc.dx = 1.0;
    r->desc.dt = 0.01;
    r->desc.order = 4;
    r->desc.precision = PF_FP32;
    if (model_create(&r->desc, s->stream, nullptr, 0, &r->m, true) != PF_OK) std::exit(2);
    r->cls = class_of(s, r->m);
    tune_served(s, r);
    return r;
}

static int run()
{
    int bad = 0;
    auto expect = [&](const char *what, double got, double want) {
        if (!(std::fabs(got - want) <= 0.02 * want)) {
            std::fprintf(stderr, "%s: %g, not %g\n", what, got, want);
            bad = 1;
        }
    };
    {
        Server s;
        s.max_slots = 4;
        (void)hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking);
        (void)hipEventCreate(&s.tev[0]);
        (void)hipEventCreate(&s.tev[1]);
        Req *a = request(&s, 2048, 2048), *b = request(&s, 4000, 4000);
        expect("four times the work of the measured grid", b->march_us, a->march_us * b->m->items / a->m->items);
        Req *c = request(&s, 100, 100), *d = request(&s, 120, 120);
        expect("both less than the chip holds", d->march_us, c->march_us);
    }
    {
        Server s;
        s.tune = false;
        s.max_slots = 4;
        (void)hipStreamCreateWithFlags(&s.stream, hipStreamNonBlocking);
        Req *a = request(&s, 100, 100), *b = request(&s, 4000, 4000);
        if (!(b->march_us > a->march_us)) {
            std::fprintf(stderr, "not tuned: %g %g\n", a->march_us, b->march_us);
            bad = 1;
        }
    }
    return bad;
}

}  // namespace pf

int main()
{
    if (pf::run()) return 1;
    std::printf("serve_estimate: ok\n");
    return 0;
}

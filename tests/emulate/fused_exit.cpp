// A fused sweep's first kernel computes the last sweep's slide in every block, and block 0 publishes
// it, the end of the sample included, while other blocks may not have started or may be between any
// two of their waves' instructions. What the others do must not depend on when that happens.
//
// A sample's first two launches, the one that ends it and those after it are run with block 1
// stopped before each of its runs of a wave in turn while block 0 runs from start to end; every one
// of them has to leave the memory the launch leaves with the blocks one after another, and no block
// may be left by some of its waves alone.
#include <math.h>

#include "pa_internal.h"

using namespace pa;

namespace {

struct Arena {
    std::vector<char> mem = std::vector<char>(1u << 20);
    size_t used = 0;
    template <class T>
    T* get(size_t n) {
        used = (used + 255) / 256 * 256;
        T* p = reinterpret_cast<T*>(reinterpret_cast<char*>(((uintptr_t)mem.data() + 255) / 256 * 256) + used);
        used += n * sizeof(T);
        if (used + 512 > mem.size()) abort();
        return p;
    }
};

int failures = 0;
void expect(bool ok, const char* what, int launch, int step) {
    if (ok) return;
    ++failures;
    printf("FAILED: %s: launch %d, block 0 before run %d of block 1\n", what, launch, step);
}

Dev sampler(Arena& a, int C, int H, int W, int T, int P) {
    Dev d{};
    d.N = 1;
    d.T = T;
    d.P = P;
    d.C = C;
    d.Himg = H;
    d.Wimg = W;
    d.D = C * H * W;
    d.delta = 0.05;
    d.tol = 1e-3;
    d.revisit_thr = 0.05;
    d.picard_blocks = picard_blocks(d.D, P);
    d.X = a.get<float>((size_t)(T + 1) * d.D);
    d.Xh = a.get<float>((size_t)T * d.D);
    d.Eh = a.get<float>((size_t)T * d.D);
    d.valid = a.get<uint8_t>(T);
    d.coef = a.get<double>(3 * T);
    d.ctrl = a.get<Ctrl>(1);
    d.progress = a.get<uint64_t>(1);
    d.counters = a.get<uint64_t>(4);
    d.epoch = 1;
    for (int i = 0; i < d.D; ++i) d.X[i] = sinf(0.37f * i);
    for (int t = 0; t < T; ++t) {
        d.coef[3 * t] = 0.02 + 0.01 * t;
        d.coef[3 * t + 1] = -0.2;
    }
    return d;
}

bool done(const Dev& d) { return (*d.progress >> 31) & 1u; }

// Runs the launch on the memory as it is, then again from there for every place of block 0.
void in_every_order(const char* what, Arena& a, int index, const std::function<bool()>& ended,
                    const std::function<void()>& launch) {
    const std::vector<char> before = a.mem;
    emu::uneven = 0;
    launch();
    expect(emu::uneven == 0, what, index, -1);
    const std::vector<char> after = a.mem;
    int steps = 0;
    for (int k = 0; index < 2 || ended(); ++k) {
        memcpy(a.mem.data(), before.data(), before.size());
        emu::hook.block = 1;
        emu::hook.step = k;
        emu::hook.reached = false;
        emu::uneven = 0;
        launch();
        emu::hook.block = -1;
        if (!emu::hook.reached) break;
        ++steps;
        expect(emu::uneven == 0, what, index, k);
        expect(memcmp(a.mem.data(), after.data(), after.size()) == 0, what, index, k);
    }
    memcpy(a.mem.data(), after.data(), after.size());
    if (steps < 2 && (index < 2 || ended())) abort();
}

void linear(int T, int P) {
    Arena a, b;
    Dev d = sampler(a, 2, 8, 8, T, P), e = sampler(b, 2, 8, 8, T, P);
    for (auto [q, m] : {std::pair<Dev*, Arena*>{&d, &a}, {&e, &b}}) {
        q->lin_c = m->get<float>(T);
        for (int t = 0; t < T; ++t) q->lin_c[t] = 0.5f + 0.1f * t;
    }
    // one launch per sweep, and two launches after the one that ends the sample
    d.fused_linear = 1;
    d.part_res = a.get<double>((size_t)2 * P * d.picard_blocks);
    d.part_dev = a.get<double>((size_t)2 * P * d.picard_blocks);
    d.pre = a.get<SlidePre>(2);
    launch_reset(d, nullptr);
    int launches = 0;
    for (int past = 0; past < 3; past += done(d)) {
        ++d.sweep_id;
        in_every_order("linear sweep", a, launches++, [&] { return done(d); },
                       [&] { launch_picard(d, nullptr, 1, nullptr, nullptr, launches > 1); });
        if (launches > 4 * T) abort();
    }
    // a slide launch per sweep
    e.part_rows = b.get<double>((size_t)2 * P * e.picard_blocks);
    launch_reset(e, nullptr);
    int sweeps = 0;
    for (; !e.ctrl->done; ++sweeps) {
        launch_picard(e, nullptr, 1, nullptr, nullptr, 0);
        launch_slide(e, nullptr, nullptr, nullptr);
    }
    const size_t row = d.D * sizeof(float);
    expect(d.ctrl->done && memcmp(d.X, e.X, (T + 1) * row) == 0 && memcmp(d.Xh, e.Xh, T * row) == 0 &&
               memcmp(d.Eh, e.Eh, T * row) == 0 && memcmp(d.counters, e.counters, 32) == 0 &&
               *d.progress == *e.progress && sweeps == (int)(*d.progress >> 32) && launches == sweeps + 3,
           "linear sample against a slide launch per sweep", launches, -1);
    printf("linear T %d P %d: %d launches ok\n", T, P, launches);
}

// The network launch that ends a sample and the ones after it (no misses, so no network).
void network(int hidden) {
    Arena a;
    const int T = 2, P = 2;
    Dev d = sampler(a, 4, 16, 32, T, P);
    d.tol = INFINITY;
    d.hidden = hidden;
    d.ntok = (d.Himg / 2) * (d.Wimg / 2);
    d.nsplit = mlp_splits(hidden);
    d.mlp_grid = 2;
    d.fine_rows = 1;
    d.Ep = a.get<float>((size_t)d.nsplit * P * d.D);
    d.part_res = a.get<double>((size_t)P * d.picard_blocks);
    d.part_dev = a.get<double>((size_t)P * d.picard_blocks);
    d.pre = a.get<SlidePre>(2);
    d.eps_mode = a.get<int32_t>(2);
    d.whole_ok = 1;
    d.fused_slide = 1;
    launch_reset(d, nullptr);
    ++d.sweep_id;
    launch_picard(d, nullptr, 0, nullptr, nullptr, 0);     // outputs of zero, in Ep
    int launches = 0;
    for (int k = 0; k < 3; ++k) {
        ++d.sweep_id;
        in_every_order("network launch", a, launches++, [&] { return done(d); },
                       [&] { launch_eps_mlp(d, nullptr, nullptr, nullptr, 0); });
        expect(done(d) && d.ctrl->done, "network launch: end of the sample", launches, -1);
        launch_picard(d, nullptr, 0, nullptr, nullptr, 0);
    }
    printf("network H %d: %d launches ok\n", hidden, launches);
}

}  // namespace

int main() {
    linear(9, 4);       // 16 rows of one slot
    linear(18, 18);     // 16 rows of two
    linear(34, 34);     // 32 rows of two (512 threads)
    network(512);
    network(1024);
    if (failures) return 1;
    printf("fused exit ok\n");
    return 0;
}

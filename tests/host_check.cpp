// Host-side checks of the library over a stand-in HIP runtime (fake_hip.hpp, no GPU use).  host_check NAME runs one
// check; exit status 0 only if it holds.
#include "fake_hip.hpp"

#include "bubbly.h"

static int failures = 0;
#define CHECK(cond, ...)                       \
    do {                                       \
        if (!(cond)) {                         \
            std::printf("%s: ", #cond);        \
            std::printf(__VA_ARGS__);          \
            std::printf("\n");                 \
            ++failures;                        \
        }                                      \
    } while (0)

struct Problem {
    bub_grid grid{};
    bub_liquid liq{7.1, 3.06e8, 1000.0, 101325.0};
    bub_gas gas{1.4, 0.0728, 1e-3, 0.0};
    bub_bins bins{5, 10e-6, 0.3};
    bub_opts opts{};
    Problem(int ndim, int nx, int ny, int nz, int nb)
    {
        grid.ndim = ndim;
        const int n[3] = {nx, ny, nz};
        for (int d = 0; d < 3; ++d) grid.n[d] = n[d], grid.dx[d] = 1e-4;
        bins.nb = nb;
        opts.cfl = 0.3;
        opts.sub_rtol = 1e-4;
        opts.max_substeps = 1000;
        opts.transfer = {1.4, 287.06, 461.52, 293.15, 0.0257, 2.42e-5, 5.0, 5.0};
    }
    Problem &kappa(double k) { return gas.kappa = k, *this; }
    Problem &mixed() { return opts.precision = BUB_PREC_MIXED, *this; }
    Problem &split() { return opts.bubble_mode = BUB_BUBBLES_SPLIT, *this; }
    Problem &viscous() { return opts.viscous = 1, *this; }
    Problem &transfer() { return opts.contents = BUB_CONTENTS_TRANSFER, *this; }
    bub_ctx *make() const
    {
        bub_ctx *c = nullptr;
        const int rc = bub_ctx_create(&grid, &liq, &gas, &bins, &opts, &c);
        CHECK(rc == BUB_OK, "bub_ctx_create: %d", rc);
        return c;
    }
};

static double *pretend(size_t at) { return (double *)(at << 40); }   // a device address that nothing reads

// A batch charges a member the device bytes that it holds: state, work, and what its context allocated.
static void budget()
{
    Problem all[] = {Problem(2, 200, 200, 1, 5), Problem(2, 200, 200, 1, 1), Problem(3, 40, 40, 40, 11), Problem(1, 400, 1, 1, 11),
                     Problem(2, 70, 37, 1, 5), Problem(2, 800, 700, 1, 3), Problem(2, 200, 200, 1, 5).kappa(5.0 / 3.0),
                     Problem(2, 300, 200, 1, 5).transfer()};
    for (const Problem &p : all) {
        const size_t before = fake().held();
        bub_ctx *c = p.make();
        const size_t ctx = fake().held() - before;
        size_t sb;
        bub_layout(c, nullptr, nullptr, nullptr, &sb, nullptr);
        const size_t need = 3 * sb + ctx;
        int slot;
        for (int fits = 0; fits < 2; ++fits) {   // (the parts of a context's buffers are counted in units of 256)
            bub_batch *b = nullptr;
            CHECK(bub_batch_create(BUB_PREC_FP64, 2, fits ? need + 1024 : need - 1, &b) == BUB_OK, "batch");
            const int rc = bub_batch_add(b, c, pretend(1), pretend(2), 1, &slot);
            CHECK(rc == (fits ? BUB_OK : BUB_ENOMEM), "%dD %d x %d x %d, %d bins, kappa %g: %d (holds %zu)", p.grid.ndim,
                  p.grid.n[0], p.grid.n[1], p.grid.n[2], p.bins.nb, p.gas.kappa, rc, need);
            bub_batch_destroy(b);
        }
        bub_ctx_destroy(c);
    }
}

// Where the device has room for one primitive scratch but not for two, a context runs with one; a failed attempt leaves
// no error behind for the launches that follow.
static void scratch()
{
    Problem all[] = {Problem(2, 200, 200, 1, 5), Problem(3, 40, 40, 40, 11), Problem(2, 800, 700, 1, 3), Problem(2, 30, 20, 1, 1)};
    for (const Problem &p : all) {
        const size_t one = 8 * (size_t)(p.grid.ndim + 6) * p.grid.n[0] * p.grid.n[1] * p.grid.n[2];
        fake().limit = one + 4096 > 16384 ? one + 4096 : 16384;
        bub_ctx *c = p.make();
        if (c) {
            CHECK(bub_rk3_steps(c, pretend(1), pretend(2), 2, 0.0, nullptr, nullptr) == BUB_OK, "steps");
            bub_ctx_destroy(c);
        }
        fake().limit = one / 2;   // not even one
        bub_ctx *none = nullptr;
        if (one / 2 > 16384)
            CHECK(bub_ctx_create(&p.grid, &p.liq, &p.gas, &p.bins, &p.opts, &none) == BUB_ENOMEM && !none, "no room");
        CHECK(fake().mem.empty(), "%zu bytes left behind", fake().held());
        fake().limit = ~(size_t)0;
        bub_ctx *c2 = p.make();
        CHECK(bub_rk3_steps(c2, pretend(1), pretend(2), 2, 0.0, nullptr, nullptr) == BUB_OK, "steps after a refusal");
        bub_ctx_destroy(c2);
    }
}

// A second scratch is held only where a stage can ever use it.
static void unused()
{
    struct { Problem p; int scratches; } all[] = {
        {Problem(2, 200, 200, 1, 5), 2}, {Problem(2, 200, 200, 1, 5).split(), 2}, {Problem(3, 40, 40, 40, 11), 2},
        {Problem(3, 40, 40, 40, 11).mixed().split(), 2}, {Problem(2, 200, 200, 1, 5).transfer(), 2},
        {Problem(2, 800, 700, 1, 3).kappa(5.0 / 3.0), 2}, {Problem(1, 600000, 1, 1, 3), 2}, {Problem(3, 90, 90, 90, 3).mixed(), 2},
        {Problem(1, 4000, 1, 1, 11), 1}, {Problem(2, 100, 100, 1, 5), 1},
        {Problem(2, 200, 200, 1, 5).kappa(5.0 / 3.0), 1},   // no tile kernel below 2^19 cells
        {Problem(2, 200, 200, 1, 5).kappa(1.35), 1}, {Problem(2, 800, 700, 1, 3).kappa(1.35), 1},
        {Problem(2, 200, 200, 1, 5).viscous(), 1}, {Problem(2, 800, 700, 1, 3).viscous(), 1}, {Problem(1, 4000, 1, 1, 1).viscous(), 1},
        {Problem(3, 40, 40, 40, 11).mixed(), 1}, {Problem(3, 40, 40, 40, 11).transfer(), 1},
    };
    for (auto &a : all) {
        const size_t before = fake().held();
        bub_ctx *c = a.p.make();
        const size_t one = 8 * (size_t)(a.p.grid.ndim + 6) * a.p.grid.n[0] * a.p.grid.n[1] * a.p.grid.n[2];
        const double held = (double)(fake().held() - before) / one;   // (and some 11 KB of tables)
        CHECK((int)(held + 0.01) == a.scratches, "%dD %d x %d x %d, kappa %g: holds %g scratches, not %d", a.p.grid.ndim,
              a.p.grid.n[0], a.p.grid.n[1], a.p.grid.n[2], a.p.gas.kappa, held, a.scratches);
        bub_ctx_destroy(c);
    }
}

// The tile-shape cache keeps polytropic air, whose shapes have kernels of their own, apart from other gases: a hit is a
// shape that the context runs and reports.  (The stand-in clock makes the last shape that is timed the fastest.)
static void cache()
{
    auto put = [](const char *text) {
        std::FILE *f = std::fopen("tiles.txt", "w");
        std::fputs(text, f);
        std::fclose(f);
    };
    auto tuned = [](const Problem &p, int want_hit, int want) {
        bub_ctx *c = p.make();
        int best = -1, hit = -1, get = -1;
        const int rc = bub_autotune_cached(c, "tiles.txt", pretend(1), pretend(2), 1, &best, &hit, nullptr);
        bub_tile_get(c, &get);
        CHECK(rc == BUB_OK && hit == want_hit && best == want && get == want, "kappa %g: %d, hit %d, best %d, tile %d; not %d %d",
              p.gas.kappa, rc, hit, best, get, want_hit, want);
        bub_ctx_destroy(c);
    };
    const Problem air(1, 400, 1, 1, 11), other = Problem(1, 400, 1, 1, 11).kappa(5.0 / 3.0);
    put("");
    tuned(air, 0, 3);     // one wave a tile, air's only
    tuned(other, 0, 2);
    tuned(air, 1, 3);
    tuned(other, 1, 2);
    put("gfx950 1 11 0 8 1\n");   // of a file from before air had kernels of its own
    tuned(other, 1, 1);
    tuned(air, 0, 3);
    put("gfx950 1 11 0 8 3\n");   // a shape that the context cannot run
    tuned(other, 0, 2);
    const Problem air2(2, 70, 37, 1, 5), other2 = Problem(2, 70, 37, 1, 5).kappa(1.0);
    put("gfx950 2 5 0 11 0\n");
    tuned(air2, 0, 5);
    tuned(other2, 1, 0);
}

// So does the class autotuner of a batch, for members present and later ones.
static void classes()
{
    bub_batch *b = nullptr;
    CHECK(bub_batch_create(BUB_PREC_FP64, 4, 0, &b) == BUB_OK, "batch");
    const Problem ps[] = {Problem(1, 400, 1, 1, 11), Problem(1, 300, 1, 1, 11).kappa(5.0 / 3.0), Problem(1, 350, 1, 1, 11).kappa(5.0 / 3.0),
                          Problem(1, 500, 1, 1, 11)};
    const int want[] = {3, 2, 2, 3};
    bub_ctx *c[4];
    int slot, n = 0, get;
    for (int i = 0; i < 4; ++i) {
        c[i] = ps[i].make();
        CHECK(bub_batch_add(b, c[i], pretend(2 * i + 1), pretend(2 * i + 2), 0, &slot) == BUB_OK, "add");
        if (i == 1) CHECK(bub_batch_autotune(b, 1, &n, nullptr) == BUB_OK && n == 2, "%d classes", n);
    }
    for (int i = 0; i < 4; ++i) {
        bub_tile_get(c[i], &get);
        CHECK(get == want[i], "member %d: shape %d", i, get);
    }
    bub_batch_destroy(b);
    for (bub_ctx *x : c) bub_ctx_destroy(x);
}

// Every shape that is listed for a polytropic gas with a fifth-root power can be set, is reported and runs; the autotuner
// writes no more times than shapes are listed.
static void shapes()
{
    for (double kappa : {1.4, 5.0 / 3.0, 1.0, 1.35})
        for (int ndim = 1; ndim <= 3; ++ndim) {
            Problem p = ndim == 1 ? Problem(1, 400, 1, 1, 11) : ndim == 2 ? Problem(2, 70, 37, 1, 5) : Problem(3, 20, 13, 11, 3);
            bub_ctx *c = p.kappa(kappa).make();
            int n = 0;
            CHECK(bub_tile_count(c, &n) == BUB_OK, "count");
            const int want[] = {0, kappa == 1.4 ? 4 : 3, 6, 5};
            CHECK(n == want[ndim], "%dD, kappa %g: %d shapes", ndim, kappa, n);
            for (int i = 0; i < n; ++i) {
                int t[4], get = -1;
                CHECK(bub_tile_info(c, i, &t[0], &t[1], &t[2], &t[3]) == BUB_OK, "info %d", i);
                const int rc = bub_tile_set(c, i);
                if (kappa == 1.35 && i) {   // the general power has one shape
                    CHECK(rc == BUB_EUNSUPPORTED, "set %d: %d", i, rc);
                    continue;
                }
                CHECK(rc == BUB_OK && bub_tile_get(c, &get) == BUB_OK && get == i, "%dD, kappa %g: set %d: %d, then %d", ndim,
                      kappa, i, rc, get);
                CHECK(bub_rhs_stage(c, pretend(1), pretend(2), nullptr) == BUB_OK, "rhs");
                CHECK(fake().launches.back().block.x == (unsigned)t[3], "%dD, kappa %g, shape %d: %u threads, listed %d", ndim,
                      kappa, i, fake().launches.back().block.x, t[3]);
            }
            CHECK(bub_tile_set(c, n) == BUB_EINVAL, "a shape past the list");
            double ms[8] = {7, 7, 7, 7, 7, 7, 7, 7};
            CHECK(bub_autotune(c, pretend(1), pretend(2), 1, ms, nullptr, nullptr) == BUB_OK, "autotune");
            for (int i = 0; i < 8; ++i) CHECK((ms[i] != 7) == (i < n), "%dD, kappa %g: time %d", ndim, kappa, i);
            bub_ctx_destroy(c);
        }
}

// The shape that transfer contents report is the one that their stages run.
static void contents()
{
    for (int ndim = 1; ndim <= 3; ++ndim) {
        Problem p = ndim == 1 ? Problem(1, 400, 1, 1, 11) : ndim == 2 ? Problem(2, 70, 37, 1, 11) : Problem(3, 20, 13, 11, 3);
        bub_ctx *c = p.transfer().make();
        int i = -1, t[4];
        CHECK(bub_tile_get(c, &i) == BUB_OK && i == 0, "shape %d", i);
        CHECK(bub_tile_info(c, i, &t[0], &t[1], &t[2], &t[3]) == BUB_OK, "info");
        CHECK(bub_tile_set(c, 0) == BUB_OK && bub_tile_set(c, 1) == BUB_EUNSUPPORTED, "set");
        bub_bin_groups(c, 1);
        CHECK(bub_rhs_stage(c, pretend(1), pretend(2), nullptr) == BUB_OK, "rhs");
        const FakeLaunch &l = fake().launches.back();
        unsigned tiles = 1;
        for (int d = 0; d < 3; ++d) tiles *= (p.grid.n[d] + t[d] - 1) / t[d];
        CHECK(l.block.x == (unsigned)t[3] && l.grid.x == 8 * ((tiles + 7) / 8), "%dD: %u workgroups of %u threads; %d x %d x %d by %d listed",
              ndim, l.grid.x, l.block.x, t[0], t[1], t[2], t[3]);
        bub_ctx_destroy(c);
    }
}

// Threads a cell of the primitive pass at the sizes that the GPU tests take for them.
static void threads()
{
    const struct { Problem p; int threads; } all[] = {
        {Problem(2, 700, 760, 1, 3), 1}, {Problem(2, 600, 500, 1, 5), 2}, {Problem(2, 150, 140, 1, 5), 4}, {Problem(2, 150, 150, 1, 7), 8},
        {Problem(2, 211, 203, 1, 11), 8}, {Problem(2, 200, 190, 1, 11), 8}, {Problem(3, 32, 32, 30, 11), 8},
        {Problem(2, 100, 100, 1, 17), 16}, {Problem(2, 45, 40, 1, 31), 32}, {Problem(1, 1800, 1, 1, 31), 32}, {Problem(2, 160, 150, 1, 1), 2},
    };
    for (auto &a : all) {
        bub_ctx *c = a.p.make();
        CHECK(bub_moments(c, pretend(1), pretend(2), nullptr) == BUB_OK, "moments");
        const FakeLaunch &l = fake().launches.back();
        const long long cells = (long long)a.p.grid.n[0] * a.p.grid.n[1] * a.p.grid.n[2];
        const double per = (double)l.grid.x * l.block.x / cells;   // (the last workgroup may be partly idle)
        CHECK(per >= a.threads && per < a.threads * 1.2, "%lld cells, %d bins: %g threads a cell, not %d", cells, a.p.bins.nb, per,
              a.threads);
        bub_ctx_destroy(c);
    }
}

int main(int argc, char **argv)
{
    const std::string name = argc > 1 ? argv[1] : "";
    if (name == "budget") budget();
    else if (name == "scratch") scratch();
    else if (name == "unused") unused();
    else if (name == "cache") cache();
    else if (name == "shapes") shapes();
    else if (name == "contents") contents();
    else if (name == "threads") threads();
    else if (name == "classes") classes();
    else return 2;
    std::printf("%d failures\n", failures);
    return failures != 0;
}

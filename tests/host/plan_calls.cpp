// The library's host code alone (no GPU code, no GPU): what a call is planned
// as, over tables and limits that only a handle has.  argv[1] names the check;
// the exit status is 0 if it holds.
#include "../../paper_2609_16389_amd/csrc/xgemm.hip"

#include <random>
#include <stdlib.h>
#include <thread>

namespace {

constexpr int kCUs = 256;

struct Shape {
    int64_t M, N, K, lda, ldb;
};

int plan(const Shape &s, bool persistent, size_t limit, PlanCache *cache, CallPlan *cp)
{
    const uintptr_t base = 1 << 20;
    return plan_call(kCUs, s.M, s.N, s.K, (void *)base, s.lda, (void *)base, s.ldb, (float *)base, s.N, nullptr, cp,
                     persistent, limit, cache);
}

bool same(const CallPlan &a, const CallPlan &b)
{
    if (a.parts != b.parts || a.ws != b.ws)
        return false;
    for (int i = 0; i < a.parts; ++i) {
        const Segment &x = a.plan[i].seg[0], &y = b.plan[i].seg[0];
        if (a.plan[i].tile != b.plan[i].tile || a.M[i] != b.M[i] || a.N[i] != b.N[i] || x.p.split != y.p.split ||
            x.p.group_m != y.p.group_m || x.grid != y.grid || x.sk != y.sk || x.reduce != y.reduce)
            return false;
    }
    return true;
}

// Shapes drawn evenly over the logarithm of their sizes, contiguous, padded
// and odd, far more than the table has slots.
std::vector<Shape> shapes(int n)
{
    std::mt19937 gen(7);
    auto size = [&](double lo, double hi) {
        return (int64_t)exp(std::uniform_real_distribution<double>(log(lo), log(hi))(gen));
    };
    std::vector<Shape> out;
    for (int i = 0; i < n; ++i) {
        Shape s{size(1, 9000), size(8, 9000), size(8, 9000), 0, 0};
        if (i % 3 == 0)
            s.M = s.M / 256 * 256 + 256, s.N = s.N / 256 * 256 + 256, s.K = s.K / 64 * 64 + 64;
        const int64_t pad = i % 4 == 1 ? 8 : i % 4 == 2 ? 3 : 0;
        s.lda = s.K + pad;
        s.ldb = s.N + pad;
        out.push_back(s);
    }
    return out;
}

// Threads that share one handle's table plan what each plans alone.
int threads(int count)
{
    const std::vector<Shape> all = shapes(600);
    std::vector<CallPlan> alone(all.size());
    for (size_t i = 0; i < all.size(); ++i)
        plan(all[i], true, 0, nullptr, &alone[i]);
    PlanCache table;
    std::vector<long> wrong(count, 0);
    std::vector<std::thread> pool;
    for (int t = 0; t < count; ++t)
        pool.emplace_back([&, t] {
            std::mt19937 gen(t);
            for (int k = 0; k < 60000; ++k) {
                const size_t i = gen() % all.size();
                CallPlan cp;
                wrong[t] += plan(all[i], true, 0, &table, &cp) != XGEMM_OK || !same(cp, alone[i]);
            }
        });
    for (std::thread &t : pool)
        t.join();
    long sum = 0;
    for (long w : wrong)
        sum += w;
    printf("%d threads, %ld plans differ\n", count, sum);
    return sum != 0;
}

// A persistent plan whose operands that kernel cannot take: the plans with and
// without it stay in the table together.
int kept()
{
    const Shape s{8192, 8192, 8192, 8192 + 1, 8192};
    PlanCache table;
    CallPlan cp;
    plan(s, true, 0, &table, &cp);
    int found = 0;
    for (const PlanCache::Band &e : table.band)
        if (e.M == s.M && e.N == s.N && e.K == s.K)
            found |= 1 << e.persistent;
    return found != 3;
}

// The plan xgemm_run_noalloc enqueues, or false where it refuses the call.
bool noalloc(const Shape &s, CallPlan *cp)
{
    if (plan(s, true, kScratchBytes, nullptr, cp) != XGEMM_OK)
        return false;
    if (cp->ws + kWsPrefix > kScratchBytes && plan(s, false, kScratchBytes, nullptr, cp) != XGEMM_OK)
        return false;
    return cp->ws + kWsPrefix <= kScratchBytes;
}

// What a limit on the workspace changes: xgemm_run_noalloc takes a call
// exactly if xgemm_run's plan fits its scratch, and then runs the same plan
// (but for the persistent kernel's partial sums); a limit in general refuses
// no call whose plan needs less.
int limits()
{
    std::vector<Shape> all = shapes(3000);
    // tile plans that fit the scratch where a deeper K split does not
    for (Shape s : {Shape{201, 571, 37855, 37855, 571}, Shape{375, 357, 38245, 38245, 357},
                    Shape{533, 177, 42183, 42183, 177}, Shape{515, 207, 41455, 41455, 207}})
        all.push_back(s);
    // decoding steps read in place, whose operand copies would not fit
    const std::vector<Shape> in_place = {{93, 13489, 12508, 12508, 13489}, {16, 10377, 8657, 8657, 10377}};
    all.insert(all.end(), in_place.begin(), in_place.end());
    std::mt19937 gen(11);
    for (int i = 0; i < 2000; ++i) {   // few outputs, long K
        Shape s{128 + (int64_t)(gen() % 896), 128 + (int64_t)(gen() % 896), 8192 + (int64_t)(gen() % 57344), 0, 0};
        s.lda = s.K;
        s.ldb = s.N;
        all.push_back(s);
    }
    int bad = 0, accepted = 0;
    auto fail = [&](const Shape &s, const char *why) {
        if (++bad < 10)
            printf("%lld x %lld x %lld (lda %lld, ldb %lld): %s\n", (long long)s.M, (long long)s.N, (long long)s.K,
                   (long long)s.lda, (long long)s.ldb, why);
    };
    for (const Shape &s : all) {
        CallPlan run, na, cp;
        plan(s, true, 0, nullptr, &run);
        const bool took = noalloc(s, &na);
        accepted += took;
        if (run.plan[0].seg[0].sk && run.ws > 0)
            plan(s, run.ws + kWsPrefix <= kScratchBytes, 0, nullptr, &run);
        if (took != (run.ws + kWsPrefix <= kScratchBytes))
            fail(s, took ? "taken, though xgemm_run's plan does not fit" : "refused, though xgemm_run's plan fits");
        else if (took && !same(run, na))
            fail(s, "another plan than xgemm_run's");
        const size_t limit = run.ws + kWsPrefix;
        plan(s, run.plan[0].seg[0].sk, limit, nullptr, &cp);
        if (!same(run, cp))
            fail(s, "another plan under the limit it keeps");
        plan(s, true, 1, nullptr, &cp);
        if (run.ws == 0 && cp.ws != 0)
            fail(s, "needs a workspace under a limit, none without");
    }
    for (const Shape &s : in_place) {
        CallPlan cp;
        if (!noalloc(s, &cp))
            fail(s, "refused");
    }
    printf("%d of %zu fit the scratch, %d wrong\n", accepted, all.size(), bad);
    return bad != 0;
}

// Batched calls: a limit changes no plan that keeps it and refuses none that
// needs less; a launch whose kernel does not apply (fewer than 8 columns or
// K, rows far apart) leaves the tile plan's as it was.
int batches()
{
    std::mt19937 gen(13);
    int bad = 0, replaced = 0, apply = 0;
    for (int i = 0; i < 4000; ++i) {
        auto size = [&](double lo, double hi) {
            return (int64_t)exp(std::uniform_real_distribution<double>(log(lo), log(hi))(gen));
        };
        const int64_t L = size(2, 129), M = size(1, 1025), N = i % 5 == 0 ? size(1, 8) : size(1, 1025),
                      K = i % 7 == 0 ? size(1, 8) : size(1, 1025);
        const int64_t pad = i % 3 == 0 ? 3 : 0;
        const int64_t lda = i % 11 == 0 ? (int64_t)1 << 28 : K + pad, ldb = N + pad;
        const int64_t sa = M * lda, sb = K * ldb, sc = M * N;
        const uintptr_t base = 1 << 20;
        xgemm_config tile;
        select_config_batched(L, M, N, K, kCUs, &tile);
        BatchPlan t, got, under;
        auto call = [&](size_t limit, BatchPlan *bp) {
            return plan_batched_call(kCUs, true, L, M, N, K, (void *)base, lda, sa, (void *)base, ldb, sb,
                                     (float *)base, N, sc, limit, nullptr, bp);
        };
        plan_batched(kCUs, true, L, M, N, K, (void *)base, lda, sa, (void *)base, ldb, sb, (float *)base, N, sc, tile,
                     &t);
        const bool ok = call(0, &got) == XGEMM_OK && call(got.ws + kWsPrefix, &under) == XGEMM_OK;
        replaced += got.plan.tile != t.plan.tile;
        apply += !(N < 8 || K < 8 || lda > ((int64_t)1 << 27));
        const bool general = !got.plan.seg[0].dma && !got.plan.seg[0].sk && !is_direct(got.plan.tile);
        const bool kept = got.plan.tile == t.plan.tile && got.plan.seg[0].p.group_m == t.plan.seg[0].p.group_m;
        if (!ok || under.plan.tile != got.plan.tile || under.ws != got.ws || (general && !kept) ||
            ((N < 8 || K < 8) && is_direct(got.plan.tile))) {
            if (++bad < 10)
                printf("%lld of %lld x %lld x %lld, lda %lld: tile %d, under its own limit %d; the tile plan's %d\n",
                       (long long)L, (long long)M, (long long)N, (long long)K, (long long)lda, got.plan.tile,
                       under.plan.tile, t.plan.tile);
        }
    }
    printf("%d of 4000 replaced, %d wrong\n", replaced, bad);
    return bad != 0 || replaced < 1000 || apply < 1000;
}

// Decoding steps of 17 to 64 rows: no K split that leaves some CUs with one
// workgroup and gives a few (under three in eight) two.
int doubled_up()
{
    std::mt19937 gen(17);
    int bad = 0, splits = 0;
    for (int i = 0; i < 4000; ++i) {
        const int64_t N = 8192 + (int64_t)(gen() % 24576), K = 1024 + (int64_t)(gen() % 12288);
        const Shape s{17 + (int64_t)(gen() % 48), N, K, K + (i % 2), N + (i % 3)};
        CallPlan cp;
        plan(s, true, 0, nullptr, &cp);
        const Segment &g = cp.plan[0].seg[0];
        if (!is_direct(cp.plan[0].tile) || g.p.split == 1)
            continue;
        ++splits;
        if (cp.plan[0].tile == XGEMM_DIRECT_32x256 && g.grid > kCUs && g.grid < 11 * kCUs / 8) {
            if (++bad < 10)
                printf("%lld x %lld x %lld: %lld workgroups of 32 x 256, split %d\n", (long long)s.M, (long long)s.N,
                       (long long)s.K, (long long)g.grid, g.p.split);
        }
    }
    // the price of a tile plan whose split does so is its own measurement: K
    // splits of 128 x 128 tiles keep their place against other launches
    for (const Shape &s : {Shape{960, 257, 60048, 60048, 257}, Shape{2112, 763, 5160, 5160, 763}}) {
        CallPlan cp;
        plan(s, true, 0, nullptr, &cp);
        bad += cp.plan[0].tile != XGEMM_TILE_128x128;
    }
    printf("%d of %d splits\n", bad, splits);
    return bad != 0 || splits < 500;
}

// Odd rows of A under 64 x 64 blocks: the K splits that were slower than the
// tile plan go to other launches, aligned rows keep theirs.
int odd_rows()
{
    CallPlan odd, even;
    int bad = 0;
    for (const Shape &s : {Shape{493, 264, 18432, 18433, 264}, Shape{50, 5552, 2752, 2753, 5552},
                           Shape{55, 6272, 2816, 2817, 6272}}) {
        plan(s, true, 0, nullptr, &odd);
        bad += odd.plan[0].tile == XGEMM_DIRECT_64x64 && odd.plan[0].seg[0].p.split > 1;
    }
    plan(Shape{384, 832, 6848, 6848, 832}, true, 0, nullptr, &even);
    bad += even.plan[0].tile != XGEMM_DIRECT_64x64 || even.plan[0].seg[0].p.split != 3;
    printf("%d wrong\n", bad);
    return bad != 0;
}

// The launch a batch takes: L, M, N, K, the pad of A's rows, one B for all.
int batch_route(char **v)
{
    const int64_t L = atoll(v[0]), M = atoll(v[1]), N = atoll(v[2]), K = atoll(v[3]), lda = K + atoll(v[4]);
    const uintptr_t base = 1 << 20;
    BatchPlan bp;
    if (plan_batched_call(kCUs, true, L, M, N, K, (void *)base, lda, M * lda, (void *)base, N, atoi(v[5]) ? 0 : K * N,
                          (float *)base, N, M * N, 0, nullptr, &bp) != XGEMM_OK)
        return 1;
    const Segment &g = bp.plan.seg[0];
    printf("%s\n", is_direct(bp.plan.tile) ? "direct" : g.sk ? "persistent" : !g.dma ? "general" :
                   bp.plan.pack.a || bp.plan.pack.b ? "copied" : "pipelined");
    return 0;
}

// Which register-direct launches of a 16-row block stream B: its size, and
// rows that are whole cache lines.
int streams()
{
    struct {
        int64_t M, N, K, ldb;
        uintptr_t B;
        bool on;
    } const cases[] = {
        {16, 14336, 4096, 14336, 1 << 20, true},     {5, 8192, 6001, 8192, 1 << 20, true},
        {16, 14336, 4096, 14344, 1 << 20, false},    {16, 14336, 4096, 14336, (1 << 20) + 16, false},
        {16, 14336, 12288, 14336, 1 << 20, true},    {16, 14336, 12288, 14339, 1 << 20, false},
        {16, 14336, 8192, 14336, 1 << 20, false},    {16, 10240, 4096, 10240, 1 << 20, false},
        {17, 14336, 4096, 14336, 1 << 20, false},
    };
    int bad = 0;
    for (const auto &c : cases) {
        CallPlan cp;
        const xgemm_config cfg{XGEMM_DIRECT_16x128, 2, 4, 0};
        bad += plan_call(kCUs, c.M, c.N, c.K, (void *)(1 << 20), c.K, (void *)c.B, c.ldb, (float *)(1 << 20), c.N, &cfg,
                         &cp) != XGEMM_OK || cp.plan[0].tile != cfg.tile || streams_b(cp.plan[0].seg[0].p) != c.on;
    }
    printf("%d wrong\n", bad);
    return bad != 0;
}

}  // namespace

int main(int argc, char **argv)
{
    const char *what = argc > 1 ? argv[1] : "";
    if (!strcmp(what, "threads"))
        return threads(atoi(argv[2]));
    if (!strcmp(what, "kept"))
        return kept();
    if (!strcmp(what, "limits"))
        return limits();
    if (!strcmp(what, "batches"))
        return batches();
    if (!strcmp(what, "doubled_up"))
        return doubled_up();
    if (!strcmp(what, "odd_rows"))
        return odd_rows();
    if (!strcmp(what, "batch_route") && argc == 8)
        return batch_route(argv + 2);
    if (!strcmp(what, "streams"))
        return streams();
    return 2;
}

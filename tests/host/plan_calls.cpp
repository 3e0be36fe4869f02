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

}  // namespace

int main(int argc, char **argv)
{
    const char *what = argc > 1 ? argv[1] : "";
    if (!strcmp(what, "threads"))
        return threads(atoi(argv[2]));
    if (!strcmp(what, "kept"))
        return kept();
    return 2;
}

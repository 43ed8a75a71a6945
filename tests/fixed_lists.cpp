/* The fixed-order loops' lists: build_fixed's pass verify_fixed over chunk sizes,
 * orders and graphs with ragged ends, and a list with any one value changed does
 * not.  Prints "ok". */
#include <cstdio>
#include <random>
#include <vector>

#include "opflux.h"
#include "planner.hpp"

using namespace opf;
static const int NT = 512;

#define CHECK(cond, ...)                            \
    do {                                            \
        if (!(cond)) {                              \
            std::fprintf(stderr, __VA_ARGS__);      \
            std::fprintf(stderr, "\n");             \
            return 1;                               \
        }                                           \
    } while (0)

// Changes single values of one array and expects each change to be found.
template <class V>
static long missed(const Plan &P, FixedLists &F, V &v, std::mt19937 &rng)
{
    long n = 0;
    for (int t = 0; t < 40 && !v.empty(); ++t) {
        auto &x = v[rng() % v.size()];
        const auto old = x;
        x = static_cast<typename V::value_type>(x ^ (1u << rng() % (8 * sizeof x)));
        n += verify_fixed(P, F, NT).ok;
        x = old;
    }
    return n;
}

static int check(const std::vector<int32_t> &e2n, int N, int K, int chunk, int renumber, std::mt19937 &rng)
{
    PlanOptions o;
    o.renumber = renumber;
    o.block_size = 64;
    o.cluster_size = K;
    Plan P;
    std::string err;
    CHECK(build_plan(N, (int64_t)e2n.size() / 2, e2n.data(), o, P, err) == OPF_OK, "%s", err.c_str());
    CHECK(verify_plan(P, e2n.data()).ok, "plan");
    FixedLists F;
    build_fixed(P, chunk, NT, F);
    const VerifyResult r = verify_fixed(P, F, NT);
    CHECK(r.ok, "N %d K %d chunk %d: %s at %ld", N, K, chunk, r.message.c_str(), (long)r.where);
    CHECK(F.fine == (chunk != K), "fine");
    long n = missed(P, F, F.cv_off, rng);
    if (F.fine)
        n += missed(P, F, F.node_off, rng) + missed(P, F, F.cv_eid, rng) + missed(P, F, F.cv_oth, rng) +
             missed(P, F, F.cv_own, rng);
    else
        n += missed(P, F, F.iblk, rng) + missed(P, F, F.rnd_off, rng) + missed(P, F, F.ent_base, rng) +
             missed(P, F, F.off, rng) + missed(P, F, F.ent, rng);
    CHECK(n == 0, "N %d K %d chunk %d: %ld changes not found", N, K, chunk, n);
    return 0;
}

int main()
{
    std::mt19937 rng(11);
    for (int N : {65, 500, 512, 513, 1025, 3000})
        for (int hub : {0, 1}) {
            std::vector<int32_t> e2n;
            auto edge = [&](int a, int b) {
                if (rng() & 1) std::swap(a, b);
                e2n.push_back(a);
                e2n.push_back(b);
            };
            for (int i = 0; i < N; ++i)
                for (int d : {1, 7, 130})
                    if (i + d < N) edge(i, i + d);
            for (int i = 1; hub && i < N; ++i) edge(0, i);
            if (!hub) edge(3, 4);  // twice in the map
            for (int renumber : {(int)OPF_RENUM_NONE, (int)OPF_RENUM_RCM})
                for (int K : {64, 100, 512}) {
                    if (check(e2n, N, K, K, renumber, rng)) return 1;
                    if (check(e2n, N, K, 32, renumber, rng)) return 1;
                }
        }
    std::puts("ok");
    return 0;
}

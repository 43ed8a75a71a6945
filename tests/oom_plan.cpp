/* Host memory that runs out while opf_plan works: every call then returns OPF_OK or
 * OPF_ENOMEM (no exception and no abort leaves the library), and the context plans
 * afterwards as if nothing had been.  The replaced operator new fails at the n-th
 * allocation of the call, alone or with every later one.  Prints "ok". */
#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <new>
#include <vector>

#include "opflux.h"

static std::atomic<long> seen(0), limit(-1);  // allocations since arm(); the one that fails, or -1
static std::atomic<bool> later(false);        // and every one after it

static void arm(long n, bool and_later)
{
    later = and_later;
    seen = 0;
    limit = n;
}
// Whether the failure came.
static bool disarm()
{
    const long n = limit.exchange(-1);
    return seen.load() > n;
}

void *operator new(std::size_t n)
{
    const long at = limit.load();
    if (at >= 0) {
        const long k = seen.fetch_add(1);
        if (k == at || (k > at && later)) throw std::bad_alloc();
    }
    void *p = std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

int main()
{
    const int N = 3000, E = 3 * N;
    std::vector<int32_t> e2n;
    for (int i = 0; i < N; ++i)
        for (int d : {1, 7, 130}) {
            e2n.push_back(i);
            e2n.push_back((i + d) % N);
        }
    opf_ctx *ctx = nullptr;
    opf_set nodes, edges;
    opf_map m;
    if (opf_init(&ctx, -1) || opf_decl_set(ctx, N, "nodes", &nodes) || opf_decl_set(ctx, E, "edges", &edges) ||
        opf_decl_map(ctx, edges, nodes, 2, e2n.data(), 0, "e2n", &m))
        return 1;
    opf_plan_opts o = {};
    o.renumber = OPF_RENUM_RCM;
    o.block_size = 64;
    o.cluster_size = 64;
    o.lane_groups = o.bank_spread = o.halo_order = 1;
    opf_plan_report rep;
    int refused = 0;
    for (int mode = 0; mode < 2; ++mode)
        for (long n = 0;; n += n < 400 ? 1 : 1 + n / 40) {
            arm(n, mode == 1);
            const int rc = opf_plan(ctx, m, &o, nullptr);
            const bool reached = disarm();
            if (rc != OPF_OK && rc != OPF_ENOMEM) {
                std::fprintf(stderr, "allocation %ld: %d %s\n", n, rc, opf_last_error(ctx));
                return 1;
            }
            refused += rc == OPF_ENOMEM;
            if (!reached) break;
            arm(n % 60, mode == 1);  // the verification allocates too
            const int rv = opf_plan_verify(ctx, m, &rep);
            disarm();
            if (rv != OPF_OK && rv != OPF_ENOMEM && rv != OPF_ESTATE) return 1;
        }
    if (refused < 100) return 1;
    if (opf_plan(ctx, m, &o, nullptr) != OPF_OK || opf_plan_verify(ctx, m, &rep) != OPF_OK || !rep.ok) return 1;
    opf_finalize(ctx);
    std::puts("ok");
    return 0;
}

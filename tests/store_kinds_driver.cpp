// The kind of store as something a search chooses, for tests/test_write_through.py: searches over costs that are made up.  Host code only.
// Argument: the test; prints "ok".
#include <stdio.h>
#include <string.h>

#include "addrms_internal.h"

using namespace addrms_host;

#define EXPECT(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

// 8192 rows of 1000, fp16 with an fp32 residual: streaming aligned spans are best, others with whole accesses 7 % behind, and what is
// written through costs `written` times as much.
constexpr int64_t kM = 8192, kN = 1000;
constexpr int kDtype = ADDRMS_FP16_RES32;
struct Costs { double written; int through; };
static int measure(void* user, const addrms_cfg* c, int, int, double* us)
{
    Costs& costs = *static_cast<Costs*>(user);
    *us = 10.0 * ((c->flags & ADDRMS_FLAG_ALIGNED_SPAN) ? 1.0 : 1.07) * ((c->flags & ADDRMS_FLAG_NONTEMPORAL) ? 1.0 : 1.2) * (c->vec == 4 ? 1.0 : 1.5) *
          (c->max_waves_per_simd ? 1.1 : 1.0) * (c->flags & ADDRMS_FLAG_PERSISTENT ? 1.3 : 1.0);
    if (launch_write_through(*c, kM, kN, kDtype, OP_ADDRMS)) {
        *us *= costs.written;
        ++costs.through;
    }
    return 0;
}
static int search(double written, int strategy, bool store_kinds, addrms_cfg* best, addrms_tune_report* rep, int* through)
{
    Costs costs{written, 0};
    addrms_backend be{&costs, nullptr, measure};
    addrms_budget b{};
    b.strategy = strategy;
    const int st = run_search(kM, kN, kDtype, &b, be, best, rep, OP_ADDRMS, store_kinds);
    *through = costs.through;
    return st;
}

static int chooses()
{
    addrms_cfg best{};
    addrms_tune_report rep{};
    int through = 0;
    for (int strategy : {ADDRMS_SEARCH_GUIDED, ADDRMS_SEARCH_EXHAUSTIVE}) {
        // from memory: the spans, streaming; what is written through was timed beside it only
        EXPECT(search(1.08, strategy, true, &best, &rep, &through) == ADDRMS_OK);
        EXPECT((best.flags & ADDRMS_FLAG_ALIGNED_SPAN) && (best.flags & ADDRMS_FLAG_STREAM_STORES) && !launch_write_through(best, kM, kN, kDtype, OP_ADDRMS));
        EXPECT(check_cfg(best, kM, kN, kDtype).status == ADDRMS_OK && rep.best.flags == best.flags && through == 2);
        // where writing through is what is fast
        EXPECT(search(0.9, strategy, true, &best, &rep, &through) == ADDRMS_OK);
        EXPECT((best.flags & ADDRMS_FLAG_ALIGNED_SPAN) && !(best.flags & ADDRMS_FLAG_STREAM_STORES) && launch_write_through(best, kM, kN, kDtype, OP_ADDRMS));
        // and of a backend that has one kind of store
        EXPECT(search(1.08, strategy, false, &best, &rep, &through) == ADDRMS_OK && !(best.flags & ADDRMS_FLAG_STREAM_STORES));
    }
    return 0;
}

// Rows by themselves in shares of 256 to 320 threads lead a little, and the way to the fastest begins at a span that is behind them.
static int measure_layouts(void*, const addrms_cfg* c, int, int, double* us)
{
    const bool deferred = c->flags & ADDRMS_FLAG_DEFER_STORE;
    const int threads = c->threads_per_row * c->rows_per_wg;
    if (c->flags & ADDRMS_FLAG_ALIGNED_SPAN) *us = threads == 1024 ? (c->rows_per_wg == 16 ? 17.4 : 18.8) : 19.4;
    else *us = c->threads_per_row == 320 ? 18.7 : c->threads_per_row == 256 ? 18.5 : c->threads_per_row == 128 ? 18.6 : 19.5;
    *us *= (c->flags & ADDRMS_FLAG_NONTEMPORAL ? 1.0 : 1.2) * (deferred ? 1.0 : 1.02) * (c->vec == 4 ? 1.0 : 1.5) * (c->max_waves_per_simd ? 1.1 : 1.0) *
           (c->flags & ADDRMS_FLAG_PERSISTENT ? 1.3 : 1.0) * (c->flags & ADDRMS_FLAG_XCD_CONTIG ? 1.02 : 1.0);
    return 0;
}
static int layouts()
{
    addrms_backend be{nullptr, nullptr, measure_layouts};
    addrms_budget b{};
    addrms_cfg best{};
    addrms_tune_report rep{};
    EXPECT(run_search(kM, kN, kDtype, &b, be, &best, &rep, OP_ADDRMS, true) == ADDRMS_OK);
    EXPECT((best.flags & ADDRMS_FLAG_ALIGNED_SPAN) && best.rows_per_wg == 16);
    return 0;
}

// One configuration for two shapes of which one writes through.
static int general()
{
    Costs costs{1.08, 0};
    const addrms_backend_factory f{&costs, [](void* u, int64_t, int64_t, int, addrms_backend* be) { *be = addrms_backend{u, nullptr, measure}; return 0; }, nullptr};
    const addrms_shape shapes[] = {{64, kN}, {kM, kN}};
    addrms_cfg c{};
    addrms_general_report rep{};
    EXPECT(run_select_general(shapes, 2, kDtype, nullptr, f, false, &c, &rep, OP_ADDRMS, true) == ADDRMS_OK);
    EXPECT(!launch_write_through(c, kM, kN, kDtype, OP_ADDRMS) && check_cfg(c, 64, kN, kDtype).status == ADDRMS_OK);
    EXPECT(!(rep.specialized[0].flags & ADDRMS_FLAG_STREAM_STORES) || cfg_equal(rep.specialized[0], c));
    return 0;
}

// Where the flag is accepted, what it leaves of the launch, and that a saved one comes back.
static int accepted()
{
    addrms_cfg c{8, 512, 1, 0, 1, ADDRMS_FLAG_NONTEMPORAL, 0, 0};
    EXPECT(launch_write_through(c, 4096, 4096, ADDRMS_BF16, OP_ADDRMS));
    c.flags |= ADDRMS_FLAG_STREAM_STORES;
    for (int64_t M : {1, 64, 4096, 32768}) {
        EXPECT(!launch_write_through(c, M, 4096, ADDRMS_BF16, OP_ADDRMS));
        addrms_cfg plain = c;
        plain.flags &= ~ADDRMS_FLAG_STREAM_STORES;
        const Feas a = check_cfg(c, M, 4096, ADDRMS_BF16), b = check_cfg(plain, M, 4096, ADDRMS_BF16);
        EXPECT(a.status == b.status && a.inst == b.inst && a.dyn_lds == b.dyn_lds && cfg_key(c) != cfg_key(plain) && !cfg_equal(c, plain));
    }
    EXPECT(check_cfg(c, 4096, 4096, ADDRMS_BF16, OP_SILUMUL).status == ADDRMS_OK);
    addrms_cfg merge{8, 32, 8, 0, 1, ADDRMS_FLAG_NONTEMPORAL, 0, 0};
    EXPECT(check_cfg(merge, 4096, 256, ADDRMS_BF16, OP_MERGE).status == ADDRMS_OK);
    merge.flags |= ADDRMS_FLAG_STREAM_STORES;
    EXPECT(check_cfg(merge, 4096, 256, ADDRMS_BF16, OP_MERGE).status == ADDRMS_ERR_INFEASIBLE_CFG);
    for (int bad : {0 | ADDRMS_FLAG_STREAM_STORES, ADDRMS_FLAG_STREAM_STORES | ADDRMS_FLAG_XCD_CONTIG, 256 | ADDRMS_FLAG_NONTEMPORAL}) {
        addrms_cfg d = c;
        d.flags = bad;
        EXPECT(check_cfg(d, 4096, 4096, ADDRMS_BF16).status == ADDRMS_ERR_INFEASIBLE_CFG);
    }
    std::vector<addrms_cfg> all;
    enumerate(4096, 4096, ADDRMS_BF16, &all, nullptr);
    for (const addrms_cfg& e : all) EXPECT(!(e.flags & ADDRMS_FLAG_STREAM_STORES));
    return 0;
}

int main(int, char** argv)
{
    const struct { const char* name; int (*run)(); } tests[] = {{"chooses", chooses}, {"layouts", layouts}, {"general", general}, {"accepted", accepted}};
    int bad = 1;
    for (const auto& t : tests)
        if (!strcmp(argv[1], t.name)) bad = t.run();
    if (!bad) printf("ok\n");
    return bad;
}

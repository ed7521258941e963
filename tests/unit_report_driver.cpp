// How launches say that they are done and how the host comes to know it (unit_report.h), on the CPU, for tests/test_unit_report.py.
// Between any two atomic operations of one thread others may come: at each of them the test may run what is pending.
// Argument: the test; prints "ok".
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <functional>
#include <vector>

static std::function<void()> between;                        // called before each atomic operation, and not while `apart` is set
static bool apart = false;
template <typename T> static T load(const T* p) { if (!apart) between(); return *p; }
template <typename T, typename F> static T change(T* p, F f) { if (!apart) between(); const T was = *p; *p = f(was); return was; }
struct Apart {
    const bool before = apart;
    Apart() { apart = true; }
    ~Apart() { apart = before; }
};

#define __device__
#define __forceinline__ inline
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_SYSTEM 1
#define __hip_atomic_load(p, order, scope) load(p)
#define __hip_atomic_store(p, v, order, scope) ((void)change(p, [&](auto) { return v; }))
#define __hip_atomic_exchange(p, v, order, scope) change(p, [&](auto) { return v; })
#define __hip_atomic_fetch_max(p, v, order, scope) change(p, [&](auto was) { return was < (v) ? (v) : was; })
#define __hip_atomic_fetch_add(p, v, order, scope) change(p, [&](auto was) { return was + (v); })
static struct { uint32_t x; } threadIdx;

#include "unit_report.h"

#define EXPECT(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

using Reports = addrms::UnitReports<1>;
static uint32_t seed = 1;
static uint32_t random(uint32_t n) { return (seed = seed * 1664525u + 1013904223u) / 65536u % n; }

// Launches of these many pieces, one after the other in one place, each told before the next: the pieces in any order, each
// interrupted by others, and told of again and again meanwhile.  The host's word has a launch's number exactly when all its
// additions have been made.
static int pieces()
{
    for (int trial = 0; trial < 200000; ++trial) {
        Reports r{};
        uint32_t word = 0, number = 0;
        for (int launch = 0; launch < 4; ++launch) {
            static const uint32_t counts[] = {1, 2, 3, 8, 9, 10, 64};
            const uint32_t all = counts[random(7)];
            number += 1 + random(3);                         // a number may have gone to a launch that failed
            std::vector<uint32_t> left;
            for (uint32_t p = 0; p < all; ++p) left.push_back(p);
            uint32_t finished = 0;
            bool early = false;
            const auto next = [&] {
                const uint32_t k = random(static_cast<uint32_t>(left.size())), p = left[k];
                left.erase(left.begin() + k);
                addrms::unit_piece_done(&r.state[0], number, p, all);
                ++finished;
            };
            const auto tell = [&] {
                const Apart alone;
                addrms::unit_tell(&r, &word, 1u);
                early = early || (word == number && finished < all);
            };
            between = [&] {
                if (random(2)) tell();
                if (!left.empty() && random(3)) next();
            };
            while (!left.empty()) next();
            EXPECT(!early);
            tell();
            EXPECT(word == number);
        }
    }
    return 0;
}

// One that tells is held up between any two of its steps, while another tells the same, the host gives the place to the next launch,
// that one ends and is told of as well.  No word goes back to an older number, nor is one lost.
static int held_up()
{
    for (int step = 0; step < 4; ++step) {
        Reports r{};
        uint32_t word = 0, most = 0;
        int steps = 0;
        bool back = false;
        between = [&] {
            const Apart alone;
            for (uint32_t n = 2; steps == step && n <= 3; ++n) {
                addrms::unit_tell(&r, &word, 1u);
                if (word + 1 != n) break;                    // not told: the place is not another launch's
                addrms::unit_done(&r.state[0], n);
                addrms::unit_tell(&r, &word, 1u);
            }
            ++steps;
            back = back || word < most;
            most = word;
        };
        {
            const Apart alone;
            addrms::unit_done(&r.state[0], 1u);
        }
        addrms::unit_tell(&r, &word, 1u);
        EXPECT(!back && word >= most);
        const Apart alone;
        addrms::unit_tell(&r, &word, 1u);
        EXPECT(word >= most && word == static_cast<uint32_t>(r.state[0] >> 32));
    }
    return 0;
}

int main(int, char** argv)
{
    const struct { const char* name; int (*run)(); } tests[] = {{"pieces", pieces}, {"held_up", held_up}};
    int bad = 1;
    for (const auto& t : tests)
        if (!strcmp(argv[1], t.name)) bad = t.run();
    if (!bad) printf("ok\n");
    return bad;
}

// Units of the memory that split rows meet in (slot_map.h) and the shapes in which rows are split, for
// tests/test_split_rows.py.  Host code only.
//   slots   who gets which units; prints "ok"
//   walk    the split of rows of many lengths and numbers; prints the number of decisions and the kernels asked for
//   (no argument)  one problem per line: dtype M N; one split per line of output
#include <stdio.h>
#include <string.h>

#include <initializer_list>
#include <set>
#include <tuple>
#include <vector>

#include "direct_route.h"
#include "slot_map.h"

using namespace addrms_host;
using namespace addrms;

#define EXPECT(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

// A launch in flight is one that has taken units and not reported: no two of them have a unit in common, whatever ends when.
static int in_any_order()
{
    static SlotMap<64> map;
    uint32_t done[64] = {};
    struct Launch { int first, units; uint32_t number; };
    std::vector<Launch> flying;
    uint32_t seed = 1;
    const auto random = [&](uint32_t n) { seed = seed * 1664525u + 1013904223u; return (seed >> 16) % n; };
    int refused = 0;
    for (int k = 0; k < 200000; ++k) {
        const int units = 1 + static_cast<int>(random(k % 3 == 0 ? 24 : 4));
        const int u = map.take(units, done);
        if (u < 0) ++refused;
        else {
            EXPECT(u + units <= 64);
            for (const Launch& l : flying) EXPECT(u + units <= l.first || l.first + l.units <= u);
            if (random(8) == 0) map.give_back(u);
            else flying.push_back({u, units, map.number(u)});
        }
        for (uint32_t ends = random(3); ends && !flying.empty(); --ends) {
            const size_t i = random(2) ? 0 : random(static_cast<uint32_t>(flying.size()));
            done[flying[i].first] = flying[i].number;
            flying.erase(flying.begin() + static_cast<long>(i));
        }
    }
    EXPECT(refused > 100 && refused < 150000);
    for (const Launch& l : flying) done[l.first] = l.number;
    EXPECT(map.take(64, done) == 0);                              // nothing is lost: when all have ended, all is free
    return 0;
}

static int slots()
{
    static SlotMap<8> map;
    uint32_t done[8] = {};
    for (int i = 0; i < 4; ++i) EXPECT(map.take(2, done) == 2 * i && map.number(2 * i) == 1u);
    EXPECT(map.take(1, done) == -1);                              // all in flight
    done[4] = 1;
    EXPECT(map.take(3, done) == -1);                              // two are free, three are not
    EXPECT(map.take(1, done) == 4 && map.number(4) == 2u);
    EXPECT(map.take(1, done) == 5 && map.take(1, done) == -1);
    map.give_back(5);
    EXPECT(map.take(1, done) == 5 && map.number(5) == 2u);        // a launch that was not made
    done[0] = done[2] = 1;
    EXPECT(map.take(4, done) == 0 && map.number(0) == 2u && map.take(1, done) == -1);
    if (in_any_order()) return 1;
    printf("ok\n");
    return 0;
}

static bool route(int dtype, int64_t M, int64_t N, DirectRoute* p)
{
    addrms_cfg c{};
    std::string why;
    return default_cfg(N, dtype, &c, &why) == ADDRMS_OK && direct_addrms_route(M, N, dtype, c.vec, 0, 0, 0, p);
}

static int walk()
{
    std::set<std::tuple<int, int, int, bool>> asked;
    long n = 0;
    for (int dt : {ADDRMS_BF16, ADDRMS_FP16, ADDRMS_FP16_RES32, ADDRMS_FP32}) {
        const int vec = direct_vec(dt);
        for (int64_t N = 32000; N < 600000; N += N < 33000 ? 7 : N / 61 + (N % 2))
            for (int64_t M : {1, 2, 3, 5, 8, 17, 31, 32, 33, 64, 127, 128, 129, 159, 160, 200, 256, 257, 447, 448, 512, 513, 900, 5000, 100000}) {
                DirectRoute p;
                if (!route(dt, M, N, &p) || !p.parts) continue;
                ++n;
                const int64_t most = N + (p.rag ? 128 / x_bytes(dt) - 1 : 0), part = int64_t(p.part_threads) * p.part_cpt * vec;
                const bool shape = p.parts >= 2 && p.parts <= unsigned(kSplitParts) && p.part_threads >= 64 && p.part_threads <= 1024 && p.part_threads % 64 == 0;
                if (!p.long_row || !shape || p.parts * part < most || (p.parts - 1) * part >= most) {
                    printf("bad split: dtype %d M %lld N %lld\n", dt, (long long)M, (long long)N);
                    return 1;
                }
                asked.insert({dt, p.part_cpt, p.part_pol, p.rag});
            }
    }
    for (const auto& k : asked)
        if (!split_instance(std::get<1>(k), std::get<2>(k))) {
            printf("no such kernel\n");
            return 1;
        }
    printf("%ld decisions, %zu kernels\n", n, asked.size());
    return asked.size() == 4u * 4u * 2u ? 0 : 1;             // and every one that is built can be asked for
}

int main(int argc, char** argv)
{
    if (argc > 1) return strcmp(argv[1], "slots") ? walk() : slots();
    int dtype;
    long long M, N;
    while (scanf("%d %lld %lld", &dtype, &M, &N) == 3) {
        DirectRoute p;
        if (!route(dtype, M, N, &p) || !p.parts) printf("whole\n");
        else printf("parts=%u threads=%u pieces=%d %s\n", p.parts, p.part_threads, p.part_cpt, p.part_pol == POL_NT ? "nontemporal" : "writethrough");
    }
    return 0;
}

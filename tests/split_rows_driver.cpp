// Slots of split rows (stream_slots.h) and the shapes in which rows are split, for tests/test_split_rows.py.  Host code only.
//   slots   who gets which slot; prints "ok"
//   walk    the split of rows of many lengths and numbers; prints the number of decisions and the kernels asked for
//   (no argument)  one problem per line: dtype M N; one split per line of output
#include <stdio.h>
#include <string.h>

#include <initializer_list>
#include <set>
#include <tuple>

#include "direct_route.h"
#include "stream_slots.h"

using namespace addrms_host;
using namespace addrms;

#define EXPECT(c) do { if (!(c)) { printf("line %d: %s\n", __LINE__, #c); return 1; } } while (0)

static int slots()
{
    StreamSlots s;
    uint32_t done[kStreamSlots * 2] = {};
    int got[kStreamSlots];
    for (int i = 0; i < kStreamSlots; ++i) {                       // streams 100, 101, ...: a slot each
        got[i] = s.take(100u + i, done, 2);
        EXPECT(got[i] >= 0);
        for (int j = 0; j < i; ++j) EXPECT(got[j] != got[i]);
        EXPECT(s.next(got[i]) == 1u);
        s.launched(got[i]);
    }
    EXPECT(s.take(7, done, 2) == -1);                             // all in flight
    for (int k = 0; k < 1000; ++k) {                              // a stream's launches share its slot, however many there are
        EXPECT(s.take(101, done, 2) == got[1] && s.next(got[1]) == 2u + k);
        s.launched(got[1]);
    }
    done[got[1] * 2] = 1000;                                      // all but the last of them
    EXPECT(s.take(7, done, 2) == -1);
    done[got[1] * 2] = 1001;
    EXPECT(s.take(7, done, 2) == got[1]);                         // idle: given to another stream, the numbers go on
    EXPECT(s.next(got[1]) == 1002u);
    EXPECT(s.take(7, done, 2) == got[1]);                         // a launch that failed was not announced
    s.launched(got[1]);
    EXPECT(s.take(101, done, 2) == -1);                           // the stream that had it before has none now
    EXPECT(s.take(100, done, 2) == got[0]);
    done[got[3] * 2] = 1;
    EXPECT(s.take(0, done, 2) == got[3]);                         // the null stream is a stream like others
    EXPECT(s.take(0, done, 2) == got[3]);
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

// Which rows in registers are split over workgroups, and how ragged ones read their single elements, for tests/test_few_rows.py and
// tests/test_shared_lines.py.  Host code only.
//   walk            every length in steps, and the numbers of rows around the limits: shapes; prints "ok"
//   singles [silu]  one problem per line: dtype M N; how its single elements, or all of a ragged activation, are read
//   (no argument)   likewise; one split per line of output
#include <stdio.h>
#include <string.h>

#include <initializer_list>

#include "direct_route.h"

using namespace addrms_host;
using namespace addrms;

static bool route(int dtype, int64_t M, int64_t N, DirectRoute* p)
{
    addrms_cfg c{};
    std::string why;
    if (default_cfg(N, dtype, &c, &why) != ADDRMS_OK || !direct_addrms_route(M, N, dtype, c.vec, 0, 0, 0, p) || p->long_row) return false;
    direct_addrms_split_few(M, N, dtype, p);
    return true;
}

int main(int argc, char** argv)
{
    const bool singles = argc > 1 && !strcmp(argv[1], "singles");
    if (argc > 1 && !singles) {
        for (int dt : {ADDRMS_BF16, ADDRMS_FP16, ADDRMS_FP16_RES32, ADDRMS_FP32})
            for (int64_t N = 64; N <= 32768; N += N < 12000 ? 331 : 37)
                for (int64_t M : {1, 2, 15, 16, 17, 40, 64, 80, 81, 127, 128, 129, 500, 5000}) {
                    DirectRoute p, whole;
                    if (!route(dt, M, N, &p) || !p.parts) continue;
                    addrms_cfg c{};
                    std::string why;
                    default_cfg(N, dt, &c, &why);
                    direct_addrms_route(M, N, dt, c.vec, 0, 0, 0, &whole);
                    const int64_t most = N + (p.rag ? 128 / x_bytes(dt) - 1 : 0), part = int64_t(p.part_threads) * p.part_cpt * 4;
                    if (direct_vec(dt) != 4 || M > 128 || N < 12226 || p.parts < 2 || p.parts > unsigned(kSplitParts) || p.part_threads % 64 ||
                        p.part_threads < 64 || p.part_threads > 1024 || p.parts * part < most || (p.parts - 1) * part >= most ||
                        !split_instance(p.part_cpt, p.part_pol) || p.grid != whole.grid ||
                        p.block_x != whole.block_x || p.block_y != whole.block_y || p.cpt != whole.cpt || p.pol != whole.pol || p.lds != whole.lds) {
                        printf("bad split: dtype %d M %lld N %lld\n", dt, (long long)M, (long long)N);
                        return 1;
                    }
                }
        printf("ok\n");
        return 0;
    }
    int dtype;
    long long M, N;
    while (scanf("%d %lld %lld", &dtype, &M, &N) == 3) {
        DirectRoute p;
        if (argc > 2) {                                      // silu_and_mul
            printf("%s\n", !direct_silumul_route(M, N, dtype, 0, 0, &p) || !p.rag ? "none" : p.keep_shared && p.pol == POL_WT ? "ordinary" : "nontemporal");
            continue;
        }
        const bool rows = route(dtype, M, N, &p);
        if (singles) printf("%s\n", !rows || !p.rag ? "none" : p.keep_shared ? "ordinary" : "nontemporal");
        else if (!rows || !p.parts) printf("whole\n");
        else printf("parts=%u threads=%u pieces=%d\n", p.parts, p.part_threads, p.part_cpt);
    }
    return 0;
}

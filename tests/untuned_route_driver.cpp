// Prints what the rules for calls without a configuration decide, for tests/test_untuned_route.py.  Host code only.
//   (no argument)  one problem per line of standard input: op dtype M N x r w, the last three being bytes past a multiple
//                  of 16; one decision per line of output
//   walk           every kernel that the rules ask for over all row lengths held in registers, with row counts at and
//                  around every size threshold, and the kernels that exist; whether they are the same
#include <stdio.h>
#include <string.h>

#include <initializer_list>
#include <set>
#include <string>
#include <tuple>

#include "direct_route.h"

using namespace addrms_host;

static const char* policy(int pol)
{
    static const char* const names[] = {"cached", "nontemporal", "writethrough", "shared"};
    return names[pol];
}

// The decision of addrms_run and its siblings for a call that names no configuration, with an empty table.
static std::string decide(const char* op, int dtype, int64_t M, int64_t N, uintptr_t x, uintptr_t r, uintptr_t w)
{
    const int o = !strcmp(op, "addrms") ? OP_ADDRMS : !strcmp(op, "silumul") ? OP_SILUMUL : OP_MERGE;
    addrms_cfg c{};
    std::string why;
    if (default_cfg(N, dtype, &c, &why, o) != ADDRMS_OK || check_cfg(c, M, N, dtype, o).status != ADDRMS_OK) return "refused";
    const uintptr_t al = static_cast<uintptr_t>(c.vec * x_bytes(dtype)), ral = o == OP_ADDRMS ? static_cast<uintptr_t>(c.vec * r_bytes(dtype)) : al;
    if (x % al || r % (ral < 16 ? ral : 16) || w % al) return "misaligned";
    DirectRoute p;
    bool yes;
    if (o == OP_ADDRMS) yes = direct_addrms_route(M, N, dtype, c.vec, x, r, w, &p);
    else if (o == OP_SILUMUL) yes = direct_silumul_route(M, N, dtype, x, r, &p);
    else yes = direct_mergestates_route(M, N, dtype, x | r | w, &p);
    if (!yes) return "default";
    char buf[160];
    if (p.long_row) snprintf(buf, sizeof buf, "long %s%s parked=%u", policy(p.pol), p.rag ? " ragged" : "", p.units);
    else if (o == OP_ADDRMS) snprintf(buf, sizeof buf, "row %s%s pieces=%d threads=%u rows=%u", policy(p.pol), p.rag ? " ragged" : "", p.cpt, p.block_x, p.block_y);
    else snprintf(buf, sizeof buf, "flat %s%s", policy(p.pol), p.rag ? " ragged" : "");
    return buf;
}

using Kernel = std::tuple<int, int, int, bool, bool>;                      // dtype, pieces, policy, ragged, shared workgroup

static int walk()
{
    std::set<Kernel> asked, exist;
    long n = 0;
    for (int dt : {ADDRMS_BF16, ADDRMS_FP16, ADDRMS_FP16_RES32, ADDRMS_FP32}) {
        const int vec = addrms::direct_vec(dt);
        for (int cpt = 1; cpt <= 8; ++cpt)
            for (int pol = 0; pol < 4; ++pol)
                for (bool rag : {false, true})
                    for (bool multi : {false, true})
                        if (addrms::direct_instance(vec, cpt, pol, rag, multi)) exist.insert({dt, cpt, pol, rag, multi});
        for (int64_t N = 16 * vec; N <= 32 * 1024; ++N) {
            const int64_t per = N * (x_bytes(dt) + r_bytes(dt));
            for (int64_t bytes : {512ll << 10, 1ll << 20, 2ll << 20, 3ll << 20, 4ll << 20, 16ll << 20, 96ll << 20, 300ll << 20})
                for (int64_t M : {bytes / per - 1, bytes / per, bytes / per + 1, int64_t(1), int64_t(511), int64_t(512)})
                    for (uintptr_t off : {uintptr_t(0), uintptr_t(x_bytes(dt))})
                        for (int default_vec : {1, 2}) {
                            DirectRoute p;
                            if (M < 1 || !direct_addrms_route(M, N, dt, default_vec, off, off / x_bytes(dt) * r_bytes(dt), off, &p) || p.long_row) continue;
                            ++n;
                            asked.insert({dt, p.cpt, p.pol, p.rag, p.block_y > 1});
                            // every piece of a row has a thread, at the first element's worst place in its line
                            const int64_t most = N + (p.rag ? 128 / x_bytes(dt) - 1 : 0);
                            if (p.block_x * p.block_y > 1024 || (p.block_x != 32 && p.block_x % 64) ||
                                int64_t(p.block_x) * p.cpt * vec < most || int64_t(p.grid) * p.block_y < M ||
                                int64_t(p.grid - 1) * p.block_y >= M || p.lds != (p.block_x > 64 ? p.block_y * 128u : 0u)) {
                                printf("bad shape: dtype %d M %lld N %lld\n", dt, (long long)M, (long long)N);
                                return 1;
                            }
                        }
        }
    }
    for (const Kernel& k : exist)
        if (!asked.count(k)) printf("never asked for: dtype %d pieces %d %s%s%s\n", std::get<0>(k), std::get<1>(k), policy(std::get<2>(k)),
                                    std::get<3>(k) ? " ragged" : "", std::get<4>(k) ? " shared" : "");
    for (const Kernel& k : asked)
        if (!exist.count(k)) printf("missing: dtype %d pieces %d %s%s%s\n", std::get<0>(k), std::get<1>(k), policy(std::get<2>(k)),
                                    std::get<3>(k) ? " ragged" : "", std::get<4>(k) ? " shared" : "");
    printf("%ld decisions, %zu kernels asked for, %zu exist\n", n, asked.size(), exist.size());
    return asked == exist ? 0 : 1;
}

int main(int argc, char**)
{
    if (argc > 1) return walk();
    char op[16];
    int dtype;
    long long M, N;
    unsigned long x, r, w;
    while (scanf("%15s %d %lld %lld %lu %lu %lu", op, &dtype, &M, &N, &x, &r, &w) == 7)
        printf("%s\n", decide(op, dtype, M, N, x, r, w).c_str());
    return 0;
}

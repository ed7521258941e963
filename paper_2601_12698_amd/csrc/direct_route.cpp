// Calls without a configuration: the rules.  Which kernel of direct_kernel.h a problem takes, and in what shape.
#include "direct_route.h"

#include <algorithm>

using namespace addrms;

namespace {

// Write-through stores up to this many bytes of output, non-temporal ones beyond: three eighths of the
// memory-side cache, so that the output is still there when the next kernel reads it.  Measured on buffers
// that a program cycles through (three sets) / on buffers from HBM, write-through against non-temporal, in us:
//   silu_and_mul  5.5 MB of traffic  2.3 / 3.0 against 2.9 / 2.8      49 MB   8.6 / 9.9 against 9.3 / 9.8
//               270 MB, 90 MB out   39.5 / 43.2 against 42.0 / 42.5  344 MB, 115 MB out  57.2 / 56.9 against 55.9 / 56.0
//              1057 MB, 352 MB out   171 / 170 against 168 / 166
//   add+RMSNorm (in place) 17 MB 6.3 / 7.0 against 6.3 / 6.6         67 MB  20.1 / 24.2 against 22.9 / 23.5
//               104 MB          34.9 / 37.6 against 34.8 / 34.9     235 MB  78.7 / 76.3 against 77.2 / 76.1
//   merge_attn_states  38 MB  7.4 / 8.6 against 7.6 / 8.3   24 MB  5.3 / 6.3 against 5.1 / 5.8
int64_t write_through_max() { return addrms_host::hw().last_level_cache_bytes / 8 * 3; }

void set_flat(addrms_host::DirectRoute* out, int64_t pieces, int64_t units, int64_t total)
{
    out->grid = static_cast<unsigned>((pieces + kFlatThreads - 1) / kFlatThreads);
    out->block_x = kFlatThreads;
    out->units = static_cast<unsigned>(units);
    out->total = static_cast<unsigned>(total);
    uint32_t l = 0;
    while ((1ll << l) < units) ++l;                           // ceil(log2 units)
    out->mul = static_cast<unsigned>(((1ull << (31 + l)) + static_cast<uint64_t>(units) - 1) / static_cast<uint64_t>(units));
    out->shift = l - 1;
}
constexpr int64_t kFlatMax = 1ll << 31;                       // positions the flat kernels divide exactly

// A launch has at most 2^32 - 1 threads.  With one thread per piece that is 137 GB of 16-bit rows, or half where a row
// fills half of its threads; what has more rows is left to the default configuration, whose threads take several pieces.
bool launchable(int64_t workgroups, int64_t threads) { return workgroups <= UINT32_MAX / threads; }

}  // namespace

namespace addrms_host {

// Rows that 32 values per thread of 1024 do not hold.  Ordinary loads and stores up to the size that the memory-side
// cache keeps (230 x 86912 bf16, 80 MB: 26.6 us against 31.6 with non-temporal ones; 8 x 123776 16.5 against 20.8),
// non-temporal beyond (1024 x 131072 bf16 210 us against 245).
static bool direct_addrms_long_route(int64_t M, int64_t N, int dtype, bool split, DirectRoute* out)
{
    const int vec = direct_vec(dtype), xb = x_bytes(dtype);
    const bool rag = split || (N * xb) % kLineBytes != 0, nt = M * N * (xb + r_bytes(dtype)) > write_through_max();
    const int64_t span = static_cast<int64_t>(kLongThreads) * vec, slot = span * 4;             // elements, LDS bytes per chunk
    const int64_t need = (N + (rag ? kLineBytes / xb - 1 : 0) + span - 1) / span;
    const int64_t fit = (hw().lds_bytes_per_cu - 128) / slot;                                   // behind one fp64 sum per wave
    out->units = static_cast<unsigned>(std::min(fit, std::max<int64_t>(0, need - kLongRegValues / vec)));
    if (!launchable(M, kLongThreads)) return false;
    out->pol = nt ? POL_NT : POL_CACHED;
    out->rag = rag;
    out->block_x = kLongThreads;
    out->grid = static_cast<unsigned>(M);
    out->lds = 128u + out->units * static_cast<unsigned>(slot);
    out->long_row = true;
    return true;
}

// Bytes of x and residual up to which rows with single elements are left to the default configuration.  Where its accesses
// are at least two elements wide, 1 MB (40 x 1030 bf16 3.2 us against 3.3), and half as much again or, for accesses of four,
// twice as much for 16-bit rows under 1024 elements, which its 256 threads hold in one access or two each (us, this against
// the walk: 268 x 932 bf16 3.1 / 3.5, 536 x 932 3.4 / 3.6, 804 x 932 the same; 500 x 514 3.0 / 3.1, 1000 x 514 the same).
// Where they are one element, 1 MB for 16-bit rows so short that its many threads are ahead of the few pieces (380 x 131
// bf16 2.6 / 2.8; 579 x 259 the same).
static int64_t ragged_min(int vec, int default_vec, int64_t N)
{
    constexpr int64_t kMB = 1 << 20;
    if (default_vec > 1) return vec == 8 && N < 128 * vec ? (default_vec > 2 ? 2 * kMB : kMB + kMB / 2) : kMB;
    return vec == 8 && N < 32 * vec ? kMB : 0;
}

// Threads per row: one per piece up to 1024, then as few pieces per thread as that allows, in equal shares: on 40 shapes
// tried with 1 to 8 the fewest were the fastest, by 2-8 % against twice as many.  Written-through rows of more than 256
// pieces take at least two, which then are stored in one go after the row sum (256 x 8192 bf16 4.0 us against 4.2 and from
// HBM 4.4 against 5.6; 512 x 8192 5.8 against 6.5; 4096 x 4096 the same; shorter rows 1-2 % slower).
// Ragged rows from 4 MB (single elements) or 16 MB to 96 MB take three pieces per thread (two where there are no single
// elements: 8192 x 1000 fp16+fp32 17.1 us against 17.5) and two rows per workgroup, so that fewer waves repeat what a
// row costs before and after its pieces (2047 x 4095 fp16 12.9 us against 14.0 with one piece per thread, 5000 x 1001
// fp32 15.5 against 16.0, 4285 x 700 bf16 6.5 against 7.3); beyond, one is as good or better (9000 x 6150 bf16 76.4-79.7 us
// against 78.1-78.9), and so it is below, where the chip is not full and a row should arrive early (41 x 6001 bf16 3.2-3.3
// us against 3.8-4.0, 1072 x 932 3.9-4.0 against 3.8-4.2).
// Store policy: as above, but non-temporal below 512 KB of x and residual, where the launch is all there is and a
// write-through store only waits longer (16 x 4096 bf16 2.2 us against 2.4; from 1 MB on write-through wins, 64 x 8192
// 2.9 against 3.4), and for rows with single elements, whose partly written lines a write-through store sends out at
// once (2047 x 4095 fp16 12.9 us and from HBM 13.5 against 13.3 and 15.9).
// Rows of whole vectors that are not whole lines: where waves share lines with the waves beside them, a non-temporal load
// gives up a line that the next wave still wants, and a non-temporal store sends out half of one.  They take ordinary loads
// and write-through stores at every size from 512 KB on: rows that are not walked by lines, whose every wave shares two,
// and walked ones of up to 3 KB of x, where the lines at a row's ends are one in twelve or more.  On three buffer sets /
// from HBM, us, the knob grid's default, non-temporal loads (with the stores of the size), this:
//   124 x 30008 fp16 (15 MB)              7.5 / 11.1       8.5 / 12.3      6.7 / 9.1    (7.5, 8.5, 6.7: one set)
//   22500 x 1000 bf16 (90 MB)            32.2 / 35.6      31.9 / 40.6     28.0 / 31.7
//   108333 x 200 fp16+fp32 (130 MB)      48.8 / 49.8      51.2 / 51.8     43.9 / 43.8
//   228658 x 328 bf16 (300 MB)          113.3 / 112.0    125.8 / 125.4    99.7 / 99.7
//   500000 x 100 fp32 (400 MB)          136.2 / 136.0    151.2 / 151.0   133.5 / 133.3
// Longer walked rows (2056 bf16, 400 MB: 127.4 against 130.3 with this; 10008 fp16, 250 MB: 82.5 against 88.4) keep the
// policy of their size.
// Ragged walk: where a vector access does not divide the row, unless it is small and the default configuration's accesses
// reach (ragged_min); and where rows are whole
// vectors but not whole lines, from 16 MB on (below, 1000 x 1000 bf16 3.6 us against 3.5) and from 64 pieces a row on
// (22500 x 1000 bf16 28.0 us and from HBM 31.7 against 30.6 and 34.9; 28846 x 520 19.6 / 24.3 against 19.8 / 21.7; 31492 x
// 516 fp32 45.3 / 44.9 against 47.0 / 46.5; shorter rows lose: 108333 x 200 fp16+fp32 56.1 / 56.3 against 43.9 / 43.8).
// A default configuration with narrower accesses than these admits bases that they do not (86912 fp32: two elements per
// access): such rows take the ragged walk, whole vectors or not.
bool direct_addrms_route(int64_t M, int64_t N, int dtype, int default_vec, uintptr_t x, uintptr_t r, uintptr_t w, DirectRoute* out)
{
    constexpr int64_t kWriteThroughMin = 512 << 10, kThreePiecesMin = 4 << 20, kLineWalkMin = 16 << 20, kSharedLinesRow = 3072;
    const int vec = direct_vec(dtype), xb = x_bytes(dtype), rb = r_bytes(dtype);
    const int64_t bytes = M * N * (xb + rb);
    const bool split = N % vec != 0 || x % (vec * xb) != 0 || r % (vec * rb) != 0 || w % (vec * xb) != 0;   // single elements
    const bool partial_lines = (N * xb) % kLineBytes != 0;
    const bool rag = split || (partial_lines && bytes >= kLineWalkMin && N >= 64 * vec);
    if (split && ((x / xb) % vec != (r / rb) % vec || bytes < ragged_min(vec, default_vec, N))) return false;
    const int line = kLineBytes / xb;                                                 // elements
    const int64_t pieces = (N + (rag ? line - 1 : 0) + vec - 1) / vec;                // a ragged row begins anywhere in a line
    if (N < 16 * vec) return false;
    if (pieces * vec > 32 * 1024) return direct_addrms_long_route(M, N, dtype, split, out);
    const bool shared_lines = partial_lines && !split && (!rag || N * xb <= kSharedLinesRow);
    const int pol = split || bytes < kWriteThroughMin ? POL_NT : shared_lines ? POL_SHARED : bytes <= write_through_max() ? POL_WT : POL_NT;
    const bool thick = rag && bytes <= write_through_max();
    const int64_t thickness = split ? (thick && bytes >= kThreePiecesMin ? 3 : 1) : thick || (pol == POL_WT && pieces > 256) ? 2 : 1;
    int64_t cpt = std::max<int64_t>((pieces + 1023) / 1024, thickness);
    int64_t tpr = (pieces + cpt - 1) / cpt;
    tpr = tpr <= 32 ? 32 : (tpr + 63) / 64 * 64;
    cpt = (pieces + tpr - 1) / tpr;
    out->block_x = static_cast<unsigned>(tpr);
    out->block_y = tpr == 32 || (thick && tpr <= 256 && M >= 512) ? 2u : 1u;
    if (vec == 4 && cpt > 4) cpt = (cpt + 1) / 2 * 2;                                 // 5 to 8: the kernels of 6 and 8 pieces
    out->cpt = static_cast<int>(cpt);
    out->pol = pol;
    out->rag = rag;
    if (!direct_instance(vec, out->cpt, pol, rag, out->block_y > 1)) return false;    // never: the tests walk the rules
    const int64_t workgroups = (M + out->block_y - 1) / out->block_y;
    if (!launchable(workgroups, tpr * out->block_y)) return false;
    out->grid = static_cast<unsigned>(workgroups);
    out->lds = tpr > 64 ? out->block_y * 16u * 8u : 0u;        // one fp64 sum per wave
    return true;
}

bool direct_silumul_route(int64_t M, int64_t d, int dtype, uintptr_t x_align, uintptr_t out_align, DirectRoute* out)
{
    const int es = x_bytes(dtype), vec = 16 / es;
    const bool rag = d % vec != 0;
    if (d < 2 * vec || M >= kFlatMax / d) return false;       // rows of one piece have no division; 32-bit positions
    if (out_align % 16 != 0 || (!rag && x_align % 16 != 0)) return false;
    out->pol = M * d * es <= write_through_max() ? POL_WT : POL_NT;
    out->rag = rag;
    if (rag) set_flat(out, (M * d + vec - 1) / vec, d, M * d);
    else set_flat(out, M * (d / vec), d / vec, M * (d / vec));
    return true;
}

// Below 4 MB of traffic the row kernels' ordinary loads are as fast (2000 x 80 bf16: 2.3 us against 2.5): the launch
// is all there is.
bool direct_mergestates_route(int64_t rows, int64_t d, int dtype, uintptr_t v_align, DirectRoute* out)
{
    constexpr int64_t kSmall = 4 << 20;
    const int vec = 16 / x_bytes(dtype);
    if (d % vec != 0 || d < 2 * vec || rows >= kFlatMax / d || v_align % 16 != 0) return false;
    if (algorithmic_bytes(OP_MERGE, rows, d, dtype) < kSmall) return false;
    out->pol = rows * d * x_bytes(dtype) <= write_through_max() ? POL_WT : POL_NT;
    set_flat(out, rows * (d / vec), d / vec, rows * (d / vec));
    return true;
}

}  // namespace addrms_host

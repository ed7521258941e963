// Calls without a configuration: the rules.  Which kernel of direct_kernel.h a problem takes, and in what shape.
//
// Times in this file are microseconds per launch, back to back in a graph, all taken on one card in one run: on one set of
// buffers / on three in rotation / on buffers from HBM; or the last two, or the last one, where the others say nothing.
#include "direct_route.h"

#include <algorithm>

using namespace addrms;

namespace {

// Write-through stores up to this many bytes of output, non-temporal ones beyond: three eighths of the memory-side cache,
// so that the output is still there when the next kernel reads it.  Write-through against non-temporal:
//   add+RMSNorm N = 4096 bf16, in place  17 MB  6.5 /  6.4 /  8.0 against  6.0 /  6.9 /  7.6
//                                        67 MB 20.0 / 19.8 / 23.5 against 21.4 / 22.5 / 23.5
//                                       105 MB 29.9 / 35.5 / 35.4 against 33.0 / 34.7 / 35.3
//                                       235 MB 64.6 / 75.3 / 75.1 against 72.9 / 73.8 / 74.8
//   silu_and_mul d = 11008 bf16, by its  24 MB  3.8 /  4.5 /  5.6 against  4.6 /  5.1 /  5.3
//   traffic, a third of it output        67 MB  9.1 / 11.2 / 11.9 against 11.2 / 12.0 / 12.2
//                                       235 MB 33.8 / 34.0 / 37.3 against 36.3 / 37.0 / 36.8
//                                       400 MB 56.1 / 63.3 / 63.0 against 62.0 / 62.7 / 62.3
//   merge_attn_states d = 256 bf16,      24 MB  3.7 /  5.2 /  6.2 against  4.9 /  5.3 /  5.7
//   by its traffic                       67 MB 10.2 / 12.8 / 13.4 against 11.4 / 12.5 / 13.1
//                                       235 MB 36.2 / 36.5 / 39.4 against 38.1 / 39.2 / 39.6
// Neither is ahead on all buffers, and neither always beats ordinary accesses: where all that a program touches between two
// calls comes to 100 to 250 MB, and so just about fits the memory-side cache, these keep more of it there.  The default
// configuration then is ahead by up to 10 % on merges of 40 to 120 MB (67 MB: 11.7 / 11.6 / 15.2), by up to 20 % on norms
// called again and again on one set of 96 to 250 MB (N = 4096, 150 MB: 44.0 / 54.7 / 56.1 against 47.8 / 48.9 / 49.2) or of
// 16 to 40 MB, in the L2s, and there by up to 35 % on the longest rows where they are not split (166 x 120004 fp32 51
// against 69; split 55).  From HBM it is 10 to 20 % behind on all of these.
using addrms_host::write_through_max;

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

// Long rows split over workgroups (addrms_split_body), where the launch can have units.  16384 elements to a part where a
// thread has eight to a piece, 12288 where it has four: four pieces per thread of 512 or 768 threads, of which a CU holds two
// (1024 x 131072 bf16 in 4 / 8 / 16 parts 183 / 173 / 180; 500 x 200000 fp32 in 13 / 17 / 25 of four pieces 265 / 259 / 271).  Fewer rows
// than that keeps the chip busy with are cut finer, down to 512 pieces, up to 512 workgroups in all, with as few pieces per
// thread as 1024 threads allow (46 x 164992 fp16 in 6 / 11 / 21 parts 17.8 / 12.2 / 14.4; 1 x 200000 in 8 / 12 / 16 7.5 / 7.2 / 6.4).
// Against one workgroup per row, on three sets / from HBM (and the numbers of parts above: measured when meeting took 0.7 to 3 us
// more than it does now, 1 x 200000 4.8, 1024 x 131072 170.5):
//   1 x 200000 bf16   23.9 / 28.7  ->  6.4 / 6.3        2048 x 65536     195.7 / 195.5 -> 174.0 / 174.3
//   8 x 123776        14.8 / 18.3  ->  6.4 / 6.4        4096 x 40960     228.4 / 227.8 -> 214.7 / 214.5
//   60 x 131072       20.2 / 30.3  -> 12.5 / 12.7       500 x 200000 fp32 354 / 354 -> 274 / 274
//   1024 x 131072    207.3 / 211.3 -> 171.6 / 172.0     512 x 81920 fp32 130.6 / 131.0 -> 111.9 / 111.7
// Left to one workgroup per row: rows that it holds (nothing is read twice), in numbers that give nearly every CU one or two,
// while all of it fits the memory-side cache, whose contents ordinary accesses keep (192 x 40960 bf16 0.68 / 0.96 of the time, 224 x
// 65536 0.88 / 1.15, 512 x 40960 0.94 / 1.12; beside them 128 x 65536 1.10 / 1.41, 288 x 40960 1.02 / 1.24, 640 x 49152 1.01 / 1.01).
// And 16-bit rows of whole lines that its registers hold without LDS, where the CUs' last turn at them is not too empty, up to
// as many turns as it is ahead; split / whole, us on three sets:
//             350 rows     447          560          650          768          900          1000
//   32832     18.8 / 18.0  22.5 / 21.1  27.1 / 27.2  32.6 / 32.1  40.7 / 38.4  46.2 / 44.3  50.4 / 48.9
//   36864     20.4 / 19.1  24.1 / 22.3  30.5 / 30.2  39.9 / 36.1  44.3 / 42.2  50.1 / 49.0  55.0 / 53.8
//   40960     21.9 / 20.4  26.2 / 24.1  36.5 / 34.1  40.9 / 39.8  46.8 / 45.8  53.6 / 54.0  58.7 / 59.1
//   49152     24.3 / 23.7  33.1 / 32.0  41.8 / 42.9  47.5 / 47.5  54.2 / 55.5  62.8 / 65.1  69.0 / 71.8
// (300 rows 16.5 / 16.9 to 20.9 / 21.7, 513 24.8 / 25.9 to 38.5 / 41.4; 1300 x 40960 73.9 / 77.4; ragged ones, which share lines with
// their neighbours, 350 x 33333 20.6 / 21.8, 800 42.8 / 48.3; 32-bit ones 350 x 32832 33.7 / 35.2, 800 73.4 / 80.4).
// Stores: write-through between 32 MB of x and residual and the limit above, non-temporal below and beyond (84 MB, 336 x 62528 bf16
// 30.5 / 35.3 against 34.2 / 34.9; 30 MB, 46 x 164992 fp16 15.2 / 17.4 against 16.4 / 17.2; 20 MB, 100 x 50000 10.1 / 11.1
// against 9.8 / 10.4; 400 MB, 500 x 200000 fp32 284.9 against 274.5).
static void direct_addrms_split(int64_t M, int64_t N, int dtype, DirectRoute* out)
{
    constexpr int64_t kBusy = 512, kFinest = 512, kNonTemporalMax = 32 << 20;
    const int vec = direct_vec(dtype), xb = x_bytes(dtype), cus = hw().compute_units;
    const int64_t bytes = M * N * (xb + r_bytes(dtype));
    const int64_t pieces = (N + (out->rag ? kLineBytes / xb - 1 : 0) + vec - 1) / vec;
    const bool held = pieces <= static_cast<int64_t>(kLongThreads) * (kLongRegValues / vec + out->units);
    const bool filling = M <= cus ? M >= cus / 8 * 5 : M <= 2 * cus && M >= cus / 4 * 7;
    if (held && filling && bytes <= write_through_max()) return;
    const int64_t turns = (M + cus - 1) / cus, most = pieces <= 4608 ? 4 : pieces <= 5120 ? 3 : 2;
    const int64_t tenths = turns == 2 ? 3 : turns == 3 ? 1 : 0;                       // of the CUs, in the last turn
    if (vec == 8 && !out->rag && out->units == 0 && turns > 1 && turns <= most && 10 * (M - (turns - 1) * cus) >= tenths * cus) return;
    const int64_t coarse = vec == 8 ? 2048 : 3072;                                    // pieces of a part
    int64_t parts = (pieces + coarse - 1) / coarse;
    parts = std::max(parts, std::min((pieces + kFinest - 1) / kFinest, kBusy / M));
    parts = std::min<int64_t>(parts, kSplitParts);
    const int64_t per = (pieces + parts - 1) / parts;
    const int64_t cpt = M * parts > kBusy || per > 2048 ? 4 : per > 1024 ? 2 : 1;
    const int64_t threads = ((per + cpt - 1) / cpt + 63) / 64 * 64;
    if (threads > 1024) return;                                                       // rows beyond 16 parts of the largest size
    parts = (pieces + threads * cpt - 1) / (threads * cpt);
    if (parts < 2) return;
    out->parts = static_cast<unsigned>(parts);
    out->part_threads = static_cast<unsigned>(threads);
    out->part_cpt = static_cast<int>(cpt);
    out->part_pol = bytes <= kNonTemporalMax || bytes > write_through_max() ? POL_NT : POL_WT;
}

// Rows that 32 values per thread of 1024 do not hold.  Ordinary loads and stores up to the size that the memory-side
// cache keeps (230 x 86912 bf16, 80 MB: 24.5 against 31.6 with non-temporal ones on three sets), non-temporal beyond
// (1525 x 40960 bf16, 250 MB: 87.2 / 87.5 / 87.6 against 77.1 / 99.4 / 99.6; 114 x 175104 fp32, 160 MB: 78.2 / 81.6 / 91.2
// against 60.4 / 100.4 / 99.4).
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
    direct_addrms_split(M, N, dtype, out);
    return true;
}

// Bytes of x and residual up to which rows with single elements are left to the default configuration.  Where its accesses
// are at least two elements wide, 1 MB, and half as much again or, for accesses of four, twice as much for 16-bit rows under
// 1024 elements, which its 256 threads hold in one access or two each.  This against the walk, on three sets / from HBM:
// 268 x 932 bf16 3.0 / 3.2 against 3.6 / 3.4, 536 x 932 3.3 / 3.5 against 3.8 / 3.7, 804 x 932 3.6 / 4.3 against 4.0 / 3.9;
// 500 x 514 3.3 / 3.4 against 3.8 / 3.6, 1000 x 514 3.7 / 3.9 against 4.0 / 3.9; 242 x 1030 3.4 / 3.6 against 3.6 / 3.4.
// Where they are one element, 1 MB for 16-bit rows so short that its many threads are ahead of the few pieces (380 x 131
// bf16 2.9 / 2.6 against 3.4 / 3.2; 579 x 259 3.3 / 3.4 against 3.5 / 3.5, and as single launches the same).
static int64_t ragged_min(int vec, int default_vec, int64_t N)
{
    constexpr int64_t kMB = 1 << 20;
    if (default_vec > 1) return vec == 8 && N < 128 * vec ? (default_vec > 2 ? 2 * kMB : kMB + kMB / 2) : kMB;
    return vec == 8 && N < 32 * vec ? kMB : 0;
}

// Rows that the registers of one workgroup hold, up to so many at a time, are split like long ones: a CU that has a row of 100 to 260 KB
// to itself takes 2 us and more to read and write it.  Formats of four elements per piece only; one workgroup / split, us on three
// sets (fp16+fp32 gains a tenth less, with 80 rows of 16416 and 50 of 18000 nothing):
//   fp32       1 row          8            16           32           64           80           96           128
//   12288      3.62 / 3.44                 4.07 / 3.87  4.17 / 4.45  4.46 / 5.09
//   14336      3.81 / 3.64    4.70 / 3.71  4.72 / 3.97  4.81 / 4.34  5.10 / 5.12  5.27 / 5.51  5.46 / 5.86  5.95 / 6.59
//   16448      4.31 / 3.82    5.26 / 3.97  5.29 / 4.14  5.43 / 4.76  5.82 / 5.39  6.05 / 5.67  6.27 / 6.09  6.92 / 7.14
//   20480      4.83 / 3.84    5.59 / 3.96  5.74 / 4.29  5.91 / 4.87  6.27 / 5.57  6.51 / 6.12  6.79 / 6.81  7.81 / 7.98
//   24577      5.63 / 4.17    6.43 / 4.42  7.06 / 4.70  7.97 / 5.47  9.00 / 6.25  9.24 / 7.22  9.50 / 7.87  10.4 / 9.39
//   28672      6.31 / 4.05    7.25 / 4.28  7.26 / 4.56  7.49 / 5.35  8.00 / 6.33  8.28 / 7.30  8.74 / 8.10  10.3 / 10.1
//   32768      6.44 / 4.10    7.78 / 4.29  8.16 / 4.71  8.03 / 5.56  8.74 / 6.87  9.18 / 7.83  9.63 / 8.90  11.4 / 11.3
// More rows than CUs gain up to 8 % split where they are ragged and lose up to 17 % otherwise (400 x 16448 17.5 / 21.1).
void direct_addrms_split_few(int64_t M, int64_t N, int dtype, DirectRoute* out)
{
    const int64_t cus = hw().compute_units, pieces = (N + (out->rag ? kLineBytes / x_bytes(dtype) - 1 : 0) + 3) / 4;
    const int64_t most = pieces > 7168 ? cus / 2 : pieces > 6144 ? cus / 8 * 3 : pieces > 5120 ? cus / 16 * 5 : pieces > 4096 ? cus / 32 * 5 :
                         pieces > 3072 ? cus / 16 : 0;
    if (direct_vec(dtype) == 4 && M <= most) direct_addrms_split(M, N, dtype, out);
}

// Threads per row: one per piece up to 1024, then as few pieces per thread as that allows, in equal shares: on 40 shapes
// tried with 1 to 8 the fewest were the fastest, by 2-8 % against twice as many.  Written-through rows of more than 256
// pieces take at least two, which then are stored in one go after the row sum (256 x 8192 bf16 4.0 / 4.2 against 4.2 / 5.3,
// 512 x 8192 5.8 / 7.3 against 6.6 / 8.3, 4096 x 4096 19.9 / 23.5 against 19.8 / 23.4; 1000 x 2048, of 256 pieces, 3.7 / 4.6
// against 3.6 / 4.6).
// Rows with single elements from 4 to 96 MB take three pieces per thread, and from 512 rows on two rows per workgroup where
// that is at most 512 threads, so that fewer waves repeat what a row costs before and after its pieces.  One piece, three,
// three and two rows: 2047 x 4095 fp16 13.5 / 14.0 / 12.6 on three sets, 2000 x 2001 bf16 8.3 / 7.2 / 7.0, 2000 x 6001 18.4 /
// 19.3 / 18.1, 5000 x 1001 fp32 15.4 / 15.8 / 15.5; 4285 x 700 bf16 7.3 with one piece, 6.4-6.6 here.  With few rows one row
// per workgroup is as good (513 x 4001 5.3 / 5.3, 300 x 10001 6.7 / 6.8), and so it is with more threads (2000 x 10001 31.1 /
// 31.7).  Below 4 MB, where the chip is not full and a row should arrive early, one piece is ahead (41 x 6001 bf16 3.5
// against 4.2, 1072 x 932 4.2 against 4.3), and beyond 96 MB too (9000 x 6150 72.8 against 75.7).
// Rows walked by lines that are whole vectors take two pieces and two rows up to 96 MB by the same rule (3000 x 2056 bf16
// 9.6 / 11.7 against 10.5 / 11.6 with one and one, 6144 x 1000 8.7 / 10.8 against 9.0 / 10.9, 8192 x 1000 fp16+fp32 the same).
// Store policy: as above, but non-temporal below 512 KB of x and residual, where the launch is all there is (16 x 4096 bf16
// 2.3 / 2.3 against 2.5 / 2.3); between that and 4 MB non-temporal stores are 0.2 faster on three sets and 0.2 slower from
// HBM.  And non-temporal for rows with single elements, whose partly written lines a write-through store sends out at once
// (2047 x 4095 fp16 12.4 / 13.2 against 13.7 / 15.2, 300 x 10001 bf16 6.5 / 6.8 against 7.1 / 8.9).
// Rows of whole vectors that are not whole lines: where waves share lines with the waves beside them, a non-temporal load
// gives up a line that the next wave still wants, and a non-temporal store sends out half of one.  They take ordinary loads
// and write-through stores at every size from 512 KB on: rows that are not walked by lines, whose every wave shares two,
// and walked ones of up to 3 KB of x, where the lines at a row's ends are one in twelve or more.  The knob grid's default,
// non-temporal loads (with the stores of the size), this:
//   124 x 30008 fp16 (15 MB)              8.6 / 11.3       8.5 / 12.3      6.9 / 9.2
//   22500 x 1000 bf16 (90 MB)            31.2 / 35.6      31.9 / 40.6     27.7 / 31.9
//   108333 x 200 fp16+fp32 (130 MB)      49.2 / 50.2      51.2 / 51.8     43.8 / 44.1
//   228658 x 328 bf16 (300 MB)          113.6 / 113.0    125.8 / 125.4    99.6 / 99.1
//   500000 x 100 fp32 (400 MB)          139.2 / 136.7    151.2 / 151.0   132.2 / 132.5
// Longer walked rows (2056 bf16, 400 MB: 127.4 against 130.3 with this; 10008 fp16, 250 MB: 82.5 against 88.4) keep the
// policy of their size.
// Ragged walk: where a vector access does not divide the row, unless it is small and the default configuration's accesses
// reach (ragged_min); and where rows are whole vectors but not whole lines, from 16 MB on and from 64 pieces a row on.  With
// and without it, 1000 bf16: 4 MB 3.2 / 3.5 against 3.0 / 3.4, 8 MB 3.9 / 5.1 against 3.7 / 4.9, 16 MB 6.5 / 7.9 against 6.6 /
// 8.7, 25 MB 8.8 / 10.9 against 9.0 / 11.7, 50 MB 15.9 / 18.9 against 16.6 / 20.7; for 4680 fp16 the line is less clear (25 MB
// 9.8 / 11.4 against 9.2 / 11.6, 50 MB 16.9 / 19.9 against 16.2 / 20.1).  Rows of fewer pieces lose with it (108333 x 200
// fp16+fp32 56.1 / 56.3 against 43.9 / 43.8; 31492 x 516 fp32 gains, 45.3 / 44.9 against 47.0 / 46.5).
// A default configuration with narrower accesses than these admits bases that they do not (86912 fp32: two elements per
// access): such rows take the ragged walk, whole vectors or not.
// Single elements are read with ordinary loads, which leave their lines for the pieces beside them and for the row that shares the
// line, but where x and residual have 16 to 36 MB and rows are longer than 3 KB of x, or 16 to 64 MB and 16 KB.  Non-temporal
// against ordinary on three sets: 74751 x 301 fp16 45.6 / 34.7, 32467 x 693 bf16 38.9 / 32.2, 12000 x 501 12.0 / 10.8, 22522 x 999 fp16 35.8 /
// 32.0, 513 x 4001 bf16 5.05 / 4.79, 488 x 4095 fp16 4.79 / 4.49, 244 x 4095 fp32 4.56 / 4.23; but 2014 x 4095 fp16 12.4 / 12.9, 1007 x 8191 12.9 /
// 13.1, 503 x 16383 12.5 / 12.8, 2015 x 2047 fp32 12.0 / 12.2.  By size, 4095 fp16: 12 MB 1.03 times as fast, 16 MB 1.03, 20 MB 0.97, 24 MB
// 0.96, 28 MB 0.99, 40 MB 1.01, 100 MB 1.02; 16383 fp16: 1.03, 1.03, 1.00, 0.99, 0.98, 0.99, and 64 MB 1.00.  From HBM the same from 24 MB
// on (74751 x 301 46.3 / 35.1), 0.98 to 1.04 below.  Rows split over workgroups,
// 300 x 33333 bf16: 17.5 / 16.8, and 16.5 with ordinary stores of them too, which change nothing in rows that are not split.
bool direct_addrms_route(int64_t M, int64_t N, int dtype, int default_vec, uintptr_t x, uintptr_t r, uintptr_t w, DirectRoute* out)
{
    constexpr int64_t kWriteThroughMin = 512 << 10, kThreePiecesMin = 4 << 20, kLineWalkMin = 16 << 20, kSharedLinesRow = 3072;
    constexpr int64_t kKeepMin = 36 << 20, kKeepLongRow = 16000, kKeepLongMin = 64 << 20;
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
    out->keep_shared = N * xb <= kSharedLinesRow || bytes <= kLineWalkMin || bytes > (N * xb >= kKeepLongRow ? kKeepLongMin : kKeepMin);
    if (!direct_instance(vec, out->cpt, pol, rag, out->block_y > 1)) return false;    // never: the tests walk the rules
    const int64_t workgroups = (M + out->block_y - 1) / out->block_y;
    if (!launchable(workgroups, tpr * out->block_y)) return false;
    out->grid = static_cast<unsigned>(workgroups);
    out->lds = tpr > 64 ? out->block_y * 16u * 8u : 0u;        // one fp64 sum per wave
    return true;
}

// Ragged rows, whose waves share the lines at their ends, are read with ordinary loads up to 26 MB of output.  Non-temporal against
// these on three sets / from HBM: 4073 x 1023 bf16 (25 MB of traffic) 5.6 / 6.6 against 5.2 / 6.5, 8146 x 1023 9.9 / 10.8 against 8.4 / 10.6, 1525 x 8191
// 13.4 against 11.9, 2033 x 4099 9.7 / 10.6 against 8.4 / 10.6, 4073 x 1023 fp32 9.2 / 10.4 against 8.3 / 10.5; 16293 x 1023 bf16 (100 MB) 17.4
// against 17.9.  (add+RMSNorm gains as much on three sets, and loses 10 to 20 % from HBM.)
bool direct_silumul_route(int64_t M, int64_t d, int dtype, uintptr_t x_align, uintptr_t out_align, DirectRoute* out)
{
    constexpr int64_t kKeepMax = 26 << 20;
    const int es = x_bytes(dtype), vec = 16 / es;
    const bool rag = d % vec != 0;
    if (d < 2 * vec || M >= kFlatMax / d) return false;       // rows of one piece have no division; 32-bit positions
    if (out_align % 16 != 0 || (!rag && x_align % 16 != 0)) return false;
    out->pol = M * d * es <= write_through_max() ? POL_WT : POL_NT;
    out->rag = rag;
    out->keep_shared = rag && M * d * es <= kKeepMax;
    if (rag) set_flat(out, (M * d + vec - 1) / vec, d, M * d);
    else set_flat(out, M * (d / vec), d / vec, M * (d / vec));
    return true;
}

// Below 4 MB of traffic the row kernels' ordinary loads are as fast or faster: this on three sets / from HBM against them,
// d = 256 bf16: 2 MB 2.4 / 2.4 against 2.2 / 2.3, 4 MB 2.6 / 2.9 against 2.4 / 3.2, 6 MB 2.8 / 3.1 against 2.6 / 3.9,
// 8 MB 2.6 / 3.4 against 2.8 / 4.4.
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

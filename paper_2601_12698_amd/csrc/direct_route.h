// Calls without a configuration: which kernel of direct_kernel.h a problem takes, and in what shape.  Host code only, no
// HIP; the rules are in direct_route.cpp, the kernels they name are instantiated in addrms_direct.hip.
#pragma once
#include <stdint.h>

#include "addrms_internal.h"

namespace addrms {

// Loads and stores.  POL_CACHED: ordinary.  POL_NT: both non-temporal.  POL_WT: non-temporal loads, write-through stores.
// POL_SHARED: ordinary loads, write-through stores, for waves that share cache lines with the waves beside them.
enum : int { POL_CACHED = 0, POL_NT = 1, POL_WT = 2, POL_SHARED = 3 };

constexpr int kFlatThreads = 256;
// Workgroups of 1024 threads leave each 128 registers: 48 values of the row stay there.  (512 threads with 144 values
// each: 204 us against 210 on 1024 x 131072 bf16, but 68 against 58 on 300 x 110592 and 27 against 20 on 8 x 123776.)
constexpr int kLongThreads = 1024, kLongRegValues = 48;

// Elements per thread and access: 16 bytes of the residual, and of x too unless the residual is wider.
constexpr int direct_vec(int dtype) { return dtype == ADDRMS_BF16 || dtype == ADDRMS_FP16 ? 8 : 4; }

// The add+RMSNorm kernels with the row in registers that the rules can ask for: at most 32 values per thread, because a
// workgroup of 1024 threads leaves each 128 registers.  Rows of whole vectors share a workgroup only where 32 threads
// take one piece each; walks by lines with write-through stores have at least two pieces per thread, and exactly two
// where rows share a workgroup; with ordinary loads two in a shared workgroup and one otherwise.
constexpr bool direct_instance(int vec, int cpt, int pol, bool rag, bool multi)
{
    if (pol == POL_CACHED || cpt < 1 || (vec == 8 ? cpt > 4 : cpt > 4 && cpt != 6 && cpt != 8)) return false;
    if (rag && pol == POL_SHARED) return cpt == (multi ? 2 : 1);
    if (rag) return pol == POL_WT ? (multi ? cpt == 2 : cpt >= 2) : (!multi || cpt <= 3);
    return !multi || cpt == 1;
}

constexpr int kSplitRows = 4096;                             // rows of one launch of split rows; more are several launches
// The memory that they meet in: units of 64 rows (24 KB), 24 MB in all.  A long row is at least 32769 elements long, 42 ns of
// bf16 at 6.2 TB/s, so that all units are taken no sooner than 2.7 ms of such launches are in flight.  The same of few wide rows on one
// stream: launches of one unit take 3.3 us and more, of two 5.4.
constexpr int kSplitUnits = 1024, kSplitUnitRows = 64;
constexpr int kSplitParts = 16;                              // workgroups a row may be split over
// The kernels of split rows: pieces per thread and store policy.  With fewer than four pieces 512 workgroups are within 32 MB.
constexpr bool split_instance(int cpt, int pol) { return cpt == 4 ? pol == POL_NT || pol == POL_WT : (cpt == 1 || cpt == 2) && pol == POL_NT; }

}  // namespace addrms

namespace addrms_host {

// A launch that is ready but for the kernel's address and the pointers.
struct DirectRoute {
    int pol = 0;                                            // as above
    int cpt = 0;                                            // pieces per thread (rows in registers)
    bool rag = false;                                       // ragged: see direct_kernel.h
    bool keep_shared = false;                               // ragged rows: ordinary loads of single elements; silu_and_mul: of all
    bool long_row = false;                                  // rows beyond the registers: units = chunks parked in LDS
    unsigned grid = 0, block_x = 0, block_y = 1, lds = 0;   // block_y: rows of a workgroup
    unsigned units = 0, total = 0, mul = 0, shift = 0;      // flat operators: see direct_kernel.h
    // Rows that are split over workgroups where the launch can have units (slot_map.h): long ones, and few ones in registers; the rest
    // of the route is what runs where it cannot.
    unsigned parts = 0, part_threads = 0;                   // 0: not split
    int part_cpt = 0, part_pol = 0;
};

// False: the default configuration runs.  x, r, w: the tensors' bases, aligned as the default configuration (of
// default_vec elements per access) asks for; *_align: bases or-ed together.
bool direct_addrms_route(int64_t M, int64_t N, int dtype, int default_vec, uintptr_t x, uintptr_t r, uintptr_t w,
                         DirectRoute* out);
// For a route of rows in registers: splits them where they are few and wide.
void direct_addrms_split_few(int64_t M, int64_t N, int dtype, DirectRoute* out);
bool direct_silumul_route(int64_t M, int64_t d, int dtype, uintptr_t x_align, uintptr_t out_align, DirectRoute* out);
bool direct_mergestates_route(int64_t rows, int64_t d, int dtype, uintptr_t v_align, DirectRoute* out);

}  // namespace addrms_host

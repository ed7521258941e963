// Launches without a configuration (kernels in direct_kernel.h, rules in direct_route.cpp).
#pragma once
#include <stdint.h>

#include "direct_route.h"

namespace addrms_host {

// A launch that is ready but for the pointers.
struct DirectPlan : DirectRoute {
    const void* fn = nullptr;
    const void *split_fn = nullptr, *alone_fn = nullptr;    // of DirectRoute::parts
    unsigned long_index = 0;                                // which of the kernels for rows beyond the registers
};

// Arguments as in direct_route.h.
bool direct_addrms_plan(int64_t M, int64_t N, int dtype, int default_vec, uintptr_t x, uintptr_t r, uintptr_t w,
                        DirectPlan* out);
bool direct_silumul_plan(int64_t M, int64_t d, int dtype, uintptr_t x_align, uintptr_t out_align, DirectPlan* out);
bool direct_mergestates_plan(int64_t rows, int64_t d, int dtype, uintptr_t v_align, DirectPlan* out);

// hipError_t of the launch.
int direct_launch_addrms(const DirectPlan& p, void* x, void* r, const void* w, float eps, int64_t M, int64_t N, int dtype,
                         void* stream);
// The kernels of rows split over workgroups; NULL where the route splits none.
void direct_split_kernels(int dtype, DirectPlan* p);
constexpr unsigned kSplitPatience = 256;                    // reads of a row's words, some hundreds of microseconds
// Only the kernel of rows split over workgroups, where the route has one (direct_launch_addrms prefers it).  Returns how many
// of the M rows have been launched: fewer where a launch failed (*status, a hipError_t) or could have no units (slot_pool.h;
// *capturing: since the stream is).  patience: see split_row_sum.
int64_t direct_launch_split(const DirectPlan& p, void* x, void* r, const void* w, float eps, int64_t M, int64_t N, int dtype,
                            unsigned patience, void* stream, int* status, bool* capturing);
// The kernels for the same rows that need no units: the one of calls that find none, and the one of captured calls.
int direct_launch_alone(const DirectPlan& p, void* x, void* r, const void* w, float eps, int64_t M, int64_t N, void* stream);
int direct_launch_whole(const DirectPlan& p, void* x, void* r, const void* w, float eps, int64_t M, int64_t N, void* stream);
int direct_launch_silumul(const DirectPlan& p, const void* x, void* out, int64_t d, void* stream);
int direct_launch_mergestates(const DirectPlan& p, const void* va, const float* sa, const void* vb, const float* sb, void* vo,
                              float* so, void* stream);

}  // namespace addrms_host

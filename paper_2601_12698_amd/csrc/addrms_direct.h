// Launches without a configuration (kernels in direct_kernel.h, rules in addrms_direct.hip).
#pragma once
#include <stdint.h>

#include "addrms_internal.h"

namespace addrms_host {

// A launch that is ready but for the pointers.
struct DirectPlan {
    const void* fn = nullptr;
    unsigned grid = 0, block_x = 0, block_y = 1, lds = 0;
    bool long_row = false;                                  // rows beyond the registers: units = chunks parked in LDS
    unsigned long_index = 0;                                // ... and which of those kernels
    unsigned units = 0, total = 0, mul = 0, shift = 0;      // flat operators: see direct_kernel.h
};

// The kernel and shape for a problem that the grid's default configuration covers, or false: the default
// configuration runs.  x, r, w: the tensors' bases, aligned as the default configuration (of default_vec elements per access)
// asks for; *_align: bases or-ed together.
bool direct_addrms_plan(int64_t M, int64_t N, int dtype, int default_vec, uintptr_t x, uintptr_t r, uintptr_t w,
                        DirectPlan* out);
bool direct_silumul_plan(int64_t M, int64_t d, int dtype, uintptr_t x_align, uintptr_t out_align, DirectPlan* out);
bool direct_mergestates_plan(int64_t rows, int64_t d, int dtype, uintptr_t v_align, DirectPlan* out);

// hipError_t of the launch.
int direct_launch_addrms(const DirectPlan& p, void* x, void* r, const void* w, float eps, int64_t M, int64_t N, void* stream);
int direct_launch_silumul(const DirectPlan& p, const void* x, void* out, int64_t d, void* stream);
int direct_launch_mergestates(const DirectPlan& p, const void* va, const float* sa, const void* vb, const float* sb, void* vo,
                              float* so, void* stream);

}  // namespace addrms_host

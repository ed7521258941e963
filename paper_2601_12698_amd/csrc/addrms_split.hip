// Long rows without a configuration, split over workgroups: the instances of addrms_split_body and addrms_alone_body, and
// their launches.  A code
// object of their own, because the memory in it is cleared when it is loaded, with the first of these launches (some
// milliseconds), and other calls should not pay for that.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "addrms_direct.h"
#include "direct_kernel.h"
#include "slot_pool.h"

using namespace addrms;

// Where the workgroups of split rows meet: memory that belongs to the loaded code object, one copy per GPU.
static __device__ SplitRow split_rows[kSplitUnits][kSplitUnitRows];
static __device__ UnitReports<kSplitUnits> split_reports;

namespace {

// tells: the first row of the grid is none of the tensors', and its first workgroup tells.
template <int DT, int VEC, int CPT, int POL, bool RAG>
__global__ __launch_bounds__(1024) void addrms_split(addr_t x, addr_t r, addr_t w, double inv_n, float eps, int N, unsigned shape,
                                                     unsigned rows, unsigned unit_tells, addr_t words, uint32_t number, uint32_t tag,
                                                     unsigned patience)
{
    // 16-bit rows of whole pieces: so many registers that a CU takes two workgroups of 512 threads, not three (1024 x 131072 bf16 170.5 us
    // against 176.2, 4096 x 40960 fp16 213.0 against 217.9).  88 of them, v87 being the last, are five waves per SIMD, and so are up to 96
    // that the compiler may come to need.
    if constexpr (VEC == 8 && CPT == 4 && !RAG) asm volatile("" ::: "v87");
    const uint32_t tpr = shape & 0xffffu, unit = unit_tells >> 1, tells = unit_tells & 1u;
    if (tells && blockIdx.y == 0u) {
        if (blockIdx.x == 0u) unit_tell(&split_reports, at_global<uint32_t>(words), tpr);
        return;
    }
    addrms_split_body<DT, VEC, CPT, POL, RAG>(at_global(x), at_global(r), at_global(w), inv_n, eps, N, tpr, shape >> 16, rows, blockIdx.y - tells,
                                              split_rows[unit], &split_reports.state[unit], tag, number, patience);
}
__global__ __launch_bounds__(1024) void split_tell(addr_t words) { unit_tell(&split_reports, at_global<uint32_t>(words), 1024u); }

template <int DT, int VEC, int CPT, bool RAG>
__global__ __launch_bounds__(1024) void addrms_alone(addr_t x, addr_t r, addr_t w, double inv_n, float eps, int N, unsigned shape)
{
    addrms_alone_body<DT, VEC, CPT, RAG>(at_global(x), at_global(r), at_global(w), inv_n, eps, N, shape & 0xffffu, shape >> 16);
}

template <int DT, int CPT> const void* addrms_alone_fn1(bool rag)
{
    constexpr int VEC = direct_vec(DT);
    return rag ? reinterpret_cast<const void*>(&addrms_alone<DT, VEC, CPT, true>)
               : reinterpret_cast<const void*>(&addrms_alone<DT, VEC, CPT, false>);
}
template <int DT> const void* addrms_alone_fn(int cpt, bool rag)
{
    switch (cpt) {
    case 1: return addrms_alone_fn1<DT, 1>(rag);
    case 2: return addrms_alone_fn1<DT, 2>(rag);
    case 4: return addrms_alone_fn1<DT, 4>(rag);
    default: return nullptr;
    }
}
const void* addrms_alone_fn(int dtype, int cpt, bool rag)
{
    switch (dtype) {
    case DT_BF16: return addrms_alone_fn<DT_BF16>(cpt, rag);
    case DT_FP16: return addrms_alone_fn<DT_FP16>(cpt, rag);
    case DT_FP16_RES32: return addrms_alone_fn<DT_FP16_RES32>(cpt, rag);
    case DT_FP32: return addrms_alone_fn<DT_FP32>(cpt, rag);
    default: return nullptr;
    }
}
template <int DT, int CPT, int POL> const void* addrms_split_fn2(bool rag)
{
    constexpr int VEC = direct_vec(DT);
    if constexpr (split_instance(CPT, POL))
        return rag ? reinterpret_cast<const void*>(&addrms_split<DT, VEC, CPT, POL, true>)
                   : reinterpret_cast<const void*>(&addrms_split<DT, VEC, CPT, POL, false>);
    else return nullptr;
}
template <int DT, int CPT> const void* addrms_split_fn1(int pol, bool rag)
{
    return pol == POL_NT ? addrms_split_fn2<DT, CPT, POL_NT>(rag) : addrms_split_fn2<DT, CPT, POL_WT>(rag);
}
template <int DT> const void* addrms_split_fn(int cpt, int pol, bool rag)
{
    switch (cpt) {
    case 1: return addrms_split_fn1<DT, 1>(pol, rag);
    case 2: return addrms_split_fn1<DT, 2>(pol, rag);
    case 4: return addrms_split_fn1<DT, 4>(pol, rag);
    default: return nullptr;
    }
}
const void* addrms_split_fn(int dtype, int cpt, int pol, bool rag)
{
    switch (dtype) {
    case DT_BF16: return addrms_split_fn<DT_BF16>(cpt, pol, rag);
    case DT_FP16: return addrms_split_fn<DT_FP16>(cpt, pol, rag);
    case DT_FP16_RES32: return addrms_split_fn<DT_FP16_RES32>(cpt, pol, rag);
    case DT_FP32: return addrms_split_fn<DT_FP32>(cpt, pol, rag);
    default: return nullptr;
    }
}

}  // namespace

namespace addrms_host {

void direct_split_kernels(int dtype, DirectPlan* p)
{
    if (!p->parts) return;
    p->split_fn = addrms_split_fn(dtype, p->part_cpt, p->part_pol, p->rag);
    p->alone_fn = addrms_alone_fn(dtype, p->part_cpt, p->rag);
}

static SlotPool<kSplitUnits> g_split_slots;

int64_t direct_launch_split(const DirectPlan& p, void* x, void* r, const void* w, float eps, int64_t M, int64_t N, int dtype,
                            unsigned patience, void* stream, int* status, bool* capturing)
{
    *status = static_cast<int>(hipSuccess);
    *capturing = false;
    if (!p.split_fn) return 0;
    double inv_n = 1.0 / static_cast<double>(N);
    int n = static_cast<int>(N);
    unsigned shape = p.part_threads | p.parts << 16;
    int64_t row = 0;
    while (row < M) {
        unsigned rows = static_cast<unsigned>(std::min<int64_t>(kSplitRows, M - row));
        SlotPool<kSplitUnits>::Lease lease;
        const int needed = (static_cast<int>(rows) + kSplitUnitRows - 1) / kSplitUnitRows;
        const Units units = g_split_slots.take(static_cast<hipStream_t>(stream), needed, &lease, [stream](uint32_t* words) {
            void* args[] = {&words};
            return hipLaunchKernel(reinterpret_cast<const void*>(&split_tell), dim3(1), dim3(1024), args, 0, static_cast<hipStream_t>(stream));
        });
        *capturing = units == Units::capturing;
        if (units != Units::taken) break;
        void *xr = static_cast<char*>(x) + row * N * x_bytes(dtype), *rr = static_cast<char*>(r) + row * N * r_bytes(dtype);
        unsigned tells = lease.tells(), unit_tells = lease.unit() << 1 | tells;
        uint32_t *words = lease.words(), number = lease.number(), tag = lease.tag();
        void* args[] = {&xr, &rr, &w, &inv_n, &eps, &n, &shape, &rows, &unit_tells, &words, &number, &tag, &patience};
        const hipError_t e = hipLaunchKernel(p.split_fn, dim3(p.parts, rows + tells), dim3(p.part_threads), args, 17u * sizeof(double),
                                             static_cast<hipStream_t>(stream));
        *status = static_cast<int>(e);
        if (e != hipSuccess) break;
        lease.launched();
        row += rows;
    }
    return row;
}

int direct_launch_alone(const DirectPlan& p, void* x, void* r, const void* w, float eps, int64_t M, int64_t N, void* stream)
{
    double inv_n = 1.0 / static_cast<double>(N);
    int n = static_cast<int>(N);
    unsigned shape = p.part_threads | p.parts << 16;
    void* args[] = {&x, &r, &w, &inv_n, &eps, &n, &shape};
    return static_cast<int>(hipLaunchKernel(p.alone_fn, dim3(static_cast<unsigned>(M)), dim3(p.part_threads), args, 32u * sizeof(double),
                                            static_cast<hipStream_t>(stream)));
}

}  // namespace addrms_host

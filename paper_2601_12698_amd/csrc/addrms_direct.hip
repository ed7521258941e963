// Launches without a configuration: the instances of direct_kernel.h, and the launches of what direct_route.cpp decides.
#include <hip/hip_runtime.h>

#include <atomic>
#include <cstdint>

#include "addrms_direct.h"
#include "direct_kernel.h"

using namespace addrms;

namespace {

// MULTI: several rows per workgroup (rpw).  KEEP: see SingleElement.  The launch shape travels as arguments: together with the rest they are preloaded
// into scalar registers, where blockDim would be another load before the first address is known.
template <int DT, int VEC, int CPT, int POL, bool RAG, bool MULTI, bool KEEP>
__global__ __launch_bounds__(1024) void addrms_direct(addr_t x, addr_t r, addr_t w, double inv_n, float eps, int N,
                                                      unsigned tpr, unsigned rpw, long long M)
{
    addrms_direct_body<DT, VEC, CPT, POL, RAG, (CPT > 1), MULTI, KEEP>(at_global(x), at_global(r), at_global(w), eps, inv_n, N, tpr, rpw, M);
}
template <int DT, int VEC, int POL, bool RAG>
__global__ __launch_bounds__(kLongThreads) void addrms_long(addr_t x, addr_t r, addr_t w, float eps, double inv_n, int N,
                                                            unsigned lds_chunks)
{
    addrms_long_body<DT, VEC, kLongRegValues / VEC, 2, POL, RAG>(at_global(x), at_global(r), at_global(w), eps, inv_n, N, lds_chunks);
}
template <int DT, int POL, bool RAG>
__global__ __launch_bounds__(kFlatThreads) void silumul_flat(addr_t x, addr_t out, uint32_t d, uint32_t units,
                                                             uint32_t total, FlatDiv fd)
{
    silumul_flat_body<DT, POL, RAG>(at_global<char>(x), at_global<char>(out), d, units, total, fd);
}
template <int DT, int POL>
__global__ __launch_bounds__(kFlatThreads) void mergestates_flat(addr_t va, addr_t sa, addr_t vb, addr_t sb, addr_t vo, addr_t so,
                                                                 uint32_t units, uint32_t total, FlatDiv fd)
{
    mergestates_flat_body<DT, POL>(at_global<char>(va), at_global<float>(sa), at_global<char>(vb), at_global<float>(sb),
                                   at_global<char>(vo), at_global<float>(so), units, total, fd);
}

template <int DT, int CPT, int POL, bool RAG, bool MULTI> const void* addrms_fn3(bool keep)
{
    constexpr int VEC = direct_vec(DT);
    if constexpr (direct_instance(VEC, CPT, POL, RAG, MULTI))
        return RAG && keep ? reinterpret_cast<const void*>(&addrms_direct<DT, VEC, CPT, POL, RAG, MULTI, RAG>)
                           : reinterpret_cast<const void*>(&addrms_direct<DT, VEC, CPT, POL, RAG, MULTI, false>);
    else return nullptr;
}
template <int DT, int CPT, int POL> const void* addrms_fn2(bool rag, bool multi, bool keep)
{
    return rag ? (multi ? addrms_fn3<DT, CPT, POL, true, true>(keep) : addrms_fn3<DT, CPT, POL, true, false>(keep))
               : (multi ? addrms_fn3<DT, CPT, POL, false, true>(keep) : addrms_fn3<DT, CPT, POL, false, false>(keep));
}
template <int DT, int CPT> const void* addrms_fn2(int pol, bool rag, bool multi, bool keep)
{
    switch (pol) {
    case POL_NT: return addrms_fn2<DT, CPT, POL_NT>(rag, multi, keep);
    case POL_WT: return addrms_fn2<DT, CPT, POL_WT>(rag, multi, keep);
    case POL_SHARED: return addrms_fn2<DT, CPT, POL_SHARED>(rag, multi, keep);
    default: return nullptr;
    }
}
template <int DT> const void* addrms_fn1(int cpt, int pol, bool rag, bool multi, bool keep)
{
    switch (cpt) {
    case 1: return addrms_fn2<DT, 1>(pol, rag, multi, keep);
    case 2: return addrms_fn2<DT, 2>(pol, rag, multi, keep);
    case 3: return addrms_fn2<DT, 3>(pol, rag, multi, keep);
    case 4: return addrms_fn2<DT, 4>(pol, rag, multi, keep);
    case 6: return addrms_fn2<DT, 6>(pol, rag, multi, keep);
    case 8: return addrms_fn2<DT, 8>(pol, rag, multi, keep);
    default: return nullptr;
    }
}
const void* addrms_fn(int dtype, int cpt, int pol, bool rag, bool multi, bool keep)
{
    switch (dtype) {
    case DT_BF16: return addrms_fn1<DT_BF16>(cpt, pol, rag, multi, keep);
    case DT_FP16: return addrms_fn1<DT_FP16>(cpt, pol, rag, multi, keep);
    case DT_FP16_RES32: return addrms_fn1<DT_FP16_RES32>(cpt, pol, rag, multi, keep);
    case DT_FP32: return addrms_fn1<DT_FP32>(cpt, pol, rag, multi, keep);
    default: return nullptr;
    }
}

template <int DT> const void* addrms_long_fn1(int pol, bool rag)
{
    constexpr int VEC = direct_vec(DT);
    if (rag) return pol == POL_NT ? reinterpret_cast<const void*>(&addrms_long<DT, VEC, POL_NT, true>)
                                  : reinterpret_cast<const void*>(&addrms_long<DT, VEC, POL_CACHED, true>);
    return pol == POL_NT ? reinterpret_cast<const void*>(&addrms_long<DT, VEC, POL_NT, false>)
                         : reinterpret_cast<const void*>(&addrms_long<DT, VEC, POL_CACHED, false>);
}
const void* addrms_long_fn(int dtype, int pol, bool rag)
{
    switch (dtype) {
    case DT_BF16: return addrms_long_fn1<DT_BF16>(pol, rag);
    case DT_FP16: return addrms_long_fn1<DT_FP16>(pol, rag);
    case DT_FP16_RES32: return addrms_long_fn1<DT_FP16_RES32>(pol, rag);
    case DT_FP32: return addrms_long_fn1<DT_FP32>(pol, rag);
    default: return nullptr;
    }
}

template <int DT> const void* silumul_fn1(int pol, bool rag, bool keep)
{
    if (rag && keep) return reinterpret_cast<const void*>(&silumul_flat<DT, POL_SHARED, true>);       // written through, being small
    if (rag) return pol == POL_NT ? reinterpret_cast<const void*>(&silumul_flat<DT, POL_NT, true>)
                                  : reinterpret_cast<const void*>(&silumul_flat<DT, POL_WT, true>);
    return pol == POL_NT ? reinterpret_cast<const void*>(&silumul_flat<DT, POL_NT, false>)
                         : reinterpret_cast<const void*>(&silumul_flat<DT, POL_WT, false>);
}
const void* silumul_fn(int dtype, int pol, bool rag, bool keep)
{
    switch (dtype) {
    case DT_BF16: return silumul_fn1<DT_BF16>(pol, rag, keep);
    case DT_FP16: return silumul_fn1<DT_FP16>(pol, rag, keep);
    case DT_FP32: return silumul_fn1<DT_FP32>(pol, rag, keep);
    default: return nullptr;
    }
}
template <int DT> const void* mergestates_fn1(int pol)
{
    return pol == POL_NT ? reinterpret_cast<const void*>(&mergestates_flat<DT, POL_NT>)
                         : reinterpret_cast<const void*>(&mergestates_flat<DT, POL_WT>);
}

}  // namespace

namespace addrms_host {

bool direct_addrms_plan(int64_t M, int64_t N, int dtype, int default_vec, uintptr_t x, uintptr_t r, uintptr_t w, DirectPlan* out)
{
    if (!direct_addrms_route(M, N, dtype, default_vec, x, r, w, out)) return false;
    if (!out->long_row) direct_addrms_split_few(M, N, dtype, out);
    direct_split_kernels(dtype, out);
    if (out->long_row) {
        out->fn = addrms_long_fn(dtype, out->pol, out->rag);
        out->long_index = static_cast<unsigned>(dtype) * 4u + (out->pol == POL_NT ? 2u : 0u) + (out->rag ? 1u : 0u);
    } else {
        out->fn = addrms_fn(dtype, out->cpt, out->pol, out->rag, out->block_y > 1, out->keep_shared);
    }
    return out->fn != nullptr;
}
bool direct_silumul_plan(int64_t M, int64_t d, int dtype, uintptr_t x_align, uintptr_t out_align, DirectPlan* out)
{
    if (!direct_silumul_route(M, d, dtype, x_align, out_align, out)) return false;
    out->fn = silumul_fn(dtype, out->pol, out->rag, out->keep_shared);
    return out->fn != nullptr;
}
bool direct_mergestates_plan(int64_t rows, int64_t d, int dtype, uintptr_t v_align, DirectPlan* out)
{
    if (!direct_mergestates_route(rows, d, dtype, v_align, out)) return false;
    out->fn = dtype == DT_BF16 ? mergestates_fn1<DT_BF16>(out->pol) : mergestates_fn1<DT_FP16>(out->pol);
    return true;
}

// Once per kernel: LDS beyond the default limit of 64 KB has to be allowed, as in launch_instance, and this loads the kernel's
// code object.
static hipError_t prepare_long(const DirectPlan& p)
{
    static std::atomic<uint64_t> allowed{0};                   // one bit per kernel
    const uint64_t bit = 1ull << p.long_index;
    if (allowed.load(std::memory_order_acquire) & bit) return hipSuccess;
    const hipError_t e = hipFuncSetAttribute(p.fn, hipFuncAttributeMaxDynamicSharedMemorySize, hw().lds_bytes_per_cu);
    if (e == hipSuccess) allowed.fetch_or(bit, std::memory_order_acq_rel);
    return p.lds > 64u * 1024u ? e : hipSuccess;
}
static int go(const DirectPlan& p, unsigned grid, void** args, void* stream)
{
    return static_cast<int>(hipLaunchKernel(p.fn, dim3(grid), dim3(p.block_x, p.block_y), args, p.lds,
                                            static_cast<hipStream_t>(stream)));
}

static int launch_rows(const DirectPlan& p, void* x, void* r, const void* w, float eps, int64_t M, int64_t N, void* stream)
{
    double inv_n = 1.0 / static_cast<double>(N);
    long long m = M;
    int n = static_cast<int>(N);
    unsigned tpr = p.block_x, rpw = p.block_y;
    void* args[] = {&x, &r, &w, &inv_n, &eps, &n, &tpr, &rpw, &m};
    return go(p, p.grid, args, stream);
}
int direct_launch_whole(const DirectPlan& p, void* x, void* r, const void* w, float eps, int64_t M, int64_t N, void* stream)
{
    if (!p.long_row) return launch_rows(p, x, r, w, eps, M, N, stream);
    if (const hipError_t e = prepare_long(p); e != hipSuccess) return static_cast<int>(e);
    double inv_n = 1.0 / static_cast<double>(N);
    int n = static_cast<int>(N);
    unsigned lds_chunks = p.units;
    void* args[] = {&x, &r, &w, &eps, &inv_n, &n, &lds_chunks};
    return go(p, static_cast<unsigned>(M), args, stream);
}
int direct_launch_addrms(const DirectPlan& p, void* x, void* r, const void* w, float eps, int64_t M, int64_t N, int dtype, void* stream)
{
    if (p.split_fn) {
        // Of the kernel that a capture of this call runs: a capture is no place for this.
        if (const hipError_t e = p.long_row ? prepare_long(p) : hipSuccess; e != hipSuccess) return static_cast<int>(e);
        int status;
        bool capturing;
        const int64_t split = direct_launch_split(p, x, r, w, eps, M, N, dtype, kSplitPatience, stream, &status, &capturing);
        if (status != static_cast<int>(hipSuccess) || split == M) return status;
        // What is in flight decides whether there are units, but not the bits: the kernel behind it adds in the same order.
        if (!capturing)
            return direct_launch_alone(p, static_cast<char*>(x) + split * N * x_bytes(dtype),
                                       static_cast<char*>(r) + split * N * r_bytes(dtype), w, eps, M - split, N, stream);
    }
    return direct_launch_whole(p, x, r, w, eps, M, N, stream);
}
int direct_launch_silumul(const DirectPlan& p, const void* x, void* out, int64_t d, void* stream)
{
    uint32_t ud = static_cast<uint32_t>(d), units = p.units, total = p.total;
    FlatDiv fd{p.mul, p.shift};
    void* args[] = {&x, &out, &ud, &units, &total, &fd};
    return go(p, p.grid, args, stream);
}
int direct_launch_mergestates(const DirectPlan& p, const void* va, const float* sa, const void* vb, const float* sb, void* vo,
                              float* so, void* stream)
{
    uint32_t units = p.units, total = p.total;
    FlatDiv fd{p.mul, p.shift};
    void* args[] = {&va, &sa, &vb, &sb, &vo, &so, &units, &total, &fd};
    return go(p, p.grid, args, stream);
}

}  // namespace addrms_host

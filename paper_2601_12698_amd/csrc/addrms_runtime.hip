// HIP side of libaddrms: kernel dispatch (addrms_run), the measurement harness
// and correctness gate used by the search (Algorithm 1: Validate, Search,
// EvaluatePerformance), and the probe kernels.
#include <hip/hip_runtime.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <mutex>
#include <vector>

#include "addrms_direct.h"
#include "addrms_internal.h"
#include "mergestates.h"
#include "mergestates_kernel.h"
#include "slot_pool.h"
#include "unit_report.h"
#include "silumul.h"
#include "silumul_kernel.h"

// Declarations of every kernel instance and the table of their addresses, in
// the order of the instance list the deriver uses.
#include "gen_dispatch_decl.inc"
struct DispatchEntry { int op, dt, vec, cpt, unr, nt, df; const void* fn; };
static const DispatchEntry kDispatch[] = {
#include "gen_dispatch_rows.inc"
};

using namespace addrms_host;
using addrms::addr_t;
using addrms::at_global;

// Partial-count slots of addrms_gate_probe_noalloc: device memory that belongs to the loaded
// code object, one copy per GPU, so the entry point needs no allocation.  Host code never
// uses this name as an address; it asks the runtime for the device address once per device
// (gate_scratch_on_current_device) and passes that pointer around.
constexpr int kGateScratchSlots = 512;
static __device__ __align__(256) unsigned scratch[kGateScratchSlots * 4];

namespace {

#define HIP_TRY(expr)                                                                              \
    do {                                                                                           \
        hipError_t e_ = (expr);                                                                    \
        if (e_ != hipSuccess)                                                                      \
            return fail(ADDRMS_ERR_HIP, "%s failed: %s", #expr, hipGetErrorString(e_));            \
    } while (0)

bool dispatch_consistent()
{
    static const bool ok = [] {
        if (static_cast<int>(sizeof(kDispatch) / sizeof(kDispatch[0])) != n_instances()) return false;
        for (int i = 0; i < n_instances(); ++i) {
            const Instance& in = instance(i);
            const DispatchEntry& d = kDispatch[i];
            if (d.op != in.op || d.dt != in.dt || d.vec != in.vec || d.cpt != in.cpt || d.unr != in.unr || d.nt != in.nt || d.df != in.df) return false;
        }
        return true;
    }();
    return ok;
}

constexpr int kDefaultDynamicLdsLimit = 64 * 1024;
std::atomic<bool> g_big_lds_enabled[sizeof(kDispatch) / sizeof(kDispatch[0])];

bool aligned(const void* p, int bytes) { return (reinterpret_cast<uintptr_t>(p) % static_cast<uintptr_t>(bytes)) == 0; }

// Launch of a kernel instance with every check already done.
int launch_instance(const Feas& f, const addrms_cfg& c, unsigned grid, void** args, hipStream_t stream)
{
    const dim3 block(static_cast<unsigned>(c.threads_per_row), static_cast<unsigned>(c.rows_per_wg));
    const int lds = f.dyn_lds;
    if (lds > kDefaultDynamicLdsLimit) {
        // Occupancy padding beyond the default per-launch limit has to be enabled once per kernel.
        std::atomic<bool>& done = g_big_lds_enabled[f.inst];
        if (!done.load(std::memory_order_acquire)) {
            HIP_TRY(hipFuncSetAttribute(kDispatch[f.inst].fn, hipFuncAttributeMaxDynamicSharedMemorySize,
                                        hw().lds_bytes_per_cu));
            done.store(true, std::memory_order_release);
        }
    }
    HIP_TRY(hipLaunchKernel(kDispatch[f.inst].fn, dim3(grid), block, args, static_cast<size_t>(lds), stream));
    return ADDRMS_OK;
}

unsigned shape_argument(const addrms_cfg& c)
{
    return static_cast<unsigned>(c.threads_per_row) | static_cast<unsigned>(c.rows_per_wg) << 16;
}

// The flags of the configuration and those that are the launch's own.
unsigned launch_flags(const addrms_cfg& c, int64_t M, int64_t N, int dtype, int op)
{
    unsigned flags = static_cast<unsigned>(c.flags);
    if (launch_paced(c, M, N, dtype, op)) flags |= static_cast<unsigned>(addrms::LAUNCH_PACED);
    if (launch_write_through(c, M, N, dtype, op)) flags |= static_cast<unsigned>(addrms::LAUNCH_WRITE_THROUGH);
    return flags;
}

int launch(const Feas& f, const addrms_cfg& c, void* x, void* r, const void* w, float eps, int64_t M, int64_t N, int dtype,
           hipStream_t stream)
{
    double inv_n = 1.0 / static_cast<double>(N);
    int n = static_cast<int>(N);
    unsigned m = static_cast<unsigned>(M), shape = shape_argument(c);                    // the callers checked M < 2^31
    unsigned mode = launch_flags(c, M, N, dtype, OP_ADDRMS) | static_cast<unsigned>(c.reduce) << 16;
    // the last argument is the number of row blocks (persistent grids walk them), or, for the forms that
    // continue the row cache in LDS, the chunks per thread the LDS allocation holds
    unsigned nblocks = f.lds_chunks >= 0 ? static_cast<unsigned>(f.lds_chunks) : static_cast<unsigned>(n_row_blocks(c, M));
    unsigned grid = static_cast<unsigned>(n_workgroups(c, M, f.res.wgs_per_cu));
    void* args[] = {&x, &r, &w, &inv_n, &eps, &n, &m, &shape, &mode, &nblocks, &grid};
    return launch_instance(f, c, grid, args, stream);
}

int launch_silumul(const Feas& f, const addrms_cfg& c, const void* x, void* out, int64_t M, int64_t d, int dtype, hipStream_t stream)
{
    int dd = static_cast<int>(d);
    unsigned m = static_cast<unsigned>(M), shape = shape_argument(c);
    unsigned flags = launch_flags(c, M, d, dtype, OP_SILUMUL);
    unsigned nblocks = static_cast<unsigned>(n_row_blocks(c, M));
    unsigned grid = static_cast<unsigned>(n_workgroups(c, M, f.res.wgs_per_cu));
    void* args[] = {&x, &out, &dd, &m, &shape, &flags, &nblocks, &grid};
    return launch_instance(f, c, grid, args, stream);
}

int launch_mergestates(const Feas& f, const addrms_cfg& c, const void* va, const float* sa, const void* vb,
                       const float* sb, void* vo, float* so, int64_t rows, int64_t d, hipStream_t stream)
{
    int dd = static_cast<int>(d);
    unsigned m = static_cast<unsigned>(rows), shape = shape_argument(c), flags = static_cast<unsigned>(c.flags);
    unsigned nblocks = static_cast<unsigned>(n_row_blocks(c, rows));
    unsigned grid = static_cast<unsigned>(n_workgroups(c, rows, f.res.wgs_per_cu));
    void* args[] = {&va, &vb, &dd, &m, &shape, &flags, &sa, &sb, &vo, &so, &nblocks, &grid};
    return launch_instance(f, c, grid, args, stream);
}

// *untuned (may be NULL): true if neither the caller nor the table names a configuration.
int resolve_cfg(const addrms_cfg* cfg, int64_t M, int64_t N, int dtype, addrms_cfg* out, int op = OP_ADDRMS, bool* untuned = nullptr)
{
    if (untuned) *untuned = false;
    if (cfg) { *out = *cfg; return ADDRMS_OK; }
    if (table_lookup(M, N, dtype, out, op) == ADDRMS_OK) return ADDRMS_OK;
    std::string why;
    const int st = default_cfg(N, dtype, out, &why, op);
    if (untuned) *untuned = st == ADDRMS_OK;
    return st == ADDRMS_OK ? st : fail(st, "%s", why.c_str());
}

// ---- resolved calls -----------------------------------------------------------------
// What a *_run call decides before it launches depends on its sizes, its configuration (if any), the table and the
// alignment of its tensors, not on their contents or addresses.  Deciding it takes from 0.8 us to 13 us (a default
// configuration behind several infeasible ones) beside a launch of 2 us, so each thread keeps decisions in 64 slots
// per operator, looked up by everything they depend on.  A problem has one slot: of two problems of an operator that fall
// into the same one, each call decides anew.
struct Resolved {
    Feas f;                  // of c, which has passed every check
    addrms_cfg c{};
    bool direct = false;     // no configuration named, and the direct kernels cover the problem: p
    DirectPlan p;
};
struct ResolvedKey {
    int64_t M, N;
    uint64_t table;          // table_generation(); 0 in an empty slot
    addrms_cfg cfg;          // zeroes where the call names none
    int32_t op, dtype, has_cfg;
    uint32_t low;            // the bases modulo 16: as much of an address as any check or rule asks for
};
bool same_key(const ResolvedKey& a, const ResolvedKey& b)
{
    return a.M == b.M && a.N == b.N && a.table == b.table && a.op == b.op && a.dtype == b.dtype && a.has_cfg == b.has_cfg &&
           a.low == b.low && cfg_equal(a.cfg, b.cfg);
}

// Fills and checks one decision.  `misaligned` is the operator's own test of its tensors against a configuration.
template <class Misaligned, class Plan>
int resolve_call(const ResolvedKey& k, Resolved* out, Misaligned misaligned, Plan plan)
{
    bool untuned = false;
    int st = resolve_cfg(k.has_cfg ? &k.cfg : nullptr, k.M, k.N, k.dtype, &out->c, k.op, &untuned);
    if (st != ADDRMS_OK) return st;
    out->f = check_cfg(out->c, k.M, k.N, k.dtype, k.op);
    if (out->f.status != ADDRMS_OK) return fail(out->f.status, "%s", out->f.reason.c_str());
    st = misaligned(out->c);
    if (st != ADDRMS_OK) return st;
    out->p = DirectPlan{};
    out->direct = untuned && plan(out->c, &out->p);
    return ADDRMS_OK;
}
template <class Misaligned, class Plan>
int find_or_resolve(int op, int64_t M, int64_t N, int dtype, const addrms_cfg* cfg, uint32_t low, const Resolved** out,
                    Misaligned misaligned, Plan plan)
{
    constexpr unsigned kSlots = 64;
    static thread_local ResolvedKey keys[kSlots];
    static thread_local Resolved values[kSlots];
    ResolvedKey k{M, N, table_generation(), cfg ? *cfg : addrms_cfg{}, op, dtype, cfg ? 1 : 0, low};
    uint64_t h = static_cast<uint64_t>(M) * 0x9e3779b97f4a7c15ull ^ static_cast<uint64_t>(N) * 0xc2b2ae3d27d4eb4full;
    h ^= (static_cast<uint64_t>(op) << 8 | static_cast<uint64_t>(dtype) << 4 | static_cast<uint64_t>(low) << 16) * 0x165667b19e3779f9ull;
    if (cfg) h ^= cfg_key(*cfg) * 0x27d4eb2f165667c5ull;
    const unsigned slot = static_cast<unsigned>(h >> 58);                  // the top six bits
    static_assert(kSlots == 64, "six bits of the hash");
    *out = &values[slot];
    if (same_key(keys[slot], k)) return ADDRMS_OK;
    keys[slot].table = 0;                                                  // nothing is kept of a call that fails
    const int st = resolve_call(k, &values[slot], misaligned, plan);
    if (st == ADDRMS_OK) keys[slot] = k;
    return st;
}
uintptr_t bits(const void* p) { return reinterpret_cast<uintptr_t>(p); }
uint32_t low4(const void* p, int place) { return static_cast<uint32_t>(bits(p) & 15u) << (4 * place); }

int run_addrms(void* x, void* r, const void* w, float eps, int64_t M, int64_t N, int dtype, const addrms_cfg* cfg, hipStream_t stream)
{
    const Resolved* call = nullptr;
    const int st = find_or_resolve(
        OP_ADDRMS, M, N, dtype, cfg, low4(x, 0) | low4(r, 1) | low4(w, 2), &call,
        [=](const addrms_cfg& c) {
            const int xa = c.vec * x_bytes(dtype), ra = std::min(16, c.vec * r_bytes(dtype));
            if (aligned(x, xa) && aligned(w, xa) && aligned(r, ra)) return static_cast<int>(ADDRMS_OK);
            return fail(ADDRMS_ERR_MISALIGNED, "x and weight must be %d-byte aligned and residual %d-byte aligned for vec=%d",
                        xa, ra, c.vec);
        },
        [=](const addrms_cfg& c, DirectPlan* p) { return direct_addrms_plan(M, N, dtype, c.vec, bits(x), bits(r), bits(w), p); });
    if (st != ADDRMS_OK) return st;
    if (!call->direct) return launch(call->f, call->c, x, r, w, eps, M, N, dtype, stream);
    HIP_TRY(static_cast<hipError_t>(direct_launch_addrms(call->p, x, r, w, eps, M, N, dtype, stream)));
    return ADDRMS_OK;
}
int run_silumul(const void* x, void* out, int64_t M, int64_t d, int dtype, const addrms_cfg* cfg, hipStream_t stream)
{
    const Resolved* call = nullptr;
    const int st = find_or_resolve(
        OP_SILUMUL, M, d, dtype, cfg, low4(x, 0) | low4(out, 1), &call,
        [=](const addrms_cfg& c) {
            const int al = c.vec * x_bytes(dtype);
            if (aligned(x, al) && aligned(out, al)) return static_cast<int>(ADDRMS_OK);
            return fail(ADDRMS_ERR_MISALIGNED, "x and out must be %d-byte aligned for vec=%d", al, c.vec);
        },
        [=](const addrms_cfg&, DirectPlan* p) { return direct_silumul_plan(M, d, dtype, bits(x), bits(out), p); });
    if (st != ADDRMS_OK) return st;
    if (!call->direct) return launch_silumul(call->f, call->c, x, out, M, d, dtype, stream);
    HIP_TRY(static_cast<hipError_t>(direct_launch_silumul(call->p, x, out, d, stream)));
    return ADDRMS_OK;
}
int run_mergestates(const void* va, const float* sa, const void* vb, const float* sb, void* vo, float* so, int64_t rows,
                    int64_t d, int dtype, const addrms_cfg* cfg, hipStream_t stream)
{
    const Resolved* call = nullptr;
    const int st = find_or_resolve(
        OP_MERGE, rows, d, dtype, cfg, low4(va, 0) | low4(vb, 1) | low4(vo, 2) | low4(sa, 3) | low4(sb, 4) | low4(so, 5), &call,
        [=](const addrms_cfg& c) {
            const int al = c.vec * x_bytes(dtype);
            if (aligned(va, al) && aligned(vb, al) && aligned(vo, al) && aligned(sa, 4) && aligned(sb, 4) && aligned(so, 4))
                return static_cast<int>(ADDRMS_OK);
            return fail(ADDRMS_ERR_MISALIGNED, "v_a, v_b and v_out must be %d-byte aligned for vec=%d, scores 4-byte aligned", al, c.vec);
        },
        [=](const addrms_cfg&, DirectPlan* p) { return direct_mergestates_plan(rows, d, dtype, bits(va) | bits(vb) | bits(vo), p); });
    if (st != ADDRMS_OK) return st;
    if (!call->direct) return launch_mergestates(call->f, call->c, va, sa, vb, sb, vo, so, rows, d, stream);
    HIP_TRY(static_cast<hipError_t>(direct_launch_mergestates(call->p, va, sa, vb, sb, vo, so, stream)));
    return ADDRMS_OK;
}

// ---- probe and harness kernels ---------------------------------------------------

__global__ void rstd_probe_kernel(const double* ss, long long n, double inv_n, float eps, float* out)
{
    const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i < n) out[i] = addrms::rsqrt_to_f32(__builtin_fma(ss[i], inv_n, static_cast<double>(eps)));
}

// Reads two streams and writes both back complemented: the operator's traffic
// pattern (one read and one write of every byte, both streams touched by the
// same lane) with no arithmetic to speak of.
// It uses the best settings a sweep of plain copy-like kernels found on this device:
// streaming (non-temporal) policy on loads and stores, and at most three 256-thread
// workgroups per CU (imposed by the dynamic LDS allocation; fewer requests in flight
// suit mixed read/write traffic better than full occupancy).
constexpr int kProbeLdsBytes = 160 * 1024 / 3 / 1280 * 1280;   // 53,760: three workgroups per CU
template <int B_PER_A>   // 16-byte pieces of b per piece of a: 1, or 2 when the residual is fp32 beside 16-bit x
__global__ __launch_bounds__(256) void stream_probe_kernel(addrms::u32x4* a, addrms::u32x4* b, long long n)
{
    const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    // every load is issued before the first value is used
    const addrms::u32x4 va = __builtin_nontemporal_load(a + i);
    addrms::u32x4 vb[B_PER_A];
#pragma unroll
    for (int k = 0; k < B_PER_A; ++k) vb[k] = __builtin_nontemporal_load(b + B_PER_A * i + k);
    __builtin_nontemporal_store(~va, a + i);
#pragma unroll
    for (int k = 0; k < B_PER_A; ++k) __builtin_nontemporal_store(~vb[k], b + B_PER_A * i + k);
}

// The same traffic under the operator's constraint: a workgroup owns one whole row, every thread reads all its
// 16-byte pieces of the row from both streams, the workgroup meets at a barrier (where the operator would have
// its row sum), and only then is anything written.  No arithmetic beyond the complement.  What this kernel
// reaches, over workgroup sizes and occupancy caps, is what holding a row across a reduction costs by itself.
template <int CPT, int B_PER_A>
__global__ __launch_bounds__(1024) void row_probe_kernel(addrms::u32x4* a, addrms::u32x4* b, long long M, unsigned pieces)
{
    const long long row = blockIdx.x;
    if (row >= M) return;                                   // uniform over the workgroup
    addrms::u32x4* ar = a + row * pieces;
    addrms::u32x4* br = b + row * pieces * B_PER_A;
    addrms::u32x4 va[CPT], vb[CPT][B_PER_A];
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const unsigned p = static_cast<unsigned>(c) * blockDim.x + threadIdx.x;
        const unsigned pc = p < pieces ? p : pieces - 1u;   // tail lanes re-read the last piece
        va[c] = __builtin_nontemporal_load(ar + pc);
#pragma unroll
        for (int k = 0; k < B_PER_A; ++k) vb[c][k] = __builtin_nontemporal_load(br + B_PER_A * pc + k);
    }
    __syncthreads();
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const unsigned p = static_cast<unsigned>(c) * blockDim.x + threadIdx.x;
        if (p < pieces) {
#pragma unroll
            for (int k = 0; k < B_PER_A; ++k) __builtin_nontemporal_store(~vb[c][k], br + B_PER_A * p + k);
        }
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const unsigned p = static_cast<unsigned>(c) * blockDim.x + threadIdx.x;
        if (p < pieces) __builtin_nontemporal_store(~va[c], ar + p);
    }
}

template <int B_PER_A>
static const void* row_probe_instance(int chunks, int* cpt_out)
{
#define ROW_PROBE_CASE(C) if (chunks <= C) { *cpt_out = C; return reinterpret_cast<const void*>(&row_probe_kernel<C, B_PER_A>); }
    ROW_PROBE_CASE(1) ROW_PROBE_CASE(2) ROW_PROBE_CASE(3) ROW_PROBE_CASE(4) ROW_PROBE_CASE(6) ROW_PROBE_CASE(8)
    ROW_PROBE_CASE(12) ROW_PROBE_CASE(16)
#undef ROW_PROBE_CASE
    return nullptr;
}

// Synthetic activations for the tuner's own buffers: a counter-based hash mapped
// to a roughly unit-variance symmetric distribution (sum of four uniforms).
__device__ __forceinline__ uint32_t mix32(uint32_t v)
{
    v ^= v >> 16; v *= 0x7feb352du; v ^= v >> 15; v *= 0x846ca68bu; v ^= v >> 16;
    return v;
}
__device__ __forceinline__ float synth_value(uint64_t i, uint32_t seed, float lo, float hi, bool bell)
{
    const uint32_t a = mix32(static_cast<uint32_t>(i) ^ seed);
    const uint32_t b = mix32(a ^ static_cast<uint32_t>(i >> 32) ^ 0x9e3779b9u);
    if (!bell) return lo + (hi - lo) * (static_cast<float>(a >> 8) * (1.0f / 16777216.0f));
    const float u = static_cast<float>(a & 0xffffu) + static_cast<float>(a >> 16) +
                    static_cast<float>(b & 0xffffu) + static_cast<float>(b >> 16);
    return (u * (1.0f / 65536.0f) - 2.0f) * 1.7320508f;   // variance 4/12 -> 1
}
template <int ES, bool BF>
__global__ void fill_kernel(void* p, long long n, uint32_t seed, float lo, float hi, int bell)
{
    const long long i = static_cast<long long>(blockIdx.x) * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const float v = synth_value(static_cast<uint64_t>(i), seed, lo, hi, bell != 0);
    if constexpr (ES == 4) static_cast<float*>(p)[i] = v;
    else static_cast<uint16_t*>(p)[i] = static_cast<uint16_t>(addrms::pack2<BF>(v, 0.0f) & 0xffffu);
}

// Correctness gate d(S~(x), S(x)) <= eps (Section 3.1): residual must match bit
// for bit; y may differ by at most `tol` units in the last place of its format
// (+0 and -0 are the same value).  Counted in two stages so that the cost and the
// result do not depend on how many elements disagree: every workgroup walks a
// grid-stride slice and writes its three counts to its own slot, and one workgroup
// folds the slots into `out`, within one launch (gate_one_kernel) or, for captured
// calls and those that can have no unit, in a second (gate_partial_kernel, whose
// slots are `partial`, and gate_finish_kernel):
//   out[0] = residual elements that differ, out[1] = y elements beyond tol,
//   out[2] = largest y distance seen, out[3] = 0.
// Every slot that is read was written by the same call, so the buffer needs no clearing.
//
// Bound by HBM reads (four streams, nothing written), so a thread takes 16 bytes of y and
// of its reference at a time (8 or 4 elements) and the matching elements of the residual
// pair, with all loads of a piece issued before the first is used; the arithmetic is about
// ten 32-bit operations per element, a quarter of what the reads leave room for.  Tensors
// are only element-aligned here, so the vector type says so.  134 MB (4096 x 4096 bf16): the
// first stage takes 21.8 us (6.2 TB/s; 24.6 with ordinary loads and 1024 workgroups, 30.6 with
// one element per access), the second 4 (6.1 over 4096 slots).
constexpr int kGateBlock = 512;
constexpr int kGateMaxGrid = kGateScratchSlots;          // slots of 4 counters each: two workgroups per CU, all of the wave slots
constexpr size_t kGateScratchBytes = static_cast<size_t>(kGateMaxGrid) * 4 * sizeof(unsigned);
constexpr long long kGateMaxElems = 0xffffffffll;        // the counters are 32 bits wide

template <int ES> struct gate_piece;                     // 16 bytes at element alignment
template <> struct gate_piece<2> { typedef addrms::u32x4 type __attribute__((aligned(2))); };
template <> struct gate_piece<4> { typedef addrms::u32x4 type __attribute__((aligned(4))); };

template <typename P> __device__ __forceinline__ addrms::u32x4 gate_load(const char* p)
{
    return __builtin_nontemporal_load(reinterpret_cast<const P*>(p));      // read once
}

// Distance in units in the last place of two bit patterns (sign and magnitude; the zeros are one value).
template <int ES>
__device__ __forceinline__ unsigned ulp_distance(unsigned a, unsigned b)
{
    constexpr unsigned kSign = ES == 4 ? 0x80000000u : 0x8000u, kMag = kSign - 1u;
    const unsigned ma = a & kMag, mb = b & kMag;
    // same sign: difference of the magnitudes; opposite signs: their sum, which fits 32 bits
    return ((a ^ b) & kSign) ? ma + mb : (ma > mb ? ma - mb : mb - ma);
}
template <int ES>
__device__ __forceinline__ void gate_count_y(unsigned a, unsigned b, unsigned tol, unsigned& bad, unsigned& most)
{
    const unsigned d = ulp_distance<ES>(a, b);
    bad += d > tol;
    most = d > most ? d : most;
}
// Sum (or largest) over the 64 lanes of a wave, in every lane.
template <bool MAX, int STEP>
__device__ __forceinline__ unsigned gate_fold(unsigned v)
{
    const unsigned o = addrms::lane_partner<STEP>(v);
    return MAX ? (o > v ? o : v) : v + o;
}
template <bool MAX>
__device__ __forceinline__ unsigned gate_wave(unsigned v)
{
    v = gate_fold<MAX, 1>(v); v = gate_fold<MAX, 2>(v); v = gate_fold<MAX, 4>(v);
    v = gate_fold<MAX, 8>(v); v = gate_fold<MAX, 16>(v); return gate_fold<MAX, 32>(v);
}
// The three counts of a workgroup, valid in thread 0.  USE: uses of one kernel have LDS of their own, and need no barrier between.
template <int USE>
__device__ __forceinline__ void gate_block(unsigned& rbad, unsigned& ybad, unsigned& ymax)
{
    __shared__ unsigned red[3][kGateBlock / 64];
    rbad = gate_wave<false>(rbad); ybad = gate_wave<false>(ybad); ymax = gate_wave<true>(ymax);
    if ((threadIdx.x & 63u) == 0u) {
        red[0][threadIdx.x >> 6] = rbad; red[1][threadIdx.x >> 6] = ybad; red[2][threadIdx.x >> 6] = ymax;
    }
    __syncthreads();
    if (threadIdx.x == 0)
        for (int w = 1; w < kGateBlock / 64; ++w) {
            rbad += red[0][w]; ybad += red[1][w];
            ymax = red[2][w] > ymax ? red[2][w] : ymax;
        }
}

// One launch: the workgroups put their counts into words of their own and end; the last one in the grid looks for the words of all
// others and folds them.  It is the only one that looks, and they need nothing of it.  Nor does it depend on them: each XCD takes
// its share of a grid by itself, so that others may still wait for room where the last one has found some.  After a number of looks
// the wave that misses a word compares that workgroup's slice itself.  Whoever comes later than that leaves its words in a unit that
// may be another launch's by then: with a number that is not that launch's, whose last workgroup may have to compare a slice, too.
// A word is a count and, in its upper half, the number of the launch, so that nothing has to be cleared and no arrival to be
// counted: what a unit's earlier launches left has other numbers (a unit's numbers do not come round, slot_map.h).  Words are
// accessed with relaxed atomics of device scope, which go to the memory side of the XCDs' L2s.
// Through the binding, us; before, up to 96 workgroups met in one launch, whose last arrival, counted on one line, folded and
// cleared the words, and more took two launches:
//   8 k elements of bf16 (2 workgroups)  4.5 -> 3.7    28 k  4.7 -> 3.9    384 k (96)  5.5 -> 4.4    860 k (209)  5.9 -> 4.3
//   2 M (512)  6.8 -> 5.8    4 M  8.8 -> 7.9    16 M  23.2 -> 22.5    64 M  77.4 -> 76.7
// (with a report to host memory at the end, as before; unit_report.h has what is written now)
// Looks that are counted cost 0.07 us of each (60 sizes of 2 to 573 workgroups' work, 4.37 -> 4.44 on average).
// Two launches with arguments instead of gridDim: 860 k 7.0 -> 6.2.  Arguments in scalar registers when a wave starts: 28 k 4.3 ->
// 3.9, 860 k 4.6 -> 4.3.
struct GateWords { uint64_t rbad, ybad, ymax; };
constexpr int kGateUnits = 256;                          // launches in flight: 1 ms of them
// Looks at a missing word, a microsecond and more each: some hundreds of them, and more than the whole comparison takes.
unsigned gate_looks(long long n) { return 256u + static_cast<unsigned>(n >> 20); }
static __device__ GateWords gate_words[kGateUnits][kGateMaxGrid];
static __device__ addrms::UnitReports<kGateUnits> gate_reports;

__device__ __forceinline__ void gate_put(uint64_t* word, unsigned count, uint32_t number)
{
    __hip_atomic_store(word, static_cast<uint64_t>(number) << 32 | count, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ uint64_t gate_look(const uint64_t* word) { return __hip_atomic_load(word, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// The counts that one workgroup leaves, added to those here once they are there.  True: they are not, after `looks` further looks.
__device__ __forceinline__ bool gate_without(const GateWords* w, uint32_t number, unsigned looks, unsigned& rbad, unsigned& ybad, unsigned& ymax)
{
    uint64_t a, b, c;
    bool without = false;
    for (unsigned k = looks;; --k, __builtin_amdgcn_s_sleep(1)) {
        a = gate_look(&w->rbad); b = gate_look(&w->ybad); c = gate_look(&w->ymax);        // in one trip to memory
        if ((a >> 32) == number && (b >> 32) == number && (c >> 32) == number) break;
        if (k == 0u) {
            a = b = c = 0;
            without = true;
            break;
        }
    }
    rbad += static_cast<unsigned>(a);
    ybad += static_cast<unsigned>(b);
    ymax = static_cast<unsigned>(c) > ymax ? static_cast<unsigned>(c) : ymax;
    return without;
}
// One element.
template <int XB, int RB>
__device__ __forceinline__ void gate_element(const char* y, const char* y_ref, const char* r, const char* r_ref, long long i, unsigned tol,
                                             unsigned& rbad, unsigned& ybad, unsigned& ymax)
{
    if constexpr (XB == 4) gate_count_y<4>(reinterpret_cast<const uint32_t*>(y)[i], reinterpret_cast<const uint32_t*>(y_ref)[i], tol, ybad, ymax);
    else gate_count_y<2>(reinterpret_cast<const uint16_t*>(y)[i], reinterpret_cast<const uint16_t*>(y_ref)[i], tol, ybad, ymax);
    if constexpr (RB == 4) rbad += reinterpret_cast<const uint32_t*>(r)[i] != reinterpret_cast<const uint32_t*>(r_ref)[i];
    else rbad += reinterpret_cast<const uint16_t*>(r)[i] != reinterpret_cast<const uint16_t*>(r_ref)[i];
}
// Adds workgroup `block`'s slice, as gate_slice counts it, to the counts of a wave.  Small rather than fast.
template <int XB, int RB>
__device__ __forceinline__ void gate_wave_slice(const char* y, const char* y_ref, const char* r, const char* r_ref, long long n, unsigned tol,
                                                unsigned block, unsigned grid, unsigned& rbad, unsigned& ybad, unsigned& ymax)
{
    constexpr unsigned E = 16 / XB, kRun = kGateBlock * E;   // elements of a piece, and of a workgroup's pieces side by side
    long long at = static_cast<long long>(block) * kRun, end = n / E * E;
    for (bool rest = block == 0u;; rest = false, at = end, end = n) {
#pragma unroll 1
        for (; at < end; at += static_cast<long long>(grid) * kRun)
#pragma unroll 1
            for (unsigned i = threadIdx.x & 63u; i < kRun && at + i < end; i += 64u)
                gate_element<XB, RB>(y, y_ref, r, r_ref, at + i, tol, rbad, ybad, ymax);
        if (!rest) break;
    }
}

// The three counts of a workgroup's grid-stride slice, valid in thread 0.
template <int XB, int RB>
__device__ __forceinline__ void gate_slice(const char* y, const char* y_ref, const char* r, const char* r_ref, long long n, unsigned tol,
                                           unsigned block, unsigned grid, unsigned& rbad, unsigned& ybad, unsigned& ymax)
{
    using YP = typename gate_piece<XB>::type;
    using RP = typename gate_piece<RB>::type;
    constexpr int E = 16 / XB, RPP = E * RB / 16;        // elements per piece; residual pieces beside it
    rbad = ybad = ymax = 0;
    const unsigned pieces = static_cast<unsigned>(n / E), step = grid * kGateBlock;
    for (unsigned long long p = block * kGateBlock + threadIdx.x; p < pieces; p += step) {
        const addrms::u32x4 a = gate_load<YP>(y + p * 16), b = gate_load<YP>(y_ref + p * 16);
        addrms::u32x4 ra[RPP], rb[RPP];
#pragma unroll
        for (int k = 0; k < RPP; ++k) {
            ra[k] = gate_load<RP>(r + (p * RPP + k) * 16);
            rb[k] = gate_load<RP>(r_ref + (p * RPP + k) * 16);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if constexpr (XB == 4) {
                gate_count_y<4>(a[j], b[j], tol, ybad, ymax);
            } else {
                gate_count_y<2>(a[j] & 0xffffu, b[j] & 0xffffu, tol, ybad, ymax);
                gate_count_y<2>(a[j] >> 16, b[j] >> 16, tol, ybad, ymax);
            }
        }
#pragma unroll
        for (int k = 0; k < RPP; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const unsigned d = ra[k][j] ^ rb[k][j];
                if constexpr (RB == 4) rbad += d != 0u;
                else rbad += ((d & 0xffffu) != 0u) + ((d >> 16) != 0u);
            }
    }
    // the last n % E elements, one per thread of the first workgroup
    const long long i = static_cast<long long>(pieces) * E + threadIdx.x;
    if (block == 0 && i < n) gate_element<XB, RB>(y, y_ref, r, r_ref, i, tol, rbad, ybad, ymax);
    gate_block<0>(rbad, ybad, ymax);
}
template <int XB, int RB>
__global__ __launch_bounds__(kGateBlock) void gate_partial_kernel(addr_t y, addr_t y_ref, addr_t r, addr_t r_ref, long long n,
                                                                   unsigned tol, unsigned grid, addr_t partial)
{
    unsigned rbad, ybad, ymax;
    gate_slice<XB, RB>(at_global<char>(y), at_global<char>(y_ref), at_global<char>(r), at_global<char>(r_ref), n, tol, blockIdx.x, grid,
                       rbad, ybad, ymax);
    if (threadIdx.x == 0)
        at_global<addrms::u32x4>(partial)[blockIdx.x] = addrms::u32x4{rbad, ybad, ymax, 0u};
}
// tells: the first workgroup compares nothing and tells.
template <int XB, int RB>
__global__ __launch_bounds__(kGateBlock) void gate_one_kernel(addr_t y_at, addr_t y_ref_at, addr_t r_at, addr_t r_ref_at, long long n,
                                                               unsigned tol, unsigned grid, addr_t out_at, unsigned unit_looks, uint32_t number,
                                                               addr_t words)
{
    const unsigned unit = unit_looks >> 1 & 0x7fffu, tells = unit_looks & 1u, block = blockIdx.x - tells;
    if (tells && blockIdx.x == 0u) {
        addrms::unit_tell(&gate_reports, at_global<uint32_t>(words), kGateBlock);
        return;
    }
    const char *y = at_global<char>(y_at), *y_ref = at_global<char>(y_ref_at), *r = at_global<char>(r_at), *r_ref = at_global<char>(r_ref_at);
    addrms::u32x4* out = at_global<addrms::u32x4>(out_at);
    unsigned rbad, ybad, ymax;
    gate_slice<XB, RB>(y, y_ref, r, r_ref, n, tol, block, grid, rbad, ybad, ymax);
    if (grid == 1u) {
        if (threadIdx.x == 0) *out = addrms::u32x4{rbad, ybad, ymax, 0u};
        return;
    }
    GateWords* all = gate_words[unit];
    if (block != grid - 1u) {
        if (threadIdx.x == 0) {
            GateWords* w = &all[block];
            gate_put(&w->rbad, rbad, number); gate_put(&w->ybad, ybad, number); gate_put(&w->ymax, ymax, number);
        }
        return;
    }
    if (threadIdx.x != 0) rbad = ybad = ymax = 0u;
    const unsigned looks = unit_looks >> 16;
    const uint32_t expected = looks ? number : ~number;      // not this launch's: nothing is found
    bool without = false;                                    // the word of workgroup threadIdx.x is missing
    if (threadIdx.x < grid - 1u) without = gate_without(&all[threadIdx.x], expected, looks, rbad, ybad, ymax);
    uint64_t left = __ballot(without);
    if (__builtin_expect(left != 0u, 0)) {                   // not expected: its instructions lie behind the kernel's end
        do {
            const unsigned first = (threadIdx.x & ~63u) + static_cast<unsigned>(__builtin_ctzll(left));
            gate_wave_slice<XB, RB>(y, y_ref, r, r_ref, n, tol, static_cast<unsigned>(__builtin_amdgcn_readfirstlane(static_cast<int>(first))),
                                    grid, rbad, ybad, ymax);
            without = without && threadIdx.x != first;
            if (without) without = gate_without(&all[threadIdx.x], expected, 0u, rbad, ybad, ymax);
            left = __ballot(without);
        } while (left);
    }
    gate_block<1>(rbad, ybad, ymax);                         // its barrier: all slices have been counted
    if (threadIdx.x != 0) return;
    *out = addrms::u32x4{rbad, ybad, ymax, 0u};
    addrms::unit_done(&gate_reports.state[unit], number);
}
__global__ __launch_bounds__(kGateBlock) void gate_tell_kernel(addr_t words) { addrms::unit_tell(&gate_reports, at_global<uint32_t>(words), kGateBlock); }
// One workgroup.  accumulate != 0 folds the new counts into what `out` already holds
// (a second comparison graded into the same verdict).
__global__ __launch_bounds__(kGateBlock) void gate_finish_kernel(addr_t partial, int nslots, addr_t out_at, int accumulate)
{
    unsigned* out = at_global<unsigned>(out_at);
    unsigned a = 0, b = 0, c = 0;
#pragma unroll
    for (int k = 0; k < kGateMaxGrid / kGateBlock; ++k) {
        const int s = k * kGateBlock + static_cast<int>(threadIdx.x);
        if (s < nslots) {
            const addrms::u32x4 v = at_global<const addrms::u32x4>(partial)[s];
            a += v.x; b += v.y;
            c = v.z > c ? v.z : c;
        }
    }
    gate_block<0>(a, b, c);
    if (threadIdx.x == 0) {
        if (accumulate) {
            out[0] += a; out[1] += b;
            if (c > out[2]) out[2] = c;
        } else {
            *reinterpret_cast<addrms::u32x4*>(out) = addrms::u32x4{a, b, c, 0u};
        }
    }
}

// Workgroups of the first stage for n elements of xb bytes: a piece per thread until the chip is full.
int gate_grid(long long n, int xb)
{
    const long long per_wg = static_cast<long long>(kGateBlock) * (16 / xb);
    return static_cast<int>(std::max<long long>(1, std::min<long long>(kGateMaxGrid, (n + per_wg - 1) / per_wg)));
}

// Both stages of the gate on `stream`: xb/rb are the element sizes of the y and residual
// streams, `partial` holds at least gate_grid(n, xb) slots, `out` four counters.  Asynchronous.
int launch_gate(const void* y, const void* y_ref, const void* r, const void* r_ref, long long n, int xb, int rb,
                unsigned tol, unsigned* partial, unsigned* out, bool accumulate, hipStream_t stream)
{
    unsigned grid = static_cast<unsigned>(gate_grid(n, xb));
    const void* fn = xb == 4   ? reinterpret_cast<const void*>(&gate_partial_kernel<4, 4>)
                     : rb == 4 ? reinterpret_cast<const void*>(&gate_partial_kernel<2, 4>)
                               : reinterpret_cast<const void*>(&gate_partial_kernel<2, 2>);
    void* args[] = {&y, &y_ref, &r, &r_ref, &n, &tol, &grid, &partial};
    HIP_TRY(hipLaunchKernel(fn, dim3(grid), dim3(kGateBlock), args, 0, stream));
    int slots = static_cast<int>(grid), more = accumulate ? 1 : 0;
    void* last[] = {&partial, &slots, &out, &more};
    HIP_TRY(hipLaunchKernel(reinterpret_cast<const void*>(&gate_finish_kernel), dim3(1), dim3(kGateBlock), last, 0, stream));
    return ADDRMS_OK;
}

SlotPool<kGateUnits> g_gate_slots;

// The gate in one launch, where one workgroup does it or the launch can have a unit.  *launched: whether it was.
int launch_gate_in_one(const void* y, const void* y_ref, const void* r, const void* r_ref, long long n, int xb, int rb, unsigned tol,
                       unsigned looks, unsigned* out, hipStream_t stream, bool* launched)
{
    unsigned workgroups = static_cast<unsigned>(gate_grid(n, xb));
    SlotPool<kGateUnits>::Lease lease;
    const auto tell = [stream](uint32_t* words) {
        void* args[] = {&words};
        return hipLaunchKernel(reinterpret_cast<const void*>(&gate_tell_kernel), dim3(1), dim3(kGateBlock), args, 0, stream);
    };
    *launched = workgroups == 1 || g_gate_slots.take(stream, 1, &lease, tell) == Units::taken;
    if (!*launched) return ADDRMS_OK;
    const bool meet = workgroups > 1;
    unsigned tells = meet && lease.tells() ? 1u : 0u, unit_looks = meet ? std::min(looks, 0xffffu) << 16 | lease.unit() << 1 | tells : 0u;
    uint32_t *words = meet ? lease.words() : nullptr, number = meet ? lease.number() : 0u;
    const void* fn = xb == 4   ? reinterpret_cast<const void*>(&gate_one_kernel<4, 4>)
                     : rb == 4 ? reinterpret_cast<const void*>(&gate_one_kernel<2, 4>)
                               : reinterpret_cast<const void*>(&gate_one_kernel<2, 2>);
    void* args[] = {&y, &y_ref, &r, &r_ref, &n, &tol, &workgroups, &out, &unit_looks, &number, &words};
    // The launch's own status: hipGetLastError may have an older error, of the caller's, for a launch that is queued.
    HIP_TRY(hipLaunchKernel(fn, dim3(workgroups + tells), dim3(kGateBlock), args, 0, stream));
    if (meet) lease.launched();
    return ADDRMS_OK;
}

int fill(void* p, int64_t n, int es, bool bf, uint32_t seed, float lo, float hi, bool bell, hipStream_t st)
{
    if (n == 0) return ADDRMS_OK;
    const dim3 block(256), grid(static_cast<unsigned>((n + 255) / 256));
    if (es == 4) hipLaunchKernelGGL((fill_kernel<4, false>), grid, block, 0, st, p, (long long)n, seed, lo, hi, bell ? 1 : 0);
    else if (bf) hipLaunchKernelGGL((fill_kernel<2, true>), grid, block, 0, st, p, (long long)n, seed, lo, hi, bell ? 1 : 0);
    else hipLaunchKernelGGL((fill_kernel<2, false>), grid, block, 0, st, p, (long long)n, seed, lo, hi, bell ? 1 : 0);
    HIP_TRY(hipGetLastError());
    return ADDRMS_OK;
}

// ---- measurement harness ------------------------------------------------------------
// Owns: one pristine input set, one reference-output set, and `nsets` working
// sets that the timed launches rotate through so that their combined footprint
// exceeds the last-level caches.
struct Harness {
    static constexpr int kOp = OP_ADDRMS;
    int64_t M = 0, N = 0;
    int dtype = 0;
    float eps = 1e-6f;
    int nsets = 0;
    size_t xbytes = 0, rbytes = 0, wbytes = 0;
    char* pool = nullptr;
    char *x0 = nullptr, *r0 = nullptr, *yref = nullptr, *rref = nullptr, *w = nullptr;
    std::vector<char*> xs, rs;
    bool untuned = false;     // measure what a call without a configuration launches
    unsigned* counts = nullptr;
    hipStream_t stream = nullptr;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;
    bool have_ref = false;
    addrms_cfg ref_cfg{};
    int relax = 0;   // efficiency rules switched off (audit only)

    // Buffers start on 64 KiB boundaries; each residual buffer is then skewed by
    // one 4 KiB interleave unit so that the x and residual accesses of a lane,
    // issued together at equal offsets, do not land on the same HBM channel.
    static constexpr size_t kAlign = 64 * 1024, kSkew = 4096;
    static size_t pad(size_t b) { return (b + kAlign - 1) / kAlign * kAlign + kAlign; }

    int init(int64_t m, int64_t n, int dt, float e, bool rotate)
    {
        M = m; N = n; dtype = dt; eps = e;
        xbytes = static_cast<size_t>(M) * N * x_bytes(dt);
        rbytes = static_cast<size_t>(M) * N * r_bytes(dt);
        wbytes = static_cast<size_t>(N) * x_bytes(dt);
        const size_t set = pad(xbytes) + pad(rbytes);
        // enough rotating sets that one lap is four times the last-level cache plus the L2s (with twice, a mid-size
        // shape still measured about 1 % fast: the memory-side cache does not evict in strict order)
        const size_t want = 4 * (static_cast<size_t>(hw().last_level_cache_bytes) +
                                 static_cast<size_t>(hw().l2_bytes_per_xcd) * hw().xcds);
        nsets = rotate ? static_cast<int>(std::min<size_t>(32, std::max<size_t>(2, (want + set - 1) / set))) : 1;
        const size_t total = set * (nsets + 2) + pad(wbytes) + pad(256 + kGateScratchBytes);
        HIP_TRY(hipMalloc(reinterpret_cast<void**>(&pool), total));
        char* p = pool;
        auto take = [&](size_t b, size_t skew) { char* q = p + skew; p += pad(b); return q; };
        x0 = take(xbytes, 0); r0 = take(rbytes, kSkew); yref = take(xbytes, 0); rref = take(rbytes, kSkew);
        w = take(wbytes, 0);
        counts = reinterpret_cast<unsigned*>(take(256 + kGateScratchBytes, 0));   // 4 result counters, then the gate's slots
        for (int i = 0; i < nsets; ++i) { xs.push_back(take(xbytes, 0)); rs.push_back(take(rbytes, kSkew)); }
        HIP_TRY(hipStreamCreateWithFlags(&stream, hipStreamNonBlocking));
        HIP_TRY(hipEventCreate(&ev0));
        HIP_TRY(hipEventCreate(&ev1));
        const bool bf = dt == ADDRMS_BF16;
        int st = fill(x0, M * N, x_bytes(dt), bf, 0x1234567u, 0, 0, true, stream);
        if (st == ADDRMS_OK) st = fill(r0, M * N, r_bytes(dt), bf, 0x89abcdeu, 0, 0, true, stream);
        if (st == ADDRMS_OK) st = fill(w, N, x_bytes(dt), bf, 0x5555aaau, 0.5f, 1.5f, false, stream);
        if (st != ADDRMS_OK) return st;
        for (int i = 0; i < nsets; ++i) {
            HIP_TRY(hipMemcpyAsync(xs[i], x0, xbytes, hipMemcpyDeviceToDevice, stream));
            HIP_TRY(hipMemcpyAsync(rs[i], r0, rbytes, hipMemcpyDeviceToDevice, stream));
        }
        HIP_TRY(hipStreamSynchronize(stream));
        return ADDRMS_OK;
    }

    ~Harness()
    {
        if (ev0) (void)hipEventDestroy(ev0);
        if (ev1) (void)hipEventDestroy(ev1);
        if (stream) (void)hipStreamDestroy(stream);
        if (pool) (void)hipFree(pool);
    }

    int run_on(const addrms_cfg& c, const Feas& f, int set)
    {
        if (untuned) return run_addrms(xs[set], rs[set], w, eps, M, N, dtype, nullptr, stream);
        return launch(f, c, xs[set], rs[set], w, eps, M, N, dtype, stream);
    }

    int make_reference(const addrms_cfg& c)
    {
        const Feas f = check_cfg(c, M, N, dtype);
        if (f.status != ADDRMS_OK) return fail(f.status, "reference cfg infeasible: %s", f.reason.c_str());
        HIP_TRY(hipMemcpyAsync(yref, x0, xbytes, hipMemcpyDeviceToDevice, stream));
        HIP_TRY(hipMemcpyAsync(rref, r0, rbytes, hipMemcpyDeviceToDevice, stream));
        const int st = launch(f, c, yref, rref, w, eps, M, N, dtype, stream);
        if (st != ADDRMS_OK) return st;
        HIP_TRY(hipStreamSynchronize(stream));
        have_ref = true;
        ref_cfg = c;
        return ADDRMS_OK;
    }

    // 0 if cfg reproduces the reference output on the pristine inputs.
    int validate(const addrms_cfg& c)
    {
        const Feas f = check_cfg(c, M, N, dtype, OP_ADDRMS, relax);
        if (f.status != ADDRMS_OK) return f.status;
        HIP_TRY(hipMemcpyAsync(xs[0], x0, xbytes, hipMemcpyDeviceToDevice, stream));
        HIP_TRY(hipMemcpyAsync(rs[0], r0, rbytes, hipMemcpyDeviceToDevice, stream));
        int st = run_on(c, f, 0);
        if (st != ADDRMS_OK) return st;
        st = launch_gate(xs[0], yref, rs[0], rref, static_cast<long long>(M) * N, x_bytes(dtype), r_bytes(dtype), 1u,
                         counts + 64, counts, false, stream);
        if (st != ADDRMS_OK) return st;
        unsigned h[4] = {0, 0, 0, 0};
        HIP_TRY(hipMemcpyAsync(h, counts, 16, hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        if (h[0] != 0 || h[1] != 0)
            return fail(ADDRMS_ERR_INFEASIBLE_CFG, "candidate %s disagrees with the reference: %u residual elements "
                        "differ, %u outputs beyond 1 ulp (max distance %u)", cfg_json(c).c_str(), h[0], h[1], h[2]);
        return ADDRMS_OK;
    }

    int measure(const addrms_cfg& c, int warmup, int reps, double* mean_us)
    {
        const Feas f = check_cfg(c, M, N, dtype, OP_ADDRMS, relax);
        if (f.status != ADDRMS_OK) return fail(f.status, "%s", f.reason.c_str());
        int set = 0;
        for (int i = 0; i < warmup; ++i) {
            const int st = run_on(c, f, set);
            if (st != ADDRMS_OK) return st;
            set = (set + 1) % nsets;
        }
        HIP_TRY(hipEventRecord(ev0, stream));
        for (int i = 0; i < reps; ++i) {
            const int st = run_on(c, f, set);
            if (st != ADDRMS_OK) return st;
            set = (set + 1) % nsets;
        }
        HIP_TRY(hipEventRecord(ev1, stream));
        HIP_TRY(hipEventSynchronize(ev1));
        float ms = 0.0f;
        HIP_TRY(hipEventElapsedTime(&ms, ev0, ev1));
        *mean_us = static_cast<double>(ms) * 1000.0 / reps;
        return ADDRMS_OK;
    }
    // Per-launch timing: an event before and after every launch.
    int measure_stats(const addrms_cfg& c, int warmup, int reps, addrms_time_stats* out)
    {
        const Feas f = check_cfg(c, M, N, dtype);
        if (f.status != ADDRMS_OK) return fail(f.status, "%s", f.reason.c_str());
        double batch = 0.0;
        int st = measure(c, warmup, reps, &batch);
        if (st != ADDRMS_OK) return st;
        std::vector<hipEvent_t> ev(static_cast<size_t>(reps) + 1, nullptr);
        auto destroy = [&] { for (hipEvent_t e : ev) if (e) (void)hipEventDestroy(e); };
        for (hipEvent_t& e : ev)
            if (hipEventCreate(&e) != hipSuccess) { destroy(); return fail(ADDRMS_ERR_HIP, "hipEventCreate failed"); }
        int set = 0;
        hipError_t err = hipEventRecord(ev[0], stream);
        for (int i = 0; i < reps && err == hipSuccess; ++i) {
            st = run_on(c, f, set);
            if (st != ADDRMS_OK) { destroy(); return st; }
            set = (set + 1) % nsets;
            err = hipEventRecord(ev[i + 1], stream);
        }
        if (err == hipSuccess) err = hipEventSynchronize(ev[reps]);
        std::vector<double> us(reps);
        for (int i = 0; i < reps && err == hipSuccess; ++i) {
            float ms = 0.0f;
            err = hipEventElapsedTime(&ms, ev[i], ev[i + 1]);
            us[i] = static_cast<double>(ms) * 1000.0;
        }
        destroy();
        if (err != hipSuccess) return fail(ADDRMS_ERR_HIP, "per-launch timing failed: %s", hipGetErrorString(err));
        std::sort(us.begin(), us.end());
        double sum = 0.0;
        for (double v : us) sum += v;
        out->mean_us = batch;
        out->per_launch_mean_us = sum / reps;
        out->median_us = (reps % 2) ? us[reps / 2] : 0.5 * (us[reps / 2 - 1] + us[reps / 2]);
        out->min_us = us.front();
        out->max_us = us.back();
        out->reps = reps;
        out->buffer_sets = nsets;
        return ADDRMS_OK;
    }
};

std::mutex g_tune_mu;

// ---- measurement harness of silu_and_mul: one pristine input, a reference output, and
// rotating (input, output) pairs; the operator is out of place, so nothing is restored.
struct SiluHarness {
    static constexpr int kOp = OP_SILUMUL;
    int64_t M = 0, d = 0;
    int dtype = 0;
    int nsets = 0;
    size_t inbytes = 0, outbytes = 0;
    char* pool = nullptr;
    char *ref = nullptr;
    std::vector<char*> ins, outs;
    bool untuned = false;     // measure what a call without a configuration launches
    unsigned* counts = nullptr;
    hipStream_t stream = nullptr;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;

    static size_t pad(size_t b) { return (b + 65535) / 65536 * 65536 + 65536; }

    int init(int64_t m, int64_t dd, int dt, float /*eps: the operator has none*/, bool rotate)
    {
        M = m; d = dd; dtype = dt;
        inbytes = static_cast<size_t>(M) * 2 * d * x_bytes(dt);
        outbytes = static_cast<size_t>(M) * d * x_bytes(dt);
        const size_t set = pad(inbytes) + pad(outbytes);
        const size_t want = 4 * (static_cast<size_t>(hw().last_level_cache_bytes) +
                                 static_cast<size_t>(hw().l2_bytes_per_xcd) * hw().xcds);
        nsets = rotate ? static_cast<int>(std::min<size_t>(32, std::max<size_t>(2, (want + set - 1) / set))) : 1;
        HIP_TRY(hipMalloc(reinterpret_cast<void**>(&pool), set * nsets + pad(outbytes) + pad(256 + kGateScratchBytes)));
        char* p = pool;
        auto take = [&](size_t b, size_t skew) { char* q = p + skew; p += pad(b); return q; };
        ref = take(outbytes, 0);
        counts = reinterpret_cast<unsigned*>(take(256 + kGateScratchBytes, 0));
        for (int i = 0; i < nsets; ++i) { ins.push_back(take(inbytes, 0)); outs.push_back(take(outbytes, 4096)); }
        HIP_TRY(hipStreamCreateWithFlags(&stream, hipStreamNonBlocking));
        HIP_TRY(hipEventCreate(&ev0));
        HIP_TRY(hipEventCreate(&ev1));
        const int st = fill(ins[0], M * 2 * d, x_bytes(dt), dt == ADDRMS_BF16, 0x2468aceu, 0, 0, true, stream);
        if (st != ADDRMS_OK) return st;
        for (int i = 1; i < nsets; ++i)
            HIP_TRY(hipMemcpyAsync(ins[i], ins[0], inbytes, hipMemcpyDeviceToDevice, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        return ADDRMS_OK;
    }
    ~SiluHarness()
    {
        if (ev0) (void)hipEventDestroy(ev0);
        if (ev1) (void)hipEventDestroy(ev1);
        if (stream) (void)hipStreamDestroy(stream);
        if (pool) (void)hipFree(pool);
    }
    int make_reference(const addrms_cfg& c)
    {
        const Feas f = check_cfg(c, M, d, dtype, OP_SILUMUL);
        if (f.status != ADDRMS_OK) return fail(f.status, "reference cfg infeasible: %s", f.reason.c_str());
        const int st = launch_silumul(f, c, ins[0], ref, M, d, dtype, stream);
        if (st != ADDRMS_OK) return st;
        HIP_TRY(hipStreamSynchronize(stream));
        return ADDRMS_OK;
    }
    int validate(const addrms_cfg& c)
    {
        const Feas f = check_cfg(c, M, d, dtype, OP_SILUMUL);
        if (f.status != ADDRMS_OK) return f.status;
        HIP_TRY(hipMemsetAsync(outs[0], 0xff, outbytes, stream));     // stale output must not pass for a result
        int st = launch_silumul(f, c, ins[0], outs[0], M, d, dtype, stream);
        if (st != ADDRMS_OK) return st;
        // the residual slots of the comparison are fed the same buffer twice: only the output is graded
        st = launch_gate(outs[0], ref, ref, ref, static_cast<long long>(M) * d, x_bytes(dtype), x_bytes(dtype), 1u,
                         counts + 64, counts, false, stream);
        if (st != ADDRMS_OK) return st;
        unsigned h[4] = {0, 0, 0, 0};
        HIP_TRY(hipMemcpyAsync(h, counts, 16, hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        if (h[1] != 0)
            return fail(ADDRMS_ERR_INFEASIBLE_CFG, "candidate %s disagrees with the reference: %u outputs beyond 1 ulp "
                        "(max distance %u)", cfg_json(c).c_str(), h[1], h[2]);
        return ADDRMS_OK;
    }
    int measure(const addrms_cfg& c, int warmup, int reps, double* mean_us)
    {
        const Feas f = check_cfg(c, M, d, dtype, OP_SILUMUL);
        if (f.status != ADDRMS_OK) return fail(f.status, "%s", f.reason.c_str());
        int set = 0;
        for (int i = 0; i < warmup + reps; ++i) {
            if (i == warmup) HIP_TRY(hipEventRecord(ev0, stream));
            const int st = untuned ? run_silumul(ins[set], outs[set], M, d, dtype, nullptr, stream)
                                   : launch_silumul(f, c, ins[set], outs[set], M, d, dtype, stream);
            if (st != ADDRMS_OK) return st;
            set = (set + 1) % nsets;
        }
        HIP_TRY(hipEventRecord(ev1, stream));
        HIP_TRY(hipEventSynchronize(ev1));
        float ms = 0.0f;
        HIP_TRY(hipEventElapsedTime(&ms, ev0, ev1));
        *mean_us = static_cast<double>(ms) * 1000.0 / reps;
        return ADDRMS_OK;
    }
};
// ---- measurement harness of merge_attn_states: rotating (v_a, v_b, s_a, s_b, v_out, s_out)
// sets plus a reference output; out of place, nothing to restore.
struct MergeHarness {
    static constexpr int kOp = OP_MERGE;
    int64_t rows = 0, d = 0;
    int dtype = 0;
    int nsets = 0;
    size_t vbytes = 0, sbytes = 0;
    char* pool = nullptr;
    char* vref = nullptr;
    float* sref = nullptr;
    struct Set { char *va, *vb, *vo; float *sa, *sb, *so; };
    std::vector<Set> sets;
    bool untuned = false;     // measure what a call without a configuration launches
    unsigned* counts = nullptr;
    hipStream_t stream = nullptr;
    hipEvent_t ev0 = nullptr, ev1 = nullptr;

    static size_t pad(size_t b) { return (b + 65535) / 65536 * 65536 + 65536; }

    int init(int64_t r, int64_t dd, int dt, float /*eps: the operator has none*/, bool rotate)
    {
        rows = r; d = dd; dtype = dt;
        vbytes = static_cast<size_t>(rows) * d * x_bytes(dt);
        sbytes = static_cast<size_t>(rows) * 4;
        const size_t set = 3 * pad(vbytes) + 3 * pad(sbytes);
        const size_t want = 4 * (static_cast<size_t>(hw().last_level_cache_bytes) +
                                 static_cast<size_t>(hw().l2_bytes_per_xcd) * hw().xcds);
        nsets = rotate ? static_cast<int>(std::min<size_t>(32, std::max<size_t>(2, (want + set - 1) / set))) : 1;
        HIP_TRY(hipMalloc(reinterpret_cast<void**>(&pool), set * nsets + pad(vbytes) + pad(sbytes) + pad(256 + kGateScratchBytes)));
        char* p = pool;
        auto take = [&](size_t b, size_t skew) { char* q = p + skew; p += pad(b); return q; };
        vref = take(vbytes, 0);
        sref = reinterpret_cast<float*>(take(sbytes, 0));
        counts = reinterpret_cast<unsigned*>(take(256 + kGateScratchBytes, 0));
        for (int i = 0; i < nsets; ++i) {
            Set s;
            s.va = take(vbytes, 0); s.vb = take(vbytes, 4096); s.vo = take(vbytes, 8192);
            s.sa = reinterpret_cast<float*>(take(sbytes, 0)); s.sb = reinterpret_cast<float*>(take(sbytes, 0));
            s.so = reinterpret_cast<float*>(take(sbytes, 0));
            sets.push_back(s);
        }
        HIP_TRY(hipStreamCreateWithFlags(&stream, hipStreamNonBlocking));
        HIP_TRY(hipEventCreate(&ev0));
        HIP_TRY(hipEventCreate(&ev1));
        const bool bf = dt == ADDRMS_BF16;
        int st = fill(sets[0].va, rows * d, x_bytes(dt), bf, 0x1357911u, 0, 0, true, stream);
        if (st == ADDRMS_OK) st = fill(sets[0].vb, rows * d, x_bytes(dt), bf, 0x2468acfu, 0, 0, true, stream);
        if (st == ADDRMS_OK) st = fill(sets[0].sa, rows, 4, false, 0x0badcafu, -4.0f, 4.0f, false, stream);
        if (st == ADDRMS_OK) st = fill(sets[0].sb, rows, 4, false, 0x0defaceu, -4.0f, 4.0f, false, stream);
        if (st != ADDRMS_OK) return st;
        for (int i = 1; i < nsets; ++i) {
            HIP_TRY(hipMemcpyAsync(sets[i].va, sets[0].va, vbytes, hipMemcpyDeviceToDevice, stream));
            HIP_TRY(hipMemcpyAsync(sets[i].vb, sets[0].vb, vbytes, hipMemcpyDeviceToDevice, stream));
            HIP_TRY(hipMemcpyAsync(sets[i].sa, sets[0].sa, sbytes, hipMemcpyDeviceToDevice, stream));
            HIP_TRY(hipMemcpyAsync(sets[i].sb, sets[0].sb, sbytes, hipMemcpyDeviceToDevice, stream));
        }
        HIP_TRY(hipStreamSynchronize(stream));
        return ADDRMS_OK;
    }
    ~MergeHarness()
    {
        if (ev0) (void)hipEventDestroy(ev0);
        if (ev1) (void)hipEventDestroy(ev1);
        if (stream) (void)hipStreamDestroy(stream);
        if (pool) (void)hipFree(pool);
    }
    int run_set(const Feas& f, const addrms_cfg& c, const Set& s, char* vo, float* so)
    {
        return untuned ? run_mergestates(s.va, s.sa, s.vb, s.sb, vo, so, rows, d, dtype, nullptr, stream)
                       : launch_mergestates(f, c, s.va, s.sa, s.vb, s.sb, vo, so, rows, d, stream);
    }
    int make_reference(const addrms_cfg& c)
    {
        const Feas f = check_cfg(c, rows, d, dtype, OP_MERGE);
        if (f.status != ADDRMS_OK) return fail(f.status, "reference cfg infeasible: %s", f.reason.c_str());
        const int st = run_set(f, c, sets[0], vref, sref);
        if (st != ADDRMS_OK) return st;
        HIP_TRY(hipStreamSynchronize(stream));
        return ADDRMS_OK;
    }
    int validate(const addrms_cfg& c)
    {
        const Feas f = check_cfg(c, rows, d, dtype, OP_MERGE);
        if (f.status != ADDRMS_OK) return f.status;
        HIP_TRY(hipMemsetAsync(sets[0].vo, 0xff, vbytes, stream));
        HIP_TRY(hipMemsetAsync(sets[0].so, 0xff, sbytes, stream));
        const int st = run_set(f, c, sets[0], sets[0].vo, sets[0].so);
        if (st != ADDRMS_OK) return st;
        // merged outputs within 1 ulp of the reference; merged scores bit-identical
        int gs = launch_gate(sets[0].vo, vref, vref, vref, static_cast<long long>(rows) * d, 2, 2, 1u, counts + 64, counts,
                             false, stream);
        if (gs == ADDRMS_OK)
            gs = launch_gate(sets[0].so, sref, sref, sref, static_cast<long long>(rows), 4, 4, 0u, counts + 64, counts, true, stream);
        if (gs != ADDRMS_OK) return gs;
        unsigned h[4] = {0, 0, 0, 0};
        HIP_TRY(hipMemcpyAsync(h, counts, 16, hipMemcpyDeviceToHost, stream));
        HIP_TRY(hipStreamSynchronize(stream));
        if (h[1] != 0)
            return fail(ADDRMS_ERR_INFEASIBLE_CFG, "candidate %s disagrees with the reference on %u values (max "
                        "distance %u)", cfg_json(c).c_str(), h[1], h[2]);
        return ADDRMS_OK;
    }
    int measure(const addrms_cfg& c, int warmup, int reps, double* mean_us)
    {
        const Feas f = check_cfg(c, rows, d, dtype, OP_MERGE);
        if (f.status != ADDRMS_OK) return fail(f.status, "%s", f.reason.c_str());
        int set = 0;
        for (int i = 0; i < warmup + reps; ++i) {
            if (i == warmup) HIP_TRY(hipEventRecord(ev0, stream));
            const int st = run_set(f, c, sets[set], sets[set].vo, sets[set].so);
            if (st != ADDRMS_OK) return st;
            set = (set + 1) % nsets;
        }
        HIP_TRY(hipEventRecord(ev1, stream));
        HIP_TRY(hipEventSynchronize(ev1));
        float ms = 0.0f;
        HIP_TRY(hipEventElapsedTime(&ms, ev0, ev1));
        *mean_us = static_cast<double>(ms) * 1000.0 / reps;
        return ADDRMS_OK;
    }
};
// ---- one implementation of the tuner's device entry points for all three operators --------
// H is the operator's harness (Harness, SiluHarness, MergeHarness): same interface, own buffers,
// own launch and own gate; H::kOp selects the operator's part of the deriver, search and table.
template <class H> int backend_validate(void* user, const addrms_cfg* cfg) { return static_cast<H*>(user)->validate(*cfg); }
template <class H> int backend_measure(void* user, const addrms_cfg* cfg, int warmup, int reps, double* us)
{
    return static_cast<H*>(user)->measure(*cfg, warmup, reps, us);
}

float budget_eps(const addrms_budget* b) { return (b && b->eps > 0.0f) ? b->eps : 1e-6f; }

// S_ref comes from the default cfg; should a tiny M make that one infeasible, from the first feasible cfg.
template <class H> int reference_cfg(int64_t M, int64_t N, int dtype, addrms_cfg* out)
{
    std::string why;
    const int st = default_cfg(N, dtype, out, &why, H::kOp);
    if (st != ADDRMS_OK) return fail(st, "%s", why.c_str());
    if (check_cfg(*out, M, N, dtype, H::kOp).status == ADDRMS_OK) return ADDRMS_OK;
    std::vector<addrms_cfg> v;
    enumerate(M, N, dtype, &v, nullptr, nullptr, H::kOp);
    if (v.empty()) return fail(ADDRMS_ERR_UNSUPPORTED_SHAPE, "feasible region is empty");
    *out = v.front();
    return ADDRMS_OK;
}

// Backend factory over the device harness: one harness per shape, reference output from that shape's default cfg.
struct HarnessFactory { float eps; };
template <class H> int factory_open(void* user, int64_t M, int64_t N, int dtype, addrms_backend* out)
{
    auto* h = new H();
    addrms_cfg ref{};
    int st = reference_cfg<H>(M, N, dtype, &ref);
    if (st == ADDRMS_OK) st = h->init(M, N, dtype, static_cast<HarnessFactory*>(user)->eps, true);
    if (st == ADDRMS_OK) st = h->make_reference(ref);
    if (st != ADDRMS_OK) { delete h; return st; }
    out->user = h;
    out->validate = backend_validate<H>;
    out->measure = backend_measure<H>;
    return 0;
}
template <class H> void factory_close(void*, addrms_backend* be) { delete static_cast<H*>(be->user); }

int check_op_shape(int op, int64_t M, int64_t N, int dtype, const char* what)
{
    if (!dtype_valid(dtype, op)) return fail(ADDRMS_ERR_UNSUPPORTED_DTYPE, "unsupported dtype %d for %s", dtype, op_name(op));
    if (M <= 0 || N <= 0) return fail(ADDRMS_ERR_INVALID_ARG, "%s needs a positive number of rows and a positive row length", what);
    if (!dispatch_consistent()) return fail(ADDRMS_ERR_INVALID_ARG, "library was built with inconsistent kernel tables");
    return ADDRMS_OK;
}

int check_shapes(const addrms_shape* shapes, int32_t n)
{
    if (!shapes) return fail(ADDRMS_ERR_INVALID_ARG, "shapes is NULL");
    if (n < 1 || n > ADDRMS_MAX_SHAPES) return fail(ADDRMS_ERR_INVALID_ARG, "n must be 1..%d", ADDRMS_MAX_SHAPES);
    return ADDRMS_OK;
}

// Algorithm 1 lines 18-21 and 23 for one shape on the current device.
template <class H> int tune_on_device(int64_t M, int64_t N, int dtype, const addrms_budget* budget, addrms_cfg* out_cfg,
                                      addrms_tune_report* report)
{
    if (!out_cfg) return fail(ADDRMS_ERR_INVALID_ARG, "out_cfg is NULL");
    int st = check_op_shape(H::kOp, M, N, dtype, "tuning");
    if (st != ADDRMS_OK) return st;
    std::lock_guard<std::mutex> lock(g_tune_mu);
    addrms_cfg ref{};
    st = reference_cfg<H>(M, N, dtype, &ref);
    if (st != ADDRMS_OK) return st;
    H h;
    st = h.init(M, N, dtype, budget_eps(budget), true);
    if (st != ADDRMS_OK) return st;
    st = h.make_reference(ref);
    if (st != ADDRMS_OK) return st;
    addrms_backend be{&h, backend_validate<H>, backend_measure<H>};
    addrms_tune_report local{};
    st = run_search(M, N, dtype, budget, be, out_cfg, &local, H::kOp, true);
    if (st != ADDRMS_OK) return st;
    if (report) *report = local;
    return table_insert(M, N, dtype, *out_cfg, local.best_us, H::kOp);
}

// Line 22 (SelectGeneral) and the outer loop, over a set of shapes.
template <class H> int select_general_on_device(const addrms_shape* shapes, int32_t n, int dtype, const addrms_budget* budget,
                                                addrms_cfg* out_general, addrms_general_report* report)
{
    if (!dispatch_consistent()) return fail(ADDRMS_ERR_INVALID_ARG, "library was built with inconsistent kernel tables");
    const int st = check_shapes(shapes, n);
    if (st != ADDRMS_OK) return st;
    std::lock_guard<std::mutex> lock(g_tune_mu);
    HarnessFactory hf{budget_eps(budget)};
    addrms_backend_factory fac{&hf, factory_open<H>, factory_close<H>};
    return run_select_general(shapes, n, dtype, budget, fac, true, out_general, report, H::kOp, true);
}
template <class H> int tune_rounds_on_device(const addrms_shape* shapes, int32_t n, int dtype, const addrms_budget* budget,
                                             addrms_cfg* out_general, addrms_rounds_report* report)
{
    if (!dispatch_consistent()) return fail(ADDRMS_ERR_INVALID_ARG, "library was built with inconsistent kernel tables");
    const int st = check_shapes(shapes, n);
    if (st != ADDRMS_OK) return st;
    std::lock_guard<std::mutex> lock(g_tune_mu);
    HarnessFactory hf{budget_eps(budget)};
    addrms_backend_factory fac{&hf, factory_open<H>, factory_close<H>};
    return run_tune_rounds(shapes, n, dtype, budget, fac, true, out_general, report, H::kOp, true);
}

// Mean time of one cfg (NULL: table, else default) on library-allocated buffers.
template <class H> int measure_on_device(const addrms_cfg* cfg, int64_t M, int64_t N, int dtype, float eps, int warmup, int reps,
                                         int rotate, double* mean_us)
{
    if (!mean_us) return fail(ADDRMS_ERR_INVALID_ARG, "mean_us is NULL");
    if (reps <= 0 || warmup < 0) return fail(ADDRMS_ERR_INVALID_ARG, "need reps > 0 and warmup >= 0");
    int st = check_op_shape(H::kOp, M, N, dtype, "measuring");
    if (st != ADDRMS_OK) return st;
    addrms_cfg c{};
    bool untuned = false;
    st = resolve_cfg(cfg, M, N, dtype, &c, H::kOp, &untuned);
    if (st != ADDRMS_OK) return st;
    std::lock_guard<std::mutex> lock(g_tune_mu);
    H h;
    h.untuned = untuned;
    st = h.init(M, N, dtype, eps, rotate != 0);
    if (st != ADDRMS_OK) return st;
    st = h.measure(c, warmup, reps, mean_us);
    if (st != ADDRMS_OK) return st;
    // A standalone measurement starts on a device that has just been idle: its clocks are still rising while a short
    // batch is timed (a 22 us kernel measured 4-5 % slow this way, and not equally for all cfgs).  Where the batch
    // took less than kSettleUs, keep the device busy with the same kernel for that long and time the batch again.
    constexpr double kSettleUs = 30000.0;
    const double batch_us = *mean_us * (warmup + reps);
    if (batch_us < kSettleUs && *mean_us > 0.0) {
        const int extra = static_cast<int>(std::min(20000.0, (kSettleUs - batch_us) / *mean_us));
        double ignored = 0.0;
        if (extra > 0) st = h.measure(c, 0, extra, &ignored);
        if (st == ADDRMS_OK) st = h.measure(c, warmup, reps, mean_us);
    }
    return st;
}

}  // namespace

extern "C" {

int addrms_run(void* x, void* residual, const void* weight, float eps, int64_t M, int64_t N, int dtype,
               const addrms_cfg* cfg, void* stream)
{
    if (!dtype_valid(dtype)) return fail(ADDRMS_ERR_UNSUPPORTED_DTYPE, "unsupported dtype %d", dtype);
    if (M < 0 || N <= 0) return fail(ADDRMS_ERR_INVALID_ARG, "M must be >= 0 and N > 0 (got M=%lld N=%lld)",
                                     (long long)M, (long long)N);
    if (M == 0) return ADDRMS_OK;
    if (!x || !residual || !weight) return fail(ADDRMS_ERR_INVALID_ARG, "x, residual and weight must not be NULL");
    if (M > (1ll << 31) - 1) return fail(ADDRMS_ERR_INVALID_ARG, "M=%lld exceeds the 2^31-1 row limit", (long long)M);
    if (!dispatch_consistent()) return fail(ADDRMS_ERR_INVALID_ARG, "library was built with inconsistent kernel tables");
    return run_addrms(x, residual, weight, eps, M, N, dtype, cfg, static_cast<hipStream_t>(stream));
}

int addrms_tune(int64_t M, int64_t N, int dtype, const addrms_budget* budget, addrms_cfg* out_cfg,
                addrms_tune_report* report)
{
    return tune_on_device<Harness>(M, N, dtype, budget, out_cfg, report);
}

int addrms_select_general(const addrms_shape* shapes, int32_t n, int dtype, const addrms_budget* budget,
                          addrms_cfg* out_general, addrms_general_report* report)
{
    return select_general_on_device<Harness>(shapes, n, dtype, budget, out_general, report);
}

int addrms_tune_rounds(const addrms_shape* shapes, int32_t n, int dtype, const addrms_budget* budget,
                       addrms_cfg* out_general, addrms_rounds_report* report)
{
    return tune_rounds_on_device<Harness>(shapes, n, dtype, budget, out_general, report);
}

int addrms_audit_rules(int64_t M, int64_t N, int dtype, const addrms_budget* budget, addrms_audit_report* report)
{
    if (!report) return fail(ADDRMS_ERR_INVALID_ARG, "report is NULL");
    if (!dtype_valid(dtype)) return fail(ADDRMS_ERR_UNSUPPORTED_DTYPE, "unsupported dtype %d", dtype);
    if (M <= 0 || N <= 0) return fail(ADDRMS_ERR_INVALID_ARG, "the audit needs M > 0 and N > 0");
    if (!dispatch_consistent()) return fail(ADDRMS_ERR_INVALID_ARG, "library was built with inconsistent kernel tables");
    std::lock_guard<std::mutex> lock(g_tune_mu);
    addrms_cfg dflt{};
    int st = reference_cfg<Harness>(M, N, dtype, &dflt);
    if (st != ADDRMS_OK) return st;
    Harness h;
    st = h.init(M, N, dtype, budget_eps(budget), true);
    if (st != ADDRMS_OK) return st;
    st = h.make_reference(dflt);     // the reference comes from a configuration every rule retains
    if (st != ADDRMS_OK) return st;
    h.relax = RELAX_ALL;
    addrms_backend be{&h, backend_validate<Harness>, backend_measure<Harness>};
    return run_audit_rules(M, N, dtype, budget, be, report);
}

int addrms_measure(const addrms_cfg* cfg, int64_t M, int64_t N, int dtype, float eps, int warmup, int reps,
                   int rotate, double* mean_us)
{
    return measure_on_device<Harness>(cfg, M, N, dtype, eps, warmup, reps, rotate, mean_us);
}

int addrms_measure_stats(const addrms_cfg* cfg, int64_t M, int64_t N, int dtype, float eps, int warmup, int reps,
                         int rotate, addrms_time_stats* out)
{
    if (!out) return fail(ADDRMS_ERR_INVALID_ARG, "out is NULL");
    if (!dtype_valid(dtype)) return fail(ADDRMS_ERR_UNSUPPORTED_DTYPE, "unsupported dtype %d", dtype);
    if (M <= 0 || N <= 0 || reps <= 0 || reps > 100000 || warmup < 0)
        return fail(ADDRMS_ERR_INVALID_ARG, "need M, N > 0, 0 < reps <= 100000 and warmup >= 0");
    if (!dispatch_consistent()) return fail(ADDRMS_ERR_INVALID_ARG, "library was built with inconsistent kernel tables");
    addrms_cfg c{};
    bool untuned = false;
    int st = resolve_cfg(cfg, M, N, dtype, &c, OP_ADDRMS, &untuned);
    if (st != ADDRMS_OK) return st;
    std::lock_guard<std::mutex> lock(g_tune_mu);
    Harness h;
    h.untuned = untuned;
    st = h.init(M, N, dtype, eps, rotate != 0);
    if (st != ADDRMS_OK) return st;
    memset(out, 0, sizeof *out);
    return h.measure_stats(c, warmup, reps, out);
}

int addrms_device_resources(const addrms_cfg* cfg, int64_t M, int64_t N, int dtype, addrms_resources* out)
{
    if (!cfg || !out) return fail(ADDRMS_ERR_INVALID_ARG, "cfg and out must not be NULL");
    if (!dispatch_consistent()) return fail(ADDRMS_ERR_INVALID_ARG, "library was built with inconsistent kernel tables");
    const Feas f = check_cfg(*cfg, M, N, dtype);
    if (f.status != ADDRMS_OK) return fail(f.status, "%s", f.reason.c_str());
    memset(out, 0, sizeof *out);
    hipFuncAttributes attr;
    HIP_TRY(hipFuncGetAttributes(&attr, kDispatch[f.inst].fn));
    const int threads = cfg->threads_per_row * cfg->rows_per_wg;
    int wgs = 0;
    HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&wgs, kDispatch[f.inst].fn, threads,
                                                         static_cast<size_t>(f.dyn_lds)));
    out->chunks_per_thread = f.res.chunks_per_thread;
    out->vgprs = attr.numRegs;
    out->scratch_bytes = static_cast<int32_t>(attr.localSizeBytes);
    out->lds_bytes = static_cast<int32_t>(attr.sharedSizeBytes) + f.dyn_lds;
    out->max_threads = attr.maxThreadsPerBlock;
    out->waves_per_wg = threads / hw().wave_size;
    out->wgs_per_cu = wgs;
    out->waves_per_simd = (wgs * out->waves_per_wg + hw().simds_per_cu - 1) / hw().simds_per_cu;
    return ADDRMS_OK;
}

int addrms_rstd_probe(const double* ss, int64_t n, int64_t N, float eps, float* out, void* stream)
{
    if (n < 0 || N <= 0) return fail(ADDRMS_ERR_INVALID_ARG, "need n >= 0 and N > 0");
    if (n == 0) return ADDRMS_OK;
    if (!ss || !out) return fail(ADDRMS_ERR_INVALID_ARG, "ss and out must not be NULL");
    const dim3 block(256), grid(static_cast<unsigned>((n + 255) / 256));
    hipLaunchKernelGGL(rstd_probe_kernel, grid, block, 0, static_cast<hipStream_t>(stream), ss, (long long)n,
                       1.0 / static_cast<double>(N), eps, out);
    HIP_TRY(hipGetLastError());
    return ADDRMS_OK;
}

// The plan of addrms_run without a configuration, for problems whose rows it splits.
static int split_plan(const void* x, const void* residual, const void* weight, int64_t M, int64_t N, int dtype, DirectPlan* p)
{
    if (!dtype_valid(dtype)) return fail(ADDRMS_ERR_UNSUPPORTED_DTYPE, "unsupported dtype %d", dtype);
    if (M < 0 || N <= 0) return fail(ADDRMS_ERR_INVALID_ARG, "M must be >= 0 and N > 0");
    if (M == 0) return ADDRMS_OK;
    if (!x || !residual || !weight) return fail(ADDRMS_ERR_INVALID_ARG, "x, residual and weight must not be NULL");
    if (M > (1ll << 31) - 1) return fail(ADDRMS_ERR_INVALID_ARG, "M=%lld exceeds the 2^31-1 row limit", (long long)M);
    addrms_cfg c{};
    std::string why;
    const int st = default_cfg(N, dtype, &c, &why);
    if (st != ADDRMS_OK) return fail(st, "%s", why.c_str());
    const int xa = c.vec * x_bytes(dtype);
    if (!aligned(x, xa) || !aligned(weight, xa) || !aligned(residual, std::min(16, c.vec * r_bytes(dtype))))
        return fail(ADDRMS_ERR_MISALIGNED, "tensors must be aligned as addrms_run asks for");
    if (!direct_addrms_plan(M, N, dtype, c.vec, bits(x), bits(residual), bits(weight), p) || !p->split_fn)
        return fail(ADDRMS_ERR_UNSUPPORTED_SHAPE, "rows of this problem are not split over workgroups");
    return ADDRMS_OK;
}

int addrms_split_probe(void* x, void* residual, const void* weight, float eps, int64_t M, int64_t N, int dtype, uint32_t patience,
                       void* stream)
{
    DirectPlan p;
    const int st = split_plan(x, residual, weight, M, N, dtype, &p);
    if (st != ADDRMS_OK || M == 0) return st;
    int e = 0;
    bool capturing = false;
    const int64_t rows = direct_launch_split(p, x, residual, weight, eps, M, N, dtype, patience, stream, &e, &capturing);
    HIP_TRY(static_cast<hipError_t>(e));
    if (rows < M) return fail(ADDRMS_ERR_NO_RESULT, "the call can have no units for split rows now (%lld rows are launched)", (long long)rows);
    return ADDRMS_OK;
}

int addrms_whole_rows_probe(void* x, void* residual, const void* weight, float eps, int64_t M, int64_t N, int dtype, int captured,
                            void* stream)
{
    DirectPlan p;
    const int st = split_plan(x, residual, weight, M, N, dtype, &p);
    if (st != ADDRMS_OK || M == 0) return st;
    HIP_TRY(static_cast<hipError_t>(captured ? direct_launch_whole(p, x, residual, weight, eps, M, N, stream)
                                             : direct_launch_alone(p, x, residual, weight, eps, M, N, stream)));
    return ADDRMS_OK;
}

int addrms_stream_probe(void* x, void* residual, int64_t M, int64_t N, int dtype, void* stream)
{
    if (!dtype_valid(dtype)) return fail(ADDRMS_ERR_UNSUPPORTED_DTYPE, "unsupported dtype %d", dtype);
    if (M < 0 || N <= 0) return fail(ADDRMS_ERR_INVALID_ARG, "M must be >= 0 and N > 0");
    if (M == 0) return ADDRMS_OK;
    if (!x || !residual) return fail(ADDRMS_ERR_INVALID_ARG, "x and residual must not be NULL");
    const int64_t xb = M * N * x_bytes(dtype), rb = M * N * r_bytes(dtype);
    if (xb % 16 != 0 || !aligned(x, 16) || !aligned(residual, 16))
        return fail(ADDRMS_ERR_MISALIGNED, "the probe moves 16 bytes per lane: M*N*element size must be a multiple of 16 "
                    "and both bases 16-byte aligned");
    const long long n = xb / 16;
    const dim3 block(256), grid(static_cast<unsigned>((n + 255) / 256));
    addrms::u32x4* xa = static_cast<addrms::u32x4*>(x);
    addrms::u32x4* ra = static_cast<addrms::u32x4*>(residual);
    if (rb == xb)
        hipLaunchKernelGGL(stream_probe_kernel<1>, grid, block, kProbeLdsBytes, static_cast<hipStream_t>(stream), xa, ra, n);
    else if (rb == 2 * xb)
        hipLaunchKernelGGL(stream_probe_kernel<2>, grid, block, kProbeLdsBytes, static_cast<hipStream_t>(stream), xa, ra, n);
    else
        return fail(ADDRMS_ERR_INVALID_ARG, "unexpected residual/x size ratio");
    HIP_TRY(hipGetLastError());
    return ADDRMS_OK;
}

int addrms_row_probe(void* x, void* residual, int64_t M, int64_t N, int dtype, int threads_per_row, int wgs_per_cu,
                     void* stream)
{
    if (!dtype_valid(dtype)) return fail(ADDRMS_ERR_UNSUPPORTED_DTYPE, "unsupported dtype %d", dtype);
    if (M < 0 || N <= 0) return fail(ADDRMS_ERR_INVALID_ARG, "M must be >= 0 and N > 0");
    if (M == 0) return ADDRMS_OK;
    if (!x || !residual) return fail(ADDRMS_ERR_INVALID_ARG, "x and residual must not be NULL");
    if (M > 0x7fffffffLL) return fail(ADDRMS_ERR_UNSUPPORTED_SHAPE, "one workgroup per row: M must fit a grid dimension");
    const int64_t row_xb = N * x_bytes(dtype), row_rb = N * r_bytes(dtype);
    if (row_xb % 16 != 0 || !aligned(x, 16) || !aligned(residual, 16))
        return fail(ADDRMS_ERR_MISALIGNED, "the probe moves 16 bytes per lane: a row of x must be a multiple of 16 bytes "
                    "and both bases 16-byte aligned");
    if (threads_per_row < 64 || threads_per_row > 1024 || threads_per_row % 64 != 0)
        return fail(ADDRMS_ERR_INVALID_ARG, "threads_per_row must be a multiple of 64 in [64, 1024]");
    if (wgs_per_cu < 0 || wgs_per_cu > 16) return fail(ADDRMS_ERR_INVALID_ARG, "wgs_per_cu must be in [0, 16]");
    const int64_t pieces = row_xb / 16;
    const int64_t chunks = (pieces + threads_per_row - 1) / threads_per_row;
    if (chunks > 16 || (chunks - 1) * threads_per_row >= pieces)
        return fail(ADDRMS_ERR_INFEASIBLE_CFG, "threads_per_row must cover the row in at most 16 pieces per thread");
    int cpt = 0;
    const void* fn = nullptr;
    if (row_rb == row_xb) fn = row_probe_instance<1>(static_cast<int>(chunks), &cpt);
    else if (row_rb == 2 * row_xb) fn = row_probe_instance<2>(static_cast<int>(chunks), &cpt);
    else return fail(ADDRMS_ERR_INVALID_ARG, "unexpected residual/x size ratio");
    if (!fn) return fail(ADDRMS_ERR_INFEASIBLE_CFG, "no probe instance for %d pieces per thread", static_cast<int>(chunks));
    // occupancy cap by LDS padding, as the operator's cfgs impose theirs
    // (just more than would let one more workgroup fit)
    const unsigned lds = wgs_per_cu > 0 ? static_cast<unsigned>(160 * 1024 / (wgs_per_cu + 1) / 1280 * 1280 + 1280) : 0u;
    if (lds > 64u * 1024u) HIP_TRY(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024));
    addrms::u32x4* xa = static_cast<addrms::u32x4*>(x);
    addrms::u32x4* ra = static_cast<addrms::u32x4*>(residual);
    long long m = M;
    unsigned np = static_cast<unsigned>(pieces);
    void* args[] = {&xa, &ra, &m, &np};
    HIP_TRY(hipLaunchKernel(fn, dim3(static_cast<unsigned>(M)), dim3(static_cast<unsigned>(threads_per_row)), args, lds,
                            static_cast<hipStream_t>(stream)));
    return ADDRMS_OK;
}

// ---- the gate on caller buffers ----------------------------------------------------------

namespace {
int check_gate_args(const void* y, const void* y_ref, const void* r, const void* r_ref, int64_t n, int dtype,
                    const addrms_gate_counts* out)
{
    if (!dtype_valid(dtype)) return fail(ADDRMS_ERR_UNSUPPORTED_DTYPE, "unsupported dtype %d", dtype);
    if (n < 0) return fail(ADDRMS_ERR_INVALID_ARG, "n must be >= 0 (got %lld)", (long long)n);
    if (n > kGateMaxElems)
        return fail(ADDRMS_ERR_INVALID_ARG, "n=%lld exceeds the %lld elements the gate's 32-bit counters can count",
                    (long long)n, kGateMaxElems);
    if (!out) return fail(ADDRMS_ERR_INVALID_ARG, "counts_out is NULL");
    if (n > 0 && (!y || !y_ref || !r || !r_ref)) return fail(ADDRMS_ERR_INVALID_ARG, "y, y_ref, residual and residual_ref must not be NULL");
    if (!aligned(y, x_bytes(dtype)) || !aligned(y_ref, x_bytes(dtype)) || !aligned(r, r_bytes(dtype)) ||
        !aligned(r_ref, r_bytes(dtype)) || !aligned(out, 16))
        return fail(ADDRMS_ERR_MISALIGNED, "tensors must be aligned to their element size and counts_out to 16 bytes");
    return ADDRMS_OK;
}

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned* g_scratch_ptr[kMaxDevices];

// Device address of `scratch` on the current device, looked up on the first call there.
int gate_scratch_on_current_device(unsigned** out)
{
    int dev = -1;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return fail(ADDRMS_ERR_HIP, "device ordinal %d outside 0..%d", dev, kMaxDevices - 1);
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        unsigned* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(reinterpret_cast<void**>(&p), HIP_SYMBOL(scratch)));
        if (!p) return fail(ADDRMS_ERR_HIP, "hipGetSymbolAddress returned a null address for the gate scratch");
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return ADDRMS_OK;
}
}  // namespace

int addrms_gate_probe(const void* y, const void* y_ref, const void* residual, const void* residual_ref, int64_t n,
                      int dtype, uint32_t tol, addrms_gate_counts* counts_out, void* stream)
{
    int st = check_gate_args(y, y_ref, residual, residual_ref, n, dtype, counts_out);
    if (st != ADDRMS_OK) return st;
    hipStream_t s = static_cast<hipStream_t>(stream);
    if (n == 0) { HIP_TRY(hipMemsetAsync(counts_out, 0, sizeof *counts_out, s)); HIP_TRY(hipStreamSynchronize(s)); return ADDRMS_OK; }
    unsigned* partial = nullptr;
    HIP_TRY(hipMalloc(reinterpret_cast<void**>(&partial), static_cast<size_t>(gate_grid(n, x_bytes(dtype))) * 4 * sizeof(unsigned)));
    st = launch_gate(y, y_ref, residual, residual_ref, n, x_bytes(dtype), r_bytes(dtype), tol, partial,
                     reinterpret_cast<unsigned*>(counts_out), false, s);
    const hipError_t e = hipStreamSynchronize(s);
    (void)hipFree(partial);
    if (st != ADDRMS_OK) return st;
    if (e != hipSuccess) return fail(ADDRMS_ERR_HIP, "hipStreamSynchronize failed: %s", hipGetErrorString(e));
    return ADDRMS_OK;
}

int addrms_gate_looks_probe(const void* y, const void* y_ref, const void* residual, const void* residual_ref, int64_t n,
                            int dtype, uint32_t tol, uint32_t looks, addrms_gate_counts* counts_out, void* stream)
{
    int st = check_gate_args(y, y_ref, residual, residual_ref, n, dtype, counts_out);
    if (st != ADDRMS_OK) return st;
    bool launched = false;
    st = launch_gate_in_one(y, y_ref, residual, residual_ref, n, x_bytes(dtype), r_bytes(dtype), tol, looks,
                            reinterpret_cast<unsigned*>(counts_out), static_cast<hipStream_t>(stream), &launched);
    if (st != ADDRMS_OK || launched) return st;
    return fail(ADDRMS_ERR_NO_RESULT, "the comparison could not be one launch");
}

int addrms_gate_probe_noalloc(const void* y, const void* y_ref, const void* residual, const void* residual_ref, int64_t n,
                              int dtype, uint32_t tol, addrms_gate_counts* counts_out, void* stream)
{
    int st = check_gate_args(y, y_ref, residual, residual_ref, n, dtype, counts_out);
    if (st != ADDRMS_OK) return st;
    bool launched = false;
    st = launch_gate_in_one(y, y_ref, residual, residual_ref, n, x_bytes(dtype), r_bytes(dtype), tol, gate_looks(n),
                            reinterpret_cast<unsigned*>(counts_out), static_cast<hipStream_t>(stream), &launched);
    if (st != ADDRMS_OK || launched) return st;
    unsigned* partial = nullptr;
    st = gate_scratch_on_current_device(&partial);
    if (st != ADDRMS_OK) return st;
    // n == 0 goes through the kernels as well (one workgroup, empty slice): nothing here may be a memset
    // that a capturing caller would record
    return launch_gate(y, y_ref, residual, residual_ref, n, x_bytes(dtype), r_bytes(dtype), tol, partial,
                       reinterpret_cast<unsigned*>(counts_out), false, static_cast<hipStream_t>(stream));
}

// ---- silu_and_mul ----------------------------------------------------------------------

int silumul_run(const void* x, void* out, int64_t M, int64_t d, int dtype, const addrms_cfg* cfg, void* stream)
{
    if (!dtype_valid(dtype, OP_SILUMUL)) return fail(ADDRMS_ERR_UNSUPPORTED_DTYPE, "unsupported dtype %d for silu_and_mul", dtype);
    if (M < 0 || d <= 0) return fail(ADDRMS_ERR_INVALID_ARG, "M must be >= 0 and d > 0 (got M=%lld d=%lld)",
                                     (long long)M, (long long)d);
    if (M == 0) return ADDRMS_OK;
    if (!x || !out) return fail(ADDRMS_ERR_INVALID_ARG, "x and out must not be NULL");
    if (M > (1ll << 31) - 1) return fail(ADDRMS_ERR_INVALID_ARG, "M=%lld exceeds the 2^31-1 row limit", (long long)M);
    if (!dispatch_consistent()) return fail(ADDRMS_ERR_INVALID_ARG, "library was built with inconsistent kernel tables");
    return run_silumul(x, out, M, d, dtype, cfg, static_cast<hipStream_t>(stream));
}

int silumul_default_cfg(int64_t d, int dtype, addrms_cfg* out) { return export_default_cfg(OP_SILUMUL, d, dtype, out); }

int silumul_cfg_feasible(const addrms_cfg* cfg, int64_t M, int64_t d, int dtype, char* reason, size_t reason_len,
                         addrms_resources* res)
{
    return export_cfg_feasible(OP_SILUMUL, cfg, M, d, dtype, reason, reason_len, res);
}

int64_t silumul_enumerate_feasible(int64_t M, int64_t d, int dtype, addrms_cfg* out, int64_t cap, int64_t* n_grid)
{
    return export_enumerate_feasible(OP_SILUMUL, M, d, dtype, out, cap, n_grid);
}

int silumul_tune_with_backend(int64_t M, int64_t d, int dtype, const addrms_budget* budget, const addrms_backend* backend,
                              addrms_cfg* out_cfg, addrms_tune_report* report)
{
    if (!backend) return fail(ADDRMS_ERR_INVALID_ARG, "backend is NULL");
    return run_search(M, d, dtype, budget, *backend, out_cfg, report, OP_SILUMUL);
}

int silumul_tune(int64_t M, int64_t d, int dtype, const addrms_budget* budget, addrms_cfg* out_cfg,
                 addrms_tune_report* report)
{
    return tune_on_device<SiluHarness>(M, d, dtype, budget, out_cfg, report);
}

int silumul_select_general(const addrms_shape* shapes, int32_t n, int dtype, const addrms_budget* budget,
                           addrms_cfg* out_general, addrms_general_report* report)
{
    return select_general_on_device<SiluHarness>(shapes, n, dtype, budget, out_general, report);
}

int silumul_tune_rounds(const addrms_shape* shapes, int32_t n, int dtype, const addrms_budget* budget,
                        addrms_cfg* out_general, addrms_rounds_report* report)
{
    return tune_rounds_on_device<SiluHarness>(shapes, n, dtype, budget, out_general, report);
}

int silumul_measure(const addrms_cfg* cfg, int64_t M, int64_t d, int dtype, int warmup, int reps, int rotate,
                    double* mean_us)
{
    return measure_on_device<SiluHarness>(cfg, M, d, dtype, 0.0f, warmup, reps, rotate, mean_us);
}

int silumul_table_lookup(int64_t M, int64_t d, int dtype, addrms_cfg* out) { return export_table_lookup(OP_SILUMUL, M, d, dtype, out); }

int64_t silumul_algorithmic_bytes(int64_t M, int64_t d, int dtype) { return export_algorithmic_bytes(OP_SILUMUL, M, d, dtype); }

// ---- merge_attn_states -----------------------------------------------------------------

int mergestates_run(const void* v_a, const float* s_a, const void* v_b, const float* s_b, void* v_out, float* s_out,
                    int64_t rows, int64_t d, int dtype, const addrms_cfg* cfg, void* stream)
{
    if (!dtype_valid(dtype, OP_MERGE)) return fail(ADDRMS_ERR_UNSUPPORTED_DTYPE, "unsupported dtype %d for merge_attn_states", dtype);
    if (rows < 0 || d <= 0) return fail(ADDRMS_ERR_INVALID_ARG, "rows must be >= 0 and d > 0 (got rows=%lld d=%lld)",
                                        (long long)rows, (long long)d);
    if (rows == 0) return ADDRMS_OK;
    if (!v_a || !s_a || !v_b || !s_b || !v_out || !s_out) return fail(ADDRMS_ERR_INVALID_ARG, "no pointer may be NULL");
    if (rows > (1ll << 31) - 1) return fail(ADDRMS_ERR_INVALID_ARG, "rows=%lld exceeds the 2^31-1 limit", (long long)rows);
    if (!dispatch_consistent()) return fail(ADDRMS_ERR_INVALID_ARG, "library was built with inconsistent kernel tables");
    return run_mergestates(v_a, s_a, v_b, s_b, v_out, s_out, rows, d, dtype, cfg, static_cast<hipStream_t>(stream));
}

int mergestates_default_cfg(int64_t d, int dtype, addrms_cfg* out) { return export_default_cfg(OP_MERGE, d, dtype, out); }

int mergestates_cfg_feasible(const addrms_cfg* cfg, int64_t rows, int64_t d, int dtype, char* reason, size_t reason_len,
                         addrms_resources* res)
{
    return export_cfg_feasible(OP_MERGE, cfg, rows, d, dtype, reason, reason_len, res);
}

int64_t mergestates_enumerate_feasible(int64_t rows, int64_t d, int dtype, addrms_cfg* out, int64_t cap, int64_t* n_grid)
{
    return export_enumerate_feasible(OP_MERGE, rows, d, dtype, out, cap, n_grid);
}

int mergestates_tune_with_backend(int64_t rows, int64_t d, int dtype, const addrms_budget* budget, const addrms_backend* backend,
                              addrms_cfg* out_cfg, addrms_tune_report* report)
{
    if (!backend) return fail(ADDRMS_ERR_INVALID_ARG, "backend is NULL");
    return run_search(rows, d, dtype, budget, *backend, out_cfg, report, OP_MERGE);
}

int mergestates_tune(int64_t rows, int64_t d, int dtype, const addrms_budget* budget, addrms_cfg* out_cfg,
                 addrms_tune_report* report)
{
    return tune_on_device<MergeHarness>(rows, d, dtype, budget, out_cfg, report);
}

int mergestates_select_general(const addrms_shape* shapes, int32_t n, int dtype, const addrms_budget* budget,
                           addrms_cfg* out_general, addrms_general_report* report)
{
    return select_general_on_device<MergeHarness>(shapes, n, dtype, budget, out_general, report);
}

int mergestates_tune_rounds(const addrms_shape* shapes, int32_t n, int dtype, const addrms_budget* budget,
                        addrms_cfg* out_general, addrms_rounds_report* report)
{
    return tune_rounds_on_device<MergeHarness>(shapes, n, dtype, budget, out_general, report);
}

int mergestates_measure(const addrms_cfg* cfg, int64_t rows, int64_t d, int dtype, int warmup, int reps, int rotate,
                    double* mean_us)
{
    return measure_on_device<MergeHarness>(cfg, rows, d, dtype, 0.0f, warmup, reps, rotate, mean_us);
}

int mergestates_table_lookup(int64_t rows, int64_t d, int dtype, addrms_cfg* out) { return export_table_lookup(OP_MERGE, rows, d, dtype, out); }

int64_t mergestates_algorithmic_bytes(int64_t rows, int64_t d, int dtype) { return export_algorithmic_bytes(OP_MERGE, rows, d, dtype); }

}  // extern "C"

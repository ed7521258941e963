// Kernels behind a call that names no configuration and has none in the specialised table.
// They are not points of the knob grid: their launch shape follows from the problem by the
// rules in direct_route.cpp.
//
// Store policy.  A workgroup's ordinary stores leave dirty lines in its XCD's L2, which are
// written back when the kernel ends: a serial tail of up to 32 MB.  Non-temporal stores have
// no such tail, but nothing of them stays in the memory-side cache either, where the next
// kernel of the program looks for its input.  Write-through stores (sc1) go to the memory
// side as they are issued and stay there.  Which one a problem takes is decided by what it
// writes (write_through_max in direct_route.cpp has both sides measured).  Loads are
// non-temporal too, except where a wave shares lines with the waves beside it (POL_SHARED).
//
// Ragged rows (RAG).  A row length that VEC does not divide used to mean accesses as narrow
// as one element, and one that 128 bytes do not divide waves whose lines are shared with the
// waves beside them.  Here the walk of a row begins at the cache line its first element lies
// in, so that every wave covers whole lines; the pieces of VEC elements inside the row go to
// the lanes, and the fewer than 2 * VEC elements before its first and after its last whole
// piece to the first lanes, one each.
#pragma once
#include <type_traits>

#include "addrms_kernel.h"
#include "direct_route.h"
#include "silumul_kernel.h"
#include "unit_report.h"

namespace addrms {

template <typename T, int AL> struct at_align { typedef T type __attribute__((aligned(AL))); };

// Load of BYTES bytes at base + off, an address that is a multiple of AL, and aligned store; base
// is the same for the whole wave.  The write-through policy exists for buffer stores only (their
// cache-policy operand).
template <int POL, int BYTES, int AL>
__device__ __forceinline__ void ld_stream(const char* base, uint64_t off, raw_t<BYTES>& v)
{
    constexpr bool NT = POL == POL_NT || POL == POL_WT;
    if constexpr (AL >= 16 || AL >= BYTES) {
        ld_raw<BYTES, NT>(base + off, v);
    } else {
        static_assert(BYTES == 8 || BYTES == 16, "one access");
        using V = typename at_align<typename std::conditional<BYTES == 16, u32x4, u32x2>::type, AL>::type;
        const V* p = reinterpret_cast<const V*>(base + off);
        V t;
        if constexpr (NT) t = __builtin_nontemporal_load(p);
        else t = *p;
#pragma unroll
        for (int k = 0; k < BYTES / 4; ++k) v.d[k] = t[k];
    }
}
template <int POL, int BYTES>
__device__ __forceinline__ void st_stream(char* base, uint32_t off, const raw_t<BYTES>& v)
{
    if constexpr (POL == POL_WT || POL == POL_SHARED) {
        st_write_through<BYTES>(base, off, v);
    } else {
        st_raw<BYTES, POL == POL_NT>(base + off, v);
    }
}

// The columns of one row as a workgroup's lanes walk them: lane `lane` of `tpr` takes the VEC elements from
// col0 + c * stride on, for c = 0, 1, ...  Ragged: `into` elements of the row's first cache line belong to the row
// before it; `head` elements precede the row's first whole piece, which is a whole piece of both streams (the host
// checked that they have the same phase), and lane i of the first ones has the single element `single`.
template <int XB, int VEC, bool RAG>
struct RowWalk {
    static constexpr int32_t LINE = 128 / XB;
    int32_t into, head, nlast, col0, stride;
    uint32_t single;
    bool has_single;
    __device__ __forceinline__ RowWalk(const char* xbase, uint32_t rowoff, int32_t N, uint32_t lane, uint32_t tpr)
    {
        into = RAG ? static_cast<int32_t>((static_cast<uint32_t>(reinterpret_cast<uintptr_t>(xbase)) / XB + rowoff) % LINE) : 0;
        head = RAG ? (LINE - into) % VEC : 0;
        const int32_t nv = RAG ? head + (N - head) / VEC * VEC : N;       // end of the last whole piece
        nlast = nv - VEC;
        col0 = static_cast<int32_t>(lane) * VEC - into;
        stride = static_cast<int32_t>(tpr) * VEC;
        single = static_cast<int32_t>(lane) < head ? lane : static_cast<uint32_t>(nv - head) + lane;
        has_single = RAG && single < static_cast<uint32_t>(N);
    }
    __device__ __forceinline__ bool in_row(int32_t col) const
    {
        return RAG ? static_cast<uint32_t>(col) <= static_cast<uint32_t>(nlast) : col <= nlast;
    }
    __device__ __forceinline__ uint32_t clamped(int32_t col) const         // idle lanes re-read valid data
    {
        const int32_t c = RAG && col < head ? head : col;
        return static_cast<uint32_t>(c < nlast ? c : nlast);
    }
};
// A lane's single element from the loads to the stores (nothing where rows are not ragged).
template <int DT, bool RAG>
struct SingleElement {
    using T = dt_traits<DT>;
    static constexpr int XB = T::XB, RB = T::RB;
    raw_t<XB> x{}, w{};
    raw_t<RB> r{};
    float h = 0.0f;
    // KEEP: ordinary loads, which leave the line to the pieces beside the elements and to the next row; else non-temporal ones
    // (direct_addrms_route has the rule).
    template <bool KEEP>
    __device__ __forceinline__ void load(const char* xrow, const char* rrow, const char* wbase, uint32_t at, bool mine)
    {
        if (RAG && mine) {
            ld_raw<XB, !KEEP>(xrow + static_cast<uint64_t>(at * XB), x);
            ld_raw<RB, !KEEP>(rrow + static_cast<uint64_t>(at * RB), r);
            ld_raw<XB, false>(wbase + static_cast<uint64_t>(at * XB), w);
        }
    }
    __device__ __forceinline__ double add(double acc)                      // 0 where a lane has none
    {
        if constexpr (RAG) {
            h = get_elem<XB, T::BF>(x, 0) + get_elem<RB, T::BF && RB == 2>(r, 0);
            const double hd = static_cast<double>(h);
            acc = __builtin_fma(hd, hd, acc);
        }
        return acc;
    }
    template <bool NT = true>
    __device__ __forceinline__ void store(char* xrow, char* rrow, uint32_t at, bool mine, float rstd) const
    {
        if (RAG && mine) {
            float f[1] = {h};
            raw_t<RB> rout;
            pack_vec<RB, T::BF, 1>(f, rout);
            st_raw<RB, NT>(rrow + static_cast<uint64_t>(at * RB), rout);
            const float t = h * rstd;
            f[0] = t * get_elem<XB, T::BF>(w, 0);
            raw_t<XB> yout;
            pack_vec<XB, T::BF, 1>(f, yout);
            st_raw<XB, NT>(xrow + static_cast<uint64_t>(at * XB), yout);
        }
    }
};

// ---- add + RMSNorm ---------------------------------------------------------------------------
// A workgroup per row (MULTI: several, for rows shorter than a wave and ragged ones), a thread
// holds CPT chunks of VEC elements from the loads to the stores.  Same arithmetic as addrms_body,
// element by element; the sum over a row is taken in fp64 as there, but in another order, so that
// rstd may round to the neighbouring fp32 value in some 1e-7 of rows.
// HBM-bound: all loads of a thread are issued before the first value is used (in two
// batches beyond 32 values), and a row is spread over many threads with few chunks each, so that it
// arrives early.  DEFER (more than one chunk): both streams written after the row sum, 1-3 % there.
// Times: us per launch, back to back in a graph, on three sets of buffers in rotation unless said
// otherwise, each pair from one run on one card (a kernel's own duration in a trace is the same within
// 0.3).
// With written-through stores and up to two chunks the weights are fetched along with the row, so
// that nothing is loaded behind a store (64 x 8192 bf16 3.4 -> 3.0, 400 x 6144 4.7 -> 4.0, 2048 x
// 1024 4.0 -> 3.8, 1000 x 4096 fp32 10.3 -> 10.1); with non-temporal ones they are fetched after it
// (20000 x 5120 bf16 126, along with it 133), and with three or more chunks after the row sum, where
// their registers are free and their odd addresses in ragged rows hold nothing up (300 x 10001 7.8 ->
// 6.7, 900 x 28672 39.3 -> 38.8, 1800 x 3001 fp16+fp32 the same and from HBM 14.0 -> 13.6; with one
// chunk 9000 x 6150 72.4 -> 75.1, 20000 x 5120 126 -> 127).
// Default of the knob grid -> here: 16 x 4096 bf16 2.9 -> 2.3, 64 x 8192 3.8 -> 3.0, 512 x 8192 8.0 ->
// 5.7, 4096 x 4096 20.9 -> 19.8, 20000 x 5120 146 -> 127 (6.5 TB/s), 32768 x 7168 329 -> 298, 2048 x
// 8192 fp32 56.1 -> 45.3, 900 x 28672 fp16 43.2 -> 38.7.
// Ragged: 2047 x 4095 fp16 18.0 -> 12.9 (from HBM 27.2 -> 13.3), 9000 x 6150 bf16 91 -> 73, 300 x
// 10001 8.9 -> 6.7, 8192 x 1000 fp16+fp32 17.9 -> 15.5 (from HBM 23.1 -> 18.7); the single elements
// cost the first 0.7 and weights at odd addresses 0.4 of what an aligned row would not.
template <int DT, int VEC, int CPT, int POL, bool RAG, bool DEFER, bool MULTI, bool KEEP>
__device__ __forceinline__ void addrms_direct_body(void* __restrict__ xp, void* __restrict__ rp,
                                                   const void* __restrict__ wp, float eps, double inv_n, int32_t N,
                                                   uint32_t tpr, uint32_t rpw, int64_t M)
{
    using T = dt_traits<DT>;
    constexpr int XB = T::XB, RB = T::RB;
    constexpr int UNR = VEC * CPT <= 32 ? CPT : (CPT + 1) / 2;
    constexpr bool BF = T::BF, EARLY_WEIGHTS = (POL == POL_WT || POL == POL_SHARED) && CPT <= 2, LAST_WEIGHTS = POL == POL_NT && CPT >= 3;
    extern __shared__ double lds[];

    const uint32_t lane = threadIdx.x, ry = MULTI ? threadIdx.y : 0u;
    RowAddr ra;
    if constexpr (MULTI) {
        ra = row_addr<XB, RB>(xp, rp, blockIdx.x, rpw, ry, M, N);
    } else {
        ra.xbase = static_cast<char*>(xp) + static_cast<int64_t>(blockIdx.x) * N * XB;
        ra.rbase = static_cast<char*>(rp) + static_cast<int64_t>(blockIdx.x) * N * RB;
        ra.rowoff = 0u;
        ra.row_ok = 1u;
    }
    const char* wbase = static_cast<const char*>(wp);
    char *xrow = ra.xbase + static_cast<uint64_t>(ra.rowoff * XB), *rrow = ra.rbase + static_cast<uint64_t>(ra.rowoff * RB);
    const RowWalk<XB, VEC, RAG> rw(ra.xbase, ra.rowoff, N, lane, tpr);
    const int32_t col0 = rw.col0, stride = rw.stride;

    float h[CPT][VEC];
    double acc = 0.0;
    SingleElement<DT, RAG> one;
    one.template load<KEEP>(xrow, rrow, wbase, rw.single, rw.has_single);
    raw_t<XB * VEC> wv[CPT];
    auto load_weights = [&] {
#pragma unroll
        for (int c = 0; c < CPT; ++c)
            ld_stream<POL_CACHED, XB * VEC, RAG ? XB : 16>(wbase, rw.clamped(col0 + c * stride) * XB, wv[c]);
    };
#pragma unroll
    for (int g = 0; g < CPT; g += UNR) {
        raw_t<XB * VEC> xv[UNR];
        raw_t<RB * VEC> rv[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            if (g + u < CPT) {
                const uint32_t colc = rw.clamped(col0 + (g + u) * stride);
                ld_stream<POL, XB * VEC, 16>(ra.xbase, (ra.rowoff + colc) * XB, xv[u]);
                ld_stream<POL, RB * VEC, 16>(ra.rbase, (ra.rowoff + colc) * RB, rv[u]);
            }
        }
        if constexpr (EARLY_WEIGHTS) {
            if (g == 0) load_weights();
            __builtin_amdgcn_sched_barrier(0);
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            if (g + u < CPT) {
                const int c = g + u;
                const int32_t col = col0 + c * stride;
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    h[c][e] = get_elem<XB, BF>(xv[u], e) + get_elem<RB, BF && RB == 2>(rv[u], e);
                if (ra.row_ok && rw.in_row(col)) {
                    if constexpr (!DEFER) {
                        raw_t<RB * VEC> out;
                        pack_vec<RB, BF, VEC>(h[c], out);
                        st_stream<POL, RB * VEC>(ra.rbase, (ra.rowoff + col) * RB, out);
                    }
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        const double hd = static_cast<double>(h[c][e]);
                        acc = __builtin_fma(hd, hd, acc);
                    }
                }
            }
        }
        if (g + UNR < CPT) __builtin_amdgcn_sched_barrier(0);
    }
    acc = one.add(acc);
    if constexpr (!EARLY_WEIGHTS && !LAST_WEIGHTS) load_weights();

    const double ss = row_sum(acc, RED_WAVE, tpr, lane, ry, lds);
    if constexpr (LAST_WEIGHTS) load_weights();
    const float rstd = rsqrt_to_f32(__builtin_fma(ss, inv_n, static_cast<double>(eps)));

    if constexpr (DEFER) {
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const int32_t col = col0 + c * stride;
            if (ra.row_ok && rw.in_row(col)) {
                raw_t<RB * VEC> out;
                pack_vec<RB, BF, VEC>(h[c], out);
                st_stream<POL, RB * VEC>(ra.rbase, (ra.rowoff + col) * RB, out);
            }
        }
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int32_t col = col0 + c * stride;
        float y[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const float t = h[c][e] * rstd;
            y[e] = t * get_elem<XB, BF>(wv[c], e);
        }
        if (ra.row_ok && rw.in_row(col)) {
            raw_t<XB * VEC> out;
            pack_vec<XB, BF, VEC>(y, out);
            st_stream<POL, XB * VEC>(ra.xbase, (ra.rowoff + col) * XB, out);
        }
    }
    one.store(xrow, rrow, rw.single, rw.has_single && ra.row_ok, rstd);
}

// ---- add + RMSNorm, rows beyond the registers ---------------------------------------------------
// For captured launches, which can have no units (slot_map.h), rows longer than 16 parts hold, and what
// direct_addrms_split leaves.  The walk of addrms_hybrid_body (its comment has the three parts: registers, parked in LDS, read
// twice) for one row per workgroup, with the store policy of the size, ragged rows, and the weights
// of the register part fetched before the row sum, so that its stores are the first to follow it
// (1-3 % against fetching each behind the stores before it).  Bound by one workgroup filling a CU:
// it reads its row, then writes it, and nothing else runs there meanwhile.  Write-through stores
// lose here (1024 x 131072 bf16 234 us against 211): the next loads wait for their acknowledgement.
// Default of the knob grid -> here, us on three sets of buffers: 1024 x 131072 bf16 246 -> 208, 2048 x
// 65536 219 -> 193, 4096 x 40960 261 -> 227, 300 x 110592 74 -> 56, 230 x 86912 fp32 85 -> 58, 500 x
// 200000 fp32 404 -> 352, 230 x 86912 bf16 33 -> 25; ragged rows, which were read one to four elements
// at a time: 300 x 33333 bf16 39 -> 21, 700 x 99991 236 -> 108, 100 x 180001 111 -> 37.  Called again
// and again on one set of 100 to 250 MB, which the memory-side cache just holds, the default's ordinary
// accesses are ahead (166 x 120004 fp32 51 against 69; 86 against 69 on three sets).
template <int DT, int VEC, int CPT, int UNR, int POL, bool RAG>
__device__ __forceinline__ void addrms_long_body(void* __restrict__ xp, void* __restrict__ rp,
                                                 const void* __restrict__ wp, float eps, double inv_n, int32_t N,
                                                 uint32_t lds_chunks)
{
    using T = dt_traits<DT>;
    constexpr int XB = T::XB, RB = T::RB;
    constexpr bool BF = T::BF;
    extern __shared__ double lds[];

    constexpr uint32_t tpr = kLongThreads;
    const uint32_t lane = threadIdx.x;
    char* xbase = static_cast<char*>(xp) + static_cast<int64_t>(blockIdx.x) * N * XB;
    char* rbase = static_cast<char*>(rp) + static_cast<int64_t>(blockIdx.x) * N * RB;
    const char* wbase = static_cast<const char*>(wp);
    const RowWalk<XB, VEC, RAG> rw(xbase, 0u, N, lane, tpr);
    const int32_t col0 = rw.col0, stride = rw.stride;
    const int32_t need = (N + (RAG ? 128 / XB - 1 : 0) + stride - 1) / stride;    // chunks per thread
    const int32_t parked = static_cast<int32_t>(lds_chunks), streamed = CPT + parked;
    float* cache = reinterpret_cast<float*>(lds + 16) + lane * VEC;                // behind one fp64 slot per wave

    float h[CPT][VEC];
    double acc = 0.0;
    auto load = [&](int32_t col, raw_t<XB * VEC>& x, raw_t<RB * VEC>& r) {
        const uint32_t c = rw.clamped(col);
        ld_stream<POL, XB * VEC, 16>(xbase, c * XB, x);
        ld_stream<POL, RB * VEC, 16>(rbase, c * RB, r);
    };
    auto weight = [&](int32_t col, raw_t<XB * VEC>& w) {
        ld_stream<POL_CACHED, XB * VEC, RAG ? XB : 16>(wbase, rw.clamped(col) * XB, w);
    };
    auto sum = [&](const raw_t<XB * VEC>& x, const raw_t<RB * VEC>& r, float (&s)[VEC]) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) s[e] = get_elem<XB, BF>(x, e) + get_elem<RB, BF && RB == 2>(r, e);
    };
    auto square = [&](const float (&s)[VEC]) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const double hd = static_cast<double>(s[e]);
            acc = __builtin_fma(hd, hd, acc);
        }
    };
    auto put_residual = [&](int32_t col, const float (&s)[VEC]) {
        raw_t<RB * VEC> out;
        pack_vec<RB, BF, VEC>(s, out);
        st_stream<POL, RB * VEC>(rbase, static_cast<uint32_t>(col) * RB, out);
    };
    auto put_y = [&](int32_t col, const float (&s)[VEC], const raw_t<XB * VEC>& w, float rstd) {
        float y[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const float t = s[e] * rstd;
            y[e] = t * get_elem<XB, BF>(w, e);
        }
        raw_t<XB * VEC> out;
        pack_vec<XB, BF, VEC>(y, out);
        st_stream<POL, XB * VEC>(xbase, static_cast<uint32_t>(col) * XB, out);
    };

    SingleElement<DT, RAG> one;
    one.template load<false>(xbase, rbase, wbase, rw.single, rw.has_single);
    // ---- register part
#pragma unroll
    for (int g = 0; g < CPT; g += UNR) {
        raw_t<XB * VEC> xv[UNR];
        raw_t<RB * VEC> rv[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) load(col0 + (g + u) * stride, xv[u], rv[u]);
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int32_t col = col0 + (g + u) * stride;
            sum(xv[u], rv[u], h[g + u]);
            if (rw.in_row(col)) {
                put_residual(col, h[g + u]);
                square(h[g + u]);
            }
        }
        if (g + UNR < CPT) __builtin_amdgcn_sched_barrier(0);
    }
    // ---- LDS part
    for (int32_t c0 = 0; c0 < parked; c0 += UNR) {
        raw_t<XB * VEC> xv[UNR];
        raw_t<RB * VEC> rv[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) load(col0 + (CPT + c0 + u) * stride, xv[u], rv[u]);
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int32_t col = col0 + (CPT + c0 + u) * stride;
            if (c0 + u < parked) {
                float s[VEC];
                sum(xv[u], rv[u], s);
                if (rw.in_row(col)) {
                    put_residual(col, s);
                    square(s);
                }
                float* slot = cache + static_cast<uint32_t>(c0 + u) * (tpr * VEC);
#pragma unroll
                for (int e = 0; e < VEC; ++e) slot[e] = s[e];
            }
        }
    }
    // ---- part that is read twice, first time: the sum only (ordinary loads: the second asks for the same lines)
    for (int32_t c0 = streamed; c0 < need; c0 += UNR) {
        raw_t<XB * VEC> xv[UNR];
        raw_t<RB * VEC> rv[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const uint32_t c = rw.clamped(col0 + (c0 + u) * stride);
            ld_raw<XB * VEC>(xbase + static_cast<uint64_t>(c * XB), xv[u]);
            ld_raw<RB * VEC>(rbase + static_cast<uint64_t>(c * RB), rv[u]);
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            float s[VEC];
            sum(xv[u], rv[u], s);
            if (rw.in_row(col0 + (c0 + u) * stride)) square(s);
        }
    }
    acc = one.add(acc);

    raw_t<XB * VEC> wreg[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) weight(col0 + c * stride, wreg[c]);
    const double ss = row_sum(acc, RED_WAVE, tpr, lane, 0u, lds);
    const float rstd = rsqrt_to_f32(__builtin_fma(ss, inv_n, static_cast<double>(eps)));

#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int32_t col = col0 + c * stride;
        if (rw.in_row(col)) put_y(col, h[c], wreg[c], rstd);
    }
    // ---- read twice, second time, backwards: what was read last is nearest
    for (int32_t k = need; k > streamed;) {
        const int32_t c0 = k - UNR > streamed ? k - UNR : streamed;
        raw_t<XB * VEC> xv[UNR], wv[UNR];
        raw_t<RB * VEC> rv[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            load(col0 + (c0 + u) * stride, xv[u], rv[u]);
            weight(col0 + (c0 + u) * stride, wv[u]);
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int32_t col = col0 + (c0 + u) * stride;
            if (c0 + u < k && rw.in_row(col)) {
                float s[VEC];
                sum(xv[u], rv[u], s);
                put_residual(col, s);
                put_y(col, s, wv[u], rstd);
            }
        }
        k = c0;
    }
    // ---- LDS part
    for (int32_t c0 = 0; c0 < parked; c0 += UNR) {
        raw_t<XB * VEC> wv[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) weight(col0 + (CPT + c0 + u) * stride, wv[u]);
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int32_t col = col0 + (CPT + c0 + u) * stride;
            if (c0 + u < parked && rw.in_row(col)) {
                const float* slot = cache + static_cast<uint32_t>(c0 + u) * (tpr * VEC);
                float s[VEC];
#pragma unroll
                for (int e = 0; e < VEC; ++e) s[e] = slot[e];
                put_y(col, s, wv[u], rstd);
            }
        }
    }
    one.store(xbase, rbase, rw.single, rw.has_single, rstd);
}

// ---- add + RMSNorm, rows beyond the registers, split over several workgroups ---------------------
// What bounds addrms_long_body is that one workgroup fills a CU and cannot hold its row: loads and stores take turns, and
// what neither registers nor LDS keep is read twice.  Here `parts` workgroups share a row, a part each, held in registers
// from the loads to the stores as in addrms_direct_body, so that a CU has several of them at different places of their
// work and nothing is read twice.  They meet once, for the sum over the row: each puts the sum of its part into words of the
// row's SplitRow and reads those of the others.
//
// Nothing has to be cleared for that.  A sum is two words, each with half of its bits and the launch's tag, which no other launch
// with these units has or had (slot_pool.h), so that what earlier ones left is told from a sum of this one.  Both are read at once,
// and those of up to eight parts are one cache line: three words of 22 bits of sum each, in three lines, 172.2 us against 170.6 for
// 1024 x 131072 bf16.  Words that had to be 0 before a launch, cleared by the last workgroup of a row to have read them, took 0.3-0.6
// us at the launch's end.
//
// No wait depends on which workgroups are on the chip.  A workgroup that finds a sum missing for long forms it itself, in the order
// in which its owner does, and puts it into the first word with a compare-and-swap that finds no sum of this launch there: no one has
// read a sum before that word is there, outputs are written only after all sums have been read, and so the inputs were untouched
// while the sum was formed.  Where the owner or another workgroup was first, the sum formed here, perhaps of outputs, goes nowhere.  An owner that comes late writes the same bits once more.  So every workgroup waits either for
// one that runs or for a sum that it may form.
//
// Words and counts are accessed with relaxed atomics of device scope, which go to the memory side of all XCDs' L2s, and
// carry all that the workgroups tell each other, so that nothing else has to be made visible.  A workgroup that has read a row's
// words, its own writes to them long over, counts itself; the last one of each row reports the row (unit_report.h), and when all
// rows have been, the units may be another launch's.  Nobody waits for what that takes.  Against words that are cleared and a report
// to host memory, through the binding on buffers in rotation: 1 x 200000 bf16 6.0 -> 4.8 us, 64 x 55296 7.5 -> 6.2, 330 x 120896 58.7 ->
// 56.0, 1024 x 131072 173.3 -> 170.4.
//
// A row's words and its count lie on 128-byte lines of their own: with eight rows to a line the atomics of a row's
// neighbours queue up, some 10 ns per workgroup of the launch (1024 x 131072 bf16 in 32 parts 281 us against 213).
// 1024 x 131072 bf16 208 -> 170 us (6.3 TB/s), 46 x 164992 fp16 25.9 -> 12.0, through the binding on buffers in rotation; more
// shapes at direct_addrms_split.  Not for rows that the registers of one workgroup hold: 2048 x 8192 fp32 in two parts 47.5
// against 45.0.
struct __align__(128) SplitRow {
    uint64_t word[kSplitParts][2];                           // tag, and the upper and the lower half of a part's sum
    __align__(128) uint32_t read;                            // workgroups that have read all words; 0 again with the last one
};

// The sum over the squares of part `part`, formed by one wave in the order in which the part's own tpr threads form it.
template <int DT, int VEC, int CPT, bool RAG>
__device__ __forceinline__ double split_part_sum(const char* xrow, const char* rrow, const char* wbase, int32_t N, uint32_t part,
                                                 uint32_t tpr)
{
    using T = dt_traits<DT>;
    constexpr int XB = T::XB, RB = T::RB;
    constexpr bool BF = T::BF;
    double mine = 0.0;                                       // lane w: sum of the part's wave w
    for (uint32_t w = 0; w * 64u < tpr; ++w) {
        const RowWalk<XB, VEC, RAG> rw(xrow, 0u, N, w * 64u + threadIdx.x, tpr);
        double acc = 0.0;
        // The wave holds its own part meanwhile, and what this needs on top decides how many workgroups a CU holds (fp32 62 registers, unrolled
        // 78: 500 x 200000 276 us against 307; 16-bit ragged rows 80, unrolled 79 or, for fp16, 81, which are one workgroup less).
#pragma unroll 1
        for (int c = 0; c < CPT; ++c) {
            const int32_t col = rw.col0 + (static_cast<int32_t>(part) * CPT + c) * rw.stride;
            const uint32_t colc = rw.clamped(col);
            raw_t<XB * VEC> x;
            raw_t<RB * VEC> r;
            ld_stream<POL_CACHED, XB * VEC, 16>(xrow, colc * XB, x);
            ld_stream<POL_CACHED, RB * VEC, 16>(rrow, colc * RB, r);
            if (rw.in_row(col)) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const double hd = static_cast<double>(get_elem<XB, BF>(x, e) + get_elem<RB, BF && RB == 2>(r, e));
                    acc = __builtin_fma(hd, hd, acc);
                }
            }
        }
        SingleElement<DT, RAG> one;
        one.template load<true>(xrow, rrow, wbase, rw.single, rw.has_single && part == 0u);
        const double sum = wave_total(one.add(acc));
        if (threadIdx.x == w) mine = sum;
    }
    return tpr == 64u ? read_lane(mine, 0) : read_lane(row16_scan(threadIdx.x < 16u ? mine : 0.0), 15);
}

// Called by the first wave: puts the part's sum into its words and returns the sum over the row once all are there.
// patience: reads of the words after which a sum that is still missing is formed here.
template <int DT, int VEC, int CPT, bool RAG>
__device__ __forceinline__ double split_row_sum(double part_sum, SplitRow* row, uint32_t tag, uint32_t part, uint32_t parts,
                                                uint32_t patience, const char* xrow, const char* rrow, const char* wbase, int32_t N,
                                                uint32_t tpr)
{
    constexpr int kSc1 = 16;
    const __amdgpu_buffer_rsrc_t words = __builtin_amdgcn_make_buffer_rsrc(row, 0, sizeof(row->word), 0x00027000);
    const auto word = [&](uint32_t half) { return static_cast<uint64_t>(tag) << 32 | half; };
    if (threadIdx.x == 0u) {
        const uint64_t s = __builtin_bit_cast(uint64_t, part_sum);
        const u32x4 both = {static_cast<uint32_t>(s >> 32), tag, static_cast<uint32_t>(s), tag};
        __builtin_amdgcn_raw_buffer_store_b128(both, words, part * 16u, 0, kSc1);
    }
    double sums;                                             // lane q: of part q, and 0 without one
    for (uint32_t reads = 0;; ++reads) {
        uint32_t lane = threadIdx.x;
        asm volatile("" : "+v"(lane));                       // what is formed from it is not worth registers while a sum is formed
        bool first = true, all = true;
        sums = 0.0;
        if (lane < parts) {
            asm volatile("" ::: "memory");                   // read anew each time
            const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(words, lane * 16u, 0, kSc1);
            first = v[1] == tag;
            all = first && v[3] == tag;
            sums = __builtin_bit_cast(double, static_cast<uint64_t>(v[0]) << 32 | v[2]);
        }
        if (__all(all)) break;
        // A sum whose first word is there will have the other soon.  The one to form is the next behind this workgroup's own.
        const uint32_t missing = static_cast<uint32_t>(__ballot(!first));
        if (missing && reads >= patience) {
            const uint32_t behind = missing & ~0u << part;
            const uint32_t q = static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(__builtin_ctz(behind ? behind : missing)));
            const uint64_t sum = __builtin_bit_cast(uint64_t, split_part_sum<DT, VEC, CPT, RAG>(xrow, rrow, wbase, N, q, tpr));
            lane = threadIdx.x;
            asm volatile("" : "+v"(lane));
            if (lane == 0u) {
                uint64_t* w = row->word[q];
                uint64_t now = __hip_atomic_load(&w[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if (now >> 32 != tag && __hip_atomic_compare_exchange_strong(&w[0], &now, word(static_cast<uint32_t>(sum >> 32)), __ATOMIC_RELAXED,
                                                                             __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                    __hip_atomic_store(&w[1], word(static_cast<uint32_t>(sum)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
        __builtin_amdgcn_s_sleep(4);
    }
    return wave_total(sums);
}

template <int DT, int VEC, int CPT, int POL, bool RAG>
__device__ __forceinline__ void addrms_split_body(void* __restrict__ xp, void* __restrict__ rp, const void* __restrict__ wp, double inv_n,
                                                  float eps, int32_t N, uint32_t tpr, uint32_t parts, uint32_t M, uint32_t at_row,
                                                  SplitRow* rows, uint64_t* state, uint32_t tag, uint32_t number, uint32_t patience)
{
    using T = dt_traits<DT>;
    constexpr int XB = T::XB, RB = T::RB;
    constexpr bool BF = T::BF;
    extern __shared__ double lds[];                          // one sum per wave, then the row's

    const uint32_t part = blockIdx.x, lane = threadIdx.x;
    SplitRow* row = rows + at_row;
    char* xrow = static_cast<char*>(xp) + static_cast<int64_t>(at_row) * N * XB;
    char* rrow = static_cast<char*>(rp) + static_cast<int64_t>(at_row) * N * RB;
    const char* wbase = static_cast<const char*>(wp);
    const RowWalk<XB, VEC, RAG> rw(xrow, 0u, N, lane, tpr);
    const int32_t stride = rw.stride, col0 = rw.col0 + static_cast<int32_t>(part) * CPT * stride;
    const bool has_single = rw.has_single && part == 0u;

    float h[CPT][VEC];
    double acc = 0.0;
    SingleElement<DT, RAG> one;
    one.template load<true>(xrow, rrow, wbase, rw.single, has_single);
    raw_t<XB * VEC> xv[CPT];
    raw_t<RB * VEC> rv[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const uint32_t colc = rw.clamped(col0 + c * stride);
        ld_stream<POL, XB * VEC, 16>(xrow, colc * XB, xv[c]);
        ld_stream<POL, RB * VEC, 16>(rrow, colc * RB, rv[c]);
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
#pragma unroll
        for (int e = 0; e < VEC; ++e) h[c][e] = get_elem<XB, BF>(xv[c], e) + get_elem<RB, BF && RB == 2>(rv[c], e);
        if (rw.in_row(col0 + c * stride)) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                const double hd = static_cast<double>(h[c][e]);
                acc = __builtin_fma(hd, hd, acc);
            }
        }
    }
    const double part_sum = row_sum(one.add(acc), RED_WAVE, tpr, lane, 0u, lds);
    raw_t<XB * VEC> wv[CPT];                                 // on their way while the sums meet
#pragma unroll
    for (int c = 0; c < CPT; ++c) ld_stream<POL_CACHED, XB * VEC, RAG ? XB : 16>(wbase, rw.clamped(col0 + c * stride) * XB, wv[c]);
    __builtin_amdgcn_sched_barrier(0);
    uint32_t before = 0;                                     // workgroups that had read the words earlier
    if (lane < 64u) {
        const double total = split_row_sum<DT, VEC, CPT, RAG>(part_sum, row, tag, part, parts, patience, xrow, rrow, wbase, N, tpr);
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // the wave's own stores to words are over
        if (lane == 0u) {
            lds[16] = total;
            before = __builtin_amdgcn_atomic_inc32(&row->read, parts - 1u, __ATOMIC_RELAXED, "agent");
        }
    }
    wg_sync_lds();
    const float rstd = rsqrt_to_f32(__builtin_fma(lds[16], inv_n, static_cast<double>(eps)));

#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int32_t col = col0 + c * stride;
        if (rw.in_row(col)) {
            raw_t<RB * VEC> out;
            pack_vec<RB, BF, VEC>(h[c], out);
            st_stream<POL, RB * VEC>(rrow, static_cast<uint32_t>(col) * RB, out);
        }
    }
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const int32_t col = col0 + c * stride;
        float y[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const float t = h[c][e] * rstd;
            y[e] = t * get_elem<XB, BF>(wv[c], e);
        }
        if (rw.in_row(col)) {
            raw_t<XB * VEC> out;
            pack_vec<XB, BF, VEC>(y, out);
            st_stream<POL, XB * VEC>(xrow, static_cast<uint32_t>(col) * XB, out);
        }
    }
    one.template store<false>(xrow, rrow, rw.single, has_single, rstd);

    if (lane < 64u && static_cast<uint32_t>(__builtin_amdgcn_readfirstlane(static_cast<int>(before))) == parts - 1u && lane == 0u)
        unit_piece_done(state, number, at_row, M);
}

// The same rows by one workgroup each, for a call that finds no units for the kernel above: whatever made it find none, its
// results are that kernel's.  The workgroup forms the parts' sums one after the other, as each part's own would, adds them as
// split_row_sum does, and then reads its row again.  Rarely run, and simple rather than fast: 1024 x 131072 bf16 311 us against
// 173 split.
template <int DT, int VEC, int CPT, bool RAG>
__device__ __forceinline__ void addrms_alone_body(void* __restrict__ xp, void* __restrict__ rp, const void* __restrict__ wp, double inv_n,
                                                  float eps, int32_t N, uint32_t tpr, uint32_t parts)
{
    using T = dt_traits<DT>;
    constexpr int XB = T::XB, RB = T::RB;
    constexpr bool BF = T::BF;
    extern __shared__ double lds[];                          // one sum per wave, twice

    const uint32_t lane = threadIdx.x;
    char* xrow = static_cast<char*>(xp) + static_cast<int64_t>(blockIdx.x) * N * XB;
    char* rrow = static_cast<char*>(rp) + static_cast<int64_t>(blockIdx.x) * N * RB;
    const char* wbase = static_cast<const char*>(wp);
    const RowWalk<XB, VEC, RAG> rw(xrow, 0u, N, lane, tpr);
    const int32_t stride = rw.stride;
    SingleElement<DT, RAG> one;
    one.template load<true>(xrow, rrow, wbase, rw.single, rw.has_single);

    double mine = 0.0;                                       // lane p of a wave: sum of part p
    for (uint32_t part = 0; part < parts; ++part) {
        const int32_t col0 = rw.col0 + static_cast<int32_t>(part) * CPT * stride;
        raw_t<XB * VEC> xv[CPT];
        raw_t<RB * VEC> rv[CPT];
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const uint32_t colc = rw.clamped(col0 + c * stride);
            ld_stream<POL_CACHED, XB * VEC, 16>(xrow, colc * XB, xv[c]);
            ld_stream<POL_CACHED, RB * VEC, 16>(rrow, colc * RB, rv[c]);
        }
        double acc = 0.0;
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            if (rw.in_row(col0 + c * stride)) {
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const double hd = static_cast<double>(get_elem<XB, BF>(xv[c], e) + get_elem<RB, BF && RB == 2>(rv[c], e));
                    acc = __builtin_fma(hd, hd, acc);
                }
            }
        }
        if (part == 0u) acc = one.add(acc);
        const double sum = row_sum(acc, RED_WAVE, tpr, lane, part & 1u, lds);
        if ((lane & 63u) == part) mine = sum;
    }
    const float rstd = rsqrt_to_f32(__builtin_fma(wave_total(mine), inv_n, static_cast<double>(eps)));

    for (uint32_t part = 0; part < parts; ++part) {
        const int32_t col0 = rw.col0 + static_cast<int32_t>(part) * CPT * stride;
        raw_t<XB * VEC> xv[CPT], wv[CPT];
        raw_t<RB * VEC> rv[CPT];
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const uint32_t colc = rw.clamped(col0 + c * stride);
            ld_stream<POL_CACHED, XB * VEC, 16>(xrow, colc * XB, xv[c]);
            ld_stream<POL_CACHED, RB * VEC, 16>(rrow, colc * RB, rv[c]);
            ld_stream<POL_CACHED, XB * VEC, RAG ? XB : 16>(wbase, colc * XB, wv[c]);
        }
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const int32_t col = col0 + c * stride;
            float h[VEC], y[VEC];
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                h[e] = get_elem<XB, BF>(xv[c], e) + get_elem<RB, BF && RB == 2>(rv[c], e);
                const float t = h[e] * rstd;
                y[e] = t * get_elem<XB, BF>(wv[c], e);
            }
            if (rw.in_row(col)) {
                raw_t<RB * VEC> rout;
                pack_vec<RB, BF, VEC>(h, rout);
                st_stream<POL_CACHED, RB * VEC>(rrow, static_cast<uint32_t>(col) * RB, rout);
                raw_t<XB * VEC> yout;
                pack_vec<XB, BF, VEC>(y, yout);
                st_stream<POL_CACHED, XB * VEC>(xrow, static_cast<uint32_t>(col) * XB, yout);
            }
        }
    }
    one.store(xrow, rrow, rw.single, rw.has_single, rstd);
}

// ---- elementwise operators over the output as one flat array -----------------------------------
// silu_and_mul and merge_attn_states have no reduction, so nothing ties a workgroup to a row: the
// output is a flat array of 16-byte pieces, piece p goes to one lane, and its row is p divided by
// the pieces of a row.  Bound by HBM; every wave reads and writes whole lines whatever the row
// length, no lane is idle for rows that a launch shape does not divide, and a small problem
// spreads over as many workgroups as it has pieces.  One piece per lane: two in flight per lane
// (half as many workgroups) lost 1-18 %; workgroups of 64 to 256 threads are the same.
// Default of the knob grid -> here, us per launch, on one set of buffers / three in rotation / from HBM:
//   silu_and_mul  4096 x 11008 bf16  43.4 / 56.3 / 56.8 -> 38.8 / 39.7 / 42.5 (6.8 TB/s on three sets: the
//                 memory-side cache serves part of it)    16000 x 11008  204 / 204 / 204 -> 158 on all
//                 (6.7 TB/s)    64 x 14336 fp16  4.3 / 4.3 / 7.4 -> 2.2 / 2.1 / 2.5
//                 2000 x 4099 bf16  12.0 / 12.0 / 16.7 -> 8.5 / 9.8 / 10.7
//   merge_attn_states  24576 x 256 bf16  6.4 / 7.5 / 10.0 -> 4.5 / 7.5 / 8.7    20480 x 128 fp16  3.6 / 4.5 /
//                 5.7 -> 2.9 / 3.8 / 4.5    38759 x 256 bf16  10.8 / 10.7 / 14.0 -> 9.1 / 11.4 / 12.2 (the one
//                 kind of buffers where the default is ahead; write_through_max in direct_route.cpp has why)

// n / d for n < 2^31 and d >= 2 as (n * mul) >> 32 >> shift, where shift = ceil(log2 d) - 1 and
// mul = ceil(2^(32 + shift) / d) < 2^32: the error of mul * d is below d <= 2^(shift + 1), so that of
// the quotient is below n / 2^31 of 1 / d.
struct FlatDiv { uint32_t mul, shift; };
__device__ __forceinline__ uint32_t flat_div(uint32_t n, FlatDiv f) { return __umulhi(n, f.mul) >> f.shift; }

// units: pieces of a row, or for ragged rows (RAG: d is no multiple of VEC) its elements; total:
// the same for the whole output.  A piece of a ragged output begins anywhere in a row: its inputs
// are read at element alignment, and the one piece in d / VEC that straddles two rows, or the end,
// element by element.
template <int DT, int POL, bool RAG>
__device__ __forceinline__ void silumul_flat_body(const char* __restrict__ x, char* __restrict__ out, uint32_t d,
                                                  uint32_t units, uint32_t total, FlatDiv fd)
{
    using T = dt_traits<DT>;
    constexpr int ES = T::XB, VEC = 16 / ES, AL = RAG ? ES : 16;
    constexpr bool BF = T::BF;
    const uint32_t p = blockIdx.x * kFlatThreads + threadIdx.x;
    const uint32_t at = RAG ? p * VEC : p;
    if (at >= total) return;
    // Outputs beyond the memory-side cache: 16000 x 11008 bf16 164.7 us -> 158.4 (6.7 TB/s), 6056 x 11008 62.4 -> 60.7, 20000 x 4096 75.8 ->
    // 74.5.  Not where the cache serves part of it (4096 x 11008 39.0 -> 40.4), for fp32 (3000 x 28672 156.9 -> 157.3), whose lanes have
    // half as many requests per byte, or where rows share lines (16000 x 8191 121.5 -> 124.2).
    if constexpr (POL == POL_NT && !RAG && ES == 2) wait_one_load(x);
    const uint32_t have = RAG && total - at < VEC ? total - at : VEC;      // elements of this piece that exist
    const uint32_t row = flat_div(at, fd), col = at - row * units;
    const char* g = x + (static_cast<uint64_t>(row) * 2u * d + (RAG ? col : col * VEC)) * ES;
    raw_t<16> gv, uv;
    if (!RAG || (col + VEC <= units && have == VEC)) {
        ld_stream<POL, 16, AL>(g, 0, gv);
        ld_stream<POL, 16, AL>(g, static_cast<uint64_t>(d) * ES, uv);
    } else {
#pragma unroll
        for (int k = 0; k < 4; ++k) gv.d[k] = uv.d[k] = 0u;
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const uint32_t i = at + e < total ? at + e : total - 1u;
            const uint32_t r = flat_div(i, fd);
            const char* q = x + (static_cast<uint64_t>(r) * 2u * d + (i - r * units)) * ES;
            raw_t<ES> ge, ue;
            ld_raw<ES>(q, ge);
            ld_raw<ES>(q + static_cast<uint64_t>(d) * ES, ue);
            const int sh = ES == 2 ? (e & 1) * 16 : 0;
            gv.d[e * ES / 4] |= ge.d[0] << sh;
            uv.d[e * ES / 4] |= ue.d[0] << sh;
        }
    }
    float y[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) y[e] = silu_times(get_elem<ES, BF>(gv, e), get_elem<ES, BF>(uv, e));
    raw_t<16> o;
    pack_vec<ES, BF, VEC>(y, o);
    if (!RAG || have == VEC) {
        st_stream<POL, 16>(out + static_cast<uint64_t>(blockIdx.x) * (kFlatThreads * 16), threadIdx.x * 16u, o);
    } else {
#pragma unroll
        for (int e = 0; e < VEC; ++e)
            if (static_cast<uint32_t>(e) < have) {
                raw_t<ES> one;
                one.d[0] = ES == 2 ? o.d[e >> 1] >> ((e & 1) * 16) : o.d[e * ES / 4];
                st_raw<ES>(out + static_cast<uint64_t>(at + e) * ES, one);
            }
    }
}

// Rows of whole pieces (d a multiple of 8, 16-byte aligned bases).  Every lane reads its row's two scores itself;
// the lane of a row's first piece writes the merged score.
template <int DT, int POL>
__device__ __forceinline__ void mergestates_flat_body(const char* __restrict__ va, const float* __restrict__ sa,
                                                      const char* __restrict__ vb, const float* __restrict__ sb,
                                                      char* __restrict__ vo, float* __restrict__ so, uint32_t units,
                                                      uint32_t total, FlatDiv fd)
{
    using T = dt_traits<DT>;
    constexpr int ES = T::XB, VEC = 16 / ES;
    constexpr bool BF = T::BF;
    constexpr float kLog2e = 1.44269504088896340736f, kLn2 = 0.69314718055994530942f;
    const uint64_t base = static_cast<uint64_t>(blockIdx.x) * (kFlatThreads * 16);
    const uint32_t off = threadIdx.x * 16u, p = blockIdx.x * kFlatThreads + threadIdx.x;
    if (p >= total) return;
    raw_t<16> av, bv;
    ld_stream<POL, 16, 16>(va + base, off, av);
    ld_stream<POL, 16, 16>(vb + base, off, bv);
    const uint32_t row = flat_div(p, fd);
    const float s_a = sa[row], s_b = sb[row];
    const float m = s_a > s_b ? s_a : s_b;
    const float ea = __builtin_amdgcn_exp2f((s_a - m) * kLog2e);
    const float eb = __builtin_amdgcn_exp2f((s_b - m) * kLog2e);
    const float denom = ea + eb;
    const float inv = __builtin_amdgcn_rcpf(denom);
    const float wa = ea * inv, wb = eb * inv;
    if (p == row * units) so[row] = m + __builtin_amdgcn_logf(denom) * kLn2;
    float y[VEC];
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        const float tb = wb * get_elem<ES, BF>(bv, e);
        y[e] = __builtin_fmaf(wa, get_elem<ES, BF>(av, e), tb);
    }
    raw_t<16> o;
    pack_vec<ES, BF, VEC>(y, o);
    st_stream<POL, 16>(vo + base, off, o);
}

}  // namespace addrms

// Kernels behind a call that names no configuration and has none in the specialised table.
// They are not points of the knob grid: their launch shape follows from the problem by the
// rules in addrms_direct.hip.
//
// Store policy.  A workgroup's ordinary stores leave dirty lines in its XCD's L2, which are
// written back when the kernel ends: a serial tail of up to 32 MB.  Non-temporal stores have
// no such tail, but nothing of them stays in the memory-side cache either, where the next
// kernel of the program looks for its input.  Write-through stores (sc1) go to the memory
// side as they are issued and stay there.  Which one a problem takes is decided by what it
// writes (write_through_max in addrms_direct.hip has both sides measured).
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
#include "silumul_kernel.h"

namespace addrms {

// POL_CACHED: ordinary loads and stores.  POL_NT: both non-temporal.  POL_WT: non-temporal loads, write-through stores.
enum : int { POL_CACHED = 0, POL_NT = 1, POL_WT = 2 };

template <typename T, int AL> struct at_align { typedef T type __attribute__((aligned(AL))); };

// Load of BYTES bytes at base + off, an address that is a multiple of AL, and aligned store; base
// is the same for the whole wave.  The write-through policy exists for buffer stores only (their
// cache-policy operand).
template <int POL, int BYTES, int AL>
__device__ __forceinline__ void ld_stream(const char* base, uint64_t off, raw_t<BYTES>& v)
{
    constexpr bool NT = POL != POL_CACHED;
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
    if constexpr (POL == POL_WT) {
        constexpr int kSc1 = 16;
        const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(base, 0, -1, 0x00027000);
        if constexpr (BYTES == 8) {
            __builtin_amdgcn_raw_buffer_store_b64(u32x2{v.d[0], v.d[1]}, rs, off, 0, kSc1);
        } else {
            static_assert(BYTES == 16, "one store");
            __builtin_amdgcn_raw_buffer_store_b128(u32x4{v.d[0], v.d[1], v.d[2], v.d[3]}, rs, off, 0, kSc1);
        }
    } else {
        st_raw<BYTES, POL == POL_NT>(base + off, v);
    }
}

// ---- add + RMSNorm ---------------------------------------------------------------------------
// A workgroup per row (several for rows shorter than a wave), a thread holds CPT chunks of VEC
// elements from the loads to the stores.  Same arithmetic as addrms_body, bit for bit.  HBM-bound:
// all loads of a thread are issued before the first value is used (in two batches beyond 32
// values), and a row is spread over as many threads as there are pieces, up to 1024, so that a
// thread has few and the row arrives early: of the 1 to 8 chunks per thread tried on 40 shapes
// the fewest were the fastest on all but four, by 2-8 % against twice as many.  DEFER (more than
// one chunk): both streams written after the row sum, 1-3 % there.
// Default of the knob grid -> here, us: 16 x 4096 bf16 3.1 -> 2.5, 256 x 5120 4.1 -> 3.5,
// 512 x 8192 8.3 -> 6.3, 4096 x 4096 21.5 -> 20.1, 20000 x 5120 152 -> 130 (6.3 TB/s),
// 32768 x 7168 340 -> 304, 2048 x 8192 fp32 56.4 -> 45.3, 900 x 28672 fp16 44.3 -> 39.8.
// Ragged: 2047 x 4095 fp16 18.6 -> 12.9 (buffers from HBM 27.4 -> 13.5), 9000 x 6150 bf16 95.5 ->
// 77, 300 x 10001 9.3 -> 7.5, 8192 x 1000 fp16+fp32 18.2 -> 17.4 (from HBM 23.5 -> 20.8); the single
// elements cost the first 0.7 us and weights at odd addresses 0.4 of what an aligned row would not.
template <int DT, int VEC, int CPT, int POL, bool RAG, bool DEFER>
__device__ __forceinline__ void addrms_direct_body(void* __restrict__ xp, void* __restrict__ rp,
                                                   const void* __restrict__ wp, float eps, double inv_n, int64_t M,
                                                   int32_t N)
{
    using T = dt_traits<DT>;
    constexpr int XB = T::XB, RB = T::RB;
    constexpr int UNR = VEC * CPT <= 32 ? CPT : (CPT + 1) / 2;
    constexpr bool BF = T::BF;
    extern __shared__ double lds[];

    const uint32_t tpr = blockDim.x, rpw = blockDim.y;
    const uint32_t lane = threadIdx.x, ry = threadIdx.y;
    const RowAddr ra = row_addr<XB, RB>(xp, rp, blockIdx.x, rpw, ry, M, N);
    const char* wbase = static_cast<const char*>(wp);
    // Ragged: `into` elements of the row's first cache line belong to the row before it; `head` elements precede the
    // row's first whole piece, which is a whole piece of both streams (the host checked that they have the same phase).
    constexpr int32_t LINE = 128 / XB;
    const int32_t into = RAG ? static_cast<int32_t>((static_cast<uint32_t>(reinterpret_cast<uintptr_t>(ra.xbase)) / XB + ra.rowoff) % LINE) : 0;
    const int32_t head = RAG ? (LINE - into) % VEC : 0;
    const int32_t nv = RAG ? head + (N - head) / VEC * VEC : N;
    const int32_t nlast = nv - VEC;
    const int32_t col0 = static_cast<int32_t>(lane) * VEC - into, stride = static_cast<int32_t>(tpr) * VEC;
    const uint32_t tcol = static_cast<int32_t>(lane) < head ? lane : static_cast<uint32_t>(nv - head) + lane;   // this lane's single element
    const bool tail = RAG && tcol < static_cast<uint32_t>(N);
    auto in_row = [=](int32_t col) { return RAG ? static_cast<uint32_t>(col) <= static_cast<uint32_t>(nlast) : col <= nlast; };
    auto clamped = [=](int32_t col) {            // idle lanes re-read valid data
        const int32_t c = RAG && col < head ? head : col;
        return static_cast<uint32_t>(c < nlast ? c : nlast);
    };

    float h[CPT][VEC], ht = 0.0f;
    raw_t<XB> xt{}, wt{};
    raw_t<RB> rt{};
    double acc = 0.0;
    if (tail) {
        ld_raw<XB, true>(ra.xbase + static_cast<uint64_t>((ra.rowoff + tcol) * XB), xt);
        ld_raw<RB, true>(ra.rbase + static_cast<uint64_t>((ra.rowoff + tcol) * RB), rt);
        ld_raw<XB, false>(wbase + static_cast<uint64_t>(tcol * XB), wt);
    }
#pragma unroll
    for (int g = 0; g < CPT; g += UNR) {
        raw_t<XB * VEC> xv[UNR];
        raw_t<RB * VEC> rv[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            if (g + u < CPT) {
                const uint32_t colc = clamped(col0 + (g + u) * stride);
                ld_stream<POL, XB * VEC, 16>(ra.xbase, (ra.rowoff + colc) * XB, xv[u]);
                ld_stream<POL, RB * VEC, 16>(ra.rbase, (ra.rowoff + colc) * RB, rv[u]);
            }
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            if (g + u < CPT) {
                const int c = g + u;
                const int32_t col = col0 + c * stride;
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    h[c][e] = get_elem<XB, BF>(xv[u], e) + get_elem<RB, BF && RB == 2>(rv[u], e);
                if (ra.row_ok && in_row(col)) {
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
    if (tail) {
        ht = get_elem<XB, BF>(xt, 0) + get_elem<RB, BF && RB == 2>(rt, 0);
        const double hd = static_cast<double>(ht);
        acc = __builtin_fma(hd, hd, acc);
    }
    raw_t<XB * VEC> wv[CPT];
#pragma unroll
    for (int c = 0; c < CPT; ++c) {
        const uint32_t colc = clamped(col0 + c * stride);
        ld_stream<POL_CACHED, XB * VEC, RAG ? XB : 16>(wbase, colc * XB, wv[c]);
    }

    const double ss = row_sum(acc, RED_WAVE, tpr, lane, ry, lds);
    const float rstd = rsqrt_to_f32(__builtin_fma(ss, inv_n, static_cast<double>(eps)));

    if constexpr (DEFER) {
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const int32_t col = col0 + c * stride;
            if (ra.row_ok && in_row(col)) {
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
        if (ra.row_ok && in_row(col)) {
            raw_t<XB * VEC> out;
            pack_vec<XB, BF, VEC>(y, out);
            st_stream<POL, XB * VEC>(ra.xbase, (ra.rowoff + col) * XB, out);
        }
    }
    if (tail && ra.row_ok) {
        float f[1] = {ht};
        raw_t<RB> rout;
        pack_vec<RB, BF, 1>(f, rout);
        st_raw<RB, true>(ra.rbase + static_cast<uint64_t>((ra.rowoff + tcol) * RB), rout);
        const float t = ht * rstd;
        f[0] = t * get_elem<XB, BF>(wt, 0);
        raw_t<XB> yout;
        pack_vec<XB, BF, 1>(f, yout);
        st_raw<XB, true>(ra.xbase + static_cast<uint64_t>((ra.rowoff + tcol) * XB), yout);
    }
}

// ---- elementwise operators over the output as one flat array -----------------------------------
// silu_and_mul and merge_attn_states have no reduction, so nothing ties a workgroup to a row: the
// output is a flat array of 16-byte pieces, piece p goes to one lane, and its row is p divided by
// the pieces of a row.  Bound by HBM; every wave reads and writes whole lines whatever the row
// length, no lane is idle for rows that a launch shape does not divide, and a small problem
// spreads over as many workgroups as it has pieces.  One piece per lane: two in flight per lane
// (half as many workgroups) lost 1-18 %; workgroups of 64 to 256 threads are the same.
// silu_and_mul, default of the knob grid -> here, buffers cycled by the program: 4096 x 11008
// bf16 57.2 -> 39.5 us (6.85 TB/s; the memory-side cache serves part of it), 16000 x 11008 208 ->
// 168 (6.3 TB/s), 64 x 14336 fp16 4.5 -> 2.3, 2000 x 4099 bf16 12.4 -> 10.3.
// merge_attn_states: 24576 x 256 bf16 7.7 -> 7.4, 20480 x 128 fp16 4.6 -> 3.9.

// n / d for n < 2^31 and d >= 2 as (n * mul) >> 32 >> shift, where shift = ceil(log2 d) - 1 and
// mul = ceil(2^(32 + shift) / d) < 2^32: the error of mul * d is below d <= 2^(shift + 1), so that of
// the quotient is below n / 2^31 of 1 / d.
struct FlatDiv { uint32_t mul, shift; };
__device__ __forceinline__ uint32_t flat_div(uint32_t n, FlatDiv f) { return __umulhi(n, f.mul) >> f.shift; }

constexpr int kFlatThreads = 256;

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

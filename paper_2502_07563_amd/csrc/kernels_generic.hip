// Plain fp32 kernels of liblasp2: the row-times-state product without a mask for the shapes that the
// matrix-core kernel does not take, and the small passes that are the same for every path: the prefix,
// suffix and total of the states, and the row sums of the softmax backward.  Fixed summation order
// (run-to-run bit-identical, no atomics).
#include "lasp2_common.h"

#include <hip/hip_bf16.h>

namespace lasp2 {
namespace {

constexpr int kThreads = 256;

__device__ __forceinline__ float ld(const float* p) { return *p; }
__device__ __forceinline__ float ld(const __hip_bfloat16* p) { return __bfloat162float(*p); }
__device__ __forceinline__ void st(float* p, float v) { *p = v; }
__device__ __forceinline__ void st(__hip_bfloat16* p, float v) { *p = __float2bfloat16(v); }

// Exclusive prefix (or suffix) over the slots of each group, restarted per document.
// One thread owns four adjacent state elements and walks the slots in order; loads are
// batched ahead of the stores so that in-place use (P == M) stays correct and the
// memory system sees several requests in flight.  The exclusive form does not touch the last slot's own state.
// user_slots: entry per slot of the caller's, walks of g.wslots of them (see launch_state_prefix): a walk's is its first, or
// reversed its last.
// PACKED, a kernel of its own: what the marks and divisions of packed batches take before the first load shows where
// a sequence has few slots (1 280 sequences of one slot: 25.1 us with them, 17.4 without).
constexpr int kScanBatch = 8;

template <bool PACKED>
__global__ __launch_bounds__(kThreads) void state_prefix_kernel(Geom g, const float* M, float* P,
                                                                int reverse, int inclusive, int user_slots,
                                                                unsigned* clear, unsigned nclear)
{
    if (clear) {
        const unsigned blk = (blockIdx.z * gridDim.y + blockIdx.y) * gridDim.x + blockIdx.x;
        for (unsigned i = blk * kThreads + threadIdx.x; i < nclear; i += gridDim.x * gridDim.y * gridDim.z * kThreads) clear[i] = 0u;
    }
    const int dd = g.d * g.d;
    const int e = (blockIdx.x * kThreads + threadIdx.x) * 4;
    if (e >= dd) return;
    const int stride = user_slots ? g.wslots : 1;   // array entries from one walk to the next inside a document
    const int entries = user_slots ? g.P_Ts : g.T_s;
    const size_t base = (size_t)blockIdx.y * (size_t)entries * dd + e;
    const float l2 = decay_log2(g, blockIdx.y);
    // a packed batch's documents of one mark, or all of them (documents are independent of each other)
    const uint32_t L = (uint32_t)min(g.L, (int64_t)INT32_MAX);
    const uint32_t Lp = PACKED && user_slots ? L / (uint32_t)g.wslots : L;   // tokens per walk, array entry
    const int k0 = PACKED ? (int)blockIdx.z * g.doc_stride : 0;
    const int k1 = !PACKED ? 1 : gridDim.z == 1 ? g.n_seqs : min(k0 + g.doc_stride, g.n_seqs);
    int first = !PACKED ? 0 : user_slots ? g.doc_pmark[blockIdx.z] : g.doc_mark[blockIdx.z];   // entries before the document
    for (int k = k0; k < k1; ++k) {
        const int dlen = PACKED ? (g.cu[k + 1] - g.cu[k]) : g.N;
        const int ns = PACKED ? (int)(((uint32_t)dlen + (L - 1u)) / L) : g.T_s;
        const int ne = PACKED ? (int)(((uint32_t)dlen + (Lp - 1u)) / Lp) : entries;
        const size_t doc = base + (size_t)first * dd;
        auto entry = [&](int r) { return (size_t)(reverse ? min((ns - r) * stride, ne) - 1 : r * stride) * dd; };
        first += ne;
        const int nm = inclusive ? ns : ns - 1;   // states that enter a result
        float4 run = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int r = 0; r < ns; r += kScanBatch) {
            float4 m[kScanBatch];
#pragma unroll
            for (int u = 0; u < kScanBatch; ++u)
                m[u] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int u = 0; u < kScanBatch; ++u)
                if (r + u < nm)
                    m[u] = *reinterpret_cast<const float4*>(M + doc + entry(r + u));
#pragma unroll
            for (int u = 0; u < kScanBatch; ++u)
                if (r + u < ns) {
                    float4* dst = reinterpret_cast<float4*>(P + doc + entry(r + u));
                    if (!inclusive) *dst = run;
                    // decay: the carried state ages by the length of the slot it crosses
                    // (slot index inside the document: r+u counted from the walk's start)
                    const int idx = reverse ? ns - 1 - (r + u) : r + u;
                    const int n = (int)min((int64_t)g.L, (int64_t)dlen - (int64_t)idx * g.L);
                    const float w = exp2f((float)n * l2);
                    run.x = fmaf(w, run.x, m[u].x); run.y = fmaf(w, run.y, m[u].y);
                    run.z = fmaf(w, run.z, m[u].z); run.w = fmaf(w, run.w, m[u].w);
                    if (inclusive) *dst = run;
                }
        }
    }
}

// S[s] = sum of M over all slots of the document that owns slot s (the state every rank holds
// after the gather and the sum when there is no mask); walks of several slots: over the entries of their first slots, which
// receive it.  Each thread owns four elements of the d x d state and sums a document's entries in ascending order
// before it writes any of them, so S may alias M.  The documents of a mark in turn, eight loads ahead (latency bounds it: 25
// entries of 16 heads one by one 19 us, 10 so).  PACKED: as above (1 280 sequences of one slot: 28.6 -> 25.0 us).
template <bool PACKED>
__global__ __launch_bounds__(kThreads) void state_total_kernel(Geom g, const float* M, float* S)
{
    const int dd = g.d * g.d;
    const int e = (blockIdx.x * kThreads + threadIdx.x) * 4;
    if (e >= dd) return;
    const size_t base = (size_t)blockIdx.y * (size_t)g.P_Ts * dd + e, step = (size_t)g.wslots * dd;
    const uint32_t L = (uint32_t)min(g.L, (int64_t)INT32_MAX), Lp = PACKED ? L / (uint32_t)g.wslots : L;
    const int k0 = PACKED ? (int)blockIdx.z * g.doc_stride : 0;
    const int k1 = !PACKED ? 1 : gridDim.z == 1 ? g.n_seqs : min(k0 + g.doc_stride, g.n_seqs);
    int first = PACKED ? g.doc_pmark[blockIdx.z] : 0;
    for (int k = k0; k < k1; ++k) {
        const uint32_t dlen = PACKED ? (uint32_t)(g.cu[k + 1] - g.cu[k]) : (uint32_t)g.N;
        const int ns = PACKED ? (int)((dlen + (L - 1u)) / L) : g.T_s;
        const float* m = M + base + (size_t)first * dd;
        float* out = S + base + (size_t)first * dd;
        float4 run = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int r = 0; r < ns; r += kScanBatch) {
            float4 x[kScanBatch];
#pragma unroll
            for (int u = 0; u < kScanBatch; ++u) x[u] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
            for (int u = 0; u < kScanBatch; ++u)
                if (r + u < ns) x[u] = *reinterpret_cast<const float4*>(m + (size_t)(r + u) * step);
#pragma unroll
            for (int u = 0; u < kScanBatch; ++u)
                if (r + u < ns) { run.x += x[u].x; run.y += x[u].y; run.z += x[u].z; run.w += x[u].w; }
        }
        for (int r = 0; r < ns; ++r) *reinterpret_cast<float4*>(out + (size_t)r * step) = run;
        if (PACKED) first += (int)((dlen + (Lp - 1u)) / Lp);
    }
}

// out = A * state (or A * state^T) for the rows of one slot.  The state sits in LDS as
// sS[r][c] = the factor of A[.,r] in out[.,c]; thread (rg, c) produces column c of the rows
// rg, rg + NRG, ... of each tile of kProjRows * NRG rows.
constexpr int kProjRows = 8;

template <typename T, int D>
__global__ __launch_bounds__(kThreads) void rows_state_generic_kernel(Geom g, const T* __restrict__ A,
                                                                      const float* __restrict__ state,
                                                                      T* __restrict__ out, int transpose)
{
    constexpr int NRG = kThreads / D, RT = kProjRows * NRG;
    extern __shared__ float smem_f[];
    float* sS = smem_f;            // [D][D]
    float* sA = smem_f + D * D;    // [RT][D]
    const int s = blockIdx.x, grp = blockIdx.y;
    int tok0, len;
    slot_range(g, s, tok0, len);
    if (len <= 0) return;
    const float* st_ = state + ((size_t)grp * g.T_s + s) * (size_t)(D * D);
    for (int i = threadIdx.x; i < D * D; i += kThreads) {
        const int r = i / D, c = i % D;
        sS[i] = transpose ? st_[c * D + r] : st_[i];
    }
    const int c = threadIdx.x % D, rg = threadIdx.x / D;
    const size_t gbase = ((size_t)grp * (size_t)g.N + tok0) * D;
    for (int r0 = 0; r0 < len; r0 += RT) {
        __syncthreads();   // state staged / previous tile consumed
        for (int i = threadIdx.x; i < RT * D; i += kThreads) {
            const int row = r0 + i / D;
            sA[i] = row < len ? ld(A + gbase + (size_t)row * D + i % D) : 0.f;
        }
        __syncthreads();
        float acc[kProjRows];
#pragma unroll
        for (int j = 0; j < kProjRows; ++j) acc[j] = 0.f;
        for (int r = 0; r < D; ++r) {
            const float w = sS[r * D + c];
#pragma unroll
            for (int j = 0; j < kProjRows; ++j) acc[j] = fmaf(sA[(rg + j * NRG) * D + r], w, acc[j]);
        }
#pragma unroll
        for (int j = 0; j < kProjRows; ++j) {
            const int row = r0 + rg + j * NRG;
            if (row < len) st(out + gbase + (size_t)row * D + c, acc[j]);
        }
    }
}

template <typename T, int D>
hipError_t rows_state_generic_TD(const Geom& g, const T* A, const float* state, T* out, int tr,
                                 hipStream_t st)
{
    constexpr size_t smem = sizeof(float) * ((size_t)D * D + (size_t)kProjRows * (kThreads / D) * D);
    auto kern = rows_state_generic_kernel<T, D>;
    if (smem > 48 * 1024) {
        hipError_t e = allow_dynamic_lds<rows_state_generic_kernel<T, D>>((int)smem);
        if (e != hipSuccess) return e;
    }
    dim3 grid(g.T_s, g.G), block(kThreads);
    hipLaunchKernelGGL(kern, grid, block, smem, st, g, A, state, out, tr);
    return hipGetLastError();
}

template <typename T>
hipError_t rows_state_generic_T(const Geom& g, const T* A, const float* state, T* out, int tr,
                                hipStream_t st)
{
    switch (g.d) {
        case 16: return rows_state_generic_TD<T, 16>(g, A, state, out, tr, st);
        case 32: return rows_state_generic_TD<T, 32>(g, A, state, out, tr, st);
        case 64: return rows_state_generic_TD<T, 64>(g, A, state, out, tr, st);
        default: return rows_state_generic_TD<T, 128>(g, A, state, out, tr, st);
    }
}

// delta_i = dO_i . O_i for every row (the row sums the softmax backward needs).  lse2, when given,
// receives the row's log-sum-exp times log2(e), the form in which the matrix-core dK/dV kernel subtracts
// it from base-2 scores.  Bound by memory: a lane takes 16 bytes of a row (both tensors are 16-byte
// aligned and a row is a multiple of that), D * sizeof(T) / 16 lanes a row, and four rows are under way
// per lane.  (One wave per row and 2-byte loads left most of a wave's work to addresses and shuffles.)
// This kernel, 16 heads, inputs out of cache, us, before -> now: bf16, d = 128, 1000 rows 7.0 -> 6.1, 8192 rows 44.6 -> 25.7, 32768
// rows 177 -> 97; bf16, d = 64, 8192 rows 27.6 -> 14.0; fp32, d = 64, 2003 rows 8.9 -> 7.8; fp32, d = 128, 8192 rows
// 48.4 -> 47.9.  A layer's 1 % at most, less than the runs of a long softmax layer differ.
constexpr int kDeltaRows = 4;   // rows per lane

template <typename T, int D>
__global__ __launch_bounds__(kThreads) void softmax_delta_kernel(Geom g, const T* __restrict__ O,
                                                                 const T* __restrict__ dO,
                                                                 const float* __restrict__ LSE,
                                                                 float* __restrict__ delta,
                                                                 float* __restrict__ lse2)
{
    constexpr int VE = 16 / (int)sizeof(T), LP = D / VE, RB = kThreads / LP;   // elements and lanes; rows at a time
    struct alignas(16) Vec { T x[VE]; };
    const size_t rows = (size_t)g.G * (size_t)g.qn;
    const size_t row0 = (size_t)blockIdx.x * (RB * kDeltaRows) + threadIdx.x / LP;
    const int part = threadIdx.x % LP;
    Vec o[kDeltaRows], w[kDeltaRows];
#pragma unroll
    for (int u = 0; u < kDeltaRows; ++u) {
        const size_t row = min(row0 + (size_t)(u * RB), rows - 1);   // (past the end: the last row again)
        o[u] = *reinterpret_cast<const Vec*>(O + row * D + part * VE);
        w[u] = *reinterpret_cast<const Vec*>(dO + row * D + part * VE);
    }
#pragma unroll
    for (int u = 0; u < kDeltaRows; ++u) {
        float acc = 0.f;
#pragma unroll
        for (int v = 0; v < VE; ++v) acc = fmaf(ld(&o[u].x[v]), ld(&w[u].x[v]), acc);
#pragma unroll
        for (int m = LP / 2; m > 0; m >>= 1) acc += __shfl_xor(acc, m, 64);
        const size_t row = row0 + (size_t)(u * RB);
        if (part == 0 && row < rows) {
            delta[row] = acc;
            if (lse2) lse2[row] = LSE[row] * 1.4426950408889634f;
        }
    }
}

template <typename T, int D>
void softmax_delta_TD(const Geom& g, size_t rows, const T* O, const T* dO, const float* LSE, float* delta, float* lse2,
                      hipStream_t st)
{
    constexpr size_t per = (size_t)(kThreads * 16 / (D * (int)sizeof(T))) * kDeltaRows;
    hipLaunchKernelGGL((softmax_delta_kernel<T, D>), dim3((unsigned)((rows + per - 1) / per)), dim3(kThreads), 0, st, g,
                       O, dO, LSE, delta, lse2);
}

template <typename T>
hipError_t softmax_delta_T(const Geom& g, size_t rows, const void* O, const void* dO, const float* LSE, float* delta,
                           float* lse2, hipStream_t st)
{
    const T *o = static_cast<const T*>(O), *w = static_cast<const T*>(dO);
    switch (g.d) {
        case 16: softmax_delta_TD<T, 16>(g, rows, o, w, LSE, delta, lse2, st); break;
        case 32: softmax_delta_TD<T, 32>(g, rows, o, w, LSE, delta, lse2, st); break;
        case 64: softmax_delta_TD<T, 64>(g, rows, o, w, LSE, delta, lse2, st); break;
        default: softmax_delta_TD<T, 128>(g, rows, o, w, LSE, delta, lse2, st); break;
    }
    return hipGetLastError();
}

}  // namespace

hipError_t launch_softmax_delta(const Geom& g, int dtype, const void* O, const void* dO, const float* LSE,
                                float* delta, float* lse2, hipStream_t st)
{
    const size_t rows = (size_t)g.G * (size_t)g.qn;
    if (rows == 0) return hipSuccess;
    if (dtype == LASP2_F32) return softmax_delta_T<float>(g, rows, O, dO, LSE, delta, lse2, st);
    return softmax_delta_T<__hip_bfloat16>(g, rows, O, dO, LSE, delta, lse2, st);
}

// The grid's third axis: a packed batch's documents are dealt out by marks, where one thread that takes them in turn would wait
// for each (documents in turn | by marks, us: 16 x 65 536 in 1 000 990 | 231; 8 x 131 072 in 40 158 | 113), or go in turn, where they have
// many slots and the groups alone give every CU a workgroup (states of 12 documents apart from each other at a time, 32 x 131 072 in slots of
// 64: suffix 1 602 | 1 770; 16 x 131 072 in 40 203 | 214, in slots of 256).
static int scan_marks(const Geom& g)
{
    if (!g.n_seqs || (g.G >= 16 && g.T_s >= 8LL * g.n_seqs)) return 1;
    return (g.n_seqs + g.doc_stride - 1) / g.doc_stride;
}

hipError_t launch_state_total(const Geom& g, const float* M, float* S, hipStream_t st)
{
    const int dd = g.d * g.d;
    const int marks = scan_marks(g);
    dim3 grid((dd / 4 + kThreads - 1) / kThreads, g.G, marks), block(kThreads);
    hipLaunchKernelGGL((g.n_seqs ? state_total_kernel<true> : state_total_kernel<false>), grid, block, 0, st, g, M, S);
    return hipGetLastError();
}

hipError_t launch_rows_state_generic(const Geom& g, int dtype, const void* A, const float* state,
                                     void* out, int transpose_state, hipStream_t st)
{
    if (dtype == LASP2_F32)
        return rows_state_generic_T(g, static_cast<const float*>(A), state, static_cast<float*>(out),
                                    transpose_state, st);
    return rows_state_generic_T(g, static_cast<const __hip_bfloat16*>(A), state,
                                static_cast<__hip_bfloat16*>(out), transpose_state, st);
}

hipError_t launch_state_prefix(const Geom& g, const float* M, float* P, int reverse, int inclusive,
                               int user_slots, unsigned* clear, unsigned nclear, hipStream_t st)
{
    const int dd = g.d * g.d;
    const int marks = scan_marks(g);
    dim3 grid((dd / 4 + kThreads - 1) / kThreads, g.G, marks), block(kThreads);
    hipLaunchKernelGGL((g.n_seqs ? state_prefix_kernel<true> : state_prefix_kernel<false>), grid, block, 0, st, g, M, P, reverse, inclusive,
                       user_slots, clear, nclear);
    return hipGetLastError();
}

}  // namespace lasp2

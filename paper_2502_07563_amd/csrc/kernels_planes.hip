// Linear attention on the matrix cores for every shape that kernels_mfma.hip does not take: fp32 of
// any head size, bf16 with d < 128, and bf16 d = 128 with decay factors too small for its kernels.
// All products go through split planes (planes.h), so scores, states and sums have fp32 accuracy
// whatever the input type.
#include "planes.h"

#include <algorithm>

namespace lasp2 {
namespace {

constexpr int kThr = 256;    // four waves
constexpr int kChunk = 128;  // rows of out per workgroup and chunk: 32 per wave

// Which 32 x 32 tiles of a D x D state wave w owns: NT = 4: row w; NT = 2: one tile; NT = 1: the
// one tile belongs to wave `solo`.
template <int NT>
struct Tiles {
    static constexpr int n = NT == 4 ? 4 : 1;
    __device__ static __forceinline__ bool mine(int w, int solo) { return NT > 1 || w == solo; }
    __device__ static __forceinline__ int row(int w) { return NT == 4 ? w : NT == 2 ? w >> 1 : 0; }
    __device__ static __forceinline__ int col(int w, int t) { return NT == 4 ? t : NT == 2 ? w & 1 : 0; }
};

// lam^e, l2 = log2 lam (the hardware exponential: 1 ulp; results below 2^-126 are zero)
__device__ __forceinline__ float decay_pow(float e, float l2) { return __builtin_amdgcn_exp2f(e * l2); }

// Rescales the elements of a transposed fetch (tokens r0 + 4h + .., planes.h) by lam^(e0 + de * token):
// the planes add up to the exact value, the product is an fp32 one and is split again.
template <int NP>
__device__ __forceinline__ void weight_frag(const bf16x8 (&f)[NP], int r0, int lane, int e0, int de, float l2, bf16x8 (&out)[3])
{
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int t = r0 + 4 * (lane >> 5) + (e < 4 ? e : e + 4);
        x[e] = frag_value(f, e) * decay_pow((float)max(e0 + de * t, 0), l2);   // (below 0: rows past the end, all zero)
    }
    split8(x, out);
}

// S[t] += X^T Y over the tokens of NKS k-steps (16 rows each, from row r0) of one stage
template <typename T, int D, int DP, int PLANE, bool DECAY, int NKS>
__device__ __forceinline__ void state_step(f32x16 (&S)[Tiles<DP / 32>::n], const char* buf, int tensor_bytes, int r0,
                                           int w, int lane, int e0, int de, float l2)
{
    constexpr int NP = planes_of<T>::n, NT = DP / 32, NA = DECAY ? 3 : NP;
    bf16x8 a[NKS][NA];
#pragma unroll
    for (int ks = 0; ks < NKS; ++ks) {
        if constexpr (DECAY) {
            bf16x8 x[NP];
            col_frag<DP>(buf, PLANE, r0 + 16 * ks, 32 * Tiles<NT>::row(w), lane, x);
            weight_frag(x, r0 + 16 * ks, lane, e0, de, l2, a[ks]);
        } else {
            col_frag<DP>(buf, PLANE, r0 + 16 * ks, 32 * Tiles<NT>::row(w), lane, a[ks]);
        }
    }
#pragma unroll
    for (int t = 0; t < Tiles<NT>::n; ++t) {
        bf16x8 b[NKS][NP];
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) col_frag<DP>(buf + tensor_bytes, PLANE, r0 + 16 * ks, 32 * Tiles<NT>::col(w, t), lane, b[ks]);
        if constexpr (NA * NP > 1) {
            f32x16 low = zero16();
#pragma unroll
            for (int ks = 0; ks < NKS; ++ks) low = mm<1, 2>(a[ks], b[ks], low);
            S[t] += low;
        }
#pragma unroll
        for (int ks = 0; ks < NKS; ++ks) S[t] = mm<0, 0>(a[ks], b[ks], S[t]);
    }
}

// sum over t < n of lam^(e0 + de t) x[t] y[t] in fp32 (columns of row-major arrays with rows of D elements)
template <typename T>
__device__ __forceinline__ float state_element(const T* x, const T* y, int D, int n, float l2, int e0, int de)
{
    float acc = 0.f;
#pragma unroll 1
    for (int t = 0; t < n; ++t)
        acc = fmaf(exp2f((float)(e0 + de * t) * l2) * load1(x + (size_t)t * D), load1(y + (size_t)t * D), acc);
    return acc;
}

// M[slot] = sum over the slot's tokens of (weighted) k^T v; one workgroup per slot.
template <typename T, int D, bool DECAY>
__global__ __launch_bounds__(kThr) void states_planes_kernel(Geom g, const T* __restrict__ K, const T* __restrict__ V,
                                                             float* __restrict__ M, int anchor_start)
{
    constexpr int DP = D < 32 ? 32 : D, NT = DP / 32;
    constexpr int ROWS = (planes_of<T>::n == 3 && D == 128) ? 32 : 64;   // two stages fit the LDS
    typedef PairStage<T, D, DP, ROWS, kThr> Stage;
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int s = blockIdx.x, grp = blockIdx.y;
    int tok0, len;
    slot_range(g, s, tok0, len);
    const size_t base = ((size_t)grp * (size_t)g.N + tok0) * D;
    const float l2 = decay_log2(g, grp);
    const int e0 = anchor_start ? 0 : len - 1, de = anchor_start ? 1 : -1;

    f32x16 S[Tiles<NT>::n];
#pragma unroll
    for (int t = 0; t < Tiles<NT>::n; ++t) S[t] = zero16();
    Stage st;
    const int nst = (len + ROWS - 1) / ROWS;
    st.fetch(K + base, V + base, 0, len, tid);
    for (int i = 0; i < nst; ++i) {
        char* buf = smem + (i & 1) * Stage::BYTES;
        st.put(buf, tid);
        if (i + 1 < nst) st.fetch(K + base, V + base, (i + 1) * ROWS, len, tid);
        __syncthreads();   // (two buffers: the one written next was last read before this barrier)
        if (NT > 1) {
#pragma unroll
            for (int r0 = 0; r0 < ROWS; r0 += 32)
                state_step<T, D, DP, Stage::PLANE, DECAY, 2>(S, buf, Stage::TENSOR, r0, w, lane, e0 + de * i * ROWS, de, l2);
        } else {           // one tile: the waves share the tokens
            state_step<T, D, DP, Stage::PLANE, DECAY, 1>(S, buf, Stage::TENSOR, 16 * w, w, lane, e0 + de * i * ROWS, de, l2);
        }
    }
    float* m = M + ((size_t)grp * g.T_s + s) * (size_t)(D * D);
    // Planes make NaN of an infinity and of what rounds to one (planes.h): such a slot is summed again in fp32.
    float odd = 0.f;
#pragma unroll
    for (int t = 0; t < Tiles<NT>::n; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            odd = fmaf(D >= 32 || (acc_row(v) + 4 * (lane >> 5) < D && (lane & 31) < D) ? S[t][v] : 0.f, 0.f, odd);
    if (__syncthreads_or(odd != 0.f)) {
        for (int e = tid; e < D * D; e += kThr)
            m[e] = state_element(K + base + e / D, V + base + e % D, D, len, l2, e0, de);
        return;
    }
    if (NT == 1) {
        float* part = reinterpret_cast<float*>(smem);
#pragma unroll
        for (int v = 0; v < 16; ++v) part[(w * 16 + v) * 64 + lane] = S[0][v];
        __syncthreads();
        for (int e = tid; e < 16 * 64; e += kThr) {
            const int v = e / 64, l = e % 64, row = acc_row(v) + 4 * (l >> 5), col = l & 31;
            const float x = (part[e] + part[1024 + e]) + (part[2048 + e] + part[3072 + e]);
            if (row < D && col < D) m[row * D + col] = x;
        }
        return;
    }
#pragma unroll
    for (int t = 0; t < Tiles<NT>::n; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            m[(32 * Tiles<NT>::row(w) + acc_row(v) + 4 * (lane >> 5)) * D + 32 * Tiles<NT>::col(w, t) + (lane & 31)] = S[t][v];
}

struct PlanesProblem {
    const void *A, *Bk, *Cv;
    const float* state;
    void* out;
    int transpose, reverse;
};
struct PlanesProblems { PlanesProblem p[3]; };

// Problem, segment x (= slot * nseg + segment) and group of a workgroup.  flat: a one-dimensional grid in which the nprob
// problems of a segment are dealt to the same XCD, one after another, and find each other's rows in its L2 (backward launch, fp32,
// 16 x 4000 x 64 64 -> 60 us; bf16, 16 x 1800 x 64 23.6 -> 21.9); otherwise (one problem, or grids past 2^32 threads) groups are
// the second axis.
__device__ __forceinline__ bool which_segment(const Geom& g, int nprob, int nseg, int flat, int& prob, int& x, int& grp)
{
    if (nprob == 1) {   // (the forward: without the divisions 64 x 4001 x 64 in bf16 takes 46.6 us instead of 47.9)
        prob = 0;
        x = blockIdx.x;
        grp = blockIdx.y;
        return true;
    }
    if (!flat) {
        prob = blockIdx.x % nprob;
        x = blockIdx.x / nprob;
        grp = blockIdx.y;
        return true;
    }
    const unsigned per = (unsigned)g.T_s * (unsigned)nseg, u = (blockIdx.x / (8u * nprob)) * 8u + (blockIdx.x & 7u);
    prob = (int)((blockIdx.x >> 3) % (unsigned)nprob);
    grp = (int)(u / per);
    x = (int)(u % per);
    return u < per * (unsigned)g.G;
}

// Tokens per LDS stage: as many of the chunk's 128 as leave room for a second workgroup on the CU
// (one workgroup with d = 128), with at most 32 registers per thread for the next stage's loads; fp32 with
// decay and d = 64 has no registers for more than 32, and spills 9 even so.  With d = 128 the operands' planes, the
// state's and the result's accumulators exceed the 512 registers of a thread at one wave per SIMD: 88 spilled
// in fp32, 140 with decay, 76 in bf16 with decay.  Layer, 2 x 16 x 4096 x 128, against one scalar product per element, us:
// fp32 forward 3470 -> 356, backward 10120 -> 908; bf16 with strong decay 2850 -> 241, 8240 -> 576.
template <typename T, int D, bool DECAY>
struct AttnLds {
    static constexpr int DP = D < 32 ? 32 : D, NP = planes_of<T>::n;
    static constexpr int ROWS = D == 128 ? (NP == 3 ? 32 : 64) : (NP == 3 && D == 64) ? (DECAY ? 32 : 64) : 128;
    typedef PairStage<T, D, DP, ROWS, kThr> Stage;
    static constexpr int SPLANE = DP * DP * 2;
    static constexpr int BYTES = Stage::BYTES + 3 * SPLANE;
};

// What attn_planes_kernel computes, in fp32 from the elements as they are, for a workgroup's chunks from `first`
// on: a row of out per wave, the running state M [D][D] in LDS.  For inputs whose planes are not finite: slow, as scalar
// products are (fp32, 8 x 2003 x 64 with a NaN in every head's V, forward + backward: 1760 us).
template <typename T, int D>
__device__ __forceinline__ void attn_scalar(const Geom& g, const PlanesProblems& probs, int nprob, int nseg, int cps, int flat,
                                            int first, float* M)
{
    asm volatile("" : "+s"(nseg));   // (all of this worked out anew, so that none of it stays in registers through the walk)
    int x, prob, grp;
    which_segment(g, nprob, nseg, flat, prob, x, grp);
    const PlanesProblem pb = probs.p[prob];
    const int tid = threadIdx.x;
    int tok0, len, ps;
    slot_range(g, x / nseg, tok0, len, ps);
    const bool rev = pb.reverse != 0;
    if (rev && g.wslots > 1) ps += (len - 1) / ((int)g.L / g.wslots);
    const size_t base = ((size_t)grp * (size_t)g.N + tok0) * D;
    const T* A = static_cast<const T*>(pb.A) + base;
    const T* Bk = static_cast<const T*>(pb.Bk) + base;
    const T* Cv = static_cast<const T*>(pb.Cv) + base;
    T* out = static_cast<T*>(pb.out) + base;
    const float* state = pb.state ? pb.state + ((size_t)grp * g.P_Ts + ps) * (size_t)(D * D) : nullptr;
    const float l2 = decay_log2(g, grp);
    const int transpose = pb.transpose, last = min((len + kChunk - 1) / kChunk, (x % nseg + 1) * cps);
    constexpr int NB = D > 64 ? 2 : 1;
    const int lane = tid & 63, nch = (len + kChunk - 1) / kChunk;
#pragma unroll 1
    for (int e = tid; e < D * D; e += kThr) M[e] = state ? state[transpose ? (e % D) * D + e / D : e] : 0.f;
#pragma unroll 1
    for (int ci = 0; ci < last; ++ci) {
        const int c0 = (rev ? nch - 1 - ci : ci) * kChunk, clen = min(kChunk, len - c0);
        __syncthreads();   // M is written
#pragma unroll 1
        for (int i = ci < first ? clen : tid >> 6; i < clen; i += kThr / 64) {
            float o[NB], t[NB];
            const T* ar = A + (size_t)(c0 + i) * D;
#pragma unroll
            for (int u = 0; u < NB; ++u) { o[u] = 0.f; t[u] = 0.f; }
#pragma unroll 1
            for (int a = 0; a < D; ++a)
#pragma unroll
                for (int u = 0; u < NB; ++u) t[u] = fmaf(load1(ar + a), M[a * D + min(lane + 64 * u, D - 1)], t[u]);
#pragma unroll 1
            for (int j = rev ? i : 0; j <= (rev ? clen - 1 : i); ++j) {
                float p = 0.f;
#pragma unroll
                for (int u = 0; u < NB; ++u)
                    if (lane + 64 * u < D)
                        p = fmaf(load1(ar + lane + 64 * u), load1(Bk + (size_t)(c0 + j) * D + lane + 64 * u), p);
#pragma unroll
                for (int k = 32; k > 0; k >>= 1) p += __shfl_xor(p, k, 64);
                p *= exp2f((float)(rev ? j - i : i - j) * l2);
#pragma unroll
                for (int u = 0; u < NB; ++u) o[u] = fmaf(p, load1(Cv + (size_t)(c0 + j) * D + min(lane + 64 * u, D - 1)), o[u]);
            }
            const float wi = exp2f((float)(rev ? clen - i : i + 1) * l2);
#pragma unroll
            for (int u = 0; u < NB; ++u)
                if (lane + 64 * u < D) store1(out + (size_t)(c0 + i) * D + lane + 64 * u, fmaf(wi, t[u], o[u]));
        }
        __syncthreads();   // M has been read
        if (ci + 1 < last) {
            const float wc = exp2f((float)clen * l2);
#pragma unroll 1
            for (int e = tid; e < D * D; e += kThr)
                M[e] = fmaf(wc, M[e], state_element(Bk + (size_t)c0 * D + e / D, Cv + (size_t)c0 * D + e % D, D, clen, l2,
                                                    rev ? 0 : clen - 1, rev ? 1 : -1));
        }
    }
}

// c += x y with the rows of the result those of x, or (TR) those of y: transposed
template <bool TR, int LO, int HI, int NX, int NY>
__device__ __forceinline__ f32x16 mm_either(const bf16x8 (&x)[NX], const bf16x8 (&y)[NY], f32x16 c)
{
    if constexpr (TR) return mm<LO, HI>(y, x, c);
    else return mm<LO, HI>(x, y, c);
}

// four columns of a row
__device__ __forceinline__ void store4(float* p, float a, float b, float c, float d)
{
    const f32x4 v = {a, b, c, d};
    *reinterpret_cast<f32x4*>(p) = v;
}
__device__ __forceinline__ void store4(__hip_bfloat16* p, float a, float b, float c, float d)
{
    const u32x2 v = {pack2(a, b), pack2(c, d)};
    *reinterpret_cast<u32x2*>(p) = v;
}

// out = [(A Bk^T) (.) mask] Cv + A * state for the rows of one segment of one slot, state += Bk^T Cv from
// chunk to chunk of 128 rows (causal: first to last; reverse: mask j >= i, last to first).
//
// A wave owns 32 rows of out: its rows of A are operands in registers, Bk and Cv pass through LDS
// in stages for all four (the next stage's loads in flight in registers), scores are formed transposed (a query per lane) and are the
// next product's operand as they stand.  The running state stays in accumulators, its planes
// are written to LDS once per chunk, as rows of the state's second index.
// With d = 128 the result is formed transposed too: a lane stores four columns of its row at a time, and the 64 addresses and
// bounds of single elements no longer compete for the registers (forward | backward launch, 16 x 1800 x 128 in fp32, us: 73 -> 63 |
// 207 -> 179; scratch 416 -> 352 bytes).  Smaller heads lose by it (bf16, 64 x 4001 x 64: 50 -> 53 | 124 -> 128): their
// stores, rows of 32 to 256 bytes, are better made by column.
// A slot may be cut into `nseg` segments of `cps` chunks, a workgroup each: a workgroup first adds up
// the states of the chunks before its own (a fifth of a chunk's work), which is worth it while the
// launch leaves CUs idle.
// Bounds: the split's vector instructions next to the matrix products in fp32, latency and HBM in bf16.
// Against one scalar fp32 product per element (and a load for each), layer forward + backward: bf16,
// 64 groups x 4001 x 64: 4200 -> 230 us (the forward launch 50 us, 3.2 TB/s); fp32, 2 x 1024 x 64: 1190 -> 58 us.
template <typename T, int D, bool DECAY>
__global__ __launch_bounds__(kThr, D == 128 ? 1 : 2) void attn_planes_kernel(Geom g, PlanesProblems probs, int nprob, int nseg,
                                                                             int cps, int flat)
{
    typedef AttnLds<T, D, DECAY> LD;
    typedef typename LD::Stage Stage;
    constexpr int DP = LD::DP, NP = planes_of<T>::n, NT = DP / 32, KS = D / 16, NTL = Tiles<NT>::n;
    constexpr int ROWS = LD::ROWS, SUB = 32 * DP * 2;   // bytes of 32 rows of a plane
    constexpr bool TR = D == 128;
    extern __shared__ __align__(16) char smem[];
    char* snap = smem + Stage::BYTES;

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, l32 = lane & 31;
    int prob, x, grp;
    if (!which_segment(g, nprob, nseg, flat, prob, x, grp)) return;
    const PlanesProblem pb = probs.p[prob];
    const int s = x / nseg, seg = x % nseg;
    int tok0, len, ps;
    slot_range(g, s, tok0, len, ps);
    const int nch = (len + kChunk - 1) / kChunk;
    const int ci0 = seg * cps, ci1 = min(nch, ci0 + cps);
    if (ci0 >= nch) return;
    const bool rev = pb.reverse != 0;
    const size_t base = ((size_t)grp * (size_t)g.N + tok0) * D;
    const T* A = static_cast<const T*>(pb.A) + base;
    const T* Bk = static_cast<const T*>(pb.Bk) + base;
    const T* Cv = static_cast<const T*>(pb.Cv) + base;
    T* out = static_cast<T*>(pb.out) + base;
    const float l2 = DECAY ? decay_log2(g, grp) : 0.f;
    const int solo = rev ? 3 : 0;   // (the wave with the fewest score tiles)
    const bool owner = Tiles<NT>::mine(w, solo);

    Stage st;
    st.fetch(Bk, Cv, (rev ? nch - 1 : 0) * kChunk, len, tid);
    f32x16 S[NTL];
    bool have_state = pb.state != nullptr;
#pragma unroll
    for (int t = 0; t < NTL; ++t) S[t] = zero16();
    if (have_state && owner) {
        // (several slots in one walk: the prefix of its first, the suffix of its last)
        if (rev && g.wslots > 1) ps += (len - 1) / ((int)g.L / g.wslots);
        const float* st0 = pb.state + ((size_t)grp * g.P_Ts + ps) * (size_t)(D * D);
#pragma unroll
        for (int t = 0; t < NTL; ++t)
#pragma unroll
            for (int v = 0; v < 16; v += 4) {
                const int a = 32 * Tiles<NT>::row(w) + acc_row(v) + 4 * h, b = 32 * Tiles<NT>::col(w, t) + l32;
                if (a >= D || b >= D) continue;
                if (pb.transpose) {
                    const f32x4 q4 = *reinterpret_cast<const f32x4*>(st0 + b * D + a);
#pragma unroll
                    for (int e = 0; e < 4; ++e) S[t][v + e] = q4[e];
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) S[t][v + e] = st0[(a + e) * D + b];
                }
            }
    }

    int redo = ci1;
    for (int ci = 0; ci < ci1; ++ci) {
        const int c0 = (rev ? nch - 1 - ci : ci) * kChunk, clen = min(kChunk, len - c0);
        const int nsub = (clen + 31) / 32;
        const bool emit = ci >= ci0, update = ci + 1 < ci1;
        f32x16 acc[NT];
        bf16x8 q[KS][NP];
        if (emit) {
            const int r = c0 + 32 * w + l32;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) to_planes(load8(A + (size_t)r * D + 16 * ks + 8 * h, r < len), q[ks]);
            // snapshot of the running state, rows = its second index
            if (have_state && owner) {
#pragma unroll
                for (int t = 0; t < NTL; ++t)
#pragma unroll
                    for (int v = 0; v < 16; v += 8) {
                        bf16x8 p[3];
                        acc_frag(S[t], v, p);
                        const int b = 32 * Tiles<NT>::col(w, t) + l32, a = 32 * Tiles<NT>::row(w) + acc_row(v) + 4 * h;
#pragma unroll
                        for (int i = 0; i < 3; ++i) {
                            const bf16x4 lo = {p[i][0], p[i][1], p[i][2], p[i][3]}, hi = {p[i][4], p[i][5], p[i][6], p[i][7]};
                            *reinterpret_cast<bf16x4*>(snap + i * LD::SPLANE + plane_off<DP>(b, a >> 3) + (a & 7) * 2) = lo;
                            *reinterpret_cast<bf16x4*>(snap + i * LD::SPLANE + plane_off<DP>(b, (a >> 3) + 1) + (a & 7) * 2) = hi;
                        }
                    }
            }
        }
        if (DECAY && update) {
            const float wc = decay_pow((float)clen, l2);
#pragma unroll
            for (int t = 0; t < NTL; ++t)
#pragma unroll
                for (int v = 0; v < 16; ++v) S[t][v] *= wc;
        }
        for (int s0 = 0; s0 < clen; s0 += ROWS) {
            // the previous stage has been read (an emitted chunk ends with a barrier)
            if (s0 > 0 || (ci > 0 && ci <= ci0)) __syncthreads();
            st.put(smem, tid);
            if (s0 + ROWS < clen) st.fetch(Bk, Cv, c0 + s0 + ROWS, len, tid);
            else if (ci + 1 < ci1) st.fetch(Bk, Cv, rev ? c0 - kChunk : c0 + kChunk, len, tid);
            __syncthreads();
            if (emit && s0 == 0) {
#pragma unroll
                for (int nt = 0; nt < NT; ++nt) {
                    acc[nt] = zero16();
                    if (have_state) {
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) {
                            bf16x8 b[3];
                            row_frag<DP>(snap, LD::SPLANE, 32 * nt + l32, 2 * ks + h, b);
                            acc[nt] = mm_either<TR, 1, 2>(q[ks], b, acc[nt]);
                        }
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) {
                            bf16x8 b[1];
                            row_frag<DP>(snap, LD::SPLANE, 32 * nt + l32, 2 * ks + h, b);
                            acc[nt] = mm_either<TR, 0, 0>(q[ks], b, acc[nt]);
                        }
                        if (DECAY) {
                            // the state sits one token before the chunk (causal) or one after it
#pragma unroll
                            for (int v = 0; v < 16; ++v) {
                                const int i = 32 * w + (TR ? l32 : acc_row(v) + 4 * h);
                                acc[nt][v] *= decay_pow((float)(rev ? max(clen - i, 0) : i + 1), l2);
                            }
                        }
                    }
                }
            }
#pragma unroll 1
            for (int u = 0; u < ROWS / 32; ++u) {
                const int sb = s0 / 32 + u;
                const char* buf = smem + u * SUB;
                if (sb >= nsub) break;
                if (emit && (rev ? sb >= w : sb <= w)) {
                    f32x16 sc = zero16();
                    if constexpr (NP > 1) {
#pragma unroll
                        for (int ks = 0; ks < KS; ++ks) {
                            bf16x8 k[NP];
                            row_frag<DP>(buf, Stage::PLANE, l32, 2 * ks + h, k);
                            sc = mm<1, 2>(k, q[ks], sc);
                        }
                    }
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        bf16x8 k[1];
                        row_frag<DP>(buf, Stage::PLANE, l32, 2 * ks + h, k);
                        sc = mm<0, 0>(k, q[ks], sc);
                    }
                    if (DECAY || sb == w) {
                        const int dist = 32 * (w - sb) + l32 - 4 * h;   // query minus key, for the first row
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const int d = dist - acc_row(v);
                            if (DECAY) sc[v] *= decay_pow((float)d, rev ? -l2 : l2);
                            if (sb == w && (rev ? d > 0 : d < 0)) sc[v] = 0.f;
                        }
                    }
                    bf16x8 p[2][3];
                    acc_frag(sc, 0, p[0]);
                    acc_frag(sc, 8, p[1]);
#pragma unroll
                    for (int nt = 0; nt < NT; ++nt) {
                        bf16x8 v[2][NP];
                        col_frag<DP>(buf + Stage::TENSOR, Stage::PLANE, 0, 32 * nt, lane, v[0]);
                        col_frag<DP>(buf + Stage::TENSOR, Stage::PLANE, 16, 32 * nt, lane, v[1]);
                        const f32x16 low = mm_either<TR, 1, 2>(p[1], v[1], mm_either<TR, 1, 2>(p[0], v[0], zero16()));
                        acc[nt] = mm_either<TR, 0, 0>(p[1], v[1], mm_either<TR, 0, 0>(p[0], v[0], acc[nt] + low));
                    }
                }
                if (update && owner)
                    state_step<T, D, DP, Stage::PLANE, DECAY, 2>(S, buf, Stage::TENSOR, 0, w, lane,
                                                                 rev ? sb * 32 : clen - 1 - sb * 32, rev ? 1 : -1, l2);
            }
        }
        if (!emit) { have_state = true; continue; }

        // A non-finite row of Cv would reach, as 0 * inf, the rows of its 32-token tile that the mask
        // keeps from it, and planes make NaN of an infinity and of what rounds to one.  Either shows as a
        // non-finite result (a state that has one makes its whole column so): from that chunk on the
        // segment is done again in fp32.
        float odd = 0.f;
#pragma unroll
        for (int nt = 0; nt < NT; ++nt)
#pragma unroll
            for (int v = 0; v < 16; ++v) odd = fmaf(TR || 32 * nt + l32 < D ? acc[nt][v] : 0.f, 0.f, odd);
        if (__syncthreads_or(odd != 0.f)) {
            redo = ci;
            break;
        }
        if constexpr (TR) {
            if (32 * w + l32 < clen) {
                T* o = out + (size_t)(c0 + 32 * w + l32) * D + 4 * h;
#pragma unroll
                for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                    for (int v = 0; v < 16; v += 4)
                        store4(o + 32 * nt + acc_row(v), acc[nt][v], acc[nt][v + 1], acc[nt][v + 2], acc[nt][v + 3]);
            }
        } else {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int i = 32 * w + acc_row(v) + 4 * h, b = 32 * nt + l32;
                    if (i < clen && b < D) store1(out + (size_t)(c0 + i) * D + b, acc[nt][v]);
                }
        }
        have_state = true;
    }
    if (redo < ci1) attn_scalar<T, D>(g, probs, nprob, nseg, cps, flat, redo, reinterpret_cast<float*>(snap));
}

template <typename T, int D, bool DECAY>
hipError_t states_TD(const Geom& g, const T* K, const T* V, float* M, int anchor, hipStream_t st)
{
    constexpr int DP = D < 32 ? 32 : D, ROWS = (planes_of<T>::n == 3 && D == 128) ? 32 : 64;
    constexpr int stages = 2 * PairStage<T, D, DP, ROWS, kThr>::BYTES, lds = stages < 16384 ? 16384 : stages;
    hipError_t e = allow_dynamic_lds<states_planes_kernel<T, D, DECAY>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((states_planes_kernel<T, D, DECAY>), dim3(g.T_s, g.G), dim3(kThr), lds, st, g, K, V, M, anchor);
    return hipGetLastError();
}

template <typename T, int D, bool DECAY>
hipError_t attn_TD(const Geom& g, const PlanesProblems& p, int n, hipStream_t st)
{
    constexpr int lds = AttnLds<T, D, DECAY>::BYTES;
    hipError_t e = allow_dynamic_lds<attn_planes_kernel<T, D, DECAY>>(lds);
    if (e != hipSuccess) return e;
    // Segments: as many as bring the launch to two workgroups per CU, at most eight per slot (the last
    // one then re-adds seven eighths of the slot's states).
    const int64_t chunks = std::min<int64_t>((std::min<int64_t>(g.L, g.N) + kChunk - 1) / kChunk, INT32_MAX / 2);
    const int64_t wgs = (int64_t)g.G * g.T_s * n;
    int64_t nseg = std::max<int64_t>(1, std::min<int64_t>({2 * (int64_t)cu_count() / wgs, chunks, 8}));
    const int64_t cps = (chunks + nseg - 1) / nseg;
    nseg = (chunks + cps - 1) / cps;
    const int64_t units = ((int64_t)g.G * g.T_s * nseg + 7) / 8 * 8;
    if (n > 1 && units * n < ((int64_t)1 << 32) / kThr) {
        hipLaunchKernelGGL((attn_planes_kernel<T, D, DECAY>), dim3((unsigned)(units * n)), dim3(kThr), lds, st, g, p, n, (int)nseg,
                           (int)cps, 1);
        return hipGetLastError();
    }
    // (a grid holds fewer than 2^32 threads per axis: past that groups are the other axis, and the problems may go one by one)
    const int per = (int64_t)g.T_s * nseg * n < ((int64_t)1 << 32) / kThr ? n : 1;
    for (int i = 0; i < n; i += per) {
        PlanesProblems sub = p;
        if (per == 1) sub.p[0] = p.p[i];
        hipLaunchKernelGGL((attn_planes_kernel<T, D, DECAY>), dim3((unsigned)(g.T_s * nseg * per), g.G), dim3(kThr), lds, st, g, sub,
                           per, (int)nseg, (int)cps, 0);
        e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename T, int D>
hipError_t states_T(const Geom& g, const void* K, const void* V, float* M, int anchor, hipStream_t st)
{
    const T *k = static_cast<const T*>(K), *v = static_cast<const T*>(V);
    return g.decay ? states_TD<T, D, true>(g, k, v, M, anchor, st) : states_TD<T, D, false>(g, k, v, M, anchor, st);
}

template <typename T, int D>
hipError_t attn_T(const Geom& g, const PlanesProblems& p, int n, hipStream_t st)
{
    return g.decay ? attn_TD<T, D, true>(g, p, n, st) : attn_TD<T, D, false>(g, p, n, st);
}

// one instance per (type, head size)
#define LASP2_FOR_TYPE_AND_SIZE(CALL, ...)                                         \
    if (dtype == LASP2_F32) switch (g.d) {                                         \
        case 16: return CALL<float, 16>(__VA_ARGS__);                              \
        case 32: return CALL<float, 32>(__VA_ARGS__);                              \
        case 64: return CALL<float, 64>(__VA_ARGS__);                              \
        default: return CALL<float, 128>(__VA_ARGS__);                             \
    }                                                                              \
    switch (g.d) {                                                                 \
        case 16: return CALL<__hip_bfloat16, 16>(__VA_ARGS__);                     \
        case 32: return CALL<__hip_bfloat16, 32>(__VA_ARGS__);                     \
        case 64: return CALL<__hip_bfloat16, 64>(__VA_ARGS__);                     \
        default: return CALL<__hip_bfloat16, 128>(__VA_ARGS__);                    \
    }

hipError_t attn_any(const Geom& g, int dtype, const PlanesProblems& p, int n, hipStream_t st)
{
    LASP2_FOR_TYPE_AND_SIZE(attn_T, g, p, n, st)
}

}  // namespace

hipError_t launch_states_planes(const Geom& g, int dtype, const void* K, const void* V, float* M, int anchor_start,
                                hipStream_t st)
{
    LASP2_FOR_TYPE_AND_SIZE(states_T, g, K, V, M, anchor_start, st)
}

hipError_t launch_attn_fwd_planes(const Geom& g, int dtype, const void* Q, const void* K, const void* V, const float* P,
                                  void* O, hipStream_t st)
{
    PlanesProblems p = {};
    p.p[0] = {Q, K, V, P, O, 0, 0};
    return attn_any(g, dtype, p, 1, st);
}

hipError_t launch_attn_bwd_planes(const Geom& g, int dtype, const void* Q, const void* K, const void* V, const void* dO,
                                  const float* P, const float* dR, void* dQ, void* dK, void* dV, hipStream_t st)
{
    PlanesProblems p = {};
    // dQ: the forward problem with (dO, V, K) in the roles of (Q, K, V); its state is
    // V^T K = (K^T V)^T, i.e. the cached prefix read transposed.
    p.p[0] = {dO, V, K, P, dQ, 1, 0};
    // dV: anti-causal problem with (K, Q, dO); state dM_{t+1:T} = sum Q^T dO.
    p.p[1] = {K, Q, dO, dR, dV, 0, 1};
    // dK: anti-causal problem with (V, dO, Q); state dO^T Q = dM^T.
    p.p[2] = {V, dO, Q, dR, dK, 1, 1};
    return attn_any(g, dtype, p, 3, st);
}

}  // namespace lasp2

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
// the planes add up to the exact value, which is multiplied and split again.
template <int NP>
__device__ __forceinline__ void weight_frag(const bf16x8 (&f)[NP], int r0, int lane, int e0, int de, float l2, bf16x8 (&out)[3])
{
    float x[8], y[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        const int t = r0 + 4 * (lane >> 5) + (e < 4 ? e : e + 4);
        x[e] = frag_value(f, e);
        y[e] = decay_pow((float)max(e0 + de * t, 0), l2);   // (below 0: rows past the end, all zero)
    }
    split8_products(x, y, out);
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

// Tokens of the caller's slots
__device__ __forceinline__ int slot_tokens(const Geom& g)
{
    return g.wslots > 1 ? (int)((uint32_t)g.L / (uint32_t)g.wslots) : (int)min(g.L, (int64_t)INT32_MAX);
}

// M[slot] = sum over the slot's tokens of (weighted) k^T v; one workgroup per slot.
template <typename T, int D, bool DECAY>
__global__ __launch_bounds__(kThr) void states_planes_kernel(Geom g, const T* __restrict__ K, const T* __restrict__ V,
                                                             float* __restrict__ M, int anchor_start, int of_slots)
{
    constexpr int DP = D < 32 ? 32 : D, NT = DP / 32;
    constexpr int ROWS = (planes_of<T>::n == 3 && D == 128) ? 32 : 64;   // two stages fit the LDS
    typedef PairStage<T, D, DP, ROWS, kThr> Stage;
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
    const int s = blockIdx.x, grp = blockIdx.y;
    int tok0, len, ps, doc0, doc1, slot0, slot1;
    slot_range<false>(g, s, tok0, len, ps, doc0, doc1, slot0, slot1);
    if (of_slots && (anchor_start ? tok0 == doc0 : tok0 + len == doc1)) return;   // (in no exclusive sum)
    const size_t base = ((size_t)grp * (size_t)g.N + tok0) * D;
    const float l2 = decay_log2(g, grp);
    const int de = anchor_start ? 1 : -1;

    f32x16 S[Tiles<NT>::n];
#pragma unroll
    for (int t = 0; t < Tiles<NT>::n; ++t) S[t] = zero16();
    // Walks of several slots (of_slots: heads of 64, slots of whole stages): a slot's rows are weighted and summed among themselves, then
    // the sum before (anchor_start: behind) them is aged and added, as it is where each slot has a state.
    constexpr bool SPLIT = D == 64;
    const bool back = SPLIT && of_slots && anchor_start;
    const int slot = SPLIT && of_slots ? slot_tokens(g) : len;
    int slot_at = back ? (len - 1) / slot * slot : 0;
    f32x16 sum = zero16();
    Stage st;
    const int nst = (len + ROWS - 1) / ROWS;
    auto row_of = [&](int i) { return (back ? nst - 1 - i : i) * ROWS; };
    st.fetch(K + base, V + base, row_of(0), len, tid);
    for (int i = 0; i < nst; ++i) {
        char* buf = smem + (i & 1) * Stage::BYTES;
        st.put(buf, tid);
        if (i + 1 < nst) st.fetch(K + base, V + base, row_of(i + 1), len, tid);
        __syncthreads();   // (two buffers: the one written next was last read before this barrier)
        const int row = row_of(i), end = min(slot_at + slot, len), e = anchor_start ? row - slot_at : end - 1 - row;
        if (NT > 1) {
#pragma unroll
            for (int r0 = 0; r0 < ROWS; r0 += 32)
                state_step<T, D, DP, Stage::PLANE, DECAY, 2>(S, buf, Stage::TENSOR, r0, w, lane, e, de, l2);
        } else {           // one tile: the waves share the tokens
            state_step<T, D, DP, Stage::PLANE, DECAY, 1>(S, buf, Stage::TENSOR, 16 * w, w, lane, e, de, l2);
        }
        if (SPLIT && (back ? row == slot_at : row + ROWS >= end)) {
            const float age = DECAY ? decay_pow((float)(end - slot_at), l2) : 1.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) sum[v] = DECAY ? fmaf(age, sum[v], S[0][v]) : sum[v] + S[0][v];
            S[0] = zero16();
            slot_at += back ? -slot : slot;
        }
    }
    if (SPLIT) S[0] = sum;
    if (of_slots && anchor_start) ps += (len - 1) / slot_tokens(g);
    float* m = M + (of_slots ? (size_t)grp * g.P_Ts + ps : (size_t)grp * g.T_s + s) * (size_t)(D * D);
    // Planes make NaN of an infinity and of what rounds to one (planes.h): such a slot is summed again in fp32.
    float odd = 0.f;
#pragma unroll
    for (int t = 0; t < Tiles<NT>::n; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v)
            odd = fmaf(D >= 32 || (acc_row(v) + 4 * (lane >> 5) < D && (lane & 31) < D) ? S[t][v] : 0.f, 0.f, odd);
    if (__syncthreads_or(odd != 0.f)) {
        for (int e = tid; e < D * D; e += kThr)
            m[e] = state_element(K + base + e / D, V + base + e % D, D, len, l2, anchor_start ? 0 : len - 1, de);
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
    float* emit;   // NULL, or the array of such states whose entries of the other slots the walks write (heads of 64)
};
struct PlanesProblems { PlanesProblem p[3]; };

// How a launch is cut: `nseg` segments of `cps` chunks per walk and `nprob` problems (1 or 3).  flat: a one-dimensional grid in which
// the problems of a segment are dealt to the same XCD, one after another, and find each other's rows in its L2 (backward launch,
// fp32, 16 x 4000 x 64 64 -> 60 us; bf16, 16 x 1800 x 64 23.6 -> 21.9); otherwise (one problem, or grids past 2^32 threads)
// groups are the second axis.
struct PlanesGrid {
    int nprob, nseg, cps, flat;
    uint32_t per, per_inv, nseg_inv;   // segments of a group; 2^32 / per and 2^32 / nseg, rounded down
};

// u / d, inv = 2^32 / d rounded down (d > 1): the product is the quotient or one less.  (A division is forty instructions, and a
// workgroup of one chunk starts with five of them: 1900 clocks of its 20000.)
__device__ __forceinline__ uint32_t div_by(uint32_t u, uint32_t d, uint32_t inv)
{
    const uint32_t q = __umulhi(u, inv);
    return q + (u - q * d >= d);
}

// Problem, walk, segment and group of a workgroup
__device__ __forceinline__ bool which_segment(const Geom& g, const PlanesGrid& pg, int& prob, int& s, int& seg, int& grp)
{
    uint32_t x = blockIdx.x;
    bool there = true;
    prob = 0;
    grp = blockIdx.y;
    if (pg.flat) {
        const uint32_t i = x >> 3, t = i / 3u, u = t * 8u + (x & 7u);
        prob = (int)(i - 3u * t);
        const uint32_t q = pg.per > 1 ? div_by(u, pg.per, pg.per_inv) : u;
        grp = (int)q;
        x = u - q * pg.per;
        there = q < (uint32_t)g.G;
    } else if (pg.nprob > 1) {
        prob = (int)(x % 3u);
        x /= 3u;
    }
    const uint32_t walk = pg.nseg > 1 ? div_by(x, (uint32_t)pg.nseg, pg.nseg_inv) : x;
    s = (int)walk;
    seg = (int)(x - walk * (uint32_t)pg.nseg);
    return there;
}

// Tokens per LDS stage: as many of the chunk's 128 as leave room for a second workgroup on the CU
// (one workgroup with d = 128), with at most 32 registers per thread for the next stage's loads.  With d = 128 the operands' planes, the
// state's and the result's accumulators exceed the 512 registers of a thread at one wave per SIMD: 88 spilled
// in fp32, 140 with decay, 76 in bf16 with decay.  Layer, 2 x 16 x 4096 x 128, against one scalar product per element, us:
// fp32 forward 3470 -> 356, backward 10120 -> 908; bf16 with strong decay 2850 -> 241, 8240 -> 576.
template <typename T, int D, bool DECAY>
struct AttnLds {
    static constexpr int DP = D < 32 ? 32 : D, NP = planes_of<T>::n;
    static constexpr int ROWS = D == 128 ? (NP == 3 ? 32 : 64) : 128;
    typedef PairStage<T, D, DP, ROWS, kThr> Stage;
    static constexpr int SPLANE = DP * DP * 2;
    static constexpr int FLAG = Stage::BYTES + 3 * SPLANE, BYTES = FLAG + 16;
};

// Where the state that a walk starts from lies, in states: the entry of its first slot (ps), reversed of its last.
__device__ __forceinline__ size_t state_index(const Geom& g, const PlanesProblem& pb, int grp, int ps, int len)
{
    return (size_t)grp * g.P_Ts + ps + (pb.reverse && g.wslots > 1 ? (len - 1) / slot_tokens(g) : 0);
}

// What attn_planes_kernel computes, in fp32 from the elements as they are, for a workgroup's chunks from `first`
// on: a row of out per wave, the running state M [D][D] in LDS.  For inputs whose planes are not finite: slow, as scalar
// products are (fp32, 8 x 2003 x 64 with a NaN in every head's V, forward + backward: 1760 us).
template <typename T, int D, int CHUNK>
__device__ __forceinline__ void attn_scalar(const Geom& g, const PlanesProblems& probs, PlanesGrid pg, int first, float* M)
{
    asm volatile("" : "+s"(pg.nseg));   // (all of this worked out anew, so that none of it stays in registers through the walk)
    int s, seg, prob, grp;
    which_segment(g, pg, prob, s, seg, grp);
    const PlanesProblem pb = probs.p[prob];
    const int tid = threadIdx.x;
    int tok0, len, ps;
    slot_range(g, s, tok0, len, ps);
    const bool rev = pb.reverse != 0;
    const size_t base = ((size_t)grp * (size_t)g.N + tok0) * D;
    const T* A = static_cast<const T*>(pb.A) + base;
    const T* Bk = static_cast<const T*>(pb.Bk) + base;
    const T* Cv = static_cast<const T*>(pb.Cv) + base;
    T* out = static_cast<T*>(pb.out) + base;
    const float* state = pb.state ? pb.state + state_index(g, pb, grp, ps, len) * (size_t)(D * D) : nullptr;
    const float l2 = decay_log2(g, grp);
    const int transpose = pb.transpose, last = min((len + CHUNK - 1) / CHUNK, (seg + 1) * pg.cps);
    constexpr int NB = D > 64 ? 2 : 1;
    const int lane = tid & 63, nch = (len + CHUNK - 1) / CHUNK;
#pragma unroll 1
    for (int e = tid; e < D * D; e += kThr) M[e] = state ? state[transpose ? (e % D) * D + e / D : e] : 0.f;
#pragma unroll 1
    for (int ci = 0; ci < last; ++ci) {
        const int c0 = (rev ? nch - 1 - ci : ci) * CHUNK, clen = min(CHUNK, len - c0);
        __syncthreads();   // M is written
        const int edge = rev ? c0 + clen : c0, slot = slot_tokens(g);
        if (pb.emit && ci >= first && (ci > 0 || !pb.state) && (edge % slot == 0 || (rev && ci == 0))) {
            float* at = pb.emit + ((size_t)grp * g.P_Ts + ps + (rev ? (edge - 1) / slot : edge / slot)) * (size_t)(D * D);
#pragma unroll 1
            for (int e = tid; e < D * D; e += kThr) at[e] = M[e];
        }
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

// Scores of a tile: times lam^(distance), zero outside the mask where the tile lies on the diagonal.  dist: query minus key, for
// the accumulator's first row.  (Bounds that hold for either direction, and one compare each: a choice of the
// direction per element had become a branch each, 1800 clocks a tile.)
template <bool DECAY>
__device__ __forceinline__ void mask_tile(f32x16& sc, int dist, bool diagonal, bool rev, float l2)
{
    const int lo = diagonal && rev ? dist : -64;                            // accumulator rows lo .. lo + span are kept
    const uint32_t span = (uint32_t)((diagonal && !rev ? dist : 64) - lo);
    const float e2 = rev ? -l2 : l2;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        if (DECAY) sc[v] *= decay_pow((float)(dist - acc_row(v)), e2);
        sc[v] = (uint32_t)(acc_row(v) - lo) <= span ? sc[v] : 0.f;
    }
}

// Whether any thread of the workgroup says `odd`, by a flag in LDS that starts at zero (and is asked no more once it is set); a
// barrier.  The wave's answer is a compare: the reduction inside __syncthreads_or takes 1000 clocks, a tenth of a chunk.
__device__ __forceinline__ bool any_odd(bool odd, int* flag)
{
    if (__any(odd)) *flag = 1;
    __syncthreads();
    return __builtin_amdgcn_readfirstlane(*static_cast<volatile int*>(flag)) != 0;
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
// 207 -> 179; scratch 416 -> 352 bytes).  Heads of 16 and 32 store by column (64 x 4001 x 32 by row, forward | backward, us: fp32 68 -> 68 |
// 119 -> 114, bf16 43 -> 43 | 65 -> 64).
// A slot may be cut into `nseg` segments of `cps` chunks, a workgroup each: a workgroup first adds up
// the states of the chunks before its own (a fifth of a chunk's work), which is worth it while the
// launch leaves CUs idle.
// Bounds: the split's vector instructions next to the matrix products in fp32, latency and HBM in bf16.
// Against one scalar fp32 product per element (and a load for each), layer forward + backward, when it took heads of 64 too: bf16,
// 64 groups x 4001 x 64: 4200 -> 230 us; fp32, 2 x 1024 x 64: 1190 -> 58 us.  Now 64 x 4001 x 32: bf16 108 us, fp32 187.
template <typename T, int D, bool DECAY>
__global__ __launch_bounds__(kThr, D == 128 ? 1 : 2) void attn_planes_kernel(Geom g, PlanesProblems probs, PlanesGrid pg)
{
    static_assert(D != 64, "heads of 64: attn64_planes_kernel");
    typedef AttnLds<T, D, DECAY> LD;
    typedef typename LD::Stage Stage;
    constexpr int DP = LD::DP, NP = planes_of<T>::n, NT = DP / 32, KS = D / 16, NTL = Tiles<NT>::n;
    constexpr int ROWS = LD::ROWS, SUB = 32 * DP * 2;   // bytes of 32 rows of a plane
    constexpr bool TR = D == 128;
    extern __shared__ __align__(16) char smem[];
    char* snap = smem + Stage::BYTES;
    int* flag = reinterpret_cast<int*>(smem + LD::FLAG);

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, l32 = lane & 31;
    if (tid == 0) *flag = 0;
    int prob, s, seg, grp;
    if (!which_segment(g, pg, prob, s, seg, grp)) return;
    const PlanesProblem pb = probs.p[prob];
    int tok0, len, ps;
    slot_range(g, s, tok0, len, ps);
    const int nch = (len + kChunk - 1) / kChunk;
    const int ci0 = seg * pg.cps, ci1 = min(nch, ci0 + pg.cps);
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
        const float* st0 = pb.state + state_index(g, pb, grp, ps, len) * (size_t)(D * D);
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
                        mask_tile<DECAY>(sc, 32 * (w - sb) + l32 - 4 * h, sb == w, rev, l2);
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
        if (any_odd(odd != 0.f, flag)) {
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
    if (redo < ci1) attn_scalar<T, D, kChunk>(g, probs, pg, redo, reinterpret_cast<float*>(snap));
}

// 8 consecutive elements of a row in all its planes
template <int NP>
__device__ __forceinline__ void frag_at(const char* tile, int plane_bytes, uint32_t off, bf16x8 (&f)[NP])
{
#pragma unroll
    for (int p = 0; p < NP; ++p) f[p] = *reinterpret_cast<const bf16x8*>(tile + p * plane_bytes + off);
}

// ---- The same for heads of 64 ----
// Chunks of 64 rows; a wave has 32 of them and 32 of the 64 columns: the scores of its rows are formed by two waves, but a
// chunk is three score tiles instead of ten per 128 rows, the longest of a wave two instead of four, and accumulators and
// state take less than half of the registers: three workgroups per CU in bf16 (48 KB of LDS and 168 registers each) where there were
// two; fp32 and decay have two.  Walks of several slots write the states of the slots inside them (emit: prefixes in the forward,
// suffixes by the backward's dV).  bf16 rows go out through
// LDS, 128 bytes at a time.  Bounds: the chain of a chunk (snapshot, stage, barrier, state product, two tiles, barrier: about
// 8000 clocks, 3000 of them the tiles), of which a CU runs two or three side by side.  With walks as pick_planes64_slots has
// them and slots of 128, us, against 128-row chunks in four waves of 32 rows and all columns: bf16, 64 x 4001, layer forward 77 -> 51, backward
// 147 -> 96 (the launches 47 -> 38 and 119 -> 87, 4.3 and 3.0 TB/s); 16 x 4000 28 -> 25, 46 -> 35; fp32, 64 x 4001 137 -> 113, 260
// -> 241; 2 x 1024 25 -> 20, 25 -> 20.
template <typename T>
struct Attn64Lds {
    typedef PairStage<T, 64, 64, 64, kThr> Stage;
    static constexpr int SPLANE = 64 * 64 * 2, PATCH = planes_of<T>::n == 1 ? 64 * 128 : 0;   // (rows of out in bf16 on their way to whole lines)
    static constexpr int FLAG = Stage::BYTES + 3 * SPLANE + PATCH, BYTES = FLAG + 16;
};
constexpr int kRows64 = 64;

template <typename T, bool DECAY>
__global__ __launch_bounds__(kThr, planes_of<T>::n == 1 && !DECAY ? 3 : 2) void attn64_planes_kernel(Geom g, PlanesProblems probs, PlanesGrid pg)
{
    typedef Attn64Lds<T> LD;
    typedef typename LD::Stage Stage;
    constexpr int D = 64, NP = planes_of<T>::n, KS = D / 16, SUB = 32 * D * 2;
    constexpr bool TR = NP == 1, LOW = NP > 1;
    extern __shared__ __align__(16) char smem[];
    char* snap = smem + Stage::BYTES;
    char* patch = snap + 3 * LD::SPLANE;
    int* flag = reinterpret_cast<int*>(smem + LD::FLAG);

    const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6, h = lane >> 5, l32 = lane & 31;
    if (tid == 0) *flag = 0;
    int prob, s, seg, grp;
    if (!which_segment(g, pg, prob, s, seg, grp)) return;
    const PlanesProblem pb = probs.p[prob];
    int tok0, len, ps;
    slot_range(g, s, tok0, len, ps);
    const int nch = (len + kRows64 - 1) / kRows64;
    const int ci0 = seg * pg.cps, ci1 = min(nch, ci0 + pg.cps);
    if (ci0 >= nch) return;
    const bool rev = pb.reverse != 0;
    const size_t base = ((size_t)grp * (size_t)g.N + tok0) * D;
    const T* A = static_cast<const T*>(pb.A) + base;
    const T* Bk = static_cast<const T*>(pb.Bk) + base;
    const T* Cv = static_cast<const T*>(pb.Cv) + base;
    T* out = static_cast<T*>(pb.out) + base;
    const float l2 = DECAY ? decay_log2(g, grp) : 0.f;
    const int rt = w >> 1, ct = w & 1;   // row and column tile; the state's tile has the same numbers

    Stage st;
    st.fetch(Bk, Cv, (rev ? nch - 1 : 0) * kRows64, len, tid);
    // The running state is the sum since the last edge of a slot, S, on top of that there, base, so that states are sums of slots' sums,
    // as accurate as those of the states and prefix kernels: one running sum rounds all of it with every 16 rows (P of 130 x 1000
    // in slots of 64, error 1.5e-7 instead of 7.6e-8).
    f32x16 S[1] = {zero16()}, base_sum = zero16();
    bool have_state = pb.state != nullptr;
    if (have_state) {
        const float* st0 = pb.state + state_index(g, pb, grp, ps, len) * (size_t)(D * D);
#pragma unroll
        for (int v = 0; v < 16; v += 4) {
            const int a = 32 * rt + acc_row(v) + 4 * h, b = 32 * ct + l32;
            if (pb.transpose) {
                const f32x4 q4 = *reinterpret_cast<const f32x4*>(st0 + b * D + a);
#pragma unroll
                for (int e = 0; e < 4; ++e) base_sum[v + e] = q4[e];
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) base_sum[v + e] = st0[(a + e) * D + b];
            }
        }
    }

    // the next edge of a slot of the caller's (where edges lie inside chunks: every 128 rows), its number in the walk, and its row
    const int tokens = slot_tokens(g), slot = tokens % kRows64 ? 2 * kRows64 : tokens;
    int at_slot = rev ? (len - 1) / slot : 0, edge = rev ? len : 0, since = 0;   // since: rows in S
    // offset of a lane's first piece of its row in a tile; the next ones differ in bits 5 and 6 alone
    uint32_t row_at = (uint32_t)plane_off<D>(l32, h);
    // ... and of its first piece of the state's snapshot, row 32 ct + l32, columns 32 rt + 4 h ..; the next ones are 8, 16 and 24 columns on
    uint32_t snap_at = (uint32_t)plane_off<D>(32 * ct + l32, 4 * rt) + 8u * h;
    auto running = [&](int v, float age) __attribute__((always_inline)) { return DECAY ? fmaf(age, base_sum[v], S[0][v]) : base_sum[v] + S[0][v]; };
    int redo = ci1;
    for (int ci = 0; ci < ci1; ++ci) {
        const int c0 = (rev ? nch - 1 - ci : ci) * kRows64, clen = min(kRows64, len - c0);
        const bool rows = ci >= ci0, update = ci + 1 < ci1;
        float age = DECAY ? decay_pow((float)since, l2) : 1.f;
        if ((rev ? c0 + clen : c0) == edge) {
            if (ci > 0) {
#pragma unroll
                for (int v = 0; v < 16; ++v) base_sum[v] = running(v, age);
                S[0] = zero16();
                since = 0;
                age = 1.f;
            }
            // (the state that the walk started from is there; stores marked, as this launch reads none of them: backward of 64 x 4 001 in
            // bf16 107 -> 104 us, forward of the same in fp32 125 -> 119)
            if (rows && pb.emit && (ci > 0 || !pb.state)) {
                int t = threadIdx.x;
                asm volatile("" : "+v"(t));   // (worked out anew, as below)
                float* at = pb.emit + ((size_t)grp * g.P_Ts + ps + at_slot) * (size_t)(D * D) + (32 * rt + (t >> 3 & 4)) * D + 32 * ct + (t & 31);
#pragma unroll
                for (int v = 0; v < 16; ++v) __builtin_nontemporal_store(base_sum[v], at + acc_row(v) * D);
            }
            at_slot += rev ? -1 : 1;
            edge = (at_slot + (rev ? 1 : 0)) * slot;
        }
        f32x16 acc, low;   // (fp32: products of the higher orders have a sum of their own for the whole chunk)
        bf16x8 q[KS][NP];
        if (rows) {
            // (rows past the end: the last one once more, whose results nobody reads; a zero instead of it would be a select
            // that waits for the load here)
            const T* row = A + (size_t)min(c0 + 32 * rt + l32, len - 1) * D + 8 * h;
#pragma unroll
            for (int ks = 0; ks < KS; ++ks) to_planes(load8(row + 16 * ks, true), q[ks]);
            // snapshot of the running state, rows = its second index
            if (have_state) {
                pin_vgpr(snap_at);
#pragma unroll
                for (int v = 0; v < 16; v += 8) {
                    float x[8];
                    bf16x8 p[3];
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[e] = running(v + e, age);
                    split8(x, p);
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const bf16x4 lo = {p[i][0], p[i][1], p[i][2], p[i][3]}, hi = {p[i][4], p[i][5], p[i][6], p[i][7]};
                        *reinterpret_cast<bf16x4*>(snap + i * LD::SPLANE + (snap_at ^ (v << 2))) = lo;
                        *reinterpret_cast<bf16x4*>(snap + i * LD::SPLANE + (snap_at ^ ((v << 2) + 16))) = hi;
                    }
                }
            }
        }
        if (DECAY && update) {
            const float wc = decay_pow((float)clen, l2);
#pragma unroll
            for (int v = 0; v < 16; ++v) S[0][v] *= wc;
        }
        if (ci > 0 && ci <= ci0) __syncthreads();   // the previous stage has been read (a chunk with rows ends with a barrier)
        st.put(smem, tid);
        if (update) st.fetch(Bk, Cv, rev ? c0 - kRows64 : c0 + kRows64, len, tid);
        __syncthreads();
        if (rows) {
            acc = zero16();
            if constexpr (LOW) low = zero16();
            if (have_state) {
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    bf16x8 b[3];
                    frag_at<3>(snap + 32 * ct * 2 * D, LD::SPLANE, row_at ^ (32 * ks), b);
                    if constexpr (LOW) low = mm_either<TR, 1, 2>(q[ks], b, low);
                    else acc = mm_either<TR, 1, 2>(q[ks], b, acc);
                }
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    bf16x8 b[1];
                    frag_at<1>(snap + 32 * ct * 2 * D, LD::SPLANE, row_at ^ (32 * ks), b);
                    acc = mm_either<TR, 0, 0>(q[ks], b, acc);
                }
                if (DECAY) {
                    // the state sits one token before the chunk (causal) or one after it
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int i = 32 * rt + (TR ? l32 : acc_row(v) + 4 * h);
                        const float f = decay_pow((float)(rev ? max(clen - i, 0) : i + 1), l2);
                        acc[v] *= f;
                        if constexpr (LOW) low[v] *= f;
                    }
                }
            }
#pragma unroll 1
            for (int u = rev ? rt : 0; u <= (rev ? 1 : rt); ++u) {
                if (32 * u >= clen) break;
                pin_vgpr(row_at);   // (four offsets worked out at each use, not kept)
                const char* buf = smem + u * SUB;
                f32x16 sc = zero16();
                if constexpr (NP > 1) {
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) {
                        bf16x8 k[NP];
                        frag_at<NP>(buf, Stage::PLANE, row_at ^ (32 * ks), k);
                        sc = mm<1, 2>(k, q[ks], sc);
                    }
                }
#pragma unroll
                for (int ks = 0; ks < KS; ++ks) {
                    bf16x8 k[1];
                    frag_at<1>(buf, Stage::PLANE, row_at ^ (32 * ks), k);
                    sc = mm<0, 0>(k, q[ks], sc);
                }
                if (DECAY || u == rt) {
                    mask_tile<DECAY>(sc, 32 * (rt - u) + l32 - 4 * h, u == rt, rev, l2);
                }
                bf16x8 p[2][3];
                acc_frag(sc, 0, p[0]);
                acc_frag(sc, 8, p[1]);
                bf16x8 v[2][NP];
                col_frag<D>(buf + Stage::TENSOR, Stage::PLANE, 0, 32 * ct, lane, v[0]);
                col_frag<D>(buf + Stage::TENSOR, Stage::PLANE, 16, 32 * ct, lane, v[1]);
                if constexpr (LOW) low = mm_either<TR, 1, 2>(p[1], v[1], mm_either<TR, 1, 2>(p[0], v[0], low));
                else acc += mm_either<TR, 1, 2>(p[1], v[1], mm_either<TR, 1, 2>(p[0], v[0], zero16()));
                acc = mm_either<TR, 0, 0>(p[1], v[1], mm_either<TR, 0, 0>(p[0], v[0], acc));
            }
        }
        if (update) {
#pragma unroll 1
            for (int r0 = 0; r0 < clen; r0 += 32)
                state_step<T, D, D, Stage::PLANE, DECAY, 2>(S, smem + (r0 / 32) * SUB, Stage::TENSOR, 0, w, lane,
                                                            rev ? r0 : clen - 1 - r0, rev ? 1 : -1, l2);
        }
        have_state = true;
        since += clen;
        if (!rows) continue;

        // (not finite: from this chunk on in fp32, as above)
        if constexpr (LOW) acc += low;
        float odd = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) odd = fmaf(acc[v], 0.f, odd);
        if constexpr (TR) {   // a lane has 16 columns of its row
            const int row = 32 * rt + l32;
#pragma unroll
            for (int v = 0; v < 16; v += 4) {
                const u32x2 two = {pack2(acc[v], acc[v + 1]), pack2(acc[v + 2], acc[v + 3])};
                *reinterpret_cast<u32x2*>(patch + row * 128 + (((4 * ct + v / 4) ^ (row >> 1 & 7)) << 4) + 8 * h) = two;
            }
        }
        if (any_odd(odd != 0.f, flag)) {
            redo = ci;
            break;
        }
        if constexpr (TR) {
            int t = threadIdx.x;
            asm volatile("" : "+v"(t));   // (worked out anew: 168 registers are what three workgroups on a CU leave)
            const int ch = t & 7;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int row = (t >> 3) + 32 * i;
                const u32x4 piece = *reinterpret_cast<const u32x4*>(patch + row * 128 + ((ch ^ (row >> 1 & 7)) << 4));
                if (row < clen) *reinterpret_cast<u32x4*>(out + (size_t)(c0 + row) * D + 8 * ch) = piece;
            }
        } else {
            int t = threadIdx.x;
            asm volatile("" : "+v"(t));   // (else the address and the answers for the rows are kept through the walk)
            const int h4 = t >> 3 & 4;
            T* o = out + (size_t)(c0 + 32 * rt + h4) * D + 32 * ct + (t & 31);
            const int left = clen - 32 * rt - h4;
            if (clen >= 32 * rt + 32) {
#pragma unroll
                for (int v = 0; v < 16; ++v) store1(o + acc_row(v) * D, acc[v]);
            } else {
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    if (acc_row(v) < left) store1(o + acc_row(v) * D, acc[v]);
            }
        }
    }
    if (redo < ci1) attn_scalar<T, D, kRows64>(g, probs, pg, redo, reinterpret_cast<float*>(snap));
}

template <typename T, int D, bool DECAY>
hipError_t states_TD(const Geom& g, const T* K, const T* V, float* M, int anchor, int of_slots, hipStream_t st)
{
    constexpr int DP = D < 32 ? 32 : D, ROWS = (planes_of<T>::n == 3 && D == 128) ? 32 : 64;
    constexpr int stages = 2 * PairStage<T, D, DP, ROWS, kThr>::BYTES, lds = stages < 16384 ? 16384 : stages;
    hipError_t e = allow_dynamic_lds<states_planes_kernel<T, D, DECAY>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((states_planes_kernel<T, D, DECAY>), dim3(g.T_s, g.G), dim3(kThr), lds, st, g, K, V, M, anchor, of_slots);
    return hipGetLastError();
}

template <typename T, int D, bool DECAY>
hipError_t attn_TD(const Geom& g, const PlanesProblems& p, int n, hipStream_t st)
{
    constexpr int lds = D == 64 ? Attn64Lds<T>::BYTES : AttnLds<T, D, DECAY>::BYTES, rows = D == 64 ? kRows64 : kChunk;
    hipError_t e;
    if constexpr (D == 64) e = allow_dynamic_lds<attn64_planes_kernel<T, DECAY>>(lds);
    else e = allow_dynamic_lds<attn_planes_kernel<T, D, DECAY>>(lds);
    if (e != hipSuccess) return e;
    // Segments: as many as bring the launch to two workgroups per CU, at most eight per slot (the last
    // one then re-adds seven eighths of the slot's states).  Heads of 64, us, one | two per CU: forward of what has more work to
    // a row, one (fp32, 16 x 2000 in slots of 512 45 | 50, 32 x 2000 52 | 59; with decay 39 | 45, 44 | 47); bf16 without decay
    // two (16 x 8000 37 | 35, 256 x 1000 53 | 45), but segments of a chunk only while there is a CU for each (16 x 2000 24 | 27).
    const int64_t chunks = std::min<int64_t>((std::min<int64_t>(g.L, g.N) + rows - 1) / rows, INT32_MAX / 2), cus = cu_count();
    const int64_t wgs = (int64_t)g.G * g.T_s * n, per_cu = D == 64 && n == 1 && (planes_of<T>::n > 1 || DECAY) ? 1 : 2;
    const int64_t most = D == 64 && wgs * chunks > cus ? (chunks + 1) / 2 : chunks;
    int64_t nseg = std::max<int64_t>(1, std::min<int64_t>({per_cu * cus / wgs, most, 8}));
    const int64_t cps = (chunks + nseg - 1) / nseg;
    nseg = (chunks + cps - 1) / cps;
    auto launch = [&](dim3 grid, const PlanesProblems& q, int per, int flat) {
        const uint32_t in_group = (uint32_t)(g.T_s * nseg);
        const PlanesGrid pg = {per, (int)nseg, (int)cps, flat, in_group, (uint32_t)(((uint64_t)1 << 32) / std::max(2u, in_group)),
                               (uint32_t)(((uint64_t)1 << 32) / std::max<int64_t>(2, nseg))};
        if constexpr (D == 64) hipLaunchKernelGGL((attn64_planes_kernel<T, DECAY>), grid, dim3(kThr), lds, st, g, q, pg);
        else hipLaunchKernelGGL((attn_planes_kernel<T, D, DECAY>), grid, dim3(kThr), lds, st, g, q, pg);
        return hipGetLastError();
    };
    const int64_t units = ((int64_t)g.G * g.T_s * nseg + 7) / 8 * 8;
    if (n == 3 && units * n < ((int64_t)1 << 32) / kThr) return launch(dim3((unsigned)(units * n)), p, n, 1);
    // (a grid holds fewer than 2^32 threads per axis: past that groups are the other axis, and the problems may go one by one)
    const int per = (int64_t)g.T_s * nseg * n < ((int64_t)1 << 32) / kThr ? n : 1;
    for (int i = 0; i < n; i += per) {
        PlanesProblems sub = p;
        if (per == 1) sub.p[0] = p.p[i];
        e = launch(dim3((unsigned)(g.T_s * nseg * per), g.G), sub, per, 0);
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

template <typename T, int D>
hipError_t states_T(const Geom& g, const void* K, const void* V, float* M, int anchor, int of_slots, hipStream_t st)
{
    const T *k = static_cast<const T*>(K), *v = static_cast<const T*>(V);
    return g.decay ? states_TD<T, D, true>(g, k, v, M, anchor, of_slots, st) : states_TD<T, D, false>(g, k, v, M, anchor, of_slots, st);
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
                                int of_slots, hipStream_t st)
{
    LASP2_FOR_TYPE_AND_SIZE(states_T, g, K, V, M, anchor_start, of_slots, st)
}

bool planes_emit(const Geom& g) { return g.d == 64 && (g.L / g.wslots) % kRows64 == 0 && (g.wslots > 1 || g.lone_slots); }

hipError_t launch_attn_fwd_planes(const Geom& g, int dtype, const void* Q, const void* K, const void* V, const float* P,
                                  float* emit, void* O, hipStream_t st)
{
    PlanesProblems p = {};
    p.p[0] = {Q, K, V, P, O, 0, 0, emit};
    return attn_any(g, dtype, p, 1, st);
}

hipError_t launch_attn_bwd_planes(const Geom& g, int dtype, const void* Q, const void* K, const void* V, const void* dO,
                                  const float* P, const float* dR, float* emit, void* dQ, void* dK, void* dV, hipStream_t st)
{
    PlanesProblems p = {};
    // dQ: the forward problem with (dO, V, K) in the roles of (Q, K, V); its state is
    // V^T K = (K^T V)^T, i.e. the cached prefix read transposed.
    p.p[0] = {dO, V, K, P, dQ, 1, 0, nullptr};
    // dV: anti-causal problem with (K, Q, dO); state dM_{t+1:T} = sum Q^T dO.
    p.p[1] = {K, Q, dO, dR, dV, 0, 1, emit};
    // dK: anti-causal problem with (V, dO, Q); state dO^T Q = dM^T.
    p.p[2] = {V, dO, Q, dR, dK, 1, 1, nullptr};
    return attn_any(g, dtype, p, 3, st);
}

}  // namespace lasp2

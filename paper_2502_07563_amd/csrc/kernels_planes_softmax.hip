// Softmax attention on the matrix cores for the shapes kernels_softmax.hip does not take (fp32 of any head
// size, bf16 with d < 128).  All products go through split planes (planes.h): scores, probabilities and
// their gradients have fp32 accuracy whatever the input type.
//
// One scheme serves the three kernels.  A wave owns 32 rows (queries, or keys for dK and dV), a row per lane, its
// operands in registers; the partner rows pass through LDS in stages.  Scores are formed transposed, so
// the row statistics are per-lane scalars and the probabilities are the next product's operand as they
// stand.  The waves of a workgroup are QW row tiles times KW shares of the partner rows, whose results are
// merged at the end: 4 x 1 when such workgroups fill the device; 2 x 4 otherwise, where the longest causal
// row sets the time.  The two row tiles are then mirrored (tile i with the i-th from the end), and a SIMD
// has one wave of each, so that every workgroup has the same number of tiles.  In the forward and in dQ the shorter tile's waves,
// once they are done, fill the stages for the longer one's (HELP): filling takes as long as a tile's scores and products, and a
// workgroup of the longest and the shortest tile is nearly all such stages.  (A middle one has half as many stages with two tiles
// each and ends first: the longest row still sets the time.)  A stage of theirs then takes 5200 clocks instead of 6700; forward,
// us, causal: fp32 8 x 2003 x 64 52 -> 50, 8 x 1500 x 128 108 -> 79, 4 x 4000 x 16 49 -> 33; bf16 16 x 2500 x 64 88 -> 70; dQ of the first
// 59 -> 55.  dK and dV read both their partners in both of their products, and own rows fill what LDS there is: not there.
// Masks are applied to tiles at the border alone.
// Bounds: vector instructions - in fp32 the splits of the stages (five and a half per element) and of the scores -
// and the matrix products beside them (six bf16 ones per fp32 one).
#include "planes.h"

#include <algorithm>

namespace lasp2 {
namespace {

constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;

template <typename T, int D, int QW_, int KW_>
struct SmCfg {
    static constexpr int NP = planes_of<T>::n, DP = D < 32 ? 32 : D, NT = DP / 32, KS = D / 16, QW = QW_, KW = KW_, THR = 64 * QW * KW;
    static constexpr int ROWS = 32 * KW < 64 && !(NP == 3 && D == 128) ? 64 : 32 * KW;   // partner rows per stage
    typedef PairStage<T, D, DP, ROWS, THR> Stage;
    static constexpr bool help = QW == 2 && ROWS == 32 * KW;   // waves whose tile is done fill the stages
    static constexpr bool own_lds = NP == 3 && D == 64 && KW == 4;   // dK, dV: own rows in LDS
    static constexpr int MERGE = (KW - 1) * QW * 64 * 4;      // bytes per merged register
    static constexpr int lds(int merged, int extra)            // stage, or the merge of `merged` registers per lane
    {
        return Stage::BYTES + extra > merged * MERGE ? Stage::BYTES + extra : merged * MERGE;
    }
};

// First row of wave tile qw of workgroup bx (tiles of 32 of `rows` rows; a start at or past `rows`: none).
template <int QW>
__device__ __forceinline__ int tile_row(int bx, int qw, int rows, bool mirrored)
{
    if (QW != 2 || !mirrored) return 32 * (bx * QW + qw);
    const int tiles = (rows + 31) / 32, last = tiles - 1 - bx;
    return 32 * (qw == 0 ? last : last == bx ? tiles : bx);
}

// First row of the workgroup's tiles and the one past its last.
template <int QW>
__device__ __forceinline__ void wg_rows(int bx, int rows, bool mirrored, int& r0, int& r1)
{
    const bool m = QW == 2 && mirrored;
    r0 = m ? 32 * bx : 32 * QW * bx;
    r1 = min(rows, m ? 32 * ((rows + 31) / 32 - bx) : 32 * QW * (bx + 1));
}

// Mirrored tiles of one causal sequence: where the stages end that the shorter one (the second) takes part in, and one more.
template <int QW>
__device__ __forceinline__ int shared_end(const Geom& g, int bx, int klo, int khi, int rows)
{
    const int wr = tile_row<QW>(bx, 1, g.qn, true);
    const int end = wr < g.qn ? g.q0 + min(wr + 32, g.qn) : klo;
    return min(khi, klo + (max(end - klo, 0) + 2 * rows - 1) / rows * rows);
}

// Document of token i: [lo, hi).
__device__ __forceinline__ void doc_of(const Geom& g, int i, int& lo, int& hi)
{
    lo = 0;
    hi = g.N;
    if (g.n_seqs == 0) return;
    int a = 0, b = g.n_seqs;   // cu[a] <= i < cu[b]
    while (b - a > 1) {
        const int m = (a + b) >> 1;
        if (g.cu[m] <= i) a = m; else b = m;
    }
    lo = g.cu[a];
    hi = g.cu[a + 1];
}

// keys of query token i
__device__ __forceinline__ void keys_of(const Geom& g, int i, int causal, int& lo, int& hi)
{
    doc_of(g, i, lo, hi);
    if (causal) hi = i + 1;
}

// the share's query tokens that see key j
__device__ __forceinline__ void queries_of(const Geom& g, int j, int causal, int& lo, int& hi)
{
    doc_of(g, j, lo, hi);
    if (causal) lo = j;
    lo = max(lo, g.q0);
    hi = min(hi, g.q0 + g.qn);
}

// s = X_tile . own rows: lane = own row, accumulator rows = the 32 partner rows at `tile`
template <int DP, int KS, int NP>
__device__ __forceinline__ f32x16 scores(const char* tile, int plane_bytes, const bf16x8 (&own)[KS][NP], int l32, int h)
{
    f32x16 s = zero16();
    if constexpr (NP > 1) {
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) {
            bf16x8 k[NP];
            row_frag<DP>(tile, plane_bytes, l32, 2 * ks + h, k);
            s = mm<1, 2>(k, own[ks], s);
        }
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        bf16x8 k[1];
        row_frag<DP>(tile, plane_bytes, l32, 2 * ks + h, k);
        s = mm<0, 0>(k, own[ks], s);
    }
    return s;
}

// the same with the own rows in LDS too
template <int DP, int KS, int NP>
__device__ __forceinline__ f32x16 scores(const char* tile, int plane_bytes, const char* own, int own_plane, int l32, int h)
{
    f32x16 s = zero16();
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        bf16x8 k[NP], o[NP];
        row_frag<DP>(tile, plane_bytes, l32, 2 * ks + h, k);
        row_frag<DP>(own, own_plane, l32, 2 * ks + h, o);
        s = mm<1, 2>(k, o, s);
    }
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
        bf16x8 k[1], o[1];
        row_frag<DP>(tile, plane_bytes, l32, 2 * ks + h, k);
        row_frag<DP>(own, own_plane, l32, 2 * ks + h, o);
        s = mm<0, 0>(k, o, s);
    }
    return s;
}

// acc[nt] (lane = own row, rows = columns of X) += X_tile^T . p over the 32 partner rows
template <int DP, int NP>
__device__ __forceinline__ void accumulate(f32x16 (&acc)[DP / 32], const char* tile, int plane_bytes, const f32x16& p, int lane)
{
    bf16x8 f[2][3];
    acc_frag(p, 0, f[0]);
    acc_frag(p, 8, f[1]);
#pragma unroll
    for (int nt = 0; nt < DP / 32; ++nt) {
        bf16x8 x[2][NP];
        col_frag<DP>(tile, plane_bytes, 0, 32 * nt, lane, x[0]);
        col_frag<DP>(tile, plane_bytes, 16, 32 * nt, lane, x[1]);
        const f32x16 low = mm<1, 2>(x[1], f[1], mm<1, 2>(x[0], f[0], zero16()));
        acc[nt] = mm<0, 0>(x[1], f[1], mm<0, 0>(x[0], f[0], acc[nt] + low));
    }
}

__device__ __forceinline__ void store4(float* p, const float (&x)[4])
{
    const f32x4 v = {x[0], x[1], x[2], x[3]};
    *reinterpret_cast<f32x4*>(p) = v;
}
__device__ __forceinline__ void store4(__hip_bfloat16* p, const float (&x)[4])
{
    const u32x2 v = {pack2(x[0], x[1]), pack2(x[2], x[3])};
    *reinterpret_cast<u32x2*>(p) = v;
}

// row of out (D elements) from a transposed accumulator, times f
template <typename T, int D>
__device__ __forceinline__ void store_row(T* row, const f32x16 (&acc)[(D < 32 ? 32 : D) / 32], float f, int h)
{
#pragma unroll
    for (int nt = 0; nt < (D < 32 ? 32 : D) / 32; ++nt)
#pragma unroll
        for (int v = 0; v < 16; v += 4) {
            const int c = 32 * nt + acc_row(v) + 4 * h;
            const float x[4] = {acc[nt][v] * f, acc[nt][v + 1] * f, acc[nt][v + 2] * f, acc[nt][v + 3] * f};
            if (c < D) store4(row + c, x);
        }
}

template <typename T, int D, int KS, int NP>
__device__ __forceinline__ void load_rows(bf16x8 (&f)[KS][NP], const T* row, bool ok, int h)
{
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) to_planes(load8(row + 16 * ks + 8 * h, ok), f[ks]);
}

// ---- Rows with a non-finite result, once more in fp32, by the row's wave ----
// A non-finite partner row reaches, as 0 * inf, the rows of its tile that the mask (or their document) keeps from it,
// and planes make NaN of an infinity and of what rounds to one (planes.h): an infinite key whose scores are -inf has
// the probability 0.  The sums below are over a row's own partners and the elements as they are.

// The lane, worked out anew, so that it does not stay in a register through the walk before.
__device__ __forceinline__ int lane_again()
{
    int t = threadIdx.x;
    asm volatile("" : "+v"(t));
    return t & 63;
}

// lanes (h = 0 and 1) of the rows whose accumulators are not all finite, as a mask of rows
template <int D>
__device__ __forceinline__ uint32_t odd_rows(const f32x16 (&acc)[(D < 32 ? 32 : D) / 32], float extra, bool valid, int h)
{
    float odd = extra * 0.f;
#pragma unroll
    for (int nt = 0; nt < (D < 32 ? 32 : D) / 32; ++nt)
#pragma unroll
        for (int v = 0; v < 16; ++v) odd = fmaf(32 * nt + acc_row(v) + 4 * h < D ? acc[nt][v] : 0.f, 0.f, odd);
    const unsigned long long m = __ballot(valid && odd != 0.f);
    return (uint32_t)m | (uint32_t)(m >> 32);
}

__device__ __forceinline__ float value_of(const raw8<float>& r, int e) { return __builtin_bit_cast(float, (uint32_t)r.w[e / 4][e % 4]); }
__device__ __forceinline__ float value_of(const raw8<__hip_bfloat16>& r, int e)
{
    const uint32_t w = r.w[0][e / 2];
    return __builtin_bit_cast(float, e % 2 ? w & 0xffff0000u : w << 16);
}

template <typename T, int D>
__device__ __forceinline__ float dot_row(const T* a, const T* b)
{
    float s = 0.f;
#pragma unroll 4
    for (int c = 0; c < D; c += 8) {
        const raw8<T> x = load8(a + c, true), y = load8(b + c, true);
#pragma unroll
        for (int e = 0; e < 8; ++e) s = fmaf(value_of(x, e), value_of(y, e), s);
    }
    return s;
}

// o += sum over n rows of X (1 .. 64) of (lane j's coefficient) * row j; a lane has the columns lane and lane + 64
template <typename T, int D>
__device__ __forceinline__ void add_rows(float (&o)[2], float coef, const T* X, int n, int lane)
{
    constexpr int NU = D > 64 ? 2 : 1;
    auto row = [&](int j, float (&x)[NU]) {
#pragma unroll
        for (int u = 0; u < NU; ++u) x[u] = load1(X + (size_t)j * D + min(lane + 64 * u, D - 1));
    };
    auto add = [&](int j, const float (&x)[NU]) {
        const float c = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, coef), j));
#pragma unroll
        for (int u = 0; u < NU; ++u) o[u] = fmaf(c, x[u], o[u]);
    };
    int j = 0;
#pragma unroll 1
    for (; j + 8 <= n; j += 8) {      // (eight rows' loads in flight)
        float x[8][NU];
#pragma unroll
        for (int e = 0; e < 8; ++e) row(j + e, x[e]);
#pragma unroll
        for (int e = 0; e < 8; ++e) add(j + e, x[e]);
    }
#pragma unroll 1
    for (; j < n; ++j) {
        float x[NU];
        row(j, x);
        add(j, x);
    }
}

// every column of the row is NaN: it stays so
template <int D>
__device__ __forceinline__ bool all_nan(const float (&o)[2])
{
    return __all(o[0] != o[0] && (D <= 64 || o[1] != o[1]));
}

template <typename T, int D>
__device__ __forceinline__ void put_row(T* row, const float (&o)[2], float f, int lane)
{
#pragma unroll
    for (int u = 0; u < (D > 64 ? 2 : 1); ++u)
        if (lane + 64 * u < D) store1(row + lane + 64 * u, o[u] * f);
}

// q, out: the row; K, V: of the group; keys [lo, hi).  known: the row's log-sum-exp, if the walk found a finite one.
template <typename T, int D>
__device__ __forceinline__ void fwd_row(const T* q, const T* K, const T* V, T* out, float* lse, float known, int lo, int hi, int lane)
{
    const float scale = rsqrtf((float)D);
    float m = known, l = 1.f, o[2] = {0.f, 0.f};
    bool nan = false;                 // a score is: so are the row's sum and every element
    const bool all = !(known - known == 0.f);
    if (all) {
        m = -INFINITY;
#pragma unroll 1
        for (int k0 = lo; k0 < hi && !nan; k0 += 64) {
            const float s = k0 + lane < hi ? dot_row<T, D>(q, K + (size_t)(k0 + lane) * D) * scale : -INFINITY;
            m = fmaxf(m, s);
            nan = __any(s != s);
        }
#pragma unroll
        for (int k = 32; k > 0; k >>= 1) m = fmaxf(m, __shfl_xor(m, k, 64));
        l = nan ? NAN : 0.f;
    }
    const float mu = m == -INFINITY ? 0.f : m;
#pragma unroll 1
    for (int k0 = lo; k0 < hi && !nan; k0 += 64) {
        const float p = k0 + lane < hi ? expf(dot_row<T, D>(q, K + (size_t)(k0 + lane) * D) * scale - mu) : 0.f;
        if (all) l += p;
        add_rows<T, D>(o, p, V + (size_t)k0 * D, min(64, hi - k0), lane);
        nan = !all && all_nan<D>(o);
    }
    if (all) {
#pragma unroll
        for (int k = 32; k > 0; k >>= 1) l += __shfl_xor(l, k, 64);
    }
    put_row<T, D>(out, o, 1.f / l, lane);
    if (lane == 0) *lse = all ? m + logf(l) : known;
}

template <typename T, int D>
__device__ __forceinline__ void dq_row(const T* q, const T* d, const T* K, const T* V, float lse, float dlt, T* out, int lo, int hi,
                                       int lane)
{
    const float scale = rsqrtf((float)D);
    float o[2] = {0.f, 0.f};
    bool nan = false;
#pragma unroll 1
    for (int k0 = lo; k0 < hi && !nan; k0 += 64) {
        float ds = 0.f;
        if (k0 + lane < hi) {
            const size_t r = (size_t)(k0 + lane) * D;
            ds = expf(dot_row<T, D>(q, K + r) * scale - lse) * (dot_row<T, D>(d, V + r) - dlt);
        }
        add_rows<T, D>(o, ds * scale, K + (size_t)k0 * D, min(64, hi - k0), lane);
        nan = all_nan<D>(o);
    }
    put_row<T, D>(out, o, 1.f, lane);
}

// k, x: the key's rows of K and V; Q, dO, LSE, delta: of the group's share, queries [lo, hi) counted from its first;
// dk, dv: where the row goes, or null for a row that is right as it is
template <typename T, int D>
__device__ __forceinline__ void dkv_row(const T* k, const T* x, const T* Q, const T* dO, const float* LSE, const float* delta, T* dk,
                                        T* dv, int lo, int hi, int lane)
{
    const float scale = rsqrtf((float)D);
    float ok[2] = {0.f, 0.f}, ov[2] = {0.f, 0.f};
    bool nan = false;
#pragma unroll 1
    for (int i0 = lo; i0 < hi && !nan; i0 += 64) {
        float p = 0.f, ds = 0.f;
        if (i0 + lane < hi) {
            const size_t r = (size_t)(i0 + lane) * D;
            p = expf(dot_row<T, D>(k, Q + r) * scale - LSE[i0 + lane]);
            if (dk) ds = p * (dot_row<T, D>(x, dO + r) - delta[i0 + lane]);
        }
        const int n = min(64, hi - i0);
        if (dk) add_rows<T, D>(ok, ds * scale, Q + (size_t)i0 * D, n, lane);
        if (dv) add_rows<T, D>(ov, p, dO + (size_t)i0 * D, n, lane);
        nan = (!dk || all_nan<D>(ok)) && (!dv || all_nan<D>(ov));
    }
    if (dk) put_row<T, D>(dk, ok, 1.f, lane);
    if (dv) put_row<T, D>(dv, ov, 1.f, lane);
}

template <typename T, int D, int QW, int KW>
__global__ __launch_bounds__(64 * QW * KW, D == 128 ? 1 : 2) void softmax_fwd_planes_kernel(
    Geom g, const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, T* __restrict__ O, float* __restrict__ LSE,
    int causal)
{
    typedef SmCfg<T, D, QW, KW> Cf;
    typedef typename Cf::Stage Stage;
    constexpr int NP = Cf::NP, DP = Cf::DP, NT = Cf::NT, KS = Cf::KS, ROWS = Cf::ROWS;
    constexpr bool HELP = Cf::help;
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, l32 = lane & 31;
    const int qw = w / KW, kw = w % KW, grp = blockIdx.y;
    const bool mirrored = causal && g.n_seqs == 0;
    // Order of the workgroups within a group.  Mirrored ones are alike.  Else documents start with their last rows,
    // which are the longest under a causal mask; one causal sequence (four row tiles) with its first.  The other order
    // is no better there, because the groups follow one another and the last one's longest workgroup comes late either
    // way (16 x 4096 x 128 in fp32, us, first rows first | last rows first: forward 903 | 923, backward 3110 | 3029).
    const int bx = mirrored ? blockIdx.x : gridDim.x - 1 - blockIdx.x;
    const int wr = tile_row<QW>(bx, qw, g.qn, mirrored), row = wr + l32;
    int r0, r1;
    wg_rows<QW>(bx, g.qn, mirrored, r0, r1);
    const size_t kbase = (size_t)grp * (size_t)g.N * D, qbase = (size_t)grp * (size_t)g.qn * D;
    const bool valid = row < g.qn;
    int lo = 0, hi = 0;
    if (valid) keys_of(g, g.q0 + row, causal, lo, hi);
    // the wave's and the workgroup's key ranges: both ends grow with the query
    int wlo = 0, whi = 0, alo = 0, ahi = 0, klo, khi, t;   // [alo, ahi): the keys that every row has
    if (wr < g.qn) {
        keys_of(g, g.q0 + wr, causal, wlo, ahi);
        keys_of(g, g.q0 + min(wr + 31, g.qn - 1), causal, alo, whi);
    }
    keys_of(g, g.q0 + r0, causal, klo, t);
    keys_of(g, g.q0 + r1 - 1, causal, t, khi);

    const unsigned span = (unsigned)max(hi - lo, 0);   // a partner row x counts if (unsigned)(x - lo) < span
    Stage st;
    st.fetch(K + kbase, V + kbase, klo, khi, tid);
    bf16x8 q[KS][NP];
    load_rows<T, D>(q, Q + qbase + (size_t)row * D, valid, h);
    const float c = rsqrtf((float)D) * kLog2e;
    float m = -INFINITY, l = 0.f;      // m: of the whole row, l: of this lane's half of the keys
    f32x16 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = zero16();
    // scores of the 32 keys at t0 -> probabilities, row statistics
    auto softmax = [&](f32x16& s, int t0) __attribute__((always_inline)) {
        if (t0 < alo || t0 + 32 > ahi) {
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = (unsigned)(t0 + 4 * h - lo + acc_row(v)) < span ? s[v] : -INFINITY;
        }
        float mx = s[0];
#pragma unroll
        for (int v = 1; v < 16; ++v) mx = fmaxf(mx, s[v]);
        mx = fmaxf(m, fmaxf(mx, __shfl_xor(mx, 32, 64)) * c);
        const float mu = mx == -INFINITY ? 0.f : mx;
        const float alpha = __builtin_amdgcn_exp2f(m - mu);
        m = mx;
        float ps = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = __builtin_amdgcn_exp2f(fmaf(s[v], c, -mu));
            ps += s[v];
        }
        l = fmaf(l, alpha, ps);
        if (__any(alpha != 1.f)) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt) acc[nt] *= alpha;
        }
    };

    const int kshared = HELP && mirrored ? shared_end<QW>(g, bx, klo, khi, ROWS) : khi;
    for (int k0 = klo; k0 < kshared; k0 += ROWS) {
        if (k0 > klo) __syncthreads();
        st.put(smem, tid);
        if (k0 + ROWS < kshared) st.fetch(K + kbase, V + kbase, k0 + ROWS, khi, tid);
        __syncthreads();
#pragma unroll 1
        for (int u = kw; u < ROWS / 32; u += KW) {
            const int t0 = k0 + 32 * u;
            if (t0 >= whi || t0 + 32 <= wlo) continue;
            const char* kt = smem + u * 64 * DP;
            f32x16 s = scores<DP, KS, NP>(kt, Stage::PLANE, q, l32, h);
            softmax(s, t0);
            accumulate<DP, NP>(acc, kt + Stage::TENSOR, Stage::PLANE, s, lane);
        }
    }
    if constexpr (HELP) {
        // The shorter tile is done (a stage ago): its waves fill the stages from here on.  V has two places, and half of the next one
        // is put beside the scores, the other half and K beside the products, which take twice as long.  (V whole beside the scores,
        // in one place: they waited for it, 5800 clocks a stage.)
        if (kshared < khi) {
            int vbuf = 2 * Stage::TENSOR;
            if (qw == 0) {
                __syncthreads();
                for (int k0 = kshared; k0 < khi; k0 += ROWS) {
                    const int t0 = k0 + 32 * kw;
                    f32x16 s;
                    __syncthreads();   // K and V are there
                    if (t0 < whi) s = scores<DP, KS, NP>(smem + kw * 64 * DP, Stage::PLANE, q, l32, h);
                    __syncthreads();   // K has been read
                    if (t0 < whi) {
                        softmax(s, t0);
                        accumulate<DP, NP>(acc, smem + kw * 64 * DP + vbuf, Stage::PLANE, s, lane);
                    }
                    vbuf = 3 * Stage::TENSOR - vbuf;
                }
            } else {
                typedef PairStage<T, D, DP, ROWS, 64 * KW> Half;
                const int t = tid - 64 * KW;
                Half hs;
                Half::fetch_one(hs.x, K + kbase, kshared, khi, t);
                Half::fetch_one(hs.y, V + kbase, kshared, khi, t);
                Half::put_one(hs.y, smem + vbuf, t);
                Half::fetch_one(hs.y, V + kbase, kshared + ROWS, khi, t);
                __syncthreads();
                Half::put_one(hs.x, smem, t);
                for (int k0 = kshared; k0 < khi; k0 += ROWS) {
                    Half::fetch_one(hs.x, K + kbase, k0 + ROWS, khi, t);   // (after the last stage too: see fetch_one)
                    vbuf = 3 * Stage::TENSOR - vbuf;
                    __syncthreads();
                    Half::template put_one<0, Half::NU / 2>(hs.y, smem + vbuf, t);
                    __syncthreads();
                    Half::template put_one<Half::NU / 2, Half::NU>(hs.y, smem + vbuf, t);
                    Half::fetch_one(hs.y, V + kbase, k0 + 2 * ROWS, khi, t);
                    Half::put_one(hs.x, smem, t);
                }
            }
        }
    }
    l += __shfl_xor(l, 32, 64);
    if constexpr (KW > 1) {
        float* part = reinterpret_cast<float*>(smem) + (((kw - 1) * QW + qw) * (16 * NT + 2)) * 64 + lane;
        __syncthreads();
        if (kw > 0) {
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 16; ++v) part[(16 * nt + v) * 64] = acc[nt][v];
            part[16 * NT * 64] = m;
            part[(16 * NT + 1) * 64] = l;
        }
        __syncthreads();
        if (kw > 0) return;
#pragma unroll 1
        for (int k = 1; k < KW; ++k) {
            const float* o = reinterpret_cast<const float*>(smem) + (((k - 1) * QW + qw) * (16 * NT + 2)) * 64 + lane;
            const float om = o[16 * NT * 64], mn = fmaxf(m, om), mu = mn == -INFINITY ? 0.f : mn;
            const float fa = __builtin_amdgcn_exp2f(m - mu), fb = __builtin_amdgcn_exp2f(om - mu);
            l = l * fa + o[(16 * NT + 1) * 64] * fb;
            m = mn;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[nt][v] = acc[nt][v] * fa + o[(16 * nt + v) * 64] * fb;
        }
    }
    const float inv = 1.f / l, lse = fmaf(m, kLn2, logf(l));
    const int ln = lane_again(), first = __builtin_amdgcn_readfirstlane(row);
    uint32_t odd = odd_rows<D>(acc, inv, valid, h);
    if (valid && !((odd >> (ln & 31)) & 1u)) {
        store_row<T, D>(O + qbase + (size_t)row * D, acc, inv, h);
        if (h == 0) LSE[(size_t)grp * g.qn + row] = lse;
    }
    for (; odd; odd &= odd - 1) {
        const int r = first + __builtin_ctz(odd);
        keys_of(g, g.q0 + r, causal, klo, khi);
        fwd_row<T, D>(Q + qbase + (size_t)r * D, K + kbase, V + kbase, O + qbase + (size_t)r * D, LSE + (size_t)grp * g.qn + r,
                      __shfl(lse, __builtin_ctz(odd), 64), klo, khi, ln);
    }
}

// dQ = scale * sum_j dS_j k_j, with dS = P (dO.v - delta), P rebuilt from the log-sum-exp
template <typename T, int D, int QW, int KW>
__global__ __launch_bounds__(64 * QW * KW, D == 128 ? 1 : 2) void softmax_bwd_dq_planes_kernel(
    Geom g, const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V, const T* __restrict__ dO,
    const float* __restrict__ LSE, const float* __restrict__ delta, T* __restrict__ dQ, int causal)
{
    typedef SmCfg<T, D, QW, KW> Cf;
    typedef typename Cf::Stage Stage;
    constexpr int NP = Cf::NP, DP = Cf::DP, NT = Cf::NT, KS = Cf::KS, ROWS = Cf::ROWS;
    constexpr bool HELP = Cf::help;
    extern __shared__ __align__(16) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, l32 = lane & 31;
    const int qw = w / KW, kw = w % KW, grp = blockIdx.y;
    const bool mirrored = causal && g.n_seqs == 0;
    const int bx = mirrored ? blockIdx.x : gridDim.x - 1 - blockIdx.x;   // as in the forward
    const int wr = tile_row<QW>(bx, qw, g.qn, mirrored), row = wr + l32;
    int r0, r1;
    wg_rows<QW>(bx, g.qn, mirrored, r0, r1);
    const size_t kbase = (size_t)grp * (size_t)g.N * D, qbase = (size_t)grp * (size_t)g.qn * D;
    const bool valid = row < g.qn;
    int lo = 0, hi = 0, wlo = 0, whi = 0, alo = 0, ahi = 0, klo, khi, t;   // [alo, ahi): the keys that every row has
    float lse2 = 0.f, dlt = 0.f;
    if (valid) {
        keys_of(g, g.q0 + row, causal, lo, hi);
        lse2 = LSE[(size_t)grp * g.qn + row] * kLog2e;
        dlt = delta[(size_t)grp * g.qn + row];
    }
    if (wr < g.qn) {
        keys_of(g, g.q0 + wr, causal, wlo, ahi);
        keys_of(g, g.q0 + min(wr + 31, g.qn - 1), causal, alo, whi);
    }
    keys_of(g, g.q0 + r0, causal, klo, t);
    keys_of(g, g.q0 + r1 - 1, causal, t, khi);

    const unsigned span = (unsigned)max(hi - lo, 0);
    Stage st;
    st.fetch(K + kbase, V + kbase, klo, khi, tid);
    bf16x8 q[KS][NP], d[KS][NP];
    load_rows<T, D>(q, Q + qbase + (size_t)row * D, valid, h);
    load_rows<T, D>(d, dO + qbase + (size_t)row * D, valid, h);
    const float scale = rsqrtf((float)D), c = scale * kLog2e;
    f32x16 acc[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) acc[nt] = zero16();
    // scores and dO.v of the 32 keys at t0 -> dS
    auto gradient = [&](f32x16& s, const f32x16& dp, int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int v = 0; v < 16; ++v) s[v] = __builtin_amdgcn_exp2f(fmaf(s[v], c, -lse2)) * (dp[v] - dlt);
        if (t0 < alo || t0 + 32 > ahi) {
#pragma unroll
            for (int v = 0; v < 16; ++v) s[v] = (unsigned)(t0 + 4 * h - lo + acc_row(v)) < span ? s[v] : 0.f;
        }
    };

    const int kshared = HELP && mirrored ? shared_end<QW>(g, bx, klo, khi, ROWS) : khi;
    for (int k0 = klo; k0 < kshared; k0 += ROWS) {
        if (k0 > klo) __syncthreads();
        st.put(smem, tid);
        if (k0 + ROWS < kshared) st.fetch(K + kbase, V + kbase, k0 + ROWS, khi, tid);
        __syncthreads();
#pragma unroll 1
        for (int u = kw; u < ROWS / 32; u += KW) {
            const int t0 = k0 + 32 * u;
            if (t0 >= whi || t0 + 32 <= wlo) continue;
            const char* kt = smem + u * 64 * DP;
            f32x16 s = scores<DP, KS, NP>(kt, Stage::PLANE, q, l32, h);
            const f32x16 dp = scores<DP, KS, NP>(kt + Stage::TENSOR, Stage::PLANE, d, l32, h);
            gradient(s, dp, t0);
            accumulate<DP, NP>(acc, kt, Stage::PLANE, s, lane);
        }
    }
    if constexpr (HELP) {
        // (as in the forward; here K has two places, as it is what the second product reads)
        if (kshared < khi) {
            int kbuf = 2 * Stage::TENSOR;
            if (qw == 0) {
                __syncthreads();
                for (int k0 = kshared; k0 < khi; k0 += ROWS) {
                    const int t0 = k0 + 32 * kw;
                    const char* kt = smem + kw * 64 * DP;
                    f32x16 s, dp;
                    __syncthreads();   // K and V are there
                    if (t0 < whi) {
                        s = scores<DP, KS, NP>(kt + kbuf, Stage::PLANE, q, l32, h);
                        dp = scores<DP, KS, NP>(kt + Stage::TENSOR, Stage::PLANE, d, l32, h);
                    }
                    __syncthreads();   // V has been read
                    if (t0 < whi) {
                        gradient(s, dp, t0);
                        accumulate<DP, NP>(acc, kt + kbuf, Stage::PLANE, s, lane);
                    }
                    kbuf = 2 * Stage::TENSOR - kbuf;
                }
            } else {
                typedef PairStage<T, D, DP, ROWS, 64 * KW> Half;
                const int t = tid - 64 * KW;
                Half hs;
                Half::fetch_one(hs.x, K + kbase, kshared, khi, t);
                Half::fetch_one(hs.y, V + kbase, kshared, khi, t);
                Half::put_one(hs.x, smem + kbuf, t);
                Half::fetch_one(hs.x, K + kbase, kshared + ROWS, khi, t);
                __syncthreads();
                Half::put_one(hs.y, smem + Half::TENSOR, t);
                for (int k0 = kshared; k0 < khi; k0 += ROWS) {
                    Half::fetch_one(hs.y, V + kbase, k0 + ROWS, khi, t);
                    kbuf = 2 * Stage::TENSOR - kbuf;
                    __syncthreads();
                    Half::put_one(hs.x, smem + kbuf, t);
                    Half::fetch_one(hs.x, K + kbase, k0 + 2 * ROWS, khi, t);
                    __syncthreads();
                    Half::put_one(hs.y, smem + Half::TENSOR, t);
                }
            }
        }
    }
    if constexpr (KW > 1) {
        __syncthreads();
        if (kw > 0) {
            float* part = reinterpret_cast<float*>(smem) + (((kw - 1) * QW + qw) * 16 * NT) * 64 + lane;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 16; ++v) part[(16 * nt + v) * 64] = acc[nt][v];
        }
        __syncthreads();
        if (kw > 0) return;
#pragma unroll 1
        for (int k = 1; k < KW; ++k) {
            const float* o = reinterpret_cast<const float*>(smem) + (((k - 1) * QW + qw) * 16 * NT) * 64 + lane;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[nt][v] += o[(16 * nt + v) * 64];
        }
    }
    const int ln = lane_again(), first = __builtin_amdgcn_readfirstlane(row);
    uint32_t odd = odd_rows<D>(acc, 0.f, valid, h);
    if (valid && !((odd >> (ln & 31)) & 1u)) store_row<T, D>(dQ + qbase + (size_t)(wr + (ln & 31)) * D, acc, scale, ln >> 5);
    for (; odd; odd &= odd - 1) {
        const int r = first + __builtin_ctz(odd);
        const size_t o = qbase + (size_t)r * D, i = (size_t)grp * g.qn + r;
        keys_of(g, g.q0 + r, causal, klo, khi);
        dq_row<T, D>(Q + o, dO + o, K + kbase, V + kbase, LSE[i], delta[i], dQ + o, klo, khi, ln);
    }
}

// dV = sum_i P_i dO_i and dK = scale * sum_i dS_i q_i: a key per lane, the share's queries pass through LDS with
// their log-sum-exp (base 2) and delta.  fp32, d = 64: with two accumulators the own rows' planes (96 registers)
// do not fit beside the rest at two waves per SIMD.  Eight waves keep them in LDS (158 -> 76 us at
// 8 x 2003, against spills of 72 registers), four run at one wave per SIMD.  fp32, d = 128, spills at one wave per SIMD too
// (107 registers with two row tiles, 55 with four); against scalar products, 16 x 4096 causal, backward: 16.5 -> 3.1 ms.
template <typename T, int D, int QW, int KW>
__global__ __launch_bounds__(64 * QW * KW, D == 128 || (D == 64 && planes_of<T>::n == 3 && KW == 1) ? 1 : 2)
void softmax_bwd_dkv_planes_kernel(Geom g, const T* __restrict__ Q, const T* __restrict__ K, const T* __restrict__ V,
                                   const T* __restrict__ dO, const float* __restrict__ LSE, const float* __restrict__ delta,
                                   T* __restrict__ dK, T* __restrict__ dV, int causal)
{
    typedef SmCfg<T, D, QW, KW> Cf;
    typedef typename Cf::Stage Stage;
    constexpr int NP = Cf::NP, DP = Cf::DP, NT = Cf::NT, KS = Cf::KS, ROWS = Cf::ROWS;
    extern __shared__ __align__(16) char smem[];
    constexpr bool OWN_LDS = Cf::own_lds;
    constexpr int OPLANE = 64 * DP, OTENSOR = NP * OPLANE;        // 32 own rows
    float* stat = reinterpret_cast<float*>(smem + Stage::BYTES);   // [2][ROWS]
    const int tid = threadIdx.x, lane = tid & 63, w = __builtin_amdgcn_readfirstlane(tid >> 6), h = lane >> 5, l32 = lane & 31;
    const int qw = w / KW, kw = w % KW, grp = blockIdx.y;
    const bool mirrored = causal && g.n_seqs == 0;
    const int wr = tile_row<QW>(blockIdx.x, qw, g.N, mirrored), row = wr + l32;   // (causal: the first keys have the most queries)
    int r0, r1;
    wg_rows<QW>(blockIdx.x, g.N, mirrored, r0, r1);
    const size_t kbase = (size_t)grp * (size_t)g.N * D, qbase = (size_t)grp * (size_t)g.qn * D;
    const bool valid = row < g.N;
    int lo = 0, hi = 0, wlo = 0, whi = 0, alo = 0, ahi = 0, ilo, ihi, t;   // [alo, ahi): the queries that every row has
    if (valid) queries_of(g, row, causal, lo, hi);
    if (wr < g.N) {
        queries_of(g, wr, causal, wlo, ahi);
        queries_of(g, min(wr + 31, g.N - 1), causal, alo, whi);
    }
    queries_of(g, r0, causal, ilo, t);
    queries_of(g, r1 - 1, causal, t, ihi);

    const unsigned span = (unsigned)max(hi - lo, 0);
    bf16x8 k[KS][NP], x[KS][NP];
    char* own = smem + Stage::BYTES + 8 * ROWS + qw * 2 * OTENSOR;
    if constexpr (OWN_LDS) {
        // (the tile's KW = 4 waves have a 16-byte chunk of K and V per lane; published by the first stage's barrier)
        static_assert(!OWN_LDS || 32 * (D / 8) == 64 * KW);
        const int u = 64 * kw + lane, r = u / (D / 8), ch = u % (D / 8), off = plane_off<DP>(r, ch);
        const size_t o = kbase + (size_t)(wr + r) * D + 8 * ch;
        bf16x8 a[NP], b[NP];
        to_planes(load8(K + o, wr + r < g.N), a);
        to_planes(load8(V + o, wr + r < g.N), b);
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            *reinterpret_cast<bf16x8*>(own + i * OPLANE + off) = a[i];
            *reinterpret_cast<bf16x8*>(own + OTENSOR + i * OPLANE + off) = b[i];
        }
    } else {
        load_rows<T, D>(k, K + kbase + (size_t)row * D, valid, h);
        load_rows<T, D>(x, V + kbase + (size_t)row * D, valid, h);
    }
    const float scale = rsqrtf((float)D), c = scale * kLog2e;
    f32x16 ak[NT], av[NT];
#pragma unroll
    for (int nt = 0; nt < NT; ++nt) ak[nt] = av[nt] = zero16();

    // rows of Q and dO are counted from the share's first query
    const T *Qg = Q + qbase, *Dg = dO + qbase;
    Stage st;
    float stv = 0.f;   // ROWS <= 128: one value per thread
    auto fetch = [&](int i0) {
        st.fetch(Qg, Dg, i0 - g.q0, ihi - g.q0, tid);
        const int r = tid % ROWS, i = i0 - g.q0 + r;
        stv = 0.f;
        if (tid < 2 * ROWS && i0 + r < ihi)
            stv = tid < ROWS ? LSE[(size_t)grp * g.qn + i] * kLog2e : delta[(size_t)grp * g.qn + i];
    };
    if (ilo < ihi) fetch(ilo);
    for (int i0 = ilo; i0 < ihi; i0 += ROWS) {
        if (i0 > ilo) __syncthreads();
        st.put(smem, tid);
        if (tid < 2 * ROWS) stat[tid] = stv;
        if (i0 + ROWS < ihi) fetch(i0 + ROWS);
        __syncthreads();
#pragma unroll 1
        for (int u = kw; u < ROWS / 32; u += KW) {
            const int t0 = i0 + 32 * u;
            if (t0 >= whi || t0 + 32 <= wlo) continue;
            const char* qt = smem + u * 64 * DP;
            f32x16 s, dp;
            if constexpr (OWN_LDS) {
                s = scores<DP, KS, NP>(qt, Stage::PLANE, own, OPLANE, l32, h);
                dp = scores<DP, KS, NP>(qt + Stage::TENSOR, Stage::PLANE, own + OTENSOR, OPLANE, l32, h);
            } else {
                s = scores<DP, KS, NP>(qt, Stage::PLANE, k, l32, h);
                dp = scores<DP, KS, NP>(qt + Stage::TENSOR, Stage::PLANE, x, l32, h);
            }
#pragma unroll
            for (int v = 0; v < 16; v += 4) {
                const f32x4 ls = *reinterpret_cast<const f32x4*>(stat + 32 * u + acc_row(v) + 4 * h);
                const f32x4 dl = *reinterpret_cast<const f32x4*>(stat + ROWS + 32 * u + acc_row(v) + 4 * h);
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    s[v + e] = __builtin_amdgcn_exp2f(fmaf(s[v + e], c, -ls[e]));
                    dp[v + e] = s[v + e] * (dp[v + e] - dl[e]);
                }
            }
            if (t0 < alo || t0 + 32 > ahi) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const bool keep = (unsigned)(t0 + 4 * h - lo + acc_row(v)) < span;
                    s[v] = keep ? s[v] : 0.f;
                    dp[v] = keep ? dp[v] : 0.f;
                }
            }
            accumulate<DP, NP>(av, qt + Stage::TENSOR, Stage::PLANE, s, lane);
            accumulate<DP, NP>(ak, qt, Stage::PLANE, dp, lane);
        }
    }
    if constexpr (KW > 1) {
        __syncthreads();
        if (kw > 0) {
            float* part = reinterpret_cast<float*>(smem) + (((kw - 1) * QW + qw) * 32 * NT) * 64 + lane;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    part[(16 * nt + v) * 64] = ak[nt][v];
                    part[(16 * (NT + nt) + v) * 64] = av[nt][v];
                }
        }
        __syncthreads();
        if (kw > 0) return;
#pragma unroll 1
        for (int e = 1; e < KW; ++e) {
            const float* o = reinterpret_cast<const float*>(smem) + (((e - 1) * QW + qw) * 32 * NT) * 64 + lane;
#pragma unroll
            for (int nt = 0; nt < NT; ++nt)
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    ak[nt][v] += o[(16 * nt + v) * 64];
                    av[nt][v] += o[(16 * (NT + nt) + v) * 64];
                }
        }
    }
    const int ln = lane_again(), first = wr, own_row = wr + (ln & 31);   // (row and what hangs on it are not kept through the walk)
    const bool there = own_row < g.N;
    const uint32_t oddk = odd_rows<D>(ak, 0.f, there, ln >> 5), oddv = odd_rows<D>(av, 0.f, there, ln >> 5);
    if (there && !((oddk >> (ln & 31)) & 1u)) store_row<T, D>(dK + kbase + (size_t)own_row * D, ak, scale, ln >> 5);
    if (there && !((oddv >> (ln & 31)) & 1u)) store_row<T, D>(dV + kbase + (size_t)own_row * D, av, 1.f, ln >> 5);
    for (uint32_t odd = oddk | oddv; odd; odd &= odd - 1) {
        const int b = __builtin_ctz(odd), r = first + b;
        const size_t o = kbase + (size_t)r * D, i = (size_t)grp * g.qn;
        queries_of(g, r, causal, ilo, ihi);
        dkv_row<T, D>(K + o, V + o, Qg, Dg, LSE + i, delta + i, (oddk >> b) & 1u ? dK + o : nullptr,
                      (oddv >> b) & 1u ? dV + o : nullptr, ilo - g.q0, ihi - g.q0, ln);
    }
}

// Workgroups of four row tiles, unless they fill less than the device twice over: then two tiles and four (fp32
// with d = 128, whose rows take too many registers for eight waves: two) shares of the partner rows.
// (fp32, 8 x 2003 x 64, causal, forward: 1 x 4 115 us, 2 x 4 mirrored 50 us.)
bool split_partners(const Geom& g, int rows) { return (int64_t)g.G * ((rows + 127) / 128) < 2 * (int64_t)cu_count(); }

template <typename T, int D, int QW, int KW>
hipError_t fwd_TD(const Geom& g, const T* Q, const T* K, const T* V, T* O, float* LSE, int causal, hipStream_t st)
{
    typedef SmCfg<T, D, QW, KW> Cf;
    constexpr int lds = Cf::lds(16 * Cf::NT + 2, Cf::help ? Cf::Stage::TENSOR : 0), R = 32 * Cf::QW;
    hipError_t e = allow_dynamic_lds<softmax_fwd_planes_kernel<T, D, QW, KW>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((softmax_fwd_planes_kernel<T, D, QW, KW>), dim3((g.qn + R - 1) / R, g.G), dim3(Cf::THR), lds, st, g, Q, K, V,
                       O, LSE, causal);
    return hipGetLastError();
}

template <typename T, int D, int QW, int KW>
hipError_t dq_TD(const Geom& g, const T* Q, const T* K, const T* V, const T* dO, const float* LSE, const float* delta, T* dQ,
                 int causal, hipStream_t st)
{
    typedef SmCfg<T, D, QW, KW> Cf;
    constexpr int lds = Cf::lds(16 * Cf::NT, Cf::help ? Cf::Stage::TENSOR : 0), R = 32 * Cf::QW;
    hipError_t e = allow_dynamic_lds<softmax_bwd_dq_planes_kernel<T, D, QW, KW>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((softmax_bwd_dq_planes_kernel<T, D, QW, KW>), dim3((g.qn + R - 1) / R, g.G), dim3(Cf::THR), lds, st, g, Q, K,
                       V, dO, LSE, delta, dQ, causal);
    return hipGetLastError();
}

template <typename T, int D, int QW, int KW>
hipError_t dkv_TD(const Geom& g, const T* Q, const T* K, const T* V, const T* dO, const float* LSE, const float* delta, T* dK,
                  T* dV, int causal, hipStream_t st)
{
    typedef SmCfg<T, D, QW, KW> Cf;
    constexpr int lds = Cf::lds(32 * Cf::NT, 8 * Cf::ROWS + (Cf::own_lds ? QW * 2 * Cf::NP * 64 * Cf::DP : 0)), R = 32 * Cf::QW;
    hipError_t e = allow_dynamic_lds<softmax_bwd_dkv_planes_kernel<T, D, QW, KW>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((softmax_bwd_dkv_planes_kernel<T, D, QW, KW>), dim3((g.N + R - 1) / R, g.G), dim3(Cf::THR), lds, st, g, Q, K,
                       V, dO, LSE, delta, dK, dV, causal);
    return hipGetLastError();
}

template <typename T, int D>
hipError_t fwd_T(const Geom& g, const void* Q_, const void* K_, const void* V_, void* O_, float* LSE, int causal, hipStream_t st)
{
    constexpr int KW = planes_of<T>::n == 3 && D == 128 ? 2 : 4;
    const T *Q = static_cast<const T*>(Q_), *K = static_cast<const T*>(K_), *V = static_cast<const T*>(V_);
    T* O = static_cast<T*>(O_);
    return split_partners(g, g.qn) ? fwd_TD<T, D, 2, KW>(g, Q, K, V, O, LSE, causal, st)
                                   : fwd_TD<T, D, 4, 1>(g, Q, K, V, O, LSE, causal, st);
}

template <typename T, int D>
hipError_t bwd_T(const Geom& g, const void* Q_, const void* K_, const void* V_, const void* dO_, const float* LSE, const float* delta,
                 void* dQ_, void* dK_, void* dV_, int causal, hipStream_t st)
{
    constexpr int KW = planes_of<T>::n == 3 && D == 128 ? 2 : 4;
    const T *Q = static_cast<const T*>(Q_), *K = static_cast<const T*>(K_), *V = static_cast<const T*>(V_);
    const T* dO = static_cast<const T*>(dO_);
    T *dQ = static_cast<T*>(dQ_), *dK = static_cast<T*>(dK_), *dV = static_cast<T*>(dV_);
    if (g.qn > 0) {
        const hipError_t e = split_partners(g, g.qn) ? dq_TD<T, D, 2, KW>(g, Q, K, V, dO, LSE, delta, dQ, causal, st)
                                                     : dq_TD<T, D, 4, 1>(g, Q, K, V, dO, LSE, delta, dQ, causal, st);
        if (e != hipSuccess) return e;
    }
    return split_partners(g, g.N) ? dkv_TD<T, D, 2, KW>(g, Q, K, V, dO, LSE, delta, dK, dV, causal, st)
                                  : dkv_TD<T, D, 4, 1>(g, Q, K, V, dO, LSE, delta, dK, dV, causal, st);
}

}  // namespace

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
        default: return CALL<__hip_bfloat16, 64>(__VA_ARGS__);                     \
    }

hipError_t launch_softmax_fwd_planes(const Geom& g, int dtype, const void* Q, const void* K, const void* V, void* O, float* LSE,
                                     int causal, hipStream_t st)
{
    LASP2_FOR_TYPE_AND_SIZE(fwd_T, g, Q, K, V, O, LSE, causal, st)
}

hipError_t launch_softmax_bwd_planes(const Geom& g, int dtype, const void* Q, const void* K, const void* V, const void* dO,
                                     const float* LSE, const float* delta, void* dQ, void* dK, void* dV, int causal, hipStream_t st)
{
    LASP2_FOR_TYPE_AND_SIZE(bwd_T, g, Q, K, V, dO, LSE, delta, dQ, dK, dV, causal, st)
}

}  // namespace lasp2

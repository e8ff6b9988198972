// Softmax attention for bf16 heads of 128 in launches that kernels_softmax.hip, whose workgroups take 256 queries (128 keys),
// would leave most of the CUs without.  A workgroup has 64 rows (queries, or keys for dK and dV): two row tiles of 32 by four
// shares of the partner rows, a wave each, whose results are merged through LDS at the end.  A wave's row is a lane, as there:
// scores are formed transposed, the row statistics are per lane and the probabilities are the next product's operand as they
// stand.  Partner rows pass through LDS in steps of 128, one 32-row tile per share, by direct loads, the next step's on their way
// while this one is worked on.  Under a causal mask the two row tiles are mirrored (tile i with the i-th from the end) and a
// SIMD has one wave of each, so that its work is the same in every workgroup.
// Bounds: latency; a step takes 0.7 us with two waves per SIMD.
#include "mfma_tile.h"

namespace lasp2 {
namespace {

constexpr int SS_KW = 4, SS_STEP = 32 * SS_KW, SS_THR = 512;
constexpr int SS_TENSOR = SS_STEP * ROWB, SS_RING = 2 * SS_TENSOR;   // bytes: one tensor of a step; a tensor's ring of two
constexpr float kLog2e = 1.4426950408889634f, kLn2 = 0.6931471805599453f;

__device__ __forceinline__ void document_of(const Geom& g, int i, int& lo, int& hi)
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
    document_of(g, i, lo, hi);
    if (causal) hi = i + 1;
}

// the call's query tokens that see key j
__device__ __forceinline__ void queries_of(const Geom& g, int j, int causal, int& lo, int& hi)
{
    document_of(g, j, lo, hi);
    if (causal) lo = j;
    lo = max(lo, g.q0);
    hi = min(hi, g.q0 + g.qn);
}

// Where a workgroup's rows are: tile qw of 32 rows from `wr` (at or past `rows`: none), all of them in [r0, r1).
struct Rows { int grp, wr, r0, r1; };

__device__ __forceinline__ bool find_rows(const Geom& g, int rows, bool mirrored, int qw, Rows& x)
{
    // groups one after another, each XCD a contiguous range, so that its workgroups share the partner rows in its L2
    const int nblk = (rows + 63) / 64;
    const unsigned units = (unsigned)g.G * (unsigned)nblk, per_xcd = (units + 7u) / 8u;
    const unsigned unit = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per_xcd || unit >= units) return false;
    x.grp = (int)(unit / (unsigned)nblk);
    const int b = (int)(unit % (unsigned)nblk), tiles = (rows + 31) / 32, last = tiles - 1 - b;
    x.wr = 32 * (!mirrored ? 2 * b + qw : qw == 0 ? last : last == b ? tiles : b);
    x.r0 = mirrored ? 32 * b : 64 * b;
    x.r1 = min(rows, mirrored ? 32 * (tiles - b) : 64 * (b + 1));
    return true;
}

// A wave's addresses inside a step's tile of 32 rows, and the two ways of reading it (mfma_tile.h)
struct TileAddr {
    uint32_t nat[8], tr[4][2];
    __device__ __forceinline__ TileAddr(int lane)
    {
        const int h = lane >> 5, i = lane & 15, cl = 16 * ((lane >> 4) & 1) + 4 * (i & 3), rl = i >> 2;
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) nat[ks] = (uint32_t)tile_off(lane & 31, 2 * ks + h);
#pragma unroll
        for (int tv = 0; tv < 4; ++tv) {
            tr[tv][0] = (uint32_t)tr_off(4 * h + rl, 32 * tv + cl);
            tr[tv][1] = (uint32_t)tr_off(8 + 4 * h + rl, 32 * tv + cl);
        }
    }
};

// tile . own rows: lane = own row, accumulator rows = the tile's
__device__ __forceinline__ f32x16 tile_scores(uint32_t tile, const TileAddr& a, const bf16x8 (&own)[8])
{
    f32x16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
    bf16x8 k[8];
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) k[ks] = lds_read16_u(tile + a.nat[ks]);
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) s = mfma(k[ks], own[ks], s);
    return s;
}

// the same with the own rows in LDS
__device__ __forceinline__ f32x16 tile_scores(uint32_t tile, const TileAddr& a, uint32_t own)
{
    f32x16 s;
#pragma unroll
    for (int v = 0; v < 16; ++v) s[v] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) s = mfma(lds_read16_u(tile + a.nat[ks]), lds_read16_u(own + a.nat[ks]), s);
    return s;
}

// acc (lane = own row, rows = columns of the tile) += tile^T . p
__device__ __forceinline__ void tile_add(f32x16 (&acc)[4], uint32_t tile, const TileAddr& a, const f32x16& p)
{
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        const u32x4 w = {pack2(p[8 * e], p[8 * e + 1]), pack2(p[8 * e + 2], p[8 * e + 3]), pack2(p[8 * e + 4], p[8 * e + 5]),
                         pack2(p[8 * e + 6], p[8 * e + 7])};
        const bf16x8 f = __builtin_bit_cast(bf16x8, w);
#pragma unroll
        for (int tv = 0; tv < 4; ++tv)
            acc[tv] = mfma(lds_read_tr8_u(tile + a.tr[tv][0] + 16 * e * ROWB, tile + a.tr[tv][1] + 16 * e * ROWB), f, acc[tv]);
    }
}

__device__ __forceinline__ void load_own(bf16x8 (&f)[8], const char* row, bool valid, int h)
{
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
        const u32x4 z = {0u, 0u, 0u, 0u};
        f[ks] = __builtin_bit_cast(bf16x8, valid ? *reinterpret_cast<const u32x4*>(row + 16 * h + 32 * ks) : z);
    }
}

__device__ __forceinline__ void zero_acc(f32x16 (&acc)[4])
{
#pragma unroll
    for (int tv = 0; tv < 4; ++tv)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[tv][v] = 0.f;
}

// a row from the transposed accumulators, times f
__device__ __forceinline__ void store_own(char* row, const f32x16 (&acc)[4], float f, int h)
{
#pragma unroll
    for (int tv = 0; tv < 4; ++tv)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const u32x2 p = {pack2(acc[tv][4 * q] * f, acc[tv][4 * q + 1] * f), pack2(acc[tv][4 * q + 2] * f, acc[tv][4 * q + 3] * f)};
            *reinterpret_cast<u32x2*>(row + 2 * (32 * tv + 8 * q + 4 * h)) = p;
        }
}

// The loads of step i of rows [lo, hi) of X and Y ([n][128], the group's) into their rings; rows at or past n are zeroed by settle().
struct Steps {
    const char *X, *Y;
    size_t base;
    int lo, hi, n;
    char *sX, *sY;
    __device__ __forceinline__ int count() const { return hi > lo ? (hi - lo + SS_STEP - 1) / SS_STEP : 0; }
    __device__ __forceinline__ void issue(int i, int w, int lane) const
    {
        uint32_t dvo[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) dvo[u] = dma_lane_off(2 * w + u, lane);
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int row = lo + i * SS_STEP + b * KB, o = (i & 1) * SS_TENSOR + b * STAGE_BYTES;
            if (row < hi) dma_block<8>(X, Y, base, row, n, sX + o, sY + o, w, lane, dvo);
        }
    }
    // step i has landed: what lies past the end is zero
    __device__ __forceinline__ void settle(int i, int w, int lane) const
    {
        wait_vmcnt<0>();
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int row = lo + i * SS_STEP + b * KB, o = (i & 1) * SS_TENSOR + b * STAGE_BYTES;
            if (row < hi && row + KB > n) zero_tail_rows<8>(row, n, sX + o, sY + o, w, lane);
        }
    }
};

// The shares' accumulators of one kind, added up in the wave of share 0 (part: the tile's 3 x 64 places of 64 lanes).
__device__ __forceinline__ float* share_part(char* smem, int k, int qw, int regs, int lane)
{
    return reinterpret_cast<float*>(smem) + (((k - 1) * 2 + qw) * regs) * 64 + lane;
}

__device__ __forceinline__ void add_shares(f32x16 (&acc)[4], char* smem, int kw, int qw, int lane)
{
    __syncthreads();
    if (kw > 0) {
        float* o = share_part(smem, kw, qw, 64, lane);
#pragma unroll
        for (int i = 0; i < 64; ++i) o[64 * i] = acc[i >> 4][i & 15];
    }
    __syncthreads();
    if (kw == 0) {
#pragma unroll 1
        for (int k = 1; k < SS_KW; ++k) {
            const float* o = share_part(smem, k, qw, 64, lane);
#pragma unroll
            for (int i = 0; i < 64; ++i) acc[i >> 4][i & 15] += o[64 * i];
        }
    }
}

__global__ __launch_bounds__(SS_THR) void softmax_fwd_small_kernel(Geom g, const char* __restrict__ Q, const char* __restrict__ K,
                                                                   const char* __restrict__ V, char* __restrict__ O,
                                                                   float* __restrict__ LSE, int causal, float c)
{
    extern __shared__ __attribute__((aligned(256))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), qw = w >> 2, kw = w & 3;
    Rows x;
    if (!find_rows(g, g.qn, causal && g.n_seqs == 0, qw, x)) return;
    const int row = x.wr + l32;
    const bool valid = row < g.qn;
    int lo = 0, hi = 0, wlo = 0, whi = 0, klo, khi, t;
    if (valid) keys_of(g, g.q0 + row, causal, lo, hi);
    if (x.wr < g.qn) {
        keys_of(g, g.q0 + x.wr, causal, wlo, t);
        keys_of(g, g.q0 + min(x.wr + 31, g.qn - 1), causal, t, whi);
    }
    keys_of(g, g.q0 + x.r0, causal, klo, t);
    keys_of(g, g.q0 + x.r1 - 1, causal, t, khi);
    const unsigned span = (unsigned)max(hi - lo, 0);   // key j counts if (unsigned)(j - lo) < span
    const Steps st = {K, V, (size_t)x.grp * g.N * ROWB, klo, khi, g.N, smem, smem + SS_RING};
    const int ns = st.count();
    if (ns > 0) st.issue(0, w, lane);

    const size_t qbase = (size_t)x.grp * g.qn * ROWB;
    bf16x8 q[8];
    load_own(q, Q + qbase + (size_t)min(row, g.qn - 1) * ROWB, valid, h);
    const TileAddr a(lane);
    f32x16 acc[4];
    zero_acc(acc);
    float m = -INFINITY, l = 0.f;   // m: of the row's keys of this share, l: of this lane's half of them
    for (int i = 0; i < ns; ++i) {
        st.settle(i, w, lane);
        __syncthreads();   // the step is complete in LDS; every wave is past the one whose place the next takes
        if (i + 1 < ns) st.issue(i + 1, w, lane);
        const int t0 = klo + i * SS_STEP + 32 * kw;
        if (t0 >= whi || t0 + 32 <= wlo) continue;
        const uint32_t tk = lds_addr_of(smem) + (i & 1) * SS_TENSOR + kw * (32 * ROWB), tv = tk + SS_RING;
        f32x16 s = tile_scores(tk, a, q);
        float mx = -INFINITY;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = (unsigned)(t0 + 8 * (v >> 2) + 4 * h + (v & 3) - lo) < span ? s[v] * c : -INFINITY;
            mx = fmaxf(mx, s[v]);
        }
        mx = fmaxf(m, fmaxf(mx, __shfl_xor(mx, 32, 64)));
        const float mu = mx == -INFINITY ? 0.f : mx, alpha = __builtin_amdgcn_exp2f(m - mu);
        m = mx;
        float ps = 0.f;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            s[v] = __builtin_amdgcn_exp2f(s[v] - mu);
            ps += s[v];
        }
        l = fmaf(l, alpha, ps);
        if (__any(alpha != 1.f)) {
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int v = 0; v < 16; ++v) acc[e][v] *= alpha;
        }
        tile_add(acc, tv, a, s);
    }
    l += __shfl_xor(l, 32, 64);
    __syncthreads();
    if (kw > 0) {
        float* o = share_part(smem, kw, qw, 66, lane);
#pragma unroll
        for (int i = 0; i < 64; ++i) o[64 * i] = acc[i >> 4][i & 15];
        o[64 * 64] = m;
        o[65 * 64] = l;
    }
    __syncthreads();
    if (kw > 0) return;
#pragma unroll 1
    for (int k = 1; k < SS_KW; ++k) {
        const float* o = share_part(smem, k, qw, 66, lane);
        const float om = o[64 * 64], mn = fmaxf(m, om), mu = mn == -INFINITY ? 0.f : mn;
        const float fa = __builtin_amdgcn_exp2f(m - mu), fb = __builtin_amdgcn_exp2f(om - mu);
        l = l * fa + o[65 * 64] * fb;
        m = mn;
#pragma unroll
        for (int i = 0; i < 64; ++i) acc[i >> 4][i & 15] = acc[i >> 4][i & 15] * fa + o[64 * i] * fb;
    }
    if (!valid) return;
    store_own(O + qbase + (size_t)row * ROWB, acc, l > 0.f ? 1.f / l : 0.f, h);
    if (h == 0) LSE[(size_t)x.grp * g.qn + row] = (m + log2f(l)) * kLn2;
}

// dQ = scale * sum_j dS_j k_j, dS = P (dO . v - delta), P rebuilt from the log-sum-exp
__global__ __launch_bounds__(SS_THR) void softmax_bwd_dq_small_kernel(Geom g, const char* __restrict__ Q, const char* __restrict__ K,
                                                                      const char* __restrict__ V, const char* __restrict__ dO,
                                                                      const float* __restrict__ LSE, const float* __restrict__ delta,
                                                                      char* __restrict__ dQ, int causal, float c, float scale)
{
    extern __shared__ __attribute__((aligned(256))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), qw = w >> 2, kw = w & 3;
    Rows x;
    if (!find_rows(g, g.qn, causal && g.n_seqs == 0, qw, x)) return;
    const int row = x.wr + l32;
    const bool valid = row < g.qn;
    int lo = 0, hi = 0, wlo = 0, whi = 0, klo, khi, t;
    if (valid) keys_of(g, g.q0 + row, causal, lo, hi);
    if (x.wr < g.qn) {
        keys_of(g, g.q0 + x.wr, causal, wlo, t);
        keys_of(g, g.q0 + min(x.wr + 31, g.qn - 1), causal, t, whi);
    }
    keys_of(g, g.q0 + x.r0, causal, klo, t);
    keys_of(g, g.q0 + x.r1 - 1, causal, t, khi);
    const unsigned span = (unsigned)max(hi - lo, 0);
    const Steps st = {K, V, (size_t)x.grp * g.N * ROWB, klo, khi, g.N, smem, smem + SS_RING};
    const int ns = st.count();
    if (ns > 0) st.issue(0, w, lane);

    const size_t qbase = (size_t)x.grp * g.qn * ROWB, at = (size_t)min(row, g.qn - 1);
    bf16x8 q[8], d[8];
    load_own(q, Q + qbase + at * ROWB, valid, h);
    load_own(d, dO + qbase + at * ROWB, valid, h);
    const float lse2 = valid ? LSE[(size_t)x.grp * g.qn + at] * kLog2e : 0.f, dlt = valid ? delta[(size_t)x.grp * g.qn + at] : 0.f;
    const TileAddr a(lane);
    f32x16 acc[4];
    zero_acc(acc);
    for (int i = 0; i < ns; ++i) {
        st.settle(i, w, lane);
        __syncthreads();
        if (i + 1 < ns) st.issue(i + 1, w, lane);
        const int t0 = klo + i * SS_STEP + 32 * kw;
        if (t0 >= whi || t0 + 32 <= wlo) continue;
        const uint32_t tk = lds_addr_of(smem) + (i & 1) * SS_TENSOR + kw * (32 * ROWB), tv = tk + SS_RING;
        f32x16 s = tile_scores(tk, a, q);
        const f32x16 dp = tile_scores(tv, a, d);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float p = __builtin_amdgcn_exp2f(fmaf(s[v], c, -lse2)), ds = p * (dp[v] - dlt);
            s[v] = (unsigned)(t0 + 8 * (v >> 2) + 4 * h + (v & 3) - lo) < span ? ds : 0.f;
        }
        tile_add(acc, tk, a, s);
    }
    add_shares(acc, smem, kw, qw, lane);
    if (kw == 0 && valid) store_own(dQ + qbase + (size_t)row * ROWB, acc, scale, h);
}

// dV = sum_i P_i dO_i, dK = scale * sum_i dS_i q_i: a key per lane, its row of K in registers and of V in LDS (with two
// accumulators both don't fit the 256 registers of two waves per SIMD); queries in steps with their statistics.
__global__ __launch_bounds__(SS_THR) void softmax_bwd_dkv_small_kernel(Geom g, const char* __restrict__ Q, const char* __restrict__ K,
                                                                       const char* __restrict__ V, const char* __restrict__ dO,
                                                                       const float* __restrict__ LSE, const float* __restrict__ delta,
                                                                       char* __restrict__ dK, char* __restrict__ dV, int causal,
                                                                       float c, float scale)
{
    extern __shared__ __attribute__((aligned(256))) char smem[];
    char* own = smem + 2 * SS_RING;                                            // [2 row tiles][32][128]
    float* stat = reinterpret_cast<float*>(own + 2 * 32 * ROWB);               // [2 steps][2][SS_STEP]
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), qw = w >> 2, kw = w & 3;
    Rows x;
    if (!find_rows(g, g.N, causal && g.n_seqs == 0, qw, x)) return;
    const int row = x.wr + l32;
    const bool valid = row < g.N;
    int lo = 0, hi = 0, wlo = 0, whi = 0, ilo, ihi, t;
    if (valid) queries_of(g, row, causal, lo, hi);
    if (x.wr < g.N) {
        queries_of(g, x.wr, causal, wlo, t);
        queries_of(g, min(x.wr + 31, g.N - 1), causal, t, whi);
    }
    queries_of(g, x.r0, causal, ilo, t);
    queries_of(g, x.r1 - 1, causal, t, ihi);
    const unsigned span = (unsigned)max(hi - lo, 0);
    // query rows are counted from the call's first
    const Steps st = {Q, dO, (size_t)x.grp * g.qn * ROWB, ilo - g.q0, ihi - g.q0, g.qn, smem, smem + SS_RING};
    const int ns = st.count();
    float sv = 0.f;
    auto fetch_stat = [&](int i) {   // one value per thread of the first four waves
        const int r = st.lo + i * SS_STEP + (tid & (SS_STEP - 1));
        sv = 0.f;
        if (tid < 2 * SS_STEP && r < st.hi)
            sv = tid < SS_STEP ? LSE[(size_t)x.grp * g.qn + r] * kLog2e : delta[(size_t)x.grp * g.qn + r];
    };
    if (ns > 0) { st.issue(0, w, lane); fetch_stat(0); }

    const size_t kbase = (size_t)x.grp * g.N * ROWB;
    bf16x8 k[8];
    load_own(k, K + kbase + (size_t)min(row, g.N - 1) * ROWB, valid, h);
    {   // the tile's four waves take eight rows of V each (published by the first step's barrier)
        char* o = own + qw * 32 * ROWB;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = 8 * kw + 4 * u + (lane >> 4), ch = lane & 15;
            const u32x4 z = {0u, 0u, 0u, 0u};
            *reinterpret_cast<u32x4*>(o + tile_off(r, ch)) =
                x.wr + r < g.N ? *reinterpret_cast<const u32x4*>(V + kbase + (size_t)(x.wr + r) * ROWB + 16 * ch) : z;
        }
    }
    const TileAddr a(lane);
    f32x16 ak[4], av[4];
    zero_acc(ak);
    zero_acc(av);
    for (int i = 0; i < ns; ++i) {
        st.settle(i, w, lane);
        float* sl = stat + (i & 1) * (2 * SS_STEP);
        if (tid < 2 * SS_STEP) sl[tid] = sv;
        __syncthreads();
        if (i + 1 < ns) { st.issue(i + 1, w, lane); fetch_stat(i + 1); }
        const int t0 = ilo + i * SS_STEP + 32 * kw;   // token of the tile's first query
        if (t0 >= whi || t0 + 32 <= wlo) continue;
        const uint32_t tq = lds_addr_of(smem) + (i & 1) * SS_TENSOR + kw * (32 * ROWB), td = tq + SS_RING;
        f32x16 s = tile_scores(tq, a, k);
        f32x16 dp = tile_scores(td, a, lds_addr_of(own) + qw * 32 * ROWB);
        const float* ls = sl + 32 * kw + 4 * h;
#pragma unroll
        for (int v = 0; v < 16; v += 4) {
            const f32x4 le = *reinterpret_cast<const f32x4*>(ls + 2 * v), de = *reinterpret_cast<const f32x4*>(ls + SS_STEP + 2 * v);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool keep = (unsigned)(t0 + 2 * v + e + 4 * h - lo) < span;
                const float p = __builtin_amdgcn_exp2f(fmaf(s[v + e], c, -le[e])), ds = p * (dp[v + e] - de[e]);
                s[v + e] = keep ? p : 0.f;
                dp[v + e] = keep ? ds : 0.f;
            }
        }
        tile_add(av, td, a, s);
        tile_add(ak, tq, a, dp);
    }
    add_shares(ak, smem, kw, qw, lane);
    add_shares(av, smem, kw, qw, lane);
    if (kw > 0 || !valid) return;
    store_own(dK + kbase + (size_t)row * ROWB, ak, scale, h);
    store_own(dV + kbase + (size_t)row * ROWB, av, 1.f, h);
}

unsigned small_grid(const Geom& g, int rows)
{
    const unsigned units = (unsigned)g.G * (unsigned)((rows + 63) / 64);
    return 8u * ((units + 7u) / 8u);
}

constexpr int kSmallLds = 2 * SS_RING, kSmallLdsKv = kSmallLds + 2 * 32 * ROWB + 2 * 2 * SS_STEP * 4;
const float kScale = 0.08838834764831845f;   // 1 / sqrt(128)

}  // namespace

hipError_t launch_softmax_fwd_small(const Geom& g, const void* Q, const void* K, const void* V, void* O, float* LSE, int causal,
                                    hipStream_t st)
{
    hipError_t e = allow_dynamic_lds<softmax_fwd_small_kernel>(kSmallLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(softmax_fwd_small_kernel, dim3(small_grid(g, g.qn)), dim3(SS_THR), kSmallLds, st, g, static_cast<const char*>(Q),
                       static_cast<const char*>(K), static_cast<const char*>(V), static_cast<char*>(O), LSE, causal, kScale * kLog2e);
    return hipGetLastError();
}

hipError_t launch_softmax_bwd_dq_small(const Geom& g, const void* Q, const void* K, const void* V, const void* dO, const float* LSE,
                                       const float* delta, void* dQ, int causal, hipStream_t st)
{
    if (g.qn == 0) return hipSuccess;
    hipError_t e = allow_dynamic_lds<softmax_bwd_dq_small_kernel>(kSmallLds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(softmax_bwd_dq_small_kernel, dim3(small_grid(g, g.qn)), dim3(SS_THR), kSmallLds, st, g,
                       static_cast<const char*>(Q), static_cast<const char*>(K), static_cast<const char*>(V),
                       static_cast<const char*>(dO), LSE, delta, static_cast<char*>(dQ), causal, kScale * kLog2e, kScale);
    return hipGetLastError();
}

hipError_t launch_softmax_bwd_dkv_small(const Geom& g, const void* Q, const void* K, const void* V, const void* dO, const float* LSE,
                                        const float* delta, void* dK, void* dV, int causal, hipStream_t st)
{
    hipError_t e = allow_dynamic_lds<softmax_bwd_dkv_small_kernel>(kSmallLdsKv);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(softmax_bwd_dkv_small_kernel, dim3(small_grid(g, g.N)), dim3(SS_THR), kSmallLdsKv, st, g,
                       static_cast<const char*>(Q), static_cast<const char*>(K), static_cast<const char*>(V),
                       static_cast<const char*>(dO), LSE, delta, static_cast<char*>(dK), static_cast<char*>(dV), causal, kScale * kLog2e,
                       kScale);
    return hipGetLastError();
}

}  // namespace lasp2

// Softmax attention for bf16 heads of 128 in launches that kernels_softmax.hip, whose workgroups take 256 queries (128 keys),
// would leave most of the CUs without.  A workgroup has 64 rows (queries, or keys for dK and dV), two row tiles of 32 by four
// shares of the partner rows, or in the forward 128 rows, four tiles by two shares: a wave each, whose results are merged through LDS
// at the end.  A wave's row is a lane, as there: scores are formed transposed, the row statistics are per lane and the
// probabilities are the next product's operand as they stand.  Partner rows pass through LDS in steps of one 32-row tile per share,
// by direct loads, the ring's other steps requested ahead.  (Forward and dQ: the own rows are ordinary loads whose first use lies inside
// the loop, and the wait that the compiler puts there takes in the step just requested, so a step's loads are not on their
// way while the one before it is computed, whatever settle() would leave outstanding.  In dK, dV they are.)  Under a causal mask half
// of the row tiles are mirrored (the i-th from the start with the i-th from the end) and a SIMD has one wave of each kind, so that its
// work is the same in every workgroup.
// Bounds: latency and the L2: 64 rows take 64 KB of partner rows per step of 1.7 us; 128 rows half as much per row, which pays in the
// forward (16 x 1 300 causal: 64 rows 34 us, 128 30) and not in the backward (92, 95).
#include "mfma_tile.h"

namespace lasp2 {
namespace {

constexpr int SS_THR = 512;

// QW row tiles by KW shares of the partner rows; RING steps of STEP partner rows in LDS, all but one of them requested ahead
template <int QW_, int RING_>
struct Cfg {
    static constexpr int QW = QW_, KW = 8 / QW, RING = RING_, STEP = 32 * KW, BLOCKS = STEP / KB;
    static constexpr int TENSOR = STEP * ROWB, RINGB = RING * TENSOR;   // bytes: one tensor of a step, of the ring
};

// One wave instruction of direct global->LDS load of 4 bytes per lane (see dma16)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void dma4(const char* sbase, uint32_t voff, uint32_t lds_base)
{
    asm volatile("s_mov_b32 m0, %0\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_base), "v"(voff), "s"(sbase) : "memory", "m0");
}
#pragma clang diagnostic pop

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

template <int QW>
__device__ __forceinline__ bool find_rows(const Geom& g, int rows, bool mirrored, int qw, Rows& x)
{
    // groups one after another, each XCD a contiguous range, so that its workgroups share the partner rows in its L2
    constexpr int HALF = QW / 2;
    const int tiles = (rows + 31) / 32, nblk = (tiles + QW - 1) / QW;
    const unsigned units = (unsigned)g.G * (unsigned)nblk, per_xcd = (units + 7u) / 8u;
    const unsigned unit = (blockIdx.x & 7u) * per_xcd + (blockIdx.x >> 3);
    if ((blockIdx.x >> 3) >= per_xcd || unit >= units) return false;
    x.grp = (int)(unit / (unsigned)nblk);
    const int b = (int)(unit % (unsigned)nblk);
    if (!mirrored) {
        x.wr = 32 * (QW * b + qw);
        x.r0 = 32 * QW * b;
        x.r1 = min(rows, 32 * QW * (b + 1));
        return true;
    }
    // HALF tiles from the end, HALF from the start (none where the two meet)
    const int late = tiles - 1 - HALF * b - qw, early = HALF * b + qw - HALF;
    if (qw < HALF) x.wr = 32 * (late >= HALF * b ? late : tiles);
    else x.wr = 32 * (early < tiles - HALF * (b + 1) ? early : tiles);
    x.r0 = 32 * HALF * b;
    x.r1 = min(rows, 32 * (tiles - HALF * b));
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

// The loads of step i of rows [lo, hi) of X and Y ([n][128], the group's) into their rings, with the rows' values of two fp32
// arrays if sx is given; rows at or past n are zeroed by settle().
template <typename Cf>
struct Steps {
    const char *X, *Y;
    size_t base;
    int lo, hi, n;
    char *sX, *sY;
    const char *vx, *vy;   // fp32 arrays of the group, or NULL
    char* sv;              // [RING][BLOCKS][2][64]
    __device__ __forceinline__ int count() const { return hi > lo ? (hi - lo + Cf::STEP - 1) / Cf::STEP : 0; }
    __device__ __forceinline__ void issue(int i, int w, int lane) const
    {
        uint32_t dvo[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) dvo[u] = dma_lane_off(2 * w + u, lane);
#pragma unroll
        for (int b = 0; b < Cf::BLOCKS; ++b) {
            const int row = lo + i * Cf::STEP + b * KB, o = (i % Cf::RING) * Cf::TENSOR + b * STAGE_BYTES;
            if (row >= hi) continue;
            dma_block<8>(X, Y, base, row, n, sX + o, sY + o, w, lane, dvo);
            if (vx) {   // (every wave the same bytes to the same place, so that all have as many loads in flight)
                const uint32_t vo = 4u * (uint32_t)min(row + lane, n - 1), d = lds_addr_of(sv) + ((i % Cf::RING) * Cf::BLOCKS + b) * 512;
                dma4(vx, vo, d);
                dma4(vy, vo, d + 256);
            }
        }
    }
    // step i has landed (with steps of one block: once only the younger ones are outstanding); what lies past the end is zero
    __device__ __forceinline__ void settle(int i, int ns, int w, int lane) const
    {
        const int younger = Cf::BLOCKS > 1 ? 0 : min(Cf::RING - 2, ns - 1 - i);
        if (younger >= 2) { if (vx) wait_vmcnt<12>(); else wait_vmcnt<8>(); }
        else if (younger == 1) { if (vx) wait_vmcnt<6>(); else wait_vmcnt<4>(); }
        else wait_vmcnt<0>();
#pragma unroll
        for (int b = 0; b < Cf::BLOCKS; ++b) {
            const int row = lo + i * Cf::STEP + b * KB, o = (i % Cf::RING) * Cf::TENSOR + b * STAGE_BYTES;
            if (row < hi && row + KB > n) zero_tail_rows<8>(row, n, sX + o, sY + o, w, lane);
        }
    }
    __device__ __forceinline__ void start(int ns, int w, int lane) const
    {
        for (int i = 0; i < Cf::RING - 1 && i < ns; ++i) issue(i, w, lane);
    }
    // block until step i is in LDS for all; the step whose place is free then starts
    __device__ __forceinline__ void enter(int i, int ns, int w, int lane) const
    {
        settle(i, ns, w, lane);
        __syncthreads();   // complete in LDS; every wave is past step i - 1
        if (i + Cf::RING - 1 < ns) issue(i + Cf::RING - 1, w, lane);
    }
};

// The shares' accumulators of one kind, added up in the wave of share 0.
template <int QW>
__device__ __forceinline__ float* share_part(char* smem, int k, int qw, int regs, int lane)
{
    return reinterpret_cast<float*>(smem) + (((k - 1) * QW + qw) * regs) * 64 + lane;
}

template <int QW>
__device__ __forceinline__ void add_shares(f32x16 (&acc)[4], char* smem, int kw, int qw, int lane)
{
    __syncthreads();
    if (kw > 0) {
        float* o = share_part<QW>(smem, kw, qw, 64, lane);
#pragma unroll
        for (int i = 0; i < 64; ++i) o[64 * i] = acc[i >> 4][i & 15];
    }
    __syncthreads();
    if (kw == 0) {
#pragma unroll 1
        for (int k = 1; k < 8 / QW; ++k) {
            const float* o = share_part<QW>(smem, k, qw, 64, lane);
#pragma unroll
            for (int i = 0; i < 64; ++i) acc[i >> 4][i & 15] += o[64 * i];
        }
    }
}

template <int QW, int RING>
__global__ __launch_bounds__(SS_THR) void softmax_fwd_small_kernel(Geom g, const char* __restrict__ Q, const char* __restrict__ K,
                                                                   const char* __restrict__ V, char* __restrict__ O,
                                                                   float* __restrict__ LSE, int causal, float c)
{
    typedef Cfg<QW, RING> Cf;
    extern __shared__ __attribute__((aligned(256))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), qw = w / Cf::KW, kw = w % Cf::KW;
    Rows x;
    if (!find_rows<QW>(g, g.qn, causal && g.n_seqs == 0, qw, x)) return;
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
    const Steps<Cf> st = {K, V, (size_t)x.grp * g.N * ROWB, klo, khi, g.N, smem, smem + Cf::RINGB, nullptr, nullptr, nullptr};
    const int ns = st.count();
    st.start(ns, w, lane);

    const size_t qbase = (size_t)x.grp * g.qn * ROWB;
    bf16x8 q[8];
    load_own(q, Q + qbase + (size_t)min(row, g.qn - 1) * ROWB, valid, h);
    const TileAddr a(lane);
    f32x16 acc[4];
    zero_acc(acc);
    float m = -INFINITY, l = 0.f;   // m: of the row's keys of this share, l: of this lane's half of them
    for (int i = 0; i < ns; ++i) {
        st.enter(i, ns, w, lane);
        const int t0 = klo + i * Cf::STEP + 32 * kw;
        if (t0 >= whi || t0 + 32 <= wlo) continue;
        const uint32_t tk = lds_addr_of(smem) + (i % RING) * Cf::TENSOR + kw * (32 * ROWB), tv = tk + Cf::RINGB;
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
        float* o = share_part<QW>(smem, kw, qw, 66, lane);
#pragma unroll
        for (int i = 0; i < 64; ++i) o[64 * i] = acc[i >> 4][i & 15];
        o[64 * 64] = m;
        o[65 * 64] = l;
    }
    __syncthreads();
    if (kw > 0) return;
#pragma unroll 1
    for (int k = 1; k < 8 / QW; ++k) {
        const float* o = share_part<QW>(smem, k, qw, 66, lane);
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
template <int QW, int RING>
__global__ __launch_bounds__(SS_THR) void softmax_bwd_dq_small_kernel(Geom g, const char* __restrict__ Q, const char* __restrict__ K,
                                                                      const char* __restrict__ V, const char* __restrict__ dO,
                                                                      const float* __restrict__ LSE, const float* __restrict__ delta,
                                                                      char* __restrict__ dQ, int causal, float c, float scale)
{
    typedef Cfg<QW, RING> Cf;
    extern __shared__ __attribute__((aligned(256))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), qw = w / Cf::KW, kw = w % Cf::KW;
    Rows x;
    if (!find_rows<QW>(g, g.qn, causal && g.n_seqs == 0, qw, x)) return;
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
    const Steps<Cf> st = {K, V, (size_t)x.grp * g.N * ROWB, klo, khi, g.N, smem, smem + Cf::RINGB, nullptr, nullptr, nullptr};
    const int ns = st.count();
    st.start(ns, w, lane);

    const size_t qbase = (size_t)x.grp * g.qn * ROWB, at = (size_t)min(row, g.qn - 1);
    bf16x8 q[8], d[8];
    load_own(q, Q + qbase + at * ROWB, valid, h);
    load_own(d, dO + qbase + at * ROWB, valid, h);
    const float lse2 = valid ? LSE[(size_t)x.grp * g.qn + at] * kLog2e : 0.f, dlt = valid ? delta[(size_t)x.grp * g.qn + at] : 0.f;
    const TileAddr a(lane);
    f32x16 acc[4];
    zero_acc(acc);
    for (int i = 0; i < ns; ++i) {
        st.enter(i, ns, w, lane);
        const int t0 = klo + i * Cf::STEP + 32 * kw;
        if (t0 >= whi || t0 + 32 <= wlo) continue;
        const uint32_t tk = lds_addr_of(smem) + (i % RING) * Cf::TENSOR + kw * (32 * ROWB), tv = tk + Cf::RINGB;
        f32x16 s = tile_scores(tk, a, q);
        const f32x16 dp = tile_scores(tv, a, d);
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const float p = __builtin_amdgcn_exp2f(fmaf(s[v], c, -lse2)), ds = p * (dp[v] - dlt);
            s[v] = (unsigned)(t0 + 8 * (v >> 2) + 4 * h + (v & 3) - lo) < span ? ds : 0.f;
        }
        tile_add(acc, tk, a, s);
    }
    add_shares<QW>(acc, smem, kw, qw, lane);
    if (kw == 0 && valid) store_own(dQ + qbase + (size_t)row * ROWB, acc, scale, h);
}

// dV = sum_i P_i dO_i, dK = scale * sum_i dS_i q_i: a key per lane, its row of K in registers and of V in LDS (with two
// accumulators both don't fit the 256 registers of two waves per SIMD); queries in steps with their statistics.
template <int QW, int RING>
__global__ __launch_bounds__(SS_THR) void softmax_bwd_dkv_small_kernel(Geom g, const char* __restrict__ Q, const char* __restrict__ K,
                                                                       const char* __restrict__ V, const char* __restrict__ dO,
                                                                       const float* __restrict__ LSE2, const float* __restrict__ delta,
                                                                       char* __restrict__ dK, char* __restrict__ dV, int causal,
                                                                       float c, float scale)
{
    typedef Cfg<QW, RING> Cf;
    extern __shared__ __attribute__((aligned(256))) char smem[];
    char* own = smem + 2 * Cf::RINGB;          // [QW row tiles][32][128]
    char* stat = own + QW * 32 * ROWB;         // [RING][BLOCKS][2][64]
    const int tid = threadIdx.x, lane = tid & 63, h = lane >> 5, l32 = lane & 31;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6), qw = w / Cf::KW, kw = w % Cf::KW;
    Rows x;
    if (!find_rows<QW>(g, g.N, causal && g.n_seqs == 0, qw, x)) return;
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
    const size_t first = (size_t)x.grp * g.qn;
    const Steps<Cf> st = {Q, dO, first * ROWB, ilo - g.q0, ihi - g.q0, g.qn, smem, smem + Cf::RINGB,
                          reinterpret_cast<const char*>(LSE2 + first), reinterpret_cast<const char*>(delta + first), stat};
    const int ns = st.count();
    st.start(ns, w, lane);

    const size_t kbase = (size_t)x.grp * g.N * ROWB;
    bf16x8 k[8];
    load_own(k, K + kbase + (size_t)min(row, g.N - 1) * ROWB, valid, h);
    {   // the tile's KW waves take 32 / KW rows of V each (published by the first step's barrier)
        char* o = own + qw * 32 * ROWB;
#pragma unroll
        for (int u = 0; u < 8 / Cf::KW; ++u) {
            const int r = (32 / Cf::KW) * kw + 4 * u + (lane >> 4), ch = lane & 15;
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
        st.enter(i, ns, w, lane);
        const int t0 = ilo + i * Cf::STEP + 32 * kw;   // token of the tile's first query
        if (t0 >= whi || t0 + 32 <= wlo) continue;
        const uint32_t tq = lds_addr_of(smem) + (i % RING) * Cf::TENSOR + kw * (32 * ROWB), td = tq + Cf::RINGB;
        f32x16 s = tile_scores(tq, a, k);
        f32x16 dp = tile_scores(td, a, lds_addr_of(own) + qw * 32 * ROWB);
        const float* ls = reinterpret_cast<const float*>(stat + ((i % RING) * Cf::BLOCKS + kw / 2) * 512) + 32 * (kw & 1) + 4 * h;
#pragma unroll
        for (int v = 0; v < 16; v += 4) {
            const f32x4 le = *reinterpret_cast<const f32x4*>(ls + 2 * v), de = *reinterpret_cast<const f32x4*>(ls + 64 + 2 * v);
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
    add_shares<QW>(ak, smem, kw, qw, lane);
    add_shares<QW>(av, smem, kw, qw, lane);
    if (kw > 0 || !valid) return;
    store_own(dK + kbase + (size_t)row * ROWB, ak, scale, h);
    store_own(dV + kbase + (size_t)row * ROWB, av, 1.f, h);
}

const float kScale = 0.08838834764831845f;   // 1 / sqrt(128)

template <int QW>
unsigned small_grid(const Geom& g, int rows)
{
    const unsigned units = (unsigned)g.G * (unsigned)((rows + 32 * QW - 1) / (32 * QW));
    return 8u * ((units + 7u) / 8u);
}

// RING: what the LDS holds (64 KB a step of 128 rows, 32 KB of 64)
template <int QW, int RING>
hipError_t fwd_small(const Geom& g, const char* Q, const char* K, const char* V, char* O, float* LSE, int causal, hipStream_t st)
{
    constexpr int lds = 2 * Cfg<QW, RING>::RINGB;
    hipError_t e = allow_dynamic_lds<softmax_fwd_small_kernel<QW, RING>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((softmax_fwd_small_kernel<QW, RING>), dim3(small_grid<QW>(g, g.qn)), dim3(SS_THR), lds, st, g, Q, K, V, O, LSE,
                       causal, kScale * kLog2e);
    return hipGetLastError();
}

template <int QW, int RING>
hipError_t dq_small(const Geom& g, const char* Q, const char* K, const char* V, const char* dO, const float* LSE, const float* delta,
                    char* dQ, int causal, hipStream_t st)
{
    constexpr int lds = 2 * Cfg<QW, RING>::RINGB;
    hipError_t e = allow_dynamic_lds<softmax_bwd_dq_small_kernel<QW, RING>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((softmax_bwd_dq_small_kernel<QW, RING>), dim3(small_grid<QW>(g, g.qn)), dim3(SS_THR), lds, st, g, Q, K, V, dO,
                       LSE, delta, dQ, causal, kScale * kLog2e, kScale);
    return hipGetLastError();
}

template <int QW, int RING>
hipError_t dkv_small(const Geom& g, const char* Q, const char* K, const char* V, const char* dO, const float* LSE2, const float* delta,
                     char* dK, char* dV, int causal, hipStream_t st)
{
    typedef Cfg<QW, RING> Cf;
    constexpr int lds = 2 * Cf::RINGB + QW * 32 * ROWB + RING * Cf::BLOCKS * 512;
    hipError_t e = allow_dynamic_lds<softmax_bwd_dkv_small_kernel<QW, RING>>(lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((softmax_bwd_dkv_small_kernel<QW, RING>), dim3(small_grid<QW>(g, g.N)), dim3(SS_THR), lds, st, g, Q, K, V, dO,
                       LSE2, delta, dK, dV, causal, kScale * kLog2e, kScale);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_softmax_fwd_small(const Geom& g, int tiles, const void* Q_, const void* K_, const void* V_, void* O_, float* LSE,
                                    int causal, hipStream_t st)
{
    const char *Q = static_cast<const char*>(Q_), *K = static_cast<const char*>(K_), *V = static_cast<const char*>(V_);
    char* O = static_cast<char*>(O_);
    return tiles == 2 ? fwd_small<2, 2>(g, Q, K, V, O, LSE, causal, st) : fwd_small<4, 4>(g, Q, K, V, O, LSE, causal, st);
}

hipError_t launch_softmax_bwd_dq_small(const Geom& g, const void* Q_, const void* K_, const void* V_, const void* dO_,
                                       const float* LSE, const float* delta, void* dQ_, int causal, hipStream_t st)
{
    if (g.qn == 0) return hipSuccess;
    const char *Q = static_cast<const char*>(Q_), *K = static_cast<const char*>(K_), *V = static_cast<const char*>(V_);
    const char* dO = static_cast<const char*>(dO_);
    char* dQ = static_cast<char*>(dQ_);
    return dq_small<2, 2>(g, Q, K, V, dO, LSE, delta, dQ, causal, st);
}

hipError_t launch_softmax_bwd_dkv_small(const Geom& g, const void* Q_, const void* K_, const void* V_, const void* dO_,
                                        const float* LSE2, const float* delta, void* dK_, void* dV_, int causal, hipStream_t st)
{
    const char *Q = static_cast<const char*>(Q_), *K = static_cast<const char*>(K_), *V = static_cast<const char*>(V_);
    const char* dO = static_cast<const char*>(dO_);
    char *dK = static_cast<char*>(dK_), *dV = static_cast<char*>(dV_);
    return dkv_small<2, 2>(g, Q, K, V, dO, LSE2, delta, dK, dV, causal, st);
}

}  // namespace lasp2

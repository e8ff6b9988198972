// Building blocks of the split-plane matrix-core kernels (kernels_planes.hip,
// kernels_planes_softmax.hip): products of fp32 accuracy on the bf16 matrix unit.
//
// A value x of 24 significant bits is the sum of three bf16 numbers, hi = bf16(x),
// mid = bf16(x - hi), lo = x - hi - mid (both differences are exact and lo fits bf16), called its
// planes.  A product of a 3-plane operand with a bf16 one is then the exact sum of three bf16
// products, accumulated in fp32; of two 3-plane operands the six products hi.hi, hi.mid, mid.hi,
// mid.mid, hi.lo, lo.hi are formed.  The dropped mid.lo and lo.mid reach 2^-25 of the product each
// (mid is at most 2^-8 of the value, lo 2^-17), lo.lo 2^-34: together 2^-24, what the rounding of one fp32
// multiplication may cost.  bf16 inputs are one plane, fp32 inputs three,
// scores, probabilities and states always three: nothing is held in fewer bits than fp32.
// Why: the matrix unit multiplies fp32 operands at 1/16 of its bf16 rate, so three or six bf16
// products are 5 or 2.7 times faster than one fp32 instruction.
// An infinity, or a finite fp32 value that rounds to one in bf16 (above 3.39e38), has planes that make every
// sum they enter NaN; the kernels do such rows again in fp32.  Planes end at 2^-133, the last bit of bf16's
// smallest numbers: below 2^-109 a value has no exact sum any more.
#ifndef LASP2_PLANES_H
#define LASP2_PLANES_H
#include "mfma_tile.h"

#include <hip/hip_bf16.h>

namespace lasp2 {
namespace {

template <typename T> struct planes_of { static constexpr int n = 3; };
template <> struct planes_of<__hip_bfloat16> { static constexpr int n = 1; };

// A residual x - bf16(x) of one half of a packed pair, by the dot product of two: (-1, 0) . (a, b) + x.  The product is
// exact, and so is the difference; the other half enters times zero (and makes the residual NaN where it is not finite: its
// row is done again either way).  Against taking the half out and subtracting, the same bits over all exponents, and seven
// instructions for two elements instead of eleven: the split is most of the vector work of the fp32 kernels (softmax, 8 x
// 2003 x 64, forward | backward, us: 57.5 -> 52.8 | 135 -> 126; 8 x 1500 x 128 117 -> 111 | 380 -> 360).  The pairs of factors are
// made out of the compiler's sight: it would write (0, -1) as the float constant -1, which is another pair to an
// instruction that takes bf16 ones.
struct Residual {
    uint32_t lo, hi;
    __device__ __forceinline__ Residual()
    {
        asm("s_mov_b32 %0, 0xbf80" : "=s"(lo));
        asm("s_mov_b32 %0, 0xbf800000" : "=s"(hi));
    }
    __device__ __forceinline__ float of(uint32_t pair, uint32_t factors, float x) const
    {
        typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
        return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, pair), __builtin_bit_cast(bf16x2, factors), x, false);
    }
};

// lower planes of values whose pairs of highest ones are w[0] and whose residuals are y
__device__ __forceinline__ void split_rest(const Residual& r, u32x4 (&w)[3], float (&y)[8], bf16x8 (&p)[3])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) w[1][e] = pack2(y[2 * e], y[2 * e + 1]);
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = r.of(w[1][e / 2], e % 2 ? r.hi : r.lo, y[e]);
#pragma unroll
    for (int e = 0; e < 4; ++e) w[2][e] = pack2(y[2 * e], y[2 * e + 1]);
#pragma unroll
    for (int i = 0; i < 3; ++i) p[i] = __builtin_bit_cast(bf16x8, w[i]);
}

__device__ __forceinline__ void split8(const float (&x)[8], bf16x8 (&p)[3])
{
    const Residual r;
    u32x4 w[3];
    float y[8];
    // (by steps: what follows a dot product has to leave it three other instructions)
#pragma unroll
    for (int e = 0; e < 4; ++e) w[0][e] = pack2(x[2 * e], x[2 * e + 1]);   // a conversion makes a pair
#pragma unroll
    for (int e = 0; e < 8; ++e) y[e] = r.of(w[0][e / 2], e % 2 ? r.hi : r.lo, x[e]);
    split_rest(r, w, y, p);
}

// Planes of the products x f.  The first residual is taken of the exact product, by an fma, so that the planes hold what
// rounding it to fp32 first would drop (decayed states, all types and head sizes, error against 64 bits: 3 to 6 % less).
__device__ __forceinline__ void split8_products(const float (&x)[8], const float (&f)[8], bf16x8 (&p)[3])
{
    const Residual r;
    u32x4 w[3];
    float y[8];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        w[0][e] = pack2(x[2 * e] * f[2 * e], x[2 * e + 1] * f[2 * e + 1]);
        y[2 * e] = fmaf(x[2 * e], f[2 * e], -__builtin_bit_cast(float, w[0][e] << 16));
        y[2 * e + 1] = fmaf(x[2 * e + 1], f[2 * e + 1], -__builtin_bit_cast(float, w[0][e] & 0xffff0000u));
    }
    split_rest(r, w, y, p);
}

// c += the plane products of one k-step (a, b: MFMA operands) whose orders i + j lie in [LO, HI], smallest
// first.  Order 0, hi.hi, carries the value, the others are below 2^-7 of it: taken through
// separate sums (orders 2 and 1 of all k-steps first, then order 0), the many small products do not
// each cost a rounding of the large sum.
template <int LO, int HI, int NA, int NB>
__device__ __forceinline__ f32x16 mm(const bf16x8 (&a)[NA], const bf16x8 (&b)[NB], f32x16 c)
{
#pragma unroll
    for (int order = HI; order >= LO; --order)
#pragma unroll
        for (int i = 0; i <= order; ++i)
            if (i < NA && order - i < NB) c = mfma(a[i], b[order - i], c);
    return c;
}

// ---- LDS tiles: rows of DP bf16 (DP = 32, 64, 128) per plane, 16-byte chunks XOR-swizzled so
// that 16 consecutive rows at one chunk, and 4 rows x 64 bytes (the transposing read), both spread
// over all banks ----
template <int DP>
__device__ __forceinline__ int plane_off(int row, int chunk)
{
    const int sw = DP == 128 ? (((row & 3) << 2) | ((row >> 2) & 3))
                 : DP == 64  ? ((((row >> 1) & 1) << 2) | ((row >> 2) & 3))
                             : ((row >> 2) & 3);
    return row * (2 * DP) + (((chunk ^ sw) & (DP / 8 - 1)) << 4);
}

// 8 consecutive elements of a row: k = 8 chunk .. 8 chunk + 7
template <int DP, int NP>
__device__ __forceinline__ void row_frag(const char* tile, int plane_bytes, int row, int chunk, bf16x8 (&f)[NP])
{
    const int off = plane_off<DP>(row, chunk);
#pragma unroll
    for (int p = 0; p < NP; ++p) f[p] = *reinterpret_cast<const bf16x8*>(tile + p * plane_bytes + off);
}

// Transposed fetch: lane's column is col0 + lane % 32, its k-slots 0..3 are rows r0 + 4h .. + 3 and
// 4..7 rows r0 + 8 + 4h .. + 3 (h = lane / 32): the order in which a 32 x 32 accumulator holds its
// rows, so a score tile is the matching operand as it stands.
template <int DP, int NP>
__device__ __forceinline__ void col_frag(const char* tile, int plane_bytes, int r0, int col0, int lane, bf16x8 (&f)[NP])
{
    const int i = lane & 15, col = col0 + 16 * ((lane >> 4) & 1) + 4 * (i & 3);
    const int ra = r0 + 4 * (lane >> 5) + (i >> 2);
    const int lo = plane_off<DP>(ra, col >> 3) + (col & 7) * 2, hi = plane_off<DP>(ra + 8, col >> 3) + (col & 7) * 2;
#pragma unroll
    for (int p = 0; p < NP; ++p) f[p] = lds_read_tr8_at(tile + p * plane_bytes, lo, hi);
}

// row of accumulator element v (C/D layout): + 4h for the lane's half
__device__ __forceinline__ constexpr int acc_row(int v) { return 8 * (v / 4) + v % 4; }

__device__ __forceinline__ f32x16 zero16()
{
    f32x16 z;
#pragma unroll
    for (int v = 0; v < 16; ++v) z[v] = 0.f;
    return z;
}

// one element in global memory
template <typename T> __device__ __forceinline__ void store1(T* p, float x);
template <> __device__ __forceinline__ void store1(float* p, float x) { *p = x; }
template <> __device__ __forceinline__ void store1(__hip_bfloat16* p, float x) { *p = __float2bfloat16(x); }
__device__ __forceinline__ float load1(const float* p) { return *p; }
__device__ __forceinline__ float load1(const __hip_bfloat16* p) { return __bfloat162float(*p); }

// 8 consecutive elements in global memory (16-byte aligned), raw, as 16-byte words
template <typename T> struct raw8;
template <> struct raw8<float> { u32x4 w[2]; };
template <> struct raw8<__hip_bfloat16> { u32x4 w[1]; };

template <typename T>
__device__ __forceinline__ raw8<T> load8(const T* p, bool ok)
{
    raw8<T> r;
    constexpr int n = sizeof(r.w) / 16;
#pragma unroll
    for (int i = 0; i < n; ++i) {
        const u32x4 z = {0u, 0u, 0u, 0u};
        r.w[i] = ok ? reinterpret_cast<const u32x4*>(p)[i] : z;
    }
    return r;
}

__device__ __forceinline__ void to_planes(const raw8<__hip_bfloat16>& r, bf16x8 (&p)[1]) { p[0] = __builtin_bit_cast(bf16x8, r.w[0]); }
__device__ __forceinline__ void to_planes(const raw8<float>& r, bf16x8 (&p)[3])
{
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = __builtin_bit_cast(float, (uint32_t)r.w[e / 4][e % 4]);
    split8(x, p);
}

// fp32 value of element e of a fragment (exact)
template <int NP>
__device__ __forceinline__ float frag_value(const bf16x8 (&f)[NP], int e)
{
    float x = (float)f[NP - 1][e];
#pragma unroll
    for (int p = NP - 2; p >= 0; --p) x += (float)f[p][e];
    return x;
}

// 8 accumulator elements v0 .. v0+7 as an operand of three planes
__device__ __forceinline__ void acc_frag(const f32x16& s, int v0, bf16x8 (&f)[3])
{
    float x[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = s[v0 + e];
    split8(x, f);
}

// Rows tok0 .. tok0 + ROWS - 1 of X and Y on their way from global memory to LDS planes, by all
// NTHR threads: fetch() issues the loads, put() splits and writes.  Rows at or past `end` are zero.
template <typename T, int D, int DP, int ROWS, int NTHR>
struct PairStage {
    static constexpr int NP = planes_of<T>::n;
    static constexpr int CPR = D / 8, UNITS = ROWS * CPR, NU = (UNITS + NTHR - 1) / NTHR;
    static constexpr int PLANE = ROWS * DP * 2, TENSOR = NP * PLANE, BYTES = 2 * TENSOR;
    raw8<T> x[NU], y[NU];
    __device__ __forceinline__ void fetch(const T* X, const T* Y, int tok0, int end, int tid)
    {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int unit = tid + u * NTHR, r = unit / CPR;
            const bool ok = (UNITS % NTHR == 0 || unit < UNITS) && tok0 + r < end;
            const size_t o = (size_t)(tok0 + r) * D + (unit % CPR) * 8;
            x[u] = load8(X + o, ok);
            y[u] = load8(Y + o, ok);
        }
    }
    __device__ __forceinline__ void put(char* buf, int tid) const
    {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int unit = tid + u * NTHR;
            if (UNITS % NTHR != 0 && unit >= UNITS) continue;
            const int off = plane_off<DP>(unit / CPR, unit % CPR);
            bf16x8 p[NP], q[NP];
            to_planes(x[u], p);
            to_planes(y[u], q);
#pragma unroll
            for (int i = 0; i < NP; ++i) {
                *reinterpret_cast<bf16x8*>(buf + i * PLANE + off) = p[i];
                *reinterpret_cast<bf16x8*>(buf + TENSOR + i * PLANE + off) = q[i];
            }
        }
    }
    // One of the two tensors (x, at buf, or y, at buf + TENSOR).  Rows past the end are the last one: loads without a condition, or the
    // next put waits for all of them, the other tensor's too.
    __device__ __forceinline__ static void fetch_one(raw8<T> (&z)[NU], const T* Z, int tok0, int end, int tid)
    {
#pragma unroll
        for (int u = 0; u < NU; ++u) {
            const int unit = tid + u * NTHR;
            z[u] = load8(Z + (size_t)min(tok0 + unit / CPR, end - 1) * D + (unit % CPR) * 8, true);
        }
    }
    template <int U0 = 0, int U1 = NU>
    __device__ __forceinline__ static void put_one(const raw8<T> (&z)[NU], char* buf, int tid)
    {
#pragma unroll
        for (int u = U0; u < U1; ++u) {
            const int unit = tid + u * NTHR;
            if (UNITS % NTHR != 0 && unit >= UNITS) continue;
            const int off = plane_off<DP>(unit / CPR, unit % CPR);
            bf16x8 p[NP];
            to_planes(z[u], p);
#pragma unroll
            for (int i = 0; i < NP; ++i) *reinterpret_cast<bf16x8*>(buf + i * PLANE + off) = p[i];
        }
    }
};

}  // namespace
}  // namespace lasp2
#endif  // LASP2_PLANES_H

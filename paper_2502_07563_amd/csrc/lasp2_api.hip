// Host side of liblasp2: argument validation, slot arithmetic and kernel dispatch
// for the entry points declared in include/lasp2.h.  Every argument error is
// reported before the first HIP call, so the error paths run on a machine
// without a GPU.
#include "lasp2_common.h"

#include <limits.h>
#include <stdlib.h>

#include <algorithm>
#include <cmath>

namespace lasp2 {
namespace {

bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

bool supported_d(int d) { return d == 16 || d == 32 || d == 64 || d == 128; }

// Slots of L tokens that n < 2^31 tokens make (a 32-bit division where there is more than one: packed batches count them by the
// thousand, several times a call)
int64_t slots_of(int64_t n, int64_t L) { return n <= L ? (n > 0 ? 1 : 0) : (int64_t)(((uint32_t)n - 1u) / (uint32_t)L) + 1; }

// Validates the descriptor and fills the kernel geometry.  *empty is set when
// there is nothing to compute.
int make_geom(const lasp2_desc_t* desc, Geom* g, bool* empty)
{
    if (!desc) return LASP2_ERR_NULL;
    if (desc->dtype != LASP2_F32 && desc->dtype != LASP2_BF16) return LASP2_ERR_DTYPE;
    if (desc->B < 0 || desc->H < 0 || desc->N < 0) return LASP2_ERR_SHAPE;
    if (!supported_d(desc->d)) return LASP2_ERR_SHAPE;
    if (desc->C < 1 || desc->C > 512) return LASP2_ERR_SHAPE;
    if (desc->L < 0) return LASP2_ERR_SHAPE;
    int64_t L = desc->L == 0 ? desc->C : desc->L;
    if (L % desc->C != 0) return LASP2_ERR_SHAPE;
    int64_t G = (int64_t)desc->B * desc->H;
    if (G > 65535) return LASP2_ERR_SHAPE;  // grid.y carries the group index
    // every element offset must fit int64 with a wide margin
    if (G > 0 && (int64_t)desc->N > (INT64_MAX / 8) / (G * desc->d)) return LASP2_ERR_SHAPE;
    if (desc->n_seqs < 0) return LASP2_ERR_SEQLENS;

    int64_t T_s = 0;
    if (desc->n_seqs > 0) {
        if (!desc->cu_seqlens_host || !desc->cu_seqlens_dev) return LASP2_ERR_SEQLENS;
        if (desc->B != 1) return LASP2_ERR_SEQLENS;
        const int32_t* cu = desc->cu_seqlens_host;
        if (cu[0] != 0 || cu[desc->n_seqs] != desc->N) return LASP2_ERR_SEQLENS;
        for (int k = 0; k < desc->n_seqs; ++k) {
            if (cu[k + 1] <= cu[k]) return LASP2_ERR_SEQLENS;
            T_s += slots_of(cu[k + 1] - cu[k], L);
        }
        if (reinterpret_cast<uintptr_t>(desc->cu_seqlens_dev) & 3u) return LASP2_ERR_ALIGN;
    } else {
        if (desc->cu_seqlens_host || desc->cu_seqlens_dev) return LASP2_ERR_SEQLENS;
        T_s = ((int64_t)desc->N + L - 1) / L;
    }
    if (T_s > INT32_MAX) return LASP2_ERR_SHAPE;
    if (G > 0 && T_s > (INT64_MAX / 8) / (G * desc->d * desc->d)) return LASP2_ERR_SHAPE;
    // one-dimensional grids carry up to three workgroups per (group, slot) pair
    if (G * T_s > (int64_t)(INT32_MAX / 4)) return LASP2_ERR_SHAPE;

    // decay: both pointers or neither; every factor in (0, 1]
    if ((desc->decay_host == nullptr) != (desc->decay_dev == nullptr)) return LASP2_ERR_DECAY;
    if (desc->decay_host) {
        for (int h = 0; h < desc->H; ++h) {
            const float lam = desc->decay_host[h];
            if (!(lam > 0.f && lam <= 1.f)) return LASP2_ERR_DECAY;
        }
        if (reinterpret_cast<uintptr_t>(desc->decay_dev) & 3u) return LASP2_ERR_ALIGN;
    }

    g->G = (int32_t)G;
    g->H = desc->H > 0 ? desc->H : 1;
    g->decay = desc->decay_dev;
    // The MFMA decay kernels weight rows by lam^(0..63) in bf16 and undo it with lam^-(0..63)
    // in fp32; 0.35^63 = 2e-29 keeps both far from the ends of the exponent range.
    g->decay_mfma = 0;
    if (desc->decay_host) {
        g->decay_mfma = 1;
        for (int h = 0; h < desc->H; ++h)
            if (desc->decay_host[h] < 0.35f) g->decay_mfma = 0;
    }
    g->N = desc->N;
    g->q0 = 0;
    g->qn = desc->N;
    g->d = desc->d;
    g->C = desc->C;
    g->L = L;
    g->T_s = (int32_t)T_s;
    g->n_seqs = desc->n_seqs;
    g->lone_slots = (T_s == (desc->n_seqs > 0 ? (int64_t)desc->n_seqs : (int64_t)1)) ? 1 : 0;
    g->cu = desc->cu_seqlens_dev;
    // marks for slot_range: the number of slots before every doc_stride-th document
    g->wslots = 1;
    g->W = 0;
    g->sub = 1;
    g->P_Ts = g->T_s;
    g->doc_stride = 1;
    for (int j = 0; j < kDocMarks; ++j) g->doc_mark[j] = j == 0 ? 0 : INT32_MAX;
    if (desc->n_seqs > 0) {
        const int32_t* cu = desc->cu_seqlens_host;
        g->doc_stride = (desc->n_seqs + kDocMarks - 1) / kDocMarks;
        int64_t before = 0;
        for (int k = 0; k < desc->n_seqs; ++k) {
            if (k % g->doc_stride == 0) g->doc_mark[k / g->doc_stride] = (int32_t)before;
            before += slots_of(cu[k + 1] - cu[k], L);
        }
    }
    for (int j = 0; j < kDocMarks; ++j) g->doc_pmark[j] = g->doc_mark[j];
    *empty = (G == 0 || desc->N == 0);
    return LASP2_OK;
}

// ---- walks of several slots ---------------------------------------------------------------
// The state a fused pass carries across a slot boundary IS the next slot's prefix (up to the
// rounding order), so a workgroup may walk `ws` consecutive slots of a document and read the
// caller's state array only at the first.  The slot length the caller chose then no longer fixes
// how many workgroups a launch has nor how much of their time goes into starting up: one state
// per chunk (the paper's layout) still runs with walks as long as the device can keep busy.

constexpr int64_t kMaxWalkTokens = (int64_t)1 << 30;

// The geometry of the walks: g with L and T_s (and the document marks) for ws slots per walk;
// the caller's arrays stay described by P_Ts, wslots and doc_pmark.
Geom regroup(const Geom& g, const int32_t* cu_host, int ws)
{
    if (ws <= 1) return g;
    Geom w = g;
    w.wslots = ws;
    w.P_Ts = g.T_s;
    w.L = g.L * ws;
    if (g.n_seqs == 0) {
        w.T_s = (int32_t)(((int64_t)g.N + w.L - 1) / w.L);
        w.lone_slots = w.T_s == 1 ? 1 : 0;
        return w;
    }
    int64_t walks = 0, slots = 0;
    for (int j = 0; j < kDocMarks; ++j) w.doc_mark[j] = w.doc_pmark[j] = j == 0 ? 0 : INT32_MAX;
    for (int k = 0; k < g.n_seqs; ++k) {
        if (k % g.doc_stride == 0) {
            w.doc_mark[k / g.doc_stride] = (int32_t)walks;
            w.doc_pmark[k / g.doc_stride] = (int32_t)slots;
        }
        const int64_t len = cu_host[k + 1] - cu_host[k];
        walks += slots_of(len, w.L);
        slots += slots_of(len, g.L);
    }
    w.T_s = (int32_t)walks;
    w.lone_slots = walks == g.n_seqs ? 1 : 0;
    return w;
}

// The geometry of walks of W tokens (a multiple of 64) inside the slots, which are longer than that.
Geom regroup_short(const Geom& g, const int32_t* cu_host, int64_t W)
{
    Geom w = g;
    w.W = (int32_t)W;
    w.sub = (int32_t)((std::min<int64_t>(g.L, g.N) + W - 1) / W);
    auto walks_of = [&](int64_t n) {
        const int64_t full = slots_of(n, g.L) - 1;
        return full * w.sub + slots_of(n - full * g.L, W);
    };
    if (g.n_seqs == 0) {
        w.T_s = (int32_t)walks_of(g.N);
        return w;
    }
    int64_t walks = 0;
    for (int k = 0; k < g.n_seqs; ++k) {
        if (k % g.doc_stride == 0) w.doc_mark[k / g.doc_stride] = (int32_t)walks;
        walks += walks_of(cu_host[k + 1] - cu_host[k]);
    }
    w.T_s = (int32_t)walks;
    return w;
}

int64_t longest_sequence(const Geom& g, const int32_t* cu_host)
{
    if (g.n_seqs == 0) return g.N;
    int64_t m = 0;
    for (int k = 0; k < g.n_seqs; ++k) m = std::max<int64_t>(m, cu_host[k + 1] - cu_host[k]);
    return m;
}

int64_t max_walk_slots(const Geom& g) { return std::max<int64_t>(1, std::min<int64_t>(kMaxWalkTokens / g.L, INT32_MAX / 2)); }

// The environment variable LASP2_WALK_SLOTS (for tests and tuning), clamped; 0 when it is not set to a
// positive number.
int forced_walk_slots(const Geom& g)
{
    const char* e = getenv("LASP2_WALK_SLOTS");
    const long v = e ? strtol(e, nullptr, 10) : 0;
    return v >= 1 ? (int)std::min<int64_t>(v, max_walk_slots(g)) : 0;
}

// Slots per walk of lasp2_attn_fwd, and of lasp2_forward where slots are not a multiple of 64 tokens: for a launch that runs `par` walks at a time and gains
// little from walks longer than `target` tokens (measured: the forward launch is flat from about 2 048 tokens on; starting a walk costs what streaming about a hundred tokens does).
//   - Equal sequences, enough of them to fill the device by themselves: one walk per sequence,
//     which needs no prefix or suffix state at all (the serial-carry order of work).
//   - Otherwise the shortest walk of at least `target` tokens (a power of two of slots), made
//     shorter again while the launch would have fewer than two rounds of workgroups: a launch of
//     one round ends at the pace of its slowest CU, and less than one leaves CUs without work.
// LASP2_WALK_SLOTS overrides the choice.
constexpr int64_t kWalkTargetFwd = 2048;

int pick_walk_slots(const Geom& g, const int32_t* cu_host, int par, int64_t target)
{
    const int64_t longest_seq = longest_sequence(g, cu_host);
    if (g.L >= longest_seq || g.G == 0) return 1;
    const int64_t ws_max = max_walk_slots(g);
    if (const int v = forced_walk_slots(g)) return v;
    if (par < 1) par = 1;
    const int64_t ws_whole = (longest_seq + g.L - 1) / g.L;   // slots of the longest sequence
    if (g.n_seqs == 0 && ws_whole <= ws_max) {
        const int64_t rounds = ((int64_t)g.G + par - 1) / par;
        if ((int64_t)g.G * 100 >= rounds * par * 85) return (int)ws_whole;
    }
    auto units = [&](int64_t ws) {
        const int64_t W = g.L * ws;
        if (g.n_seqs == 0) return (int64_t)g.G * ((g.N + W - 1) / W);
        int64_t nw = 0;
        for (int k = 0; k < g.n_seqs; ++k) nw += slots_of(cu_host[k + 1] - cu_host[k], W);
        return (int64_t)g.G * nw;
    };
    int64_t ws = 1;
    while (ws * g.L < target && ws * 2 <= ws_max && ws < ws_whole) ws *= 2;
    while (ws > 1 && units(ws) < 2 * (int64_t)par) ws /= 2;
    return (int)ws;
}

// How lasp2_forward (walks that write states in passing, kernels_mfma.hip) and the backward cut the sequences: slots per
// walk, and whether the walks gather the state they start from themselves (`direct`: one launch, no states and prefix
// before it); also which long slots lasp2_attn_fwd takes in parts.  From an estimate in us of what each choice costs; the candidates are the
// shortest walks that fit into one to sixteen rounds of workgroups, the shortest at all, and powers of two for documents of different lengths.
// The rates are measured, the rest is fitted to 284 shapes (1 to 300 sequences of 3 to 200 000 tokens, packed batches among them) with every choice
// timed: the chosen one takes 2.2 % more than the best in the forward and 2.5 % in the backward (geometric means; 71 packed batches alone, half of
// them long documents in long slots, 6 % and 5 %: which workgroups start last, and beside which, is not followed).
//   - A row of a walk takes 0.03 us forward (dQ 0.031, the pair of the backward 0.0376; with decay 0.033 each, and 0.009 gathered), starting a walk what 256 (180)
//     rows do, a row that is gathered 0.0068 (16 heads, walks of 256, gathered | states first, us: 300 rows 15 | 22; 1 024
//     20 | 24; 2 048 28 | 30; 3 000 37 | 31; 4 096 45 | 36; backward 20 | 27, 25 | 32, 34 | 37, 44 | 46, 58 | 50).  Rows come 128 at
//     a time, with decay 256 (4 x 8 000 decayed, backward, walks of 256 51, 384 66, 512 47; 2 x 16 x 271, whole 25.7, 256 21.6).
//   - `crowded`: parts of slots gather the same rows at once, past the L2s (32 MB) at less than half that rate (2 x 4 x 38 206, slots of 2 560,
//     lasp2_attn_fwd 84 whole, 100 in parts of 640; backward 2 x 50 000, slots of 2 048, 121 whole, 128 to 145 in parts of 384 to 576).
//   - Memory: 5.2 TB/s, 8 where the tensors fit the 256 MB cache.  The one-launch backward reads four tensors more, as its two
//     workgroups per walk don't keep in step (256 sequences of 2 000: 305 | 262), large ones ten (64 of 43 174: 2420 | 2190).
//   - Of two choices that memory bounds alike the one with less work (0.05 of the walks' time on top).  Documents of
//     different lengths: the last to start is a long one, and takes 0.05 us per row beside the others, 0.6 of a walk on average (32 heads, 131 072 in
//     40 documents, forward, walks of 2 048 1434 us, 4 096 1275, 8 192 1212, whole documents 2411).
//   - States: read at 6 TB/s, 0.0118 us per row of one slot (128 slots of 20 000 rows: 236; backward with its suffix 0.0127), and 10 us for two launches; beyond 16 of
//     a sequence's states 0.1 each, as they are combined one after another (1 x 39 086, forward, walks of 192 66, 384 56); documents of different lengths spread unevenly:
//     a third more.  (32 heads, 131 072 tokens in 40 documents, forward 1500 -> 1212 us direct in walks of 8 192; 16 heads,
//     32 768 in 50 322 -> 187, backward 486 -> 341; 32 heads, 8 000 in 20 100 -> 72, 239 -> 155.)
//   - Forward walks have more than 128 rows: shorter ones take the 128-row kernel and write no states in passing (16 heads x 3 000,
//     64-token slots: walks of 128 58 us, 192 or 256 38; 2 x 2 581, slots of 192, 23 one by one, 33 by two).  Backward walks have 96 or more; the kernels for up to 128 rows, with three
//     workgroups a walk, pay while all of them fit (4 x 1 000 21 us, 26 with 256; 32 x 1 000 49, 33), and gathering walks of 128 while there are few (4 x 300 16, 21).
//   - One round ends at the pace of the slowest CU: 8 % more in the backward (16 heads, one round | two, us: 8 192 85 | 93;
//     16 384 149 | 151; 32 768 281 | 271; 262 144 2058 | 1949), 3 % in the forward (65 536: 346 | 361; 262 144, 4 096-token
//     slots: 1209 | 1153), 4 % more where it is long and memory bounds it.  Backward (`busy`): a device with few workgroups runs them a fifth faster, and every round
//     past the first, to the third, costs 6 % more than it alone (states first, 64 x 1 000 0.89 of the estimate, 64 x 4 000 in two rounds 1.07, 64 x 8 000 in four 1.12).
//   - A gathering backward of a few rounds lasts as long as they do, however short the walks (8 x 20 sequences of 59 rows, two rounds, 24; states first 22; parts of
//     slots gather in each, 1 x 100 003 in slots of 4 096, parts of 448, two rounds, 196, of 832, one, 156).  With decay
//     and one walk per document there is nothing to gather: a kernel of its own for that is slower (32 x 4 of 13 rows 27; 13).
//   - Margins: gathering where the estimate errs more (backward 1.05, packed with decay 1.07 (8 heads, 20 000 in 50, slots of 1 024, 176; 163), forward parts of slots
//     1.12), and up to 6 us for parts of short slots that are given states (lasp2_attn_fwd, slots of 512, in halves | whole: 4 x 13 887, 217 workgroups, 23.6 | 21.2; 8 x 3 297, 104, 18.0 | 19.9).
enum class Start {
    states,   // states and prefix kernels first, a walk is `ws` slots
    gather,   // the walks gather them, from or to the document's end; a walk is `ws` slots, or W > 0 tokens
    both      // states and prefix per slot, and walks of W tokens gather from there
};
struct WalkPlan { int ws; int64_t W; Start start; };

Geom regroup(const Geom& g, const int32_t* cu_host, const WalkPlan& p)
{
    return p.W ? regroup_short(g, cu_host, p.W) : regroup(g, cu_host, p.ws);
}

// What walks of W tokens are, per group; walks no longer than a slot don't cross its border
struct WalkCount {
    double walks = 0, longest = 0;       // how many; rows of the longest
    double before = 0, after = 0;        // rows that lie before (from the start of, to the end of the document) each, summed
    double farthest = 0;                 // ... the largest single one of `before`
    double before_in = 0, after_in = 0, farthest_in = 0;   // ... the same, as far as the slot's borders
    double inner = 0, parts = 0;         // rows of slots (walks, if longer) that are not their document's last; how many there are
    double longest_part = 0;
};

// The counts of walks of W, 2 W, 4 W .. tokens (W: some slots), `n` of them: from one to the next a document's full walks halve, so the
// batch is passed through once for all of them (a plan used to pass through it for every candidate and kind of start: 4 000
// documents 468 us of host time, now 21; 40 documents 8.6, now 2.2).
constexpr int kMostDoubled = 32;
void count_whole(const Geom& g, const int32_t* cu_host, int64_t longest, int64_t W, int n, WalkCount* out)
{
    double full[kMostDoubled] = {}, pairs[kMostDoubled] = {}, rows[kMostDoubled] = {};   // full walks; sum of f (f + 1) / 2; of tokens times f
    const int docs = std::max(1, (int)g.n_seqs);
    if (longest > W) {
        for (int k = 0; k < docs; ++k) {
            const int64_t len = g.n_seqs ? cu_host[k + 1] - cu_host[k] : g.N;
            int64_t f = slots_of(len, W) - 1;
            for (int i = 0; f > 0 && i < n; ++i, f >>= 1) {
                full[i] += (double)f;
                pairs[i] += 0.5 * (double)f * (double)(f + 1);
                rows[i] += (double)len * (double)f;
            }
        }
    }
    for (int i = 0; i < n; ++i) {
        WalkCount& c = out[i];
        const double w = (double)W * (double)((int64_t)1 << i);
        c = WalkCount{};
        c.walks = c.parts = full[i] + docs;
        c.longest = c.longest_part = std::min((double)longest, w);
        c.before = w * pairs[i];
        c.after = (double)g.N + rows[i] - c.before;
        c.after_in = g.N;
        c.farthest = w * (double)((slots_of(longest, W) - 1) >> i);
        c.inner = w * full[i];
    }
}

// ... of walks of W tokens inside the slots, which are longer
WalkCount count_inside(const Geom& g, const int32_t* cu_host, int64_t longest, int64_t W)
{
    WalkCount c;
    c.longest = (double)std::min(longest, W);
    c.longest_part = (double)std::min<int64_t>(longest, g.L);
    int64_t short_docs = 0, short_rows = 0;   // documents of one walk
    const double w = (double)W, S = (double)g.L;
    const int64_t in_slot = slots_of(std::min<int64_t>(g.L, INT32_MAX), W);
    const double mf = (double)in_slot, bf = 0.5 * w * mf * (mf - 1.0);
    for (int k = 0; k < std::max(1, (int)g.n_seqs); ++k) {
        const int64_t len = g.n_seqs ? cu_host[k + 1] - cu_host[k] : g.N;
        if (len <= W) {
            ++short_docs;
            short_rows += len;
            continue;
        }
        const int64_t slots = slots_of(len, g.L) - 1, last = len - slots * g.L;
        const double n = (double)len, full = (double)slots, rest = (double)last, mr = (double)slots_of(last, W);
        const double br = 0.5 * w * mr * (mr - 1.0), m = full * mf + mr;
        const double before = 0.5 * full * (full - 1.0) * S * mf + full * bf + full * S * mr + br;
        c.walks += m;
        c.parts += full + 1.0;
        c.before += before;
        c.after += n * m - before;
        c.before_in += full * bf + br;
        c.after_in += full * (S * mf - bf) + rest * mr - br;
        c.farthest = std::max(c.farthest, full * S + (mr - 1.0) * w);
        c.farthest_in = std::max(c.farthest_in, (slots > 0 ? mf - 1.0 : mr - 1.0) * w);
        c.inner += full * S;
    }
    c.walks += (double)short_docs;
    c.parts += (double)short_docs;
    c.after += (double)short_rows;
    c.after_in += (double)short_rows;
    return c;
}

// may_states = false: the states are there already (lasp2_attn_fwd, slots only)
WalkPlan pick_walks(const Geom& g, const int32_t* cu_host, bool backward, bool may_states)
{
    const int64_t longest = longest_sequence(g, cu_host), slots = slots_of(longest, g.L);
    const int wgs = !backward ? 1 : g.decay ? 3 : 2;   // workgroups per walk
    const int ncu = cu_count();
    const double G = g.G, N = g.N, cus = ncu, par = cus / wgs, start = backward ? 180.0 : 256.0;
    const double row = g.decay ? 0.033 : backward ? 0.0376 : 0.03, gather = g.decay ? 0.009 : 0.0068;
    const int part = g.decay ? 256 : 128;   // rows that a walk takes at a time
    const double per_row = g.decay ? 3.0 * row : row + 0.031, ends = g.decay ? 2.0 : 1.0;   // backward: of all workgroups of a walk; that gather `after`
    auto estimate = [&](const WalkCount& c, int64_t W, Start how) {
        const double tensor = G * N * 256.0, states = G * N / (double)g.L * 65536.0;
        const double rate = (backward ? 7.0 : 4.0) * tensor < 2.56e8 ? 8e6 : 5.2e6;
        const double memory = (backward ? 7.0 * tensor : 4.0 * tensor + states) / rate * (!backward && c.walks * G <= par && W > (g.decay ? 4096 : 8192) ? 1.04 : 1.0);
        const double rows_of_one = c.longest < 2048.0 ? std::ceil(c.longest / part) * part : c.longest;
        const double crowded = how != Start::both || 2.0 * tensor < 2.4e7 ? gather : backward ? (g.decay ? 0.012 : 0.0113) : g.decay ? 0.02 : 0.015;
        const double one = (rows_of_one + start) * row, units = c.walks * G * wgs, rounds = std::ceil(units / cus);
        const double busy = g.n_seqs || !backward ? 1.0 : units <= cus ? 0.8 + 0.2 * units / cus
                                                        : 1.0 + (g.decay ? 0.0 : 0.06) * std::min(3.0, rounds - 1.0);
        const double walk = g.n_seqs ? std::max(one, G * (N + start * c.walks) * row / par)
                                     : rounds * one * busy * (rounds > 1.0 ? 1.0 : backward ? 1.08 : 1.03);
        const double tail = 0.05 * walk + (g.n_seqs && rounds > 1.0 ? 0.6 * one : 0.0);
        const double again = 256.0 * row * std::max(0.0, (g.n_seqs ? c.walks * G / par : rounds) - 1.0);   // gathering starts once more
        const double cache = 2.0 * tensor < 2e8 ? 2e7 : 8e6, unsure = !backward ? (W >= g.L ? 1.0 : 1.12) : g.decay && g.n_seqs ? 1.07 : 1.05;
        const double moved = g.n_seqs ? 4.0 * G * 65536.0 / 5.2e6 : 0.0;   // a walk's state: written, combined, read
        const double uneven = g.n_seqs ? 1.33 : 1.0;
        const double chain = g.n_seqs ? 0.0 : 0.1 * std::max(0.0, (double)longest / (double)(how == Start::states ? W : g.L) - 16.0);   // states combined one after another
        if (!backward) {
            const double first = c.inner == 0.0 || !may_states ? 0.0
                                 : 10.0 + std::max(G * c.inner * 512.0 / 6e6 * uneven, c.longest_part * 0.0118) + moved * c.parts + chain;
            if (how == Start::states) return std::max(walk, memory) + tail + first;
            const bool in = how == Start::both;
            const double rows = G * (in ? c.before_in : c.before);
            return unsure * (std::max({walk + again + rows * crowded / par, one + (in ? c.farthest_in : c.farthest) * gather,
                                       memory + rows * 512.0 / cache}) + tail + (!in ? 0.0 : may_states ? first : g.L <= 1024 ? 6.0 * std::min(1.0, units / cus) : 0.0));
        }
        const double first = g.decay && c.inner == 0.0 ? 0.0   // (exclusive suffixes, all zero)
                             : 10.0 + std::max(2.0 * tensor / 6e6 * uneven, std::ceil(c.longest_part / part) * part * 0.0127) + moved * c.parts + chain;
        if (how == Start::states && W <= 128) {   // the kernels for 128 rows, three workgroups per walk
            const double wide = 3.0 * c.walks * G / cus;
            if (c.inner == 0.0) return (g.decay ? 12.0 : 15.0) + std::max(0.0, wide - 1.0) * (7.0 + 0.05 * c.longest) + 2.0 * tensor / 6e6 + moved * c.parts;
            return std::max(18.0, 10.0 + 13.5 * wide * (c.longest + 64.0) / 192.0) + 2.0 * tensor / 6e6 + 0.19 * (double)longest / (double)W +
                   moved * c.parts;
        }
        if (how == Start::states) return std::max(walk, memory) + tail + first;
        const bool in = how == Start::both;
        const double far = in ? std::min((double)longest, (double)g.L) : (double)longest;
        const double rows = G * (ends * (in ? c.after_in : c.after) + (W < g.L ? c.before_in : 0.0));
        const double all = (rows * crowded + G * (N + start * c.walks) * per_row) / cus;
        const double passes = tensor < 2e8 ? 11.0 : 17.0;
        double slowest = 1.5 * far * gather + 1.08 * one * std::min(1.0, busy) + 0.1 * all;
        const double full = std::ceil(units * std::min(1.0, N / (c.walks * c.longest)) / cus);   // rounds of whole walks
        if (!g.n_seqs && full > 1.0 && full <= 4.0)
            slowest = std::max(slowest, g.decay ? full * one : W >= g.L ? full * ((rows_of_one + start) * 0.031 + 3.3)
                                        : far * gather + one + (full - 1.0) * ((rows_of_one + start) * 0.031 + 3.3 + 0.5 * far * crowded));
        return unsure * (std::max({slowest, 1.1 * all, passes * tensor / rate + rows * 512.0 / 1e7}) + 0.15 * all + (in ? first : 0.0));
    };
    const int forced = forced_walk_slots(g);
    const int64_t ws_max = std::min(slots, max_walk_slots(g)), ws_min = std::min(backward ? slots_of(96, g.L) : 128 / g.L + 1, ws_max);
    WalkPlan best = {1, 0, Start::states};
    double cost = -1.0;
    auto take = [&](const WalkPlan& p, const WalkCount& c) {
        const double e = estimate(c, p.W ? p.W : p.ws * g.L, p.start);
        if (cost < 0.0 || e < cost) { cost = e; best = p; }
    };
    const bool lone = slots <= 1;
    auto offer_counted = [&](int64_t ws, const WalkCount& c) {
        if (!backward || lone || forced || ws * g.L >= 256 || 3.0 * c.walks * G <= cus) take({(int)ws, 0, Start::states}, c);
        if (backward ? !(lone && g.decay) : may_states) take({(int)ws, 0, Start::gather}, c);
    };
    auto offer = [&](int64_t ws) {
        WalkCount c;
        count_whole(g, cu_host, longest, ws * g.L, 1, &c);
        offer_counted(ws, c);
    };
    // walks of about W tokens inside the slots
    auto offer_short = [&](int64_t W) {
        W = std::max<int64_t>(256, (W + 63) / 64 * 64);
        if (forced || W >= std::min(g.L, longest)) return;
        const WalkCount c = count_inside(g, cu_host, longest, W);
        if (may_states || lone) take({1, W, Start::gather}, c);
        if (!lone) take({1, W, Start::both}, c);
    };
    if (lone) {
        offer(1);
    } else if (forced) {
        offer(forced);
    } else if (g.n_seqs) {
        WalkCount c[kMostDoubled];
        const int64_t base = std::min((256 + g.L - 1) / g.L, ws_max);
        int n = 0;   // base, 2 base, .. below ws_max, and the shortest
        while (base << n < ws_max) ++n;
        count_whole(g, cu_host, longest, base * g.L, n, c);
        for (int i = 0; i < n; ++i) offer_counted(base << i, c[i]);
        if (ws_min < base) offer(ws_min);
        offer(ws_max);
    }
    if (g.n_seqs) {
        for (int64_t W = (std::min(g.L, longest) + 1) / 2; W >= 256; W /= 2) offer_short(W);
    } else {
        for (int k = 1; k <= 16; ++k) {
            const int64_t m = (int64_t)k * ncu / ((int64_t)wgs * g.G);   // walks per sequence
            if (m < 1) continue;
            const int64_t ws = std::min(ws_max, std::max(ws_min, (slots + m - 1) / m)), W = (g.N + m - 1) / m;
            if (!lone && !forced) {
                offer(ws);
                const int64_t whole = std::min(ws_max, (ws * g.L + part - 1) / part * part / g.L);   // whole rounds of a walk's rows
                if (whole > ws) offer(whole);
            }
            offer_short(W);
            if (m >= 2 * slots) offer_short((std::min<int64_t>(g.L, g.N) + m / slots - 1) / (m / slots));   // as many walks in every slot
            if (ws == ws_min && W <= 256) break;
        }
        if (!lone && !forced && ws_min < ws_max) offer(std::min(2 * ws_min, ws_max));
        if (cost < 0.0) offer(ws_max);
    }
    return best;
}

WalkPlan pick_bwd_walks(const Geom& g, const int32_t* cu_host)
{
    if (g.G == 0) return {1, 0, Start::states};
    return pick_walks(g, cu_host, true, true);
}

// (slots of other lengths: no state of theirs stands between two blocks of a walk)
WalkPlan pick_forward_walks(const Geom& g, const int32_t* cu_host)
{
    if (g.L % 64 == 0) return pick_walks(g, cu_host, false, true);
    return {pick_walk_slots(g, cu_host, cu_count(), kWalkTargetFwd), 0, Start::states};
}

// Walks of 128 rows where lasp2_forward's gather anyway and all of these run at once: the last one then gathers half a walk more and walks
// half as many rows (skew_walk ends after half a chunk there).  Forward, us, walks of 256 | 128: 16 heads x 300 16.5 | 12.5, x 1 024 21.1 | 17.7, x
// 2 048 (256 workgroups) 28.5 | 26.0; 32 x 1 200 (320) 22.7 | 22.9; slots of 64, whose states take longer to write, 16 x 1 500 26.1 | 26.8;
// with decay 8 x 500 20.6 | 16.8, 16 x 1 024 27.7 | 24.3, 16 x 2 048 41.0 | 38.3.  Walks end with their slots, so the launch has its remainders too, and
// these are counted: slots of 192 (there walks of 192) 16 x 1 000 (176) 19.6 | 16.2, 32 x 1 000 (352) 19.8 | 22.3, 16 x 1 920 (320) 27.1 | 25.6; slots
// of 320 16 x 1 280 (240) 25.1 | 18.6, 16 x 2 048 (304) 25.8 | 24.9.
WalkPlan in_halves(const Geom& g, const int32_t* cu_host, const WalkPlan& p)
{
    if (p.start != Start::gather || g.n_seqs || g.L < 128 || g.N <= 128 || forced_walk_slots(g)) return p;
    const WalkPlan half = {1, g.L > 128 ? 128 : 0, Start::gather};
    return (int64_t)g.G * regroup(g, cu_host, half).T_s <= cu_count() ? half : p;   // (walks end with their slots)
}

// Slots per walk of the split-plane kernels, `nprob` workgroups per walk.  They work on chunks of 128
// rows: slots that leave chunks partly empty (one state per 64 tokens, say) are taken two, four or
// eight at a time while that still gives every CU a workgroup, and P is read at the first only.  (d = 32, fp32,
// 64-token slots: forward pass 123 -> 92 us.)  Slots of whole chunks gain nothing and are walked one by one.
// LASP2_WALK_SLOTS overrides the choice where there is one.
int pick_planes_slots(const Geom& g, const int32_t* cu_host, int nprob)
{
    if (g.L % 128 == 0 || g.G == 0 || g.L >= longest_sequence(g, cu_host)) return 1;
    if (const int v = forced_walk_slots(g)) return v;
    int ws = 1;
    while (ws < 8 && g.L * ws < 512 && (g.L * ws) % 128 != 0) {
        const Geom w = regroup(g, cu_host, 2 * ws);
        if (w.T_s == g.T_s || (int64_t)w.G * w.T_s * nprob < cu_count()) break;
        ws *= 2;
    }
    return ws;
}

// The same for heads of 64 in lasp2_forward and the backward, which build the states: one per walk (the walks write the others in
// passing, planes_emit).  A walk starts with the rows of its predecessors read once more and one state each written, combined
// and read, and holds a third of a CU (half in fp32); so about two walks per CU, and not below the length under which states cost
// more than CUs without work.
//   - Layer forward | backward, us, tokens per walk, slots of 64: bf16, 64 x 4001 64 tokens 82 | 140, 128 69 | 120, 256 60 | 110, 512 54 | 103,
//     1024 60 | 104, 2048 84 | 150; 16 x 4000 64 36 | 46, 128 28 | 41, 256 27 | 36, 512 31 | 44; 16 x 2000 128 22 | 26, 256 22 | 28; fp32, 64 x 4001
//     128 134 | 264, 256 124 | 255, 512 119 | 246, 1024 137 | 255; 16 x 4000 64 54 | 78, 128 43 | 73, 256 43 | 72, 512 53 | 85; 4 x 1000 64 19 | 19,
//     128 20 | 21; with decay 16 x 512 64 16 | 17, 128 18 | 21.
//   - Short sequences whole, in one launch without states (in segments that add up the rows before them, where CUs are free),
//     three launches | one, forward and backward: bf16, 16 x 600 16 + 17 | 14 + 15, 40 x 768 19 + 24 | 17 + 22, 8 x 768 14 + 16 | 16 + 16, 16 x 1000
//     17 + 20 | 19 + 22, 128 x 500 24 + 35 | 17 + 32, 256 x 1000 66 + 119 | 43 + 87; with decay 4 x 320 15 + 16 | 13 + 13, 16 x 384 15 + 17 | 15 + 17, 16 x 512
//     16 + 17 | 18 + 21, 100 x 384 30 + 38 | 21 + 37; fp32 4 x 1000 19 + 19 | 37 + 37, 128 x 500 39 + 68 | 33 + 64, 256 x 1000 132 + 262 | 102 + 227.
int pick_planes64_slots(const Geom& g, const int32_t* cu_host, int dtype, bool backward)
{
    const int64_t longest = longest_sequence(g, cu_host);
    if (g.G == 0 || g.L >= longest) return 1;
    if (const int v = forced_walk_slots(g)) return v;
    const bool light = dtype == LASP2_BF16 && !g.decay;
    const int64_t slots = slots_of(longest, g.L), cus = cu_count(), ws_max = std::min(slots, max_walk_slots(g));
    if (g.n_seqs == 0 && longest <= 1024 && slots == ws_max &&
        (g.G >= cus / 2 || longest <= (light ? 768 : dtype == LASP2_BF16 ? 384 : 0)))
        return (int)slots;
    const int64_t tokens = (int64_t)g.G * g.N, least = light ? (tokens >= 160 * cus ? 256 : 128) : tokens >= 64 * cus ? 128 : 64;
    const int64_t target = std::max<int64_t>(least, std::min<int64_t>(1024, tokens / (backward && light ? cus : 2 * cus)));
    int64_t ws = 1;
    while (ws * g.L < target && 2 * ws <= ws_max && !(backward && tokens * 3 < 2 * ws * g.L * cus)) ws *= 2;
    return (int)ws;
}

// What each call does with its descriptor: what they launch by, and what lasp2_walk_slots and lasp2_walk_plan report.
WalkPlan plan_of(const Geom& g, const int32_t* cu_host, int dtype, int call)
{
    const bool backward = call == LASP2_CALL_ATTN_BWD;
    if (!mfma_path_supported(g, dtype)) {
        const bool builds = call != LASP2_CALL_ATTN_FWD;   // (lasp2_attn_fwd is given the states)
        return {g.d == 64 && builds ? pick_planes64_slots(g, cu_host, dtype, backward) : pick_planes_slots(g, cu_host, backward ? 3 : 1), 0, Start::states};
    }
    if (backward) return pick_bwd_walks(g, cu_host);
    if (call == LASP2_CALL_FORWARD) return in_halves(g, cu_host, pick_forward_walks(g, cu_host));
    // long slots that leave CUs without work: walks of parts of them
    if (g.L >= 512) {
        const WalkPlan wp = pick_walks(g, cu_host, false, false);
        if (wp.W) return {1, wp.W, g.lone_slots ? Start::gather : Start::both};
    }
    return {pick_walk_slots(g, cu_host, cu_count(), kWalkTargetFwd), 0, Start::states};
}

int check_ptrs(std::initializer_list<const void*> ptrs)
{
    for (const void* p : ptrs)
        if (!p) return LASP2_ERR_NULL;
    for (const void* p : ptrs)
        if (!aligned16(p)) return LASP2_ERR_ALIGN;
    return LASP2_OK;
}

int from_hip(hipError_t e) { return e == hipSuccess ? LASP2_OK : LASP2_ERR_LAUNCH; }

// Layout of the backward's workspace: the fp32 state array [G][T_s][d][d], then one 32-bit
// counter per (group, slot) through which the workgroups that share a slot's reads keep in
// step (used by the matrix-core kernels only; always part of the size).
size_t states_bytes(const Geom& g) { return (size_t)g.G * (size_t)g.T_s * (size_t)g.d * (size_t)g.d * sizeof(float); }
size_t pace_bytes(const Geom& g) { return (((size_t)g.G * (size_t)g.T_s * sizeof(unsigned)) + 15u) & ~(size_t)15u; }

// anchor_start matters with decay only: states as the slot's first token sees them (backward)
hipError_t run_states(const Geom& g, int dtype, const void* K, const void* V, float* M,
                      int anchor_start, hipStream_t st)
{
    if (mfma_path_supported(g, dtype)) return launch_states_mfma(g, K, V, M, anchor_start, WalkStates::none, st);
    return launch_states_planes(g, dtype, K, V, M, anchor_start, 0, st);
}

// Without a mask a document has one state, whatever its slots: it is summed and applied by walks of several slots, and
// the `nprob` products' launch hands it to the slots inside a walk.  One state per 128 tokens, 8 x 16 x
// 6233, forward 499 -> 265 us, backward 793 -> 441; 40 documents in 8 x 30 000, one per 64, 453 -> 126, 628 -> 178.
// Walks of about 2 048 tokens, fewer while there are not two workgroups per CU; slots of 1 024 and more stay as they are, but
// the products take parts of them where a launch would leave three of four CUs without work (2 x 20 x 1349, 80 of 256: 81 us whole,
// 85 in parts).
Geom nomask_walks(const Geom& g, const int32_t* cu_host, int nprob)
{
    const int64_t longest = longest_sequence(g, cu_host), cus = cu_count();
    const int64_t wanted = std::max<int64_t>(128, std::min<int64_t>(2048, (int64_t)g.G * g.N * nprob / (2 * cus)));
    if (g.L >= 1024) {
        const int64_t part = std::max<int64_t>(256, (wanted + 63) / 64 * 64);
        return (int64_t)g.G * g.T_s * nprob < cus / 4 && part <= g.L / 2 && longest > part ? regroup_short(g, cu_host, part) : g;
    }
    return regroup(g, cu_host, (int)std::max<int64_t>(1, std::min(wanted / g.L, (longest + g.L - 1) / g.L)));
}

// S = sum X^T Y of each document, then the products; gw: as nomask_walks gives them
hipError_t run_nomask(const Geom& g, const Geom& gw, const void* X, const void* Y, float* S, const RowsStateProblem* p, int n, hipStream_t st)
{
    const Geom& gs = gw.W ? g : gw;
    hipError_t e = launch_states_mfma(gs, X, Y, S, 0, gs.wslots > 1 ? WalkStates::all : WalkStates::none, st);
    if (e != hipSuccess) return e;
    e = launch_state_total(gs, S, S, st);
    if (e != hipSuccess) return e;
    return launch_rows_state_mfma(gw, p, n, st);
}

// What lasp2_attn_bwd and lasp2_attn_bwd_noalloc have in common: the checks that need no
// workspace, and the launches.
struct BwdPlan {
    Geom g;             // the caller's slots (argument checks, workspace size)
    Geom gw;            // the walks of the kernels (= g unless the matrix-core kernels take several slots per walk)
    bool empty;
    bool fast;          // matrix-core kernels
    bool inclusive;     // suffix states in the inclusive form
    bool lone;          // every document a single slot
    bool need_states;   // dM_t go through a state array of `need` bytes
    size_t need;
    bool lone_w;        // every document a single walk
    bool need_states_w; // (matrix-core kernels)
    Start start;        // what the walks start from (matrix-core kernels)
};

// `workspace`: address of the caller's workspace pointer, or NULL for an entry point that has none.
int plan_attn_bwd(const lasp2_desc_t* desc, const void* Q, const void* K, const void* V, const void* dO,
                  const float* P, void* dQ, void* dK, void* dV, void* const* workspace, BwdPlan* pl)
{
    pl->empty = false;
    int rc = make_geom(desc, &pl->g, &pl->empty);
    if (rc != LASP2_OK || pl->empty) return rc;
    const Geom& g = pl->g;
    pl->fast = mfma_path_supported(g, desc->dtype);
    // Which suffix states the kernels want: the split-plane kernels and the MFMA kernels with decay walk
    // each slot backwards from the EXCLUSIVE suffix; the MFMA kernels without decay walk forwards
    // from the INCLUSIVE suffix and subtract (see attn_mfma_kernel), which lets the three
    // problems of a slot share their reads.
    pl->inclusive = pl->fast && !g.decay;
    // Every document a single slot (serial-carry schedule): all exclusive prefixes and suffixes are
    // zero.  P is then not read (and may be NULL), kernels that start from the exclusive suffix need
    // neither states nor workspace, and the inclusive suffix of a lone slot is its own state, so
    // the combine is skipped.
    pl->lone = g.lone_slots != 0;
    pl->need_states = !pl->lone || pl->inclusive;
    pl->need = states_bytes(g) + pace_bytes(g);
    const bool ws = workspace && pl->need_states;
    if ((!pl->lone && !P) || (ws && !*workspace)) return LASP2_ERR_NULL;   // NULL before alignment, as everywhere
    rc = check_ptrs({Q, K, V, dO, dQ, dK, dV});
    if (rc != LASP2_OK) return rc;
    if ((!pl->lone && !aligned16(P)) || (ws && !aligned16(*workspace))) return LASP2_ERR_ALIGN;
    // The kernels' own walks.  The matrix-core kernels' dM states are built per walk, not per slot of the caller: fewer
    // of them, never more bytes than `need`.
    pl->gw = g;
    pl->start = Start::states;
    const int32_t* cu = desc->cu_seqlens_host;
    const WalkPlan wp = plan_of(g, cu, desc->dtype, LASP2_CALL_ATTN_BWD);
    pl->gw = regroup(g, cu, wp);
    pl->start = wp.start;
    pl->lone_w = pl->gw.lone_slots != 0;
    pl->need_states_w = !pl->lone_w || pl->inclusive;
    return LASP2_OK;
}

// Split planes.  dR holds the exclusive suffix of every slot of the caller's afterwards, however long the walks are.  Where the walks
// write the entries of the slots inside them, the launches before make those at the walks' ends only.
// (P: a walk's first state is taken as it is given, zero or not.)
int run_attn_bwd_planes(const BwdPlan& pl, int dtype, const void* Q, const void* K, const void* V, const void* dO, const float* P,
                        void* dQ, void* dK, void* dV, float* dR, hipStream_t st)
{
    const bool emit = dR && planes_emit(pl.gw);
    const Geom& g = emit ? pl.gw : pl.g;
    if (dR && !(emit && pl.lone_w)) {
        if (launch_states_planes(g, dtype, Q, dO, dR, 1, emit ? 1 : 0, st) != hipSuccess) return LASP2_ERR_LAUNCH;
        if (launch_state_prefix(g, dR, dR, 1, 0, emit ? 1 : 0, nullptr, 0, st) != hipSuccess) return LASP2_ERR_LAUNCH;
    }
    return from_hip(launch_attn_bwd_planes(pl.gw, dtype, Q, K, V, dO, P, emit && pl.lone_w ? nullptr : dR, emit ? dR : nullptr, dQ, dK, dV, st));
}

int run_attn_bwd(const BwdPlan& pl, int dtype, const void* Q, const void* K, const void* V, const void* dO,
                 const float* P, void* dQ, void* dK, void* dV, float* dR, hipStream_t st)
{
    const Geom& g = pl.gw;
    if (!pl.fast) return run_attn_bwd_planes(pl, dtype, Q, K, V, dO, pl.lone ? nullptr : P, dQ, dK, dV, dR, st);
    if (pl.lone_w) P = nullptr;
    hipError_t e = hipSuccess;
    if (pl.start == Start::gather) return from_hip(launch_attn_bwd_direct_mfma(g, Q, K, V, dO, P, dR, 0, dQ, dK, dV, st));
    if (pl.start == Start::both) {   // suffix states per slot
        if (run_states(pl.g, dtype, Q, dO, dR, 1, st) != hipSuccess) return LASP2_ERR_LAUNCH;
        if (launch_state_prefix(pl.g, dR, dR, 1, pl.inclusive ? 1 : 0, 0, nullptr, 0, st) != hipSuccess) return LASP2_ERR_LAUNCH;
        return from_hip(launch_attn_bwd_direct_mfma(g, Q, K, V, dO, P, dR, 1, dQ, dK, dV, st));
    }
    unsigned* pace = dR ? reinterpret_cast<unsigned*>(reinterpret_cast<char*>(dR) + states_bytes(g)) : nullptr;
    const bool clear = pl.inclusive && !pl.lone_w && pace;   // (the prefix launch clears the counters in passing)
    if (pl.need_states_w) {
        // dM_t = Q_t^T dO_t per walk, then its suffix combine in place
        e = run_states(g, dtype, Q, dO, dR, 1, st);
        if (e != hipSuccess) return LASP2_ERR_LAUNCH;
    }
    if (!pl.lone_w) {
        e = launch_state_prefix(g, dR, dR, 1, pl.inclusive ? 1 : 0, 0, clear ? pace : nullptr, (unsigned)(g.T_s * g.G), st);
        if (e != hipSuccess) return LASP2_ERR_LAUNCH;
    }
    return from_hip(launch_attn_bwd_mfma(g, Q, K, V, dO, P, pl.need_states_w ? dR : nullptr, pace, clear ? 0 : 1, dQ, dK, dV, st));
}

// Scratch of lasp2_attn_bwd_noalloc: device memory that belongs to the loaded library itself, one
// copy per GPU, held until the process ends.  In host code `scratch` is only a handle for the
// symbol, not a device address: the address is asked for once per device, with that device
// current, and kept; kernels and launchers only ever see that address.
static __device__ __align__(256) unsigned char scratch[LASP2_NOALLOC_SCRATCH_BYTES];

void* scratch_on_current_device()
{
    static std::atomic<void*> addr[kMaxDevices] = {};
    const int dev = current_device_index();
    if (dev < 0) return nullptr;
    void* p = addr[dev].load(std::memory_order_acquire);
    if (p) return p;
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) return nullptr;
    addr[dev].store(p, std::memory_order_release);   // the same value from whichever thread asks first
    return p;
}

}  // namespace
}  // namespace lasp2

using namespace lasp2;

extern "C" {

int lasp2_num_slots(const lasp2_desc_t* desc, int64_t* T_s)
{
    if (!T_s) return LASP2_ERR_NULL;
    Geom g;
    bool empty = false;
    int rc = make_geom(desc, &g, &empty);
    if (rc != LASP2_OK) return rc;
    *T_s = g.T_s;
    return LASP2_OK;
}

int lasp2_walk_slots(const lasp2_desc_t* desc, int backward, int64_t* slots_per_walk)
{
    if (!slots_per_walk) return LASP2_ERR_NULL;
    Geom g;
    bool empty = false;
    int rc = make_geom(desc, &g, &empty);
    if (rc != LASP2_OK) return rc;
    *slots_per_walk = empty ? 1 : plan_of(g, desc->cu_seqlens_host, desc->dtype, backward ? LASP2_CALL_ATTN_BWD : LASP2_CALL_ATTN_FWD).ws;
    return LASP2_OK;
}

int lasp2_walk_plan(const lasp2_desc_t* desc, int call, int64_t* walk_tokens, int* start)
{
    if (!walk_tokens || !start) return LASP2_ERR_NULL;
    Geom g;
    bool empty = false;
    int rc = make_geom(desc, &g, &empty);
    if (rc != LASP2_OK) return rc;
    if (call < LASP2_CALL_ATTN_FWD || call > LASP2_CALL_FORWARD) return LASP2_ERR_SHAPE;
    const WalkPlan wp = empty ? WalkPlan{1, 0, Start::states} : plan_of(g, desc->cu_seqlens_host, desc->dtype, call);
    *walk_tokens = wp.W ? wp.W : wp.ws * g.L;
    *start = wp.start == Start::gather ? LASP2_START_GATHER : wp.start == Start::both ? LASP2_START_SLOTS : LASP2_START_STATES;
    return LASP2_OK;
}

int lasp2_workspace_size(const lasp2_desc_t* desc, size_t* bytes)
{
    if (!bytes) return LASP2_ERR_NULL;
    Geom g;
    bool empty = false;
    int rc = make_geom(desc, &g, &empty);
    if (rc != LASP2_OK) return rc;
    *bytes = states_bytes(g) + pace_bytes(g);
    return LASP2_OK;
}

int lasp2_chunk_states(const lasp2_desc_t* desc, const void* K, const void* V, float* M,
                       void* stream)
{
    Geom g;
    bool empty = false;
    int rc = make_geom(desc, &g, &empty);
    if (rc != LASP2_OK) return rc;
    if (empty) return LASP2_OK;
    rc = check_ptrs({K, V, M});
    if (rc != LASP2_OK) return rc;
    return from_hip(run_states(g, desc->dtype, K, V, M, 0, (hipStream_t)stream));
}

int lasp2_state_prefix(const lasp2_desc_t* desc, const float* M, float* P, int reverse,
                       void* stream)
{
    Geom g;
    bool empty = false;
    int rc = make_geom(desc, &g, &empty);
    if (rc != LASP2_OK) return rc;
    if (empty) return LASP2_OK;
    rc = check_ptrs({M, P});
    if (rc != LASP2_OK) return rc;
    return from_hip(launch_state_prefix(g, M, P, reverse ? 1 : 0, 0, 0, nullptr, 0, (hipStream_t)stream));
}

int lasp2_attn_fwd(const lasp2_desc_t* desc, const void* Q, const void* K, const void* V,
                   const float* P, void* O, void* stream)
{
    Geom g;
    bool empty = false;
    int rc = make_geom(desc, &g, &empty);
    if (rc != LASP2_OK) return rc;
    if (empty) return LASP2_OK;
    // Serial-carry schedule: when every document is one slot, each slot starts from a zero state
    // and P may be left out (NULL); the states and prefix calls are then not needed at all.
    rc = (P == nullptr && g.lone_slots) ? check_ptrs({Q, K, V, O}) : check_ptrs({Q, K, V, P, O});
    if (rc != LASP2_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    const WalkPlan wp = plan_of(g, desc->cu_seqlens_host, desc->dtype, LASP2_CALL_ATTN_FWD);
    const Geom gw = regroup(g, desc->cu_seqlens_host, wp);
    if (wp.W) return from_hip(launch_attn_fwd_direct_mfma(gw, Q, K, V, g.lone_slots ? nullptr : P, nullptr, O, st));
    if (mfma_path_supported(g, desc->dtype))
        return from_hip(launch_attn_fwd_mfma(gw, Q, K, V, gw.lone_slots ? nullptr : P, O, st));
    return from_hip(launch_attn_fwd_planes(gw, desc->dtype, Q, K, V, P, nullptr, O, st));
}

int lasp2_forward(const lasp2_desc_t* desc, const void* Q, const void* K, const void* V,
                  float* P, void* O, void* stream)
{
    Geom g;
    bool empty = false;
    int rc = make_geom(desc, &g, &empty);
    if (rc != LASP2_OK) return rc;
    if (empty) return LASP2_OK;
    rc = check_ptrs({Q, K, V, P, O});
    if (rc != LASP2_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    const int32_t* cu = desc->cu_seqlens_host;
    const bool fast = mfma_path_supported(g, desc->dtype);
    const WalkPlan wp = plan_of(g, cu, desc->dtype, LASP2_CALL_FORWARD);
    const Geom gw = regroup(g, cu, wp);
    hipError_t e;
    if (wp.start == Start::gather) return from_hip(launch_attn_fwd_direct_mfma(gw, Q, K, V, nullptr, P, O, st));
    if (walk_emits(gw, desc->dtype)) {
        // The attention walks write the states of the slots inside them, so states and prefix are
        // needed where a walk starts only, and not at all where every document is one walk.
        if (!gw.lone_slots) {
            e = launch_states_mfma(gw, K, V, P, 0, WalkStates::before_last, st);
            if (e != hipSuccess) return LASP2_ERR_LAUNCH;
            e = launch_state_prefix(gw, P, P, 0, 0, 1, nullptr, 0, st);
            if (e != hipSuccess) return LASP2_ERR_LAUNCH;
        }
        return from_hip(launch_attn_fwd_emit_mfma(gw, Q, K, V, P, O, st));
    }
    if (!fast && planes_emit(gw)) {   // likewise
        if (!gw.lone_slots) {
            e = launch_states_planes(gw, desc->dtype, K, V, P, 0, 1, st);
            if (e != hipSuccess) return LASP2_ERR_LAUNCH;
            e = launch_state_prefix(gw, P, P, 0, 0, 1, nullptr, 0, st);
            if (e != hipSuccess) return LASP2_ERR_LAUNCH;
        }
        return from_hip(launch_attn_fwd_planes(gw, desc->dtype, Q, K, V, gw.lone_slots ? nullptr : P, P, O, st));
    }
    e = run_states(g, desc->dtype, K, V, P, 0, st);
    if (e != hipSuccess) return LASP2_ERR_LAUNCH;
    e = launch_state_prefix(g, P, P, 0, 0, 0, nullptr, 0, st);
    if (e != hipSuccess) return LASP2_ERR_LAUNCH;
    if (wp.start == Start::both) return from_hip(launch_attn_fwd_direct_mfma(gw, Q, K, V, P, nullptr, O, st));
    if (fast) return from_hip(launch_attn_fwd_mfma(gw, Q, K, V, gw.lone_slots ? nullptr : P, O, st));
    return from_hip(launch_attn_fwd_planes(gw, desc->dtype, Q, K, V, gw.lone_slots ? nullptr : P, nullptr, O, st));
}

int lasp2_attn_bwd(const lasp2_desc_t* desc, const void* Q, const void* K, const void* V,
                   const void* dO, const float* P, void* dQ, void* dK, void* dV,
                   void* workspace, size_t workspace_bytes, void* stream)
{
    BwdPlan pl;
    int rc = plan_attn_bwd(desc, Q, K, V, dO, P, dQ, dK, dV, &workspace, &pl);
    if (rc != LASP2_OK) return rc;
    if (pl.empty) return LASP2_OK;
    if (pl.need_states && workspace_bytes < pl.need) return LASP2_ERR_WORKSPACE;
    return run_attn_bwd(pl, desc->dtype, Q, K, V, dO, P, dQ, dK, dV,
                        pl.need_states ? static_cast<float*>(workspace) : nullptr, (hipStream_t)stream);
}

int lasp2_attn_bwd_noalloc(const lasp2_desc_t* desc, const void* Q, const void* K, const void* V,
                           const void* dO, const float* P, void* dQ, void* dK, void* dV, void* stream)
{
    BwdPlan pl;
    int rc = plan_attn_bwd(desc, Q, K, V, dO, P, dQ, dK, dV, nullptr, &pl);
    if (rc != LASP2_OK) return rc;
    if (pl.empty) return LASP2_OK;
    float* dR = nullptr;
    if (pl.need_states) {
        if (pl.need > (size_t)LASP2_NOALLOC_SCRATCH_BYTES) return LASP2_ERR_WORKSPACE;
        dR = static_cast<float*>(scratch_on_current_device());
        if (!dR) return LASP2_ERR_LAUNCH;
    }
    // Nothing in the array has to start at zero: the states kernel writes every slot's state
    // before the combine and the attention kernels read any of it.
    return run_attn_bwd(pl, desc->dtype, Q, K, V, dO, P, dQ, dK, dV, dR, (hipStream_t)stream);
}

int lasp2_state_total(const lasp2_desc_t* desc, const float* M, float* S, void* stream)
{
    Geom g;
    bool empty = false;
    int rc = make_geom(desc, &g, &empty);
    if (rc != LASP2_OK) return rc;
    if (g.decay) return LASP2_ERR_DECAY;   // decay is defined for the masked path only
    if (empty) return LASP2_OK;
    rc = check_ptrs({M, S});
    if (rc != LASP2_OK) return rc;
    return from_hip(launch_state_total(g, M, S, (hipStream_t)stream));
}

int lasp2_nomask_fwd(const lasp2_desc_t* desc, const void* Q, const float* S, void* O, void* stream)
{
    Geom g;
    bool empty = false;
    int rc = make_geom(desc, &g, &empty);
    if (rc != LASP2_OK) return rc;
    if (g.decay) return LASP2_ERR_DECAY;   // decay is defined for the masked path only
    if (empty) return LASP2_OK;
    rc = check_ptrs({Q, S, O});
    if (rc != LASP2_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    if (mfma_path_supported(g, desc->dtype)) {
        const RowsStateProblem p = {Q, S, O, 0, nullptr};
        return from_hip(launch_rows_state_mfma(nomask_walks(g, desc->cu_seqlens_host, 1), &p, 1, st));
    }
    return from_hip(launch_rows_state_generic(g, desc->dtype, Q, S, O, 0, st));
}

int lasp2_nomask_forward(const lasp2_desc_t* desc, const void* Q, const void* K, const void* V,
                         float* S, void* O, void* stream)
{
    Geom g;
    bool empty = false;
    int rc = make_geom(desc, &g, &empty);
    if (rc != LASP2_OK) return rc;
    if (g.decay) return LASP2_ERR_DECAY;   // decay is defined for the masked path only
    if (empty) return LASP2_OK;
    rc = check_ptrs({Q, K, V, S, O});
    if (rc != LASP2_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    if (mfma_path_supported(g, desc->dtype)) {
        const Geom gw = nomask_walks(g, desc->cu_seqlens_host, 1);
        const RowsStateProblem p = {Q, S, O, 0, S};
        return from_hip(run_nomask(g, gw, K, V, S, &p, 1, st));
    }
    hipError_t e = launch_states_planes(g, desc->dtype, K, V, S, 0, 0, st);
    if (e != hipSuccess) return LASP2_ERR_LAUNCH;
    e = launch_state_total(g, S, S, st);
    if (e != hipSuccess) return LASP2_ERR_LAUNCH;
    return from_hip(launch_rows_state_generic(g, desc->dtype, Q, S, O, 0, st));
}

int lasp2_nomask_bwd(const lasp2_desc_t* desc, const void* Q, const void* K, const void* V,
                     const void* dO, const float* S, void* dQ, void* dK, void* dV,
                     void* workspace, size_t workspace_bytes, void* stream)
{
    Geom g;
    bool empty = false;
    int rc = make_geom(desc, &g, &empty);
    if (rc != LASP2_OK) return rc;
    if (g.decay) return LASP2_ERR_DECAY;   // decay is defined for the masked path only
    if (empty) return LASP2_OK;
    rc = check_ptrs({Q, K, V, dO, S, dQ, dK, dV, workspace});
    if (rc != LASP2_OK) return rc;
    if (workspace_bytes < states_bytes(g) + pace_bytes(g)) return LASP2_ERR_WORKSPACE;   // one size for both backward calls

    hipStream_t st = (hipStream_t)stream;
    float* dS = static_cast<float*>(workspace);
    // dM_t = Q_t^T dO_t, then the sum over the document's slots in place
    if (mfma_path_supported(g, desc->dtype)) {
        const RowsStateProblem p[3] = {{dO, S, dQ, 1, nullptr}, {V, dS, dK, 1, dS}, {K, dS, dV, 0, nullptr}};
        return from_hip(run_nomask(g, nomask_walks(g, desc->cu_seqlens_host, 3), Q, dO, dS, p, 3, st));
    }
    hipError_t e = launch_states_planes(g, desc->dtype, Q, dO, dS, 0, 0, st);
    if (e != hipSuccess) return LASP2_ERR_LAUNCH;
    e = launch_state_total(g, dS, dS, st);
    if (e != hipSuccess) return LASP2_ERR_LAUNCH;
    e = launch_rows_state_generic(g, desc->dtype, dO, S, dQ, 1, st);    // dQ = dO M^T
    if (e != hipSuccess) return LASP2_ERR_LAUNCH;
    e = launch_rows_state_generic(g, desc->dtype, V, dS, dK, 1, st);    // dK = V dM^T
    if (e != hipSuccess) return LASP2_ERR_LAUNCH;
    return from_hip(launch_rows_state_generic(g, desc->dtype, K, dS, dV, 0, st));   // dV = K dM
}

// Softmax attention for the queries [q_begin, q_begin + q_len) of the sequence; the entry points
// without a range are the whole sequence.
static int softmax_geom(const lasp2_desc_t* desc, int64_t q_begin, int64_t q_len, Geom* g, bool* empty)
{
    int rc = make_geom(desc, g, empty);
    if (rc != LASP2_OK) return rc;
    if (g->decay) return LASP2_ERR_DECAY;   // decay belongs to the linear layers
    if (q_begin < 0 || q_len < 0 || q_begin + q_len > (int64_t)g->N) return LASP2_ERR_SHAPE;
    g->q0 = (int32_t)q_begin;
    g->qn = (int32_t)q_len;
    return LASP2_OK;
}

// Launches of at most one workgroup of 64 rows (forward: or 128) per CU: 256 queries (128 keys) a workgroup would leave most CUs idle
// while the longest row sets the time.  With more of them the small kernels' traffic costs more than the idle CUs.  bf16 x
// 128, 256-row kernels | 64 rows, 128 rows, us: 16 heads x 1 000 causal, forward 37 | 20, 25, backward 82 | 53; 4 x 4 000 112 | 54, 74,
// 260 | 139; 16 heads, the last 1 000 of 16 000 438 | 231, 357; 32 x 1 000 (512 and 256 of them) 36 | 33, 26, 84 | 92; and beyond
// the lines 20 x 1 692 (540, 280) 57 | 67, 61, 132 | 170; 16 x 4 000 124 | 163, 134, 315 | 410.
// `partners`: the rows that the call's rows can see (keys of its queries, queries of its keys).  A few of them are one or two steps of either
// kernel, and merging the shares costs more than splitting them gains: 16 heads causal, forward | backward, 64 rows 6.0 -> 8.3 | 17.3 -> 23.7,
// 128 8.1 -> 8.5 | 22.5 -> 24.4, 160 9.4 -> 9.6 | 26.6 -> 27.2, 192 10.4 -> 9.6 | 27.2 -> 27.6, 200 11.4 -> 9.6 | 31.4 -> 27.7.
constexpr int64_t kFewKeysFwd = 160, kFewPartnersBwd = 192;
static bool softmax_rows_fit(const Geom& g, int rows, int per, int64_t partners, int64_t few)
{
    return partners > few && (int64_t)g.G * ((rows + per - 1) / per) <= cu_count();
}
static int64_t softmax_keys(const Geom& g, int causal) { return causal ? (int64_t)g.q0 + g.qn : g.N; }

static int softmax_fwd_impl(const lasp2_desc_t* desc, int64_t q_begin, int64_t q_len, const void* Q,
                            const void* K, const void* V, void* O, float* LSE, int causal, void* stream)
{
    Geom g;
    bool empty = false;
    int rc = softmax_geom(desc, q_begin, q_len, &g, &empty);
    if (rc != LASP2_OK) return rc;
    if (empty || g.qn == 0) return LASP2_OK;
    rc = check_ptrs({Q, K, V, O, LSE});
    if (rc != LASP2_OK) return rc;
    hipStream_t st = (hipStream_t)stream;
    const int64_t keys = softmax_keys(g, causal);
    const int small = softmax_rows_fit(g, g.qn, 64, keys, kFewKeysFwd) ? 2 : softmax_rows_fit(g, g.qn, 128, keys, kFewKeysFwd) ? 4 : 0;   // row tiles per workgroup
    if (softmax_mfma_supported(g, desc->dtype))
        return from_hip(small ? launch_softmax_fwd_small(g, small, Q, K, V, O, LSE, causal ? 1 : 0, st)
                                               : launch_softmax_fwd_mfma(g, Q, K, V, O, LSE, causal ? 1 : 0, st));
    return from_hip(launch_softmax_fwd_planes(g, desc->dtype, Q, K, V, O, LSE, causal ? 1 : 0, st));
}

static int softmax_bwd_impl(const lasp2_desc_t* desc, int64_t q_begin, int64_t q_len, const void* Q,
                            const void* K, const void* V, const void* O, const void* dO, const float* LSE,
                            void* dQ, void* dK, void* dV, void* workspace, size_t workspace_bytes,
                            int causal, void* stream)
{
    Geom g;
    bool empty = false;
    int rc = softmax_geom(desc, q_begin, q_len, &g, &empty);
    if (rc != LASP2_OK) return rc;
    if (empty) return LASP2_OK;
    // with no queries dK and dV are still written (zeros); the query-side arrays are not touched
    rc = g.qn == 0 ? check_ptrs({K, V, dK, dV}) : check_ptrs({Q, K, V, O, dO, LSE, dQ, dK, dV, workspace});
    if (rc != LASP2_OK) return rc;
    const size_t rows = (size_t)g.G * (size_t)g.qn;
    if (workspace_bytes < 2 * rows * sizeof(float)) return LASP2_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    float* delta = static_cast<float*>(workspace);
    float* lse2 = delta + rows;
    const bool fast = softmax_mfma_supported(g, desc->dtype);
    hipError_t e = launch_softmax_delta(g, desc->dtype, O, dO, LSE, delta, fast ? lse2 : nullptr, st);
    if (e != hipSuccess) return LASP2_ERR_LAUNCH;
    if (fast) {
        e = softmax_rows_fit(g, g.qn, 64, softmax_keys(g, causal), kFewPartnersBwd)
                ? launch_softmax_bwd_dq_small(g, Q, K, V, dO, LSE, delta, dQ, causal ? 1 : 0, st)
                : launch_softmax_bwd_dq_mfma(g, Q, K, V, dO, LSE, delta, dQ, causal ? 1 : 0, st);
        if (e != hipSuccess) return LASP2_ERR_LAUNCH;
        return from_hip(softmax_rows_fit(g, g.N, 64, g.qn, kFewPartnersBwd)
                            ? launch_softmax_bwd_dkv_small(g, Q, K, V, dO, lse2, delta, dK, dV, causal ? 1 : 0, st)
                            : launch_softmax_bwd_dkv_mfma(g, Q, K, V, dO, lse2, delta, dK, dV, causal ? 1 : 0, st));
    }
    return from_hip(launch_softmax_bwd_planes(g, desc->dtype, Q, K, V, dO, LSE, delta, dQ, dK, dV,
                                              causal ? 1 : 0, st));
}

int lasp2_softmax_fwd(const lasp2_desc_t* desc, const void* Q, const void* K, const void* V,
                      void* O, float* LSE, int causal, void* stream)
{
    return softmax_fwd_impl(desc, 0, desc ? desc->N : 0, Q, K, V, O, LSE, causal, stream);
}

int lasp2_softmax_workspace_size(const lasp2_desc_t* desc, size_t* bytes)
{
    return lasp2_softmax_share_workspace_size(desc, desc ? desc->N : 0, bytes);
}

int lasp2_softmax_bwd(const lasp2_desc_t* desc, const void* Q, const void* K, const void* V,
                      const void* O, const void* dO, const float* LSE, void* dQ, void* dK, void* dV,
                      void* workspace, size_t workspace_bytes, int causal, void* stream)
{
    return softmax_bwd_impl(desc, 0, desc ? desc->N : 0, Q, K, V, O, dO, LSE, dQ, dK, dV, workspace,
                            workspace_bytes, causal, stream);
}

int lasp2_softmax_fwd_share(const lasp2_desc_t* desc, int64_t q_begin, int64_t q_len, const void* Q_t,
                            const void* K, const void* V, void* O_t, float* LSE_t, int causal, void* stream)
{
    return softmax_fwd_impl(desc, q_begin, q_len, Q_t, K, V, O_t, LSE_t, causal, stream);
}

int lasp2_softmax_share_workspace_size(const lasp2_desc_t* desc, int64_t q_len, size_t* bytes)
{
    if (!bytes) return LASP2_ERR_NULL;
    Geom g;
    bool empty = false;
    int rc = softmax_geom(desc, 0, q_len, &g, &empty);
    if (rc != LASP2_OK) return rc;
    *bytes = 2 * (size_t)g.G * (size_t)g.qn * sizeof(float);   // delta, and the log-sum-exp in base 2
    return LASP2_OK;
}

int lasp2_softmax_bwd_share(const lasp2_desc_t* desc, int64_t q_begin, int64_t q_len, const void* Q_t,
                            const void* K, const void* V, const void* O_t, const void* dO_t,
                            const float* LSE_t, void* dQ_t, void* dK, void* dV, void* workspace,
                            size_t workspace_bytes, int causal, void* stream)
{
    return softmax_bwd_impl(desc, q_begin, q_len, Q_t, K, V, O_t, dO_t, LSE_t, dQ_t, dK, dV, workspace,
                            workspace_bytes, causal, stream);
}

const char* lasp2_status_string(int status)
{
    switch (status) {
        case LASP2_OK: return "ok";
        case LASP2_ERR_NULL: return "a required pointer is NULL";
        case LASP2_ERR_SHAPE: return "unsupported or inconsistent shape (B,H,N,d,C,L)";
        case LASP2_ERR_DTYPE: return "unsupported dtype";
        case LASP2_ERR_SEQLENS: return "invalid packed-sequence offsets";
        case LASP2_ERR_WORKSPACE: return "workspace too small";
        case LASP2_ERR_ALIGN: return "device pointer not 16-byte aligned";
        case LASP2_ERR_LAUNCH: return "HIP launch failed";
        case LASP2_ERR_DECAY: return "invalid decay factors, or decay given to an entry point without masking";
        default: return "unknown status";
    }
}

}  // extern "C"

// C ABI entry points: argument validation, tile choice, variant dispatch, launch.
#include <hip/hip_runtime_api.h>
#include <math.h>
#include <stdio.h>
#include <string.h>

#include "mcf_geometry.h"
#include "mcf_internal.h"

namespace mcf {

static thread_local char g_last_error[256] = "";
void set_last_error(const char *msg) { snprintf(g_last_error, sizeof(g_last_error), "%s", msg ? msg : ""); }

static bool all_zero(const int64_t s[3]) { return s[0] == 0 && s[1] == 0 && s[2] == 0; }

static void packed(int64_t out[3], int64_t rows, int64_t cols) {
    out[0] = rows * cols; out[1] = cols; out[2] = 1;
}

// An output [batch, rows, cols] (col stride 1): a batch must end before the next one starts.
static bool batches_disjoint(int64_t batch, int64_t rows, int64_t cols, const int64_t s[3]) {
    if (batch <= 1 || rows <= 0 || cols <= 0) return true;
    if (s[1] > (1ll << 40) || rows > (1ll << 31)) return false; // keeps the product below in range
    return s[0] >= (rows - 1) * s[1] + cols;
}

// Whether 1 + (batch-1) s0 + (rows-1) s1 + (cols-1) s2 stays below 2^60 elements.
static bool span_fits(int64_t batch, int64_t rows, int64_t cols, const int64_t s[3]) {
    const int64_t n[3] = {batch, rows, cols};
    __int128 total = 1;
    for (int d = 0; d < 3; ++d)
        if (n[d] > 1) total += (__int128)(n[d] - 1) * s[d];
    return total < ((__int128)1 << 60);
}

int decode_layout(const mcf_problem *p, Layout *o) {
    if (p->in_dtype != MCF_F16 && p->in_dtype != MCF_BF16) return MCF_EUNSUPPORTED;
    if (p->out_dtype != p->in_dtype && p->out_dtype != MCF_F32) return MCF_EUNSUPPORTED;
    if (p->K > 65536 || p->L > 4096 || !resolve_group(p->in_dtype, p->K, p->L)) return MCF_EUNSUPPORTED;
    if (p->M >= (1ll << 31) - 512 || p->N >= (1ll << 31) - 512 || p->batch >= (1ll << 31)) return MCF_EUNSUPPORTED;
    const int64_t *in[4] = {p->a_stride, p->b_stride, p->d_stride, p->e_stride};
    int64_t *out[4] = {o->sa, o->sb, o->sd, o->se};
    const int64_t rows[4] = {p->M, p->K, p->N, p->M}, cols[4] = {p->K, p->N, p->L, p->L};
    for (int t = 0; t < 4; ++t) {
        if (all_zero(in[t])) packed(out[t], rows[t], cols[t]);
        else memcpy(out[t], in[t], 3 * sizeof(int64_t));
        for (int d = 0; d < 3; ++d)
            if (out[t][d] < 0) return MCF_EINVAL;
    }
    // contiguous index of each tensor
    if (o->sa[2] != 1 || o->sd[2] != 1 || o->se[2] != 1) return MCF_EUNSUPPORTED;
    // B: N contiguous (col stride 1) or K contiguous (row stride 1); N-contiguous wins a tie
    // unless only the K-contiguous kernels can take this N.
    if (o->sb[2] == 1 && !(o->sb[1] == 1 && p->N % 8 != 0)) o->b_kcontig = 0;
    else if (o->sb[1] == 1) o->b_kcontig = 1;
    else return MCF_EUNSUPPORTED;
    // rows must not overlap themselves
    if (p->M > 1 && o->sa[1] < p->K) return MCF_EINVAL;
    if (p->N > 1 && o->sd[1] < p->L) return MCF_EINVAL;
    if (p->M > 1 && o->se[1] < p->L) return MCF_EINVAL;
    if (o->b_kcontig ? (p->N > 1 && o->sb[2] < p->K) : (p->K > 1 && o->sb[1] < p->N)) return MCF_EINVAL;
    // Batches of the output must not overlap one another: blocks of different batches would
    // store to the same rows.  (The inputs are only read: a zero or overlapping batch stride
    // is a legal broadcast there.)
    if (!batches_disjoint(p->batch, p->M, p->L, o->se)) return MCF_EINVAL;
    // and every tensor's extent in elements must fit 64-bit arithmetic with room to spare
    for (int t = 0; t < 4; ++t)
        if (!span_fits(p->batch, rows[t], cols[t], out[t])) return MCF_EUNSUPPORTED;
    // 16-byte vector accesses: leading strides and batch strides in multiples of 8 elements
    const int64_t lead[4] = {o->sa[1], o->b_kcontig ? o->sb[2] : o->sb[1], o->sd[1], o->se[1]};
    const int64_t bstr[4] = {o->sa[0], o->sb[0], o->sd[0], o->se[0]};
    for (int t = 0; t < 4; ++t)
        if (lead[t] % 8 != 0 || bstr[t] % 8 != 0) return MCF_EALIGN;
    if (!o->b_kcontig && p->N % 8 != 0) return MCF_EUNSUPPORTED;
    // the kernels address a tile with 32-bit byte offsets from a 64-bit tile base
    for (int t = 0; t < 4; ++t)
        if (lead[t] >= (1ll << 21)) return MCF_EUNSUPPORTED;
    return MCF_OK;
}

// Elements spanned by a [batch, rows, cols] tensor with the given strides.
static int64_t span(int64_t batch, int64_t rows, int64_t cols, const int64_t s[3]) {
    if (batch == 0 || rows == 0 || cols == 0) return 0;
    return 1 + (batch - 1) * s[0] + (rows - 1) * s[1] + (cols - 1) * s[2];
}

// x: xe elements of xs bytes; y: ye elements of 2 bytes
static bool overlaps(const void *x, int64_t xe, int64_t xs, const void *y, int64_t ye) {
    const char *a = (const char *)x, *b = (const char *)y;
    return xe > 0 && ye > 0 && a < b + 2 * ye && b < a + xs * xe;
}

// Variant of the three-GEMM chain for (dtype, K, L, P) and an arrangement, or nullptr.
static const Built *find_variant3(int dtype, int64_t K, int64_t L, int64_t P, int softmax, int b_kcontig, int mb, int rg,
                                    int ns, int nj) {
    const Group *g = group3(dtype, K, L, P);
    if (!g) return nullptr;
    for (const Built *v : g->of[softmax][b_kcontig])
        if (v->mb == mb && v->rg == rg && v->ns == ns && v->nj == nj) return v;
    return nullptr;
}

// The arrangements built for the three-GEMM chain on (dtype, K, L, P, layout of B), each with
// the model terms of its two-GEMM part (the third GEMM adds the same work to all of them) and
// the LDS bytes of the three-GEMM kernel, in registry order.
template <typename F> static int each_candidate3(const mcf_problem *p, int softmax, int b_kcontig, int64_t P, F &&f) {
    const Group *g = group3(p->in_dtype, p->K, p->L, P);
    bool any = false;
    if (g)
        for (const Built *v : g->of[softmax != 0][b_kcontig]) {
            if (v->scratch_bytes != 0 || !v->two) continue;
            mcf_tiles t;
            eval_model(p, v->two, &t);
            t.lds_bytes = v->lds_bytes; // with the F tile
            any = true;
            f(t);
        }
    return any ? MCF_OK : MCF_EUNSUPPORTED;
}
int candidates3(const mcf_problem *p, int softmax, int b_kcontig, int64_t P, std::vector<mcf_tiles> *out) {
    out->clear();
    return each_candidate3(p, softmax, b_kcontig, P, [&](const mcf_tiles &t) { out->push_back(t); });
}

// Tile choice for the three-GEMM chain: the arrangement (among those built for it) whose
// two-GEMM part the model ranks best (ties broken as for the two-GEMM chain); the third GEMM
// adds the same work to each of them.
static int pick3(const mcf_problem *p, int softmax, int b_kcontig, int64_t P, mcf_tiles *out) {
    bool first = true;
    return each_candidate3(p, softmax, b_kcontig, P, [&](const mcf_tiles &t) {
        if (first || better(t, *out, softmax, p->K, chain3_f_bytes((int)p->L, (int)P))) *out = t;
        first = false;
    });
}

// The arrangement a call without one runs, from the model's pick.  The model does not see what an n-tile costs
// a block beside its loads and flops (a barrier, an LDS round trip, the load latency a short ring leaves bare).
//  * Where a ragged N pads least with it, it takes the narrowest n-tile.  Four waves with an n-tile of 32 columns
//    give way to eight with 128 (or 64) on the same rows: 15 x [1635,64].[64,4048].[4048,128] 85 -> 40 us, softmax
//    5 x 3887 x 2207, K = L = 64: 34 -> 24 us.
//    Plain chains also with many blocks (45 drawn calls of 260 to 3300 blocks: where it acts 0.71 to 0.92 of the time, none
//    slower; 32 x [2881,128].[128,976].[976,128], 736 blocks: 65 -> 56 us).
//    A softmax chain with more blocks than compute units stays: two blocks of four waves share a unit as well
//    (causal, 2376 blocks, K = L = 64: 1.10 of the time with eight).
//    Plain chains in eight waves across m take two slices a wave for one, where that pads N by an eighth of it at most (one n-tile
//    of 64 columns costs a block less than two of 32): 40 x [1000,96].[96,776].[776,96] 21.0 -> 17.9 us, the same with K = L = 64
//    14.7 -> 13.4 and with 128 22.4 -> 21.5; 80 x [500,64].[64,520].[520,128] 15.4 -> 13.9 us.  Not with more blocks than compute
//    units, where the registers of one slice let two blocks share one: 70 x [2707,96].[96,2464].[2464,96] 173 against 188 us.
//  * Among equal estimates it takes the wider n-tile.  Softmax kernels of four waves whose rows are padded to the
//    LDS pitch (K = 80) run better with one slice a wave: 40 x 333 x 1357, causal: 19.9 us with two, 18.7 with one.
// Chains of three GEMMs keep the pick: a wave that holds part of a row's n range rounds its part of E to 16 bits before the
// third GEMM, which is the caller's or the model's choice and not one to be made behind it (parts that cancel, or that
// leave fp16, are lost).
static int64_t padding_of(int64_t n, int64_t tn) { return (n + tn - 1) / tn * tn - n; }
static bool built(const mcf_problem *p, int softmax, int b_kcontig, int64_t tn_now, mcf_tiles *t) {
    if (eval_tiles(p, softmax, b_kcontig, t) != MCF_OK) return false;
    const int64_t pad = padding_of(p->N, t->tn);
    return 20 * pad < p->N || pad <= padding_of(p->N, tn_now); // Rule 3
}
// Columns that the m-tiles of tm rows see under a mask of that offset, and the last row: m-tile m sees tm (m + 1) + off of them, within 0 .. N.
static int64_t visible_columns(int64_t M, int64_t N, int64_t tm, int64_t off, int64_t *last) {
    const auto within = [](int64_t x, int64_t lo, int64_t hi) { return x < lo ? lo : x > hi ? hi : x; };
    const int64_t tiles = (M + tm - 1) / tm;
    const int64_t none = within(off < 0 ? -off / tm : 0, 0, tiles);                     // m-tiles [0, none) see nothing,
    const int64_t all = within(N > off ? (N - off + tm - 1) / tm - 1 : 0, none, tiles);  // [all, tiles) everything
    const int64_t rising = all - none;
    *last = within(M + off, 0, N);
    return rising * off + tm * (rising * (none + 1 + all) / 2) + (tiles - all) * N;
}

// Time of a chain in us from how many blocks a compute unit holds, which the model's estimate does not see: its units
// take their blocks in rounds of as many as LDS and registers let them hold, a round lasts as long as the
// matrix and vector work of its blocks at the rate that their waves reach together, or as its n-tiles take whatever their width,
// and ends with a fill and a drain; and no plain call is faster than its bytes (softmax calls are, by this estimate: decode calls of one
// m-tile that it moves take 0.80 to 1.00 of the pick's time all the same).
// Under a mask (off: its offset) a call takes as long as its longest block at least.  Constants fitted to 419 softmax chains in nine
// arrangements and 312 plain ones in fourteen and T_L, drawn with 129 blocks or more.
struct TimeFit {
    double mac, column, ends, first, tile, bytes_per_us;
    double rate[4]; // of 1 to 4 waves a SIMD, against two
};
static double chain_time(const TimeFit &fit, const mcf_problem *p, const Built *v, double cost, const int64_t *off) {
    const int waves = v->rg * v->ns, simd = waves > 4 ? waves / 4 : 1;
    const int tm = 32 * v->mb * v->rg, tn = 32 * v->ns * v->nj;
    int held = kVgprBudget / ((v->vgprs + 7) / 8 * 8) / simd;
    held = held < kLdsBytesPerBlock / v->lds_bytes ? held : kLdsBytesPerBlock / v->lds_bytes;
    if (held < 1) held = 1;
    const int64_t m_tiles = (p->M + tm - 1) / tm, n_tiles = (p->N + tn - 1) / tn, blocks = p->batch * m_tiles * (p->L / v->L);
    const double padded = (double)(n_tiles * tn);
    double mean = padded, longest = padded;
    if (off) {
        int64_t last;
        mean = (double)visible_columns(p->M, p->N, tm, *off, &last) / (double)m_tiles + 0.5 * tn;
        mean = mean < padded ? mean : padded;
        longest = (double)((last + tn - 1) / tn * tn);
    }
    const double column = tm * (fit.mac * (double)(p->K + v->L) + fit.column) * cost * 1e-6;
    const auto round = [&](int64_t blocks_a_unit, double columns) {
        const double work = (double)blocks_a_unit * column * columns / fit.rate[blocks_a_unit * simd < 4 ? blocks_a_unit * simd - 1 : 3];
        const double tiles = fit.tile * (double)n_tiles;
        return (work > tiles ? work : tiles) + fit.ends;
    };
    const int64_t slots = (int64_t)kComputeUnits * held, full = blocks / slots, rest = blocks - full * slots;
    double t = (double)full * round(held, mean);
    if (rest > 0) t += round((rest + kComputeUnits - 1) / kComputeUnits, mean);
    if (longest > mean) {
        int64_t beside = (blocks + kComputeUnits - 1) / kComputeUnits;
        const double alone = round(beside < held ? beside : held, longest);
        t = blocks > slots && t > alone ? t : alone;
    }
    if (fit.bytes_per_us > 0.) {
        const double bytes = 2.0 * (double)p->batch * ((double)p->M * p->K + (double)p->K * p->N + (double)p->N * p->L + (double)p->M * p->L * (p->out_dtype == MCF_F32 ? 2 : 1));
        if (t < bytes / fit.bytes_per_us) t = bytes / fit.bytes_per_us;
    }
    return t + fit.first;
}
// A call that n is not split for (more blocks than half the compute units): another arrangement where that is a tenth faster at
// least by chain_time (softmax chains: of whole L); a fifth where the rules of settle_tiles have acted, whose arrangements it underrates (128 x
// [2881,128].[128,976].[976,128]: 1.19 by chain_time, 1.10 measured).  Rule 3 (padding) is left aside.  Calls outside the fit whose arrangement is not the
// model's pick, against that: 220 softmax chains 0.35 to 1.09 of the time (0.76 in the mean), 250 under a mask 0.27 to 1.43 (0.79; 13 of them more
// than 3 % longer), 60 plain ones 0.43 to 1.03 (0.80).
static void settle_many(const mcf_problem *p, int softmax, int b_kcontig, const int64_t *off, bool settled, mcf_tiles *t) {
    struct Cost { int mb, rg, ns, nj; double cost; }; // of a column of an m-tile, against each other
    static const Cost kSoftmax[] = {{1, 8, 1, 2, 0.88}, {1, 8, 1, 1, 1.00}, {1, 4, 1, 2, 0.92}, {1, 4, 1, 1, 1.01}, {1, 4, 2, 2, 0.98},
                                    {1, 4, 2, 1, 1.12}, {1, 2, 2, 2, 1.27}, {1, 2, 2, 1, 1.22}, {1, 1, 4, 1, 1.82}};
    static const Cost kPlain[] = {{1, 8, 1, 2, 0.65}, {1, 8, 1, 1, 0.72}, {1, 4, 1, 2, 0.83}, {1, 4, 1, 1, 1.08}, {1, 4, 2, 2, 0.70},
                                  {1, 4, 2, 1, 0.76}, {1, 2, 2, 2, 0.81}, {1, 2, 2, 1, 0.91}, {1, 1, 4, 1, 1.17}, {2, 4, 2, 2, 0.59},
                                  {2, 4, 2, 1, 0.66}, {2, 2, 4, 1, 0.69}, {2, 2, 2, 1, 0.72}, {4, 2, 4, 1, 0.57}};
    static const TimeFit kSoftmaxFit = {0.325, 20.1, 4.3, 1.0, 0., 0., {0.72, 1.0, 1.08, 1.08}};
    static const TimeFit kPlainFit = {0.519, 1.86, 3.16, 1.5, 0.356, 2.92e6, {0.71, 1.0, 0.95, 1.11}};
    const TimeFit &fit = softmax ? kSoftmaxFit : kPlainFit;
    const Cost *costs = softmax ? kSoftmax : kPlain;
    const int n_costs = softmax ? (int)(sizeof(kSoftmax) / sizeof(Cost)) : (int)(sizeof(kPlain) / sizeof(Cost));
    if (p->N <= 0 || 2 * t->blocks <= kComputeUnits || t->tk < p->K || (softmax && t->tl != p->L)) return;
    // (K, L of 64 and fewer, three blocks a unit and more: the softmax fit is least sure of these, so a call does not leave them)
    if (softmax && t->mb == 1 && t->rg == 2 && t->ns == 2 && t->nj == 1 && p->K <= 64) return;
    const Built *best = nullptr;
    double now = 0., least = 0.;
    for (int parts = 1; parts == 1 || (!softmax && p->L / parts >= 32); ++parts) {
        if (p->L % parts != 0) continue;
        const Group *g = resolve_group(p->in_dtype, p->K, p->L / parts);
        if (!g || g->ksplit) continue;
        for (const Built *v : g->of[softmax][b_kcontig]) {
            if (!v->fits || v->vgprs <= 0) continue;
            for (int i = 0; i < n_costs; ++i) {
                const Cost &c = costs[i];
                if (v->mb != c.mb || v->rg != c.rg || v->ns != c.ns || v->nj != c.nj) continue;
                const double us = chain_time(fit, p, v, c.cost, off);
                if (t->mb == c.mb && t->rg == c.rg && t->ns == c.ns && t->nj == c.nj && t->tl == v->L) now = us;
                const int64_t tm = 32ll * c.mb * c.rg, blocks = p->batch * ((p->M + tm - 1) / tm) * parts;
                // (plain chains: not to m-tiles of 32 and 64 rows in four waves, of which the fit is least sure: 108 x [607,32].[32,608].[608,32] 12.6
                // -> 13.7 us, 2 x [2152,128].[128,3808].[3808,128] 32.4 -> 33.8)
                if (!softmax && c.mb * c.rg <= 2 && c.rg * c.ns == 4) continue;
                if (2 * blocks > kComputeUnits && (!best || us < least)) { best = v; least = us; }
            }
        }
    }
    if (best && now > 0. && (settled ? 1.2 : 1.1) * least < now) eval_model(p, best, t);
}
static bool settle_tiles(const mcf_problem *p, int softmax, int b_kcontig, mcf_tiles *t) {
    if (t->tk < p->K) return false; // a k loop: measured as it is
    mcf_tiles w;
    memset(&w, 0, sizeof(w));
    w.mb = t->mb; w.rg = t->rg; w.ns = t->ns; w.tl = t->tl;
    if (t->mb == 1 && t->rg == 4 && t->ns == 1 && t->nj == 1 && (!softmax || t->blocks <= kComputeUnits)) {
        w.ns = 2;
        for (w.nj = 2; w.nj >= 1; --w.nj)
            if (built(p, softmax, b_kcontig, t->tn, &w)) { *t = w; return true; }
    } else if (!softmax && t->mb == 1 && t->rg == 8 && t->ns == 1 && t->nj == 1 && t->blocks <= kComputeUnits) {
        w.nj = 2;
        if (eval_tiles(p, softmax, b_kcontig, &w) == MCF_OK && 8 * padding_of(p->N, w.tn) <= p->N) { *t = w; return true; }
    } else if (softmax && t->rg * t->ns == 4 && t->mb == 1 && t->nj == 2 && pitch_elems(t->tk) != t->tk) {
        w.nj = 1;
        if (built(p, softmax, b_kcontig, t->tn, &w)) { *t = w; return true; }
    }
    return false;
}

// Ranges of n of a call that may have a workspace and leaves the choice to the library.  They pay where
// the blocks leave more than half of the compute units idle and each range is long enough: the second
// kernel and its launch cost about 4 us, eight to ten ring items of a block (an n-tile; a k loop has K / T_K + 1 to
// each n-tile), so the ranges have to shorten a block by ten of them at least, and hold two items each; by eight
// with a k loop, whose items bring A as well (1 x [512,1024].[1024,512].[512,256], nine items fewer: 19 -> 15 us; the 20 calls
// of the sweep with a k loop that are split take 0.93 of their time or less, one with six items fewer 1.01).
// No more ranges than give every compute unit one block.  Measured over 373 calls drawn from the ranges of the chains,
// 318 of them with 256 blocks or fewer: those that it splits run 1.05 to 5 times as fast and none slower than unsplit; with
// eight items instead of ten the first lose (4 x [320,32].. with 11 n-tiles 6.7 -> 8.1 us).  Of 90 more calls drawn near the line
// (10 to 18 items saved) five take 1.00 to 1.17 of their time, K = L of 32 and 64, the others less.  32 rows against 8192 keys of 128:
// 92 -> 33 us; 1 x [639,1024].[1024,664].[664,128]: 100 -> 19 us.  Chains of three are not split unasked: each range would
// round its part of E before the third GEMM.
// An n-tile of more than 28 KiB of B and D counts by its bytes (tile_bytes): 3 x 300 x 1500, K = L = 128, twelve of 48 KiB: 15.4 unsplit, 10.7 us in four
// ranges; 2 x [500,160].[160,1400].[1400,160], eleven of 80 KiB: 16.7 and 12.2; 1 x [132,160].[160,816].[816,160], seven: 12.5 and 11.0 in three.
// Where fewer than ten n-tiles are saved, the results of the ranges (range_bytes each), written and read again, count as well: 2 x [1241,192].[192,616].[616,192], 9.8 MB in
// five: 13.5 and 15.6; 2 x 3983 x 399, K = L = 256, 33 MB in four: 20.1 and 27.5.
static int64_t ranges_for(int64_t blocks, int64_t n_tiles, int64_t items_per_tile, int64_t tile_bytes, int64_t range_bytes) {
    if (blocks <= 0 || 2 * blocks > kComputeUnits) return 1;
    const int64_t least = items_per_tile >= 2 ? 1 : 2; // n-tiles of a range
    int64_t s = kComputeUnits / blocks;
    if (s > n_tiles / least) s = n_tiles / least;
    if (s < 2) return 1;
    const int64_t per = (n_tiles + s - 1) / s;
    if (items_per_tile >= 2) return (n_tiles - per) * items_per_tile >= 8 ? s : 1;
    const int64_t unit = 28 * 1024;
    if (n_tiles - per >= 10 || tile_bytes <= unit) return n_tiles - per >= 10 ? s : 1;
    return (n_tiles - per) * tile_bytes >= 10 * unit + s * range_bytes / 40 ? s : 1;
}

// Longest first pays where blocks wait for a compute unit and differ in length; otherwise the order that keeps a batch
// within one L2 is the faster one: where each block has a unit of its own from the start by 4-7 % (15 x 757 x 757, K = L =
// 64, 180 blocks: 9.8 against 10.5 us; 125 x 128 x 128, 250 blocks: 5.0 against 5.2 us), and where a mask hides little by more:
// 79 x 704 x 3200, K = L = 64, nothing hidden: 70 against 100 us; 102 x 538 x 6145, the last row seeing all: 294 against 347.
// Over 100 calls with 257 to 4000 blocks, longest first took 0.88 to 1.43 of the time (1.05 in the mean) where the
// longest block is less than an eighth longer than the mean one, 0.70 to 1.02 (0.88) where it is more.
bool longest_first(int64_t M, int64_t N, int64_t tm, int64_t off) {
    if (M <= 0 || N <= 0) return false;
    int64_t last;
    const int64_t sum = visible_columns(M, N, tm, off, &last);
    return 8 * last * ((M + tm - 1) / tm) >= 9 * sum && sum > 0;
}

// Validation, tile choice and kernel arguments of one call.  P == 0: the two-GEMM chain into
// E[b, M, L].  P > 0: the three-GEMM chain; F[b, L, P] with strides f_stride (all zero = packed),
// and E / e_stride describe the output [b, M, P].
int prepare(const mcf_call *call, Launch *o) {
    set_last_error("");
    o->v = nullptr;
    o->workspace_bytes = 0;
    if (!call || call->P < 0 || call->n_split < 0) return MCF_EINVAL;
    mcf_problem pc = call->problem;
    const mcf_problem *p = &pc;
    const int softmax = call->softmax != 0 || call->causal != 0;
    const int64_t P = call->P;
    const float scale = call->scale;
    const void *A = call->A, *B = call->B, *D = call->D, *F = call->F;
    void *E = call->E;
    if (p->batch < 0 || p->M < 0 || p->K < 0 || p->N < 0 || p->L < 0) return MCF_EINVAL;
    const bool ch3 = P > 0;
    if (ch3 && call->causal) return MCF_EUNSUPPORTED;
    int64_t sg[3] = {0, 0, 0}, sf[3] = {0, 0, 0};
    if (ch3) {
        // A, B, D are laid out as in the two-GEMM chain; the output and F are checked here
        memcpy(sg, p->e_stride, sizeof(sg));
        memset(pc.e_stride, 0, sizeof(pc.e_stride));
        if (all_zero(sg)) packed(sg, p->M, P);
        memcpy(sf, call->f_stride, sizeof(sf));
        if (all_zero(sf)) packed(sf, p->L, P);
        for (int d = 0; d < 3; ++d)
            if (sg[d] < 0 || sf[d] < 0) return MCF_EINVAL;
        if (sg[2] != 1 || sf[2] != 1) return MCF_EUNSUPPORTED;
        if ((p->M > 1 && sg[1] < P) || (p->L > 1 && sf[1] < P)) return MCF_EINVAL;
        if (sg[1] % 8 || sg[0] % 8 || sf[1] % 8 || sf[0] % 8) return MCF_EALIGN;
        if (sg[1] >= (1ll << 21) || sf[1] >= (1ll << 21)) return MCF_EUNSUPPORTED;
        if (!batches_disjoint(p->batch, p->M, P, sg)) return MCF_EINVAL;
        if (!span_fits(p->batch, p->M, P, sg) || !span_fits(p->batch, p->L, P, sf)) return MCF_EUNSUPPORTED;
    }
    Layout lay;
    int st = decode_layout(p, &lay);
    if (st != MCF_OK) return st;
    if (ch3) memcpy(lay.se, sg, sizeof(sg));
    if (softmax && !(scale == scale && fabsf(scale) <= 3.0e38f)) return MCF_EINVAL; // NaN / inf scale
    if (p->batch == 0 || p->M == 0 || p->L == 0) return MCF_OK;
    if (softmax && p->N == 0) return MCF_EINVAL;
    if (!A || !E || (p->N > 0 && (!B || !D)) || (ch3 && !F)) return MCF_EINVAL;

    const int64_t ea = span(p->batch, p->M, p->K, lay.sa), eb = span(p->batch, p->K, p->N, lay.sb);
    const int64_t ed = span(p->batch, p->N, p->L, lay.sd), ee = span(p->batch, p->M, ch3 ? P : p->L, lay.se);
    const int64_t ef = ch3 ? span(p->batch, p->L, P, sf) : 0;
    const int64_t es = p->out_dtype == MCF_F32 ? 4 : 2; // bytes per element of the output
    if (overlaps(E, ee, es, A, ea) || overlaps(E, ee, es, B, eb) || overlaps(E, ee, es, D, ed) || (ch3 && overlaps(E, ee, es, F, ef)))
        return MCF_EINVAL;
    const uintptr_t ptrs[5] = {(uintptr_t)A, (uintptr_t)B, (uintptr_t)D, (uintptr_t)E, (uintptr_t)F};
    for (int t = 0; t < 5; ++t)
        if (ptrs[t] % 16 != 0) return MCF_EALIGN;

    mcf_tiles chosen;
    if (call->tiles) {
        chosen = *call->tiles;
    } else {
        st = ch3 ? pick3(p, softmax, lay.b_kcontig, P, &chosen) : pick_tiles(p, softmax, lay.b_kcontig, &chosen);
        if (st != MCF_OK) return st;
        if (!ch3) {
            const bool settled = settle_tiles(p, softmax, lay.b_kcontig, &chosen);
            const int64_t off = call->causal_offset > p->N ? p->N : call->causal_offset < -p->M ? -p->M : call->causal_offset;
            settle_many(p, softmax, lay.b_kcontig, call->causal ? &off : nullptr, settled, &chosen);
        }
    }
    const int64_t tl = ch3 ? p->L : (chosen.tl > 0 ? chosen.tl : p->L);
    if (p->L % tl != 0) return MCF_EINVAL;
    const int nj_ = chosen.nj > 0 ? chosen.nj : 1;
    const Built *v = ch3 ? find_variant3(p->in_dtype, p->K, p->L, P, softmax, lay.b_kcontig, chosen.mb, chosen.rg, chosen.ns, nj_)
                           : find_variant(p->in_dtype, p->K, tl, softmax, lay.b_kcontig, chosen.mb, chosen.rg, chosen.ns, nj_);
    if (!v) {
        if (!ch3) return call->tiles ? MCF_EINVAL : MCF_EUNSUPPORTED;
        // no kernels for this (K, L, P) at all, or only this arrangement is missing?
        mcf_tiles any;
        return pick3(p, softmax, lay.b_kcontig, P, &any) == MCF_OK ? MCF_EINVAL : MCF_EUNSUPPORTED;
    }
    if (v->lds_bytes > kLdsBytesPerBlock)
        return MCF_EINVAL; // more LDS than a compute unit has

    const int64_t tm = 32ll * v->mb * v->rg;
    const int64_t m_tiles = (p->M + tm - 1) / tm;
    const int64_t h_tiles = p->L / tl;
    if (p->batch * m_tiles * h_tiles >= (1ll << 31)) return MCF_EUNSUPPORTED;

    KParams &k = o->k;
    memset(&k, 0, sizeof(k));
    k.A = A; k.B = B; k.D = D; k.E = E;
    k.sa_b = lay.sa[0]; k.sa_r = lay.sa[1];
    k.sb_b = lay.sb[0]; k.sb_r = lay.b_kcontig ? lay.sb[2] : lay.sb[1];
    k.sd_b = lay.sd[0]; k.sd_r = lay.sd[1];
    k.se_b = lay.se[0]; k.se_r = lay.se[1];
    k.M = (int32_t)p->M; k.N = (int32_t)p->N;
    k.m_tiles = (int32_t)m_tiles;
    k.h_tiles = (int32_t)h_tiles;
    k.n_blocks = (int32_t)(p->batch * m_tiles * h_tiles);
    k.lpt = 0;
    if (call->causal && k.n_blocks > kComputeUnits) {
        const int64_t off = call->causal_offset;
        k.lpt = longest_first(p->M, p->N, tm, off > p->N ? p->N : off < -p->M ? -p->M : off);
    }
    k.divisor = (int32_t)(k.lpt ? p->batch : m_tiles * h_tiles);
    division_magic((uint32_t)k.divisor, &k.d_magic, &k.d_shift);
    division_magic((uint32_t)h_tiles, &k.h_magic, &k.h_shift);
    k.c1 = 1.0f; k.a_mode = 0;
    k.k_chunks = (int32_t)(p->K / v->K);
    k.F = F; k.sf_b = sf[0]; k.sf_r = sf[1];
    if (p->out_dtype == MCF_F32) k.E = (void *)((uintptr_t)E | 1); // the kernels read bit 0 as "store fp32"
    if (softmax) {
        // row i sees the columns n <= i + causal_off, which the kernel forms in 32 bits; an offset
        // of N - 1 (or more) hides nothing and stands for "no mask", below -M nothing is seen either
        if (p->M + p->N >= (1ll << 31) - 1024) { set_last_error("softmax chain: M + N must stay below 2^31 - 1024"); return MCF_EUNSUPPORTED; }
        const int64_t off = call->causal_offset;
        k.causal_off = (int32_t)(!call->causal || off > p->N - 1 ? p->N - 1 : off < -p->M - 1 ? -p->M - 1 : off);
    }
    if (softmax) {
        // exp(scale*s - max) = exp2(|scale|*log2(e) * (s' - max')) with s' = +-s; a zero scale
        // makes every logit equal, which is what A := 0 gives.
        const float log2e = 1.4426950408889634f;
        if (scale == 0.0f) { k.a_mode = 2; k.c1 = log2e; }
        else { k.a_mode = scale < 0.0f ? 1 : 0; k.c1 = fabsf(scale) * log2e; }
    }

    // n ranges of whole n-tiles, each a row of blocks of its own; more would leave some empty.  Where the library chooses,
    // of the columns that the last row sees under a mask (33 x 7 x 6282, K = L = 192, of which 7 are seen, was split into seven
    // ranges: 15 us for 9).
    const int64_t tn = 32ll * v->ns * v->nj;
    int64_t n_tiles = (p->N + tn - 1) / tn, n_split = call->n_split;
    if (n_split == 0 && (call->tiles || ch3)) n_split = 1;
    if (n_split == 0) {
        if (softmax) {
            const int64_t seen = p->M + k.causal_off < p->N ? p->M + k.causal_off : p->N;
            n_tiles = seen > 0 ? (seen + tn - 1) / tn : 0;
        }
        n_split = ranges_for(k.n_blocks, n_tiles, v->ksplit ? k.k_chunks + 1 : 1, stage_bytes(v->K, v->L, (int)tn), p->batch * p->M * (p->L + 4) * 4);
    }
    int64_t per = n_split < n_tiles ? (n_tiles + n_split - 1) / n_split : 1;
    n_split = n_tiles > 0 ? (n_tiles + per - 1) / per : 1;
    k.n_split = (int32_t)n_split;
    k.split_cols = n_split > 1 ? (int32_t)(per * tn) : k.N;
    o->dtype = p->in_dtype;
    o->softmax = softmax;
    if (n_split > 1) {
        if (n_split > 65535) return MCF_EINVAL;
        CombineParams &c = o->c;
        c.L = (int32_t)(ch3 ? P : p->L);
        c.pitch = c.L + (softmax ? 4 : 0);
        c.rows = p->batch * p->M; c.M = p->M;
        c.split_stride = c.rows * c.pitch;
        c.se_b = k.se_b; c.se_r = k.se_r;
        c.E = E; c.n_split = (int32_t)n_split; c.out_f32 = p->out_dtype == MCF_F32;
        k.se_b = p->M * c.pitch; k.se_r = c.pitch; k.se_s = c.split_stride;
        o->workspace_bytes = n_split * c.split_stride * 4;
        // (rows and their places are formed in 32 bits: a workspace of more would be 550 GB at least)
        if (c.rows >= (1ll << 31) || c.split_stride > (1ll << 40)) return MCF_EUNSUPPORTED;
        c.block_rows = 256 / (c.L >> 2);
        division_magic((uint32_t)(c.L >> 2), &c.quads_magic, &c.quads_shift);
        division_magic((uint32_t)p->M, &c.m_magic, &c.m_shift);
    }
    o->v = v;
    o->tiles.mb = v->mb; o->tiles.rg = v->rg; o->tiles.ns = v->ns; o->tiles.nj = v->nj; o->tiles.tl = (int32_t)tl;
    return MCF_OK;
}

// Launches what prepare() laid out.  Host errors of the launches as MCF_ELAUNCH.
int launch(Launch *o, void *workspace, int64_t workspace_bytes, void *stream) {
    if (!o->v) return MCF_OK; // nothing to compute
    if (o->workspace_bytes > 0) {
        if (!workspace || workspace_bytes < o->workspace_bytes) return MCF_EINVAL;
        if ((uintptr_t)workspace % 16 != 0) return MCF_EALIGN;
        o->c.part = (const float *)workspace;
        o->k.E = (void *)((uintptr_t)workspace | 2); // the kernels read bit 1 as "results of n ranges"
    }
    int err = o->v->launch(o->k, stream);
    if (err == 0 && o->workspace_bytes > 0) err = launch_combine(o->c, o->dtype, o->softmax, stream);
    if (err != 0) {
        set_last_error(hipGetErrorString((hipError_t)err));
        return MCF_ELAUNCH;
    }
    return MCF_OK;
}

bool stream_capturing(void *stream) {
    hipStreamCaptureStatus status = hipStreamCaptureStatusNone;
    if (hipStreamIsCapturing((hipStream_t)stream, &status) == hipSuccess) return status != hipStreamCaptureStatusNone;
    (void)hipGetLastError(); // (the default stream while another one is captured): the launch will say so itself
    return false;
}

// The calls without a workspace: n is never split.
static int run(const mcf_problem *p, int softmax, float scale, const void *A, const void *B, const void *D, void *E,
               const mcf_tiles *tiles, void *stream, int64_t P = 0, const int64_t *fstr = nullptr,
               const void *F = nullptr, bool causal = false, int64_t causal_off = 0) {
    if (!p) return MCF_EINVAL;
    mcf_call call;
    memset(&call, 0, sizeof(call));
    call.problem = *p;
    call.P = P;
    if (fstr) memcpy(call.f_stride, fstr, sizeof(call.f_stride));
    call.softmax = softmax; call.causal = causal; call.scale = scale; call.causal_offset = causal_off;
    call.n_split = 1;
    call.A = A; call.B = B; call.D = D; call.F = F; call.E = E; call.tiles = tiles;
    Launch o;
    const int st = prepare(&call, &o);
    return st != MCF_OK ? st : launch(&o, nullptr, 0, stream);
}

} // namespace mcf

extern "C" int mcf_gemm_chain(const mcf_problem *p, const void *A, const void *B, const void *D, void *E,
                              const mcf_tiles *tiles, void *stream) {
    return mcf::run(p, 0, 1.0f, A, B, D, E, tiles, stream);
}

extern "C" int mcf_softmax_gemm_chain(const mcf_problem *p, float scale, const void *A, const void *B, const void *D,
                                      void *E, const mcf_tiles *tiles, void *stream) {
    return mcf::run(p, 1, scale, A, B, D, E, tiles, stream);
}

extern "C" int mcf_causal_softmax_gemm_chain(const mcf_problem *p, float scale, int64_t causal_offset, const void *A,
                                             const void *B, const void *D, void *E, const mcf_tiles *tiles, void *stream) {
    return mcf::run(p, 1, scale, A, B, D, E, tiles, stream, 0, nullptr, nullptr, true, causal_offset);
}

extern "C" int mcf_gemm_chain3(const mcf_problem *p, int softmax, float scale, int64_t P, const int64_t *f_stride,
                               const void *A, const void *B, const void *D, const void *F, void *G,
                               const mcf_tiles *tiles, void *stream) {
    if (P <= 0) return P == 0 && p && p->batch >= 0 ? MCF_OK : MCF_EINVAL; // no output columns: nothing to do
    return mcf::run(p, softmax != 0, softmax ? scale : 1.0f, A, B, D, G, tiles, stream, P, f_stride, F);
}

extern "C" int mcf_call_workspace(const mcf_call *call, int64_t *bytes) {
    if (!bytes) return MCF_EINVAL;
    mcf::Launch o;
    const int st = mcf::prepare(call, &o);
    *bytes = st == MCF_OK ? o.workspace_bytes : 0;
    return st;
}

extern "C" int mcf_call_tiles(const mcf_call *call, mcf_tiles *tiles, int32_t *n_split) {
    if (!tiles || !n_split) return MCF_EINVAL;
    memset(tiles, 0, sizeof(*tiles));
    *n_split = 0;
    mcf::Launch o;
    int st = mcf::prepare(call, &o);
    if (st != MCF_OK || !o.v) return st;
    mcf_problem p = call->problem;
    if (call->P > 0) memset(p.e_stride, 0, sizeof(p.e_stride)); // they describe G there
    memcpy(tiles, &o.tiles, sizeof(o.tiles));
    st = mcf_eval_tiles(&p, o.softmax, tiles);
    if (st != MCF_OK && st != MCF_EINVAL) return st; // (MCF_EINVAL: over a budget of the model, which given tiles may be)
    if (call->P > 0) {
        tiles->lds_bytes = o.v->lds_bytes;
        tiles->stages = o.v->stages;
        tiles->vgpr_used = o.v->vgprs;
        tiles->scratch_bytes = o.v->scratch_bytes;
    }
    *n_split = o.k.n_split;
    return MCF_OK;
}

extern "C" int mcf_call_run(const mcf_call *call, void *workspace, int64_t workspace_bytes, void *stream) {
    mcf::Launch o;
    const int st = mcf::prepare(call, &o);
    return st != MCF_OK ? st : mcf::launch(&o, workspace, workspace_bytes, stream);
}

extern "C" int mcf_pick_tiles3(const mcf_problem *p, int64_t P, int softmax, mcf_tiles *out) {
    mcf::Layout lay;
    if (!p || !out || P <= 0) return MCF_EINVAL;
    mcf_problem pc = *p;
    memset(pc.e_stride, 0, sizeof(pc.e_stride)); // describes G, which the tile choice does not depend on
    const int st = mcf::decode_layout(&pc, &lay);
    if (st != MCF_OK) return st;
    return mcf::pick3(&pc, softmax != 0, lay.b_kcontig, P, out);
}

namespace mcf {
// Problem of the two-GEMM part and layout of B for a three-GEMM problem (e_stride describes G).
int problem3(const mcf_problem *p, int64_t P, mcf_problem *pc, int *b_kcontig) {
    mcf::Layout lay;
    if (!p || P <= 0) return MCF_EINVAL;
    *pc = *p;
    memset(pc->e_stride, 0, sizeof(pc->e_stride));
    const int st = mcf::decode_layout(pc, &lay);
    if (st == MCF_OK) *b_kcontig = lay.b_kcontig;
    return st;
}
} // namespace mcf

extern "C" int mcf_list_candidates3(const mcf_problem *p, int64_t P, int softmax, mcf_tiles *out, int cap) {
    mcf_problem pc;
    int bk = 0;
    std::vector<mcf_tiles> c;
    if (mcf::problem3(p, P, &pc, &bk) != MCF_OK || mcf::candidates3(&pc, softmax != 0, bk, P, &c) != MCF_OK) return 0;
    for (int i = 0; i < (int)c.size() && out && i < cap; ++i) out[i] = c[i];
    return (int)c.size();
}

extern "C" int mcf_list_variants3(const mcf_problem *p, int64_t P, int softmax, int32_t *out, int cap) {
    mcf::Layout lay;
    if (!p) return 0;
    mcf_problem pc = *p;
    memset(pc.e_stride, 0, sizeof(pc.e_stride));
    if (mcf::decode_layout(&pc, &lay) != MCF_OK) return 0;
    int total = 0;
    const mcf::Group *g = mcf::group3(p->in_dtype, p->K, p->L, P);
    if (!g) return 0;
    for (const mcf::Built *v : g->of[softmax != 0][lay.b_kcontig]) {
        if (out && total < cap) {
            out[4 * total] = v->mb; out[4 * total + 1] = v->rg; out[4 * total + 2] = v->ns; out[4 * total + 3] = v->nj;
        }
        ++total;
    }
    return total;
}

extern "C" const char *mcf_status_string(int s) {
    switch (s) {
    case MCF_OK: return "MCF_OK";
    case MCF_EINVAL: return "MCF_EINVAL: invalid argument";
    case MCF_EUNSUPPORTED: return "MCF_EUNSUPPORTED: no kernel variant covers this problem";
    case MCF_EALIGN: return "MCF_EALIGN: pointer or stride not 16-byte aligned";
    case MCF_ELAUNCH: return "MCF_ELAUNCH: HIP launch failed";
    default: return "unknown mcf status";
    }
}

extern "C" const char *mcf_last_error(void) { return mcf::g_last_error; }

// Table of every built kernel variant, gathered from the instantiation files.
#include <utility>
#include <vector>

#include "mcf_internal.h"

namespace mcf {

#define MCF_GROUPS(X)                                                                                      \
    X(f16_32_32) X(f16_64_64) X(f16_128_128) X(f16_64_128) X(f16_128_64) X(f16_64_256) X(f16_256_256)         \
    X(bf16_32_32) X(bf16_64_64) X(bf16_128_128) X(bf16_64_128) X(bf16_128_64) X(bf16_64_256) X(bf16_256_256)      \
    X(f16_k128x_64) X(f16_k128x_128) X(f16_k128x_256) X(bf16_k128x_64) X(bf16_k128x_128) X(bf16_k128x_256)      \
    X(f16_80_80) X(bf16_80_80) X(f16_96_96) X(bf16_96_96) X(f16_160_160) X(bf16_160_160) X(f16_192_192) X(bf16_192_192)
#define MCF_GROUPS3(X)                                                                                     \
    X(f16_c3_64_64_64) X(f16_c3_128_128_128) X(bf16_c3_64_64_64) X(bf16_c3_128_128_128)                    \
    X(f16_c3_64_128_128) X(f16_c3_128_64_64) X(f16_c3_64_64_128) X(bf16_c3_64_128_128) X(bf16_c3_128_64_64) X(bf16_c3_64_64_128)
#define MCF_DECL(NAME) const Variant *variants_##NAME(int *count);
MCF_GROUPS(MCF_DECL)
MCF_GROUPS3(MCF_DECL)

// Registers / scratch of every kernel as the compiler built it (generated at build time).
struct Resources {
    int dtype, K, L, mb, rg, ns, nj, softmax, b_kcontig, ksplit, P, vgprs, sgprs, scratch_bytes, spills_in_loops;
};
static const Resources kResources[] = {
#include "mcf_resources.inc"
};

#define MCF_ADD(NAME) add(&t, variants_##NAME);
static void add(std::vector<Built> *t, const Variant *(*group)(int *)) {
    int n = 0;
    const Variant *v = group(&n);
    for (int i = 0; i < n; ++i) {
        if (!v[i].launch) continue;
        Built b = {};
        (Variant &)b = v[i];
        b.vgprs = -1;
        b.scratch_bytes = 0;
        for (const Resources &r : kResources)
            if (r.dtype == b.dtype && r.K == b.K && r.L == b.L && r.mb == b.mb && r.rg == b.rg && r.ns == b.ns &&
                r.nj == b.nj && r.softmax == b.softmax && r.b_kcontig == b.b_kcontig && r.ksplit == b.ksplit && r.P == b.P) {
                b.vgprs = r.vgprs;
                // registers parked in scratch across the n loop (stored before it, fetched after it)
                // cost a block a handful of instructions and do not count; spill code inside a loop does
                b.scratch_bytes = r.spills_in_loops ? r.scratch_bytes : 0;
            }
        describe(&b);
        t->push_back(b);
    }
}

// The groups of a table: the variants of one (dtype, K, L, P) stand together in it.
static std::vector<Group> group_index(const std::vector<Built> &t) {
    std::vector<Group> out;
    for (const Built &v : t) {
        if (out.empty() || out.back().dtype != v.dtype || out.back().K != v.K || out.back().L != v.L || out.back().ksplit != v.ksplit ||
            out.back().P != v.P)
            out.push_back({v.dtype, v.K, v.L, v.ksplit, v.P, {}});
        out.back().of[v.softmax][v.b_kcontig].push_back(&v);
    }
    return out;
}

// Every variant of the two-GEMM chain and its groups; those that hold the whole K on chip also by (dtype, K / 16, L / 16),
// because a call looks for several.
struct Table {
    std::vector<Built> all;
    std::vector<Group> groups;
    const Group *whole[2][17][17] = {};
    Table() {
        std::vector<Built> t;
        MCF_GROUPS(MCF_ADD)
        all = std::move(t);
        groups = group_index(all);
        for (const Group &g : groups)
            if (!g.ksplit) whole[g.dtype][g.K / 16][g.L / 16] = &g;
    }
};
// ... and of the three-GEMM chain (P > 0).
struct Table3 {
    std::vector<Built> all;
    std::vector<Group> groups;
    Table3() {
        std::vector<Built> t;
        MCF_GROUPS3(MCF_ADD)
        for (Built &v : t) v.two = find_variant(v.dtype, v.K, v.L, v.softmax, v.b_kcontig, v.mb, v.rg, v.ns, v.nj);
        all = std::move(t);
        groups = group_index(all);
    }
};

const Group *resolve_group(int dtype, int64_t K, int64_t L) {
    static const Table table;
    if (K >= 0 && K <= 256 && L >= 0 && L <= 256 && K % 16 == 0 && L % 16 == 0)
        if (const Group *g = table.whole[dtype][K / 16][L / 16]) return g;
    const Group *best = nullptr;
    for (const Group &g : table.groups)
        if (g.ksplit && g.dtype == dtype && g.L == L && K > g.K && K % g.K == 0 && (!best || g.K > best->K)) best = &g; // the largest chunk that divides K
    return best;
}

const Group *group3(int dtype, int64_t K, int64_t L, int64_t P) {
    static const Table3 table;
    for (const Group &g : table.groups)
        if (g.dtype == dtype && g.K == K && g.L == L && g.P == P) return &g;
    return nullptr;
}

const Built *find_variant(int dtype, int64_t K, int64_t L, int softmax, int b_kcontig, int mb, int rg, int ns, int nj) {
    const Group *g = resolve_group(dtype, K, L);
    if (!g) return nullptr;
    for (const Built *v : g->of[softmax][b_kcontig])
        if (v->mb == mb && v->rg == rg && v->ns == ns && v->nj == nj) return v;
    return nullptr;
}

} // namespace mcf

// Table of every built kernel variant, gathered from the instantiation files.
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

#define MCF_ADD(NAME)                                    \
    {                                                    \
        int n = 0;                                       \
        const Variant *v = variants_##NAME(&n);          \
        for (int i = 0; i < n; ++i)                      \
            if (v[i].launch) t.push_back(v[i]);          \
    }
static void attach_resources(std::vector<Variant> &t) {
    for (Variant &v : t) {
        v.vgprs = -1;
        v.scratch_bytes = 0;
        for (const Resources &r : kResources)
            if (r.dtype == v.dtype && r.K == v.K && r.L == v.L && r.mb == v.mb && r.rg == v.rg && r.ns == v.ns &&
                r.nj == v.nj && r.softmax == v.softmax && r.b_kcontig == v.b_kcontig && r.ksplit == v.ksplit && r.P == v.P) {
                v.vgprs = r.vgprs;
                // registers parked in scratch across the n loop (stored before it, fetched after it)
                // cost a block a handful of instructions and do not count; spill code inside a loop does
                v.scratch_bytes = r.spills_in_loops ? r.scratch_bytes : 0;
            }
    }
}

static const std::vector<Variant> &all() {
    static const std::vector<Variant> table = [] {
        std::vector<Variant> t;
        MCF_GROUPS(MCF_ADD)
        attach_resources(t);
        return t;
    }();
    return table;
}

static const std::vector<Variant> &all3() {
    static const std::vector<Variant> table = [] {
        std::vector<Variant> t;
        MCF_GROUPS3(MCF_ADD)
        attach_resources(t);
        return t;
    }();
    return table;
}

const Variant *variants3(int *count) {
    const auto &t = all3();
    *count = (int)t.size();
    return t.data();
}

const Variant *variants(int *count) {
    const auto &t = all();
    *count = (int)t.size();
    return t.data();
}

// The groups of a table: the variants of one (dtype, K, L, P) stand together in it.
static std::vector<Group> group_index(const std::vector<Variant> &t) {
    std::vector<Group> out;
    for (int i = 0; i < (int)t.size(); ++i) {
        const Variant &v = t[i];
        if (out.empty() || out.back().dtype != v.dtype || out.back().K != v.K || out.back().L != v.L || out.back().ksplit != v.ksplit ||
            out.back().P != v.P)
            out.push_back({v.dtype, v.K, v.L, v.ksplit, v.P, i, i});
        out.back().end = i + 1;
    }
    return out;
}

const Group *resolve_group(int dtype, int64_t K, int64_t L) {
    static const std::vector<Group> groups = group_index(all());
    const Group *best = nullptr;
    for (const Group &g : groups) {
        if (g.dtype != dtype || g.L != L) continue;
        if (!g.ksplit && g.K == K) return &g;
        if (g.ksplit && K > g.K && K % g.K == 0 && (!best || g.K > best->K)) best = &g; // the largest chunk that divides K
    }
    return best;
}

const Group *group3(int dtype, int64_t K, int64_t L, int64_t P) {
    static const std::vector<Group> groups = group_index(all3());
    for (const Group &g : groups)
        if (g.dtype == dtype && g.K == K && g.L == L && g.P == P) return &g;
    return nullptr;
}

const Variant *find_variant(int dtype, int64_t K, int64_t L, int softmax, int b_kcontig, int mb, int rg, int ns, int nj) {
    const Group *g = resolve_group(dtype, K, L);
    if (!g) return nullptr;
    const Variant *t = all().data();
    for (int i = g->begin; i < g->end; ++i)
        if (t[i].softmax == softmax && t[i].b_kcontig == b_kcontig && t[i].mb == mb && t[i].rg == rg && t[i].ns == ns && t[i].nj == nj)
            return &t[i];
    return nullptr;
}

} // namespace mcf

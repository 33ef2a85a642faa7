// What the planner says of paged calls that tests/test_gather_routes.py describes on standard input,
// one call after the other:
//   dtype layers page flags planes, then per plane: row heads head_stride rot_offset rot_dim style
//   sequences, then their lengths; directives, then per directive: sequence start end replacement
// Prints per call "<gathered rows> <fresh pages> <spans> <short spans> <row table>".
#include <cstdio>
#include <vector>

#include "plan.hpp"

using namespace leyline;

int main() {
    alignas(16) static char dummy[16];
    leyline_cache cache{};
    uint32_t flags = 0;
    while (std::scanf("%d %d %d %u %d", &cache.dtype, &cache.n_layers, &cache.page_size, &flags, &cache.n_planes) == 5) {
        cache.capacity = 1 << 24;
        for (int p = 0; p < cache.n_planes; ++p) {
            leyline_plane& pl = cache.planes[p];
            if (std::scanf("%d %d %d %d %d %d", &pl.row_elems, &pl.n_heads, &pl.head_stride, &pl.rot_offset,
                           &pl.rot_dim, &pl.rope_style) != 6)
                return 1;
            pl.base = dummy;
            pl.token_stride = pl.row_elems;
            pl.page_stride = pl.token_stride * cache.page_size;
            pl.layer_stride = pl.page_stride * cache.capacity;
            pl.rope_base = 1e4;
        }
        int n_seqs = 0, n_dirs = 0;
        if (std::scanf("%d", &n_seqs) != 1) return 1;
        std::vector<int32_t> lens(n_seqs);
        for (int32_t& n : lens)
            if (std::scanf("%d", &n) != 1) return 1;
        if (std::scanf("%d", &n_dirs) != 1) return 1;
        std::vector<leyline_directive> dirs(n_dirs);
        for (leyline_directive& d : dirs) {
            long long s, e, r;
            if (std::scanf("%d %lld %lld %lld", &d.seq, &s, &e, &r) != 4) return 1;
            d.mode = LEYLINE_AMORTIZE;
            d.span_start = s;
            d.span_end = e;
            d.stub_len = r;
            for (const void*& q : d.stub) q = dummy;
        }
        KPlane planes[LEYLINE_MAX_PLANES];
        int n_planes = 0;
        PagedPlan plan;
        PagedImage img;
        if (describe_cache(&cache, true, planes, &n_planes) != LEYLINE_OK ||
            plan_paged(cache.page_size, n_seqs, lens.data(), dirs.data(), n_dirs, n_planes, !flags, &plan) != LEYLINE_OK ||
            build_paged_image(&cache, plan, n_seqs, plan.dirs, n_dirs, 1 << 24, &img) != LEYLINE_OK)
            return 2;
        const KPagedTables& t = img.tables;
        std::printf("%d %d %d %d %d\n", t.n_rows, t.n_asm, t.n_spans, short_gather_spans(t.n_rows, t.n_spans) ? 1 : 0,
                    gather_row_table(planes, n_planes, t, cache.n_layers) ? 1 : 0);
    }
    return 0;
}

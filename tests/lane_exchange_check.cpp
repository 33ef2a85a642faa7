// Half-split planes whose partner chunks the planner exchanges between lanes (neox_lanes), checked
// on the host: with rows laid end to end over wavefronts of 64 units, every band chunk and its
// partner sit in the same wavefront at every row, and with neox_dpp the partner is lane ^ 8 of the
// same 16 lanes.  Prints "<neox_lanes> <neox_dpp>" per plane; exits non-zero on a violation.
#include <cstdio>

#include "plan.hpp"

using namespace leyline;

int main() {
    struct { int32_t dtype, row, heads, stride, off, dim; } cases[] = {
        {LEYLINE_BF16, 1024, 8, 128, 0, 128}, {LEYLINE_BF16, 128, 1, 128, 0, 128},  // whole wavefronts, a divisor
        {LEYLINE_BF16, 576, 1, 576, 512, 64}, {LEYLINE_F32, 576, 1, 576, 512, 64},  // MLA rows
        {LEYLINE_BF16, 640, 5, 128, 0, 128},  {LEYLINE_BF16, 1280, 10, 128, 0, 128},
        {LEYLINE_BF16, 640, 10, 64, 0, 64},   {LEYLINE_F32, 192, 3, 64, 32, 32},
        {LEYLINE_BF16, 768, 8, 96, 0, 96},    {LEYLINE_BF16, 800, 10, 80, 0, 80},   // heads across wavefronts
        {LEYLINE_BF16, 576, 1, 576, 480, 64}, {LEYLINE_BF16, 576, 1, 576, 496, 64}, // a band off its window
        {LEYLINE_BF16, 520, 1, 520, 456, 64},                                       // an odd row
    };
    alignas(16) static char dummy[16];
    for (const auto& c : cases) {
        leyline_cache cache{};
        cache.dtype = c.dtype;
        cache.n_layers = cache.n_planes = 1;
        cache.capacity = 1 << 20;
        leyline_plane& pl = cache.planes[0];
        pl.base = dummy;
        pl.token_stride = pl.row_elems = c.row;
        pl.n_heads = c.heads;
        pl.head_stride = c.stride;
        pl.rot_offset = c.off;
        pl.rot_dim = c.dim;
        pl.rope_style = LEYLINE_ROPE_NEOX;
        pl.rope_base = 1e4;
        KPlane k[LEYLINE_MAX_PLANES];
        int n = 0;
        if (describe_cache(&cache, false, k, &n) != LEYLINE_OK) return 1;
        const KPlane& p = k[0];
        if (p.neox_lanes)
            for (int r = 0; r < 64; ++r)
                for (int h = 0; h < p.n_heads; ++h)
                    for (int j = 0; j < p.rot_chunks / 2; ++j) {
                        const int t = r * p.tpr + h * p.head_chunks + p.rot_lo + j, o = t + p.rot_chunks / 2;
                        if (p.tpr != p.row_chunks || t / 64 != o / 64) return 2;
                        if (p.neox_dpp && (t / 16 != o / 16 || (t ^ 8) != o)) return 3;
                    }
        std::printf("%d %d\n", p.neox_lanes, p.neox_dpp);
    }
    return 0;
}

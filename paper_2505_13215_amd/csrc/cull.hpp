// The conservative ellipse test of binning and of the quadrant blending kernels:
// which tiles (or quadrants) hold a pixel centre that a splat can reach with
// alpha >= 1/255.  Host and device.
#pragma once

#include "common.hpp"
#include "launch.hpp"

namespace h4d {

// Margin (log2 units) between the FP64 tile test and the FP32 per-pixel test:
// the FP32 exponent of a pixel is within about 1e-5 of its exact value, so a
// tile none of whose pixel centres reaches alpha = 1/255 * 2^-margin in exact
// arithmetic has no pixel that the blending kernels would blend.
constexpr double kCullMargin = 1e-3;

// Root of a normal x > 0: on the device the hardware's reciprocal root and one
// step on it, which gives sqrtf's bits (all 2^24 floats of [1, 4)) in a third of its
// instructions (1M splats, 2704 x 2028: counting 0.073 -> 0.067 ms).
__host__ __device__ __forceinline__ float cull_root(float x) {
#ifdef __HIP_DEVICE_COMPILE__
    const float r = __builtin_amdgcn_rsqf(x), y = x * r;
    return __builtin_fmaf(__builtin_fmaf(-y, y, x), 0.5f * r, y);
#else
    return sqrtf(x);
#endif
}
// (the hardware's approximation, one ulp, on the device)
__host__ __device__ __forceinline__ float cull_rcp(float x) {
#ifdef __HIP_DEVICE_COMPILE__
    return __builtin_amdgcn_rcpf(x);
#else
    return 1.f / x;
#endif
}
constexpr float kRootLeast = 1.17549435e-38f, kRootMost = 3.4e38f;  // the range of its argument

// The alpha >= 1/255 region of one splat as the tile test needs it:
// -p2 = a dx^2 - b dx dy + c dy^2 <= t, with dx, dy offsets from the centre.
// Set up in FP64 once per splat by the binning; the per-row test runs in FP32 on
// intervals widened by pad_x / pad_y: 2e-3 of the ellipse's half-extent plus 0.01 px,
// several times the FP32 rounding of the extent (whose worst case, near the
// ellipse's top and bottom, is about 5e-4 of the half-width).
// FP64 = false: for the quadrant kernels, which pick their quadrants' splats from a
// list that is already the tile's, once per tile and splat.  Only the determinant,
// which cancels, is FP64; the rest is within a few roundings, far inside the pads
// (1785 tiles, 73k Gaussians: forward and binning 0.132 ms against 0.146).
template <bool FP64 = true>
__host__ __device__ inline CullShape cull_shape(const Rec& rec) {
#pragma clang fp contract(off)
    CullShape cs;
    const float a = -rec.a.z, b = rec.a.w, c = -rec.b.x, op = rec.b.y;
    cs.ui = rec.c.y; cs.uf = rec.a.x; cs.vi = rec.c.z; cs.vf = rec.a.y;
    cs.px0 = (int)(rec.d.x & 0xFFFFu); cs.px1 = (int)(rec.d.x >> 16);
    cs.py0 = (int)(rec.d.y & 0xFFFFu); cs.py1 = (int)(rec.d.y >> 16);
    const double ac4 = 4.0 * (double)a * (double)c, det4 = ac4 - (double)b * (double)b;
    cs.mode = 0;
    cs.b = cs.inv2a = cs.four_at = cs.det4 = cs.y_full = cs.y_ext = cs.pad_x = cs.pad_y = 0.f;
    // a proper ellipse only (of a size whose products float32 holds); otherwise keep
    // every overlapped tile
    if (!(fminf(a, c) > 1e-30f && fmaxf(a, c) < 1e25f && det4 > 1e-12 * ac4 && det4 > 1e-30 && det4 < 1e37 &&
          op > 0.f && op < 1e30f))
        return cs;
    cs.b = b;
    cs.det4 = (float)det4;
    if constexpr (FP64) {
        const double t = log2(255.0 * (double)op) + kCullMargin;
        cs.mode = t <= 0.0 ? 2 : 1;
        if (cs.mode == 2) return cs;
        const double ia = 0.5 / (double)a, ic = 0.5 / (double)c, t4 = 4.0 * t / det4;
        const double y_full = sqrt((double)a * t4), x_ext = sqrt((double)c * t4);
        cs.inv2a = (float)ia;
        cs.four_at = (float)(4.0 * (double)a * t);
        cs.y_full = (float)y_full;
        cs.y_ext = (float)((double)b * x_ext * ic);
        cs.pad_y = (float)(2e-3 * y_full + 1e-2);
        cs.pad_x = (float)(2e-3 * (x_ext + fabs((double)b) * y_full * ia) + 1e-2);
    } else {
        // (a centre that is not a number fails no test of the blending's: keep it)
        if (!(fabsf(cs.uf) <= 1.f && fabsf(cs.vf) <= 1.f)) return cs;
        const float t = log2f(255.f * op) + (float)kCullMargin;
        cs.mode = t <= 0.f ? 2 : 1;
        if (cs.mode == 2) return cs;
        const float t4 = 4.f * t * cull_rcp(cs.det4), x_ext = cull_root(fminf(fmaxf(kRootLeast, c * t4), kRootMost));
        cs.inv2a = 0.5f * cull_rcp(a);
        cs.four_at = 4.f * a * t;
        cs.y_full = cull_root(fminf(fmaxf(kRootLeast, a * t4), kRootMost));
        cs.y_ext = 0.5f * b * x_ext * cull_rcp(c);
        cs.pad_y = 2e-3f * cs.y_full + 1e-2f;
        cs.pad_x = 2e-3f * (x_ext + fabsf(b) * cs.y_full * cs.inv2a) + 1e-2f;
    }
    return cs;
}

// The tests below compare pixel centres with the ellipse's extents: a tile
// column is kept when its last pixel centre (inside the splat's square) is not
// left of the extent and its first not right of it.  Centres are integers plus
// the splat's fractional offset, so both ends become integer pixels once per
// row and the rest is integer arithmetic.  (No contraction: every kernel that
// evaluates a test decides alike.)
// First pixel whose centre lies at or past centre + x, and last at or before it,
// as whole numbers (i: integer part of the centre, f: fractional part).
// The sum of the two whole numbers is exact wherever it lies near the image,
// however far off the centre is and the ellipse reaches (each is a multiple of its
// own unit in the last place); beyond, only its side counts.
__host__ __device__ __forceinline__ float first_pixel(float i, float f, float x) {
#pragma clang fp contract(off)
    return i + ceilf(x + f - 0.5f);
}
__host__ __device__ __forceinline__ float last_pixel(float i, float f, float x) {
#pragma clang fp contract(off)
    return i + floorf(x + f - 0.5f);
}
// Such a number as an integer; what is not a number counts as far right (left).
__host__ __device__ __forceinline__ int to_right(float p) { return (int)fmaxf(fminf(p, 1e9f), -1e9f); }
__host__ __device__ __forceinline__ int to_left(float p) { return (int)fminf(fmaxf(p, -1e9f), 1e9f); }
// The tile that holds pixel p (rounded down for pixels left of the image).
template <int TILE>
__host__ __device__ __forceinline__ int tile_of(int p) {
    return p >> (TILE == 8 ? 3 : TILE == 16 ? 4 : 5);
}
// Pixel-centre offsets of the first and last pixel row of tile row ty inside
// the splat's square.
template <int TILE>
__host__ __device__ __forceinline__ float row_y0(const CullShape& cs, int ty) {
#pragma clang fp contract(off)
    return ((float)max(ty * TILE, cs.py0) + 0.5f - cs.vi) - cs.vf;
}
template <int TILE>
__host__ __device__ __forceinline__ float row_y1(const CullShape& cs, int ty) {
#pragma clang fp contract(off)
    return ((float)min(ty * TILE + TILE - 1, cs.py1) + 0.5f - cs.vi) - cs.vf;
}
// The tile rows [r0, r1] of [ty0, ty1] whose slab of pixel centres meets the
// ellipse's height, widened by pad_y (r1 < r0: none; all for a height or a centre that
// is not a number).
template <int TILE>
__host__ __device__ __forceinline__ void slab_rows(const CullShape& cs, int ty0, int ty1, int& r0, int& r1) {
#pragma clang fp contract(off)
    const float h = cs.y_full + cs.pad_y;
    const int lo = to_left(first_pixel(cs.vi, cs.vf, -h)), hi = to_right(last_pixel(cs.vi, cs.vf, h));
    r0 = max(ty0, tile_of<TILE>(lo));
    r1 = min(ty1, tile_of<TILE>(hi));
    if (lo > cs.py1 || hi < cs.py0) r1 = r0 - 1;
}
// The ellipse's x-extent [xl, xr] over tile row ty's slab (from its leftmost
// and rightmost points clamped into the slab), widened by pad_x.
template <int TILE>
__host__ __device__ __forceinline__ void row_extent(const CullShape& cs, int ty, float& xl, float& xr) {
#pragma clang fp contract(off)
    const float Y0 = row_y0<TILE>(cs, ty), Y1 = row_y1<TILE>(cs, ty);
    const float yr = fminf(fmaxf(cs.y_ext, Y0), Y1), yl = fminf(fmaxf(-cs.y_ext, Y0), Y1);
    xr = (cs.b * yr + cull_root(fmaxf(kRootLeast, cs.four_at - yr * yr * cs.det4))) * cs.inv2a + cs.pad_x;
    xl = (cs.b * yl - cull_root(fmaxf(kRootLeast, cs.four_at - yl * yl * cs.det4))) * cs.inv2a - cs.pad_x;
}
// The tile columns of tile row ty (one of slab_rows') that the test keeps, as
// one word: first column | (last + 1) << 16 (0: none, also for an extent or a centre
// that is not a number).
template <int TILE>
__host__ __device__ __forceinline__ uint32_t row_columns(const CullShape& cs, int ty, int tx0, int tx1) {
    float xl, xr;
    row_extent<TILE>(cs, ty, xl, xr);
    const int lo = to_right(first_pixel(cs.ui, cs.uf, xl)), hi = to_left(last_pixel(cs.ui, cs.uf, xr));
    const int cl = max(tx0, tile_of<TILE>(lo)), cr = min(tx1, tile_of<TILE>(hi));
    return lo <= cs.px1 && hi >= cs.px0 && cl <= cr ? (uint32_t)cl | ((uint32_t)(cr + 1) << 16) : 0u;
}
// The same for any tile row.
template <int TILE>
__host__ __device__ __forceinline__ uint32_t row_span(const CullShape& cs, int ty, int tx0, int tx1) {
    int r0, r1;
    slab_rows<TILE>(cs, ty, ty, r0, r1);
    return r0 <= r1 ? row_columns<TILE>(cs, ty, tx0, tx1) : 0u;
}

// Tiles (bit ly * S + lx) of the super-tile at tile origin (bx, by) that the
// splat's tile rectangle [tx0, tx1] x [ty0, ty1] overlaps and, when cull is
// set, the rows' tests keep (per entry: splats taller than the span table).
template <int TILE>
__host__ __device__ inline uint32_t tile_mask(const CullShape& cs, bool cull, uint32_t tx0, uint32_t tx1, uint32_t ty0,
                                     uint32_t ty1, uint32_t bx, uint32_t by) {
    constexpr uint32_t S = (uint32_t)super_factor(TILE);
    uint32_t mask = 0u;
#pragma unroll
    for (uint32_t ly = 0; ly < S; ++ly) {
        const uint32_t ty = by + ly;
        if (ty < ty0 || ty > ty1) continue;
        const uint32_t e = cull ? row_span<TILE>(cs, (int)ty, (int)tx0, (int)tx1) : tx0 | ((tx1 + 1u) << 16);
        const uint32_t lo = max(e & 0xFFFFu, bx), hi = min(e >> 16, bx + S);
        mask |= lo < hi ? ((1u << (hi - bx)) - (1u << (lo - bx))) << (ly * S) : 0u;
    }
    return mask;
}

}  // namespace h4d

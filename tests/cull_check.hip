// Host-side check of the tile test against the blending rule in FP64 (built and
// run by test_cull_reach.py; no GPU is used).  For random splats of one kind it
// goes through every pixel of the splat's square in every tile that tile_mask
// leaves out and counts those that would blend: power <= 0 and opacity
// exp(power) >= 1/255, the power evaluated in FP64 from the record's float32 values
// or as the kernels do in FP32.  It also counts the ellipses whose extents are not
// their FP64 values rounded to float32 (to a unit in the last place; not for the
// quadrants' shapes).  Prints "kind K tile T dropped D blending B rounded R" per kind
// of splat and tile size.
#include "../paper_2505_13215_amd/csrc/sort.hip"

#include <algorithm>
#include <cmath>
#include <cstdio>
#include <random>

using namespace h4d;

// A splat: centre and covariance as the projection has them.
struct Splat2 {
    double u, v, l1, l2, angle;  // squared half-axes, the first one's angle
};
struct Kind {
    const char* name;
    int W, H;
    Splat2 (*draw)(std::mt19937_64&, int W, int H);
};
static double uni(std::mt19937_64& g) { return std::uniform_real_distribution<double>(0.0, 1.0)(g); }
static double log_uni(std::mt19937_64& g, double a, double b) {
    return std::exp(std::log(a) + uni(g) * (std::log(b) - std::log(a)));
}
static Splat2 near_image(std::mt19937_64& g, int W, int H) {
    const double l1 = log_uni(g, 0.05, uni(g) < 0.05 ? 40000.0 : 400.0);
    return {-80.0 + uni(g) * (W + 160), -80.0 + uni(g) * (H + 160), l1, l1 * log_uni(g, 1e-3, 1.0), uni(g) * 3.141592653589793};
}
// needles: half-axes from a few pixels to far beyond the image, thin down to the dilation
static Splat2 thin(std::mt19937_64& g, int W, int H) {
    return {uni(g) * W, uni(g) * H, log_uni(g, 10.0, 1e7), log_uni(g, 1e-4, 1.0), uni(g) * 3.141592653589793};
}
// centres off the image by more than a float32 holds to the pixel, ellipses that reach it or just miss
template <int LG>
static Splat2 far_off(std::mt19937_64& g, int W, int H) {
    const double d = log_uni(g, std::pow(10.0, LG), std::pow(10.0, LG + 1)), th = uni(g) * 6.283185307179586;
    const double a = d * (0.4 + 3.0 * uni(g));
    return {0.5 * W + d * std::cos(th), 0.5 * H + d * std::sin(th), a * a, a * a * log_uni(g, 1e-2, 1.0),
            uni(g) * 3.141592653589793};
}

// The power as the blending kernels evaluate it (eval_col, eval_pix).
static float kernel_power(const Rec& r, int px, int py) {
#pragma clang fp contract(off)
    const float dx = (((float)px + 0.5f) - r.c.y) - r.a.x, dy = (((float)py + 0.5f) - r.c.z) - r.a.y;
    const float qadx = r.a.z * dx;
    return std::fmaf(dy, std::fmaf(r.b.x, dy, r.a.w * dx), qadx * dx);
}

// FP64: as the binning sets the shapes up; otherwise as the quadrant kernels do.
template <int TILE, bool FP64 = true>
static void check(const Kind& kind, int splats) {
    constexpr int S = super_factor(TILE);
    std::mt19937_64 g(20250513);
    const int W = kind.W, H = kind.H;
    long dropped = 0, blending = 0, rounded = 0;
    for (int it = 0; it < splats; ++it) {
        const Splat2 z = kind.draw(g, W, H);
        const double c = std::cos(z.angle), s = std::sin(z.angle);
        const double sa = c * c * z.l1 + s * s * z.l2 + 0.3, sb = c * s * (z.l1 - z.l2), sc = s * s * z.l1 + c * c * z.l2 + 0.3;
        // (the determinant from the axes: sa sc - sb sb cancels for needles)
        const double det = (z.l1 + 0.3) * (z.l2 + 0.3), k = -0.5 * 1.4426950408889634;
        const double r = std::ceil(3.0 * std::sqrt(std::max(z.l1, z.l2) + 0.3));
        const int x0 = (int)std::max(0.0, std::ceil(z.u - r - 0.5)), x1 = (int)std::min(W - 1.0, std::floor(z.u + r - 0.5));
        const int y0 = (int)std::max(0.0, std::ceil(z.v - r - 0.5)), y1 = (int)std::min(H - 1.0, std::floor(z.v + r - 0.5));
        if (x0 > x1 || y0 > y1) continue;
        const double fu = std::floor(z.u), fv = std::floor(z.v), op = uni(g) < 0.1 ? 0.01 * uni(g) : uni(g);
        Rec rec;
        rec.a = make_float4((float)(z.u - fu), (float)(z.v - fv), (float)(sc / det * k), (float)(-sb / det * 2.0 * k));
        rec.b = make_float4((float)(sa / det * k), (float)op, 0.f, 0.f);
        rec.c = make_float4(0.f, (float)fu, (float)fv, 1.f);
        rec.d = make_uint4((uint32_t)x0 | ((uint32_t)x1 << 16), (uint32_t)y0 | ((uint32_t)y1 << 16), 1u, 1u);
        const CullShape cs = cull_shape<FP64>(rec);
        if (FP64 && cs.mode == 1) {
            const double a = -(double)rec.a.z, b = rec.a.w, cc = -(double)rec.b.x, det4 = 4.0 * a * cc - b * b;
            const double t = std::log2(255.0 * (double)rec.b.y) + kCullMargin;
            const double y_full = std::sqrt(4.0 * a * t / det4), x_ext = std::sqrt(4.0 * cc * t / det4);
            const auto off = [](float f, double x) { return std::fabs(f - x) > std::ldexp(std::fabs(x), -23); };
            rounded += off(cs.y_full, y_full) || off(cs.four_at, 4.0 * a * t) || off(cs.inv2a, 0.5 / a) ||
                       off(cs.y_ext, 0.5 * b * x_ext / cc);
        }
        const uint32_t tx0 = x0 / TILE, tx1 = x1 / TILE, ty0 = y0 / TILE, ty1 = y1 / TILE;
        for (uint32_t ty = ty0; ty <= ty1; ++ty)
            for (uint32_t tx = tx0; tx <= tx1; ++tx) {
                const uint32_t m =
                    cs.mode == 2 ? 0u : tile_mask<TILE>(cs, cs.mode == 1, tx0, tx1, ty0, ty1, tx / S * S, ty / S * S);
                if ((m >> ((ty % S) * S + tx % S)) & 1u) continue;
                for (int py = std::max(y0, (int)ty * TILE); py <= std::min(y1, (int)ty * TILE + TILE - 1); ++py)
                    for (int px = std::max(x0, (int)tx * TILE); px <= std::min(x1, (int)tx * TILE + TILE - 1); ++px) {
                        const double dx = px + 0.5 - rec.c.y - (double)rec.a.x, dy = py + 0.5 - rec.c.z - (double)rec.a.y;
                        const double p2 = (double)rec.a.z * dx * dx + (double)rec.a.w * dx * dy + (double)rec.b.x * dy * dy;
                        ++dropped;
                        const auto blends = [&](double power) {
                            return power <= 0.0 && power + std::log2((double)rec.b.y) >= -std::log2(255.0);
                        };
                        if (blends(p2) || blends(kernel_power(rec, px, py))) ++blending;
                    }
            }
    }
    std::printf("kind %s%s tile %d dropped %ld blending %ld rounded %ld\n", kind.name, FP64 ? "" : "-quadrants", TILE, dropped, blending, rounded);
}

int main(int argc, char** argv) {
    const int splats = argc > 1 ? std::atoi(argv[1]) : 4000;
    const Kind kinds[] = {{"near", 640, 480, near_image},   {"thin", 640, 480, thin},
                          {"far4", 160, 120, far_off<4>},   {"far6", 160, 120, far_off<6>},
                          {"far7", 160, 120, far_off<7>},   {"far8", 160, 120, far_off<8>}};
    for (const Kind& k : kinds) {
        check<8>(k, splats);
        check<16>(k, splats);
        check<32>(k, splats);
        check<8, false>(k, splats);
    }
    return 0;
}

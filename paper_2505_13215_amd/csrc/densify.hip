// Adaptive densification and pruning on gfx950, applied to the static 3D and
// the dynamic 4D set separately (Sec. 4.3, which adopts the clone / split /
// prune scheme of 3D Gaussian Splatting): per row a selection from the
// accumulated image-plane gradient, clone or split by the largest spatial
// scale, prune by opacity and size; then three stable compactions (kept
// originals, clones, split children) and a scatter of the output rows.
// Decisions compare float32 values widened to double against double limits,
// so they are exact; split children are placed in FP64.
#include "common.hpp"
#include "launch.hpp"
#include "rotation.hpp"

namespace h4d {

struct RowFlags {
    bool keep_orig, keep_clone, keep_child;
};

// Decisions of one row.  ls: its three spatial log-scales; opacity: its logit.
__device__ inline RowFlags densify_row(const DensifyP& p, float grad, float vis, const float* ls, float opacity) {
    const bool sel = vis > 0.0f && (double)grad >= (double)p.thr * (double)vis;
    double L = (double)ls[0], Lc = (double)(float)((double)ls[0] - p.log_shrink);
    for (int k = 1; k < 3; ++k) {
        L = fmax(L, (double)ls[k]);
        Lc = fmax(Lc, (double)(float)((double)ls[k] - p.log_shrink));
    }
    const bool large = L > p.log_dense;
    const bool low = (double)opacity < p.logit_min;
    const bool pr = low || L > p.log_max_scale;
    const bool prc = low || Lc > p.log_max_scale;
    RowFlags f;
    f.keep_orig = !(sel && large) && !pr;
    f.keep_clone = sel && !large && !pr;
    f.keep_child = sel && large && !prc;
    return f;
}

// Flags of row i of set d.
__device__ __forceinline__ RowFlags densify_flags(const DensifySet& d, int i) {
    float ls[3];
    for (int k = 0; k < 3; ++k) ls[k] = d.log_scale[(size_t)k * d.n + i];
    return densify_row(d.p, d.grad[i], d.vis[i], ls, d.opacity[i]);
}

// Kept originals, clones and split rows of each block of kScanTile rows.
// blockIdx.y: the set; partials: [3][blocks] per set.
__global__ void __launch_bounds__(256) k_densify_count(DensifySets sets) {
    __shared__ uint32_t s_c[3][4];
    const DensifySet& d = sets.s[blockIdx.y];
    if ((int)blockIdx.x * kScanTile >= d.n) return;  // uniform
    uint32_t c[3] = {0u, 0u, 0u};
#pragma unroll
    for (int k = 0; k < kScanTile / 256; ++k) {
        const int i = blockIdx.x * kScanTile + k * 256 + (int)threadIdx.x;
        RowFlags f{false, false, false};
        if (i < d.n) f = densify_flags(d, i);
        c[0] += (uint32_t)__popcll(__ballot(f.keep_orig));
        c[1] += (uint32_t)__popcll(__ballot(f.keep_clone));
        c[2] += (uint32_t)__popcll(__ballot(f.keep_child));
    }
    if ((threadIdx.x & 63) == 0)
        for (int q = 0; q < 3; ++q) s_c[q][threadIdx.x >> 6] = c[q];
    __syncthreads();
    if (threadIdx.x < 3) {
        const uint32_t* t = s_c[threadIdx.x];
        d.partials[(size_t)threadIdx.x * d.stride + blockIdx.x] = (unsigned long long)(t[0] + t[1] + t[2] + t[3]);
    }
}

// Source row of every output row (kept originals, then clones, then the
// children, child k of every split row after child k - 1 of all of them):
// itself, or -(1 + parent).  partials scanned.
__global__ void __launch_bounds__(256) k_densify_src(DensifySets sets) {
    constexpr int R = kScanTile / 256;
    __shared__ uint32_t s_c[3][R * 4];  // rows per (round, wave), in row order
    const DensifySet& d = sets.s[blockIdx.y];
    if ((int)blockIdx.x * kScanTile >= d.n) return;  // uniform
    const int tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
    unsigned long long m[3][R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int i = blockIdx.x * kScanTile + k * 256 + tid;
        RowFlags f{false, false, false};
        if (i < d.n) f = densify_flags(d, i);
        m[0][k] = __ballot(f.keep_orig);
        m[1][k] = __ballot(f.keep_clone);
        m[2][k] = __ballot(f.keep_child);
        if (lane < 3) s_c[lane][k * 4 + w] = (uint32_t)__popcll(lane == 0 ? m[0][k] : lane == 1 ? m[1][k] : m[2][k]);
    }
    __syncthreads();
    const size_t K0 = d.k0, K1 = d.k1, K2 = d.k2;
    // (counts of these inputs; a caller's others place nothing outside)
    const auto put = [&](size_t r, size_t end, int32_t v) {
        if (r < end) d.src[r] = v;
    };
    size_t run[3];
    for (int q = 0; q < 3; ++q) run[q] = (size_t)d.partials[(size_t)q * d.stride + blockIdx.x];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int i = blockIdx.x * kScanTile + k * 256 + tid;
        size_t at[3];
        for (int q = 0; q < 3; ++q) {
            at[q] = run[q] + (size_t)__popcll(m[q][k] & ((1ull << lane) - 1ull));
            for (int u = 0; u < 4; ++u) {
                if (u < w) at[q] += s_c[q][k * 4 + u];
                run[q] += s_c[q][k * 4 + u];
            }
        }
        if ((m[0][k] >> lane) & 1ull) put(at[0], K0, i);
        if ((m[1][k] >> lane) & 1ull) put(K0 + at[1], K0 + K1, -1 - i);
        if ((m[2][k] >> lane) & 1ull)
            for (int c = 0; c < d.p.split_n; ++c) put(K0 + K1 + (size_t)c * K2 + at[2], K0 + K1 + (size_t)(c + 1) * K2, -1 - i);
    }
}

// Centres and log-scales of the children (one per thread).  noise:
// [split_n][3][n] standard normal draws
__global__ void __launch_bounds__(256) k_densify_children3(G3Ptr g, const int32_t* __restrict__ src, int first, int k2,
                                                           const float* __restrict__ noise, DensifyP p, G3Grad o) {
    const int ch = blockIdx.x * 256 + (int)threadIdx.x;
    if (ch >= k2 * p.split_n) return;
    const size_t n = (size_t)g.n, no = (size_t)o.n, r = (size_t)first + ch;
    const int i = -1 - src[r], c = ch / k2;
    if (i < 0 || i >= g.n) return;  // (never so: a child's source is its parent)
    double q[4], R[3][3], z[3];
    load_unit4(g.quat, g.n, i, q);
    quat_rot3(q, R);
    for (int k = 0; k < 3; ++k) z[k] = exp((double)g.log_scale[k * n + i]) * (double)noise[((size_t)c * 3 + k) * n + i];
    for (int a = 0; a < 3; ++a)
        o.mean[a * no + r] = (float)((double)g.mean[a * n + i] + R[a][0] * z[0] + R[a][1] * z[1] + R[a][2] * z[2]);
    for (int k = 0; k < 3; ++k) o.log_scale[k * no + r] = (float)((double)g.log_scale[k * n + i] - p.log_shrink);
}

// noise: [split_n][4][n]; children move in space and time along R_l R_r (Eq. 4)
__global__ void __launch_bounds__(256) k_densify_children4(G4Ptr g, const int32_t* __restrict__ src, int first, int k2,
                                                           const float* __restrict__ noise, DensifyP p, G4Grad o) {
    const int ch = blockIdx.x * 256 + (int)threadIdx.x;
    if (ch >= k2 * p.split_n) return;
    const size_t n = (size_t)g.n, no = (size_t)o.n, r = (size_t)first + ch;
    const int i = -1 - src[r], c = ch / k2;
    if (i < 0 || i >= g.n) return;  // (never so: a child's source is its parent)
    double ql[4], qr[4], L[4][4], Rr[4][4], z[4], d[4];
    load_unit4(g.quat_l, g.n, i, ql);
    load_unit4(g.quat_r, g.n, i, qr);
    rot_left(ql, L);
    rot_right(qr, Rr);
    for (int k = 0; k < 4; ++k) z[k] = exp((double)g.log_scale[k * n + i]) * (double)noise[((size_t)c * 4 + k) * n + i];
    for (int a = 0; a < 4; ++a) {
        double R[4];
        for (int b = 0; b < 4; ++b) {
            double acc = 0.0;
            for (int k = 0; k < 4; ++k) acc += L[a][k] * Rr[k][b];
            R[b] = acc;
        }
        d[a] = R[0] * z[0] + R[1] * z[1] + R[2] * z[2] + R[3] * z[3];
    }
    for (int a = 0; a < 3; ++a) o.mean[a * no + r] = (float)((double)g.mean[a * n + i] + d[a]);
    o.mean_t[r] = (float)((double)g.mean_t[i] + d[3]);
    for (int k = 0; k < 4; ++k) o.log_scale[k * no + r] = (float)((double)g.log_scale[k * n + i] - p.log_shrink);
}

// The rows of each kind of both sets: counted, and scanned over the blocks.
void launch_densify_plan(const DensifySets& s, hipStream_t st) {
    const int nb = std::max(scan_blocks(s.s[0].n), scan_blocks(s.s[1].n));
    if (nb > 0) k_densify_count<<<dim3((unsigned)nb, 2), 256, 0, st>>>(s);
    for (int q = 0; q < 2; ++q)
        launch_scan_top(s.s[q].partials, scan_blocks(s.s[q].n), 3, s.s[q].stride, s.s[q].totals, st);
}

// The source rows (k0, k1, k2 of s filled in), the rows gathered and the
// children placed.
void launch_densify_rows(const DensifySets& s, const G3Ptr& g3, const G4Ptr& g4, const float* noise3,
                         const float* noise4, const G3Grad& o3, const G4Grad& o4, hipStream_t st) {
    const int nb = std::max(scan_blocks(s.s[0].n), scan_blocks(s.s[1].n));
    if (nb > 0) k_densify_src<<<dim3((unsigned)nb, 2), 256, 0, st>>>(s);
    const DensifySet &a = s.s[0], &b = s.s[1];
    const int f3 = a.k0 + a.k1, c3 = a.k2 * a.p.split_n, f4 = b.k0 + b.k1, c4 = b.k2 * b.p.split_n;
    launch_rows_gather(slabs3(g3, o3, f3), a.src, f3 + c3, kNegativeParent, st);
    launch_rows_gather(slabs4(g4, o4, nullptr, f4), b.src, f4 + c4, kNegativeParent, st);
    if (c3 > 0) k_densify_children3<<<ceil_div(c3, 256), 256, 0, st>>>(g3, a.src, f3, a.k2, noise3, a.p, o3);
    if (c4 > 0) k_densify_children4<<<ceil_div(c4, 256), 256, 0, st>>>(g4, b.src, f4, b.k2, noise4, b.p, o4);
}

// Rows of the optimiser state after densification: out row r takes in row
// src[r] (src >= 0) or zeros (a new row).
void launch_gather_rows(const G3Ptr& g3, const int32_t* src3, int rows3, const G3Grad& o3, const G4Ptr& g4,
                        const int32_t* src4, int rows4, const G4Grad& o4, hipStream_t st) {
    launch_rows_gather(slabs3(g3, o3, INT32_MAX), src3, rows3, kNegativeZero, st);
    launch_rows_gather(slabs4(g4, o4, nullptr, INT32_MAX), src4, rows4, kNegativeZero, st);
}

}  // namespace h4d

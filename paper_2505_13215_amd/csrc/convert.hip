// Static identification and 4D -> 3D conversion on gfx950 (Sec. 4.1-4.2,
// Eq. 7-9): mask, stable compaction of the 4D set, append of the converted rows
// to the 3D set with the Eq. 9 quaternion of the spatial rotation block.  A
// converted row keeps its time-independent SH coefficients; its time
// coefficients (if any) are dropped with the time axis.
#include "common.hpp"
#include "launch.hpp"

namespace h4d {

// Row i is converted iff (double)s_t > log((double)tau).
__device__ __forceinline__ bool is_static(const float* __restrict__ ls4, int n4, int i, double log_tau) {
    return (double)ls4[(size_t)3 * n4 + i] > log_tau;
}

// The row order is found in three small launches: the converted rows of each
// block of kScanTile, their scan, and perm (kept rows need no scan of their own:
// a row's kept predecessors are those that are not converted).
__global__ void __launch_bounds__(256) k_convert_count(const float* __restrict__ ls4, int n4, double log_tau,
                                                       unsigned long long* __restrict__ partials) {
    __shared__ uint32_t s_c[4];
    uint32_t c = 0;
#pragma unroll
    for (int k = 0; k < kScanTile / 256; ++k) {
        const int i = blockIdx.x * kScanTile + k * 256 + (int)threadIdx.x;
        c += (uint32_t)__popcll(__ballot(i < n4 && is_static(ls4, n4, i, log_tau)));
    }
    if ((threadIdx.x & 63) == 0) s_c[threadIdx.x >> 6] = c;
    __syncthreads();
    if (threadIdx.x == 0) partials[blockIdx.x] = (unsigned long long)(s_c[0] + s_c[1] + s_c[2] + s_c[3]);
}

// perm[i] = new 4D row, or -(1 + new 3D row); partials scanned.
__global__ void __launch_bounds__(256) k_convert_perm(const float* __restrict__ ls4, int n4, double log_tau, int n3,
                                                      const unsigned long long* __restrict__ partials,
                                                      int32_t* __restrict__ perm) {
    constexpr int R = kScanTile / 256;
    __shared__ uint32_t s_c[R * 4];  // converted rows per (round, wave), in row order
    const int tid = (int)threadIdx.x, lane = tid & 63, w = tid >> 6;
    unsigned long long m[R];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        const int i = blockIdx.x * kScanTile + k * 256 + tid;
        m[k] = __ballot(i < n4 && is_static(ls4, n4, i, log_tau));
        if (lane == 0) s_c[k * 4 + w] = (uint32_t)__popcll(m[k]);
    }
    __syncthreads();
    uint32_t run = (uint32_t)partials[blockIdx.x];
#pragma unroll
    for (int k = 0; k < R; ++k) {
        uint32_t before = run;
        for (int q = 0; q < 4; ++q) {
            if (q < w) before += s_c[k * 4 + q];
            run += s_c[k * 4 + q];
        }
        const int i = blockIdx.x * kScanTile + k * 256 + tid;
        const uint32_t off = before + (uint32_t)__popcll(m[k] & ((1ull << lane) - 1ull));
        if (i < n4) perm[i] = ((m[k] >> lane) & 1ull) ? -(int32_t)(1u + (uint32_t)n3 + off) : (int32_t)((uint32_t)i - off);
    }
}

__device__ inline void mat2quat(const double R[3][3], double q[4]) {
    const double tr = R[0][0] + R[1][1] + R[2][2];
    if (1.0 + tr > 1e-6) {
        const double w = 0.5 * sqrt(1.0 + tr);
        const double i4w = 1.0 / (4.0 * w);
        q[0] = w;
        q[1] = (R[2][1] - R[1][2]) * i4w;
        q[2] = (R[0][2] - R[2][0]) * i4w;
        q[3] = (R[1][0] - R[0][1]) * i4w;
        return;
    }
    // largest-diagonal branch (Shepperd) where the printed formula degenerates
    if (R[0][0] >= R[1][1] && R[0][0] >= R[2][2]) {
        const double x = 0.5 * sqrt(fmax(0.0, 1.0 + R[0][0] - R[1][1] - R[2][2]));
        const double i4 = 1.0 / (4.0 * x);
        q[1] = x; q[0] = (R[2][1] - R[1][2]) * i4; q[2] = (R[0][1] + R[1][0]) * i4; q[3] = (R[0][2] + R[2][0]) * i4;
    } else if (R[1][1] >= R[2][2]) {
        const double y = 0.5 * sqrt(fmax(0.0, 1.0 - R[0][0] + R[1][1] - R[2][2]));
        const double i4 = 1.0 / (4.0 * y);
        q[2] = y; q[0] = (R[0][2] - R[2][0]) * i4; q[1] = (R[0][1] + R[1][0]) * i4; q[3] = (R[1][2] + R[2][1]) * i4;
    } else {
        const double z = 0.5 * sqrt(fmax(0.0, 1.0 - R[0][0] - R[1][1] + R[2][2]));
        const double i4 = 1.0 / (4.0 * z);
        q[3] = z; q[0] = (R[1][0] - R[0][1]) * i4; q[1] = (R[0][2] + R[2][0]) * i4; q[2] = (R[1][2] + R[2][1]) * i4;
    }
}

__device__ inline void unit4(const float* q, int n, int i, double o[4]) {
    double a[4];
    for (int k = 0; k < 4; ++k) a[k] = (double)q[(size_t)k * n + i];
    const double inv = 1.0 / sqrt(a[0] * a[0] + a[1] * a[1] + a[2] * a[2] + a[3] * a[3]);
    for (int k = 0; k < 4; ++k) o[k] = a[k] * inv;
}

// ---------------------------------------------------------------------------
// Moving rows of component-major arrays.
// ---------------------------------------------------------------------------
// Bound by memory: 4 bytes per component and row, in and out.  A row per thread
// with its 59 or 65 components one after another kept one load in flight and
// a sixteenth of the chip's waves busy; here blockIdx.y takes a slab of up to
// eight components, all loaded before any is stored, so a launch has ten times
// the waves and eight loads in flight each.  Rows go to outputs of the exact size
// instead of being copied out of larger ones afterwards.  500k 4D rows, half of
// them converted, 250 MB: 0.062 ms (4.1 TB/s); the densified rows of 175k 3D and
// 75k 4D Gaussians 0.030 + 0.016 ms, from 0.090 + 0.077 ms and a copy.
__global__ void __launch_bounds__(256) k_rows_gather(RowSlabs t, const int32_t* __restrict__ src, int rows,
                                                     int negative) {
    const RowSlab& s = t.s[blockIdx.y];
    const int r = blockIdx.x * 256 + (int)threadIdx.x;
    if (r >= rows || r >= s.limit) return;
    int32_t i = src ? src[r] : r;
    if (negative == kNegativeParent && i < 0) i = -1 - i;
    const bool ok = i >= 0 && (size_t)i < t.ni;
    float v[kSlabComps];
#pragma unroll
    for (int k = 0; k < kSlabComps; ++k) v[k] = (ok && k < s.comps) ? s.in[(size_t)k * t.ni + i] : 0.0f;
#pragma unroll
    for (int k = 0; k < kSlabComps; ++k)
        if (k < s.comps) s.out[(size_t)k * t.no + r] = v[k];
}

// Rows of the 4D set to their places: perm >= 0 to out4's row, else to out3's
// (the components both sets have).
__global__ void __launch_bounds__(256) k_rows_split(RowSlabs t, const int32_t* __restrict__ perm, int n4) {
    const RowSlab& s = t.s[blockIdx.y];
    const int i = blockIdx.x * 256 + (int)threadIdx.x;
    if (i >= n4) return;
    const int32_t p = perm[i];
    const bool conv = p < 0;
    const size_t r = conv ? (size_t)(-1 - (int64_t)p) : (size_t)p;
    float* out = conv ? s.out3 : s.out;
    const size_t no = conv ? t.no3 : t.no;
    const int comps = conv ? s.comps3 : s.comps;
    if (r >= no) return;  // (never so for a perm of the same sets)
    float v[kSlabComps];
#pragma unroll
    for (int k = 0; k < kSlabComps; ++k) v[k] = k < comps ? s.in[(size_t)k * t.ni + i] : 0.0f;
#pragma unroll
    for (int k = 0; k < kSlabComps; ++k)
        if (k < comps) out[(size_t)k * no + r] = v[k];
}

// Eq. 8-9: the converted rows' quaternions, of the top-left 3x3 block of R_l
// R_r; zeros for moments.
__global__ void __launch_bounds__(256) k_convert_quat(const float* __restrict__ ql, const float* __restrict__ qr, int n4,
                                                      const int32_t* __restrict__ perm, float* __restrict__ quat3,
                                                      size_t no, int zero) {
    const int i = blockIdx.x * 256 + (int)threadIdx.x;
    if (i >= n4) return;
    const int32_t p = perm[i];
    if (p >= 0) return;
    const size_t r = (size_t)(-1 - (int64_t)p);
    if (r >= no) return;
    double q[4] = {0.0, 0.0, 0.0, 0.0};
    if (!zero) {
        double a[4], b[4];
        unit4(ql, n4, i, a);
        unit4(qr, n4, i, b);
        const double L[4][4] = {{a[0], -a[1], -a[2], -a[3]}, {a[1], a[0], -a[3], a[2]},
                                {a[2], a[3], a[0], -a[1]}, {a[3], -a[2], a[1], a[0]}};
        const double Rr[4][4] = {{b[0], -b[1], -b[2], -b[3]}, {b[1], b[0], b[3], -b[2]},
                                 {b[2], -b[3], b[0], b[1]}, {b[3], b[2], -b[1], b[0]}};
        double R3[3][3];
        for (int r2 = 0; r2 < 3; ++r2)
            for (int c = 0; c < 3; ++c) {
                double acc = 0;
                for (int k = 0; k < 4; ++k) acc += L[r2][k] * Rr[k][c];
                R3[r2][c] = acc;
            }
        mat2quat(R3, q);
    }
    for (int k = 0; k < 4; ++k) quat3[k * no + r] = (float)q[k];
}

namespace {
// Adds the slabs of one array of `comps` components to t.
void add_slabs(RowSlabs& t, const float* in, float* out, float* out3, int comps, int comps3, int limit) {
    for (int c = 0; c < comps; c += kSlabComps) {
        RowSlab& s = t.s[t.n++];
        s.in = in + (size_t)c * t.ni;
        s.out = out ? out + (size_t)c * t.no : nullptr;
        s.out3 = out3 ? out3 + (size_t)c * t.no3 : nullptr;
        s.comps = std::min(kSlabComps, comps - c);
        s.comps3 = out3 ? std::max(0, std::min(kSlabComps, comps3 - c)) : 0;
        s.limit = limit;
    }
}
}  // namespace

// placed: rows from there on take their means and log-scales elsewhere.
RowSlabs slabs3(const G3Ptr& in, const G3Grad& out, int placed) {
    RowSlabs t{};
    t.ni = (size_t)in.n;
    t.no = (size_t)out.n;
    add_slabs(t, in.mean, out.mean, nullptr, 3, 0, placed);
    add_slabs(t, in.log_scale, out.log_scale, nullptr, 3, 0, placed);
    add_slabs(t, in.quat, out.quat, nullptr, 4, 0, INT32_MAX);
    add_slabs(t, in.opacity, out.opacity, nullptr, 1, 0, INT32_MAX);
    add_slabs(t, in.sh, out.sh, nullptr, 48, 0, INT32_MAX);
    return t;
}
RowSlabs slabs4(const G4Ptr& in, const G4Grad& out, const G3Grad* out3, int placed) {
    RowSlabs t{};
    t.ni = (size_t)in.n;
    t.no = (size_t)out.n;
    t.no3 = out3 ? (size_t)out3->n : 0;
    add_slabs(t, in.mean, out.mean, out3 ? out3->mean : nullptr, 3, 3, placed);
    add_slabs(t, in.mean_t, out.mean_t, nullptr, 1, 0, placed);
    add_slabs(t, in.log_scale, out.log_scale, out3 ? out3->log_scale : nullptr, 4, 3, placed);
    add_slabs(t, in.quat_l, out.quat_l, nullptr, 4, 0, INT32_MAX);
    add_slabs(t, in.quat_r, out.quat_r, nullptr, 4, 0, INT32_MAX);
    add_slabs(t, in.opacity, out.opacity, out3 ? out3->opacity : nullptr, 1, 1, INT32_MAX);
    add_slabs(t, in.sh, out.sh, out3 ? out3->sh : nullptr, 48, 48, INT32_MAX);
    if (in.sh_t) add_slabs(t, in.sh_t, out.sh_t, nullptr, 48 * in.sh_t_deg, 0, INT32_MAX);
    return t;
}

void launch_rows_gather(const RowSlabs& t, const int32_t* src, int rows, int negative, hipStream_t st) {
    if (rows <= 0) return;
    k_rows_gather<<<dim3((unsigned)ceil_div(rows, 256), (unsigned)t.n), 256, 0, st>>>(t, src, rows, negative);
}

// partials: scan_blocks(n4) + 1 words; the last receives the converted rows.
void launch_convert_plan(const G4Ptr& in4, int n3, double log_tau, int32_t* perm, unsigned long long* partials,
                         hipStream_t st) {
    const int n4 = in4.n, nb = scan_blocks(n4);
    if (n4 > 0) k_convert_count<<<nb, 256, 0, st>>>(in4.log_scale, n4, log_tau, partials);
    launch_scan_top(partials, nb, 1, 0, partials + nb, st);
    if (n4 > 0) k_convert_perm<<<nb, 256, 0, st>>>(in4.log_scale, n4, log_tau, n3, partials, perm);
}

// The 3D rows copied, the 4D rows moved by perm; moments: zeros for the
// converted rows' quaternions.
void launch_convert_rows(const G4Ptr& in4, const G3Ptr& in3, const int32_t* perm, const G4Grad& out4,
                         const G3Grad& out3, int moments, hipStream_t st) {
    launch_rows_gather(slabs3(in3, out3, INT32_MAX), nullptr, in3.n, kNegativeZero, st);
    if (in4.n <= 0) return;
    const RowSlabs t = slabs4(in4, out4, &out3, INT32_MAX);
    k_rows_split<<<dim3((unsigned)ceil_div(in4.n, 256), (unsigned)t.n), 256, 0, st>>>(t, perm, in4.n);
    k_convert_quat<<<ceil_div(in4.n, 256), 256, 0, st>>>(in4.quat_l, in4.quat_r, in4.n, perm, out3.quat,
                                                         (size_t)out3.n, moments);
}

}  // namespace h4d

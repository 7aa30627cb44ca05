// Forward projector for gfx950: the exact adjoint of the backprojector.
//
// The backprojection of Eq. 2 (arXiv 2109.02174, section "Computed tomography")
// with linear interpolation is a linear map from filtered rows to pixels; its
// adjoint maps an image to projection rows:
//     sino[k][j] = w_k sum_{r,c} img[r][c] max(0, 1 - |u_k(x_c, y_r) - j|),
//     u_k(x, y) = (x cos(theta_k) + y sin(theta_k)) / dt + (D-1)/2,
// with w_k = pi/K (or the angle-gap weights).
//
// It is computed gather-only, one lane per detector bin, walking image lines across
// the ray.  On a line the bin's ray crosses at p* (pixel units along the line); the
// pixels with a nonzero weight are the integers in (p* - r, p* + r), r = 1/|a| with a
// the slope of u along the line: at most T = ceil(2r), T consecutive pixels from
// floor(p* - r) + 1.  Each bin is written once; no atomics; fixed summation order.
// Two forms: the staged projector (image rows through LDS, several bins per walk) where
// neighbouring angles share a window of its LDS rows, and project_kernel for the rest.
#include "fbp_internal.hpp"

#include <algorithm>
#include <cmath>
#include <type_traits>

namespace fbp {

namespace {

constexpr int kProjThreads = 256;
constexpr int kTrTile = 64;
constexpr int kAnchorLines = 256;                   // FP64 re-anchoring period (power of 2)
constexpr double kTwo32 = 4294967296.0;
constexpr float kPhase = 0x1p-32f;                  // of a 32-bit phase
constexpr int kRawWord3 = 0x00020000;               // buffer resource word 3: 32-bit data, raw (stride 0)
constexpr int kOffImage = 0x7FFFFFF0;               // byte offset past every image: reads as 0

// ---------------------------------------------------------------- staged projector
//
// A lane owns a bin of one base angle and walks image lines as above, but the lines
// come from LDS, and each position and weight it makes serves two or four bins:
//  * Turning the image by a quarter turn moves a projection to the angle a quarter
//    turn on, bin by bin (u_{theta+pi/2}(R X) = u_theta(X), R(x, y) = (-y, x)), and
//    turning it by a half reverses the bins.  So with I_m(X) = img(R^m X), the walk of
//    bin j at a base angle phi gives, from I_0 .. I_3, the bins j and D-1-j at phi and
//    at phi + pi/2 (M = 4: lists closed under +pi/2); any list has I_0 and I_2 (M = 2:
//    bins j and D-1-j).  The base angle is the turn of theta with |tan phi| <= 1, so
//    every walk runs along rows.  The rows of the turned images are rows of the image
//    and of its transpose, read forwards or backwards: one transposed copy is the only
//    extra memory.
//  * A workgroup of eight waves owns A neighbouring base angles and kBins bins.  Per
//    chunk of kLines image rows it stages the pixels those bins can reach as cells
//    {I_0, I_1, I_2, I_3} (at most kCells a row: the host checks the group's bound), the
//    next chunk's pixels loading while the current one is summed (double-buffered, one
//    barrier per chunk).  A lane of a wave takes every fourth row (16 bins by 4 rows).
//  * Positions are 6.26 fixed point, local to the angle's window and anchored in FP64 per
//    chunk, so that a phase carries the 24 bits of its FP32 conversion wherever in the
//    window it lies (an FP32 position of up to 64 pixels would leave it 18: on pixel noise
//    4 to 6 times the error against 64 bits).  Weights are scaled by r = 1/a, which leaves
//    three taps at 1 <= r <= 1.5 as 1 - f, r - |f - (2 - r)| and max(0, f + 2r - 3) of the
//    phase f; the sum is scaled by a.
//  * Every bin has 16 sums: rows = i + 4 q (mod 16) for lane row i and step q.  They
//    are added in that order through LDS, whichever waves made them, so the number of
//    angles per workgroup never changes a bit.  No atomics; each bin is written once.
// Bound by VALU issue, with LDS reads close behind: a step of a wave (64 lane-rows, 256
// bin-rows at M = 4) is 23 VALU instructions (20 with FP32 positions) and three 16-byte LDS
// reads, and staging, anchors and steps off the image add a quarter (512^2, 720 angles:
// 23.4 M VALU instructions, 38 us at full issue; with FP32 positions the staging loads taken
// out left 38 of 39 us a slice, the LDS bank conflicts 35).  Measured there: 63 us one slice,
// 41 us a slice in stacks of 16 (FP32 positions 62 and 40), against 110 and 84 us for one lane
// per bin reading padded copies from memory.
// 16 bins by 4 rows per wave rather than 32 by 2: the blocks are half as large, four to
// a CU for one slice; 4 or 2 angles instead of 8 stage more per bin (70 and 104 us).
constexpr int kStThreads = 512;
constexpr int kStWaves = kStThreads / 64;
constexpr int kBins = kProjBins;                    // bins per workgroup and angle
constexpr int kLines = kProjLines;                  // image rows per chunk
constexpr int kCells = kProjCells;                  // staged pixels per row
constexpr int kSteps = 4;                           // rows of a chunk a lane takes: kLines / (64 / kBins)
constexpr int kPosBits = 26;                        // fraction bits of a window-local position (six for the pixel)
constexpr double kPosOne = 1 << kPosBits;
static_assert(kCells <= 1 << (32 - kPosBits), "a window's positions fit");
static_assert(kBins * (kLines / kSteps) == 64 && kLines == 2 * kStWaves && kCells == 64, "staged projector layout");

template <int M>
struct Cell;
template <>
struct Cell<4> {
    using type = float4;
};
template <>
struct Cell<2> {
    using type = float2;
};
__device__ __forceinline__ void unpack(const float4& c, float (&v)[4]) { v[0] = c.x; v[1] = c.y; v[2] = c.z; v[3] = c.w; }
__device__ __forceinline__ void unpack(const float2& c, float (&v)[2]) { v[0] = c.x; v[1] = c.y; }
__device__ __forceinline__ void pack(const float (&v)[4], float4& c) { c = make_float4(v[0], v[1], v[2], v[3]); }
__device__ __forceinline__ void pack(const float (&v)[2], float2& c) { c = make_float2(v[0], v[1]); }

// Loads of one chunk by one lane: pixel `px` of two rows of the M turned images, as
//     I_0[l][p] = img[l][p]            I_1[l][p] = tr[N-1-l][p]
//     I_2[l][p] = img[N-1-l][N-1-p]    I_3[l][p] = tr[l][N-1-p]
// (tr the transposed image).  M = 4: all four; M = 2: I_s, I_{s+2}.
// Rows and pixels off the image read as 0 (range-checked buffer loads).
template <int M>
struct TurnRows {
    __amdgpu_buffer_rsrc_t img, tr;
    int N, s;
    __device__ __forceinline__ TurnRows(const float* im, const float* t, int n, int sel) : N(n), s(sel) {
        img = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(im), (short)0, n * n * 4, kRawWord3);
        tr = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(t), (short)0, n * n * 4, kRawWord3);
    }
    __device__ __forceinline__ float at(const __amdgpu_buffer_rsrc_t& b, int row, int off) const {
        return __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(b, off, row * N * 4, 0));
    }
    // pixel px < end of row l (uniform); pixels from `end` on are not loaded (0)
    __device__ __forceinline__ void load(float (&v)[M], int l, int px, int end) const {
        const bool in = (unsigned)px < (unsigned)min(N, end) && l < N;
        const int fwd = in ? px * 4 : kOffImage, rev = in ? (N - 1 - px) * 4 : kOffImage;
        const int la = l < N ? l : 0, lb = N - 1 - la;
        if constexpr (M == 4) {
            v[0] = at(img, la, fwd);
            v[1] = at(tr, lb, fwd);
            v[2] = at(img, lb, rev);
            v[3] = at(tr, la, rev);
        } else {
            v[0] = s ? at(tr, lb, fwd) : at(img, la, fwd);
            v[1] = s ? at(tr, la, rev) : at(img, lb, rev);
        }
    }
};

// T taps; FAST3: T == 3 and 1 <= r <= 1.5 on every angle.  P: parts the rows of a chunk
// are split over (P waves per angle, A = 8 / P angles per workgroup).
template <int M, int T, bool FAST3, int P>
__global__ __launch_bounds__(kStThreads) void project_staged_kernel(ProjStagedJob job) {
    using C = typename Cell<M>::type;
    constexpr int A = kStWaves / P;
    constexpr int NS = kSteps / P;                  // steps of this wave
    __shared__ __attribute__((aligned(16))) C win[2][kLines][kCells];
    extern __shared__ int2 wlo_lds[];               // [chunks] first staged pixel and one past the last (equal: none)
    const int per_slice = job.groups * job.bin_blocks;
    // Workgroups of one stratum (one per CU) are dealt out in turn; every second stratum
    // is taken backwards, so that a CU's workgroups add up to about the same work
    int b = blockIdx.x;
    if (job.stratum > 0) {
        const int q = b / job.stratum;
        if ((q & 1) && (q + 1) * job.stratum <= (int)gridDim.x) b = (2 * q + 1) * job.stratum - 1 - b;
    } else {
        b = xcd_logical(b, gridDim.x);
    }
    const int s = b / per_slice;
    const int rest = b - s * per_slice;
    // bin blocks from the middle of the detector outwards: the longest walks first
    const int jb = job.bin_blocks - 1 - rest / job.groups;
    const int g = rest - (rest / job.groups) * job.groups;
    const int sel = g >= job.groups0 ? 1 : 0;       // M = 2: which pair of turns this group reads
    const int first = sel ? job.n0 + (g - job.groups0) * job.per : g * job.per;
    const int n_ang = min(job.per, (sel ? job.n_base : job.n0) - first);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int N = job.N, D = job.D;
    const double half = job.half_pix, cd = job.centre_det;
    const int j0 = jb * kBins;
    const int nch = (N + kLines - 1) / kLines;

    // windows of the chunks: first staged pixel over the group's angles, bins and rows
    // (X = p* - r, linear in the bin and the row), or none when no pixel is reached
    for (int c = tid; c < nch; c += kStThreads) {
        double lo = INFINITY, hi = -INFINITY;
        for (int i = 0; i < n_ang; ++i) {
            const ProjAngle* e = job.tab + first + i;
            const double inv = 1.0 / e->a, dl = -e->b * inv;
            const double x = ((double)j0 - cd + e->b * half) * inv + half - inv + (double)(c * kLines) * dl;
            const double run = (double)(kLines - 1) * dl;
            lo = fmin(lo, x + fmin(0.0, run));
            hi = fmax(hi, x + (double)(kBins - 1) * inv + fmax(0.0, run));
        }
        // taps of a lane: floor(X) + 1 .. floor(X) + T; one pixel of margin below for FP32
        const bool none = hi + (double)(T + 1) < 0.0 || lo > (double)N;
        const int w = none ? 0 : (int)floor(lo) - 1;
        wlo_lds[c] = make_int2(w, none ? 0 : (int)floor(hi) + T + 2);
    }

    // this wave's angle, and this lane's bin and rows
    const int ia = wave & (A - 1), part = wave / A;
    const bool active = ia < n_ang;
    const ProjAngle* e = job.tab + first + (active ? ia : 0);
    const double inv_a = 1.0 / e->a, dl = -e->b * inv_a;
    const int li = lane / kBins;                    // row of the lane within a step
    const int j = j0 + (lane & (kBins - 1));
    const double xj = ((double)j - cd + e->b * half) * inv_a + half - inv_a;   // X on row 0
    const float r = (float)inv_a, r2 = (float)(2.0 - inv_a), r3 = (float)(2.0 * inv_a - 3.0);
    float tap[T];                                   // 1 + m - r
#pragma unroll
    for (int m = 0; m < T; ++m) tap[m] = (float)((double)(m + 1) - inv_a);
    uint32_t step[NS];                              // X from row li of a chunk to the lane's row of step q
#pragma unroll
    for (int q = 0; q < NS; ++q) step[q] = (uint32_t)(int)rint((double)(4 * (part + P * q)) * dl * kPosOne);
    // smallest X of the angle's bins on a chunk's rows, from the chunk's first row on row 0
    const double x_min = ((double)j0 - cd + e->b * half) * inv_a + half - inv_a + fmin(0.0, (double)(kLines - 1) * dl);

    const size_t pix = (size_t)N * N;
    const TurnRows<M> rows(job.img + (size_t)s * pix, job.tr + (size_t)s * pix, N, sel);
    float pf[2][M];
    auto load = [&](int c, int2 w) {
#pragma unroll
        for (int h = 0; h < 2; ++h) rows.load(pf[h], c * kLines + 2 * wave + h, w.x + lane, max(w.y, 0));
    };
    auto store = [&](int buf) {
#pragma unroll
        for (int h = 0; h < 2; ++h) pack(pf[h], win[buf][2 * wave + h][lane]);
    };
    float acc[NS][M];
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int m = 0; m < M; ++m) acc[q][m] = 0.0f;
    auto next = [&](int c, int2& w) {               // the next chunk with a window
        for (++c; c < nch; ++c) {
            const int2 v = wlo_lds[c];
            w = make_int2(__builtin_amdgcn_readfirstlane(v.x), __builtin_amdgcn_readfirstlane(v.y));
            if (w.x != w.y) break;
        }
        return c;
    };
    auto compute = [&](int buf, int c, int wlo) {
        // positions local to the angle's own window (not the group's, so that the grouping
        // does not round them differently)
        const double own = floor(fma((double)(c * kLines), dl, x_min)) - 1.0;
        const uint32_t xr = (uint32_t)((fma((double)(c * kLines + li), dl, xj) - own) * kPosOne);
        const C* __restrict__ row0 = &win[buf][li + 4 * part][0] + ((int)own - wlo);
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const uint32_t x = xr + step[q];        // 1 <= x < 64 up to rounding
            const C* __restrict__ px = row0 + 4 * P * q * kCells + (x >> kPosBits);
            const float f = (float)(x << (32 - kPosBits));      // phase * 2^32
            float w[T];
            if constexpr (FAST3) {
                w[0] = fmaf(f, -kPhase, 1.0f);
                w[1] = r - fabsf(fmaf(f, kPhase, -r2));
                w[2] = fmaxf(fmaf(f, kPhase, r3), 0.0f);
            } else {
#pragma unroll
                for (int m = 0; m < T; ++m) w[m] = fmaxf(r - fabsf(fmaf(f, kPhase, -tap[m])), 0.0f);
            }
#pragma unroll
            for (int m = 0; m < T; ++m) {
                float v[M];
                unpack(px[m + 1], v);
#pragma unroll
                for (int z = 0; z < M; ++z) acc[q][z] = fmaf(w[m], v[z], acc[q][z]);
            }
        }
    };
    __syncthreads();                                // windows made
    int2 w0 = make_int2(0, 0), w1 = w0;
    int c = next(-1, w0);
    if (c < nch) load(c, w0);
    for (int buf = 0; c < nch; buf ^= 1) {
        store(buf);
        const int cn = next(c, w1);
        if (cn < nch) load(cn, w1);
        // one barrier per chunk: a wave stores into a buffer two chunks after reading it,
        // and it passed the barrier between with every wave done reading
        __syncthreads();
        if (active) compute(buf, c, w0.x);
        c = cn;
        w0 = w1;
    }

    // the 16 sums of each bin, in step and row order
    __syncthreads();
    float* part_lds = reinterpret_cast<float*>(&win[0][0][0]);   // [A][kSteps][M][64]
    static_assert(sizeof(float) * A * kSteps * M * 64 <= sizeof(win), "sums fit the windows");
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int m = 0; m < M; ++m) part_lds[((ia * kSteps + part + P * q) * M + m) * 64 + lane] = acc[q][m];
    __syncthreads();
    for (int o = tid; o < n_ang * M * kBins; o += kStThreads) {
        const int bin = o & (kBins - 1), m = (o / kBins) % M, i = o / (kBins * M);
        float sum = 0.0f;
#pragma unroll
        for (int q = 0; q < kSteps; ++q)
#pragma unroll
            for (int z = 0; z < 64 / kBins; ++z) sum += part_lds[((i * kSteps + q) * M + m) * 64 + z * kBins + bin];
        // turn m of the base angle: m = t is the angle itself, t + 1 (M = 4) a quarter turn
        // on, t + 2 and t + 3 the same with the bins reversed
        const ProjAngle* ea = job.tab + first + i;
        const int turn = M == 4 ? (m - ea->t) & 3 : ((sel + 2 * m) - ea->t) & 3;
        const int k = (turn & 1) ? ea->k1 : ea->k0;
        const int jj = j0 + bin, out = (turn & 2) ? D - 1 - jj : jj;
        if (jj < job.Dh && !((turn & 2) && out == jj)) {
            const float wk = job.wscale ? job.wscale[k] * job.scale : job.scale;
            job.sino[((size_t)s * job.K + k) * D + out] = sum * (float)ea->a * wk;
        }
    }
}

// ---------------------------------------------------------------- staged fan-beam projector
//
// The adjoint of the fan-beam backprojection
//     img(X) = (2 pi / K) sum_k (R / L_k)^2 Q~_k(u_k(X)),  L_k = R - (x cos b_k + y sin b_k),
//     u_k(X) = R (-x sin b_k + y cos b_k) / (L_k ds) + (D-1)/2
// (Kak & Slaney 1988, ch. 3), i.e.
//     sino[k][j] = (2 pi / K) sum_X img(X) (R / L_k)^2 max(0, 1 - |u_k(X) - j|),
// in the staged projector's manner: a lane owns a bin of one base view and walks rows
// that come from LDS; the four turned images (M = 4: lists closed under quarter turns)
// and S slices share every position and weight.  What the fan beam changes:
//  * Turning the image by a quarter turn moves bin j of a view to bin j of the view a
//    quarter turn on; there are no reversed bins.  M = 4 serves views b + m pi/2 from
//    I_0 .. I_3, M = 1 (any other list) the view itself from one turned image.
//  * The turn is chosen per (views of the workgroup, its bins) by the direction of the
//    rays, not per view, so that every walked ray runs within about 45 degrees of the
//    columns whatever the fan's opening: windows stay narrow and pixels few per row.
//  * On a row the pixels with a nonzero weight lie exactly between the crossings of the
//    neighbouring rays, u = j - 1 and u = j + 1.  Every crossing is affine in the row, so
//    the first tap follows ray j - 1 in fixed-point steps (7.25, for the reason given above)
//    anchored in FP64 per chunk, and the tap count is a number of the chunk
//    (workgroup-uniform), from 1 to kFanTaps.
//  * With d the tap's distance from ray j along the row, l the ray's depth L/R there:
//    L/R at the tap is l + d L'/R and u - j = d E'/R / (L/R); one reciprocal per tap
//    serves the hat and the (R/L)^2 weight, for M S pixels.
//  * The turned images are laid out once per call with a border of zeros, M = 4 as cells
//    {I_0, I_1, I_2, I_3}, so that staging is one 16-byte load and one LDS store per cell.
// Bound by VALU issue: per tap six instructions, a quarter-rate reciprocal and M S
// multiply-adds (512^2, 720 views, two slices: 61.3 M wave instructions, 100 of 156 us at
// full issue; LDS 66 us).  Measured there: 156 us, against 1450 us for one lane per bin
// reading padded copies from memory.  Eight views a workgroup rather than four: 160 and
// 201 us (a staged cell serves twice the bins); two slices rather than one: 160 and 203 us.
// 16 rows of at most 64 cells, which only two views fit, gathered from the image and its
// transpose a pixel at a time: 277 us, 145 of them in staging alone.
constexpr int kFanTaps = 6;                         // most taps per row (wider hats take fan_project_kernel)
constexpr int kFanLines = 8;                        // image rows per chunk
constexpr int kFanCells = 96;                       // staged pixels per row
constexpr int kFanBorder = kFanCells;               // zeros on both sides of a row of the turned images
constexpr int kFanPosBits = 25;                     // fraction bits of a window-local position (seven for the pixel)
constexpr double kFanPosOne = 1 << kFanPosBits;
static_assert(kFanCells <= 1 << (32 - kFanPosBits), "a window's positions fit");
constexpr double kFanMinDepth = 16.0;               // depths are kept above this (the image lies beyond it)

struct FanRay {                                     // crossing of ray u = cd - g with row l: p0 + l dp (pixels)
    double p0, dp;
};
__host__ __device__ inline FanRay fan_ray(double cb, double sb, double R, double inv_ds, double half, double g) {
    const double inv = 1.0 / (-R * sb * inv_ds - g * cb);
    const double El = R * cb * inv_ds - g * sb;
    FanRay r;
    r.dp = -El * inv;
    r.p0 = half - g * R * inv - r.dp * half;
    return r;
}
__host__ __device__ inline void turn_by(int q, double& c, double& s) {   // q quarter turns, exactly
    const double x = c, y = s;
    if (q == 1) { c = -y; s = x; }
    else if (q == 2) { c = -x; s = -y; }
    else if (q == 3) { c = y; s = -x; }
}
// Quarter turns that bring the ray of view (cb, sb) to bin offset g nearest to +y.
__host__ __device__ inline int fan_turns(double cb, double sb, double R, double ds, double g) {
    const double dx = g * ds * sb - R * cb, dy = -g * ds * cb - R * sb;
    if (fabs(dy) >= fabs(dx)) return dy > 0.0 ? 0 : 2;
    return dx > 0.0 ? 1 : 3;
}
// What the rows r0 .. r1 ask of a window: the first taps of the bins j0 .. j0 + 15 of one
// view lie in (lo, hi], and no bin has more than ceil(width) pixels (crossings are monotone
// and their differences monotone in the bin, both affine in the row: extremes at the corners).
struct FanEdges {
    FanRay a, b, c, d;                              // rays j0 - 1, j0 + 1, j0 + 14, j0 + 16
};
struct FanReach {
    double lo, hi, width;
};
__host__ __device__ inline FanEdges fan_edges(double cb, double sb, double R, double inv_ds, double half, double g0) {
    FanEdges e;
    e.a = fan_ray(cb, sb, R, inv_ds, half, g0 + 1.0);
    e.b = fan_ray(cb, sb, R, inv_ds, half, g0 - 1.0);
    e.c = fan_ray(cb, sb, R, inv_ds, half, g0 - (kProjBins - 2));
    e.d = fan_ray(cb, sb, R, inv_ds, half, g0 - kProjBins);
    return e;
}
__host__ __device__ inline FanReach fan_reach(const FanEdges& e, double r0, double r1) {
    const double a0 = e.a.p0 + r0 * e.a.dp, a1 = e.a.p0 + r1 * e.a.dp, c0 = e.c.p0 + r0 * e.c.dp, c1 = e.c.p0 + r1 * e.c.dp;
    FanReach f;
    f.lo = fmin(fmin(a0, a1), fmin(c0, c1));
    f.hi = fmax(fmax(a0, a1), fmax(c0, c1));
    f.width = fmax(fmax(fabs(e.b.p0 + r0 * e.b.dp - a0), fabs(e.b.p0 + r1 * e.b.dp - a1)),
                   fmax(fabs(e.d.p0 + r0 * e.d.dp - c0), fabs(e.d.p0 + r1 * e.d.dp - c1)));
    return f;
}

// Geometry of the turned images of one slice: `rows` rows of `pitch` pixels, pixel p at
// kFanBorder + p; M = 4: one float4 per pixel, M = 1: four planes of floats.
__host__ __device__ inline int fan_pitch(int N) { return N + 2 * kFanBorder; }
__host__ __device__ inline int fan_rows(int N) { return (N + kFanLines - 1) / kFanLines * kFanLines; }

template <int M>
struct FanCell {
    using type = float __attribute__((ext_vector_type(4)));
};
template <>
struct FanCell<1> {
    using type = float;
};

// M turned images, S slices, A views per workgroup (P waves per view take the rows of a
// chunk between them).
template <int M, int S, int A>
__global__ __launch_bounds__(A == 8 ? 512 : 128 * A, A >= 4 ? 4 : 1) void fan_staged_kernel(FanStagedJob job) {
    using C = typename FanCell<M>::type;
    constexpr int P = A == 8 ? 1 : 2;
    constexpr int W = A * P, kThreads = 64 * W;
    constexpr int NS = 2 / P;                       // steps of this wave (four rows each)
    constexpr int RW = kFanLines / W;               // rows staged per wave
    __shared__ __attribute__((aligned(16))) C win[2][S][kFanLines][kFanCells];
    extern __shared__ int fan_lds[];                // [chunks]{first pixel, end, taps}, [A][chunks] own origins, own ends
    const int N = job.N, D = job.D;
    const int nch = (N + kFanLines - 1) / kFanLines;
    int* own_lds = fan_lds + 3 * nch;
    const int per_slice = job.groups * job.bin_blocks;
    int b = blockIdx.x;
    if (job.stratum > 0) {                          // balanced order (see project_staged_kernel)
        const int q = b / job.stratum;
        if ((q & 1) && (q + 1) * job.stratum <= (int)gridDim.x) b = (2 * q + 1) * job.stratum - 1 - b;
    } else {
        b = xcd_logical(b, gridDim.x);
    }
    const int s0 = (b / per_slice) * S;
    const int rest = b % per_slice;
    // bin blocks from the middle of the detector outwards: the longest walks first
    const int out = rest / job.groups, mid = (job.bin_blocks - 1) >> 1;
    const int jb = (out & 1) ? mid + ((out + 1) >> 1) : mid - (out >> 1);
    const int first = (rest - out * job.groups) * A;
    const int n_ang = min(A, job.n_base - first);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const double half = job.half_pix, R = job.R, inv_ds = job.inv_ds;
    const int j0 = jb * kBins;
    const double g0 = job.centre_det - (double)j0;
    // the turn of the walks: by the middle bin's ray of the middle view of the largest
    // group, so that smaller groups walk the same rows
    const int set = first / job.most * job.most;
    const ProjAngle* em = job.tab + set + (min(job.most, job.n_base - set) >> 1);
    const int turn = __builtin_amdgcn_readfirstlane(fan_turns(em->a, em->b, R, 1.0 / inv_ds, g0 - 0.5 * (kBins - 1)));

    // per view and chunk, then per chunk over the views: the window and its tap count
    int* end_lds = own_lds + A * nch;               // 8 * (last first tap) + taps
    for (int i = tid / (kThreads / A); i < n_ang; i += A) {
        double cb = job.tab[first + i].a, sb = job.tab[first + i].b;
        turn_by(turn, cb, sb);
        const FanEdges ed = fan_edges(cb, sb, R, inv_ds, half, g0);
        for (int c = tid % (kThreads / A); c < nch; c += kThreads / A) {
            const FanReach f = fan_reach(ed, (double)(c * kFanLines), (double)(c * kFanLines + kFanLines - 1));
            own_lds[i * nch + c] = (int)floor(f.lo) - 1;
            end_lds[i * nch + c] = (int)floor(f.hi) * 8 + max(1, min(kFanTaps, (int)ceil(f.width)));
        }
    }
    __syncthreads();
    for (int c = tid; c < nch; c += kThreads) {
        int lo = INT32_MAX, hi = INT32_MIN, taps = 1;
        for (int i = 0; i < n_ang; ++i) {
            lo = min(lo, own_lds[i * nch + c]);
            hi = max(hi, end_lds[i * nch + c] >> 3);
            taps = max(taps, end_lds[i * nch + c] & 7);
        }
        fan_lds[3 * c] = lo;
        fan_lds[3 * c + 1] = hi + taps + 2;
        fan_lds[3 * c + 2] = taps;
    }

    // this wave's view, and this lane's bin and rows
    const int ia = wave & (A - 1), part = wave / A;
    const bool active = ia < n_ang;
    const ProjAngle* e = job.tab + first + (active ? ia : 0);
    double cb = e->a, sb = e->b;
    turn_by(turn, cb, sb);
    const int li = lane / kBins;
    const double g = g0 - (double)(lane & (kBins - 1));
    const FanRay below = fan_ray(cb, sb, R, inv_ds, half, g + 1.0), ray = fan_ray(cb, sb, R, inv_ds, half, g);
    const float gap0 = (float)(ray.p0 - below.p0), dgap = (float)(ray.dp - below.dp);    // ray j - ray j-1, row 0 and per row
    const double inv_R = 1.0 / R;
    // depth / R along ray j: L = R - x cb - y sb with x = p - half, y = l - half
    const float dep0 = (float)(1.0 - ((ray.p0 - half) * cb - half * sb) * inv_R), ddep = (float)(-(ray.dp * cb + sb) * inv_R);
    const float lq = (float)(-cb * inv_R), eq = (float)((-R * sb * inv_ds - g * cb) * inv_R);
    const float min_dep = (float)(kFanMinDepth * inv_R);
    uint32_t step[NS];                              // first-tap position from row li of a chunk to the row of step q
#pragma unroll
    for (int q = 0; q < NS; ++q) step[q] = (uint32_t)(int)rint((double)(4 * (part + P * q)) * below.dp * kFanPosOne);

    const int pitch = fan_pitch(N);
    const size_t plane = (size_t)fan_rows(N) * pitch;      // pixels
    // M = 1: the turned image the walk reads
    const C* __restrict__ turned = reinterpret_cast<const C*>(job.turned) + (M == 1 ? (size_t)((4 - turn) & 3) * plane : 0);
    const C* src[S];
#pragma unroll
    for (int z = 0; z < S; ++z) src[z] = turned + (size_t)min(s0 + z, job.n_slices - 1) * plane * (4 / M) + kFanBorder;
    C pf[S][RW], px[S] = {};                        // px: cells 64 .. 95 of two rows per wave, of wide windows only
    const int xrow = wave * 2 + (lane >> 5), xcol = 64 + (lane & 31);
    auto wide = [&](const int2& w) { return w.y - w.x > 64; };
    auto load = [&](int c, const int2& w) {
        const int base = c * kFanLines * pitch + w.x, col = min(lane, w.y - w.x - 1);   // nothing past the window
#pragma unroll
        for (int z = 0; z < S; ++z)
#pragma unroll
            for (int h = 0; h < RW; ++h) pf[z][h] = src[z][base + (wave * RW + h) * pitch + col];
        if (W >= 4 && wide(w) && xrow < kFanLines)
#pragma unroll
            for (int z = 0; z < S; ++z) px[z] = src[z][base + xrow * pitch + xcol];
    };
    auto store = [&](int buf, int c, const int2& w) {
#pragma unroll
        for (int z = 0; z < S; ++z)
#pragma unroll
            for (int h = 0; h < RW; ++h) win[buf][z][wave * RW + h][lane] = pf[z][h];
        if (wide(w)) {
            if constexpr (W >= 4) {
                if (xrow < kFanLines)
#pragma unroll
                    for (int z = 0; z < S; ++z) win[buf][z][xrow][xcol] = px[z];
            } else {                                // few waves: the wide windows' cells as they come
                for (int o = tid; o < kFanLines * 32; o += kThreads)
#pragma unroll
                    for (int z = 0; z < S; ++z)
                        win[buf][z][o >> 5][64 + (o & 31)] = src[z][(c * kFanLines + (o >> 5)) * pitch + w.x + 64 + (o & 31)];
            }
        }
    };
    float acc[NS][S][M];
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int z = 0; z < S; ++z)
#pragma unroll
            for (int m = 0; m < M; ++m) acc[q][z][m] = 0.0f;
    auto next = [&](int c, int2& w, int& taps) {    // the next chunk whose window meets the image
        for (++c; c < nch; ++c) {
            taps = __builtin_amdgcn_readfirstlane(fan_lds[3 * c + 2]);
            w.x = __builtin_amdgcn_readfirstlane(fan_lds[3 * c]);
            w.y = __builtin_amdgcn_readfirstlane(fan_lds[3 * c + 1]);
            if (w.x < N && w.y > 0) break;
        }
        return c;
    };
    auto compute = [&](auto taps, int buf, int c, int wlo) {
        constexpr int T = decltype(taps)::value;
        const int own = own_lds[(active ? ia : 0) * nch + c];
        const int l0 = c * kFanLines + li;
        const uint32_t xr = (uint32_t)((fma((double)l0, below.dp, below.p0) - (double)own) * kFanPosOne);
        const C* __restrict__ row0 = &win[buf][0][li + 4 * part][0] + (own - wlo);
#pragma unroll
        for (int q = 0; q < NS; ++q) {
            const uint32_t x = xr + step[q];        // 1 <= x < kFanCells up to rounding
            const C* __restrict__ at = row0 + 4 * P * q * kFanCells + (x >> kFanPosBits);
            const float f = (float)(x << (32 - kFanPosBits));         // phase * 2^32
            const float fl = (float)(l0 + 4 * (part + P * q));
            const float d0 = fmaf(f, -kPhase, 1.0f) - fmaf(fl, dgap, gap0);       // first tap - ray j
            const float dep = fmaxf(fmaf(fl, ddep, dep0), min_dep);
#pragma unroll
            for (int m = 0; m < T; ++m) {
                const float d = d0 + (float)m;
                const float inv = __builtin_amdgcn_rcpf(fmaf(lq, d, dep));            // R / L
                const float h = __builtin_amdgcn_fmed3f(1.0f - fabsf(d) * (eq * inv), 0.0f, 1.0f);
                const float w = h * inv * inv;
#pragma unroll
                for (int z = 0; z < S; ++z) {
                    const C v = at[z * kFanLines * kFanCells + m + 1];
                    if constexpr (M == 1) {
                        acc[q][z][0] = fmaf(w, v, acc[q][z][0]);
                    } else {
#pragma unroll
                        for (int y = 0; y < M; ++y) acc[q][z][y] = fmaf(w, v[y], acc[q][z][y]);
                    }
                }
            }
        }
    };
    __syncthreads();                                // windows made
    int2 w0 = make_int2(0, 0), w1 = w0;
    int t0 = 1, t1 = 1;
    int c = next(-1, w0, t0);
    if (c < nch) load(c, w0);
    for (int buf = 0; c < nch; buf ^= 1) {
        store(buf, c, w0);
        const int cn = next(c, w1, t1);
        if (cn < nch) load(cn, w1);
        __syncthreads();                            // one per chunk, as in project_staged_kernel
        if (active) {
            switch (t0) {
                case 1: compute(std::integral_constant<int, 1>{}, buf, c, w0.x); break;
                case 2: compute(std::integral_constant<int, 2>{}, buf, c, w0.x); break;
                case 3: compute(std::integral_constant<int, 3>{}, buf, c, w0.x); break;
                case 4: compute(std::integral_constant<int, 4>{}, buf, c, w0.x); break;
                case 5: compute(std::integral_constant<int, 5>{}, buf, c, w0.x); break;
                default: compute(std::integral_constant<int, kFanTaps>{}, buf, c, w0.x); break;
            }
        }
        c = cn;
        w0 = w1;
        t0 = t1;
    }

    // the eight sums of each bin, in step and row order
    __syncthreads();
    constexpr int V = S * M;
    float* part_lds = reinterpret_cast<float*>(&win[0][0][0][0]);   // [A][2][V][64]
    static_assert(sizeof(float) * A * 2 * V * 64 <= sizeof(win), "sums fit the windows");
#pragma unroll
    for (int q = 0; q < NS; ++q)
#pragma unroll
        for (int z = 0; z < S; ++z)
#pragma unroll
            for (int m = 0; m < M; ++m) part_lds[((ia * 2 + part + P * q) * V + z * M + m) * 64 + lane] = acc[q][z][m];
    __syncthreads();
    for (int o = tid; o < n_ang * V * kBins; o += kThreads) {
        const int bin = o & (kBins - 1), v = (o / kBins) % V, i = o / (kBins * V);
        float sum = 0.0f;
#pragma unroll
        for (int q = 0; q < 2; ++q)
#pragma unroll
            for (int z = 0; z < 64 / kBins; ++z) sum += part_lds[((i * 2 + q) * V + v) * 64 + z * kBins + bin];
        const ProjAngle* ea = job.tab + first + i;
        const int k = M == 4 ? ea->k0 + ((turn - ea->t + v % M) & 3) * (job.K >> 2) : ea->k0;
        const int s = s0 + v / M, j = j0 + bin;
        if (j < D && s < job.n_slices) job.sino[((size_t)s * job.K + k) * D + j] = sum * job.scale;
    }
}

// The turned images of n slices for fan_staged_kernel (fan_pitch, fan_rows), zeros around
// them: I_0[l][p] = img[l][p], I_1[l][p] = img[p][N-1-l], I_2[l][p] = img[N-1-l][N-1-p],
// I_3[l][p] = img[N-1-p][l].  Tiles of 32 x 32 pixels, I_1 and I_3 transposed through LDS.
constexpr int kTurnTile = 32;
template <int M>
__global__ __launch_bounds__(256) void turn_kernel(const float* __restrict__ img, float* __restrict__ turned, int N,
                                                   int tiles_l, int tiles_p) {
    __shared__ float t1[kTurnTile][kTurnTile + 1], t3[kTurnTile][kTurnTile + 1];
    const int per = tiles_l * tiles_p;
    const int s = blockIdx.x / per, t = blockIdx.x - s * per;
    const int l0 = (t / tiles_p) * kTurnTile, p0 = (t % tiles_p) * kTurnTile - kFanBorder;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;
    const int pitch = fan_pitch(N), rows = fan_rows(N);
    const float* __restrict__ src = img + (size_t)s * N * N;
#pragma unroll
    for (int i = 0; i < kTurnTile; i += 8) {
        const int p = p0 + ty + i, l = l0 + tx;
        const bool in = (unsigned)p < (unsigned)N && l < N;
        t1[ty + i][tx] = in ? src[(size_t)p * N + (N - 1 - l)] : 0.0f;
        t3[ty + i][tx] = in ? src[(size_t)(N - 1 - p) * N + l] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kTurnTile; i += 8) {
        const int l = l0 + ty + i, p = p0 + tx;
        if (l >= rows || p + kFanBorder >= pitch) continue;
        const bool in = (unsigned)p < (unsigned)N && l < N;
        const float v0 = in ? src[(size_t)l * N + p] : 0.0f, v2 = in ? src[(size_t)(N - 1 - l) * N + (N - 1 - p)] : 0.0f;
        const float v1 = t1[tx][ty + i], v3 = t3[tx][ty + i];
        const size_t plane = (size_t)rows * pitch, at = (size_t)l * pitch + (p + kFanBorder);
        if constexpr (M == 4) {
            reinterpret_cast<float4*>(turned)[(size_t)s * plane + at] = make_float4(v0, v1, v2, v3);
        } else {
            float* dst = turned + (size_t)s * 4 * plane + at;
            dst[0] = v0;
            dst[plane] = v1;
            dst[2 * plane] = v2;
            dst[3 * plane] = v3;
        }
    }
}

// Transposed copies of n N x N slices, 64 x 64 tiles through LDS.
__global__ __launch_bounds__(256) void transpose_kernel(const float* __restrict__ img, float* __restrict__ out, int N,
                                                        int tiles) {
    __shared__ float tile[kTrTile][kTrTile + 1];
    const int per = tiles * tiles;
    const int s = blockIdx.x / per;
    const int t = blockIdx.x - s * per;
    const int r0 = (t / tiles) * kTrTile, c0 = (t % tiles) * kTrTile;
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const float* src = img + (size_t)s * N * N;
    float* dst = out + (size_t)s * N * N;
#pragma unroll
    for (int i = 0; i < kTrTile; i += 4)
        if (r0 + ty + i < N && c0 + tx < N) tile[ty + i][tx] = src[(size_t)(r0 + ty + i) * N + c0 + tx];
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kTrTile; i += 4)
        if (c0 + ty + i < N && r0 + tx < N) dst[(size_t)(c0 + ty + i) * N + r0 + tx] = tile[tx][ty + i];
}

// ---------------------------------------------------------------- one lane per bin
//
// Lists too sparse for neighbouring angles to share a staged window, small images (where
// both take the time of their launches), and detectors too coarse to stage (five or more
// taps).  Rows when |cos| >= |sin|, else columns.  The slice is first copied twice, rows
// and transposed, each line padded with zeros on both sides (pad P) and followed by one
// zero line, so that both walks read along memory and a lane's window never needs a bounds
// test.  p* advances by the same step on every line, so it is carried in 32.32 fixed point
// (integer part = window start, fraction = phase of the window), stepped with a 64-bit
// integer add and re-anchored from FP64 every 256 lines.  A wave walks only the lines its
// 64 bins can reach; on those every bin of the wave lies within 65 r + 3 pixels of the
// image (it is within 63 bins of one that reaches it), which bounds the pad.
// Taps of one line: T > 0 fixed, T == 0 job.T at run time.  FAST3: three taps
// with 1 <= r <= 1.5 on every angle (unit detector spacing), where the first tap
// lies left of p* and the third right of it, so only the middle one needs |.|.
template <int T, bool FAST3>
__global__ __launch_bounds__(kProjThreads) void project_kernel(ProjJob job) {
    // block b: (slice, angle, block of 256 bins), bins fastest
    const int nbj = (job.D + kProjThreads - 1) / kProjThreads;
    const int rest = blockIdx.x / nbj;
    const int k = rest % job.K;                     // angle
    const int s = rest / job.K;                     // slice
    const int jw = (blockIdx.x - rest * nbj) * kProjThreads + (threadIdx.x & ~63);   // first bin of the wave
    if (jw >= job.D) return;                        // whole wave past the last bin
    const int j = jw + (threadIdx.x & 63);
    const int N = job.N;
    const int taps = T > 0 ? T : job.T;
    const double c = job.cs[2 * k];                 // cos/dt
    const double sn = job.cs[2 * k + 1];            // sin/dt
    const double half = job.half_pix;               // (N-1)/2
    const double cd = job.centre_det;               // (D-1)/2
    const bool rows = fabs(c) >= fabs(sn);
    const double a = rows ? c : sn;                 // slope of u along the line
    const double b = rows ? sn : c;                 // slope of u across lines
    const double inv_a = 1.0 / a;
    const double r = fabs(inv_a);                   // hat half-width along the line
    const double dl = -b * inv_a;                   // change of p* from one line to the next
    // p*(l) = p0(j) + l dl on line l (y = l - half for rows, x = l - half for columns)
    auto p0_of = [&](int jj) { return ((double)jj - cd + b * half) * inv_a + half; };
    // lines on which some bin of the wave can have a nonzero weight: p* in (-r, N-1+r);
    // p0 is linear in the bin, so the wave's two end bins bound the range
    const int jl = min(jw + 63, job.D - 1);
    const double e0 = p0_of(jw), e1 = p0_of(jl);
    const double lo_p = -r, hi_p = (double)(N - 1) + r;
    int l_lo, l_hi;
    if (dl != 0.0) {
        const double la0 = (lo_p - e0) / dl, lb0 = (hi_p - e0) / dl;
        const double la1 = (lo_p - e1) / dl, lb1 = (hi_p - e1) / dl;
        const double lo = fmin(fmin(la0, lb0), fmin(la1, lb1));
        const double hi = fmax(fmax(la0, lb0), fmax(la1, lb1));
        l_lo = (int)fmin(fmax(floor(lo) - 1.0, 0.0), (double)N);
        l_hi = (int)fmax(fmin(ceil(hi) + 1.0, (double)(N - 1)), -1.0);
    } else {                                        // p* the same on every line
        const bool inside = fmax(e0, e1) > lo_p && fmin(e0, e1) < hi_p;
        l_lo = 0;
        l_hi = inside ? N - 1 : -1;
    }
    l_lo = __builtin_amdgcn_readfirstlane(l_lo);
    l_hi = __builtin_amdgcn_readfirstlane(l_hi);
    float acc = 0.0f;
    if (l_lo <= l_hi) {
        const int pitch = job.pitch;
        const size_t plane = (size_t)(N + 1) * pitch;
        const float* __restrict__ line = job.pimg + (size_t)s * 2 * plane + (rows ? 0 : plane) + (size_t)l_lo * pitch;
        // X(l) = p*(l) - r + P + 1: integer part = window start in the padded line
        const double shift = (double)job.pad + 1.0 - r;
        const double p0 = p0_of(j);
        auto anchor = [&](int l) -> uint64_t {
            const double X = p0 + (double)l * dl + shift;
            const double h = floor(X);
            const double f = fmin((X - h) * kTwo32, kTwo32 - 1.0);
            return ((uint64_t)(uint32_t)(int)h << 32) | (uint64_t)(uint32_t)f;
        };
        const uint64_t step = (uint64_t)(int64_t)llrint(dl * kTwo32);
        const uint32_t st_max = (uint32_t)(pitch - taps);
        const float aa = (float)fabs(a);
        const float na = (float)(-fabs(a) / kTwo32), pa = (float)(fabs(a) / kTwo32);
        const float c1 = (float)(fabs(a) * (2.0 - r)), c2 = (float)(2.0 - 3.0 * fabs(a));
        const float sa = (float)(-a / kTwo32);
        float cm[T > 0 ? T : 1];                    // a (1 - r + m): hat argument of tap m at phase 0
        if constexpr (T > 0) {
#pragma unroll
            for (int m = 0; m < T; ++m) cm[m] = (float)(a * (1.0 - r + (double)m));
        }
        if constexpr (T > 0) {
            auto load = [&](const float* ln, uint64_t x, float& ph, float (&v)[T]) {
                const uint32_t st = min((uint32_t)(x >> 32), st_max);    // in bounds whatever x holds
                ph = (float)(uint32_t)x;                                  // phase * 2^32
                const float* __restrict__ px = ln + st;
#pragma unroll
                for (int m = 0; m < T; ++m) v[m] = px[m];        // one T-dword load
            };
            auto accumulate = [&](float ph, const float (&v)[T]) {
                if constexpr (FAST3) {
                    const float w0 = fmaf(na, ph, aa);                    // |a| (1 - phase)
                    const float w1 = 1.0f - fabsf(fmaf(na, ph, c1));
                    const float w2 = __builtin_amdgcn_fmed3f(fmaf(pa, ph, c2), 0.0f, 1.0f);
                    acc = fmaf(w0, v[0], acc);
                    acc = fmaf(w1, v[1], acc);
                    acc = fmaf(w2, v[2], acc);
                } else {
#pragma unroll
                    for (int m = 0; m < T; ++m) {
                        const float t = fmaf(sa, ph, cm[m]);              // a (tap - p*)
                        const float w = __builtin_amdgcn_fmed3f(1.0f - fabsf(t), 0.0f, 1.0f);
                        acc = fmaf(w, v[m], acc);
                    }
                }
            };
            // lines in runs of kAnchorLines from an FP64 anchor; four lines per round,
            // all four loads issued before the first line's weights
            for (int l0 = l_lo; l0 <= l_hi; l0 += kAnchorLines) {
                const int l1 = min(l0 + kAnchorLines - 1, l_hi);
                uint64_t x = anchor(l0);
                int l = l0;
                for (; l + 3 <= l1; l += 4) {
                    float ph[4];
                    float v[4][T];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        load(line + u * pitch, x, ph[u], v[u]);
                        x += step;
                        asm volatile("" : "+v"(x));         // one 64-bit add per line, no unrolled copies
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) accumulate(ph[u], v[u]);
                    line += 4 * pitch;
                }
                for (; l <= l1; ++l) {
                    float ph;
                    float v[T];
                    load(line, x, ph, v);
                    accumulate(ph, v);
                    x += step;
                    asm volatile("" : "+v"(x));
                    line += pitch;
                }
            }
        } else {
            uint64_t x = anchor(l_lo);
            for (int l = l_lo; l <= l_hi; ++l, line += pitch) {
                if (l != l_lo) x = ((l & (kAnchorLines - 1)) == 0) ? anchor(l) : x + step;
                const uint32_t st = min((uint32_t)(x >> 32), st_max);
                const float ph = (float)(uint32_t)x;
                const float* __restrict__ px = line + st;
                for (int m = 0; m < taps; ++m) {
                    const float t = fmaf(sa, ph, (float)(a * (1.0 - r + (double)m)));
                    const float w = __builtin_amdgcn_fmed3f(1.0f - fabsf(t), 0.0f, 1.0f);
                    acc = fmaf(w, px[m], acc);
                }
            }
        }
    }
    if (j < job.D) {
        const float wk = job.wscale ? job.wscale[k] * job.scale : job.scale;
        job.sino[((size_t)s * job.K + k) * job.D + j] = acc * wk;
    }
}

// Fan-beam forward projector: the adjoint of the fan-beam backprojection
//     img(X) = (2 pi / K) sum_k (R / L_k)^2 Q~_k(u_k(X)),  L_k = R - (x cos b_k + y sin b_k),
//     u_k(X) = R (-x sin b_k + y cos b_k) / (L_k ds) + (D-1)/2
// (Kak & Slaney 1988, ch. 3), i.e.
//     sino[k][j] = (2 pi / K) sum_X img(X) (R / L_k)^2 max(0, 1 - |u_k(X) - j|).
// One lane per (view, bin), walking image lines across the rays (rows when
// |sin b| >= |cos b|, else columns) in the padded copies.  On a line u - j = E / L
// with E and L linear in the position q along the line, so the bin's ray crosses
// the line at q* = -E(0) / E'.  Every pixel with a nonzero weight lies within r of
// q*, r bounding the ray spacing 1 / |du/dq| on the line grown by a margin m >= r
// (fan_line_half_width; the same for the whole block, one view and one line):
// T = floor(2r) + 1 taps from floor(q* - r) + 1.  Each tap's weight comes from the
// exact E and L at that pixel (FP64 at the line's first tap, FP32 steps after
// it), so pixels the window takes in beyond the neighbouring rays weigh zero.
// Each bin is written once by its lane, summed line by line in a fixed order; no
// atomics.
__global__ __launch_bounds__(kProjThreads) void fan_project_kernel(FanProjJob job) {
    const int nbj = (job.D + kProjThreads - 1) / kProjThreads;
    const int rest = blockIdx.x / nbj;
    const int k = rest % job.K;                     // view
    const int s = rest / job.K;                     // slice
    const int j = (blockIdx.x - rest * nbj) * kProjThreads + threadIdx.x;
    if (j >= job.D) return;                         // no barrier follows
    const int N = job.N;
    const double cb = job.cs[2 * k], sb = job.cs[2 * k + 1];
    const double R = job.R, hp = job.half_pix;
    const bool rows = fabs(sb) >= fabs(cb);
    // u - j = E / L, E = Ea + Ex x + Ey y
    const double g = job.centre_det - (double)j;
    const double Ea = g * R;
    const double Ex = -R * sb / job.ds - g * cb, Ey = R * cb / job.ds - g * sb;
    const double Eq = rows ? Ex : Ey, El = rows ? Ey : Ex;      // along the line, across lines
    const double Lq = rows ? -cb : -sb, Ll = rows ? -sb : -cb;
    const double inv_Eq = 1.0 / Eq;
    const double q_off = (double)job.pad + hp;      // padded index of line coordinate 0
    const size_t plane = (size_t)(N + 1) * job.pitch;
    const float* __restrict__ line = job.pimg + (size_t)s * 2 * plane + (rows ? 0 : plane);
    const float Eq32 = (float)Eq, Lq32 = (float)Lq, R32 = (float)R;
    const float cb32 = (float)cb, sb32 = (float)sb, ds32 = (float)job.ds, hp32 = (float)hp,
                m32 = (float)job.margin;
    float acc = 0.0f;
    for (int l = 0; l < N; ++l, line += job.pitch) {
        const double lc = (double)l - hp;
        const float r = fan_line_half_width<float>(cb32, sb32, R32, ds32, hp32, m32, (float)lc, rows);
        const int T = (int)(2.0f * r) + 1;          // floor(2r) + 1 (r > 0)
        const double qs = -(Ea + El * lc) * inv_Eq;
        // first tap, clamped into the padded line: a window that leaves the line lies
        // wholly in its zero padding (pad >= T), which the clamped window reads instead
        const int st = (int)fmin(fmax(floor(qs + q_off - (double)r) + 1.0, 0.0), (double)(job.pitch - T));
        const double q0 = (double)st - q_off;
        const float E0 = (float)(Ea + Eq * q0 + El * lc);
        const float L0 = (float)(R + Lq * q0 + Ll * lc);
        const float* __restrict__ px = line + st;
        for (int m = 0; m < T; ++m) {
            const float E = fmaf((float)m, Eq32, E0);
            const float inv = __builtin_amdgcn_rcpf(fmaf((float)m, Lq32, L0));
            const float w = fmaxf(0.0f, 1.0f - fabsf(E * inv));
            const float rl = R32 * inv;
            acc = fmaf(w * rl * rl, px[m], acc);
        }
    }
    job.sino[((size_t)s * job.K + k) * job.D + j] = acc * job.scale;
}

// Padded copies of n slices: per slice, plane 0 holds the rows and plane 1 the
// columns (transposed), each of N+1 lines of `pitch` floats: line l < N holds
// pixel p of the line at index pad + p, zeros elsewhere; line N is all zeros.
// Tiles of 64 x 64 outputs; the transposed plane goes through a padded LDS tile.
__global__ __launch_bounds__(256) void pad_kernel(const float* __restrict__ img, float* __restrict__ out, int N,
                                                  int pad, int pitch, int tiles_l, int tiles_c) {
    __shared__ float tile[kTrTile][kTrTile + 1];
    const int per_plane = tiles_l * tiles_c;
    const int q = blockIdx.x / per_plane;           // slice * 2 + plane
    const int t = blockIdx.x - q * per_plane;
    const int s = q >> 1, transposed = q & 1;
    const int l0 = (t / tiles_c) * kTrTile, c0 = (t % tiles_c) * kTrTile;   // output line, column
    const int tx = threadIdx.x & 63, ty = threadIdx.x >> 6;
    const float* src = img + (size_t)s * N * N;
    float* dst = out + (size_t)q * (N + 1) * pitch;
    if (!transposed) {
#pragma unroll
        for (int i = 0; i < kTrTile; i += 4) {
            const int l = l0 + ty + i, cc = c0 + tx, p = cc - pad;
            if (l <= N && cc < pitch)
                dst[(size_t)l * pitch + cc] = (l < N && p >= 0 && p < N) ? src[(size_t)l * N + p] : 0.0f;
        }
        return;
    }
    // output (line l = image column, index cc = pad + image row): read image rows
    // p0.. p0+63 at columns l0.. l0+63 along memory, write them transposed
    const int p0 = c0 - pad;
#pragma unroll
    for (int i = 0; i < kTrTile; i += 4) {
        const int p = p0 + ty + i, col = l0 + tx;
        tile[ty + i][tx] = (p >= 0 && p < N && col < N) ? src[(size_t)p * N + col] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kTrTile; i += 4) {
        const int l = l0 + ty + i, cc = c0 + tx;
        if (l <= N && cc < pitch) dst[(size_t)l * pitch + cc] = tile[tx][ty + i];
    }
}

}  // namespace

ProjLayout project_layout(const double* cs, int K, int N) {
    double r_min = INFINITY, r_max = 0.0;
    for (int k = 0; k < K; ++k) {
        const double r = 1.0 / fmax(fabs(cs[2 * k]), fabs(cs[2 * k + 1]));
        r_min = fmin(r_min, r);
        r_max = fmax(r_max, r);
    }
    ProjLayout L;
    L.fast3 = r_min >= 1.0 && r_max <= 1.5;
    L.T = L.fast3 ? 3 : (int)fmin(ceil(2.0 * r_max), 1e9);
    const double pad = ceil(65.0 * r_max) + L.T + 4.0;
    const double pitch = (double)N + 2.0 * pad;
    if (!(pitch < 1e9)) {
        L.T = 0;                                    // unsupported (detector spacing far above the pixel size)
        return L;
    }
    L.pad = (int)pad;
    L.pitch = (int)pitch;
    L.slice_floats = (size_t)2 * (size_t)(N + 1) * (size_t)L.pitch;
    return L;
}

// The staged window of a group of neighbouring base angles (see project_staged_kernel):
// a bin of one of them that crosses row y at p, |dp/dphi| = |v| / cos phi with v the
// distance of (p, y) from the foot of the ray, at most N/sqrt(2) plus the window beyond
// the image.  Pixels: 15 bin steps of r, 15 rows of slope |tan phi|, the spread over the
// group's angles, T taps, and the rounding margins.
int project_group_angles(const std::vector<ProjAngle>& tab, int n0, int T, int N) {
    if (T > kProjMaxTaps) return 0;
    for (int A = kProjWaves; A >= 1; A >>= 1) {
        bool fits = true;
        for (int part = 0; part < 2 && fits; ++part) {
            const int lo = part ? n0 : 0, hi = part ? (int)tab.size() : n0;
            for (int i = lo; i < hi && fits; i += A) {
                double r = 0.0, slope = 0.0, sec = 0.0, p0 = INFINITY, p1 = -INFINITY;
                for (int q = i; q < std::min(i + A, hi); ++q) {
                    const double phi = std::atan2(tab[q].b, tab[q].a);
                    r = std::max(r, 1.0 / tab[q].a);
                    slope = std::max(slope, std::fabs(tab[q].b) / tab[q].a);
                    sec = std::max(sec, 1.0 / std::cos(phi));
                    p0 = std::min(p0, phi);
                    p1 = std::max(p1, phi);
                }
                const double spread = (p1 - p0) * sec * (0.70710678118654752 * N + kProjCells + kProjLines);
                fits = (kProjBins - 1) * r + (kProjLines - 1) * slope + spread + T + 4.0 <= (double)kProjCells;
            }
        }
        if (fits) return A;
    }
    return 0;
}

template <int M, int T, bool FAST3>
hipError_t launch_staged_parts(const ProjStagedJob& job, int A, dim3 grid, size_t lds, hipStream_t stream) {
    const dim3 block(kStThreads);
    switch (A) {
        case 8: return launch_kernel(project_staged_kernel<M, T, FAST3, 1>, grid, block, lds, stream, job);
        case 4: return launch_kernel(project_staged_kernel<M, T, FAST3, 2>, grid, block, lds, stream, job);
        default: return launch_kernel(project_staged_kernel<M, T, FAST3, 4>, grid, block, lds, stream, job);
    }
}

template <int M>
hipError_t launch_staged_taps(const ProjStagedJob& job, int A, int T, bool fast3, dim3 grid, size_t lds,
                              hipStream_t stream) {
    if (fast3) return launch_staged_parts<M, 3, true>(job, A, grid, lds, stream);
    if (T == 2) return launch_staged_parts<M, 2, false>(job, A, grid, lds, stream);
    if (T == 3) return launch_staged_parts<M, 3, false>(job, A, grid, lds, stream);
    if constexpr (M == 4) return launch_staged_parts<4, 4, false>(job, A, grid, lds, stream);
    return hipErrorInvalidValue;                        // four taps: quarter-turn lists only
}

hipError_t launch_project_staged(ProjStagedJob job, int M, int A_max, int T, bool fast3, int n_slices,
                                 hipStream_t stream) {
    if (n_slices <= 0) return hipSuccess;
    if (T < 2 || T > kProjMaxTaps || A_max < 1 || A_max > kProjWaves || (M != 2 && M != 4) || (fast3 && T != 3))
        return hipErrorInvalidValue;
    job.Dh = (job.D + 1) / 2;
    job.bin_blocks = (job.Dh + kBins - 1) / kBins;
    // Angles per workgroup: as many as share a window, unless that leaves fewer than two
    // workgroups per CU (the same bits either way)
    int A = A_max;
    auto blocks_of = [&](int a) {
        job.groups0 = (job.n0 + a - 1) / a;
        job.groups = job.groups0 + (job.n_base - job.n0 + a - 1) / a;
        return (int64_t)job.groups * job.bin_blocks * n_slices;
    };
    while (A > 2 && blocks_of(A) < 2 * (int64_t)current_device_cus()) A >>= 1;
    const int64_t blocks = blocks_of(A);
    job.per = A;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    // Short stacks: the balanced order; long ones: whole slices to one XCD, whose L2 they share
    job.stratum = n_slices < 8 ? current_device_cus() : 0;
    const size_t lds = sizeof(int2) * (size_t)((job.N + kLines - 1) / kLines);
    const dim3 grid((unsigned)blocks);
    return M == 4 ? launch_staged_taps<4>(job, A, T, fast3, grid, lds, stream)
                  : launch_staged_taps<2>(job, A, T, fast3, grid, lds, stream);
}

// Views per workgroup of the staged fan projector, the largest power of two whose windows
// fit for every group and bin block; 0: none does, or a bin has more than kFanTaps pixels
// on a row, or rays run too far from the columns, or the source is too close to the image
// for the depth clamp.  A window's width is convex in the row, so the first and the last
// chunk that meet the image bound every chunk between them.
int fan_group_views(const std::vector<ProjAngle>& tab, int N, int D, double R, double ds) {
    const double half = 0.5 * (N - 1), cd = 0.5 * (D - 1), inv_ds = 1.0 / ds;
    if (N > 4096 || !(R - 0.70710678118654752 * N >= kFanMinDepth + kFanTaps + 2.0)) return 0;
    const int n = (int)tab.size(), nch = (N + kFanLines - 1) / kFanLines;
    auto group_fits = [&](int i0, int na, int j0) {
        const double g0 = cd - j0;
        const ProjAngle& em = tab[(size_t)i0 + (na >> 1)];
        const int q = fan_turns(em.a, em.b, R, ds, g0 - 0.5 * (kProjBins - 1));
        FanEdges ed[kProjWaves];
        for (int i = 0; i < na; ++i) {
            double c = tab[(size_t)i0 + i].a, s = tab[(size_t)i0 + i].b;
            turn_by(q, c, s);
            for (double g : {g0 + 1.0, g0 - kProjBins}) {              // rays stay within 60 degrees of the columns
                const double dx = g * ds * s - R * c, dy = -g * ds * c - R * s;
                if (!(dy >= 0.0 && 3.0 * dy * dy >= dx * dx)) return false;
            }
            ed[i] = fan_edges(c, s, R, inv_ds, half, g0);
        }
        auto reach = [&](int c) {                   // of all the views on the rows of a chunk
            FanReach all{INFINITY, -INFINITY, 0.0};
            for (int i = 0; i < na; ++i) {
                const FanReach f = fan_reach(ed[i], (double)(c * kFanLines), (double)(c * kFanLines + kFanLines - 1));
                all.lo = std::min(all.lo, f.lo);
                all.hi = std::max(all.hi, f.hi);
                all.width = std::max(all.width, f.width);
            }
            return all;
        };
        auto left = [](const FanReach& f) { return f.hi + f.width + 4.0 < 0.0; };      // of every pixel of the image
        auto right = [&](const FanReach& f) { return f.lo - 2.0 > (double)N; };
        // the first chunk from c towards `end` that meets the image, past `end` if none does:
        // the chunks left of it are consecutive (hi and width are convex), those right of it
        // too (lo is concave), so their ends are found by bisection
        auto seek = [&](int c, int end, int step) {
            while (c != end + step) {
                const FanReach f = reach(c);
                const bool l = left(f);
                if (!l && !right(f)) return c;
                auto out = [&](int x) { return l ? left(reach(x)) : right(reach(x)); };
                int in = end;
                if (out(in)) return end + step;
                while (in - c != step) {
                    const int mid = c + (in - c) / 2;
                    (out(mid) ? c : in) = mid;
                }
                c = in;
            }
            return c;
        };
        auto fits = [](const FanReach& f) {
            return f.width <= kFanTaps - 0.01 && f.hi - f.lo + std::ceil(f.width) + 4.5 <= (double)kFanCells;
        };
        const int c0 = seek(0, nch - 1, 1);
        return c0 == nch || (fits(reach(c0)) && fits(reach(seek(nch - 1, 0, -1))));
    };
    for (int A = kProjWaves; A >= 1; A >>= 1) {
        bool fits = true;
        for (int i0 = 0; i0 < n && fits; i0 += A)
            for (int j0 = 0; j0 < D && fits; j0 += kProjBins) fits = group_fits(i0, std::min(A, n - i0), j0);
        if (fits) return A;
    }
    return 0;
}

size_t fan_turned_floats(int N) { return (size_t)4 * fan_rows(N) * fan_pitch(N); }

hipError_t launch_turn(const float* img, float* turned, int N, int M, int n_slices, hipStream_t stream) {
    if (n_slices <= 0) return hipSuccess;
    const int tiles_l = (fan_rows(N) + kTurnTile - 1) / kTurnTile, tiles_p = (fan_pitch(N) + kTurnTile - 1) / kTurnTile;
    const int64_t blocks = (int64_t)tiles_l * tiles_p * n_slices;
    if (blocks > INT32_MAX || (M != 1 && M != 4)) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(256);
    return M == 4 ? launch_kernel(turn_kernel<4>, grid, block, 0, stream, img, turned, N, tiles_l, tiles_p)
                  : launch_kernel(turn_kernel<1>, grid, block, 0, stream, img, turned, N, tiles_l, tiles_p);
}

template <int M, int S>
hipError_t launch_fan_views(const FanStagedJob& job, int A, dim3 grid, size_t lds, hipStream_t stream) {
    switch (A) {
        case 8: return launch_kernel(fan_staged_kernel<M, S, 8>, grid, dim3(512), lds, stream, job);
        case 4: return launch_kernel(fan_staged_kernel<M, S, 4>, grid, dim3(512), lds, stream, job);
        case 2: return launch_kernel(fan_staged_kernel<M, S, 2>, grid, dim3(256), lds, stream, job);
        default: return launch_kernel(fan_staged_kernel<M, S, 1>, grid, dim3(128), lds, stream, job);
    }
}

hipError_t launch_fan_project_staged(FanStagedJob job, int M, int A_max, int n_slices, hipStream_t stream) {
    if (n_slices <= 0) return hipSuccess;
    if (A_max < 1 || A_max > kProjWaves || (A_max & (A_max - 1)) || (M != 1 && M != 4) || (M == 4 && job.K % 4 != 0))
        return hipErrorInvalidValue;
    job.n_slices = n_slices;
    job.most = A_max;
    job.bin_blocks = (job.D + kBins - 1) / kBins;
    // slices that share positions and weights
    const int S = n_slices == 1 ? 1 : M == 4 ? 2 : 4;
    const int sets = (n_slices + S - 1) / S;
    int A = A_max;
    auto blocks_of = [&](int a) {
        job.groups = (job.n_base + a - 1) / a;
        return (int64_t)job.groups * job.bin_blocks * sets;
    };
    while (A > 2 && blocks_of(A) < 2 * (int64_t)current_device_cus()) A >>= 1;
    const int64_t blocks = blocks_of(A);
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    job.stratum = sets < 8 ? current_device_cus() : 0;
    const size_t lds = sizeof(int) * (3 + 2 * A) * (size_t)((job.N + kFanLines - 1) / kFanLines);
    const dim3 grid((unsigned)blocks);
    if (M == 4)
        return S == 1 ? launch_fan_views<4, 1>(job, A, grid, lds, stream) : launch_fan_views<4, 2>(job, A, grid, lds, stream);
    return S == 1 ? launch_fan_views<1, 1>(job, A, grid, lds, stream) : launch_fan_views<1, 4>(job, A, grid, lds, stream);
}

hipError_t launch_transpose(const float* img, float* out, int N, int n_slices, hipStream_t stream) {
    if (n_slices <= 0) return hipSuccess;
    const int tiles = (N + kTrTile - 1) / kTrTile;
    const int64_t blocks = (int64_t)tiles * tiles * n_slices;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    return launch_kernel(transpose_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, img, out, N, tiles);
}

hipError_t launch_project(const ProjJob& job, int n_slices, hipStream_t stream) {
    if (n_slices <= 0) return hipSuccess;
    if (job.T < 1 || job.pitch < job.N + 2 * job.T || job.pad < job.T) return hipErrorInvalidValue;
    const int64_t blocks = (int64_t)((job.D + kProjThreads - 1) / kProjThreads) * job.K * n_slices;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(kProjThreads);
    if (job.fast3) {
        if (job.T != 3) return hipErrorInvalidValue;
        return launch_kernel(project_kernel<3, true>, grid, block, 0, stream, job);
    }
    switch (job.T) {
        case 1: return launch_kernel(project_kernel<1, false>, grid, block, 0, stream, job);
        case 2: return launch_kernel(project_kernel<2, false>, grid, block, 0, stream, job);
        case 3: return launch_kernel(project_kernel<3, false>, grid, block, 0, stream, job);
        case 4: return launch_kernel(project_kernel<4, false>, grid, block, 0, stream, job);
        default: return launch_kernel(project_kernel<0, false>, grid, block, 0, stream, job);
    }
}

hipError_t launch_fan_project(const FanProjJob& job, int n_slices, hipStream_t stream) {
    if (n_slices <= 0) return hipSuccess;
    if (job.pad < 1 || job.pitch < job.N + 2 * job.pad) return hipErrorInvalidValue;
    const int64_t blocks = (int64_t)((job.D + kProjThreads - 1) / kProjThreads) * job.K * n_slices;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    return launch_kernel(fan_project_kernel, dim3((unsigned)blocks), dim3(kProjThreads), 0, stream, job);
}

hipError_t launch_pad(const float* img, float* out, int N, int pad, int pitch, int n_slices, hipStream_t stream) {
    if (n_slices <= 0) return hipSuccess;
    const int tiles_l = (N + 1 + kTrTile - 1) / kTrTile, tiles_c = (pitch + kTrTile - 1) / kTrTile;
    const int64_t blocks = (int64_t)tiles_l * tiles_c * 2 * n_slices;
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    return launch_kernel(pad_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, img, out, N, pad, pitch, tiles_l,
                         tiles_c);
}

}  // namespace fbp

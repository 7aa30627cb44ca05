// Cone-beam (FDK) backprojection for gfx950: circular source orbit, flat
// detector through the rotation axis.
//
// The 3D extension (Feldkamp, Davis & Kress 1984; Kak & Slaney 1988, ch. 3) of
// the filtered backprojection of arXiv 2109.02174 (section "Computed
// tomography", Eq. 2).  View k has its source at (R cos b_k, R sin b_k, 0);
// detector column i sits at s_i = (i - (Du-1)/2) du along (-sin b, cos b, 0) and
// row j at z_j = (j - (Dv-1)/2) dv along z.  A voxel X = (x, y, z) at depth
// L = R - (x cos b + y sin b) is seen at s = R (x, y) . e / L, z' = R z / L, and
//     vol(X) = (2 pi / K) sum_k (R/L)^2 Q~_k(s/du + (Du-1)/2, z'/dv + (Dv-1)/2)
// with bilinear interpolation, zero beyond the detector.  (The pre-weighting and
// row filter run through the pre-weight kernel and the filter GEMM.)
//
// A workgroup owns a 16 x 16 column tile of the volume and a block of 32 slices
// in z (one column per lane, 32 voxels each).  Per block of views it stages, for
// each view, exactly the detector window the block's voxels can see (found in
// FP64 from the tile's corners and the block's z extent) as raw values in LDS,
// windows packed back to back.  The in-plane map is that of the fan beam (per
// (tile, view) an FP64 origin and six FP32 coefficients; per column rho = R/L,
// the column coordinate u and the weight rho^2); along z the row coordinate is
// v = z rho / dv + const, one FMA per voxel, and the four detector values come
// from two two-dword LDS reads at one address.  Views are summed in a fixed
// order, each voxel is written once, no atomics.
#include "fbp_internal.hpp"

#include <algorithm>
#include <type_traits>

namespace fbp {

namespace {

constexpr int kConeThreads = kConeTile * kConeTile;
constexpr int kConeCoef = 12;                           // per-view floats in LDS
constexpr int kConeSerial = 8;                          // slices a workgroup of the serial form takes

// Copies units of G consecutive detector columns (G = 4: one 16-byte load and
// LDS store; the window origins, Du, the pitch and the view base are then
// multiples of four floats, so a unit lies wholly on or off the detector) of the
// windows of views kq .. kq+3 into LDS, one unit per lane and view in flight.
template <int G>
__device__ __forceinline__ void cone_stage(const ConeJob& job, const int* org, float* win, int kq, int nk, int k0,
                                           int pitch) {
    using V = typename std::conditional<G == 4, float4, float>::type;
    int i0[4], j0[4], ng[4], nr[4], units[4], off[4];
    float inv_ng[4];
    int most = 0;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int kk = min(kq + u, nk - 1);
        const int4 o = *reinterpret_cast<const int4*>(org + 8 * kk);
        i0[u] = o.x;
        j0[u] = o.y;
        ng[u] = o.z / G;
        nr[u] = o.w;
        off[u] = org[8 * kk + 4];
        units[u] = kq + u < nk ? ng[u] * nr[u] : 0;
        inv_ng[u] = 1.0f / (float)ng[u];
        most = max(most, units[u]);
    }
    for (int e = threadIdx.x; e < most; e += kConeThreads) {
        V val[4];
        int at[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            // unit e is (row e / ng, group e % ng); the quotient from a float
            // reciprocal is exact: e < 2^16, and (e + 1/2) / ng is at least
            // 1 / (2 ng) away from an integer
            const int rr = (int)(((float)e + 0.5f) * inv_ng[u]);
            const int cc = G * (e - __mul24(rr, ng[u]));
            const int row = j0[u] + rr, col = i0[u] + cc;
            at[u] = e < units[u] ? off[u] + __mul24(rr, pitch) + cc : -1;
            const float* __restrict__ src = job.q + (size_t)(k0 + kq + u) * job.Dv * job.Du;
            const unsigned gb = (unsigned)(__mul24(row, job.Du) + col) * 4u;   // < 2^28
            if (e < units[u] && (unsigned)row < (unsigned)job.Dv && (unsigned)col < (unsigned)job.Du)
                val[u] = *reinterpret_cast<const V*>(reinterpret_cast<const char*>(src) + gb);
            else
                val[u] = V{};
        }
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (at[u] >= 0) *reinterpret_cast<V*>(win + at[u]) = val[u];
    }
}

// STAGED: each view's detector window goes through LDS with a row pitch of P
// floats (P = 0: the pitch is job.pitch; a fixed P lets the two rows of a bilinear
// sample come from one LDS address with constant offsets).  Windows are packed
// back to back by their actual row count, so a block takes as many of the next
// KB views as fit job.cap floats (at least one: the host checks that the largest
// possible window fits).  Otherwise the four values come from global memory with
// detector bounds checks.  Both read the same per-view window and share the
// arithmetic.
//
// ZS slices of the block of kConeZB per workgroup: all of them, or (ZS < kConeZB) the form
// for views in parts without planes for the parts' sums: the workgroup takes the parts one
// after another and adds their sums in registers, in the order and so with the bits of the
// planes.  There are few blocks then, so each goes to kConeZB / ZS workgroups, which stage
// the same windows; no voxel's arithmetic depends on ZS.  64^3, 361 views: 593 us against 868
// unsplit and 90 with planes; quarter-turn form, 100^2 x 60, 360 views: 471, 1244 and 127.
template <bool STAGED, int P, int ZS>
__global__ __launch_bounds__(kConeThreads) void cone_bp_kernel(ConeJob job) {
    extern __shared__ __align__(16) char smem[];
    const int KB = job.KB, N = job.N, K = job.K, Du = job.Du, Dv = job.Dv;
    const int pitch = P > 0 ? P : job.pitch;
    const int RW = job.WV + 1;                         // rows of the largest window
    const int A = job.vec4 ? 4 : 1;                    // column alignment of the windows
    // per view: n0 n1 n2 cvj | d0 d1 d2 umax | vmax - - - (floats); column
    // origin, row origin, columns, rows, LDS offset, - - - (ints); then the
    // number of views in the block
    float* coef = reinterpret_cast<float*>(smem);
    int* org = reinterpret_cast<int*>(coef + kConeCoef * KB);
    int* nk_lds = org + 8 * KB;
    float* win = reinterpret_cast<float*>(nk_lds + 4);
    const int tiles = job.tiles_x * job.tiles_x;
    const int zblocks = (job.Nz + kConeZB - 1) / kConeZB;
    constexpr bool kSerial = ZS < kConeZB;
    constexpr int kSubs = kConeZB / ZS;
    const int block = blockIdx.x / kSubs, zs = blockIdx.x % kSubs * ZS;
    const int view_part = block / (tiles * zblocks);                   // views [K part / split, K (part+1) / split)
    const int zb = block / tiles - view_part * zblocks;
    const int tile = block % tiles;
    const int c0 = (tile % job.tiles_x) * kConeTile, r0 = (tile / job.tiles_x) * kConeTile;
    const int z0 = zb * kConeZB;
    const int zn = min(kConeZB, job.Nz - z0);
    const int dx = threadIdx.x & (kConeTile - 1), dy = threadIdx.x / kConeTile;
    const bool inside = c0 + dx < N && r0 + dy < N;
    const int cw = min(kConeTile, N - c0), rh = min(kConeTile, N - r0);
    const float fdx = (float)dx, fdy = (float)dy;
    const double zlo = (double)z0 - job.half_z, zhi = zlo + (double)(zn - 1);
    const float zlo_dv = (float)(zlo / job.dv), inv_dv = (float)(1.0 / job.dv);
    if (zs >= zn) return;                               // the whole workgroup
    float acc[ZS];
    auto walk = [&](int part) {
#pragma unroll
        for (int q = 0; q < ZS; ++q) acc[q] = 0.0f;
        const int k_end = (int)((int64_t)K * (part + 1) / job.split);
        for (int k0 = (int)((int64_t)K * part / job.split); k0 < k_end;) {
            const int nmax = min(KB, k_end - k0);
            __syncthreads();                                // previous block's reads done
            if (threadIdx.x < 64) {                         // wave 0: one view per lane (KB <= 64)
                int size = 0;
                if ((int)threadIdx.x < nmax) {
                    // FP64, per view: the in-plane map (as the fan beam) and the window
                    // of detector cells the tile's voxels can reach.  u = N/L and
                    // rho = R/L are linear-fractional in (x, y), so over the tile their
                    // extremes sit at the corners; v = z rho / dv + cv is then extreme
                    // at a corner of (z, rho).  One cell of margin on each side covers
                    // FP32 rounding, and the clamps below keep every read inside the
                    // window regardless.
                    const int k = k0 + threadIdx.x;
                    const double c = job.cs[2 * k], sn = job.cs[2 * k + 1];
                    const double R = job.R, du = job.du;
                    const double xt = (double)c0 - job.half_pix, yt = (double)r0 - job.half_pix;
                    const double Lt = R - (c * xt + sn * yt);
                    const double Nt = R * (-sn * xt + c * yt);
                    double Lmin = INFINITY, Lmax = -INFINITY, umin = INFINITY, umax = -INFINITY;
                    for (int q = 0; q < 4; ++q) {
                        const double ex = (q & 1) ? (double)(cw - 1) : 0.0, ey = (q & 2) ? (double)(rh - 1) : 0.0;
                        const double L = Lt - c * ex - sn * ey;
                        const double u = (Nt + R * (-sn * ex + c * ey)) / (L * du);
                        Lmin = fmin(Lmin, L);
                        Lmax = fmax(Lmax, L);
                        umin = fmin(umin, u);
                        umax = fmax(umax, u);
                    }
                    const double rlo = R / Lmax, rhi = R / Lmin;
                    const double vmin = fmin(fmin(zlo * rlo, zlo * rhi), fmin(zhi * rlo, zhi * rhi)) / job.dv;
                    const double vmax = fmax(fmax(zlo * rlo, zlo * rhi), fmax(zhi * rlo, zhi * rhi)) / job.dv;
                    // column origin rounded down to the alignment, width up to it
                    const int i0 = (int)floor(umin + job.cu) - 1;
                    const int i0a = i0 - (((i0 % A) + A) % A);
                    const int j0 = (int)floor(vmin + job.cv) - 1;
                    const int ncw = (int)floor(umax + job.cu) + 3 - i0a;
                    const int nc = min(pitch, (ncw + A - 1) / A * A);
                    const int nr = min(RW, (int)floor(vmax + job.cv) + 4 - j0);   // one more row: see the clamp
                    const double G = ((double)i0a - job.cu) * du;
                    const double a0 = Nt - G * Lt, a1 = -R * sn + G * c, a2 = R * c + G * sn;
                    float* cf = coef + kConeCoef * threadIdx.x;
                    cf[0] = (float)(a0 * job.inv_duR);
                    cf[1] = (float)(a1 * job.inv_duR);
                    cf[2] = (float)(a2 * job.inv_duR);
                    cf[3] = (float)(job.cv - (double)j0);
                    cf[4] = (float)(Lt * job.inv_R);
                    cf[5] = (float)(-c * job.inv_R);
                    cf[6] = (float)(-sn * job.inv_R);
                    cf[7] = (float)(nc - 2);
                    cf[8] = (float)(nr - 2);
                    int* og = org + 8 * threadIdx.x;
                    og[0] = i0a;
                    og[1] = j0;
                    og[2] = nc;
                    og[3] = nr;
                    size = nr * pitch;
                }
                if constexpr (STAGED) {
                    // pack the windows: LDS offsets from a prefix sum over the lanes; the
                    // block takes the views whose windows end within cap (a prefix of them)
                    int incl = size;
#pragma unroll
                    for (int d = 1; d < 64; d <<= 1) {
                        const int y = __shfl_up(incl, d, 64);
                        if ((int)threadIdx.x >= d) incl += y;
                    }
                    if ((int)threadIdx.x < nmax) org[8 * threadIdx.x + 4] = incl - size;
                    const unsigned long long fit = __ballot((int)threadIdx.x < nmax && incl <= job.cap);
                    if (threadIdx.x == 0) nk_lds[0] = __popcll(fit);
                }
            }
            __syncthreads();
            int nk = nmax;
            if constexpr (STAGED) {
                nk = nk_lds[0];
                for (int kq = 0; kq < nk; kq += 4) {
                    if (job.vec4)
                        cone_stage<4>(job, org, win, kq, nk, k0, pitch);
                    else
                        cone_stage<1>(job, org, win, kq, nk, k0, pitch);
                }
                __syncthreads();
            }
            if (inside) {
                for (int kk = 0; kk < nk; ++kk) {
                    const float4 nf = *reinterpret_cast<const float4*>(coef + kConeCoef * kk);
                    const float4 df = *reinterpret_cast<const float4*>(coef + kConeCoef * kk + 4);
                    const float vmax = coef[kConeCoef * kk + 8];
                    const float den = fmaf(df.z, fdy, fmaf(df.y, fdx, df.x));
                    const float num = fmaf(nf.z, fdy, fmaf(nf.y, fdx, nf.x));
                    const float rho = __builtin_amdgcn_rcpf(den);          // R / L
                    const float u = __builtin_amdgcn_fmed3f(num * rho, 0.0f, df.w);
                    const float w = rho * rho;
                    const int iu = (int)u;
                    const float fu = u - (float)iu;
                    const float wb = w * fu, wa = w - wb;                  // column weights
                    const float a = rho * inv_dv;                          // rows per slice
                    const float v0 = fmaf(zlo_dv, rho, nf.w);              // window row of the block's first slice
                    if constexpr (STAGED) {
                        // byte offset of the sample's window column in LDS, kept in one
                        // register so each sample's address is one 24-bit multiply-add
                        unsigned boff = (unsigned)((const char*)(win + org[8 * kk + 4] + iu) - smem);
                        asm volatile("" : "+v"(boff));
                        auto sample = [&](int q, float v) {
                            const int iv = (int)v;
                            const float fv = __builtin_amdgcn_fractf(v);   // v >= 0: v - floor(v)
                            const float* __restrict__ p =
                                reinterpret_cast<const float*>(smem + __umul24((unsigned)iv, (unsigned)(4 * pitch)) + boff);
                            const float c0v = fmaf(fv, p[pitch] - p[0], p[0]);
                            const float c1v = fmaf(fv, p[pitch + 1] - p[1], p[1]);
                            acc[q] = fmaf(wb, c1v, fmaf(wa, c0v, acc[q]));
                        };
                        // v is monotone in q (a > 0, and FP32 rounding keeps the order), so
                        // when the first and last slices' rows lie in the window every
                        // slice's does and the clamp can be left out
                        if (v0 >= 0.0f && fmaf((float)(kConeZB - 1), a, v0) <= vmax) {
#pragma unroll
                            for (int q = 0; q < ZS; ++q) sample(q, fmaf((float)(zs + q), a, v0));
                        } else {
#pragma unroll
                            for (int q = 0; q < ZS; ++q)
                                sample(q, __builtin_amdgcn_fmed3f(fmaf((float)(zs + q), a, v0), 0.0f, vmax));
                        }
                    } else {
                        const float* __restrict__ qv = job.q + (size_t)(k0 + kk) * Dv * Du;
                        const int col = org[8 * kk] + iu;
                        const int row0 = org[8 * kk + 1];
                        auto at = [&](int cc, int rr) {
                            return ((unsigned)cc < (unsigned)Du && (unsigned)rr < (unsigned)Dv) ? qv[rr * Du + cc] : 0.0f;
                        };
#pragma unroll 4
                        for (int q = 0; q < ZS; ++q) {
                            const float v = __builtin_amdgcn_fmed3f(fmaf((float)(zs + q), a, v0), 0.0f, vmax);
                            const int iv = (int)v;
                            const float fv = __builtin_amdgcn_fractf(v);
                            const int row = row0 + iv;
                            const float p00 = at(col, row), p01 = at(col + 1, row);
                            const float p10 = at(col, row + 1), p11 = at(col + 1, row + 1);
                            const float c0v = fmaf(fv, p10 - p00, p00);
                            const float c1v = fmaf(fv, p11 - p01, p01);
                            acc[q] = fmaf(wb, c1v, fmaf(wa, c0v, acc[q]));
                        }
                    }
                }
            }
            k0 += nk;
        }
    };
    walk(kSerial ? 0 : view_part);
    if constexpr (kSerial) {
        float sum[ZS];
#pragma unroll
        for (int q = 0; q < ZS; ++q) sum[q] = acc[q];
        for (int part = 1; part < job.split; ++part) {
            walk(part);
#pragma unroll
            for (int q = 0; q < ZS; ++q) sum[q] += acc[q];
        }
#pragma unroll
        for (int q = 0; q < ZS; ++q) acc[q] = sum[q];
    }
    if (inside) {
        // split views: unscaled sums into the part's plane
        const bool planes = !kSerial && job.split > 1;
        float* __restrict__ vol = planes ? job.part + (size_t)view_part * job.Nz * N * N : job.vol;
        const float scale = planes ? 1.0f : job.scale;
#pragma unroll
        for (int q = 0; q < ZS; ++q)
            if (zs + q < zn)
                vol[((size_t)(z0 + zs + q) * N + (r0 + dy)) * N + (c0 + dx)] = acc[q] * scale;
    }
}

// ---------------------------------------------------------------- quarter-turn form
//
// View lists closed under quarter turns (K = 4 K4, view k + j K4 at angle b_k + j pi/2).
// Turning a column by a quarter turn and the view with it leaves (u, v, rho) unchanged,
// so column R^t p at a base view k < K4 sees the detector where column R^(t+j) p sees it
// at view k + j K4: one set of coordinates and bilinear weights serves four samples.
//  * A workgroup owns a 16 x 16 tile of the base region (rows [0, N/2), columns
//    [0, (N+1)/2): for odd N a pinwheel piece, the centre column apart) and its three
//    turns, kConeRotZB slices deep; a lane holds 4 kConeRotZB voxels.
//  * An item is (base view k, turn t): the tile's window at view b_k turned back by t, of
//    the views k + j K4, j = 0..3, staged as cells of four values, so that the four
//    corners of a sample are four 16-byte LDS reads for four voxels.
//  * The next item's cells load into registers while the current one is summed; items are
//    summed in a fixed order, each voxel is written once, no atomics.
// Bound by VALU issue (256^3, 360 views, 256 x 384 detector: 0.71 G wave instructions, 7.5
// a sample against 13.3 of one column per lane, 1.16 ms at full issue; LDS 1.1 ms), with
// four waves a SIMD.  Measured there, filter included: 1.73 ms against 2.54 ms.  Three
// waves a SIMD without spills: 2.14 ms; 12 slices a workgroup 2.00 ms; one end of the
// window area for every item (two barriers an item): 1.86 ms.
constexpr int kConeRotSerial = 4;                       // slices a workgroup of the serial form takes
constexpr int kConeRotItems = 32;                       // items whose windows are made at once
constexpr int kConeRotRegs = 3;                         // cells a thread prefetches (the rest, of the largest windows, load late)
constexpr int kConeRotInts = 16;                        // per-item words in LDS

template <int ZS>                                       // slices per workgroup (see cone_bp_kernel)
__global__ __launch_bounds__(kConeThreads, 4) void cone_rot_kernel(ConeJob job) {
    extern __shared__ __align__(16) char smem[];
    const int N = job.N, K4 = job.K >> 2, Du = job.Du, Dv = job.Dv;
    // per item: n0 n1 n2 cvj | d0 d1 d2 umax | vmax (floats), column origin, row origin, columns, rows (ints)
    float* coef = reinterpret_cast<float*>(smem);
    float4* win = reinterpret_cast<float4*>(coef + kConeRotInts * kConeRotItems);
    const int tiles_y = ((N >> 1) + kConeTile - 1) / kConeTile;
    const int tiles = job.tiles_x * tiles_y;
    const int zblocks = (job.Nz + kConeRotZB - 1) / kConeRotZB;
    constexpr bool kSerial = ZS < kConeRotZB;
    constexpr int kSubs = kConeRotZB / ZS;
    const int block = blockIdx.x / kSubs, zs = blockIdx.x % kSubs * ZS;
    const int view_part = block / (tiles * zblocks);         // base views [K4 part / split, K4 (part+1) / split)
    const int zb = block / tiles - view_part * zblocks;
    const int tile = block % tiles;
    const int c0 = (tile % job.tiles_x) * kConeTile, r0 = (tile / job.tiles_x) * kConeTile;
    const int z0 = zb * kConeRotZB;
    const int zn = min(kConeRotZB, job.Nz - z0);
    const int tid = threadIdx.x;
    const int dx = tid & (kConeTile - 1), dy = tid / kConeTile;
    const int nbx = (N + 1) >> 1, nby = N >> 1;          // base region
    const int cw = min(kConeTile, nbx - c0), rh = min(kConeTile, nby - r0);
    const float fdx = (float)dx, fdy = (float)dy;
    const double zlo = (double)z0 - job.half_z, zhi = zlo + (double)(zn - 1);
    const float zlo_dv = (float)(zlo / job.dv), inv_dv = (float)(1.0 / job.dv);
    if (zs >= zn) return;                                // the whole workgroup
    auto part_begin = [&](int part) { return 4 * (int)((int64_t)K4 * part / job.split); };
    int first = part_begin(kSerial ? 0 : view_part);     // items of the part in hand: its first, one past its last
    int items = part_begin(kSerial ? 1 : view_part + 1);
    const size_t view = (size_t)Dv * Du;

    float acc[4][ZS];
#pragma unroll
    for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int q = 0; q < ZS; ++q) acc[m][q] = 0.0f;

    // windows of the items i0 .. i0 + kConeRotItems - 1 (see cone_bp_kernel), one per lane of wave 0
    auto windows = [&](int i0) {
        const int it = i0 + tid;
        if (tid < kConeRotItems && it < items) {
            double c = job.cs[2 * (it >> 2)], sn = job.cs[2 * (it >> 2) + 1];
            const double cx = c, sx = sn;
            switch (it & 3) {                            // back by t quarter turns
                case 1: c = sx; sn = -cx; break;
                case 2: c = -cx; sn = -sx; break;
                case 3: c = -sx; sn = cx; break;
                default: break;
            }
            const double R = job.R, du = job.du;
            const double xt = (double)c0 - job.half_pix, yt = (double)r0 - job.half_pix;
            const double Lt = R - (c * xt + sn * yt);
            const double Nt = R * (-sn * xt + c * yt);
            double Lmin = INFINITY, Lmax = -INFINITY, umin = INFINITY, umax = -INFINITY;
            for (int q = 0; q < 4; ++q) {
                const double ex = (q & 1) ? (double)(cw - 1) : 0.0, ey = (q & 2) ? (double)(rh - 1) : 0.0;
                const double L = Lt - c * ex - sn * ey;
                const double u = (Nt + R * (-sn * ex + c * ey)) / (L * du);
                Lmin = fmin(Lmin, L);
                Lmax = fmax(Lmax, L);
                umin = fmin(umin, u);
                umax = fmax(umax, u);
            }
            const double rlo = R / Lmax, rhi = R / Lmin;
            const double vmin = fmin(fmin(zlo * rlo, zlo * rhi), fmin(zhi * rlo, zhi * rhi)) / job.dv;
            const double vmax = fmax(fmax(zlo * rlo, zlo * rhi), fmax(zhi * rlo, zhi * rhi)) / job.dv;
            const int i0c = (int)floor(umin + job.cu) - 1;
            const int j0 = (int)floor(vmin + job.cv) - 1;
            const int nc = min(job.WL + 1, (int)floor(umax + job.cu) + 3 - i0c);
            const int nr = min(job.WV + 1, (int)floor(vmax + job.cv) + 4 - j0);
            const double G = ((double)i0c - job.cu) * du;
            const double a0 = Nt - G * Lt, a1 = -R * sn + G * c, a2 = R * c + G * sn;
            float* cf = coef + kConeRotInts * tid;
            cf[0] = (float)(a0 * job.inv_duR);
            cf[1] = (float)(a1 * job.inv_duR);
            cf[2] = (float)(a2 * job.inv_duR);
            cf[3] = (float)(job.cv - (double)j0);
            cf[4] = (float)(Lt * job.inv_R);
            cf[5] = (float)(-c * job.inv_R);
            cf[6] = (float)(-sn * job.inv_R);
            cf[7] = (float)(nc - 2);
            cf[8] = (float)(nr - 2);
            int* og = reinterpret_cast<int*>(cf + 9);
            og[0] = i0c;
            og[1] = j0;
            og[2] = nc;
            og[3] = nr;
        }
    };
    // one cell of an item: the four views' value at window position e (0 off the detector)
    struct Window {
        int i0, j0, nc, cells;
        float inv_nc;
    };
    auto window = [&](int it) {
        const int* og = reinterpret_cast<const int*>(coef + kConeRotInts * ((it - first) & (kConeRotItems - 1)) + 9);
        Window w;
        w.i0 = __builtin_amdgcn_readfirstlane(og[0]);
        w.j0 = __builtin_amdgcn_readfirstlane(og[1]);
        w.nc = __builtin_amdgcn_readfirstlane(og[2]);
        w.cells = w.nc * __builtin_amdgcn_readfirstlane(og[3]);
        w.inv_nc = 1.0f / (float)w.nc;
        return w;
    };
    __amdgpu_buffer_rsrc_t src[4];
    auto sources = [&](int it) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            src[j] = __builtin_amdgcn_make_buffer_rsrc(const_cast<float*>(job.q + (size_t)((it >> 2) + j * K4) * view),
                                                       (short)0, (int)(view * 4), 0x00020000);
    };
    auto cell = [&](const Window& w, int e, float (&v)[4]) {
        // row e / nc, column e % nc (exact, as in cone_stage); past the window's end or off the
        // detector the offset is past the view, which reads as 0
        const int rr = (int)(((float)e + 0.5f) * w.inv_nc);
        const int row = w.j0 + rr, col = w.i0 + e - __mul24(rr, w.nc);
        const bool in = e < w.cells && (unsigned)row < (unsigned)Dv && (unsigned)col < (unsigned)Du;
        const int off = in ? (row * Du + col) * 4 : 0x7FFFFFF0;
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(src[j], off, 0, 0));
    };
    float pf[kConeRotRegs][4];
    Window nxt;
    auto load = [&](int it) {
        nxt = window(it);
        sources(it);
#pragma unroll
        for (int i = 0; i < kConeRotRegs; ++i)
            if (i * kConeThreads < nxt.cells) cell(nxt, tid + i * kConeThreads, pf[i]);
    };
    auto store = [&](float4* dst) {
#pragma unroll
        for (int i = 0; i < kConeRotRegs; ++i) {
            const int e = tid + i * kConeThreads;
            if (e < nxt.cells) dst[e] = make_float4(pf[i][0], pf[i][1], pf[i][2], pf[i][3]);
        }
        for (int e = tid + kConeRotRegs * kConeThreads; e < nxt.cells; e += kConeThreads) {
            float v[4];
            cell(nxt, e, v);
            dst[e] = make_float4(v[0], v[1], v[2], v[3]);
        }
    };
    auto compute = [&](auto turn, int it, int pitch, const float4* cells) {
        constexpr int t = decltype(turn)::value;
        const float* cf = coef + kConeRotInts * ((it - first) & (kConeRotItems - 1));
        const float4 nf = *reinterpret_cast<const float4*>(cf);
        const float4 df = *reinterpret_cast<const float4*>(cf + 4);
        const float vmax = cf[8];
        const float den = fmaf(df.z, fdy, fmaf(df.y, fdx, df.x));
        const float num = fmaf(nf.z, fdy, fmaf(nf.y, fdx, nf.x));
        const float rho = __builtin_amdgcn_rcpf(den);          // R / L
        const float u = __builtin_amdgcn_fmed3f(num * rho, 0.0f, df.w);
        const float w = rho * rho;
        const int iu = (int)u;
        const float fu = u - (float)iu;
        const float wb = w * fu, wa = w - wb;                  // column weights
        const float a = rho * inv_dv;                          // rows per slice
        const float v0 = fmaf(zlo_dv, rho, nf.w);              // window row of the block's first slice
        // byte offset of the column in LDS, in one register: a sample's address is one
        // 24-bit multiply-add
        unsigned boff = (unsigned)((const char*)(cells + iu) - smem);
        asm volatile("" : "+v"(boff));
        const unsigned pitch16 = 16u * (unsigned)pitch;
        auto sample = [&](int q, float v) {
            const int iv = (int)v;
            const float fv = __builtin_amdgcn_fractf(v);       // v >= 0: v - floor(v)
            const unsigned o = __umul24((unsigned)iv, pitch16) + boff;
            const float4* __restrict__ p = reinterpret_cast<const float4*>(smem + o);
            const float4* __restrict__ n = reinterpret_cast<const float4*>(smem + (o + pitch16));
            const float4 p00 = p[0], p01 = p[1], p10 = n[0], p11 = n[1];
            const float w10 = wa * fv, w11 = wb * fv, w00 = wa - w10, w01 = wb - w11;
            acc[t][q] = fmaf(w11, p11.x, fmaf(w10, p10.x, fmaf(w01, p01.x, fmaf(w00, p00.x, acc[t][q]))));
            acc[(t + 1) & 3][q] = fmaf(w11, p11.y, fmaf(w10, p10.y, fmaf(w01, p01.y, fmaf(w00, p00.y, acc[(t + 1) & 3][q]))));
            acc[(t + 2) & 3][q] = fmaf(w11, p11.z, fmaf(w10, p10.z, fmaf(w01, p01.z, fmaf(w00, p00.z, acc[(t + 2) & 3][q]))));
            acc[(t + 3) & 3][q] = fmaf(w11, p11.w, fmaf(w10, p10.w, fmaf(w01, p01.w, fmaf(w00, p00.w, acc[(t + 3) & 3][q]))));
        };
        // clamped into the window whatever the rounding (leaving the clamp out where the first
        // and last slices' rows lie inside measured no faster)
#pragma unroll
        for (int q = 0; q < ZS; ++q) sample(q, __builtin_amdgcn_fmed3f(fmaf((float)(zs + q), a, v0), 0.0f, vmax));
    };
    const bool inside = dx < cw && dy < rh;
    // The items' windows lie at the two ends of the window area in turn, so that one barrier
    // per item suffices: a wave stores an item's window once every wave is done with the item
    // before the last (same end).  Two neighbours that do not fit together wait for the reads.
    int last = 0;
    auto step = [&](auto turn, int it) {
        constexpr int t = decltype(turn)::value;
        const int pitch = nxt.nc, size = nxt.cells;
        float4* dst = (t & 1) ? win + (job.cap - size) : win;
        if (last + size > job.cap) __syncthreads();
        store(dst);
        __syncthreads();
        if (it + 1 < items && ((it + 1 - first) & (kConeRotItems - 1))) load(it + 1);
        if (inside) compute(turn, it, pitch, dst);
        last = size;
    };
    auto walk = [&]() {
        for (int i0 = first; i0 < items; i0 += kConeRotItems) {
            __syncthreads();
            windows(i0);
            __syncthreads();
            load(i0);
            const int end = min(items, i0 + kConeRotItems);
            for (int it = i0; it < end; it += 4) {
                step(std::integral_constant<int, 0>{}, it);
                step(std::integral_constant<int, 1>{}, it + 1);
                step(std::integral_constant<int, 2>{}, it + 2);
                step(std::integral_constant<int, 3>{}, it + 3);
            }
        }
    };
    walk();
    if constexpr (kSerial) {
        float sum[4][ZS];
        auto each = [&](auto f) {
#pragma unroll
            for (int m = 0; m < 4; ++m)
#pragma unroll
                for (int q = 0; q < ZS; ++q) f(sum[m][q], acc[m][q]);
        };
        each([](float& s, float& a) { s = a; a = 0.0f; });
        for (int part = 1; part < job.split; ++part) {
            first = items;
            items = part_begin(part + 1);
            walk();
            each([](float& s, float& a) { s += a; a = 0.0f; });
        }
        each([](float& s, float& a) { a = s; });
    }

    // turns 0 and 2 lie along rows; 1 and 3 along columns, transposed through LDS so that
    // consecutive lanes write consecutive addresses
    const size_t plane = (size_t)N * N;
    const bool planes = !kSerial && job.split > 1;
    float* __restrict__ vol = (planes ? job.part + (size_t)view_part * job.Nz * plane : job.vol) + (z0 + zs) * plane;
    const float scale = planes ? 1.0f : job.scale;             // split views: unscaled sums into the part's plane
    const int zq = zn - zs;                                    // slices of the workgroup that exist
    if (inside) {
        const int r = r0 + dy, c = c0 + dx;
#pragma unroll
        for (int q = 0; q < ZS; ++q)
            if (q < zq) {
                vol[q * plane + (size_t)r * N + c] = acc[0][q] * scale;
                vol[q * plane + (size_t)(N - 1 - r) * N + (N - 1 - c)] = acc[2][q] * scale;
            }
    }
    float* tr = reinterpret_cast<float*>(win);               // [ZS][16][17]
#pragma unroll
    for (int m = 1; m < 4; m += 2) {
        __syncthreads();
#pragma unroll
        for (int q = 0; q < ZS; ++q) tr[(q * kConeTile + dx) * (kConeTile + 1) + dy] = acc[m][q];
        __syncthreads();
        // lane (dx, dy) now holds column c0 + dy, row r0 + dx of the tile
        if (dy < cw && dx < rh) {
            const int r = r0 + dx, c = c0 + dy;
            const size_t o = m == 1 ? (size_t)c * N + (N - 1 - r) : (size_t)(N - 1 - c) * N + r;
#pragma unroll
            for (int q = 0; q < ZS; ++q)
                if (q < zq) vol[q * plane + o] = tr[(q * kConeTile + dy) * (kConeTile + 1) + dx] * scale;
        }
    }
}

// Odd N: the centre column (x = y = 0, so rho = 1 and u = (Du-1)/2 on every view), one
// slice per lane, all views in order.  A serial walk behind the main kernel, bound by the
// latency of its loads: 44 us for 316 views (the main kernel 59 at 53^3), 90 for 360 (1680
// at 255^3).
__global__ __launch_bounds__(kConeThreads) void cone_centre_kernel(ConeJob job) {
    const int z = blockIdx.x * kConeThreads + threadIdx.x;
    if (z >= job.Nz) return;                                 // no barrier follows
    const double v = ((double)z - job.half_z) / job.dv + job.cv, u = job.cu;
    const int j0 = (int)floor(v), i0 = (int)floor(u);
    const float fv = (float)(v - (double)j0), fu = (float)(u - (double)i0);
    auto at = [&](const float* q, int row, int col) {
        return (unsigned)row < (unsigned)job.Dv && (unsigned)col < (unsigned)job.Du ? q[(size_t)row * job.Du + col] : 0.0f;
    };
    float sum = 0.0f;
#pragma unroll 8
    for (int k = 0; k < job.K; ++k) {
        const float* q = job.q + (size_t)k * job.Dv * job.Du;
        const float a = fmaf(fu, at(q, j0, i0 + 1), (1.0f - fu) * at(q, j0, i0));
        const float b = fmaf(fu, at(q, j0 + 1, i0 + 1), (1.0f - fu) * at(q, j0 + 1, i0));
        sum += fmaf(fv, b, (1.0f - fv) * a);
    }
    const int c = job.N >> 1;
    job.vol[((size_t)z * job.N + c) * job.N + c] = sum * job.scale;
}

// fixed row pitches (floats) of the staged windows; the second row of a bilinear
// sample sits at an LDS offset of P + 1 <= 255 dwords
constexpr int kConePitches[] = {16, 24, 32, 40, 48, 64, 80, 96, 128, 160, 192, 248};

template <int I>
hipError_t launch_pitch(int pitch, const ConeJob& job, dim3 grid, size_t lds, hipStream_t stream) {
    if constexpr (I < (int)(sizeof(kConePitches) / sizeof(int))) {
        if (pitch == kConePitches[I])
            return launch_kernel(cone_bp_kernel<true, kConePitches[I], kConeZB>, grid, dim3(kConeThreads), lds, stream, job);
        return launch_pitch<I + 1>(pitch, job, grid, lds, stream);
    } else {
        return launch_kernel(cone_bp_kernel<true, 0, kConeZB>, grid, dim3(kConeThreads), lds, stream, job);
    }
}

}  // namespace

int cone_pitch(int WL) {
    for (int p : kConePitches)
        if (p >= WL + 1) return p;
    return (WL + 4) / 4 * 4;
}

size_t cone_lds_bytes(int KB, int cap, bool staged) {
    return sizeof(float) * kConeCoef * (size_t)KB + sizeof(int) * 8 * (size_t)KB + sizeof(int) * 4 +
           (staged ? sizeof(float) * (size_t)cap : 0);
}

// LDS of a workgroup whose window area holds `cells` cells (and, at the end, the
// transposed voxels of one turn)
size_t cone_rot_lds_bytes(int cells) {
    const int least = kConeRotZB * kConeTile * (kConeTile + 1) / 4;
    return sizeof(float) * kConeRotInts * kConeRotItems + sizeof(float4) * (size_t)std::max(cells, least);
}

hipError_t launch_cone_rot(ConeJob job, hipStream_t stream) {
    if (job.N < 2 || job.K % 4 != 0 || job.WL < 2 || job.WV < 2 ||
        cone_rot_lds_bytes((job.WL + 1) * (job.WV + 1)) > kConeLdsBudget)
        return hipErrorInvalidValue;
    // room for two of the largest windows, up to a quarter of a CU's LDS
    job.cap = std::min(2 * (job.WL + 1) * (job.WV + 1), (int)((kConeLdsBudget - sizeof(float) * kConeRotInts * kConeRotItems) / sizeof(float4)));
    job.cap = std::max(job.cap, (job.WL + 1) * (job.WV + 1));
    const size_t lds = cone_rot_lds_bytes(job.cap);
    if ((int64_t)job.Dv * job.Du * 4 > 0x7FFFFFF0) return hipErrorInvalidValue;     // a view's buffer range
    const int64_t tiles = (int64_t)job.tiles_x * (((job.N >> 1) + kConeTile - 1) / kConeTile);
    if (job.split < 1 || job.split > job.K / 4) return hipErrorInvalidValue;
    const bool serial = job.split > 1 && !job.part;
    const int64_t blocks = tiles * ((job.Nz + kConeRotZB - 1) / kConeRotZB) * (serial ? kConeRotZB / kConeRotSerial : job.split);
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    return launch_kernel(serial ? cone_rot_kernel<kConeRotSerial> : cone_rot_kernel<kConeRotZB>, dim3((unsigned)blocks),
                         dim3(kConeThreads), lds, stream, job);
}

hipError_t launch_cone_centre(const ConeJob& job, hipStream_t stream) {
    return launch_kernel(cone_centre_kernel, dim3((unsigned)((job.Nz + kConeThreads - 1) / kConeThreads)), dim3(kConeThreads),
                         0, stream, job);
}

hipError_t launch_cone_bp(const ConeJob& job, bool staged, hipStream_t stream) {
    if (job.KB < 1 || job.KB > 64 || job.WL < 2 || job.WV < 2 || job.pitch < job.WL + 1)
        return hipErrorInvalidValue;
    if (job.vec4 && (job.Du % 4 != 0 || job.pitch % 4 != 0 || job.pitch < job.WL + 7 ||
                     reinterpret_cast<uintptr_t>(job.q) % 16 != 0))
        return hipErrorInvalidValue;
    if (staged && (int64_t)(job.WV + 1) * job.pitch > job.cap) return hipErrorInvalidValue;   // one window must fit
    const size_t lds = cone_lds_bytes(job.KB, job.cap, staged);
    if (lds > kConeLdsBudget) return hipErrorInvalidValue;
    if (job.split < 1 || job.split > job.K) return hipErrorInvalidValue;
    const bool serial = job.split > 1 && !job.part;
    const int64_t blocks = (int64_t)job.tiles_x * job.tiles_x * ((job.Nz + kConeZB - 1) / kConeZB) *
                           (serial ? kConeZB / kConeSerial : job.split);
    if (blocks > INT32_MAX) return hipErrorInvalidValue;
    const dim3 grid((unsigned)blocks), block(kConeThreads);
    if (serial)
        return launch_kernel(staged ? cone_bp_kernel<true, 0, kConeSerial> : cone_bp_kernel<false, 0, kConeSerial>, grid, block,
                             lds, stream, job);
    return staged ? launch_pitch<0>(job.pitch, job, grid, lds, stream)
                  : launch_kernel(cone_bp_kernel<false, 0, kConeZB>, grid, block, lds, stream, job);
}

}  // namespace fbp

// HIP kernels (gfx950) of one RSF level-set iteration.
//
// One iteration = three passes plus a tiny reduction:
//   z(H)     : (phi, I) -> Kz*(H I), Kz*H           H = H_eps(phi)      (Sec. 3)
//   xy       : -> A1 = K*(H I), B1 = K*H, with A2 = K*I - A1, B2 = K*1 - B1
//              f1 = A1/B1, f2 = A2/B2, g1 = l1 f1 - l2 f2,
//              g2 = l1 f1^2 - l2 f2^2                                    (Sec. 3)
//              -> Kxy*g1, Kxy*g2
//   z(upd)   : Fd = (l1-l2) I^2 K*1 - 2 I K*g1 + K*g2 = l1 e1 - l2 e2,
//              curvature, regulariser, Dirac-weighted explicit update   (Sec. 2-3)
//              and per-block FP64 partial sums of |phi' - phi|
//   reduce   : fixed-order FP64 sum of the partials.
// The separable Gaussian is applied as z passes (each thread marches one
// (x, y) column through a z chunk with a register ring of 2R+1 slices) and an
// xy pass (a workgroup marches down the rows of a slice, convolving each of
// them on the matrix cores), so every global access is coalesced along x.
// Stage 1 runs z first, so H_eps is evaluated once per voxel; stage 2 runs z
// last, so the update sees the z window it needs.  Every pass is one launch
// over a batch of tiles; workgroups are numbered so that each of the 8 XCDs
// works on one contiguous range, keeping halo re-reads within one L2.
#include <algorithm>
#include <cmath>

#include "rsf_device.hpp"

namespace rsf {

namespace {

// ---------------------------------------------------------------------------
// Per-tile set-up and reduction (one workgroup per tile)
// ---------------------------------------------------------------------------

// K * 1 = cx[x] cy[y] cz[z]: partial sums of the taps that land inside; the
// tile's flags cleared.
__global__ __launch_bounds__(kThreads) void setup_kernel(Batch bt, Taps t, int R)
{
    const TileDesc &d = bt.tiles[blockIdx.x];
    const Grid3 g = d.g;
    if (threadIdx.x < 2) d.flags[threadIdx.x] = 0;
    for (int i = threadIdx.x; i < g.nx + g.ny + g.nz; i += kThreads) {
        int n, p;
        float *dst;
        if (i < g.nx) { n = g.nx; p = i; dst = d.cx; }
        else if (i < g.nx + g.ny) { n = g.ny; p = i - g.nx; dst = d.cy; }
        else { n = g.nz; p = i - g.nx - g.ny; dst = d.cz; }
        float acc = 0.f;
        for (int k = -R; k <= R; ++k)
            if (p + k >= 0 && p + k < n) acc += t.w[k + R];
        dst[p] = acc;
    }
}

// The tile table of a batch from the kernel argument (one workgroup).
__global__ __launch_bounds__(kThreads) void put_table_kernel(uint32_t *dst, TableBlob blob,
                                                             int words)
{
    for (int i = threadIdx.x; i < words; i += kThreads) dst[i] = blob.w[i];
}

// Fixed-order FP64 sum of one tile's update-pass partials into hist[iters
// run]; sets the tile's stop flag when the tolerance is met.
__global__ __launch_bounds__(kThreads) void reduce_kernel(Batch bt, Coeffs c)
{
    const TileDesc &d = bt.tiles[blockIdx.x];
    if (d.flags[0]) return;
    const int64_t n = u_blocks(d.g, d.sp);
    double acc = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += kThreads) acc += d.partials[i];
    __shared__ double sh[kThreads];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) sh[threadIdx.x] += sh[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const int k = d.flags[1];
        if (k < d.hist_cap) d.hist[k] = sh[0];
        *reinterpret_cast<double *>(d.flags + 2) = sh[0];   // last sum, 8-byte aligned
        d.flags[1] = k + 1;
        const double voxels = (double)d.g.nx * d.g.ny * d.g.nz;
        if (c.tol > 0.0 && sh[0] < c.tol * voxels) d.flags[0] = 1;
        else if (k + 1 >= d.hist_cap) d.flags[0] = 2;   // all its iterations done
    }
}

// After the last iteration: a tile whose final iterate n is odd has it in the
// workspace buffer phi[1]; copy it to the caller's phi[0].  Workgroups as in
// the stage-1 z pass.
__global__ __launch_bounds__(kThreads) void finish_kernel(Batch bt)
{
    Where wh;
    if (!locate(bt, wh)) return;
    const TileDesc &d = bt.tiles[wh.t];
    if (!(glb(d.flags)[1] & 1)) return;
    const Grid3 g = d.g;
    const ZCols zt = z_cols(g, d.sp.z, wh.lb);
    if (!zt.active) return;
    const int col = zt.col;
    const gptr<const float> src = glb(d.phi[1]);
    const gptr<float> dst = glb(d.phi[0]);
    for (int z = zt.z0; z < zt.z1; ++z) (dst + (int64_t)z * g.sxy)[col] = (src + (int64_t)z * g.sxy)[col];
}

// ---------------------------------------------------------------------------
// Volume-level driver: gather a sub-volume, merge it back (Sec. 4.1)
// ---------------------------------------------------------------------------

template <class T>
__global__ __launch_bounds__(kThreads) void gather_kernel(const T *src, T *dst, int64_t nx,
                                                          int64_t ny, SubBox b)
{
    const int64_t n = (int64_t)b.ext[0] * b.ext[1] * b.ext[2];
    const gptr<const T> s = glb(src);
    const gptr<T> d = glb(dst);
    for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads) {
        const int64_t x = i % b.ext[0], yz = i / b.ext[0];
        const int64_t y = yz % b.ext[1], z = yz / b.ext[1];
        d[i] = s[((z + b.lo[2]) * ny + (y + b.lo[1])) * nx + (x + b.lo[0])];
    }
}

// Weight of a box at volume coordinate c along one axis: 1 inside its core,
// a linear ramp across the 2C voxels straddling each core face it shares
// with a neighbour (the neighbour's ramp is its complement, so the weights
// of all boxes sum to one).
__device__ __forceinline__ float ramp(int c, int core_lo, int core_hi, int nb_lo, int nb_hi, int C)
{
    const float inv = 1.f / (2.f * (float)C);
    if (nb_lo && c < core_lo + C) return ((float)(c - (core_lo - C)) + 0.5f) * inv;
    if (nb_hi && c >= core_hi - C) return ((float)((core_hi + C) - c) - 0.5f) * inv;
    return 1.f;
}

__global__ __launch_bounds__(kThreads) void merge_kernel(float *acc, const float *tile, int64_t nx,
                                                         int64_t ny, SubBox b, int C)
{
    const int64_t n = (int64_t)b.ext[0] * b.ext[1] * b.ext[2];
    const gptr<float> a = glb(acc);
    const gptr<const float> t = glb(tile);
    for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads) {
        const int x = (int)(i % b.ext[0]);
        const int64_t yz = i / b.ext[0];
        const int y = (int)(yz % b.ext[1]), z = (int)(yz / b.ext[1]);
        const int gx = x + b.lo[0], gy = y + b.lo[1], gz = z + b.lo[2];
        const float w = ramp(gx, b.core_lo[0], b.core_hi[0], b.nb_lo[0], b.nb_hi[0], C) *
                        ramp(gy, b.core_lo[1], b.core_hi[1], b.nb_lo[1], b.nb_hi[1], C) *
                        ramp(gz, b.core_lo[2], b.core_hi[2], b.nb_lo[2], b.nb_hi[2], C);
        a[((int64_t)gz * ny + gy) * nx + gx] += w * t[i];
    }
}

__global__ __launch_bounds__(kThreads) void fill_kernel(float *dst, int64_t n, float v)
{
    const gptr<float> d = glb(dst);
    for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads)
        d[i] = v;
}

// ---------------------------------------------------------------------------
// Initialisation (Sec. 4.3): determinant-of-Hessian seeds, fast sweeping
// ---------------------------------------------------------------------------

template <class IT>
__global__ __launch_bounds__(kThreads) void smooth_x_kernel(const IT *img, float *out, int64_t nx,
                                                            int64_t n, Taps t, int R)
{
    const gptr<const IT> in = glb(img);
    const gptr<float> o = glb(out);
    for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads) {
        const int64_t x = i % nx, row = i - x;
        float acc = 0.f;
        for (int k = -R; k <= R; ++k) {
            const int64_t xx = x + k;
            if (xx >= 0 && xx < nx) acc = fmaf(t.w[k + R], to_f(in[row + xx]), acc);
        }
        o[i] = acc;
    }
}

__global__ __launch_bounds__(kThreads) void smooth_y_kernel(const float *src, float *out,
                                                            int64_t nx, int64_t ny, int64_t n,
                                                            Taps t, int R)
{
    const gptr<const float> in = glb(src);
    const gptr<float> o = glb(out);
    for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads) {
        const int64_t yz = i / nx;
        const int64_t y = yz % ny, base = i - y * nx;   // (z, 0, x)
        float acc = 0.f;
        for (int k = -R; k <= R; ++k) {
            const int64_t yy = y + k;
            if (yy >= 0 && yy < ny) acc = fmaf(t.w[k + R], in[base + yy * nx], acc);
        }
        o[i] = acc;
    }
}

__device__ __forceinline__ int64_t refl(int64_t i, int64_t n)
{
    return i < 0 ? -i : (i > n - 1 ? 2 * (n - 1) - i : i);
}

__global__ __launch_bounds__(kThreads) void hessian_kernel(const float *Lp, float *doh, float *tr,
                                                           float *part, int64_t nx, int64_t ny,
                                                           int64_t n)
{
    const gptr<const float> L = glb(Lp);
    __shared__ float sm[kThreads];
    float best = -kFar;
    for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads) {
        const int64_t x = i % nx, yz = i / nx;
        const int64_t y = yz % ny, base = i - x - y * nx;
        auto at = [&](int64_t xx, int64_t yy) { return L[base + refl(yy, ny) * nx + refl(xx, nx)]; };
        const float c = at(x, y);
        const float lxx = at(x + 1, y) - 2.f * c + at(x - 1, y);
        const float lyy = at(x, y + 1) - 2.f * c + at(x, y - 1);
        const float lxy = (at(x + 1, y + 1) - at(x + 1, y - 1) - at(x - 1, y + 1) +
                           at(x - 1, y - 1)) * 0.25f;
        const float d = lxx * lyy - lxy * lxy;
        glb(doh)[i] = d;
        glb(tr)[i] = lxx + lyy;
        best = fmaxf(best, d);
    }
    sm[threadIdx.x] = best;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) sm[threadIdx.x] = fmaxf(sm[threadIdx.x], sm[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) glb(part)[blockIdx.x] = sm[0];
}

__global__ __launch_bounds__(kThreads) void max_kernel(const float *part, int n, float *out)
{
    __shared__ float sm[kThreads];
    float best = -kFar;
    for (int i = threadIdx.x; i < n; i += kThreads) best = fmaxf(best, glb(part)[i]);
    sm[threadIdx.x] = best;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) sm[threadIdx.x] = fmaxf(sm[threadIdx.x], sm[threadIdx.x + w]);
        __syncthreads();
    }
    if (threadIdx.x == 0) glb(out)[0] = sm[0];
}

// A seed is a bright blob (trace < 0) whose determinant exceeds threshold x
// the volume's largest and is a local maximum of its 3x3 in-slice
// neighbourhood: strictly above the neighbours earlier in raster order, at
// least the later ones (so a plateau gives one seed).
__global__ __launch_bounds__(kThreads) void seeds_kernel(const float *dohp, const float *trp,
                                                         const float *maxv, float threshold,
                                                         unsigned char *mask, float *u,
                                                         unsigned *cnt, int64_t nx, int64_t ny,
                                                         int64_t n)
{
    const gptr<const float> doh = glb(dohp);
    __shared__ unsigned sc[kThreads];
    unsigned mine = 0;
    const float thr = threshold * glb(maxv)[0];
    for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads) {
        const int64_t x = i % nx, yz = i / nx;
        const int64_t y = yz % ny, base = i - x - y * nx;
        const float d = doh[i];
        bool seed = d > thr && glb(trp)[i] < 0.f;
        for (int dy = -1; dy <= 1 && seed; ++dy)
            for (int dx = -1; dx <= 1 && seed; ++dx) {
                if (dx == 0 && dy == 0) continue;
                const int64_t xx = x + dx, yy = y + dy;
                if (xx < 0 || xx >= nx || yy < 0 || yy >= ny) continue;
                const float nb = doh[base + yy * nx + xx];
                const bool earlier = dy < 0 || (dy == 0 && dx < 0);
                seed = earlier ? d > nb : d >= nb;
            }
        glb(mask)[i] = seed ? 1 : 0;
        glb(u)[i] = seed ? 0.f : kFar;
        mine += seed ? 1u : 0u;
    }
    sc[threadIdx.x] = mine;
    __syncthreads();
    for (int w = kThreads / 2; w > 0; w >>= 1) {
        if (threadIdx.x < w) sc[threadIdx.x] += sc[threadIdx.x + w];
        __syncthreads();
    }
    if (threadIdx.x == 0) glb(cnt)[blockIdx.x] = sc[0];
}

// Godunov update of |grad u| = 1 on the unit grid from the smallest
// neighbour value along each axis (x, y, z; kFar when absent).  The roots
// are written in the differences d1 = b - a, d2 = c - a, which are O(1)
// where they are used: the textbook discriminant (a+b+c)^2 - 3(a^2+b^2+c^2-1)
// cancels to O(1) from O(u^2) terms and loses most FP32 digits at large u.
// All three candidates are computed (their chains overlap) and one selected;
// the others may be NaN.
// sqrt correctly rounded, for a normal x (here 0.03..3: the library's scaling
// of denormal and huge arguments is left out; others give some value that is
// not used): the hardware root, within an ulp, moved to the neighbour that a
// Tuckerman test of the residuals selects.
__device__ __forceinline__ float sqrt_normal(float x)
{
    const float s = __builtin_amdgcn_sqrtf(x);
    const float lo = __int_as_float(__float_as_int(s) - 1);
    const float hi = __int_as_float(__float_as_int(s) + 1);
    float r = fmaf(-lo, s, x) <= 0.f ? lo : s;
    if (fmaf(-hi, s, x) > 0.f) r = hi;
    return r;
}
// The smaller of two values, or the one that is a number (as fminf; one
// instruction, where fminf first quiets operands that come from memory).
__device__ __forceinline__ float min_num(float x, float y)
{
    float r;
    __asm__("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}
__device__ __forceinline__ float godunov(float &a, float b, float c)
{
    // sorted by comparisons (not min/max, which would drop a NaN)
    float t;
    if (a > b) { t = a; a = b; b = t; }
    if (b > c) { t = b; b = c; c = t; }
    if (a > b) { t = a; a = b; b = t; }
    const float d1 = b - a;
    const float r2 = 0.5f * (d1 + sqrt_normal(2.f - d1 * d1));
    const float d2 = c - a, d3 = d2 - d1;
    const float v3 =
        a + (d1 + d2 + sqrt_normal(3.f - (d1 * d1 + d2 * d2 + d3 * d3))) * (1.f / 3.f);
    return a + 1.f <= b ? a + 1.f : (a + r2 <= c ? a + r2 : v3);
}

// One wavefront of blocks of a sweep.  In the sweep's orientation (i' = i or
// nx-1-i by its x order, likewise j', k') the points of a hyperplane
// s = i' + j' + k' do not depend on each other: each needs its upwind
// neighbours (s - 1) as already swept and its downwind ones (s + 1) as not
// yet.  A block is kSj x kSj lines (j', k') times kSs consecutive hyperplanes,
// so in the skewed coordinates (s; j', k') it needs the blocks (b - 1; J, K),
// (b; J - 1, K) and (b; J, K - 1) before it, and the blocks with
// b + J + K = W form one launch.  Every point is updated after its upwind
// neighbours and before its downwind ones, which gives exactly the sequential
// Gauss-Seidel sweep.
//
// The block's lines and one line around them are loaded skewed, [s][k'][j'],
// kSs + 2 planes (absent points as kFar); thread (j', k') updates its point of
// one plane after the other, one barrier each, and a block that changed is
// written back.  The load also takes in points that no update reads, on lines
// and planes off the block along two axes at once: those of the blocks
// (b - 1; J + 1, K), (b + 1; J - 1, K), (b; J + 1, K - 1) and the like, which
// belong to the same launch and may be writing them.  An update reads the
// points one step along one axis only: planes s - 1 and s + 1 of its own line,
// s - 1 of the lines j' - 1 and k' - 1, s + 1 of j' + 1 and k' + 1; those lie in
// blocks of launches before or after this one.
//
// What bounds it is the chain of dependent steps: (nx + ny + nz) / kSs +
// (ny + nz) / kSj launches a sweep, each a block's load, kSs steps and its
// store.  512^3, 2 rounds: 1760 launches of 21 us, 103 -> 43 ms a call;
// unskewed blocks of 32 x 8 x 8, whose 46 inner hyperplanes are mostly idle,
// took 2272 launches of 43 us.  The wave runs alone on its SIMD and issues an
// instruction every 5 to 6 clocks, so instructions count, not operations:
// dividing out each element's coordinates while staging cost 38 us a launch.
constexpr int kSj = 16, kSs = 32;
__global__ __launch_bounds__(kSj * kSj) void sweep_block_kernel(float *up, int nx, int ny, int nz,
                                                                int dir, int W, int nb, int nbj,
                                                                int kblo)
{
    constexpr int T = kSj + 2, NT = kSj * kSj;
    constexpr int PL = T * T + 1;   // plane pitch, odd: the skewed writes spread over the banks
    static_assert(kSs == 32 && NT == 256, "eight half-waves, each a line's 32 planes");
    __shared__ float tile[(kSs + 2) * PL];
    __shared__ int any;
    const int bj = (int)blockIdx.x % nbj, bk = kblo + (int)blockIdx.x / nbj;
    const int b = W - bj - bk;
    const int j0 = bj * kSj, k0 = bk * kSj, s0 = b * kSs;   // oriented origin
    if (b < 0 || b >= nb) return;                           // the whole workgroup
    // hyperplanes of the block's lines: none of this block's kSs, no work
    const int lo = j0 + k0, hi = min(j0 + kSj, ny) - 1 + min(k0 + kSj, nz) - 1 + nx - 1;
    if (s0 + kSs <= lo || s0 > hi) return;
    const int tid = threadIdx.x;
    const gptr<float> u = glb(up);
    // The point of line (j', k') on hyperplane s has i' = s - j' - k', so its
    // element index is linear in (s, j', k'): a lane's addresses along the
    // block are additions.
    const int sx = (dir & 1) ? -1 : 1;
    const int64_t dj = ((dir & 2) ? -(int64_t)nx : (int64_t)nx) - sx;
    const int64_t dk = ((dir & 4) ? -(int64_t)nx * ny : (int64_t)nx * ny) - sx;
    const int64_t org = ((dir & 4) ? (int64_t)(nz - 1) * nx * ny : 0) +
                        ((dir & 2) ? (int64_t)(ny - 1) * nx : 0) + ((dir & 1) ? nx - 1 : 0);
    // Staging: half-wave h takes lines lj = h, h + 8, (h + 16) of each lk, its
    // lanes the 32 planes of the block, which are consecutive in memory.  All
    // loads are issued before any is used (an absent point loads element 0,
    // so none sits under a branch), then staged with those points as kFar.
    const int h = tid >> 5, tp = tid & 31;
    constexpr int NJ = 3;
    float v[T][NJ], ve[3];
    uint32_t in[T];
#pragma unroll
    for (int lk = 0; lk < T; ++lk) {
        const int k = k0 + lk - 1;
        const bool kok = k >= 0 && k < nz;
        const int64_t rk = org + (int64_t)k * dk + (int64_t)sx * s0;   // uniform
        in[lk] = 0;
#pragma unroll
        for (int q = 0; q < NJ; ++q) {
            const int lj = h + 8 * q, j = j0 + lj - 1, i = s0 + tp - j - k;
            const bool ok = kok && lj < T && j >= 0 && j < ny && (uint32_t)i < (uint32_t)nx;
            const int64_t at = rk + j * dj + sx * tp;
            v[lk][q] = u[ok ? at : 0];
            in[lk] |= ok ? 1u << q : 0u;
        }
    }
    // the planes before and after the block's, for all lines
    bool ine[3];
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int c = tid + NT * r, t = c < T * T ? -1 : kSs, l = c < T * T ? c : c - T * T;
        const int j = j0 + l % T - 1, k = k0 + l / T - 1, i = s0 + t - j - k;
        ine[r] = c < 2 * T * T && j >= 0 && j < ny && k >= 0 && k < nz && (uint32_t)i < (uint32_t)nx;
        ve[r] = u[ine[r] ? org + (int64_t)k * dk + j * dj + (int64_t)sx * (s0 + t) : 0];
    }
    if (tid == 0) any = 0;
#pragma unroll
    for (int lk = 0; lk < T; ++lk)
#pragma unroll
        for (int q = 0; q < NJ; ++q) {
            const float w = in[lk] >> q & 1 ? v[lk][q] : kFar;
            if (q < 2 || h < T - 16) tile[(tp + 1) * PL + lk * T + h + 8 * q] = w;
        }
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const int c = tid + NT * r, t = c < T * T ? 0 : kSs + 1, l = c < T * T ? c : c - T * T;
        if (c < 2 * T * T) tile[t * PL + l] = ine[r] ? ve[r] : kFar;
    }
    __syncthreads();
    const int lj = tid % kSj, lk = tid / kSj;
    // planes on which the thread's line has a point: ta .. ta + tn - 1
    const int i0 = s0 - (j0 + lj) - (k0 + lk);              // i' at the first plane
    const bool line_in = j0 + lj < ny && k0 + lk < nz;
    const int ta = max(0, -i0), tn = line_in ? max(min(kSs, nx - i0) - ta, 0) : 0;
    float *p = &tile[(lk + 1) * T + lj + 1];                // own line, plane s - 1
    float prev = p[0], me = p[PL];
#pragma unroll 2
    for (int t = 0; t < kSs; ++t, p += PL) {
        const float next = p[2 * PL];
        const float bb = min_num(p[-1], p[2 * PL + 1]);
        const float c = min_num(p[-T], p[2 * PL + T]);
        float a = min_num(prev, next);
        const float w = godunov(a, bb, c);   // a: the smallest of the three now
        if (w < me && (uint32_t)(t - ta) < (uint32_t)tn && !(a >= kFar)) {
            me = w;
            p[PL] = w;
            any = 1;
        }
        prev = me;
        me = next;
        __syncthreads();
    }
    if (!any) return;
    // planes 1..kSs of the block's own lines
#pragma unroll 4
    for (int lk2 = 0; lk2 < kSj; ++lk2) {
        const int k = k0 + lk2;
        const int64_t rk = org + (int64_t)k * dk + (int64_t)sx * s0;
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int lj2 = h + 8 * q, j = j0 + lj2, i = s0 + tp - j - k;
            if (k < nz && j < ny && (uint32_t)i < (uint32_t)nx)
                u[rk + j * dj + sx * tp] = tile[(tp + 1) * PL + (lk2 + 1) * T + lj2 + 1];
        }
    }
}

__global__ __launch_bounds__(kThreads) void offset_kernel(const float *u, float *phi, int64_t n,
                                                          float offset)
{
    for (int64_t i = blockIdx.x * (int64_t)kThreads + threadIdx.x; i < n;
         i += (int64_t)gridDim.x * kThreads)
        glb(phi)[i] = offset - glb(u)[i];
}

unsigned stride_grid(int64_t n)
{
    const int64_t g = (n + kThreads - 1) / kThreads;
    return (unsigned)std::min<int64_t>(std::max<int64_t>(g, 1), 65536);
}

}  // namespace

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------

hipError_t launch_gather(const void *src, void *dst, int elem_bytes, int64_t nx, int64_t ny,
                         const SubBox &b, hipStream_t s)
{
    const int64_t n = (int64_t)b.ext[0] * b.ext[1] * b.ext[2];
    if (elem_bytes == 4)
        hipLaunchKernelGGL(gather_kernel<float>, dim3(stride_grid(n)), dim3(kThreads), 0, s,
                           static_cast<const float *>(src), static_cast<float *>(dst), nx, ny, b);
    else if (elem_bytes == 2)
        hipLaunchKernelGGL(gather_kernel<uint16_t>, dim3(stride_grid(n)), dim3(kThreads), 0, s,
                           static_cast<const uint16_t *>(src), static_cast<uint16_t *>(dst), nx, ny,
                           b);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_merge(float *acc, const float *tile, int64_t nx, int64_t ny, const SubBox &b,
                        int curtain, hipStream_t s)
{
    const int64_t n = (int64_t)b.ext[0] * b.ext[1] * b.ext[2];
    hipLaunchKernelGGL(merge_kernel, dim3(stride_grid(n)), dim3(kThreads), 0, s, acc, tile, nx, ny,
                       b, curtain);
    return hipGetLastError();
}

// dtype codes as in rsf.h
constexpr int F32 = 0, F16 = 1, BF16 = 2, U16 = 3;

hipError_t launch_smooth_x(const void *img, int image_dtype, float *out, int64_t nx, int64_t ny,
                           int64_t nz, const Taps &t, int R, hipStream_t s)
{
    const int64_t n = nx * ny * nz;
    if (image_dtype == U16)
        hipLaunchKernelGGL(smooth_x_kernel<uint16_t>, dim3(stride_grid(n)), dim3(kThreads), 0, s,
                           static_cast<const uint16_t *>(img), out, nx, n, t, R);
    else
        hipLaunchKernelGGL(smooth_x_kernel<float>, dim3(stride_grid(n)), dim3(kThreads), 0, s,
                           static_cast<const float *>(img), out, nx, n, t, R);
    return hipGetLastError();
}

hipError_t launch_smooth_y(const float *in, float *out, int64_t nx, int64_t ny, int64_t nz,
                           const Taps &t, int R, hipStream_t s)
{
    const int64_t n = nx * ny * nz;
    hipLaunchKernelGGL(smooth_y_kernel, dim3(stride_grid(n)), dim3(kThreads), 0, s, in, out, nx, ny,
                       n, t, R);
    return hipGetLastError();
}

hipError_t launch_hessian(const float *L, float *doh, float *tr, float *part, int64_t nx,
                          int64_t ny, int64_t nz, int *blocks, hipStream_t s)
{
    const int64_t n = nx * ny * nz;
    const unsigned g = stride_grid(n);
    *blocks = (int)g;
    hipLaunchKernelGGL(hessian_kernel, dim3(g), dim3(kThreads), 0, s, L, doh, tr, part, nx, ny, n);
    return hipGetLastError();
}

hipError_t launch_max(const float *part, int n, float *out, hipStream_t s)
{
    hipLaunchKernelGGL(max_kernel, dim3(1), dim3(kThreads), 0, s, part, n, out);
    return hipGetLastError();
}

hipError_t launch_seeds(const float *doh, const float *tr, const float *maxv, float threshold,
                        unsigned char *mask, float *u, unsigned *cnt, int64_t nx, int64_t ny,
                        int64_t nz, hipStream_t s)
{
    const int64_t n = nx * ny * nz;
    hipLaunchKernelGGL(seeds_kernel, dim3(stride_grid(n)), dim3(kThreads), 0, s, doh, tr, maxv,
                       threshold, mask, u, cnt, nx, ny, n);
    return hipGetLastError();
}

int64_t sweep_wavefronts(int64_t nx, int64_t ny, int64_t nz)
{
    const int64_t nbj = (ny + kSj - 1) / kSj, nbk = (nz + kSj - 1) / kSj;
    return (nx + ny + nz - 2 + kSs - 1) / kSs + nbj + nbk - 2;
}

hipError_t launch_sweep_blocks(float *u, int64_t nx, int64_t ny, int64_t nz, int dir, int64_t W,
                               hipStream_t s)
{
    // (hyperplane numbers and block indices are 32 bits wide: nx ny <= 2^28 and
    // nz <= 2^30, so nx + ny + nz fits)
    const int64_t nbj = (ny + kSj - 1) / kSj, nbk = (nz + kSj - 1) / kSj,
                  nb = (nx + ny + nz - 2 + kSs - 1) / kSs;
    // block diagonals D = J + K for which b = W - D is one of the nb blocks of
    // hyperplanes; those whose lines have no point on them leave in the kernel
    const int64_t dlo = std::max<int64_t>(0, W - (nb - 1));
    const int64_t dhi = std::min<int64_t>(nbj + nbk - 2, W);
    if (dhi < dlo) return hipSuccess;
    const int64_t klo = std::max<int64_t>(0, dlo - (nbj - 1)), khi = std::min<int64_t>(nbk - 1, dhi);
    if (khi < klo) return hipSuccess;
    const int64_t g = nbj * (khi - klo + 1);
    if (g > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL(sweep_block_kernel, dim3((unsigned)g), dim3(kSj * kSj), 0, s, u, (int)nx,
                       (int)ny, (int)nz, dir, (int)W, (int)nb, (int)nbj, (int)klo);
    return hipGetLastError();
}

hipError_t launch_offset(const float *u, float *phi, int64_t n, float offset, hipStream_t s)
{
    hipLaunchKernelGGL(offset_kernel, dim3(stride_grid(n)), dim3(kThreads), 0, s, u, phi, n, offset);
    return hipGetLastError();
}

hipError_t launch_fill(float *dst, int64_t n, float v, hipStream_t s)
{
    hipLaunchKernelGGL(fill_kernel, dim3(stride_grid(n)), dim3(kThreads), 0, s, dst, n, v);
    return hipGetLastError();
}

hipError_t launch_setup(const Batch &b, const Taps &t, int R, hipStream_t s)
{
    hipLaunchKernelGGL(setup_kernel, dim3(b.n), dim3(kThreads), 0, s, b, t, R);
    return hipGetLastError();
}

hipError_t launch_put_table(void *dst, const TableBlob &blob, int bytes, hipStream_t s)
{
    if (bytes < 0 || bytes > kTableBlobBytes || bytes % 4) return hipErrorInvalidValue;
    hipLaunchKernelGGL(put_table_kernel, dim3(1), dim3(kThreads), 0, s,
                       static_cast<uint32_t *>(dst), blob, bytes / 4);
    return hipGetLastError();
}

hipError_t launch_reduce(const Batch &b, const Coeffs &c, hipStream_t s)
{
    hipLaunchKernelGGL(reduce_kernel, dim3(b.n), dim3(kThreads), 0, s, b, c);
    return hipGetLastError();
}

hipError_t launch_finish(const Batch &b, int64_t blocks, hipStream_t s)
{
    hipLaunchKernelGGL(finish_kernel, dim3((unsigned)blocks), dim3(kThreads), 0, s, b);
    return hipGetLastError();
}


bool types_supported(int R, int it, int st)
{
    if (R < 1 || R > kMaxR) return false;
    if (it == F32 && st == F32) return true;
    if (R < kMinRMixed || R > kMaxRMixed) return false;
    return (it == F32 || it == U16) && (st == F32 || st == F16 || st == BF16);
}

// Expand CALL(RR, IT, ST) for the built (radius, image, storage) combination
// matching the runtime (R, it, st).
#define RSF_R_ALL(X, IT, ST) \
    X(1, IT, ST) X(2, IT, ST) X(3, IT, ST) X(4, IT, ST) X(5, IT, ST) X(6, IT, ST) X(7, IT, ST) \
    X(8, IT, ST) X(9, IT, ST) X(10, IT, ST) X(11, IT, ST) X(12, IT, ST) X(13, IT, ST)          \
    X(14, IT, ST) X(15, IT, ST) X(16, IT, ST)
#define RSF_R_MIXED(X, IT, ST) \
    X(4, IT, ST) X(5, IT, ST) X(6, IT, ST) X(7, IT, ST) X(8, IT, ST) X(9, IT, ST) X(10, IT, ST) \
    X(11, IT, ST) X(12, IT, ST)
#define RSF_DISPATCH(CALL)                                                              \
    if (!types_supported(R, it, st)) return hipErrorInvalidValue;                       \
    if (it == F32 && st == F32) {                                                       \
        switch (R) { RSF_R_ALL(CALL, float, float) default: break; }                     \
    } else if (it == U16 && st == F16) {                                                \
        switch (R) { RSF_R_MIXED(CALL, uint16_t, _Float16) default: break; }             \
    } else if (it == U16 && st == BF16) {                                               \
        switch (R) { RSF_R_MIXED(CALL, uint16_t, __bf16) default: break; }               \
    } else if (it == U16 && st == F32) {                                                \
        switch (R) { RSF_R_MIXED(CALL, uint16_t, float) default: break; }                \
    } else if (it == F32 && st == F16) {                                                \
        switch (R) { RSF_R_MIXED(CALL, float, _Float16) default: break; }                \
    } else if (it == F32 && st == BF16) {                                               \
        switch (R) { RSF_R_MIXED(CALL, float, __bf16) default: break; }                  \
    }                                                                                   \
    return hipErrorInvalidValue;

hipError_t launch_xy_one(int R, int it, int st, const Batch &b, int64_t blocks, const Taps &t,
                         const Coeffs &c, hipStream_t s)
{
#define C(RR, IT, ST) \
    case RR: return launch_xy_one_r<RR, IT, ST>(b, blocks, t, c, s);
    RSF_DISPATCH(C)
#undef C
}

hipError_t launch_xyf(int R, int mode, int it, int st, const Batch &b, int64_t blocks,
                      int nw, int threads, int lds, const Taps &t, const Coeffs &c, bool probe, hipStream_t s)
{
#define C(RR, IT, ST) \
    case RR: return launch_xyf_r<RR, IT, ST>(mode, b, blocks, nw, threads, lds, t, c, probe, s);
    RSF_DISPATCH(C)
#undef C
}

hipError_t launch_z_plain(int R, int st, const Batch &b, int64_t blocks, const Taps &t,
                          int target, hipStream_t s)
{
    const int it = F32;   // the plain z pass only touches the storage type
#define C(RR, IT, ST) \
    case RR: return launch_z_plain_r<RR, ST>(b, blocks, t, target, s);
    RSF_DISPATCH(C)
#undef C
}

hipError_t launch_z_heaviside(int R, int it, int st, const Batch &b, int64_t blocks,
                              const Taps &t, const Coeffs &c, bool probe, hipStream_t s)
{
#define C(RR, IT, ST) \
    case RR: return launch_z_heaviside_r<RR, IT, ST>(b, blocks, t, c, probe, s);
    RSF_DISPATCH(C)
#undef C
}

hipError_t launch_z_update(int R, int it, int st, const Batch &b, int64_t blocks, const Taps &t,
                           const Coeffs &c, bool probe, hipStream_t s)
{
#define C(RR, IT, ST) \
    case RR: return launch_z_update_r<RR, IT, ST>(b, blocks, t, c, probe, s);
    RSF_DISPATCH(C)
#undef C
}

hipError_t launch_z_update_fused(int R, int it, int st, const Batch &b, int64_t blocks,
                                 const Taps &t, const Coeffs &c, bool paper, hipStream_t s)
{
#define C(RR, IT, ST) \
    case RR: return launch_z_update_fused_r<RR, IT, ST>(b, blocks, t, c, paper, s);
    RSF_DISPATCH(C)
#undef C
}

hipError_t launch_z_update_paper(int it, int st, const Batch &b, int64_t blocks, const Coeffs &c,
                                 bool probe, hipStream_t s)
{
    if (it == F32 && st == F32) return launch_z_update_paper_r<float, float>(b, blocks, c, probe, s);
    if (it == U16 && st == F16) return launch_z_update_paper_r<uint16_t, _Float16>(b, blocks, c, probe, s);
    if (it == U16 && st == BF16) return launch_z_update_paper_r<uint16_t, __bf16>(b, blocks, c, probe, s);
    if (it == U16 && st == F32) return launch_z_update_paper_r<uint16_t, float>(b, blocks, c, probe, s);
    if (it == F32 && st == F16) return launch_z_update_paper_r<float, _Float16>(b, blocks, c, probe, s);
    if (it == F32 && st == BF16) return launch_z_update_paper_r<float, __bf16>(b, blocks, c, probe, s);
    return hipErrorInvalidValue;
}

}  // namespace rsf

// Internal declarations shared by the kernels (rsf_kernels.hpp / .hip) and
// the C-ABI host code (rsf_api.hip).  gfx950 only.
//
// Every pass runs over a batch of tiles (independent volumes); a single
// volume is a batch of one.  A pass launches one grid for the whole batch:
// each tile owns a contiguous range of the pass's workgroups, found from a
// prefix table, so uneven tiles share one launch.
#pragma once

#include <hip/hip_runtime.h>

#include <cstddef>
#include <cstdint>
#include <type_traits>

namespace rsf {

constexpr int kMaxR = 16;          // largest Gaussian radius (sigma <= 16/3)
constexpr int kXcds = 8;           // accelerator complex dies, each with its own L2
constexpr int kCus = 256;           // compute units
constexpr int kThreads = 256;      // z pass block: consecutive columns
constexpr int kUx = 64;            // update pass: columns per block along x
constexpr int kUy = 8;             // update pass: columns per block along y
constexpr int kUThreads = kUx * kUy;
// Largest xy plane (voxels): every in-slice byte offset of an 8-byte
// element, with a workgroup's overhang, fits a 32-bit unsigned offset.
constexpr int64_t kMaxPlane = (int64_t)1 << 28;

// Image/storage combinations other than (F32, F32) are built for radii
// kMinRMixed..kMaxRMixed.
constexpr int kMinRMixed = 4;
constexpr int kMaxRMixed = 12;

// Sampled, truncated, unit-sum Gaussian taps w[k + R], k = -R..R.
struct Taps {
    float w[2 * kMaxR + 1];
};

struct Grid3 {
    int nx, ny, nz;
    int64_t sxy;  // nx * ny
};

// How each pass cuts a tile into workgroups: row chunks of the xy passes,
// z chunks of the stage-1 z pass and of the update pass.
struct Split {
    int xy, z, u;
    int f = 1;   // row chunks of the iteration's xy pass
};

// One tile of a batch as the kernels see it (device pointers).
struct TileDesc {
    Grid3 g;
    Split sp;
    const void *I;          // image, in the image type
    float *phi[2];          // phi ping-pong: [0] the caller's buffer, [1] workspace
    void *P, *Q;            // interleaved pair fields, storage type
    void *KI;               // K * I, storage type
    void *K2I, *K2I2;       // K2 * I and K2 * I^2 (Sec. 4.2 force, sigma2 > 0), storage type
    float *cx, *cy, *cz;    // K * 1 = cx[x] cy[y] cz[z]
    double *partials;       // one sum |dphi| per update-pass block
    double *hist;           // sum |dphi| per iteration run
    int hist_cap;           // entries of hist = iterations asked of this tile
    int *flags;             // [0] 0 running, 1 stopped by tol, 2 done; [1] iterations run
    // one-step probe outputs (float fields), null when unused
    float *probe_H, *probe_f1, *probe_f2, *probe_Fd, *probe_kappa, *probe_lap, *probe_R,
        *probe_E;
};

// Scalars shared by every tile of a batch.
struct Coeffs {
    float l1, l2, nu, mu, dt;
    float eps, eps_over_pi, eps2;   // delta = eps_over_pi / (eps2 + phi^2)
    float eta;
    int reg;                        // 0 double well, 1 single well
    int force;                      // 0 RSF e_i (sigma), 1 Sec. 4.2 form (sigma2)
    int square;                     // xy pass of K*I: convolve I^2 instead of I
    double tol;                     // stop a tile once sum|dphi| / voxels < tol (0: never)
};

// A pass over a batch: the tiles and the pass's workgroup prefix table (n + 1
// entries: tile t owns workgroups [start[t], start[t+1])).  A tile's current
// iterate n (flags[1]) is in phi[n & 1], so tiles of one batch may be at
// different iterations.
//
// Workgroups are dispatched to the XCDs round robin (hardware workgroup b on
// XCD b % 8).  XCD k takes the contiguous range [xcd[k], xcd[k+1]) of the
// batch's workgroups, the ranges cut for equal estimated cost; the grid is 8
// times the longest range and the surplus workgroups exit at once.
struct Batch {
    const TileDesc *tiles;
    const int *start;
    int n;
    int xcd[kXcds + 1];
};

// Workgroup counts of one tile under a split.
__host__ __device__ inline int nbx64(int nx) { return (nx + 63) / 64; }
__host__ __device__ inline int64_t xy_blocks(const Grid3 &g, const Split &s)
{
    return (int64_t)nbx64(g.nx) * s.xy * g.nz;
}
// z passes: workgroups of kThreads consecutive columns (y nx + x) times a z
// chunk.
__host__ __device__ inline int64_t z_cols(const Grid3 &g) { return (g.sxy + kThreads - 1) / kThreads; }
__host__ __device__ inline int64_t z_blocks(const Grid3 &g, const Split &s)
{
    return z_cols(g) * s.z;
}
__host__ __device__ inline int64_t u_blocks(const Grid3 &g, const Split &s)
{
    return (int64_t)((g.nx + kUx - 1) / kUx) * ((g.ny + kUy - 1) / kUy) * s.u;
}

// Strips of the iteration's xy pass: a workgroup of up to `nw` waves (64
// columns each) computes `width` columns and stores all but the `halo` columns
// it shares with a neighbouring strip.  Of the few smallest strip counts, the
// one with the fewest waves in all.  With more than one strip (4 or 8 waves)
// every strip is at least 128 wide, so that its threads can load a group's x
// halo (8 R elements) at one each; the last one is moved left to its full width.
struct XyfStrips {
    int n, width, step;
};
__host__ __device__ inline XyfStrips xyf_strips(int nx, int halo, int nw)
{
    const int most = 64 * nw;
    if (nx <= most) return XyfStrips{1, nx, nx};
    const int full = most - 2 * halo;
    const int least = (nx - 2 * halo + full - 1) / full;
    XyfStrips best{0, 0, 0};
    int waves = 0;
    for (int n = least; n < least + 4; ++n) {
        const int w = (int)(((int64_t)nx + (int64_t)2 * halo * (n - 1) + n - 1) / n);
        if (n > least && w < 128) break;
        const int step = w - 2 * halo;
        const int m = (nx - 2 * halo + step - 1) / step;   // strips that hold a column of their own
        const int k = m * ((w + 63) / 64);
        if (best.n == 0 || k < waves) {
            best = XyfStrips{m, w, step};
            waves = k;
        }
    }
    return best;
}
// Threads of the workgroup that covers a strip.
__host__ __device__ inline int xyf_threads(int nx, int halo, int nw)
{
    return (xyf_strips(nx, halo, nw).width + 63) / 64 * 64;
}
// Workgroups of a tile in the iteration's xy pass.
__host__ __device__ inline int64_t xyf_blocks(const Grid3 &g, const Split &s, int halo, int nw)
{
    return (int64_t)xyf_strips(g.nx, halo, nw).n * s.f * g.nz;
}

// Workgroups a whole batch aims at per pass: xy waves, z-pass workgroups,
// update-pass workgroups.
struct Targets {
    int64_t xy, z, u;
};
constexpr Targets kDefaultTargets{16384, 2048, 1024};

// Split of one volume aiming at the given workgroup counts per pass (the
// autotuner varies them); every chunk is non-empty and at least 8 long.
// R, halo: Gaussian radius and halo of the iteration's xy pass.
Split make_split(const Grid3 &g, int64_t xy_waves, int64_t z_target, int64_t u_target, int R = 9,
                 int halo = 9);
// Split of a tile holding fraction `share` of its batch's voxels: that share
// of the batch's targets.
Split default_split(const Grid3 &g, double share = 1.0, const Targets &tg = kDefaultTargets,
                    int R = 9, int halo = 9);
// Split of a single volume from the resident capacity of the z and update
// passes (R: Gaussian radius): z chunks are chosen so that the launches' last
// round of workgroups is not left nearly empty, and down to 2 slices long where
// the volume is too small to fill the GPU.
Split capacity_split(const Grid3 &g, int R, int halo);
// Workgroups the GPU keeps resident at once: z passes (256-thread groups at
// 8 per CU) and the update pass (512-thread groups at 2 per CU), on 256 CUs.
constexpr int64_t kResidentZ = 2048;
constexpr int64_t kResidentU = 512;
// Waves of the xy pass's march that a SIMD holds (registers): what the kernels
// are compiled for (`two`: with both Gaussian stages), the most each radius
// allows without a spill.
__host__ __device__ constexpr int xyf_simd_waves(int R, bool two)
{
    return two ? (R <= 7 ? 4 : R <= 10 ? 3 : 2) : (R <= 4 ? 5 : R <= 10 ? 4 : R <= 15 ? 3 : 2);
}
// Workgroups of `waves` waves that a CU holds: by registers, and by LDS 4 of up
// to 4 waves or 2 of up to 8.  One stage is planned with 3 waves per SIMD up to
// R = 9, 2 above and 4 workgroups, which is fewer than fit: its large volumes are
// bound by HBM, and a plan that fills every place once, so that all chunks march
// in step, is the slower one (512^3, R = 9: one chunk in one round of 4 per CU
// 606 us, three chunks 567).
int xyf_resident(int R, bool two, int nw, int waves);
// Load of the busiest SIMD while a CU holds `k` such workgroups, in waves: a
// step of four rows takes a SIMD about 2600 clocks per wave (R = 9; it is bound by
// the matrix and vector units) and no less than about 3900, one wave's own
// latency, hence 1.5 or more.
double xyf_load(int waves, int64_t k);
// The small-volume form of the xy pass (RSF force): a workgroup of 8 waves
// holds a chunk's rows in LDS.  Groups of four rows that are x-convolved in
// stage 1, whose fits are taken, and that are stored, for `len` rows.
constexpr int kXysThreads = 512;
struct XysRows {
    int a, b, c;
};
__host__ __device__ inline XysRows xys_rows(int len, int R)
{
    XysRows n{};
    n.c = (len + 3) / 4;
    n.b = (4 * n.c + 2 * R + 3) / 4;
    n.a = (4 * n.b + 2 * R + 3) / 4;
    return n;
}
// Row stride (floats) of its rows of 64 nw columns and their halo.
__host__ __device__ inline int xys_stride(int nw, int R)
{
    const int need = 64 * nw + (2 * R + 4 + 3) / 4 * 4;
    const int m = need % 64;
    return need + (m <= 16 ? 16 - m : (m <= 48 ? 48 - m : 80 - m));
}
inline int64_t xys_lds(int len, int R, int nw)
{
    return (int64_t)xys_rows(len, R).a * 4 * 2 * (xys_stride(nw, R) + 64 * nw) * 4;
}
constexpr int64_t kXysLds = 156 * 1024;   // of a CU's 160 KB

// Workgroup size (4 or 8 waves) and row chunks of the xy pass for a single
// volume, or nw = 2: the small-volume form with f chunks.  For the march: the
// least time of the busiest CU, in rows: rounds of resident workgroups x rows
// (the chunk, R + `halo` rows of its neighbours' on either side, two groups of
// latency) x load.  192 x 320 x 352, R = 9, FP16 fields: two strips of 3 waves in
// two chunks 0.76 x the time of one strip of 6 waves.  The small form's time is
// that of its products on the busiest CU (each group of four rows of 64 columns
// 2 (2R + 4) instructions of 8 clocks, 3.6 x that with two waves per SIMD and
// the rest) plus its chain of loads and barriers (about 6 us); 1 us is 3.5 rows
// in the march's unit.  64^3: 20 -> 12 us; at 108 x 172 x 140, R = 6 it would take
// 64 us where the march takes 36.  It is taken in one round of workgroups only: a
// second one has nothing to overlap its chain with (169 x 304 x 56, R = 5: 39 us
// in two rounds, the march 27).
struct XyfPick {
    int nw, f;
};
XyfPick xyf_pick(const Grid3 &g, int R, int halo);
// Workgroup size (4 or 8 waves) for a batch of several tiles with row chunks f:
// the least sum of their workgroups' times.  Two stages recompute a 2R-column
// halo per strip, so long rows go to 8 waves (512^3, R = 9: one 512-column strip
// 0.62 ms, three of 183 columns 0.74 ms) unless the strips leave much of such a
// workgroup's LDS unused and put two waves on one SIMD and one on the others
// (114- to 274-column tiles: 0.74 ms with 4, 1.33 ms with 8).  Taken over all
// tiles, not the narrowest: 400 and 600 columns 109 -> 74 us (4 instead of 8),
// one tile of 100 and six of 512, R = 12, FP16 356 -> 272 (8 instead of 4).
int xyf_batch_waves(const Grid3 *g, const Split *sp, int n, int R, int halo);
// Update-pass workgroups of a tile under any valid split are at most this:
// chunks of 8 slices, or, where those are fewer than the GPU holds, of 2.
__host__ __device__ inline int64_t u_blocks_max(const Grid3 &g)
{
    const int64_t cols = (int64_t)((g.nx + kUx - 1) / kUx) * ((g.ny + kUy - 1) / kUy);
    const int64_t by8 = cols * ((g.nz + 7) / 8), by2 = cols * ((g.nz + 1) / 2);
    const int64_t small = by2 < kResidentU ? by2 : kResidentU;
    return by8 > small ? by8 : small;
}
bool split_valid(const Grid3 &g, const Split &s);

bool types_supported(int R, int image_dtype, int storage_dtype);

// Modes of the iteration's xy pass: XY_RSF reads the pair P and K*I and writes
// the pair Q = Kxy*(g1, g2); XY_PAPER reads the pair P, K*I and the image and
// writes the Sec. 4.2 force with sigma2 = 0 to Q as float; XY_PAPER2 reads
// K2*I and K2*I^2 in place of the image (sigma2 > 0).  (The numbers follow
// those the profiles name.)
enum XyMode { XY_PAPER = 3, XY_PAPER2 = 4, XY_RSF = 5 };
// Where the plain z pass writes: K*I, K2*I or K2*I^2.
enum ZTarget { Z_TO_KI = 0, Z_TO_K2I = 1, Z_TO_K2I2 = 2 };

// One workgroup per tile: K*1 edge tables, flags cleared.
hipError_t launch_setup(const Batch &b, const Taps &t, int R, hipStream_t s);
// A small host-built table written to device memory by a kernel from its own
// argument: no pinned staging buffer and no copy, for the entry point that
// allocates nothing.
constexpr int kTableBlobBytes = 2048;
struct TableBlob {
    uint32_t w[kTableBlobBytes / 4];
};
hipError_t launch_put_table(void *dst, const TableBlob &blob, int bytes, hipStream_t s);
// The image (or its square) -> the field P, for K*I.
hipError_t launch_xy_one(int R, int image_dtype, int storage_dtype, const Batch &b, int64_t blocks,
                         const Taps &t, const Coeffs &c, hipStream_t s);
// The iteration's xy pass: P (and K*I, ...) -> Q (mode XY_RSF, XY_PAPER, XY_PAPER2).
// `nw`: 4 or 8 (the march) with `threads`, 64 times the most waves a strip of
// the batch's tiles holds; or 2 (the small-volume form) with its `lds` bytes.
hipError_t launch_xyf(int R, int mode, int image_dtype, int storage_dtype, const Batch &b,
                      int64_t blocks, int nw, int threads, int lds, const Taps &t,
                      const Coeffs &c, bool probe, hipStream_t s);
// K*I: the z pass of P into KI.
hipError_t launch_z_plain(int R, int storage_dtype, const Batch &b, int64_t blocks,
                          const Taps &t, int target, hipStream_t s);
// Stage-1 z pass: (phi, I) -> the pair P = (Kz*(H I), Kz*H).
hipError_t launch_z_heaviside(int R, int image_dtype, int storage_dtype, const Batch &b,
                              int64_t blocks, const Taps &t, const Coeffs &c, bool probe,
                              hipStream_t s);
// Stage-2 z pass of the pair Q = (Kxy*g1, Kxy*g2) and the update into the
// other phi buffer, with per-block |dphi| partial sums.
hipError_t launch_z_update(int R, int image_dtype, int storage_dtype, const Batch &b,
                           int64_t blocks, const Taps &t, const Coeffs &c, bool probe,
                           hipStream_t s);
// The update reading the Sec. 4.2 force (sigma2 = 0) that XY_PAPER wrote.
hipError_t launch_z_update_paper(int image_dtype, int storage_dtype, const Batch &b,
                                 int64_t blocks, const Coeffs &c, bool probe, hipStream_t s);
// Largest Gaussian radius whose RSF-force update is fused with the next
// stage-1 pass (the Sec. 4.2 force's update has no stage-2 ring: any radius).
// A stage-2 ring slot holds two floats with FP32 or BF16 storage and one
// packed pair with FP16 storage, which leaves room for the stage-1 ring and
// the prefetched stage with no spill in the march up to radius 9 (8 with a
// uint16 image), resp. 12 (storage and image dtypes as in rsf_dtype: 1 is
// FP16, 3 uint16).
constexpr int kFuseMaxR = 9;
constexpr int kFuseMaxRU16 = 8;
constexpr int kFuseMaxRPacked = 12;
template <class ST, class IT>
constexpr int fuse_max_r_t = std::is_same<ST, _Float16>::value
                                 ? kFuseMaxRPacked
                                 : (std::is_same<IT, uint16_t>::value ? kFuseMaxRU16 : kFuseMaxR);
inline int fuse_max_r(int storage_dtype, int image_dtype)
{
    return storage_dtype == 1 ? kFuseMaxRPacked : (image_dtype == 3 ? kFuseMaxRU16 : kFuseMaxR);
}
// The update (RSF force, or the Sec. 4.2 force if `paper`) fused with the
// next iteration's stage-1 z pass (writes P from phi' as launch_z_heaviside
// would); every tile marched whole in z.
hipError_t launch_z_update_fused(int R, int image_dtype, int storage_dtype, const Batch &b,
                                 int64_t blocks, const Taps &t, const Coeffs &c, bool paper,
                                 hipStream_t s);
// One workgroup per tile: fixed-order FP64 sum of the partials; counts the
// iteration and stops the tile at its tolerance or its last iteration.
hipError_t launch_reduce(const Batch &b, const Coeffs &c, hipStream_t s);
// Copy an odd final iterate from phi[1] to phi[0] (workgroups of the z pass).
hipError_t launch_finish(const Batch &b, int64_t blocks, hipStream_t s);

// Volume-level driver (Sec. 4.1): one sub-volume box of a large volume.
struct SubBox {
    int lo[3], ext[3];              // x, y, z origin and extent in the volume
    int core_lo[3], core_hi[3];     // its core (the part it owns outright)
    int nb_lo[3], nb_hi[3];         // 1 when a neighbour shares the face
};
// Copy box `b` of the volume (elements of elem_bytes, 2 or 4) into a dense
// tile buffer.
hipError_t launch_gather(const void *src, void *dst, int elem_bytes, int64_t nx, int64_t ny,
                         const SubBox &b, hipStream_t s);
// acc += w * tile over box b, w the product of per-axis linear ramps across
// the 2C-wide overlaps with the box's neighbours (the curtain).
hipError_t launch_merge(float *acc, const float *tile, int64_t nx, int64_t ny, const SubBox &b,
                        int curtain, hipStream_t s);
hipError_t launch_fill(float *dst, int64_t n, float v, hipStream_t s);

// Initialisation (Sec. 4.3).  Slices smoothed by the 2D Gaussian (x pass from
// the image, then y pass), the determinant and trace of the in-slice Hessian
// with per-workgroup maxima of the determinant, the seed mask, and one fast
// sweeping hyperplane.
constexpr float kFar = 1e30f;        // distance of a voxel no seed has reached
hipError_t launch_smooth_x(const void *img, int image_dtype, float *out, int64_t nx, int64_t ny,
                           int64_t nz, const Taps &t, int R, hipStream_t s);
hipError_t launch_smooth_y(const float *in, float *out, int64_t nx, int64_t ny, int64_t nz,
                           const Taps &t, int R, hipStream_t s);
// doh, trace from L; partial maxima of doh into part[blocks]; returns blocks
hipError_t launch_hessian(const float *L, float *doh, float *tr, float *part, int64_t nx,
                          int64_t ny, int64_t nz, int *blocks, hipStream_t s);
// max of part[0..n) into out[0] (one workgroup, fixed order)
hipError_t launch_max(const float *part, int n, float *out, hipStream_t s);
// mask and u (0 at seeds, kFar elsewhere); per-workgroup seed counts into cnt
hipError_t launch_seeds(const float *doh, const float *tr, const float *maxv, float threshold,
                        unsigned char *mask, float *u, unsigned *cnt, int64_t nx, int64_t ny,
                        int64_t nz, hipStream_t s);
// Fast sweeping by wavefronts of blocks: a sweep with axis orders dir (bit
// 0: x descending, bit 1: y, bit 2: z) is sweep_wavefronts() launches of
// launch_sweep_blocks with W = 0, 1, ...
int64_t sweep_wavefronts(int64_t nx, int64_t ny, int64_t nz);
hipError_t launch_sweep_blocks(float *u, int64_t nx, int64_t ny, int64_t nz, int dir, int64_t W,
                               hipStream_t s);
// phi = offset - u
hipError_t launch_offset(const float *u, float *phi, int64_t n, float offset, hipStream_t s);

// Per-radius, per-type launchers behind the dispatchers (rsf_kernels.hpp).
template <int R, class IT, class ST>
hipError_t launch_xy_one_r(const Batch &b, int64_t blocks, const Taps &t, const Coeffs &c,
                           hipStream_t s);
template <int R, class IT, class ST>
hipError_t launch_xyf_r(int mode, const Batch &b, int64_t blocks, int nw, int threads, int lds,
                        const Taps &t, const Coeffs &c, bool probe, hipStream_t s);
template <int R, class ST>
hipError_t launch_z_plain_r(const Batch &b, int64_t blocks, const Taps &t, int target,
                            hipStream_t s);
template <int R, class IT, class ST>
hipError_t launch_z_heaviside_r(const Batch &b, int64_t blocks, const Taps &t, const Coeffs &c,
                                bool probe, hipStream_t s);
template <int R, class IT, class ST>
hipError_t launch_z_update_r(const Batch &b, int64_t blocks, const Taps &t, const Coeffs &c,
                             bool probe, hipStream_t s);
template <class IT, class ST>
hipError_t launch_z_update_paper_r(const Batch &b, int64_t blocks, const Coeffs &c, bool probe,
                                   hipStream_t s);
template <int R, class IT, class ST>
hipError_t launch_z_update_fused_r(const Batch &b, int64_t blocks, const Taps &t, const Coeffs &c,
                                   bool paper, hipStream_t s);

}  // namespace rsf

// The xy pass of an iteration: both Gaussian stages' x and y convolutions of
// one z slice, with the region fits between them, in one kernel (RSF force),
// or the one stage of the Sec. 4.2 force with its pointwise epilogue.
#pragma once

#include <type_traits>
#include <utility>

#include "rsf_device.hpp"

namespace rsf {

namespace {

template <int I>
using ic = std::integral_constant<int, I>;
template <class F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>)
{
    (f(ic<I>{}), ...);
}
// f(ic<0>), ..., f(ic<N - 1>): indices that reach an instruction as immediates
template <int N, class F>
__device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}
template <class F, int... I>
__device__ __forceinline__ bool all_of_impl(F &&f, std::integer_sequence<int, I...>)
{
    return (f(ic<I>{}) && ...);
}

using f4 = float __attribute__((ext_vector_type(4)));
using f4u = float __attribute__((ext_vector_type(4), aligned(4)));

// The 2R + 1 taps as operands of v_mfma_f32_4x4x1 (16 blocks of a 4 x 4 outer
// product; lane l is column l % 4 of block l / 4 as operand B and row l % 4
// as operand A).  Four consecutive outputs of a convolution take one input
// element with four consecutive taps: pattern p holds w[p - 3 + 0..3], zero
// outside 0..2R, for p = 0 .. 2R + 3.
//   y: operand A, block b of register q is pattern 16 q + b; the instruction
//      broadcasts one block to all (cbsz 4, abid b), so every lane's column
//      receives the same four taps.
//   x: operand B, 16-lane group g of register q is the pattern of input
//      4 q + g (w[k - 0..3], the mirrored one), broadcast by blgp 4 + g.
template <int R>
struct TapOps {
    static constexpr int N = 2 * R + 4;
    float y[(N + 15) / 16], x[(N + 3) / 4];
    __device__ __forceinline__ void load(const Taps &t, int lane)
    {
        auto w = [&](int i) { return i >= 0 && i <= 2 * R ? t.w[min(max(i, 0), 2 * R)] : 0.f; };
#pragma unroll
        for (int q = 0; q < (N + 15) / 16; ++q) y[q] = w(16 * q + lane / 4 - 3 + lane % 4);
#pragma unroll
        for (int q = 0; q < (N + 3) / 4; ++q) x[q] = w(4 * q + lane / 16 - lane % 4);
    }
};

// The zeros of a pattern stand for taps outside the window.  They add nothing
// while the element is finite; an Inf or NaN times such a zero is a NaN up to
// three rows or columns past the window, which ones depending on where the
// groups of four begin, that is on the split.  So sums that hold a NaN are
// taken again without the zeros, and a non-finite voxel reaches R voxels under
// any split, as it does in the one-field pass of K*I.  A wrong value is a NaN
// that its own output row takes in, so the march looks at the sums it completes
// last (512^3, R = 9: FP32 fields 670 -> 673 us, FP16 588 -> 599) and runs its
// chunk once more; the small form looks at each of its sums (64^3: 13.8 -> 13.4).
//
// The wave's lanes with a NaN among the values (an instruction for two of them).
__device__ __forceinline__ uint64_t nan_lanes(const f4 &a, const f4 &b)
{
    float m = 0.f;
#pragma unroll
    for (int i = 0; i < 4; ++i)
        m = __builtin_elementwise_maximum(__builtin_elementwise_maximum(m, __builtin_fabsf(a[i])),
                                          __builtin_fabsf(b[i]));
    return __builtin_amdgcn_ballot_w64(m != m);
}
// Sums a[i] of w[k] src[i si + k sk] in the order of k; field b is `fb` on.
template <int R>
__device__ __forceinline__ void conv_exact(const float *src, int si, int sk, int fb, const Taps &t,
                                           f4 &a, f4 &b)
{
    a = b = f4{};
#pragma clang loop unroll(disable)
    for (int k = 0; k <= 2 * R; ++k) {
        const float w = t.w[k];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            a[i] = fmaf(w, src[i * si + k * sk], a[i]);
            b[i] = fmaf(w, src[fb + i * si + k * sk], b[i]);
        }
    }
}
// acc + the taps of pattern P inside the window times v
template <int R, int P>
__device__ __forceinline__ void tap4_exact(f4 &acc, float v, const TapOps<R> &tp, const Taps &t)
{
    if constexpr (P >= 3 && P <= 2 * R) {
        acc = __builtin_amdgcn_mfma_f32_4x4x1f32(tp.y[P / 16], v, acc, 4, P % 16, 0);
    } else {
        static_for<4>([&](auto jc) {
            constexpr int j = jc, k = P - 3 + j;
            if constexpr (k >= 0 && k <= 2 * R) acc[j] = fmaf(tap<R>(t, k), v, acc[j]);
        });
    }
}

// Raw buffer of exactly `bytes` (at most 2 GiB): a load at an offset outside
// it returns 0, a store is dropped.  Rows above or below the slice (offsets
// that are negative, hence huge, or past its end) are then the zero padding
// with no mask, and a lane with nothing to load or store sets the top bit of
// its offset.
constexpr uint32_t kOut = 0x80000000u;
__device__ __forceinline__ rsrc_t rsrc_n(const void *base, uint32_t bytes)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0, (int)bytes,
                                             kRsrcFlags);
}
template <class T>
__device__ __forceinline__ T bld_at(rsrc_t r, uint32_t off)
{
    if constexpr (sizeof(T) == 2)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b16(r, off, 0, 0));
    else if constexpr (sizeof(T) == 4)
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b32(r, off, 0, 0));
    else
        return __builtin_bit_cast(T, __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, 0));
}
template <class T>
__device__ __forceinline__ void bst_at(rsrc_t r, uint32_t off, T v)
{
    if constexpr (sizeof(T) == 4) {
        __builtin_amdgcn_raw_buffer_store_b32(__builtin_bit_cast(unsigned int, v), r, off, 0, 0);
    } else {
        static_assert(sizeof(T) == 8, "4 or 8-byte elements");
        using U2 = unsigned int __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(U2, v), r, off, 0, 0);
    }
}

// A workgroup owns a strip of at most 64 NW columns of one slice (64 per
// wave) and a chunk of rows, and marches down it four rows per step.  Step G:
//   - rows of group G (with an R halo in x) are in LDS; each lane x-convolves
//     them for its column (operand A: lane 4 b + i reads row i from column
//     4 b; the result's register is the row, its lane the column);
//   - each of the four x-convolved rows is added into the sums of every
//     output row it reaches (y): NG groups of four rows are open at a time,
//     the oldest of which is complete at the end of the step;
//   - its region fits give g1, g2 of four rows, which go to LDS and are
//     convolved the same way in step G + 1 (RSF force), or the force of
//     Sec. 4.2, which is stored.
// Rows of group G + 1 are written to the other LDS buffer and those of G + 2
// loaded meanwhile; one barrier per step.
template <int R, int MODE, bool PROBE, int NW, class ST, class IMG>
__global__ __launch_bounds__(64 * NW)
__attribute__((amdgpu_waves_per_eu(PROBE ? 2 : xyf_simd_waves(R, MODE == XY_RSF))))
void xyf_kernel(Batch bt, Taps t, Coeffs c)
{
    constexpr bool TWO = MODE == XY_RSF;
    constexpr int NG = (2 * R + 3) / 4 + 1;          // open output groups
    constexpr int NK = TapOps<R>::N, NQ = (NK + 3) / 4;
    // a staged row: columns -R .. 64 * waves + R, read in 16-byte pieces up to
    // 4 * NQ - 4 past the last column's piece.  Row stride 16 or 48 mod 64
    // words: the 16-byte reads of 16 consecutive lanes (4 rows x 4 columns)
    // then fall on all 64 banks.
    constexpr int need = (64 * NW) + 4 * NQ;
    constexpr int S = need + ((16 - need % 64 + 64) % 64 < (48 - need % 64 + 64) % 64
                                  ? (16 - need % 64 + 64) % 64
                                  : (48 - need % 64 + 64) % 64);
    constexpr int BUF = 2 * 4 * S;                   // [field][row][column]
    __shared__ __attribute__((aligned(16))) float lds[(TWO ? 4 : 2) * BUF];
    __shared__ int redo;                             // a sum of the workgroup's is NaN

    Where wh;
    if (!locate(bt, wh)) return;
    const TileDesc &d = bt.tiles[wh.t];
    if (glb(d.flags)[0]) return;
    const Grid3 g = d.g;
    const XyfStrips sg = xyf_strips(g.nx, MODE == XY_RSF ? R : 0, NW);
    const int strip = wh.lb % sg.n, rest = wh.lb / sg.n;
    const int yc = rest % d.sp.f, z = rest / d.sp.f;
    const int ly = (g.ny + d.sp.f - 1) / d.sp.f;
    const int y0 = yc * ly, y1 = min(y0 + ly, g.ny);
    constexpr int H = TWO ? R : 0;                   // columns a strip shares with the next
    const int c0 = min(strip * sg.step, g.nx - sg.width);   // first column of the strip
    const int nw = (sg.width + 63) / 64;             // its waves
    // Waves past the strip leave.  Which of the workgroup's waves these are
    // turns with the workgroup, so that no SIMD is left with fewer waves.
    const int waves = (int)blockDim.x / 64;
    const int wave = ((int)__builtin_amdgcn_readfirstlane(threadIdx.x / 64) + wh.lb) % waves;
    if (wave >= nw) return;
    const int tid = 64 * wave + (int)(threadIdx.x & 63);

    const int lane = tid & 63;
    const int64_t zb = (int64_t)z * g.sxy;
    const int x = c0 + tid;
    const bool xin = x < g.nx;
    constexpr uint32_t PB = sizeof(Vec2<ST>);
    TapOps<R> tp;
    tp.load(t, lane);

    const uint32_t plane = (uint32_t)g.sxy, nx = (uint32_t)g.nx;
    constexpr uint32_t SB = sizeof(ST), IB = sizeof(IMG);
    const rsrc_t rin = rsrc_n(static_cast<const char *>(d.P) + zb * (int64_t)PB, plane * PB);
    const rsrc_t rki = rsrc_n(static_cast<const ST *>(d.KI) + zb, plane * SB);
    const rsrc_t rim = rsrc_n(static_cast<const IMG *>(d.I) + zb, plane * IB);
    const rsrc_t rk2i = rsrc_n(static_cast<const ST *>(d.K2I) + zb, plane * SB);
    const rsrc_t rk2q = rsrc_n(static_cast<const ST *>(d.K2I2) + zb, plane * SB);
    constexpr uint32_t OB = TWO ? PB : 4u;           // bytes of an output element
    // the chunk's rows only: the output rows of priming steps and past the
    // chunk's end are dropped
    const rsrc_t rout = rsrc_n(static_cast<char *>(d.Q) + (zb + (int64_t)y0 * g.nx) * (int64_t)OB,
                               (uint32_t)(y1 - y0) * nx * OB);
    // columns this strip stores: all but the halo it shares with a neighbour
    const int o0 = strip == 0 ? 0 : strip * sg.step + H;
    const int o1 = strip == sg.n - 1 ? g.nx : c0 + sg.width - H;
    const uint32_t ibad = xin ? 0u : kOut, obad = x >= o0 && x < o1 ? 0u : kOut;
    const int xkeep = xin ? -1 : 0;
    const float cxz = glb(d.cx)[min(x, g.nx - 1)] * glb(d.cz)[z];
    const float *const cyp = d.cy;

    // x halo of the four rows of a group: thread k < 8 R takes row k / 2R,
    // halo column k % 2R (left, then right of the strip's 64 nw columns); the
    // others write to an element of the row's padding that is never read
    const int hr = tid / (2 * R), hc = tid % (2 * R);
    const bool has_h = tid < 8 * R;
    const int hx = hc < R ? c0 - R + hc : c0 + 64 * nw + hc - R;
    const uint32_t hbad = has_h && hx >= 0 && hx < g.nx ? 0u : kOut;
    const int hdst = has_h ? hr * S + (hc < R ? hc : 64 * nw + hc) : S - 1;
    static_assert((64 * NW) + 4 * NQ - 4 <= S - 1, "the padding element is past every read");

    // first input row of group 0, so that the first output row is y0
    constexpr int PAD = TWO ? 0 : (4 - 2 * R % 4) % 4;
    const int r0 = y0 - (TWO ? 2 * R : R + PAD);
    constexpr int GF = TWO ? R + 1 : (2 * R + PAD) / 4;   // step of the first output row
    const int gend = GF + (y1 - y0 + 3) / 4;
    // steps before GP complete no row the chunk uses: they only convolve and
    // sum.  A chunk that starts the volume skips the groups of zeros above it.
    constexpr int GP = TWO ? 2 * R / 4 : GF, GZ = TWO ? GP : (R + PAD) / 4;
    static_assert(GZ <= GP, "the loop starts at step GP");

    // element offset of row r of n (clamped to one row outside: on planes of
    // a few very long rows, more would wrap around to valid offsets)
    auto at_row = [&](int r, int n) { return (uint32_t)min(max(r, -1), n) * nx; };
    const uint32_t e0 = (uint32_t)x;
    struct Rows {
        Vec2<ST> m[4], h;
    };
    auto fetch = [&](int grp) {
        Rows v;
        const int row = r0 + 4 * grp;
#pragma unroll
        for (int i = 0; i < 4; ++i)
            v.m[i] = bld_at<Vec2<ST>>(rin, ((e0 + at_row(row + i, g.ny)) * PB) | ibad);
        v.h = bld_at<Vec2<ST>>(rin, (((uint32_t)hx + at_row(row + hr, g.ny)) * PB) | hbad);
        return v;
    };
    float *const wr = lds + R + tid;                 // own column of row 0
    auto put = [&](const Rows &v, int buf) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            wr[buf + i * S] = to_f(v.m[i].x);
            wr[buf + (4 + i) * S] = to_f(v.m[i].y);
        }
        lds[buf + hdst] = to_f(v.h.x);
        lds[buf + hdst + 4 * S] = to_f(v.h.y);
    };
    // pointwise inputs of the fits of the group completed in step grp
    struct Point {
        ST ki[4], k2i[4], k2q[4];
        IMG im[4];
        f4 cy;
    };
    auto point = [&](int grp) {
        Point p;
        const int rb = r0 - R + 4 * grp;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t e = e0 + at_row(rb + i, g.ny);
            p.ki[i] = bld_at<ST>(rki, e * SB);
            if constexpr (MODE == XY_PAPER) p.im[i] = bld_at<IMG>(rim, e * IB);
            if constexpr (MODE == XY_PAPER2) {
                p.k2i[i] = bld_at<ST>(rk2i, e * SB);
                p.k2q[i] = bld_at<ST>(rk2q, e * SB);
            }
        }
        // one scalar load; rows outside the table (at most 2 R + 8 entries on
        // either side) are their neighbours' in the tile's workspace, each at
        // least 64 entries long, and go nowhere
        p.cy = *(const __attribute__((address_space(4))) f4u *)(cyp + rb);
        return p;
    };
    const int aoff = (lane & 3) * S + (tid & ~63) + (lane & ~3);
    // x convolution of the four staged rows of a buffer, both fields; the LDS
    // reads run one piece (4 columns) ahead of the products
    auto xconv = [&](int buf, f4 &xa, f4 &xb) {
        f4 a{}, b{}, va[2], vb[2];
        const float *const src = lds + buf + aoff;
        auto read = [&](int q) {
            va[q & 1] = *reinterpret_cast<const f4 *>(src + 4 * q);
            vb[q & 1] = *reinterpret_cast<const f4 *>(src + 4 * S + 4 * q);
        };
        read(0);
        static_for<NQ>([&](auto qc) {
            constexpr int q = qc;
            if constexpr (q + 1 < NQ) read(q + 1);
            // (opaque: kept as 16-byte reads)
            __asm__ volatile("" : "+v"(va[q & 1]), "+v"(vb[q & 1]));
            static_for<4>([&](auto kc) {
                constexpr int k = kc;
                if constexpr (4 * q + k < NK) {
                    a = __builtin_amdgcn_mfma_f32_4x4x1f32(va[q & 1][k], tp.x[q], a, 0, 0, 4 + k);
                    b = __builtin_amdgcn_mfma_f32_4x4x1f32(vb[q & 1][k], tp.x[q], b, 0, 0, 4 + k);
                }
            });
            __builtin_amdgcn_sched_barrier(0);
        });
        xa = a;
        xb = b;
    };
    // add the four rows to the open groups (group m of the step in slot
    // (T + m) % NG; group NG - 1 starts here), rows in order
    auto ysum = [&](auto T, auto exact, f4 *sa, f4 *sb, const f4 &xa, const f4 &xb) {
        static_for<4>([&](auto ci) {
            static_for<NG>([&](auto cm) {
                constexpr int i = ci, m = cm;
                constexpr int p = 4 * m - i + 3;     // tap pattern
                if constexpr (p >= 0 && p < NK) {
                    constexpr int s = (T + m) % NG;
                    // the first row that reaches the newest group
                    constexpr bool first = m == NG - 1 && (i == 0 || p + 1 >= NK);
                    const f4 zero{};
                    if constexpr (exact) {
                        if constexpr (first) sa[s] = sb[s] = zero;
                        tap4_exact<R, p>(sa[s], xa[i], tp, t);
                        tap4_exact<R, p>(sb[s], xb[i], tp, t);
                    } else {
                        sa[s] = __builtin_amdgcn_mfma_f32_4x4x1f32(
                            tp.y[p / 16], xa[i], first ? zero : sa[s], 4, p % 16, 0);
                        sb[s] = __builtin_amdgcn_mfma_f32_4x4x1f32(
                            tp.y[p / 16], xb[i], first ? zero : sb[s], 4, p % 16, 0);
                    }
                }
            });
        });
        // opaque, or the compiler would sink sums to the step that completes
        // them and keep their inputs instead
#pragma unroll
        for (int m = 0; m < NG; ++m) __asm__ volatile("" : "+v"(sa[m]), "+v"(sb[m]));
    };
    auto conv = [&](auto T, auto exact, int buf, f4 *sa, f4 *sb) {
        f4 xa, xb;
        if constexpr (exact) conv_exact<R>(wr + buf - R, S, 1, 4 * S, t, xa, xb);
        else xconv(buf, xa, xb);
        ysum(T, exact, sa, sb, xa, xb);
    };

    const gptr<float> probe_f1 = glb(d.probe_f1), probe_f2 = glb(d.probe_f2),
                      probe_fd = glb(d.probe_Fd);
    // One march down the chunk; true if one of its sums is NaN (`exact`: the
    // sums without the patterns' zeros, one step at a time).
    auto march = [&](auto exact) -> bool {
        f4 a1[NG], b1[NG], a2[TWO ? NG : 1], b2[TWO ? NG : 1];
#pragma unroll
        for (int m = 0; m < NG; ++m) a1[m] = b1[m] = f4{};
        if constexpr (TWO) {
#pragma unroll
            for (int m = 0; m < NG; ++m) a2[m] = b2[m] = f4{};
        }
        uint64_t nans = 0;
        int G = y0 > 0 ? 0 : GZ;
        int cur = 0;                                     // LDS buffer of group G
        // the first rows are on their way while the LDS is cleared (by the 64 nw
        // threads that are left)
        const Rows first = fetch(G);
        Rows nxt = fetch(G + 1);
        for (int i = 4 * ((int)(wr - lds) - R); i < (TWO ? 4 : 2) * BUF; i += 256 * nw)
            *reinterpret_cast<f4 *>(lds + i) = f4{};
        if constexpr (!exact) redo = 0;
        __syncthreads();
        put(first, cur);

        Point pt;
        int oth = BUF;
        // stage 1 of step G; the fits' inputs are loaded here and used after it
        auto stage1 = [&](auto T, auto fits) {
            // opaque, or the compiler would keep every LDS address of both
            // buffers in a register
            __asm__ volatile("" : "+s"(cur));
            oth = BUF - cur;
            __asm__ volatile("" : "+s"(oth));
            __syncthreads();
            put(nxt, oth);
            if constexpr (fits) pt = point(G);
            nxt = fetch(G + 2);
            conv(T, exact, cur, a1, b1);
            __builtin_amdgcn_sched_barrier(0);
        };
        auto step = [&](auto T) -> bool {
            stage1(T, std::true_type{});
            const f4 A = a1[T], B = b1[T];
            const int rb = r0 - R + 4 * G;               // rows of the completed group
            float u[4], v[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                // region fits (Sec. 3 local_intensity)
                const float K1 = cxz * pt.cy[i];
                const float A2 = to_f(pt.ki[i]) - A[i];
                const float B2 = K1 - B[i];
                const float f1 = A[i] * rcp(B[i]);
                const float f2 = A2 * rcp(B2);
                if constexpr (MODE == XY_PAPER) {
                    // F+- = (I - r+-)^2 (Sec. 4.2 expansion, sigma2 = 0)
                    const float im = to_f(pt.im[i]);
                    float r1 = f1, r2 = f2;
                    if constexpr (std::is_same<IMG, uint16_t>::value) {
                        // rounded fits, so that the image's scaling is the product
                        // that contracts with the difference
                        pin(r1);
                        pin(r2);
                    }
                    const float d1 = im - r1, d2 = im - r2;
                    u[i] = c.l1 * d1 * d1 - c.l2 * d2 * d2;
                } else if constexpr (MODE == XY_PAPER2) {
                    // F+- = K2*I^2 - 2 r+- K2*I + r+-^2 (Sec. 4.2 expansion)
                    const float a = to_f(pt.k2i[i]), q = to_f(pt.k2q[i]);
                    const float F1 = q - 2.f * f1 * a + f1 * f1;
                    const float F2 = q - 2.f * f2 * a + f2 * f2;
                    u[i] = c.l1 * F1 - c.l2 * F2;
                } else {
                    // inputs of the force convolution; zero outside the volume
                    // (the row's mask opaque: a select would go through VCC)
                    int rk = ~(((rb + i) | (g.ny - 1 - rb - i)) >> 31);
                    __asm__ volatile("" : "+s"(rk));
                    const int keep = xkeep & rk;
                    float g1 = c.l1 * f1 - c.l2 * f2, g2 = c.l1 * f1 * f1 - c.l2 * f2 * f2;
                    if constexpr (!std::is_same<ST, float>::value) {
                        // rounded to FP32, then to the storage type (opaque: not
                        // in one step), as every field of an iteration is
                        pin(g1);
                        pin(g2);
                        g1 = to_f(from_f<ST>(g1));
                        g2 = to_f(from_f<ST>(g2));
                    }
                    u[i] = __int_as_float(__float_as_int(g1) & keep);
                    v[i] = __int_as_float(__float_as_int(g2) & keep);
                }
                if constexpr (PROBE) {
                    if (rb + i >= y0 && rb + i < y1 && x >= o0 && x < o1) {
                        const int64_t at = zb + (int64_t)(rb + i) * g.nx + x;
                        if (probe_f1) probe_f1[at] = f1;
                        if (probe_f2) probe_f2[at] = f2;
                        if (!TWO && probe_fd) probe_fd[at] = u[i];
                    }
                }
            }
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (TWO) {
                // this step's g into the other buffer; the previous step's is
                // convolved
                float *const wg = wr + 2 * BUF + oth;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    wg[i * S] = u[i];
                    wg[(4 + i) * S] = v[i];
                }
                conv(T, exact, 2 * BUF + cur, a2, b2);
                if constexpr (!exact) nans |= nan_lanes(a2[T], b2[T]);
            } else if constexpr (!exact) {
                nans |= nan_lanes(A, B);
            }
            const int orow = TWO ? rb - R - 4 - y0 : rb - y0;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const uint32_t off = ((e0 + at_row(orow + i, y1 - y0)) * OB) | obad;
                if constexpr (TWO) {
                    Vec2<ST> w;
                    w.x = from_f<ST>(a2[T][i]);
                    w.y = from_f<ST>(b2[T][i]);
                    bst_at<Vec2<ST>>(rout, off, w);
                } else {
                    bst_at<float>(rout, off, u[i]);
                }
            }
            cur = oth;
            return ++G < gend;
        };
        if constexpr (exact) {
            // (steps before GP too: what they complete is not stored)
            while (step(ic<0>{})) {
#pragma unroll
                for (int m = 0; m + 1 < NG; ++m) {
                    a1[m] = a1[m + 1];
                    b1[m] = b1[m + 1];
                    if constexpr (TWO) {
                        a2[m] = a2[m + 1];
                        b2[m] = b2[m + 1];
                    }
                }
            }
            return false;
        } else {
            auto prime = [&](auto j) {   // (the loop below starts in slot 0)
                G = j;
                stage1(ic<((j - GP) % NG + NG) % NG>{}, std::false_type{});
                cur = oth;
            };
            if (y0 > 0) static_for<GP>(prime);
            else static_for<GP - GZ>([&](auto j) { prime(ic<j + GZ>{}); });
            G = GP;
            while (all_of_impl(step, std::make_integer_sequence<int, NG>{})) {
            }
            return nans != 0;
        }
    };
    if (march(std::false_type{})) redo = 1;
    __syncthreads();
    if (__builtin_expect(!redo, 1)) return;
    march(std::true_type{});
}

// The xy pass of a small volume (RSF force): instead of marching down the
// rows, a workgroup of 8 waves holds all rows of its chunk in LDS and its
// waves convolve the groups of four rows side by side, one stage after the
// other.  The same products in the same order, so bitwise the same fields;
// more rows are convolved twice (the chunk's 4 R halo rows), but the chain is
// four group convolutions long instead of one for every group of the chunk.
// The march's 11 steps at 64^3, R = 9 took 20 us; this takes 12 us.
//
//   rows of P -> A (LDS, with the x halo) -> x -> B -> y, fits -> A (g1, g2)
//   -> x -> B -> y -> Q
//
// Row stride of A as in the march; B holds 64 columns per wave and no halo.
template <int R, class ST>
__global__ __launch_bounds__(kXysThreads, 4) void xys_kernel(Batch bt, Taps t, Coeffs c)
{
    constexpr int NK = TapOps<R>::N, NQ = (NK + 3) / 4, NWAVES = kXysThreads / 64;
    extern __shared__ __attribute__((aligned(16))) float lds[];

    Where wh;
    if (!locate(bt, wh)) return;
    const TileDesc &d = bt.tiles[wh.t];
    if (glb(d.flags)[0]) return;
    const Grid3 g = d.g;
    const XyfStrips sg = xyf_strips(g.nx, R, 2);
    const int strip = wh.lb % sg.n, rest = wh.lb / sg.n;
    const int yc = rest % d.sp.f, z = rest / d.sp.f;
    const int len = (g.ny + d.sp.f - 1) / d.sp.f;
    const int y0 = yc * len, y1 = min(y0 + len, g.ny);
    const XysRows n = xys_rows(len, R);
    const int c0 = min(strip * sg.step, g.nx - sg.width), nw = (sg.width + 63) / 64;
    const int S = xys_stride(nw, R), BS = 64 * nw;
    const int FA = 4 * n.a * S, FB = 4 * n.a * BS;          // a field of A, of B
    float *const A = lds, *const B = lds + 2 * FA;

    const int lane = threadIdx.x & 63;
    const int wave = (int)__builtin_amdgcn_readfirstlane(threadIdx.x / 64);
    const int64_t zb = (int64_t)z * g.sxy;
    constexpr uint32_t PB = sizeof(Vec2<ST>), SB = sizeof(ST);
    const uint32_t plane = (uint32_t)g.sxy, nx = (uint32_t)g.nx;
    auto at_row = [&](int r, int rows) { return (uint32_t)min(max(r, -1), rows) * nx; };
    const rsrc_t rin = rsrc_n(static_cast<const char *>(d.P) + zb * (int64_t)PB, plane * PB);
    const rsrc_t rki = rsrc_n(static_cast<const ST *>(d.KI) + zb, plane * SB);
    const rsrc_t rout = rsrc_n(static_cast<char *>(d.Q) + (zb + (int64_t)y0 * g.nx) * (int64_t)PB,
                               (uint32_t)(y1 - y0) * nx * PB);
    TapOps<R> tp;
    tp.load(t, lane);

    // rows y0 - 2R .. of P into A, a row per wave and turn, columns
    // c0 - R + (0 .. S - 1) (past the halo: zeros)
    constexpr int NC = 3, NR = 4;
    uint32_t xb[NC], xbad[NC];
#pragma unroll
    for (int h = 0; h < NC; ++h) {
        const int j = lane + 64 * h, x = c0 - R + j;
        xb[h] = (uint32_t)x;
        xbad[h] = x >= 0 && x < g.nx && j < BS + 2 * R ? 0u : kOut;
    }
    for (int r0 = wave; r0 < 4 * n.a; r0 += NR * NWAVES) {
        Vec2<ST> v[NR][NC];
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const uint32_t row = at_row(y0 - 2 * R + r0 + i * NWAVES, g.ny);
#pragma unroll
            for (int h = 0; h < NC; ++h)
                v[i][h] = bld_at<Vec2<ST>>(rin, ((xb[h] + row) * PB) | xbad[h]);
        }
#pragma unroll
        for (int i = 0; i < NR; ++i) {
            const int r = r0 + i * NWAVES;
#pragma unroll
            for (int h = 0; h < NC; ++h) {
                const int j = lane + 64 * h;
                if (r < 4 * n.a && j < S) {
                    A[r * S + j] = to_f(v[i][h].x);
                    A[FA + r * S + j] = to_f(v[i][h].y);
                }
            }
        }
    }
    __syncthreads();

    // x convolution of the groups of four rows of A into B
    auto xpass = [&](int groups) {
        for (int k = wave; k < groups * nw; k += NWAVES) {
            const int gr = k / nw, w = k % nw;
            const float *const src = A + (4 * gr + (lane & 3)) * S + 64 * w + (lane & ~3);
            f4 a{}, b{};
            static_for<NQ>([&](auto qc) {
                constexpr int q = qc;
                f4 va = *reinterpret_cast<const f4 *>(src + 4 * q);
                f4 vb = *reinterpret_cast<const f4 *>(src + FA + 4 * q);
                __asm__ volatile("" : "+v"(va), "+v"(vb));   // (kept as 16-byte reads)
                static_for<4>([&](auto kc) {
                    constexpr int e = kc;
                    if constexpr (4 * q + e < NK) {
                        a = __builtin_amdgcn_mfma_f32_4x4x1f32(va[e], tp.x[q], a, 0, 0, 4 + e);
                        b = __builtin_amdgcn_mfma_f32_4x4x1f32(vb[e], tp.x[q], b, 0, 0, 4 + e);
                    }
                });
            });
            if (__builtin_expect(nan_lanes(a, b) != 0, 0))
                conv_exact<R>(A + 4 * gr * S + 64 * w + lane, S, 1, FA, t, a, b);
            float *const dst = B + 4 * gr * BS + 64 * w + lane;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                dst[i * BS] = a[i];
                dst[FB + i * BS] = b[i];
            }
        }
    };
    // y convolution: four rows from row 4 gr of B on, columns 64 w ..
    auto yconv = [&](int gr, int w, f4 &a, f4 &b) {
        const float *src = B + 4 * gr * BS + 64 * w + lane;
        a = f4{};
        b = f4{};
        static_for<NK>([&](auto kc) {
            constexpr int k = kc, p = 2 * R + 3 - k;
            a = __builtin_amdgcn_mfma_f32_4x4x1f32(tp.y[p / 16], src[k * BS], a, 4, p % 16, 0);
            b = __builtin_amdgcn_mfma_f32_4x4x1f32(tp.y[p / 16], src[FB + k * BS], b, 4, p % 16, 0);
        });
        if (__builtin_expect(nan_lanes(a, b) != 0, 0)) conv_exact<R>(src, BS, BS, FB, t, a, b);
    };

    xpass(n.a);
    __syncthreads();
    const float *const cyp = d.cy;
    const float cz = glb(d.cz)[z];
    // the columns around the strip hold no g: zero padding at the volume's
    // edges, not used elsewhere
    for (int k = threadIdx.x; k < 4 * n.b * 2 * R; k += kXysThreads) {
        const int r = k / (2 * R), j = k % (2 * R), at = r * S + (j < R ? j : BS + j);
        A[at] = A[FA + at] = 0.f;
    }
    for (int k = wave; k < n.b * nw; k += NWAVES) {
        const int gr = k / nw, w = k % nw;
        const int x = c0 + 64 * w + lane, rb = y0 - R + 4 * gr;
        const uint32_t e0 = (uint32_t)x;
        ST ki[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) ki[i] = bld_at<ST>(rki, (e0 + at_row(rb + i, g.ny)) * SB);
        const float cxz = glb(d.cx)[min(x, g.nx - 1)] * cz;
        f4 a1, b1;
        yconv(gr, w, a1, b1);
        const int xkeep = x < g.nx ? -1 : 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // region fits (Sec. 3 local_intensity), as in the march
            const float K1 = cxz * uniform_ld(cyp, min(max(rb + i, 0), g.ny - 1));
            const float A2 = to_f(ki[i]) - a1[i];
            const float B2 = K1 - b1[i];
            const float f1 = a1[i] * rcp(b1[i]);
            const float f2 = A2 * rcp(B2);
            float g1 = c.l1 * f1 - c.l2 * f2, g2 = c.l1 * f1 * f1 - c.l2 * f2 * f2;
            if constexpr (!std::is_same<ST, float>::value) {
                pin(g1);
                pin(g2);
                g1 = to_f(from_f<ST>(g1));
                g2 = to_f(from_f<ST>(g2));
            }
            int rk = ~(((rb + i) | (g.ny - 1 - rb - i)) >> 31);
            __asm__ volatile("" : "+s"(rk));
            const int keep = xkeep & rk, at = (4 * gr + i) * S + R + 64 * w + lane;
            A[at] = __int_as_float(__float_as_int(g1) & keep);
            A[FA + at] = __int_as_float(__float_as_int(g2) & keep);
        }
    }
    __syncthreads();
    xpass(n.b);
    __syncthreads();
    const int o0 = strip == 0 ? 0 : strip * sg.step + R;
    const int o1 = strip == sg.n - 1 ? g.nx : c0 + sg.width - R;
    for (int k = wave; k < n.c * nw; k += NWAVES) {
        const int gr = k / nw, w = k % nw;
        const int x = c0 + 64 * w + lane;
        const uint32_t obad = x >= o0 && x < o1 ? 0u : kOut;
        f4 a2, b2;
        yconv(gr, w, a2, b2);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            Vec2<ST> v;
            v.x = from_f<ST>(a2[i]);
            v.y = from_f<ST>(b2[i]);
            bst_at<Vec2<ST>>(rout, (((uint32_t)x + at_row(4 * gr + i, y1 - y0)) * PB) | obad, v);
        }
    }
}

}  // namespace

}  // namespace rsf

// How each pass cuts a tile into workgroups (host code): row chunks of the xy
// passes, z chunks of the z passes and of the update pass.
#include <algorithm>
#include <cmath>
#include <utility>
#include <vector>

#include "rsf_internal.hpp"

namespace rsf {

// The fewest chunks giving at least `want_blocks` over `cols` columns, each
// chunk at least `least` long; re-derived so every chunk is non-empty.
static int chunks(int64_t n, int64_t cols, int64_t want_blocks, int64_t least)
{
    int64_t want = (want_blocks + cols - 1) / cols;
    const int64_t most = (n + least - 1) / least;
    if (want > most) want = most;
    if (want < 1) want = 1;
    const int64_t len = (n + want - 1) / want;
    return (int)((n + len - 1) / len);
}

Split make_split(const Grid3 &g, int64_t xy_waves, int64_t z_target, int64_t u_target, int R,
                 int halo)
{
    Split s;
    const int64_t strips = nbx64(g.nx);
    s.xy = chunks(g.ny, strips * g.nz, xy_waves, 8);
    s.z = chunks(g.nz, z_cols(g), z_target, 8);
    s.u = chunks(g.nz, (int64_t)((g.nx + kUx - 1) / kUx) * ((g.ny + kUy - 1) / kUy), u_target, 8);
    // an xy-pass workgroup holds several waves and pays a halo of up to 4 R rows
    const int nw = xyf_batch_waves(&g, &s, 1, R, halo);
    s.f = chunks(g.ny, (int64_t)xyf_strips(g.nx, halo, nw).n * g.nz, xy_waves / 16, 32);
    return s;
}

// A tile holding fraction `share` of a batch's voxels gets that fraction of
// the batch's workgroup targets (by default xy ~16K waves, rows in chunks of
// at most 128; z ~2K workgroups; update ~1K workgroups).  Fewer chunks per tile means fewer
// halo slices re-read, so small tiles in a big batch run unchunked.
Split default_split(const Grid3 &g, double share, const Targets &tg, int R, int halo)
{
    const auto part = [&](int64_t n) {
        return (int64_t)std::max(1.0, std::ceil((double)n * share));
    };
    Split s = make_split(g, part(tg.xy), part(tg.z), part(tg.u), R, halo);
    const int base = (g.ny + 127) / 128;
    if (s.xy < base) {
        const int64_t len = (g.ny + base - 1) / base;
        s.xy = (int)((g.ny + len - 1) / len);
    }
    return s;
}

// z chunks c in 1..ceil(nz/8) for a pass whose workgroups each march a chunk
// plus `halo` extra slices: the cost of c is ceil(groups / resident) x (chunk
// length + halo), the launch's rounds of workgroups.  Among the c that keep at
// least `min_fill` of the resident slots busy, take the fewest chunks whose
// cost is within 3 % of the least (fewer halo re-reads); if none keeps the
// slots that busy, `few` picks the chunks of a volume too small for that.
template <class Few>
static int capacity_chunks(int64_t nz, int64_t cols, int64_t resident, double min_fill,
                           int64_t halo, Few &&few)
{
    const int64_t most = (nz + 7) / 8;
    std::vector<std::pair<int64_t, double>> ok;
    double least = -1.0;
    for (int64_t c = 1; c <= most; ++c) {
        const int64_t len = (nz + c - 1) / c;
        if ((nz + len - 1) / len != c) continue;   // not c non-empty chunks
        const int64_t groups = cols * c;
        if ((double)groups < min_fill * (double)resident) continue;
        const double cost = (double)((groups + resident - 1) / resident) * (double)(len + halo);
        ok.push_back({c, cost});
        if (least < 0.0 || cost < least) least = cost;
    }
    for (const auto &cc : ok)
        if (cc.second <= 1.03 * least) return (int)cc.first;
    if (nz <= 8) return 1;
    const int64_t len = (nz + most - 1) / most;
    return few((nz + len - 1) / len);
}

// The update pass of a small volume is bound by the latency of one
// workgroup's march, so its chunks go down to 2 slices: the least (length +
// halo), times 1.3 where a CU holds two workgroups (45 x 71 x 67: 216
// workgroups of 4 slices 13.0 us, 270 of 3 slices 15.3, 414 of 2 slices 14.3).
// 64^3, R = 9: 64 workgroups of 8 slices 16.2 us, 256 of 2 slices 11.7.
static int few_u(int64_t nz, int64_t cols, int64_t halo)
{
    int best = 1;
    double least = -1.0;
    for (int64_t c = 1; c <= (nz + 1) / 2; ++c) {
        const int64_t len = (nz + c - 1) / c;
        if ((nz + len - 1) / len != c) continue;
        if (c > 1 && cols * c > kResidentU) break;
        const double cost = (double)(len + halo) * (cols * c > kCus ? 1.3 : 1.0);
        if (least < 0.0 || cost < least) {
            least = cost;
            best = (int)c;
        }
    }
    return best;
}

// A small volume's z pass: chunks of 8 slices, or down to 2 while every
// workgroup has a CU of its own (64^3: 128 workgroups of 8 slices 10.3 us, 256
// of 4 slices 9.6; 96^3: 432 of 8 slices are 0.9 us faster than 864 of 4).
static int few_z(int64_t nz, int64_t cols, int64_t most)
{
    int best = (int)most;
    for (int64_t c = most + 1; c <= (nz + 1) / 2 && cols * c <= kCus; ++c) {
        const int64_t len = (nz + c - 1) / c;
        if ((nz + len - 1) / len == c) best = (int)c;
    }
    return best;
}

int xyf_resident(int R, bool two, int nw, int waves)
{
    const int simd = two ? xyf_simd_waves(R, true) : (R <= 9 ? 3 : 2);
    return std::max(1, std::min(4 * simd / waves, nw == 8 ? 2 : 4));
}

double xyf_load(int waves, int64_t k)
{
    // (more than four waves load the busiest SIMD as a multiple of four)
    const int on_simds = waves > 4 ? (waves + 3) / 4 * 4 : waves;
    return std::max(1.5, 0.25 * (double)(k * on_simds));
}

// Rows of a chunk of `len` rows, one of c: its own, `reach` rows above and below
// where it has neighbours, and two groups of latency.
static int xyf_rows(int len, int c, int reach)
{
    return len + (c == 1 ? 0 : c == 2 ? reach : 2 * reach) + 8;
}

// f(c, length) for the chunk counts c <= most of n rows that give c non-empty
// chunks of ceil(n / c): about 2 sqrt(n) of them.
template <class F>
static void each_chunking(int n, int most, F &&f)
{
    for (int c = 1; c <= most;) {
        const int len = (n + c - 1) / c;
        f(c, len);
        if (len == 1) break;
        c = (n + len - 2) / (len - 1);
    }
}

// Where strips times slices fill the CUs by themselves, the time of a row lies
// between the SIMDs' mean load and the busiest one's whole waves: 257 x 301 x 316,
// R = 6, FP16, has two workgroups of three waves on most CUs and takes 201 us uncut,
// 157 in three chunks; 300 x 300 x 100, R = 6, FP16, 83 in two and 63 in three.  Of
// 212 volumes of 1 to 60 million voxels that 0.6 cuts otherwise than the mean does,
// the call takes 0.946 of the time on average, four 2 to 3.4 % more (184 x 639 x 298,
// R = 3, FP32, one stage: 166 -> 180 us); 1.0 also loses 192 x 320 x 352, R = 3, by
// 4.5 %, and 0.5 leaves 257 x 301 x 316 uncut.  On smaller volumes a finer cut hides
// latency, and the mean serves better (128^3, R = 6, FP16: 6 chunks 8 % faster than
// the 4 of the busiest one).
XyfPick xyf_pick(const Grid3 &g, int R, int halo)
{
    XyfPick best{4, 1};
    double least = -1.0;
    const bool two = halo > 0;
    const int most = (g.ny + 3) / 4;
    const auto better = [&](double cost, int nw, int c) {
        if (least >= 0.0 && cost >= 0.97 * least) return;
        least = cost;
        best = XyfPick{nw, c};
    };
    for (int nw = 4; nw <= (two ? 8 : 4); nw += 4) {
        const XyfStrips st = xyf_strips(g.nx, halo, nw);
        const int waves = (st.width + 63) / 64;
        const int64_t slots = xyf_resident(R, two, nw, waves);
        each_chunking(g.ny, most, [&](int c, int len) {
            const int64_t per_cu = ((int64_t)st.n * g.nz * c + kCus - 1) / kCus;
            const int64_t at_once = std::min(per_cu, slots);
            double load = xyf_load(waves, at_once);
            if ((int64_t)st.n * g.nz >= kCus) load += 0.6 * (std::ceil(load) - load);
            better((double)((per_cu + at_once - 1) / at_once) * xyf_rows(len, c, R + halo) * load,
                   nw, c);
        });
    }
    if (!two) return best;
    const XyfStrips st = xyf_strips(g.nx, halo, 2);
    const int waves = (st.width + 63) / 64;
    each_chunking(g.ny, most, [&](int c, int len) {
        const int64_t lds = xys_lds(len, R, waves);
        if (lds > kXysLds) return;
        const XysRows n = xys_rows(len, R);
        const int64_t per_cu = ((int64_t)st.n * g.nz * c + kCus - 1) / kCus;
        if (per_cu > std::min<int64_t>(2, kXysLds / lds)) return;   // one round
        const double work =
            (n.a + 2 * n.b + n.c) * waves * 2.0 * (2 * R + 4) * 8.0 / 4.0 * 3.6 / 2300.0;
        better(3.5 * (6.0 + per_cu * work), 2, c);
    });
    return best;
}

int xyf_batch_waves(const Grid3 *g, const Split *sp, int n, int R, int halo)
{
    if (halo == 0) return 4;
    double cost[2] = {0.0, 0.0};
    for (int k = 0; k < 2; ++k)
        for (int t = 0; t < n; ++t) {
            const int nw = 4 + 4 * k;
            const XyfStrips st = xyf_strips(g[t].nx, halo, nw);
            const int waves = (st.width + 63) / 64, slots = xyf_resident(R, true, nw, waves);
            const int len = (g[t].ny + sp[t].f - 1) / sp[t].f;
            cost[k] += (double)st.n * g[t].nz * sp[t].f * xyf_rows(len, sp[t].f, R + halo) *
                       xyf_load(waves, slots) / slots;
        }
    return cost[1] < cost[0] ? 8 : 4;
}

Split capacity_split(const Grid3 &g, int R, int halo)
{
    Split s = default_split(g, 1.0, kDefaultTargets);
    // a z-pass chunk primes its ring with 2R slices; an update chunk reads R
    // extra slices of the pair ring on average and 4 of phi
    s.f = xyf_pick(g, R, halo).f;
    const int64_t zc = z_cols(g);
    const int64_t uc = (int64_t)((g.nx + kUx - 1) / kUx) * ((g.ny + kUy - 1) / kUy);
    s.z = capacity_chunks(g.nz, zc, kResidentZ, 0.5, 2 * R,
                          [&](int64_t most) { return few_z(g.nz, zc, most); });
    s.u = capacity_chunks(g.nz, uc, kResidentU, 0.75, R + 2,
                          [&](int64_t) { return few_u(g.nz, uc, R + 2); });
    return s;
}

static bool chunks_ok(int n, int c)
{
    if (c < 1 || c > n) return false;
    const int len = (n + c - 1) / c;
    return (c - 1) * len < n;
}

bool split_valid(const Grid3 &g, const Split &s)
{
    return chunks_ok(g.ny, s.xy) && chunks_ok(g.nz, s.z) && chunks_ok(g.nz, s.u) &&
           chunks_ok(g.ny, s.f) && u_blocks(g, s) <= u_blocks_max(g);
}

}  // namespace rsf

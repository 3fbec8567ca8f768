// Host check of how the iteration's xy pass is cut: strips, row chunks, the
// small-volume form and the batched launch.  Host code only.
//   xyf_check              run the checks
//   xyf_check R force nz ny nx [nz ny nx ...]   the pass's form for a volume or
//                          a batch: waves (2: the small form), row chunks of each
#include <algorithm>
#include <chrono>
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "rsf_host.hpp"

using namespace rsf;
using namespace rsf::host;

#define CHECK(c)                                                              \
    do {                                                                      \
        if (!(c)) {                                                           \
            std::fprintf(stderr, "check failed line %d: %s\n", __LINE__, #c); \
            return 1;                                                         \
        }                                                                     \
    } while (0)

static Grid3 grid(int nz, int ny, int nx) { return Grid3{nx, ny, nz, (int64_t)nx * ny}; }

// strips of nx columns: every column stored once, with `halo` computed columns
// on either side of each inner edge
static int strips(int nx, int halo, int nw)
{
    const XyfStrips s = xyf_strips(nx, halo, nw);
    CHECK(s.n >= 1 && s.width <= 64 * nw && s.width <= nx);
    CHECK(s.n == 1 || nw < 4 || s.width >= 128);
    int next = 0;
    for (int k = 0; k < s.n; ++k) {
        const int c0 = std::min(k * s.step, nx - s.width);
        const int o0 = k == 0 ? 0 : k * s.step + halo;
        const int o1 = k == s.n - 1 ? nx : c0 + s.width - halo;
        CHECK(c0 >= 0 && o0 == next && o1 > o0);
        CHECK(k == 0 || o0 - halo >= c0);
        CHECK(k == s.n - 1 || o1 + halo <= c0 + s.width);
        next = o1;
    }
    CHECK(next == nx);
    return 0;
}

// the launch of a batch: every workgroup in exactly one XCD range
static int launch(const std::vector<Grid3> &g, const std::vector<Split> &sp, int R, int halo, int nw)
{
    std::vector<int> start(1, 0);
    for (size_t t = 0; t < g.size(); ++t)
        start.push_back(start.back() + (int)xyf_blocks(g[t], sp[t], halo, nw));
    Batch b{nullptr, nullptr, (int)g.size(), {}};
    const int64_t blocks = balance_xcds(b, PASS_F, g, sp, R, halo, nw);
    CHECK(b.xcd[0] == 0 && b.xcd[kXcds] == start.back() && blocks % kXcds == 0);
    double most = 0.0, sum = 0.0, one = 0.0;
    int64_t longest = 0;
    std::vector<double> cost(kXcds, 0.0);
    for (int x = 0; x < kXcds; ++x) {
        CHECK(b.xcd[x] <= b.xcd[x + 1]);
        longest = std::max<int64_t>(longest, b.xcd[x + 1] - b.xcd[x]);
    }
    CHECK(blocks == kXcds * longest);
    for (size_t t = 0; t < g.size(); ++t) {
        const int n = xyf_strips(g[t].nx, halo, nw).n;
        one = std::max(one, (double)g[t].ny + 2 * (R + halo));
        for (int gb = start[t]; gb < start[t + 1]; ++gb) {
            const int x = (int)(std::upper_bound(b.xcd, b.xcd + kXcds, gb) - b.xcd) - 1;
            cost[x] += (double)span_cost(g[t].ny, sp[t].f, (gb - start[t]) / n % sp[t].f, R + halo);
        }
    }
    for (double c : cost) {
        most = std::max(most, c);
        sum += c;
    }
    // balanced in cost, or, where all workgroups of a volume run at once, in number
    if (g.size() == 1 && start.back() <= 4 * kCus)
        CHECK(longest <= (start.back() + kCus - 1) / kCus * (kCus / kXcds));
    else
        CHECK(most <= sum / kXcds + one + 1e-9);
    return 0;
}

static int run()
{
    for (int halo : {0, 1, 4, 9, 12, 16})
        for (int nw : {2, 4, 8})
            for (int nx = 3; nx < 3000; nx += nx < 700 ? 1 : 7)
                if (strips(nx, halo, nw)) return 1;

    std::mt19937 rng(11);
    for (int trial = 0; trial < 600; ++trial) {
        const int R = 1 + rng() % 16, big = trial % 3 == 0 ? 700 : 130;
        const int force = rng() % 2 ? RSF_FORCE_PAPER : RSF_FORCE_RSF, halo = xyf_halo(force, R);
        const Grid3 q = grid(3 + rng() % big, 3 + rng() % big, 3 + rng() % big);
        // a single volume's own split
        const Split s = capacity_split(q, R, halo);
        CHECK(split_valid(q, s) && u_blocks(q, s) <= u_blocks_max(q));
        const XyfShape f = xyf_shape({q}, {s}, force, R, false);
        CHECK(f.nw == 4 || (force == RSF_FORCE_RSF && (f.nw == 2 || f.nw == 8)));
        CHECK(f.nw == 2 ? f.lds > 0 && f.lds <= kXysLds && f.threads == kXysThreads
                        : f.threads <= 64 * f.nw && f.threads >= std::min(xyf_strips(q.nx, halo, f.nw).width, 64));
        // the small form's workgroups run in one round
        if (f.nw == 2)
            CHECK(xyf_blocks(q, s, halo, 2) <= kCus * std::min<int64_t>(2, kXysLds / f.lds));
        if (launch({q}, {s}, R, halo, f.nw)) return 1;
        // a batch
        std::vector<Grid3> g;
        std::vector<Split> sp;
        for (unsigned t = 0, n = 2 + rng() % 12; t < n; ++t) {
            g.push_back(grid(3 + rng() % 60, 3 + rng() % 200, 3 + rng() % big));
            sp.push_back(trial % 2 ? default_split(g[t], 1.0 / n) : make_split(g[t], 1 + rng() % 30000, 100, 100));
            CHECK(split_valid(g[t], sp[t]));
        }
        const XyfShape b = xyf_shape(g, sp, force, R, false);
        CHECK(b.nw == 4 || (b.nw == 8 && force == RSF_FORCE_RSF));
        for (const Grid3 &t : g) CHECK(b.threads >= xyf_threads(t.nx, halo, b.nw));
        CHECK(b.threads <= 64 * b.nw);
        if (launch(g, sp, R, halo, b.nw)) return 1;
    }

    // the plan of a very long volume takes no time that counts beside a launch
    const auto t0 = std::chrono::steady_clock::now();
    for (int force : {RSF_FORCE_RSF, RSF_FORCE_PAPER}) {
        const Grid3 q = grid(3, 80000000, 3);
        const Split s = capacity_split(q, 9, xyf_halo(force, 9));
        xyf_shape({q}, {s}, force, 9, false);
    }
    const double ms = std::chrono::duration<double, std::milli>(std::chrono::steady_clock::now() - t0).count();
    CHECK(ms < 50.0);
    std::printf("xyf ok %.3f ms\n", ms);
    return 0;
}

int main(int argc, char **argv)
{
    if (argc < 6) return run();
    const int R = std::atoi(argv[1]), force = std::atoi(argv[2]), halo = xyf_halo(force, R);
    std::vector<Grid3> g;
    std::vector<Split> sp;
    double voxels = 0.0;
    for (int k = 3; k + 2 < argc; k += 3) {
        g.push_back(grid(std::atoi(argv[k]), std::atoi(argv[k + 1]), std::atoi(argv[k + 2])));
        voxels += (double)g.back().sxy * g.back().nz;
    }
    for (const Grid3 &q : g)
        sp.push_back(g.size() == 1 ? capacity_split(q, R, halo)
                                   : default_split(q, (double)q.sxy * q.nz / voxels, kDefaultTargets, R, halo));
    std::printf("%d", xyf_shape(g, sp, force, R, false).nw);
    for (const Split &s : sp) std::printf(" %d", s.f);
    std::printf("\n");
    return 0;
}

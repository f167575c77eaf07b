// Host-side planning of resident lanes: how a grid is cut into the rectangles of a
// group's workgroups, and which groups a launch gets. No HIP call and no device
// code, so that a host program can include it.
#pragma once

#include <math.h>

#include <algorithm>
#include <vector>

#include "../../include/pt.h"
#include "pt_internal.h"

namespace pt {

namespace {

// How a lane is cut up on its group: nodes per streaming tile, or the rectangle,
// polynomial degree and window rows per thread of a resident lane.
struct Shape {
    int tile, tw, th, deg, nr;
};

// One kind of lane and how its lanes are queued on groups.
struct LanePlan {
    int kind;
    int count;        // lanes
    int slice0;       // first slice in queue order
    int dir;          // +1 ascending, -1 descending slices
    double weight;    // work per lane (relative)
    bool latency;     // sweep-like: fixed group size
    int queues = 0;   // groups (0: one lane per group)
    int fixed_nwg = 0;  // workgroups per group if > 0 (same fine shape in both passes)
    int lead_kind = -1, lead_slice = 0;  // a lane the group runs first (one group only)
};

// ---------------------------------------------------------------------------
// Shapes of resident lanes
// ---------------------------------------------------------------------------

// Window rows per thread the kernel is built for.
constexpr int kResRowChoices[] = {2, 4, 6};
static_assert(kResRowChoices[2] == kResRows, "the largest variant");
constexpr int kResMaxColumns = 480;  // columns of a window, at most
static_assert(kResMaxColumns <= kThreads, "a thread for each");

// A workgroup's window: the rectangle with its rings where the grid is cut, and the
// rows of it that the threads hold.
struct Window {
    int wc, wr, rows;
    Window(const Shape &s, int W, int HN)
        : wc(s.tw + (s.tw < W ? 2 * (s.deg + 1) : 0)),
          wr(s.th + (s.th < HN ? 2 * (s.deg + 1) : 0)),
          rows(wc > kResMaxColumns ? 0 : std::min(kThreads / wc, (wr + s.nr - 1) / s.nr) * s.nr) {}
};

// LDS bytes of a resident lane: two operand windows with a rim and two values
// per node slot (the p and x of the solve).
size_t res_lds_bytes(const Shape &s, int W, int HN) {
    const Window w(s, W, HN);
    return sizeof(double) *
           (2 * (size_t)(w.wc + 2) * (w.rows + 2) + 2 * (size_t)s.nr * kThreads);
}

// Whether a workgroup holds its window of a shape: the threads its rows, the LDS its
// operands, and kRim cells per thread the cells around it (those above and below first;
// where the grid is not cut into columns the ones beside it lie outside).
bool res_window_fits(const Shape &s, int W, int HN, size_t lds_cap) {
    const Window w(s, W, HN);
    return w.wc <= kResMaxColumns && w.wr <= w.rows &&
           2 * (w.wc + 2) + (s.tw < W ? 2 * w.rows : 0) <= kRim * kThreads &&
           res_lds_bytes(s, W, HN) <= lds_cap;
}

// The rectangles for a grid of W x HN nodes on at most max_wg workgroups: the
// fewest window rows per thread, then the smallest window. False if the grid
// does not fit. `wgs`: the workgroups used.
bool res_shape(int W, int HN, int max_wg, int deg, int rows_max, size_t lds_cap, Shape &best,
               int &wgs) {
    for (int nr : kResRowChoices) {
        if (nr > rows_max) break;
        double best_cost = INFINITY;
        for (int TX = 1; TX <= std::min(max_wg, W); ++TX) {
            const int tw = (W + TX - 1) / TX;
            if ((W + tw - 1) / tw != TX) continue;  // the same width with fewer columns
            const int th = (HN + std::min(max_wg / TX, HN) - 1) / std::min(max_wg / TX, HN);
            const int TY = (HN + th - 1) / th;
            const Shape s{0, tw, th, deg, nr};
            if (!res_window_fits(s, W, HN, lds_cap)) continue;
            const Window w(s, W, HN);
            const double cost = (double)w.wc * w.wr;
            if (cost < best_cost) {
                best_cost = cost;
                best = s;
                wgs = TX * TY;
            }
        }
        if (best_cost < INFINITY) return true;
    }
    return false;
}

// The shape of lanes of degree d0 on at most max_wg workgroups: that degree, or the
// largest below it whose window fits; then, among the degrees from one less up to
// kResMaxDeg and the rows per thread, the least time per application of the operator.
// A round of n = degree + 1 applications takes about 3 + 0.5 rows + n (0.1 + 0.12 rows)
// us (measured: 5.4 at 2 rows and n = 4, 9.3 at 6 rows), and the polynomial's part in
// the convergence falls off by some 3% per degree. More applications per round pay
// until the window's rings need more rows (101^2 nodes, sequential: 105 ms at degree 3,
// 71 at 8; sweep of 30 slices 13.2 ms at 4, 11.5 at 6; solves ended at cg_rtol itself).
// `more` false: that degree only. Coarse-mesh solves are well conditioned, with 6 to 24
// rounds at degree 4, and the search gives their passes 0 to 5% warm, up to 12% cold
// (256^2 with 8 slices: 9.15 against 9.02 ms, 12.3 against 11.0); but it leaves them
// so few rounds, 4 on 17^2 nodes as the fine solves take, that an iteration cap hardly
// tells them apart any more.
bool res_fit(int W, int HN, int max_wg, int d0, int rows_max, size_t cap, Shape &s, int &n,
             bool more = true) {
    bool ok = false;
    for (int deg = d0; deg >= 0 && !ok; --deg)
        ok = res_shape(W, HN, max_wg, deg, rows_max, cap, s, n);
    if (!ok || !more || d0 < 2 || s.deg < d0) return ok;
    auto cost = [](int nr, int apps) {
        return (3.0 + 0.5 * nr + apps * (0.1 + 0.12 * nr)) / apps * (1.0 + 0.03 * apps);
    };
    for (int deg = d0 - 1; deg <= kResMaxDeg; ++deg) {
        Shape t;
        int m;
        if (!res_shape(W, HN, max_wg, deg, rows_max, cap, t, m)) break;
        // (one degree less only for the fastest rounds: at 512^2, 4 rows and degree 2
        // instead of 6 and 3 took 314 ms against 291)
        if (deg < d0 && t.nr > kResRowChoices[0]) continue;
        if (cost(t.nr, deg + 1) < cost(s.nr, s.deg + 1)) {
            s = t;
            n = m;
        }
    }
    return ok;
}

// The fewest workgroups that hold the grid (0: none do).
int res_min_wgs(int W, int HN, int deg, int rows_max, size_t lds_cap) {
    int best = 0;
    for (int nr : kResRowChoices) {
        if (nr > rows_max) break;
        for (int TX = 1; TX <= W && (best == 0 || TX < best); ++TX) {
            const int tw = (W + TX - 1) / TX;
            const int wc = tw + (TX > 1 ? 2 * (deg + 1) : 0);
            if (wc > kResMaxColumns) continue;
            const int wr = kThreads / wc * nr;
            const int th = HN <= wr ? HN : wr - 2 * (deg + 1);
            if (th < 1 || !res_window_fits(Shape{0, tw, th, deg, nr}, W, HN, lds_cap)) continue;
            const int n = TX * ((HN + th - 1) / th);
            if (best == 0 || n < best) best = n;
        }
    }
    return best;
}

// Plans a launch whose lanes are all resident: group counts and sizes and the
// lanes' shapes. False if the lanes do not fit the grid. one_queue (of a plan): the sweeps
// have no groups of their own, all lanes go through the shared queue.
bool plan_resident(const Consts &C, const std::vector<LanePlan> &plans, const pt_tuning &T,
                   int grid, int lds_cap_d, int sweep_wgs, const CoarseMesh *cm,
                   std::vector<int> &ngroups, std::vector<int> &nwg, std::vector<Shape> &shape,
                   std::vector<Shape> &lead_shape, size_t &lds, bool &one_queue) {
    const int HN = C.ny + 1;
    const size_t cap = (size_t)lds_cap_d * sizeof(double);
    const int rows_max = std::max(2, T.resident_npt_max);
    const int deg_f = 3, deg_c = 4;
    auto deg_of = [&](int kind) {
        if (kind == F_PRI || kind == F_ADJ) return deg_f;
        if (is_cm_kind(kind)) return deg_c;
        return C.coarse_iters > 0 ? 0 : deg_c;
    };
    auto rows_of = [&](int kind) { return is_cm_kind(kind) ? C.ny / 2 + 1 : HN; };
    auto width_of = [&](int kind) { return is_cm_kind(kind) ? C.nx / 2 + 1 : C.W; };
    auto fit = [&](int kind, int max_wg, Shape &s, int &n) {
        return res_fit(width_of(kind), rows_of(kind), max_wg, deg_of(kind), rows_max, cap, s, n,
                       !is_cm_kind(kind));
    };
    auto min_wgs = [&](int kind, int deg) {
        return res_min_wgs(width_of(kind), rows_of(kind), deg, rows_max, cap);
    };
    auto lds_of = [&](int kind, const Shape &s) {
        return res_lds_bytes(s, width_of(kind), rows_of(kind));
    };
    lds = 0;
    one_queue = false;
    // the least workgroups that hold the grid for every kind of batched lane
    int g_min = 0, nb = 0, lanes = 0, lat = 0, fk = -1;
    bool sweeps = false;
    for (size_t k = 0; k < plans.size(); ++k) {
        const LanePlan &p = plans[k];
        ngroups[k] = 0;
        nwg[k] = 1;
        if (p.latency) sweeps |= p.count > 0;
        if (p.latency || p.count == 0) continue;
        ++nb;
        lanes += p.count;
        if (p.kind == F_PRI || p.kind == F_ADJ) fk = p.kind;
        const int g = min_wgs(p.kind, deg_of(p.kind));
        if (g == 0) return false;
        g_min = std::max(g_min, g);
    }
    // sequential sweeps on groups of their own
    bool own = true;
    for (size_t k = 0; own && k < plans.size(); ++k) {
        const LanePlan &p = plans[k];
        if (!p.latency || p.count == 0) continue;
        const int want = p.fixed_nwg > 0 ? p.fixed_nwg : std::min(sweep_wgs, grid / 4);
        int n = want;
        own = fit(p.kind, std::max(want, min_wgs(p.kind, deg_of(p.kind))), shape[k], n);
        if (own && p.lead_kind >= 0) {
            int m = 0;
            own = fit(p.lead_kind, std::max(n, min_wgs(p.lead_kind, deg_of(p.lead_kind))),
                      lead_shape[k], m);
            n = std::max(n, m);
            lds = std::max(lds, lds_of(p.lead_kind, lead_shape[k]));
        }
        lds = std::max(lds, lds_of(p.kind, shape[k]));
        ngroups[k] = p.count;
        nwg[k] = n;
        lat += n * p.count;
    }
    const bool share = T.shared_queue != 0;
    // the rest of the grid for the batched lanes, on groups of one size
    int avail = g_min > 0 ? (grid - lat) / g_min : nb;
    if (!own || grid < lat) avail = 0;
    // A grid so large that beside the sweep's group only one other is left: the
    // sweep's workgroups, which mostly wait for that group's lanes, are better used
    // for such lanes too, the sweep following as the queue's last lane. With 32
    // slices of 16 steps the fine and batched coarse lanes are about four times the
    // sweep's work, so two groups and then the sweep take 4/2 + 1 against 4; where
    // two groups are left beside the sweep, 4/2 against 4/3 + 1.
    if (share && sweeps && !cm && fk >= 0 && avail < 2) {
        int g = 0;
        for (int deg = deg_f; deg >= 1; --deg) {
            g = min_wgs(fk, deg);
            if (g > 0 && g <= grid) break;
        }
        const int G = g > 0 ? std::min(grid / g, lanes) : 0;
        if (G > avail) {
            const int gsz = grid / G;
            lds = 0;
            int used = 1;
            for (size_t k = 0; k < plans.size(); ++k) {
                const LanePlan &p = plans[k];
                if (p.count == 0) continue;
                int n = 1, m = 1;
                if (!fit(p.kind, gsz, shape[k], n)) return false;
                if (!fit(p.lead_kind >= 0 ? p.lead_kind : p.kind, gsz, lead_shape[k], m))
                    return false;
                lds = std::max(lds, std::max(res_lds_bytes(shape[k], C.W, HN),
                                             res_lds_bytes(lead_shape[k], C.W, HN)));
                used = std::max(used, std::max(n, m));
            }
            for (size_t k = 0; k < plans.size(); ++k) {
                ngroups[k] = plans[k].kind == fk ? G : 0;
                nwg[k] = used;
            }
            one_queue = true;
            return true;
        }
    }
    // (a sweep that is its launch's only lane needs no group beside it, but has to fit:
    // the cold coarse-mesh sweep takes 260 workgroups at 1500 x 1500 elements)
    if (!own || lat > grid) return false;
    if (nb > 0 && (avail < 1 || (avail < nb && (!share || nb > 2)))) return false;
    avail = std::min(avail, lanes);
    const int gsz = g_min > 0 ? std::max(g_min, (grid - lat) / std::max(1, avail)) : 1;
    int left = avail, kinds = nb;
    double wF = 0.0;
    for (const auto &p : plans)
        if (!p.latency && p.count > 0) wF += p.weight * p.count;
    int used_max = 1;
    for (size_t k = 0; k < plans.size(); ++k) {
        const LanePlan &p = plans[k];
        if (p.latency || p.count == 0) continue;
        --kinds;
        int q = p.queues > 0 ? p.queues : (int)floor(avail * p.weight * p.count / wF);
        q = std::max(1, std::min(q, std::min(p.count, left - kinds)));
        // (one group for two kinds: they share a queue)
        q = std::min(q, left);
        ngroups[k] = q;
        left -= q;
        int n = 1;
        if (!fit(p.kind, gsz, shape[k], n)) return false;
        lds = std::max(lds, lds_of(p.kind, shape[k]));
        used_max = std::max(used_max, n);
    }
    for (size_t k = 0; k < plans.size(); ++k)
        if (!plans[k].latency && plans[k].count > 0) nwg[k] = used_max;
    for (size_t k = 0; k < plans.size(); ++k)
        if (plans[k].lead_kind < 0) lead_shape[k] = shape[k];
    return true;
}

}  // namespace

}  // namespace pt

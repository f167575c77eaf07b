// Runs the planner of resident lanes (pt_plan.h) on the host, for
// tests/test_plan_host.py. Reads one request per line from stdin and answers each
// with one line:
//   shape W HN max_wg deg rows      -> ok tw th deg nr wgs lds | min_wgs
//   window W HN tw th deg nr        -> fits lds
//   plan nx ny Ntau M grid rows sweep_wgs share cm, then 9 numbers per kind of lane
//        (kind count slice0 dir weight latency queues fixed_nwg lead_kind)
//                                   -> ok one_queue lds, then per kind of lane
//                                      ngroups nwg tw th deg nr
#include "../paper_2411_19030_amd/csrc/pt_plan.h"

#include <iostream>
#include <sstream>
#include <string>

using namespace pt;

constexpr int kLdsDoubles = (160 * 1024 - 1024) / 8;

static void shape(std::istream &in) {
    int W, HN, wg, deg, rows, n = 0;
    in >> W >> HN >> wg >> deg >> rows;
    const size_t cap = kLdsDoubles * sizeof(double);
    Shape s{};
    const bool ok = res_fit(W, HN, wg, deg, rows, cap, s, n);
    std::cout << ok << ' ' << s.tw << ' ' << s.th << ' ' << s.deg << ' ' << s.nr << ' ' << n << ' '
              << (ok ? res_lds_bytes(s, W, HN) : 0) << ' ' << res_min_wgs(W, HN, deg, rows, cap)
              << '\n';
}

static void window(std::istream &in) {
    int W, HN;
    Shape s{};
    in >> W >> HN >> s.tw >> s.th >> s.deg >> s.nr;
    std::cout << res_window_fits(s, W, HN, kLdsDoubles * sizeof(double)) << ' '
              << res_lds_bytes(s, W, HN) << '\n';
}

static void plan(std::istream &in) {
    Consts C{};
    pt_tuning T{};
    CoarseMesh M{};
    int grid, sweep_wgs, cm;
    in >> C.nx >> C.ny >> C.Ntau >> C.M >> grid >> T.resident_npt_max >> sweep_wgs >>
        T.shared_queue >> cm;
    C.W = C.nx + 1;
    C.Nn = C.W * (C.ny + 1);
    std::vector<LanePlan> plans;
    LanePlan p{};
    int latency;
    while (in >> p.kind >> p.count >> p.slice0 >> p.dir >> p.weight >> latency >> p.queues >>
           p.fixed_nwg >> p.lead_kind) {
        p.latency = latency != 0;
        plans.push_back(p);
    }
    std::vector<int> ngroups(plans.size()), nwg(plans.size());
    std::vector<Shape> s(plans.size()), lead(plans.size());
    size_t lds = 0;
    bool one_queue = false;
    const bool ok = plan_resident(C, plans, T, grid, kLdsDoubles, sweep_wgs, cm ? &M : nullptr,
                                  ngroups, nwg, s, lead, lds, one_queue);
    std::cout << ok << ' ' << one_queue << ' ' << lds;
    for (size_t k = 0; k < plans.size(); ++k)
        std::cout << ' ' << ngroups[k] << ' ' << nwg[k] << ' ' << s[k].tw << ' ' << s[k].th << ' '
                  << s[k].deg << ' ' << s[k].nr;
    std::cout << '\n';
}

int main() {
    std::string line, what;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        in >> what;
        if (what == "shape") shape(in);
        else if (what == "window") window(in);
        else plan(in);
    }
}

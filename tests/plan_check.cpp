// plan_check.cpp -- host-only driver: the launch plan of n equal cells (one
// branch of 8 CVs, n_syn synapses each) as planned, and the plan under which the
// autotuner times the library's own shape and an explicit one on a sample.
// Usage: plan_check n_cells n_sample n_syn; prints threads, slots and most cells
// per workgroup of four plans: full model, sample, and both trials.
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../paper_1901_07454_amd/csrc/sim.hpp"

using namespace arbmi;

int main(int argc, char** argv) {
    if (argc < 4) return 2;
    const int n = std::atoi(argv[1]), k = std::atoi(argv[2]), ns = std::atoi(argv[3]);
    std::vector<arb_cell> cells(static_cast<size_t>(n));
    std::vector<arb_branch> br(static_cast<size_t>(n) * 20);
    std::vector<arb_synapse> syn;
    for (int c = 0; c < n; ++c) {
        cells[c].branch_begin = 20 * c;
        cells[c].n_branch = 20;
        for (int b = 0; b < 20; ++b) {
            br[20 * c + b].parent = b - 1;
            br[20 * c + b].n_cv = 8;
        }
        for (int q = 0; q < ns; ++q) {
            syn.emplace_back();
            syn.back().cell = c;
        }
    }
    auto view = [&](int m) {
        ModelView v{};
        v.cells = cells.data();
        v.n_cells = m;
        v.br = br.data();
        v.n_br = 20 * int64_t(m);
        v.syn = syn.data();
        v.n_syn = int64_t(ns) * m;
        return v;
    };
    const DeviceLimits d;
    arb_params p{};
    auto show = [](const Plan& pl) {
        std::printf("%d %d %d %lld\n", pl.coef_mode, pl.block_threads, pl.reg_slots, (long long)pl.max_cells_per_pack);
    };
    const ModelView full = view(n), smp = view(k);
    for (const ModelView& v : {full, smp})
        show(choose_plan(v.cells, v.n_cells, v.br, v.n_br, v.syn, v.n_syn, p, d.lds_max, d.n_cu));
    show(trial_plan(full, smp, p, d));
    p.coef_mode = 3;
    p.block_threads = 128;
    show(trial_plan(full, smp, p, d));
    return 0;
}

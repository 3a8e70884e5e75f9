// plan.cpp -- launch shape and packing limits for a model.
#include <algorithm>
#include <cmath>
#include <vector>

#include "sim.hpp"

namespace arbmi {

namespace {

// A model's mean cell, for the estimate below.
struct MeanCell {
    double tasks, hh, nl, syn;  // branches with the soma, CVs with hh, nonlinear CVs, synapses
    int levels;                 // of the deepest tree, the soma's with them
};

// LDS of a workgroup of c such cells with at most binary branch points.
int64_t mean_lds(int len, int64_t c, const MeanCell& m, bool grads = false) {
    PackDesc D{};
    D.ntk = int32_t(double(c) * m.tasks);
    D.nslot = len * D.ntk;
    D.nhh = int32_t(double(c) * m.hh);
    D.nnl = int32_t(double(c) * m.nl);
    D.nsyn = int32_t(double(c) * m.syn);
    D.binary = 1;
    return grads ? std::max(pack_lds_bytes(D, 3), reg_adjoint_lds_bytes(D)) : pack_lds_bytes(D, 3);
}

// Time of a step (us) of n cells, c to a workgroup of T threads whose branches
// take `len` registers: the workgroups a CU holds at once by registers and LDS
// run in rounds of that many, and a round takes the time of its chain of phases
// (local solve, tree levels, nonlinear CVs and gates one after another in a
// thread) and of its instructions on the SIMDs, which overlap in part.  The
// constants are a fit to 14,400 measured shapes of 917 models (30 to 9,000 cells
// of 1 to 126 branches of 4, 8, 13 or 16 CVs, none to all of them hh, 1 to 120
// synapses): 12% off in the mean, 6% at the median.
double step_us(int T, int len, int64_t c, int64_t n, int n_cu, int64_t lds_max, const MeanCell& m) {
    const double tasks = double(c) * m.tasks, hh = double(c) * m.hh, nl = double(c) * m.nl;
    const double held = std::ceil(tasks / T) * len / 8;  // 8-CV branches a thread holds
    const int64_t lds = mean_lds(len, c, m);
    const int by_reg = (held <= 1 ? 3 : held <= 2 ? 2 : 1) * 256 / T;
    const int64_t on_cu = std::max<int64_t>(1, std::min<int64_t>(by_reg, lds_max / lds));
    const bool spread = hh <= kSpreadHH;  // a thread for every gate
    const double chain = (T == 64 ? 0.91 : T == 128 ? 1.1 : 1.07) + 0.12 * (m.levels + 1) + 0.23 * (held - 1) +
                         (spread ? 0.17 : 0.92 * std::ceil(hh / T)) + 0.28 * std::ceil(nl / T);
    const double waves = T / 64.0;
    const double issue = 0.24 * held + (spread ? 0.085 : 0.31 * std::ceil(hh / 64) / waves) +
                         0.15 * std::ceil(nl / 64) / waves;
    auto round = [&](int64_t on) {
        return std::pow(std::pow(chain, 1.2) + std::pow(double(on) * waves / 4 * issue, 1.2), 1 / 1.2);
    };
    const int64_t packs = (n + c - 1) / c, at_once = n_cu * on_cu, rest = packs % at_once;
    return double(packs / at_once) * round(on_cu) + (rest ? round((rest + n_cu - 1) / n_cu) : 0.0);
}

}  // namespace

Plan choose_plan(const arb_cell* cells, int32_t n_cells, const arb_branch* br, int64_t n_br, const arb_synapse* syn,
                 int64_t n_syn, const arb_params& p, int64_t lds_max, int n_cu) {
    Plan pl;
    lds_max -= 256;  // static LDS of the kernels
    // largest cell (CVs), widest branch level, longest branch, most branches,
    // branches of all cells, most CVs with nonlinear or point currents
    int64_t max_cv = 1, max_width = 1, max_len = 1, max_tasks = 1, max_tasks8 = 1, all_tasks8 = 0, max_nl = 0,
            max_hh = 0, max_syn = 0, max_lds = 1, max_depth = 0, all_tasks = 0, all_hh = 0, all_nl = 0,
            all_syn = 0;
    std::vector<int> depth, count;
    std::vector<int64_t> n_syn_of(size_t(std::max(n_cells, 0)), 0);
    for (int64_t q = 0; q < n_syn && syn; ++q)
        if (syn[q].cell >= 0 && syn[q].cell < n_cells) n_syn_of[syn[q].cell]++;
    for (int32_t c = 0; c < n_cells && cells; ++c) {
        const arb_cell& C = cells[c];
        if (C.branch_begin < 0 || C.n_branch < 0 || C.branch_begin + C.n_branch > n_br) continue;
        int64_t n = 1, seg8 = 1, hh = (C.soma_mech & ARB_MECH_HH) ? 1 : 0;
        depth.assign(C.n_branch, 0);
        count.assign(C.n_branch + 2, 0);
        for (int32_t b = 0; b < C.n_branch; ++b) {
            const arb_branch& B = br[C.branch_begin + b];
            n += std::max(0, B.n_cv);
            seg8 += (std::max(1, B.n_cv) + 7) / 8;
            if (B.mech & ARB_MECH_HH) hh += std::max(0, B.n_cv);
            max_len = std::max<int64_t>(max_len, B.n_cv);
            depth[b] = (B.parent < 0 || B.parent >= b) ? 1 : depth[B.parent] + 1;
            max_depth = std::max<int64_t>(max_depth, depth[b]);
            if (depth[b] <= C.n_branch) count[depth[b]]++;
        }
        for (int v : count) max_width = std::max<int64_t>(max_width, v);
        max_cv = std::max(max_cv, n);
        max_tasks = std::max<int64_t>(max_tasks, int64_t(C.n_branch) + 1);
        max_tasks8 = std::max(max_tasks8, seg8);
        all_tasks8 += seg8;
        max_hh = std::max(max_hh, hh);
        max_syn = std::max(max_syn, n_syn_of[c]);
        all_tasks += C.n_branch + 1;
        all_hh += hh;
        all_syn += n_syn_of[c];
        const int64_t nl = p.n_densities > 0 ? n : std::min(n, hh + n_syn_of[c]);
        max_nl = std::max(max_nl, nl);
        all_nl += nl;
        // the register layout's LDS of the cell, near enough (pack_lds_bytes)
        const int64_t syn_lds = 24 * n_syn_of[c] > kSynLdsMax ? 0 : 24 * n_syn_of[c];
        max_lds = std::max(max_lds, (128 + 24) * seg8 + syn_lds + 44 * hh + (p.n_densities > 0 ? 37 : 24) * nl);
    }
    const bool grads = (p.flags & ARB_FLAG_GRADIENTS) != 0;
    // some cell has too many synapses for LDS, and they are of more than one kind
    // (near enough: the model's are)
    bool streams = false;
    if (24 * max_syn > kSynLdsMax)
        for (int64_t q = 1; q < n_syn && !streams; ++q)
            streams = syn[q].tau_ms != syn[0].tau_ms || syn[q].e_rev_mV != syn[0].e_rev_mV;

    // Streamed coefficients (mode 2): 16 B of LDS per CV, 256 threads, enough
    // cells per pack that the widest branch level fills the workgroup.  Also
    // the fallback of the other modes.
    const int T2 = p.block_threads ? p.block_threads : 256;
    pl.fallback_cells_per_pack = std::max<int64_t>(1, std::min<int64_t>(T2, T2 / max_width));
    pl.fallback_lds_budget = lds_max / 2;
    pl.fallback_lds_hard_max = lds_max;
    if (grads) {  // the streamed adjoint kernel keeps 32 B per CV (forward: 16 B)
        pl.fallback_lds_budget = lds_max / 3;
        pl.fallback_lds_hard_max = lds_max / 2 - 1024;
    }

    // Register-resident coefficients (mode 3) by default when every branch
    // fits the registers: L = 8 CVs with up to 3 branches per thread, or
    // L = 16 with 1.  On request (and for the autotuner) longer branches are
    // cut into chains of 8-CV segments.  An explicit request is honoured or
    // refused by the lowering, never changed.  With gradients the packs must
    // also fit the register-resident adjoint kernel (the lowering checks).
    // The same cut is the default for longer branches, where the caller left
    // everything to the library: streamed, a step walks each branch as one
    // chain of CVs, whose length bounds it (64 cells of 7 sections of 27 CVs:
    // 16.4 us a step streamed, 2.3 cut into segments; 8192 of them 22.5 / 5.5,
    // with every CV hh 75 / 31; one cell of a 2000-CV cable 363 / 26).  Up to
    // the segments that 256 threads hold, whose packs fit the adjoint's LDS
    // (lower_planned).  Models with generated mechanisms, which have no
    // gradients, get it on request only.  arb_get_info still says coef_mode 2
    // for them.
    pl.long_cut = p.coef_mode == 0 && max_len > 16 && p.block_threads == 0 && p.cells_per_pack == 0 && !grads &&
                  !(p.flags & ARB_FLAG_AUTOTUNE) && p.n_densities == 0 && max_tasks8 <= 768;
    const bool reg_ok = p.coef_mode == 3 || (p.coef_mode == 0 && max_len <= 16) || pl.long_cut;
    if (reg_ok) {
        pl.coef_mode = 3;
        pl.reg_len = (max_len > 8 && max_len <= 16) ? 16 : 8;
        pl.lds_budget = lds_max / 2;
        pl.lds_hard_max = lds_max;
        const int64_t tasks = pl.reg_len == 8 ? std::max(max_tasks, max_tasks8) : max_tasks;
        if (p.block_threads == 0 && p.cells_per_pack == 0) {
            // One wave per workgroup where its register slots hold the largest
            // cell: a step is a chain of short phases, and in one wave they
            // follow each other without barriers (8192 cells of 1017 CVs:
            // 12.2 us a step, against 15.6 with four cells in 256 threads;
            // 96 of them 2.3 against 3.3).  More threads pay while there are
            // fewer waves than the GPU has SIMDs and a cell has work for
            // them: several rounds of branches or of nonlinear CVs per thread
            // (256 cells of 200 hh CVs: 6.6 / 4.8 / 3.7 us a step with 64 / 128
            // / 256 threads, 1024 of them 9.0 / 11.3 / 16.7).
            const int64_t slots = pl.reg_len == 8 ? 3 : 1;
            int T = 64;
            while (T < 256 && tasks > slots * T) T *= 2;
            // Where LDS holds few of these cells per CU and they have several
            // nonlinear CVs for each thread, two waves per SIMD by threads
            // (1024 cells with every CV hh: 505 CVs, 44 KB: 26.0 / 16.8 / 11.1
            // us a step with 64 / 128 / 256 threads; 249 CVs, 22 KB: 7.5 / 6.8
            // / 7.5).
            const int64_t heavy = p.n_densities > 0 ? max_nl : max_hh;  // costly ones
            while (T < 256 && heavy > T && (lds_max / max_lds) * (T / 64) < 8) T *= 2;
            // two such cells of more than 64 branches share 256 threads
            // better than they fill 128 each (2048 cells of 1017 CVs, a
            // quarter of them hh: 15.9 against 18.0 us a step), while there are
            // more of them than CUs take at once (512 cells: 6.6 against 6.0)
            int64_t pair = 0;
            if (T == 128 && heavy > 128 && tasks > 64 && tasks <= 128) {
                T = 256;
                pair = int64_t(n_cells) * (T / 64) <= 8 * int64_t(n_cu) ? 1 : 2;
            }
            const int64_t avg = std::max<int64_t>(1, all_tasks8 / std::max(1, n_cells));
            // Cells with generated mechanisms, two or more for each CU: 256
            // threads shared by cells of up to four nonlinear CVs a thread,
            // which keep its waves evenly busy with instances and its lanes with
            // branches (us a step, a wave for each cell / so / 256 threads
            // filled to half the LDS: 8192 cells of 57 CVs 28.6 / 11.8 / 18.4, of
            // 121 37.8 / 21.6 / 29.5, of 249 50.3 / 39.5 / 47.1; 600 cells of 121
            // 7.7 / 5.7 / 16.2), and whose synapses stay in LDS together, as
            // generated mechanisms need.
            int64_t share = 0;
            if (p.n_densities > 0 && pl.reg_len == 8)
                share = std::min({256 / avg, 4 * 256 / std::max<int64_t>(1, max_nl), int64_t(n_cells) / n_cu,
                                  kSynLdsMax / (24 * std::max<int64_t>(1, max_syn))});
            if (T < 256 && share >= 2) T = 256;
            // Cells whose synapses stream from HBM each step want as many loads
            // in flight as there are threads, and branches for all of them (914
            // cells of 130 branches and 2177 synapses of two kinds: 30.5 us a
            // step with 64 threads, 15.1 with 256).
            if (T < 256 && streams && tasks > T) T = 256;
            // Cells of which the largest, more than one wave takes, is more
            // than twice the mean share 256 threads or more (below).
            const bool mixed = tasks > slots * 64 && max_tasks > 2 * all_tasks / std::max(1, n_cells);
            if (T < 256 && mixed) T = 256;
            const int want = (max_nl > 128 || tasks > 128) ? 256 : max_nl > 64 ? 128 : 64;
            while (T < want && int64_t(n_cells) * (2 * T / 64) <= 4 * int64_t(n_cu)) T *= 2;
            // Cells of more than 256 branches in 512 threads, two waves per SIMD,
            // where the kernels have it (uneven cells of up to 5000 CVs, us a
            // step with 256 threads / 512: 64 cells 14.2 / 11.2, 512 of them
            // 15.2 / 12.1, 2000 of them 30.5 / 26.6), where each has a CU to
            // itself by number or by LDS (256 threads let two share one: 312
            // cells of 300 branches, 74 KB, 6.6 / 8.8, 403 of 450, 70 KB, 5.3 /
            // 6.9; 404 of 378, 110 KB, 15.1 / 13.1).  Branches of up to 8 CVs,
            // and where the caller asked for this layout no more of them than
            // it takes with any other workgroup (an explicit request is
            // honoured or refused).
            if (T == 256 && pl.reg_len == 8 && tasks > 256 && tasks <= (p.coef_mode == 3 ? 768 : 1024) &&
                !grads && !pl.long_cut && p.n_densities == 0 && (n_cells <= n_cu || 2 * max_lds > lds_max || mixed))
                T = 512;
            // Cells with generated mechanisms and more nonlinear CVs than 256
            // threads, where each has a CU to itself (by number, or by LDS):
            // a step is mostly visits of their instances, in series per
            // thread (256 cells: 1017 CVs 8.7 us a step with 256 threads, 7.7
            // with 512; 2041 CVs 13.0 / 10.8; 505 CVs 6.3 / 6.1; 249 CVs 5.4 /
            // 6.0).
            if (T == 256 && p.n_densities > 0 && pl.reg_len == 8 && max_nl > 256 && tasks <= 512 &&
                (n_cells <= n_cu || 2 * max_lds > lds_max))
                T = 512;
            pl.block_threads = T;
            pl.reg_slots = pl.reg_len == 8 ? int(std::min<int64_t>(3, std::max<int64_t>(1, (tasks + T - 1) / T))) : 1;
            // Several cells in a workgroup only where its lanes would idle
            // otherwise: as many average cells as its slots take, and no more
            // nonlinear CVs than threads (two cells of 200 hh CVs in 64
            // threads: 11.9 us a step, one 7.4).  Four cells of 16 branches in
            // one wave cost what one costs (16,000 of them 4.1 against 11.2
            // us a step).  Cells that differ much in size (T = 256) fill a
            // workgroup up to half the LDS, unless every cell can have a CU.
            if (T == 256) pl.wide_slots = pl.reg_len == 8 ? (tasks <= 2 * T ? 2 : 3) : 1;
            if (pair) {
                pl.max_cells_per_pack = pair;
            } else if (T == 256 && share >= 2) {
                pl.max_cells_per_pack = share;
            } else if (T >= 256 && mixed && tasks <= slots * 128) {
                // as many as leave every CU a workgroup, in 512 threads with
                // more than 256 branches (us a step, 256 threads filled / by the
                // mean cell, one or four to a workgroup / so: 846 cells of 20 to
                // 3000 CVs, a quarter hh, 9.9 / 15.5 / 9.0; 848 of them, soma hh,
                // 5.5 / 6.8 / 5.4)
                pl.max_cells_per_pack = (n_cells + n_cu - 1) / n_cu;
                pl.estimated = T > 256;  // (a state header of its own)
            } else if (T >= 256 && tasks > slots * 128) {
                pl.max_cells_per_pack = n_cells <= n_cu ? 1 : T;
            } else {
                int64_t c = std::min(pl.reg_slots * T / avg, T / std::max<int64_t>(1, max_nl));
                // while that leaves SIMDs idle, no more cells than have a
                // thread for every gate
                const int64_t spread = kSpreadHH / std::max<int64_t>(1, max_hh);
                if (spread >= 1 && n_cells <= 4 * int64_t(n_cu) * spread) c = std::min(c, spread);
                pl.max_cells_per_pack = std::max<int64_t>(1, c);
            }
            // The rules weigh one thing at a time, and lose to 256 threads
            // filled to half the LDS where a last round of workgroups is nearly
            // empty, or a wave that could take more cells has one.  For many
            // similar cells that fit two waves, where the estimate says so, the
            // shape with the least estimated step (us a step, filled / by the
            // rules / so: 7578 cells of 40 CVs, 14 hh, 6.6 / 10.2 / 4.8; 5152 of
            // 121, 65 hh, 8.1 / 13.0 / 7.9; 1443 of 1281, soma hh, 4.2 / 6.8 /
            // 4.3).  Of 799 models of 256 cells and more, 84 were more than 3%
            // slower by the rules than filled, and 21 are so.
            const double n = std::max(1, n_cells);
            const MeanCell mean{double(all_tasks) / n, double(all_hh) / n, double(all_nl) / n, double(all_syn) / n,
                                int(max_depth) + 1};
            const bool similar = double(max_tasks) <= 1.25 * mean.tasks + 1 && double(max_nl) <= 1.25 * mean.nl + 8;
            const int64_t cap = pl.reg_len == 8 ? 2 : 1;  // branches a thread holds
            // The adjoint kernel gains less from small workgroups than the step
            // kernel: 256 threads, filled, wherever that leaves two thirds of
            // the CUs a workgroup (867 cells of 201 hh CVs, forward and gradient,
            // us a step: a wave for each 39.5, filled 30.4), and for more than 40
            // branches of up to 16 CVs (98 cells of 820 CVs: 15.8 / 13.3).  Of 250
            // models 18 were more than 3% slower by the rules above than filled,
            // and 5 are so.
            if (grads && similar && pl.block_threads < 256 && max_tasks <= cap * 256) {
                int64_t fill = 1;
                while (fill < 256 && (fill + 1) * max_tasks <= cap * 256 &&
                       mean_lds(pl.reg_len, fill + 1, mean, true) <= pl.lds_budget)
                    ++fill;
                if (3 * n_cells >= 2 * n_cu * fill || (pl.reg_len == 16 && max_tasks > 40)) {
                    pl.block_threads = 256;
                    pl.reg_slots = pl.wide_slots = int(cap);
                    pl.max_cells_per_pack = 256;
                }
            }
            if (n_cells >= n_cu && max_tasks <= 128 && max_len <= 16 && similar && !grads && p.n_densities == 0 &&
                24 * max_syn <= kSynLdsMax) {
                auto fits = [&](int threads, int64_t c) {
                    return c == 1 || (c * max_tasks <= cap * threads && 24 * c * max_syn <= kSynLdsMax &&
                                      c <= threads && mean_lds(pl.reg_len, c, mean) <= pl.lds_budget);
                };
                auto us = [&](int threads, int64_t c) {
                    return step_us(threads, pl.reg_len, c, n_cells, n_cu, lds_max, mean);
                };
                int64_t fill = 1;  // cells of 256 threads filled
                while (fits(256, fill + 1)) ++fill;
                // (a shape has to win by more than the estimate's ties)
                double least = 0.985 * us(pl.block_threads, std::min(pl.max_cells_per_pack, fill));
                const bool lost = us(256, fill) < least;
                int best_T = 0;
                int64_t best_c = 0;
                for (const int threads : {64, 128, 256})
                    for (int64_t c = 1; c <= fill && lost; ++c) {
                        if (max_tasks > cap * threads || !fits(threads, c) || us(threads, c) >= least) continue;
                        least = us(threads, c);
                        best_T = threads;
                        best_c = c;
                    }
                if (best_T) {
                    pl.estimated = true;
                    pl.block_threads = best_T;
                    pl.max_cells_per_pack = best_c;
                    pl.reg_slots = pl.reg_len == 8 ? int((best_c * max_tasks + best_T - 1) / best_T) : 1;
                    pl.wide_slots = best_T == 256 ? int(cap) : 0;
                }
            }
            return pl;
        }
        pl.block_threads = p.block_threads ? p.block_threads : 256;
        if (pl.reg_len == 8)
            pl.reg_slots = (tasks <= 2 * pl.block_threads) ? 2 : 3;
        else
            pl.reg_slots = 1;
        pl.max_cells_per_pack = p.cells_per_pack > 0 ? std::min(p.cells_per_pack, pl.block_threads) : pl.block_threads;
        if (p.cells_per_pack > 0) pl.lds_budget = lds_max;
        return pl;
    }

    pl.block_threads = T2;
    const int64_t need_lds1 = (max_cv + max_cv / 4) * 6 * 8 + max_cv * 3 * 8;
    pl.coef_mode = (p.coef_mode == 1 || p.coef_mode == 2) ? p.coef_mode : 2;
    if (pl.coef_mode == 1 && need_lds1 > lds_max && p.coef_mode == 0) pl.coef_mode = 2;
    pl.lds_budget = lds_max / 2;
    pl.lds_hard_max = lds_max;
    if (grads) {
        // the adjoint kernel keeps 32 B per CV (forward, streamed: 16 B)
        pl.coef_mode = 2;
        pl.lds_budget = lds_max / 3;
        pl.lds_hard_max = lds_max / 2 - 1024;
    }
    if (p.cells_per_pack > 0) {
        pl.max_cells_per_pack = std::min(p.cells_per_pack, pl.block_threads);
        pl.lds_budget = lds_max;  // an explicit pack size wins over the LDS target
    } else {
        pl.max_cells_per_pack = pl.fallback_cells_per_pack;
    }
    return pl;
}

Plan trial_plan(const ModelView& full, const ModelView& sample, const arb_params& p, const DeviceLimits& d) {
    const bool own = p.coef_mode == 0 && p.block_threads == 0 && p.cells_per_pack == 0;
    const ModelView& m = own ? full : sample;
    return choose_plan(m.cells, m.n_cells, m.br, m.n_br, m.syn, m.n_syn, p, d.lds_max, d.n_cu);
}

}  // namespace arbmi

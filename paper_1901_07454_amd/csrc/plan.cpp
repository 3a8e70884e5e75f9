// plan.cpp -- launch shape and packing limits for a model.
#include <algorithm>
#include <vector>

#include "sim.hpp"

namespace arbmi {

Plan choose_plan(const arb_cell* cells, int32_t n_cells, const arb_branch* br, int64_t n_br, const arb_synapse* syn,
                 int64_t n_syn, const arb_params& p, int64_t lds_max, int n_cu) {
    Plan pl;
    lds_max -= 256;  // static LDS of the kernels
    // largest cell (CVs), widest branch level, longest branch, most branches,
    // branches of all cells, most CVs with nonlinear or point currents
    int64_t max_cv = 1, max_width = 1, max_len = 1, max_tasks = 1, max_tasks8 = 1, all_tasks8 = 0, max_nl = 0,
            max_hh = 0, max_syn = 0, max_lds = 1;
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
            if (depth[b] <= C.n_branch) count[depth[b]]++;
        }
        for (int v : count) max_width = std::max<int64_t>(max_width, v);
        max_cv = std::max(max_cv, n);
        max_tasks = std::max<int64_t>(max_tasks, int64_t(C.n_branch) + 1);
        max_tasks8 = std::max(max_tasks8, seg8);
        all_tasks8 += seg8;
        max_hh = std::max(max_hh, hh);
        max_syn = std::max(max_syn, n_syn_of[c]);
        const int64_t nl = p.n_densities > 0 ? n : std::min(n, hh + n_syn_of[c]);
        max_nl = std::max(max_nl, nl);
        // the register layout's LDS of the cell, near enough (pack_lds_bytes)
        const int64_t syn_lds = 24 * n_syn_of[c] > kSynLdsMax ? 0 : 24 * n_syn_of[c];
        max_lds = std::max(max_lds, (128 + 24) * seg8 + syn_lds + 44 * hh + (p.n_densities > 0 ? 37 : 24) * nl);
    }
    const bool grads = (p.flags & ARB_FLAG_GRADIENTS) != 0;

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
            const int want = (max_nl > 128 || tasks > 128) ? 256 : max_nl > 64 ? 128 : 64;
            while (T < want && int64_t(n_cells) * (2 * T / 64) <= 4 * int64_t(n_cu)) T *= 2;
            // Cells of more than 256 branches in 512 threads, two waves per SIMD,
            // where the kernels have it (uneven cells of up to 5000 CVs, us a
            // step with 256 threads / 512: 64 cells 14.2 / 11.2, 512 of them
            // 15.2 / 12.1, 2000 of them 30.5 / 26.6): branches of up to 8 CVs, and
            // where the caller asked for this layout no more of them than it
            // takes with any other workgroup (an explicit request is honoured
            // or refused).
            if (T == 256 && pl.reg_len == 8 && tasks > 256 && tasks <= (p.coef_mode == 3 ? 768 : 1024) &&
                !grads && !pl.long_cut && p.n_densities == 0)
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

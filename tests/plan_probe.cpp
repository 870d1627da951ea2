// Prints the plans of maps (the runtime's plan_job, host code only): one map
// per input line, one line of "name=value" fields per map.
//   kind precision K bins t_sft exact32 anchor_most smaller n_t0 t0... n_tau tau...
// kind: 0 rect, 1 exp; precision: tfstat_precision; anchor_most: bytes of
// anchors, -1 the default; smaller: times to plan with less workspace; t0
// relative to the data's start.
#include "../paper_1805_05652_amd/csrc/runtime.cpp"

#include <iostream>

int main() {
    int kind, prec, exact32, smaller;
    int64_t K, bins, T, anchor_most;
    while (std::cin >> kind >> prec >> K >> bins >> T >> exact32 >> anchor_most >> smaller) {
        AtomsSet at;
        at.K = (int32_t)K;
        at.n_bins = (int32_t)bins;
        at.t_sft = T;
        at.slide_ok = at.slide_ok64 = (K + 1) * bins * 32 < ((int64_t)1 << 31);
        at.exact32 = exact32 != 0;
        at.half_ok = true;
        at.amax = at.bmax = 1.0;
        Job j;
        j.at = &at;
        j.prec = prec;
        j.win.type = kind == 0 ? TFSTAT_WIN_RECT : TFSTAT_WIN_EXP;
        int64_t n = 0;
        std::cin >> n;
        j.win.t0.resize(n);
        for (auto &v : j.win.t0) std::cin >> v;
        std::cin >> n;
        j.win.tau.resize(n);
        for (auto &v : j.win.tau) std::cin >> v;
        j.runs_min_spread = kRunsAuto;
        j.split_min_bins = kSplitMinBins;
        if (anchor_most >= 0) j.anchor_most = (size_t)anchor_most;
        plan_job(j);
        int done = 0;
        while (done < smaller && plan_smaller(j)) ++done;
        std::cout << "smaller=" << done << " anchors=" << (j.slide ? anchor_bytes(j, j.pass_tt, j.pass_bg) : 0) << " no_slide=" << j.no_slide << " ";
        std::cout << "slide=" << j.slide << " bg=" << j.bg << " n_bg=" << j.n_bg << " n_tt=" << j.n_tt << " n_seg=" << j.n_seg
                  << " seg_rows=" << j.seg_rows << " range_len=" << j.range_len << " n_range=" << j.n_range << " n_sup=" << j.n_sup
                  << " kbeg=" << j.kbeg << " waves=" << j.waves << " stage=" << j.stage << " rect_rows=" << j.rect_rows
                  << " scan_blk=" << j.scan_blk << " ws=" << j.ws_bytes;
        // (passes: first tau tile, tau tiles, first bin group, bin groups)
        for (int32_t pass = 0; j.slide && pass < n_passes(j); ++pass) {
            const tfs::SlideParams q = slide_params(j, pass);
            std::cout << " pass" << pass << "=" << q.tt0 << "," << q.pass_tt << "," << q.bg0 << "," << q.pass_bg;
        }
        std::cout << std::endl;
    }
    return 0;
}

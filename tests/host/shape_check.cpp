// Host-side view of the launch rules (csrc/hexi_shapes.h).  Reads one ring step per line from stdin:
//   head_dim nq nkv forced_run_len  n_q_segs (start len)...  n_kv_segs (start len)...  [kv_of_q ...]
// and prints: rows per forward workgroup (0: 256), rows per dQ workgroup (0: 256), keys per dK / dV workgroup, q heads per dK / dV
// workgroup, whether dk / dv are summed with atomics, and that of the 128-key launch the step would otherwise take; then, for
// calls for one half alone, the rows per dQ workgroup and the keys per dK / dV workgroup; for fp32 inputs the workgroup
// shape (0 shared, 1 split, 2 split with two on a CU) of the forward, of dQ, of dK / dV and of dQ alone; and the q heads per
// dK / dV workgroup of a call for dK / dV alone, and of a whole step that adds to dk and dv; the
// forward's 256-row tiles and those left to 64-row workgroups in a launch behind it.
#include <cstdio>
#include <cstring>
#include <iostream>
#include <sstream>
#include <string>
#include "hexi_internal.h"
#include "hexi_shapes.h"
#include "read_segs.h"

int main()
{
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream is(line);
        AttnGeom g;
        std::memset(&g, 0, sizeof(g));
        int forced;
        is >> g.d >> g.nq >> g.nkv >> forced;
        g.qs = read_segs(is);
        g.ks = read_segs(is);
        g.lq = g.qs.total; g.lc = g.ks.total;
        int m;
        for (int h = 0; h < g.nq; ++h) g.kv_of_q[h] = (signed char)((is >> m) ? m : h / (g.nq / g.nkv));
        BwdPlan plan;
        hexi_plan_bwd(g, forced, true, true, false, &plan);
        HeadRuns runs;
        const bool shared = hexi_build_head_runs(g.kv_of_q, g.nq, g.nkv, plan.run_len, &runs);
        const bool shared_128 = hexi_build_head_runs(g.kv_of_q, g.nq, g.nkv, plan.run_len_128, &runs);
        BwdPlan dq_alone, dkdv_alone;
        hexi_plan_bwd(g, forced, true, false, false, &dq_alone);
        hexi_plan_bwd(g, forced, false, true, false, &dkdv_alone);
        BwdPlan added;
        hexi_plan_bwd(g, forced, true, true, true, &added);
        QShare share;
        const int fwd_rows = hexi_fwd_split_rows(g, &share), n_q_tiles = (g.lq + 255) / 256, fwd_tiles = share.n_units(g.nq);
        F32Shape kv32, q32, q32_alone, unused;
        hexi_f32_bwd_shapes(g, true, true, &kv32, &q32);
        hexi_f32_bwd_shapes(g, true, false, &unused, &q32_alone);
        std::printf("%d %d %d %d %d %d %d %d %d %d %d %d %d %d %d %d\n", fwd_rows, plan.dq_rows, plan.split_keys ? plan.keys : 128, plan.run_len, (int)shared,
                    (int)shared_128, dq_alone.dq_rows, dkdv_alone.split_keys ? dkdv_alone.keys : 128,
                    (int)hexi_f32_fwd_shape(g), (int)q32, (int)kv32, (int)q32_alone, dkdv_alone.run_len, added.run_len, fwd_tiles, g.nq * n_q_tiles - fwd_tiles);
    }
    return 0;
}

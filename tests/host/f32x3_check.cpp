// Host-side view of the launch rules of the split-operand fp32 kernels (csrc/hexi_shapes.h).  Reads one step per line from stdin: nq nkv
// head_dim, then the shard's and the chunk's segments as in shape_check.cpp, and prints whether the forward takes them, its 64-row tiles taken as such
// and all of them; for the backward, and again for one under HEXI_ACCUMULATE, whether it does, keys of a dK / dV unit, whether its dQ units have 64
// rows, and the units that the heads of a group are dealt to; then the chains of a score in the other kernels; and for a call for dQ alone whether it
// takes them and in 64 rows, for dK / dV alone and under HEXI_ACCUMULATE whether and in how many units a group; and the units to a group of a whole step with a run
// length forced to one head, and to all of them.
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
        is >> g.nq >> g.nkv >> g.d;
        for (int h = 0; h < g.nq; ++h) g.kv_of_q[h] = (signed char)(h / (g.nq / g.nkv));
        g.qs = read_segs(is);
        g.ks = read_segs(is);
        g.lq = g.qs.total;
        g.lc = g.ks.total;
        const F32x3Fwd f = hexi_f32x3_fwd(g);
        std::printf("%d %d %d", f.use, f.n64, (g.lq + 63) / 64 * g.nq);
        for (const bool accumulate : {false, true}) {
            const F32x3Bwd b = hexi_f32x3_bwd(g, accumulate);
            std::printf(" %d %d %d %d", b.use, 32 * b.key_blocks, b.rows64, b.runs);
        }
        const F32x3Bwd q = hexi_f32x3_bwd(g, false, true, false), kv = hexi_f32x3_bwd(g, false, false, true), added = hexi_f32x3_bwd(g, true, false, true);
        std::printf(" %d %d %d %d %d %d %d", hexi_f32_chains(g), q.use, q.rows64, kv.use, kv.runs, added.use, added.runs);
        std::printf(" %d %d\n", hexi_f32x3_bwd(g, false, true, true, 1).runs, hexi_f32x3_bwd(g, false, true, true, g.nq).runs);
    }
}

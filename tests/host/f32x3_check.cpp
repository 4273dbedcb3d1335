// Host-side view of the launch rules of the split-operand fp32 kernels (csrc/hexi_shapes.h).  Reads one step per line from stdin: nq nkv
// head_dim, then the shard's and the chunk's segments as in shape_check.cpp, and prints whether the forward takes them, its 64-row tiles taken as such
// and all of them, whether the backward does, keys of a dK / dV unit, whether its dQ units have 64 rows, and the units that the heads of a group are dealt to.
#include <cstdio>
#include <cstring>
#include <iostream>
#include <sstream>
#include <string>
#include "hexi_internal.h"
#include "hexi_shapes.h"

static SegTable read_segs(std::istringstream& is)
{
    SegTable t;
    std::memset(&t, 0, sizeof(t));
    is >> t.n;
    for (int s = 0; s < t.n; ++s) {
        int len;
        is >> t.start[s] >> len;
        t.row0[s] = t.total;
        t.total += len;
    }
    for (int s = t.n; s <= HEXI_MAX_SEGS; ++s) t.row0[s] = t.total;
    return t;
}

int main()
{
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream is(line);
        AttnGeom g;
        std::memset(&g, 0, sizeof(g));
        is >> g.nq >> g.nkv >> g.d;
        g.qs = read_segs(is);
        g.ks = read_segs(is);
        g.lq = g.qs.total;
        g.lc = g.ks.total;
        const F32x3Fwd f = hexi_f32x3_fwd(g);
        const F32x3Bwd b = hexi_f32x3_bwd(g, false);
        std::printf("%d %d %d %d %d %d %d\n", f.use, f.n64, (g.lq + 63) / 64 * g.nq, b.use, 32 * b.key_blocks, b.rows64, b.runs);
    }
}

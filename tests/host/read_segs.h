// A range as the host checks read it: n_segs (start len)...
#pragma once
#include <cstring>
#include <istream>
#include "hexi_internal.h"

static SegTable read_segs(std::istream& is)
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

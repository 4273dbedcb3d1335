// Which workgroup shapes a ring step is launched with, from its sizes: the rules of the bf16 and fp32 launchers, host code alone.
#pragma once
#include <cmath>
#include "hexi_internal.h"

namespace hexi_shapes {
constexpr int Q_TILE = 256;            // q rows of the large forward and dQ workgroups
constexpr int KV_STREAM_TILE = 64;     // keys per tile that they stream
constexpr int KV_TILE = 128;           // keys of the large dK / dV workgroups
constexpr int Q_STREAM_TILE = 64;      // q rows per tile that they stream
constexpr double SMALL_MARGIN = 1.03;  // the large workgroups are kept unless smaller ones are expected to be faster by this
constexpr double ORDER_MARGIN = 1.15;  // and sums in a fixed order unless others are (see BwdPlan)
}  // namespace hexi_shapes

// The units of a launch by the length of their serial chains (key tiles, q tiles, or 32-row blocks per wavefront).
struct Units {
    double sum = 0.0, longest = 0.0;
    long long n = 0;
    void add(double chain, long long k) { sum += chain * (double)k; n += k; longest = chain > longest ? chain : longest; }
};

// Time of a launch in us: a fixed part, rounds of units over 256 CUs, and its row-wise reads and writes.
struct LaunchFit {
    double fixed;
    double unit;       // per round
    double lo, hi;     // per chain step in a round that leaves most CUs idle, and in one that uses three quarters of them or more
    double mb;         // per MB read and written once per row (q, o, dO, dq, dk, dv)

    double us(const Units& u, double mbytes) const
    {
        if (u.n <= 0) return fixed;
        const double mean = u.sum / (double)u.n, rest = (double)(u.n % 256) / 256.0;
        const double busy = rest < 0.75 ? rest * rest / 0.5625 : 1.0;
        double last = u.n % 256 ? 1.0 : 0.0;
        if (u.n > 256) {           // units of unequal length fill each other's last round
            const double uneven = 2.0 * (u.longest / mean - 1.0);
            last *= 1.0 - (uneven < 1.0 ? uneven : 1.0) * (1.0 - rest);
        }
        const double full = (double)(u.n / 256);
        const double t = (full + last) * unit + mean * (full * hi + last * (lo + (hi - lo) * busy));
        const double chain = unit + u.longest * lo;
        return fixed + (t > chain ? t : chain) + mbytes * mb;
    }
};

// dK / dV: whole groups of heads write their sums once; runs of heads clear dk and dv first and add with atomics.
struct DkdvFit {
    LaunchFit launch;
    double atomic_mb, clear;       // per MB of atomics; the clearing launch
};

// dK / dV and dQ workgroups of one width in one launch, dK / dV first: whole rounds of all units shared out, or the longest one.
struct JointFit {
    double fixed;
    double kv_unit, kv_step, q_unit, q_step;     // per unit, and per step of its chain
    double shared_out, tail;   // of the work over 256 CUs when there are more units than those, and of a dQ unit behind it
    double idle;               // what a unit takes beside idle CUs, of that in a full round
    double mb, atomic_mb, clear;
    double us(const Units& kv, const Units& q, double mbytes) const
    {
        const long long n = kv.n + q.n;
        if (n <= 0) return fixed;
        const double kv_sum = (double)kv.n * kv_unit + kv.sum * kv_step, q_sum = (double)q.n * q_unit + q.sum * q_step;
        const double kv_longest = kv.n > 0 ? kv_unit + kv.longest * kv_step : 0.0, q_longest = q.n > 0 ? q_unit + q.longest * q_step : 0.0;
        const double busy = n < 256 ? (double)n / 256.0 : 1.0;
        double t = (kv_longest > q_longest ? kv_longest : q_longest) * (idle + (1.0 - idle) * busy * busy);
        if (n > 256) {
            const double all = shared_out * (kv_sum + q_sum) / 256.0 + (q.n > 0 ? tail * q_sum / (double)q.n : 0.0);
            t = all > t ? all : t;
        }
        return fixed + t + mb * mbytes;
    }
};

// Fitted to 33000 calls (half of them ring steps of zigzag, even and uneven shards, half with rows and keys drawn from 64 to 12000 over
// their logarithm, 1 to 64 heads, groups of 1 to 8, chunks visible wholly, partly or diagonally), every shape measured for each: 4 to
// 9 % rms off.  First index: head_dim 64, 128; second: 256, 64, 32 rows, or 128, 64, 32 keys; of JOINT: 64, 32.
namespace hexi_shapes {
constexpr LaunchFit FWD[2][3] = {{{5.28, 5.11, 1.15, 1.11, 0.195}, {7.16, 0.429, 0.63, 0.527, 0.286}, {5.7, 0.412, 0.719, 0.661, 0.333}},
                                        {{6.79, 7.91, 1.4, 1.57, 0.222}, {5.99, 3.25, 0.846, 0.956, 0.229}, {4.59, 2.13, 1.08, 1.27, 0.226}}};
constexpr LaunchFit DQ[2][3] = {{{5.54, 5.64, 1.54, 1.45, 0.113}, {5.01, 1.97, 0.768, 0.789, 0.165}, {4.11, 1.67, 0.744, 0.876, 0.119}},
                                        {{7.91, 9.65, 1.78, 2.06, 0.149}, {6.19, 2.32, 1.11, 1.26, 0.137}, {4.62, 1.88, 1.18, 1.47, 0.131}}};
constexpr DkdvFit DKDV[2][3] = {{{{3.28, 6.13, 1.31, 1.24, 0.168}, 0.469, 1.56}, {{2.41, 5.48, 1.3, 1.11, 0.0366}, 0.286, 3.21}, {{4.06, 2.2, 1.3, 1.28, 0.188}, 0.321, 2.48}},
                                        {{{3.44, 10.8, 1.49, 1.72, 0.151}, 0.468, 1.85}, {{2.56, 8, 1.72, 1.91, 0.0383}, 0.325, 4.42}, {{4.65, 3.35, 1.74, 2.07, 0.156}, 0.406, 2.67}}};
constexpr JointFit JOINT[2][2] = {{{2.64, 5.28, 1.29, 3.53, 0.826, 0.81, 0.776, 0.982, 0.0758, 0.266, 3.14}, {3.87, 2.34, 1.26, 1.64, 0.831, 0.98, 0.726, 0.998, 0.112, 0.206, 2.58}},
                                        {{2.63, 7.95, 1.74, 3.7, 1.26, 0.963, 0.652, 0.976, 0.0532, 0.284, 4.54}, {4.34, 3.89, 1.74, 2, 1.4, 1.11, 0.557, 0.953, 0.0673, 0.259, 2.89}}};
}  // namespace hexi_shapes

// The units of a q-stationary launch (forward, dQ) in workgroups of 256, 64 and 32 rows.  false: too large for the split kernels
// (four rounds of full-size units: their tail no longer matters).
inline bool hexi_q_units(const AttnGeom& g, Units (&u)[3])
{
    using namespace hexi_shapes;
    const int n_q_tiles = (g.lq + Q_TILE - 1) / Q_TILE;
    if (n_q_tiles > 4096) return false;
    for (int t = 0; t < n_q_tiles; ++t) {
        const int rows = t == n_q_tiles - 1 ? g.lq - t * Q_TILE : Q_TILE;
        const int seen = seg_rows_le(g.ks, seg_pos_of_row(g.qs, t * Q_TILE + rows - 1));
        if (seen == 0) continue;
        const int nt = (seen + KV_STREAM_TILE - 1) / KV_STREAM_TILE;
        u[0].add(nt, g.nq);
        u[1].add((nt + 1) / 2, (long long)g.nq * ((rows + 63) / 64));
        u[2].add((nt + 3) / 4, (long long)g.nq * ((rows + 31) / 32));
    }
    return u[0].n < 1024;
}

// Which tiles of a forward step are given to 256-row workgroups where it is shared between these and 64-row ones in a second launch: as many as
// fill whole rounds of 256 units; the rest of the rows has to fit one round of 64-row workgroups.  All of them: not to be shared.  A nearly
// empty last round costs as much as a whole one, a round of 64-row workgroups a quarter of that and a launch.  Units have to be of about
// the same length: unequal ones fill each other's last round already.  us: the expected time.
inline QShare hexi_fwd_share(const AttnGeom& g, const Units (&u)[3], double* us)
{
    using namespace hexi_shapes;
    const int n_q_tiles = (g.lq + Q_TILE - 1) / Q_TILE;
    const QShare all = {n_q_tiles, 0};
    if (g.d != 128) return all;            // head_dim 64: 64-row workgroups alone are the better choice wherever sharing would be one
    if (u[0].n != (long long)g.nq * n_q_tiles || u[0].longest * (double)u[0].n > 1.1 * u[0].sum) return all;
    const double mb = (double)g.lq * g.nq * g.d * 6.0 * 1e-6;      // q read, o written
    const int n = (int)u[0].n, big = n / 256 * 256, small = n - big;
    if (small == 0 || 4 * small > 256 || big / g.nq == 0) return all;
    const double mean = u[0].sum / n, part = (double)big / n;
    Units first, rest;
    first.add(mean, big);
    rest.add(ceil(mean / 2.0), 4LL * small);
    *us = FWD[1][0].us(first, mb * part) + FWD[1][1].us(rest, mb * (1.0 - part));
    return {big / g.nq, big % g.nq};
}

// Rows per forward workgroup of the smaller kernels (32 or 64), or 0 for the 256-row kernel, which is kept unless another is expected
// to be 8 % faster: of 8000 of the calls 3 are then slower than in 256-row workgroups by more than 3 %, at most 8 % (14 by more than 10 % at
// a margin of 5 %), and the choice is 0.8 % slower than the best of the three in the mean.  32-row workgroups beyond three rounds stream
// too much.  Measured, us in 256 / 64 / 32 rows, head_dim 128: 300 rows x 700 keys x 4 heads 28.3 / 13.1 / 9.3; 512 x 1024 x 24 34.1 / 15.7 / 19.7;
// 1024 x 1024 x 24 37.9 / 28.4 / 28.9; 2048 x 2048 x 24 64.7 / 69.8 / 88.5; head_dim 64: 2048 x 4096 x 24 80.7 / 68.7 / 82.0.
// share: the 256-row workgroups' part of a step for which 0 is returned.  It is shared with 64-row ones where that is expected to be 10 % faster,
// more than the estimates are off.  Whole passes of four visible steps, merged inside or by a launch of their own, us in one kernel / shared, units left
// over a round: 5612 x 24 heads 2172 / 1891 (16), 11725 x 12 4193 / 3635 (40), 6128 x 24 2254 / 2001 (64), 4862 x 16 1019 / 912 (48), 4184 x 16 917 / 912 (16),
// 5714 x 12 1187 / 1193 (20, the least of ten).  Left out: more than a round of 64-row workgroups, 5705 x 16 1425 / 1486 (112), 7769 x 12 1858 / 1956
// (116), eight steps of 4096 x 24 1144 / 1169 (128), though 7321 x 12 1652 / 1555 (92).
inline int hexi_fwd_split_rows(const AttnGeom& g, QShare* share)
{
    using namespace hexi_shapes;
    constexpr double SHARE_MARGIN = 1.1;
    Units u[3];
    *share = {(g.lq + Q_TILE - 1) / Q_TILE, 0};
    if (!hexi_q_units(g, u)) return 0;
    const auto& fit = FWD[g.d == 128];
    const double mb = (double)g.lq * g.nq * g.d * 6.0 * 1e-6;      // q read, o written
    const double t256 = fit[0].us(u[0], mb), t64 = fit[1].us(u[1], mb), t32 = u[2].n <= 768 ? fit[2].us(u[2], mb) : INFINITY;
    const double small = t64 < t32 ? t64 : t32;
    const bool large = t256 <= 1.08 * small;
    double shared = INFINITY;
    const QShare part = hexi_fwd_share(g, u, &shared);
    if ((large ? t256 : small) > SHARE_MARGIN * shared) { *share = part; return 0; }
    return large ? 0 : (t64 <= t32 ? 64 : 32);
}

// How a backward step is launched.
struct BwdPlan {
    int dq_rows = 0;              // rows per dQ workgroup of the split kernel; 0: the 256-row workgroups
    bool split_keys = false;      // dK / dV in workgroups of `keys` instead of the 128-key ones
    int keys = 32;                // 64 or 32; dQ workgroups of as many rows share the launch
    int run_len = 0;              // q heads per dK / dV workgroup
    int run_len_128 = 0;          // the same if the 128-key workgroups are taken
    int group = 0;                // q heads of the largest group
    double whole_cost = 1.0;      // expected time of the step with whole groups in workgroups of the same width, over that of the plan
    // Whether runs of len heads leave every element of dk and dv with the same bits whatever order they come in: one run of the whole
    // group, or two that add into a cleared element (0 + a + b = 0 + b + a).
    bool fixed_order(int len) const { return 2 * len >= group; }
    bool small = false;           // not large enough for the 128-key workgroups as a matter of course
    bool unused = false;          // some kv head is read by no local q head: zero gradient
    int n_kv_tiles = 0;           // 128-key tiles of the chunk
    int n_known = 0;              // entries of seen
    float seen[4096];             // 64-row q tiles of one head that a key tile sees
};

// The units of a dK / dV launch in workgroups of `keys` (128, 64, 32) over runs of len heads, n_runs of them.
inline Units hexi_kv_units(const AttnGeom& g, const BwdPlan& plan, int keys, int len, long long n_runs)
{
    using namespace hexi_shapes;
    Units u;
    for (int t = 0; t < plan.n_known; ++t) {
        if (plan.seen[t] < 1.0f) continue;
        const int cols = t == plan.n_kv_tiles - 1 ? g.lc - t * KV_TILE : KV_TILE;
        const double tiles = (double)len * plan.seen[t];
        u.add(keys == KV_TILE ? tiles : ceil(tiles * (keys == 64 ? 0.5 : 0.25)), n_runs * ((cols + keys - 1) / keys));
    }
    return u;
}

// The shapes of a whole step.  forced_run_len: hexi_set_dkdv_run_len().
inline void hexi_plan_bwd_step(const AttnGeom& g, int forced_run_len, BwdPlan* plan)
{
    using namespace hexi_shapes;
    const bool wide = g.d == 128;
    // dQ by itself: rows per workgroup, 0 for 256
    Units q[3];
    int& dq_rows = plan->dq_rows;
    const bool dq_small = hexi_q_units(g, q);
    const double q_mb = (double)g.lq * g.nq * g.d * 12.0 * 1e-6;       // q and dO read, dq read and written
    double dq_us = 0.0, dq_256_us = 0.0;
    if (dq_small) {
        dq_us = dq_256_us = DQ[wide][0].us(q[0], q_mb);
        for (int w = 1; w < 3; ++w) {
            const double t = SMALL_MARGIN * DQ[wide][w].us(q[w], q_mb);
            if (t < dq_us) { dq_us = t; dq_rows = w == 1 ? 64 : 32; }
        }
    }
    const int n_kv_tiles = (g.lc + KV_TILE - 1) / KV_TILE;
    plan->n_kv_tiles = n_kv_tiles;
    // q heads per kv head, in head order
    int cnt[HEXI_MAX_HEADS] = {0};
    int max_cnt = 0;
    bool& unused = plan->unused;
    for (int h = 0; h < g.nq; ++h) {
        const int c = ++cnt[g.kv_of_q[h]];
        max_cnt = c > max_cnt ? c : max_cnt;
    }
    plan->group = max_cnt;
    for (int kh = 0; kh < g.nkv; ++kh) unused |= (cnt[kh] == 0);   // a kv head no local q head reads: zero gradient
    // Run length: the longest divisor of the largest group's size (so that its runs are equally long) for which
    // the launch still has about three workgroups per CU and a workgroup walks at most 512 q tiles.  A run
    // amortises the workgroup's prologue and epilogue (about 20 tiles' worth) and, when it covers the whole
    // group, needs no atomics; but the workgroups of an XCD stream the same Q / dO tiles only while they stay
    // in step, and long tile sequences let them drift apart (measured: more L2 misses, slower launches).
    auto n_runs_for = [&](int len) {
        int n = 0;
        for (int kh = 0; kh < g.nkv; ++kh) n += (cnt[kh] + len - 1) / len;
        return n;
    };
    // q tiles that see the chunk's first key: the longest tile sequence of one head
    const int n_qtiles = (g.lq + Q_STREAM_TILE - 1) / Q_STREAM_TILE;
    const int max_tiles = g.lc > 0 ? n_qtiles - seg_rows_le(g.qs, seg_pos_of_row(g.ks, 0) - 1) / Q_STREAM_TILE : 0;
    int& run_len = plan->run_len;
    run_len = max_cnt;
    while (run_len > 1 && (max_cnt % run_len != 0 || (long long)run_len * max_tiles > 512 ||
                           (long long)n_runs_for(run_len) * n_kv_tiles < 3 * 256))
        --run_len;
    if (forced_run_len >= 1)      // tuning / test override of the heuristic
        run_len = forced_run_len < max_cnt ? forced_run_len : max_cnt;
    plan->run_len_128 = run_len;
    // cost of a unit: the q tiles its key tile sees, once per head of the run, plus the prologue and epilogue
    // (about 20 tiles' worth)
    float (&seen)[4096] = plan->seen;
    const int n_known = n_kv_tiles < 4096 ? n_kv_tiles : 4096;     // (longer chunks: the remaining tiles count like the last known one)
    plan->n_known = n_known;
    for (int t = 0; t < n_known; ++t) {
        const int k_min = seg_pos_of_row(g.ks, t * KV_TILE);
        const int before = seg_rows_le(g.qs, k_min - 1);
        seen[t] = before < g.lq ? (float)(n_qtiles - before / Q_STREAM_TILE) : 0.0f;
    }
    // Of 7350 of the calls none is then slower than 128-key and 256-row launches by more than 3 %, and the choice (but for the order of
    // sums, below) is 0.8 % slower than the best of all shapes in the mean.  Measured, both halves, head_dim 128, us in 128 keys and 256 rows / 64 and 64 / 32 and 32:
    // 300 rows x 700 keys x 4 / 2 heads 58 / 19.1 / 12.4; 512 x 1024 x 24 / 8 95 / 35 / 40.6; 2048 x 2048 x 24 / 8 242 / 178 / 212; 4096 x
    // 4096 x 12 / 3 394 / 336 / 402; 8192 x 8192 x 24 / 8 2367 / 2594 / 3060; head_dim 64: 4096 x 4096 x 24 / 8 468 / 384 / 459.
    // Launches that do not fill the chip take workgroups of 64 or 32 keys instead (whole groups where the 128-key ones take whole
    // groups: no atomics that these would not have), in one launch with dQ workgroups of as many rows: the two kinds of unit fill
    // each other's last rounds.  Where the chip is full the 128-key workgroups stream a quarter as much per key.  A forced run length
    // keeps the 128-key workgroups that it is defined for.
    // A fixed order of the sums is given up only where that is expected to be 15 % faster (an estimate is 4 to 9 % rms off).  Measured, of 100
    // steps of a smaller expected gain: the order costs 9 % in the mean, between 27 % less and 26 % more; of 50 between 15 and 20 %: 16 %.
    if (forced_run_len >= 1 || n_kv_tiles > 4096) return;
    const Units kv_128 = hexi_kv_units(g, *plan, KV_TILE, run_len, n_runs_for(run_len));
    if (kv_128.n >= 2048) return;
    plan->small = true;
    const double run_mb = (double)g.lc * g.d * 8.0 * 1e-6;      // dk and dv of a run
    auto added = [&](int len, double clear, double atomic_mb) {
        return (len < max_cnt || unused ? clear : 0.0) + (len < max_cnt ? run_mb * n_runs_for(len) * atomic_mb : 0.0);
    };
    const int len_128 = run_len;
    const DkdvFit& k128 = DKDV[wide][0];
    auto margin = [&](int len) { return plan->fixed_order(len) ? 1.0 : ORDER_MARGIN; };
    double best = margin(len_128) * (k128.launch.us(kv_128, run_mb * g.nkv) + added(len_128, k128.clear, k128.atomic_mb) + dq_us);
    for (int w = 1; w < 3; ++w) {
        const int keys = w == 1 ? 64 : 32;
        double whole_us[2];        // beside 256-row dQ workgroups, and in one launch with dQ workgroups of as many rows
        for (int len = max_cnt; len >= 1; --len) {
            if (max_cnt % len != 0 || (len_128 >= max_cnt && len < max_cnt)) continue;
            const Units kv = hexi_kv_units(g, *plan, keys, len, n_runs_for(len));
            auto consider = [&](double us, int rows) {
                const double t = SMALL_MARGIN * margin(len) * us;
                if (len == max_cnt) whole_us[rows > 0] = us;
                if (t < best) { best = t; run_len = len; plan->split_keys = true; plan->keys = keys; dq_rows = rows; plan->whole_cost = whole_us[rows > 0] / us; }
            };
            const JointFit& j = JOINT[wide][w - 1];
            if (dq_small) consider(j.us(kv, q[w], run_mb * g.nkv + q_mb) + added(len, j.clear, j.atomic_mb), keys);
            const DkdvFit& k = DKDV[wide][w];
            consider(k.launch.us(kv, run_mb * g.nkv) + added(len, k.clear, k.atomic_mb) + dq_256_us, 0);
        }
    }
}

// The shapes of a call for both halves or for one of them.  One by itself keeps the step's shape (and so the bits that it gives with the other)
// unless another is expected to be faster: what a joint launch gains for the step by filling last rounds, and what it chooses for the other half's
// sake, the half alone does not have.  Margins: dQ 15 %, also for the 256-row workgroups where the step has others; dK / dV, whose bits depend on
// more than the width, 3 %, fixed orders of sums counting as in the step.  Of 9828 random calls for dQ alone 2.6 % are then slower than with the kernels
// before by more than 10 %, of 13400 for dK / dV alone 0.9 % (6.5 and 8.5 % where a half took the step's shape or the large workgroups and nothing
// else), and they take 0.81 and 0.92 of the time in the mean (0.84 and 0.97).  us in 256 / 64 / 32 rows, dQ alone: 8245 x 74 keys x 2 heads
// x 64 21.9 / 11.4 / 11.1, 582 x 9338 x 8 x 128 236 / 65.9 / 39.0; dK / dV alone in 128 / 64 / 32 keys, the best run lengths: 3078 x 283 x 16 / 4 x 64
// 75.7 / 44.2 / 25.4, 1016 x 390 x 64 / 8 x 64 36.2 / 31.4 / 29.5.
// accumulate: two runs that add to what dk and dv hold have no fixed order, so whole groups are taken instead, in workgroups of the same width,
// where these are expected to be at most 15 % slower.
inline void hexi_plan_bwd(const AttnGeom& g, int forced_run_len, bool want_dq, bool want_dkdv, bool accumulate, BwdPlan* plan)
{
    using namespace hexi_shapes;
    constexpr double MARGIN = 1.15;
    hexi_plan_bwd_step(g, forced_run_len, plan);
    const bool wide = g.d == 128;
    Units u[3];
    if (!want_dkdv && hexi_q_units(g, u)) {
        const double mb = (double)g.lq * g.nq * g.d * 12.0 * 1e-6;      // q and dO read, dq read and written
        const double us[3] = {DQ[wide][0].us(u[0], mb), DQ[wide][1].us(u[1], mb), DQ[wide][2].us(u[2], mb)};
        const double small_us = us[1] < us[2] ? us[1] : us[2];
        if (us[0] <= MARGIN * small_us) plan->dq_rows = 0;
        else if (plan->dq_rows == 0 || us[plan->dq_rows == 64 ? 1 : 2] > MARGIN * small_us) plan->dq_rows = us[1] <= us[2] ? 64 : 32;
    }
    if (!want_dkdv || forced_run_len >= 1 || plan->n_kv_tiles > 4096) return;
    auto estimate = [&](int keys, int len) {
        const DkdvFit& f = DKDV[wide][keys == KV_TILE ? 0 : (keys == 64 ? 1 : 2)];
        HeadRuns runs;
        const bool shared = hexi_build_head_runs(g.kv_of_q, g.nq, g.nkv, len, &runs);
        const double run_mb = (double)g.lc * g.d * 8.0 * 1e-6;      // dk and dv of a run
        return f.launch.us(hexi_kv_units(g, *plan, keys, len, runs.n), run_mb * g.nkv) + (shared || plan->unused ? f.clear : 0.0) +
               (shared ? run_mb * runs.n * f.atomic_mb : 0.0);
    };
    double whole_cost = plan->whole_cost;
    if (!want_dq && plan->small) {
        auto priced = [&](int keys, int len) { return (plan->fixed_order(len) ? 1.0 : ORDER_MARGIN) * estimate(keys, len); };
        const double step_us = priced(plan->split_keys ? plan->keys : KV_TILE, plan->run_len);
        double best = priced(KV_TILE, plan->run_len_128);
        int best_keys = KV_TILE, best_len = plan->run_len_128;
        for (int keys = 64; keys >= 32; keys /= 2)
            for (int len = plan->group; len >= 1; --len) {
                if (plan->group % len != 0 || (plan->run_len_128 >= plan->group && len < plan->group)) continue;
                const double t = priced(keys, len);
                if (t < best) { best = t; best_keys = keys; best_len = len; }
            }
        if (step_us > SMALL_MARGIN * best) {
            plan->split_keys = best_keys != KV_TILE;
            plan->keys = plan->split_keys ? best_keys : 32;
            plan->run_len = best_len;
        }
        if (plan->split_keys) whole_cost = estimate(plan->keys, plan->group) / estimate(plan->keys, plan->run_len);
    }
    if (accumulate && plan->split_keys && plan->fixed_order(plan->run_len) && whole_cost <= ORDER_MARGIN) plan->run_len = plan->group;
}

// The fp32 kernels on the fp32 instruction (hexi_f32_units.h): 64-row workgroups that share their tiles, or 16-row ones whose wavefronts split the streamed
// rows, one or (head_dim 64) two of them on a CU.
enum class F32Shape { SHARED, SPLIT, SPLIT_TWO };

// Shared or split at head_dim 128: the shorter makespan on 256 CUs when all workgroups are equally long (shared: two share a
// CU; split: one takes all of it), the split one being a little slower per row (measured on a launch that fills the chip
// either way, 4096 x 4096 x 16 heads x 128: forward 109 against 120 TFLOP/s, dQ 130 / 132, dK/dV 125 / 132).
inline bool hexi_f32_split(int n_rows, int n_heads)
{
    const long long shared = (long long)((n_rows + 63) / 64) * n_heads, split = (long long)((n_rows + 15) / 16) * n_heads;
    return 0.25 * (double)((split + 255) / 256) < 0.93 * (double)((shared + 255) / 256);
}

// Keys that a row sees, averaged over 32 rows spread over the shard: the rules below weigh launches, they need no exact count.
inline double hexi_mean_seen(const AttnGeom& g)
{
    long long seen = 0;
    for (int i = 0; i < 32; ++i) seen += seg_rows_le(g.ks, seg_pos_of_row(g.qs, (int)((2 * i + 1) * (long long)g.lq / 64)));
    return (double)seen / 32.0;
}

// Two workgroups on a CU finish more units in a given time (5/6 of the time per unit, measured), but each of them takes longer.
// So they are taken where the sum of the units, dealt evenly to the CUs, is longer (by 2 %) than the longest unit, which is what the launch waits
// for otherwise.  us with one / two a CU, and that quotient: backward of 1024 x 1024 keys x 8/2 heads 92 / 96 (0.88), 1500 x 1500 x 8/2
// 175 / 163 (1.28), 300 x 600 x 16/4 48 / 43 (1.04); diagonal 2048 x 8/2 174 / 187 (0.88), 768 x 8/8 42 / 38 (1.31); forward, diagonal,
// 4096 x 2 heads 55 / 62 (1.0), 1500 x 6 heads 32 / 28 (1.1).
inline F32Shape hexi_f32_split_shape(double sum, double longest) { return sum > 262.0 * longest ? F32Shape::SPLIT_TWO : F32Shape::SPLIT; }

// head_dim 64: us of a launch whose units are about equally long (x 1000 streamed rows), besides the launch itself.  Shared: in rounds of
// 256 workgroups, the first of them 14.5 us longer per 1000 rows of the longest unit; split, two a CU: in rounds of 512, a part of one costs half of the
// rest of it, and 4.5 us of each are start and combination.  Within 10 % of the measured forward, dK/dV and (x 1.35) dQ
// for 70 to 4096 streamed rows and 1/4 to 6 shared rounds.  us forward, shared / split / two a CU: 2048 x 70 keys x 16 heads
// 15 / 42 / 28, x 300 31 / 60 / 41, x 1000 85 / 123 / 92, x 2048 160 / 203 / 163; 1500 x 1500 x 24 168 / 181 / 143, 3000 x 3000 x 24 537 / 623 / 511,
// 4096 x 4096 x 24 859 / 1106 / 902; 6703 x 4962 x 16, mean 0.63 of the longest, 747 shared, 818 split.  Units less equal than that
// fill each other's last rounds: split (diagonal 4096 x 24 heads 512 / 602 / 481, 300 x 24 heads 20 / 13 / 11).
inline bool hexi_f32_shared_64(int n_rows, int n_heads, double mean, double longest, double margin, double start = 0.0)
{
    if (mean + start <= 0.6 * (longest + start)) return false;
    const long long shared = (long long)((n_rows + 63) / 64) * n_heads, split = (long long)((n_rows + 15) / 16) * n_heads;
    const double x = mean * 1e-3, r = (double)((shared + 255) / 256), s = 0.5 * ((double)((split + 511) / 512) + (double)split / 512.0);
    return margin * (3.0 * r + 14.5e-3 * longest + 31.5 * r * x) < s * (4.5 + 17.7 * x);
}

inline F32Shape hexi_f32_fwd_shape(const AttnGeom& g)
{
    if (g.d != 64) return hexi_f32_split(g.lq, g.nq) ? F32Shape::SPLIT : F32Shape::SHARED;
    const double mean = hexi_mean_seen(g), longest = (double)seg_rows_le(g.ks, seg_pos_of_row(g.qs, g.lq - 1));
    if (hexi_f32_shared_64(g.lq, g.nq, mean, longest, 0.97)) return F32Shape::SHARED;
    return hexi_f32_split_shape((double)((g.lq + 15) / 16) * g.nq * mean, longest);
}

// Backward.  Two split halves, or two shared ones, are one launch and fill each other's rounds.  At head_dim 64 dK/dV is shared where that is
// expected to be 5 % faster (70 rows x 2740 keys x 12/12 heads: 33 us, with dQ 76, against 60 and 90 as one split launch), dQ where 20 %,
// which a launch of its own besides dK/dV's has to gain: 2048 rows x 70 keys x 16/4 heads 21 us / 33 split, with dK/dV 186 / 171 as one
// launch; 2048 x 512 x 16/4 61 / 67, 207 / 176; 3500 x 512 x 16/4 110 / 112, 349 / 288.  As one launch, shared / split / split, two a CU:
// 4096 x 4096 x 24/8 2781 / 3302 / 2769, 2048 x 2048 x 8/8 254 / 302 / 245, diagonal 249 / 179 / 146.
// dQ is also split where it fits on the CUs that few long dK/dV units leave idle: 1662 x 141 x 24/3 heads 277 us, dK/dV alone 275; a call
// for dQ alone has no such units beside it and may be shared where the step's is split.  A dQ unit has three products per
// block of scores, a dK/dV unit four, and walks the rows of every q head that reads its keys.
// Keys that no row sees are units too, of a start and an end: where there are such keys these count like 500 rows in the comparison of unit lengths
// and in the sum (fitted to 3400 calls; 400 and 800 give the same choices but for a few), and dQ units of up to 400 keys join shared dK/dV ones
// in their launch: 209 rows x 2390 keys x 4/4 heads, the first 209 seen, 26 us, 35 as two launches.  us shared / split / two a CU, dK/dV alone: 117 x 4743 keys x 16/16
// heads, the first 117 keys seen, 32 / 174 / 114; 53 x 3065 x 64/16, 1608 seen, 64 / 261 / 162.
inline void hexi_f32_bwd_shapes(const AttnGeom& g, bool want_dq, bool want_dkdv, F32Shape* kv, F32Shape* q)
{
    if (g.d != 64) {
        *kv = hexi_f32_split(g.lc, g.nkv) ? F32Shape::SPLIT : F32Shape::SHARED;
        *q = hexi_f32_split(g.lq, g.nq) ? F32Shape::SPLIT : F32Shape::SHARED;
        return;
    }
    const double group = (double)g.nq / g.nkv, seen = hexi_mean_seen(g);
    const double q_longest = (double)seg_rows_le(g.ks, seg_pos_of_row(g.qs, g.lq - 1));
    const double kv_longest = g.lc > 0 ? group * (double)(g.lq - seg_rows_le(g.qs, seg_pos_of_row(g.ks, 0) - 1)) : 0.0;
    const double kv_mean = g.lc > 0 ? group * (double)g.lq * seen / (double)g.lc : 0.0;
    const double start = q_longest < (double)g.lc ? 500.0 : 0.0;
    const bool kv_shared = hexi_f32_shared_64(g.lc, g.nkv, kv_mean, kv_longest, 1.05, start);
    const double pairs = (double)g.nq * g.lq / 16.0 * seen, starts = (double)((g.lc + 15) / 16) * g.nkv * start;
    const bool beside_dkdv = want_dkdv && !kv_shared && hexi_f32_split_shape(7.0 * pairs + 4.0 * starts, 4.0 * (kv_longest + start)) == F32Shape::SPLIT;
    const bool beside_shared = want_dq && want_dkdv && kv_shared && start > 0.0 && q_longest <= 400.0;
    const bool q_shared = beside_shared || (!beside_dkdv && hexi_f32_shared_64(g.lq, g.nq, seen, q_longest, 1.2));
    const bool split_dq = want_dq && !q_shared, split_dkdv = want_dkdv && !kv_shared;
    double longest = split_dq ? 3.0 * q_longest : 0.0;
    if (split_dkdv && 4.0 * (kv_longest + start) > longest) longest = 4.0 * (kv_longest + start);
    const F32Shape split = hexi_f32_split_shape(pairs * ((split_dq ? 3.0 : 0.0) + (split_dkdv ? 4.0 : 0.0)) + (split_dkdv ? 4.0 * starts : 0.0), longest);
    *kv = kv_shared ? F32Shape::SHARED : split;
    *q = q_shared ? F32Shape::SHARED : split;
}

// Split-operand fp32 kernels (hexi_f32_bf16x3.hip), 32 or 64 stationary rows to a workgroup, one workgroup on a CU: taken where they are expected to
// be 5 % faster than the kernels above.  Their matrix work takes under half of the time, but their units are two and four times as long as
// the 16-row ones, so a launch with few units is better off with those.  us: a launch, a unit, and 1000 streamed rows of its chain,
// fitted to 300 random calls of 60 to 7000 rows and keys and 1 to 32 heads (90 % of them within 12 %; the 16-row fit stands for all shapes of
// those kernels, 90 % within 25 %).  Over 320 other random calls, geometric mean of the time before / after at head_dim 128: forward 1.19, whole
// backward 1.11, under HEXI_ACCUMULATE 1.05; at 64, where few take them, 1.04, 1.02, 1.02.  us before / after, all keys visible: 4096 x 4096 x 16/4
// heads x 128 forward 1139 / 759, backward 3634 / 3049; 3056 x 3000 x 6/2 x 128 295 / 215, 865 / 740; the other way round
// 100 x 4000 x 8/2 x 128 forward 79 / 100, dQ 107 / 149, 777 x 1000 x 8/2 x 128 dK / dV with heads in one run 118 / 170.
struct F32Fit { double launch, unit, per_k; };
struct F32x3Fwd { bool use = false; int n64 = 0; };                                     // the last n64 64-row tiles (of all heads) as such, the others as two units
struct F32x3Bwd { bool use = false; int key_blocks = 1, runs = 1; bool rows64 = false; }; // keys of a dK / dV unit / 32, parts of a head group, dQ units of 64 rows

inline double hexi_f32_launch_us(const F32Fit& f, long long n, double mean, double longest, double tail = 0.5)
{
    const double rounds = (double)((n + 255) / 256);
    double chain = longest;
    if (n > 256) chain = mean >= 0.9 * longest ? rounds * mean : std::fmax(longest, mean * (double)n / 256.0 + tail * longest);
    return f.launch + f.unit * rounds + 1e-3 * f.per_k * chain;
}

inline F32x3Fwd hexi_f32x3_fwd_by_itself(const AttnGeom& g)
{
    const bool wide = g.d == 128;
    const F32Fit r16 = wide ? F32Fit{6.6, 1.5, 19.3} : F32Fit{6.4, 0.5, 9.9}, r32 = wide ? F32Fit{2.0, 7.2, 23.6} : F32Fit{2.8, 4.7, 14.6},
                 r64 = wide ? F32Fit{0.5, 11.2, 35.2} : F32Fit{2.4, 6.9, 20.2};
    const double mean = hexi_mean_seen(g), longest = (double)hexi_keys_seen(g);
    auto units = [&](int rows) { return (long long)((g.lq + rows - 1) / rows) * g.nq; };
    const long long tiles = units(64), rest = tiles % 256;
    const double us32 = hexi_f32_launch_us(r32, units(32), mean, longest), us64 = hexi_f32_launch_us(r64, tiles, mean, longest);
    F32x3Fwd plan;
    double us = us32;
    if (us64 < us) { us = us64; plan.n64 = (int)tiles; }
    if (tiles > 256 && rest > 0 && rest <= 128 && mean >= 0.9 * longest) {      // whole rounds of 64-row units, a last one of 32-row units
        const double mixed = hexi_f32_launch_us(r64, tiles - rest, mean, longest) + r32.unit + 1e-3 * r32.per_k * mean;
        if (mixed < us) { us = mixed; plan.n64 = (int)(tiles - rest); }
    }
    plan.use = 1.05 * us + 2.0 < hexi_f32_launch_us(r16, units(16), mean, longest, 0.2);
    return plan;
}

// A step's halves are one launch whose units fill each other's rounds.
// A few long dK / dV units are what such a launch waits for: the heads of a group may be dealt to two of them, which add to cleared elements (not
// where dk and dv hold a running value, whose sum would show the order: the margin is wider there, 1.1 lost up to 9 % in some of the calls).
// 128 columns, one run / two: 6000 x 800 x 8/1 heads 1888 / 1294 us, 3056 x 3000 x 6/2 703 / 701, 2048 x 2048 x 16/4 737 / 743; 16-row kernels / two
// runs: 1500 x 2500 x 8/2 492 / 403, 777 x 1000 x 8/2 126 / 113.
inline F32x3Bwd hexi_f32x3_bwd_by_itself(const AttnGeom& g, bool accumulate, bool whole_groups = false)
{
    struct Part { long long n; double mean, longest; F32Fit f; };
    const bool wide = g.d == 128;
    const double group = (double)g.nq / g.nkv, q_mean = hexi_mean_seen(g), q_longest = (double)hexi_keys_seen(g);
    const double kv_longest = group * (double)(g.lq - seg_rows_le(g.qs, seg_pos_of_row(g.ks, 0) - 1)), kv_mean = group * (double)g.lq * q_mean / (double)g.lc;
    auto q_part = [&](int rows, F32Fit f) { return Part{(long long)((g.lq + rows - 1) / rows) * g.nq, q_mean, q_longest, f}; };
    auto kv_part = [&](int keys, F32Fit f) { return Part{(long long)((g.lc + keys - 1) / keys) * g.nkv, kv_mean, kv_longest, f}; };
    const Part q16 = q_part(16, wide ? F32Fit{7.2, 3.0, 25.5} : F32Fit{6.7, 1.0, 12.6}), kv16 = kv_part(16, wide ? F32Fit{7.2, 6.0, 33.5} : F32Fit{6.7, 2.9, 18.2});
    const Part q32 = q_part(32, wide ? F32Fit{3.5, 9.0, 35.3} : F32Fit{3.0, 5.2, 20.3}), q64 = q_part(64, wide ? F32Fit{3.5, 13.0, 55.0} : F32Fit{3.0, 8.2, 30.7});
    auto halves = [&](Part p) {        // two runs: twice the units, of the longer half at most; the clearing launch
        const double longer = std::ceil(0.5 * group) / group;
        return Part{2 * p.n, 0.5 * p.mean, longer * p.longest, F32Fit{p.f.launch + 5.0, p.f.unit, p.f.per_k}};
    };
    const Part kv32 = kv_part(32, wide ? F32Fit{3.5, 8.0, 54.0} : F32Fit{3.0, 6.3, 31.5}), kv64 = kv_part(64, F32Fit{3.0, 11.2, 50.0});
    // (the 16-row kernels' units fill each other's rounds better, two of them on a CU at head_dim 64)
    auto us = [](const Part* kv, const Part* q, double tail) {
        double sum = 0.0, longest = 0.0, launch = 0.0;
        long long n = 0;
        for (const Part* p : {kv, q}) {
            if (!p) continue;
            sum += (double)p->n * (p->f.unit + 1e-3 * p->f.per_k * p->mean);
            longest = std::fmax(longest, p->f.unit + 1e-3 * p->f.per_k * p->longest);
            launch = std::fmax(launch, p->f.launch);
            n += p->n;
        }
        return launch + (n <= 256 ? longest : std::fmax(longest, sum / 256.0 + tail * longest));
    };
    // the best units for a number of runs to a group
    struct Choice { double us; int key_blocks; bool rows64; };
    auto best_of = [&](const Part& k32, const Part& k64) {
        Choice best{us(&k32, &q32, 0.35), 1, false};
        if (const double t = us(&k32, &q64, 0.35); t < best.us) best = {t, 1, true};
        if (const double t = wide ? best.us : us(&k64, &q64, 0.35); t < best.us) best = {t, 2, true};
        return best;
    };
    F32x3Bwd plan;
    Choice best = best_of(kv32, kv64);
    if (!accumulate && !whole_groups && group >= 2.0) {
        const Choice two = best_of(halves(kv32), halves(kv64));
        if (1.03 * two.us < best.us) {      // (a fixed cost of atomics that the fits do not hold)
            best = two;
            plan.runs = 2;
        }
    }
    plan.key_blocks = best.key_blocks;
    plan.rows64 = best.rows64;
    plan.use = (!wide ? 1.15 : accumulate ? 1.25 : 1.1) * best.us < us(&kv16, &q16, wide ? 0.1 : 0.0);
    return plan;
}

// At head_dim 64 a step takes them forward and backward or not at all: the score of the 16-row backward is one chain of sums there (four have no
// room in its 128 registers), whose rounding errors cancel in P with those of a forward of the same chain alone.  Measured with the
// split-operand forward before it, K scaled by 3: errors of dq, dk, dv 1.6, 1.5, 1.6 times as large (310 x 1040 x 16/2 heads).
inline bool hexi_f32x3_at_64(const AttnGeom& g)
{
    return hexi_f32x3_fwd_by_itself(g).use && hexi_f32x3_bwd_by_itself(g, false).use && hexi_f32x3_bwd_by_itself(g, true).use;
}
inline F32x3Fwd hexi_f32x3_fwd(const AttnGeom& g)
{
    F32x3Fwd plan = hexi_f32x3_fwd_by_itself(g);
    if (plan.use && g.d != 128) plan.use = hexi_f32x3_at_64(g);
    return plan;
}
// A half of a backward step by itself at head_dim 128: us expected with the 16-row kernels (in the shape hexi_f32_split() says) and with the plan's units.
// Fitted to 260 random halves, 90 % of each kind within 10 % (split dK / dV 20 %).
struct F32Half { double us16, us; };
inline F32Half hexi_f32x3_dq_alone(const AttnGeom& g, const F32x3Bwd& plan)
{
    const double mean = hexi_mean_seen(g), longest = (double)hexi_keys_seen(g);
    auto us = [&](int rows, F32Fit f, double tail) { return hexi_f32_launch_us(f, (long long)((g.lq + rows - 1) / rows) * g.nq, mean, longest, tail); };
    return {hexi_f32_split(g.lq, g.nq) ? us(16, {2.7, 6.9, 25.0}, 0.29) : us(64, {7.7, 7.2, 98.7}, 0.27),
            plan.rows64 ? us(64, {0.0, 16.3, 52.1}, 0.3) : us(32, {1.8, 9.7, 35.9}, 0.37)};
}
inline F32Half hexi_f32x3_dkdv_alone(const AttnGeom& g, const F32x3Bwd& plan)
{
    const double group = (double)g.nq / g.nkv, longer = std::ceil(0.5 * group) / group;
    const int seen = hexi_keys_seen(g);
    const double longest = group * (double)(g.lq - seg_rows_le(g.qs, seg_pos_of_row(g.ks, 0) - 1)), mean = group * (double)g.lq * hexi_mean_seen(g) / seen;
    // unseen: us of a round of units of keys that no row sees
    auto us = [&](int keys, int runs, F32Fit f, double tail, double unseen) {
        const long long n = (long long)((seen + keys - 1) / keys) * g.nkv * runs, all = (long long)((g.lc + keys - 1) / keys) * g.nkv * runs;
        return hexi_f32_launch_us(f, n, mean / runs, runs == 2 ? longer * longest : longest, tail) + unseen * (double)(all - n) / 256.0;
    };
    return {hexi_f32_split(g.lc, g.nkv) ? us(16, 1, {2.3, 14.1, 33.1}, 0.26, 13.0) : us(64, 1, {12.5, 7.6, 139.5}, 0.17, 3.9),
            plan.runs == 2 ? us(32, 2, {0.0, 21.3, 54.9}, 0.24, 4.6) : us(32, 1, {0.1, 19.7, 53.8}, 0.3, 1.9)};
}

// At head_dim 128 a half in a call of its own has rounds to itself, and takes the units of the whole step only where those are expected 5 % faster
// than the 16-row ones by themselves (us, 16-row / the whole step's: dQ of 329 rows x 1509 keys x 24 heads 92 / 126, of 124 x 1387 x 32 46 / 58, dK / dV of
// 93 x 2465 x 24/24 with half of the keys seen 66 / 97).  A whole step wants the sum of its halves not 15 % slower: 135 x 4439 keys x 24/24, four
// blocks of rows to a dK / dV unit, 318 / 496.
// forced_run_len: hexi_set_dkdv_run_len(); there are whole groups and halves of them here, so one that holds a whole group forbids the halves.
inline F32x3Bwd hexi_f32x3_bwd(const AttnGeom& g, bool accumulate, bool want_dq = true, bool want_dkdv = true, int forced_run_len = 0)
{
    int heads[HEXI_MAX_HEADS] = {}, largest = 0;
    for (int h = 0; h < g.nq; ++h) largest = ++heads[(int)g.kv_of_q[h]] > largest ? heads[(int)g.kv_of_q[h]] : largest;
    F32x3Bwd plan = hexi_f32x3_bwd_by_itself(g, accumulate, forced_run_len >= largest);
    if (!plan.use) return plan;
    if (g.d != 128) {
        plan.use = hexi_f32x3_at_64(g);
        return plan;
    }
    const F32Half q = hexi_f32x3_dq_alone(g, plan), kv = hexi_f32x3_dkdv_alone(g, plan);
    plan.use = 0.85 * (q.us + kv.us) < q.us16 + kv.us16;
    if (!want_dkdv) plan.use = plan.use && 1.05 * q.us < q.us16;
    if (!want_dq) plan.use = plan.use && 1.05 * kv.us < kv.us16;
    return plan;
}

// Chains of sums of a score in the 16-row kernels (hexi_f32_units.h): four at head_dim 128 where any part of the step, forward or backward, may take the
// split-operand kernels.
inline int hexi_f32_chains(const AttnGeom& g)
{
    return g.d == 128 && (hexi_f32x3_fwd(g).use || hexi_f32x3_bwd(g, false).use || hexi_f32x3_bwd(g, true).use) ? 4 : 1;
}

// Which workgroup shapes a bf16 ring step is launched with, from its sizes: the rules of the launchers, host code alone.
#pragma once
#include <cmath>
#include "hexi_internal.h"

namespace hexi_shapes {
constexpr int Q_TILE = 256;            // q rows of the large forward and dQ workgroups
constexpr int KV_STREAM_TILE = 64;     // keys per tile that they stream
constexpr int KV_TILE = 128;           // keys of the large dK / dV workgroups
constexpr int Q_STREAM_TILE = 64;      // q rows per tile that they stream
}  // namespace hexi_shapes

// Time of a launch of n units, one per CU at a time, that take `sum` in total and at most `longest` each: whole rounds
// of the mean unit on 256 CUs (the launches start the longest units first), or the longest one.
inline double hexi_makespan(double sum, double longest, long long n)
{
    if (n <= 0) return 0.0;
    const double rounds = sum / (double)n * (double)((n + 255) / 256);
    return rounds > longest ? rounds : longest;
}

// The units of a launch shape: estimated times in us.
struct UnitTimes {
    double sum = 0.0, longest = 0.0;
    long long n = 0;
    void add(double t, long long k) { sum += t * (double)k; n += k; longest = t > longest ? t : longest; }
    double makespan() const { return hexi_makespan(sum, longest, n); }
    // the same for units whose speed depends on how much of the chip is busy: `lo` per unit of `sum` in a round that leaves
    // most CUs idle, `hi` in one that uses three quarters of them or more
    double makespan(double lo, double hi) const
    {
        if (n <= 0) return 0.0;
        const double rest = (double)(n % 256) / 192.0, f = rest < 1.0 ? rest * rest : 1.0;
        const double t = sum / (double)n * ((double)(n / 256) * hi + (rest > 0.0 ? lo + (hi - lo) * f : 0.0));
        return t > longest * lo ? t : longest * lo;
    }
};
// Estimated times of a step's dQ: a launch of 256-row workgroups (us, 0 where nothing is visible), and the units of the split
// kernel's 64- and 32-row ones.
struct DqTimes {
    double t256 = 0.0;
    UnitTimes rows64, rows32;
};

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

// Fitted to 7300 calls (5300 with rows and keys drawn from 64 to 12000 over their logarithm, 1 to 64 heads, groups of 1 to 8, chunks
// visible wholly, partly or diagonally; 2000 ring steps of zigzag, even and uneven shards), every shape measured for each: 4 to
// 9 % rms off, 13 % for the 256-row dQ.  First index: head_dim 64, 128; second: 256, 64, 32 rows, or 128, 32 keys.
namespace hexi_shapes {
constexpr LaunchFit FWD[2][3] = {{{5.21, 3.75, 1.16, 1.13, 0.168}, {5.11, 0.429, 0.800, 0.613, 0.251}, {4.90, 0.669, 0.708, 0.686, 0.300}},
                                 {{5.90, 7.31, 1.42, 1.60, 0.153}, {3.87, 3.25, 1.12, 1.20, 0.159}, {3.64, 3.51, 1.04, 1.29, 0.197}}};
constexpr LaunchFit DQ[2][3] = {{{10.9, 3.05, 1.31, 1.46, 0.168}, {3.20, 2.93, 0.833, 0.861, 0.126}, {3.16, 2.69, 0.727, 0.879, 0.128}},
                                {{11.4, 13.0, 1.51, 2.11, 0.155}, {3.79, 5.09, 1.28, 1.47, 0.0999}, {3.66, 4.18, 1.21, 1.51, 0.127}}};
constexpr DkdvFit DKDV[2][2] = {{{{2.29, 6.21, 1.32, 1.22, 0.166}, 0.485, 1.33}, {{3.36, 2.21, 1.26, 1.31, 0.166}, 0.288, 2.18}},
                                {{{3.16, 10.2, 1.50, 1.72, 0.150}, 0.489, 1.46}, {{3.28, 3.83, 1.75, 2.12, 0.123}, 0.347, 2.67}}};
}  // namespace hexi_shapes

// The units of a q-stationary launch (forward, dQ) in workgroups of 256, 64 and 32 rows.  false: too large for the split kernels
// (four rounds of full-size units: their tail no longer matters).
inline bool hexi_q_units(const AttnGeom& g, Units (&u)[3])
{
    using namespace hexi_shapes;
    const int n_q_tiles = (g.lq + Q_TILE - 1) / Q_TILE;
    if ((long long)g.nq * n_q_tiles >= 1024 || n_q_tiles > 4096) return false;
    for (int t = 0; t < n_q_tiles; ++t) {
        const int rows = t == n_q_tiles - 1 ? g.lq - t * Q_TILE : Q_TILE;
        const int seen = seg_rows_le(g.ks, seg_pos_of_row(g.qs, t * Q_TILE + rows - 1));
        if (seen == 0) continue;
        const int nt = (seen + KV_STREAM_TILE - 1) / KV_STREAM_TILE;
        u[0].add(nt, g.nq);
        u[1].add((nt + 1) / 2, (long long)g.nq * ((rows + 63) / 64));
        u[2].add((nt + 3) / 4, (long long)g.nq * ((rows + 31) / 32));
    }
    return true;
}

// Rows per forward workgroup of the split kernel (32 or 64), or 0 for the 256-row kernel, which is kept unless the other is expected
// to be 5 % faster (of the 7300 calls 5 are then slower than in 256-row workgroups by more than 3 %, at most 10 %; an estimate
// without the rows' own reads and writes left 116 so, at most 24 %).  32-row workgroups beyond three rounds stream too much: 666
// rows x 6831 keys x 48 heads x 128: 150 / 212 / 243 us in 256 / 64 / 32 rows.  Others, head_dim 128: 300 x 700 x 4 heads
// 27.5 / 12.3 / 9.7; 512 x 1024 x 24 32.0 / 16.3 / 20.8; 1024 x 1024 x 24 35 / 30.6 / 31.6; 2048 x 2048 x 24 69 / 78 / 99;
// 1091 x 118 x 32 19.4 / 23.0 / 30.5; head_dim 64: 1024 x 1024 x 24 24.2 / 16.8 / 16.9; 6523 x 181 x 8 15.3 / 17.7 / 22.5.
inline int hexi_fwd_split_rows(const AttnGeom& g)
{
    using namespace hexi_shapes;
    Units u[3];
    if (!hexi_q_units(g, u)) return 0;
    const auto& fit = FWD[g.d == 128];
    const double mb = (double)g.lq * g.nq * g.d * 6.0 * 1e-6;      // q read, o written
    const double t256 = fit[0].us(u[0], mb), t64 = fit[1].us(u[1], mb), t32 = u[2].n <= 768 ? fit[2].us(u[2], mb) : INFINITY;
    if (t256 <= 1.05 * (t64 < t32 ? t64 : t32)) return 0;
    return t64 <= t32 ? 64 : 32;
}

// Estimates for the choice of a whole step's shapes, fitted to launches of 64 to 4096 rows x 96 to 4096 keys x 2 to 24 heads.  Measured,
// head_dim 128, us of 256 / 64 / 32 rows: 300 x 700 x 4 heads 35.3 / 15.2 / 11.2; 512 x 1024 x 24 47.6 / 20.3 / 24.9;
// 1024 x 1024 x 24 52 / 40 / 41; 2048 x 2048 x 24 95 / 104 / 111; head_dim 64: 1024 x 1024 x 24 30 / 23 / 23;
// 2048 x 4096 x 24 112 / 116.
inline bool hexi_bwd_dq_times(const AttnGeom& g, DqTimes* t)
{
    using namespace hexi_shapes;
    const int n_q_tiles = (g.lq + Q_TILE - 1) / Q_TILE;
    if ((long long)g.nq * n_q_tiles >= 1024 || n_q_tiles > 4096) return false;     // four rounds of full-size units: their tail no longer matters
    const bool wide = g.d == 128;
    UnitTimes b256;
    for (int p = 0; p < n_q_tiles; ++p) {
        const int row0 = (n_q_tiles - 1 - p) * Q_TILE, rows = g.lq - row0 < Q_TILE ? g.lq - row0 : Q_TILE;
        const double nt = (seg_rows_le(g.ks, seg_pos_of_row(g.qs, row0 + rows - 1)) + KV_STREAM_TILE - 1) / KV_STREAM_TILE;
        if (nt < 1.0) continue;
        b256.add((wide ? 2.0 : 6.0) + nt, g.nq);
        t->rows64.add(wide ? 2.0 + 1.85 * ceil(nt / 2.0) : 1.0 + 1.14 * ceil(nt / 2.0), (long long)g.nq * ((rows + 63) / 64));
        t->rows32.add(wide ? 2.0 + 2.1 * ceil(nt / 4.0) : 1.0 + 1.4 * ceil(nt / 4.0), (long long)g.nq * ((rows + 31) / 32));
    }
    if (b256.n == 0) return true;
    t->t256 = wide ? 11.0 + b256.makespan(1.8, 2.2) : 7.0 + b256.makespan(1.1, 1.45);
    return true;
}

// How a backward step is launched.
struct BwdPlan {
    int dq_rows = 0;              // rows per dQ workgroup of the split kernel; 0: the 256-row workgroups
    bool split_keys = false;      // dK / dV in the split kernel's 32-key workgroups instead of the 128-key ones
    int run_len = 0;              // q heads per dK / dV workgroup
    int run_len_128 = 0;          // the same if the 128-key workgroups are taken
    bool unused = false;          // some kv head is read by no local q head: zero gradient
    int n_kv_tiles = 0;           // 128-key tiles of the chunk
    int n_known = 0;              // entries of seen
    float seen[4096];             // 64-row q tiles of one head that a key tile sees
};

// The shapes of a whole step.  forced_run_len: hexi_set_dkdv_run_len().
inline void hexi_plan_bwd_step(const AttnGeom& g, int forced_run_len, BwdPlan* plan)
{
    using namespace hexi_shapes;
    // dQ: rows per split workgroup, or 0 for the 256-row ones; by itself, the shape that is expected to finish first
    DqTimes dqt;
    int& dq_rows = plan->dq_rows;
    double dq_us = 0.0;
    const bool dq_small = hexi_bwd_dq_times(g, &dqt);
    if (dq_small) {
        const double t64 = 3.0 + dqt.rows64.makespan(), t32 = 3.0 + dqt.rows32.makespan();
        dq_us = dqt.t256;
        if (t64 < dq_us) { dq_us = t64; dq_rows = 64; }
        if (t32 < dq_us) { dq_us = t32; dq_rows = 32; }
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
        const int n_all = n_qtiles - seg_rows_le(g.qs, k_min - 1) / Q_STREAM_TILE;
        seen[t] = (float)(n_all > 0 ? n_all : 0);
    }
    // Launches that do not fill the chip take the split kernel's 32-key workgroups instead (whole groups where
    // they fill it: no atomics), in one launch with split dQ workgroups where that is shorter: the two kinds of unit
    // fill each other's last rounds.  Estimated times in us, fitted like those of dQ.  Measured, head_dim 128,
    // us of 128 / 32 keys: 300 rows x 700 keys x 4 / 2 heads 23.9 / 11.5; 512 x 1024 x 24 / 8 46 / 21; 1024 x 1024 x 24 / 8
    // 56 / 34; 2048 x 2048 x 24 / 8 154 / 118; 4096 x 4096 x 12 / 3 256 / 239 (runs of one and of two heads); head_dim 64:
    // 1024 x 1024 x 24 / 8 37 / 22, 4096 x 4096 x 24 / 8 270 / 260.  A forced run length keeps the 128-key workgroups that it is
    // defined for.
    bool& split_keys = plan->split_keys;
    if (forced_run_len < 1 && (long long)n_runs_for(run_len) * n_kv_tiles < 2048 && n_kv_tiles <= 4096) {
        const bool wide = g.d == 128;
        const double fill_us = 6.0;                        // zero-filling dk and dv where runs add into them
        const double atomic_us = (double)g.lc * g.d * 8.0 / 1.2e6;     // one run's atomics (1.2 TB/s)
        auto units = [&](int len, int keys) {
            const long long n_runs = n_runs_for(len);
            UnitTimes u;
            for (int t = 0; t < n_kv_tiles; ++t) {
                if (seen[t] < 1.0f) continue;
                const int cols = t == n_kv_tiles - 1 ? g.lc - t * KV_TILE : KV_TILE;
                u.add(keys == KV_TILE ? (wide ? 3.0 + 1.8 * len * seen[t] : 2.0 + 1.5 * len * seen[t])
                                      : (wide ? 3.0 + 2.2 * ceil(len * seen[t] / 4.0) : 1.0 + 1.5 * ceil(len * seen[t] / 4.0)),
                      n_runs * ((cols + keys - 1) / keys));
            }
            return u;
        };
        // dK / dV units, then dQ units, in one launch.  More than a round of them: all work shared out, a tenth longer
        // than the units take among their like (measured 1.1 to 1.3 at head_dim 128), plus half a unit of tail; 64-row dQ units then (as
        // 32-row ones they stream twice as much beside the dK / dV units: 54 us against 46 at 512 x 1024 x 24 / 8).
        auto joint = [&](const UnitTimes& kv, const UnitTimes& dq) {
            const double longest = kv.longest > dq.longest ? kv.longest : dq.longest;
            if (kv.n + dq.n <= 256) return longest;
            const double shared_out = (wide ? 1.1 : 1.0) * (kv.sum + dq.sum) / 256.0 + (dq.n > 0 ? 0.5 * dq.sum / (double)dq.n : 0.0);
            return shared_out > longest ? shared_out : longest;
        };
        double best = 11.0 + (run_len < max_cnt || unused ? fill_us : 0.0) + units(run_len, KV_TILE).makespan() + dq_us;
        const int len_128 = run_len;
        for (int len = max_cnt; len >= 1; --len) {
            if (max_cnt % len != 0 || (len_128 >= max_cnt && len < max_cnt)) continue;     // whole groups stay whole: reproducible sums
            const UnitTimes kv = units(len, 32);
            const double t0 = 3.0 + (len < max_cnt || unused ? fill_us : 0.0) + (len < max_cnt ? atomic_us * n_runs_for(len) : 0.0);
            auto consider = [&](double t, int rows) {
                if (t < best) { best = t; run_len = len; split_keys = true; dq_rows = rows; }
            };
            consider(t0 + kv.makespan() + dqt.t256, 0);
            if (dq_small && dqt.rows64.n > 0) {
                consider(t0 + joint(kv, dqt.rows64), 64);
                if (kv.n + dqt.rows32.n <= 256) consider(t0 + joint(kv, dqt.rows32), 32);
            }
        }
    }
}

// The shapes of a call for both halves or for one of them.  One by itself keeps the step's shape (and so the bits that it gives with
// the other) where that is expected to be 15 % faster there than the large workgroups, and takes those where not: what a joint launch
// gains for the step by filling last rounds, the half alone does not have.  Measured alone, us of the large / of the step's
// workgroups: dQ of 7496 rows x 634 keys x 16 heads x 128 90 / 120, 7696 x 530 x 32 x 64 97 / 134; dK / dV of 7599 x 1171 x 24 / 8 x 64
// 155 / 220, 5042 x 519 x 32 / 16 x 128 132 / 166.  Of the 7300 calls, 323 dQ and 125 dK / dV halves were more than 3 % slower than
// in the large workgroups, up to 59 %; so 1 and 12, up to 18 %.
inline void hexi_plan_bwd(const AttnGeom& g, int forced_run_len, bool want_dq, bool want_dkdv, BwdPlan* plan)
{
    using namespace hexi_shapes;
    constexpr double MARGIN = 1.15;
    hexi_plan_bwd_step(g, forced_run_len, plan);
    if (want_dq && want_dkdv) return;
    const bool wide = g.d == 128;
    if (want_dq && plan->dq_rows > 0) {
        Units u[3];
        const int r = plan->dq_rows == 64 ? 1 : 2;
        const double mb = (double)g.lq * g.nq * g.d * 12.0 * 1e-6;      // q and dO read, dq read and written
        if (hexi_q_units(g, u) && MARGIN * DQ[wide][r].us(u[r], mb) >= DQ[wide][0].us(u[0], mb)) plan->dq_rows = 0;
    }
    if (want_dkdv && plan->split_keys) {
        auto estimate = [&](int keys, int len) {
            const DkdvFit& f = DKDV[wide][keys == KV_TILE ? 0 : 1];
            HeadRuns runs;
            const bool shared = hexi_build_head_runs(g.kv_of_q, g.nq, g.nkv, len, &runs);
            Units u;
            for (int t = 0; t < plan->n_known; ++t) {
                if (plan->seen[t] < 1.0f) continue;
                const int cols = t == plan->n_kv_tiles - 1 ? g.lc - t * KV_TILE : KV_TILE;
                u.add(keys == KV_TILE ? len * plan->seen[t] : ceil(len * plan->seen[t] / 4.0), (long long)runs.n * ((cols + keys - 1) / keys));
            }
            const double run_mb = (double)g.lc * g.d * 8.0 * 1e-6;      // dk and dv of a run
            return f.launch.us(u, run_mb * g.nkv) + (shared || plan->unused ? f.clear : 0.0) + (shared ? run_mb * runs.n * f.atomic_mb : 0.0);
        };
        if (MARGIN * estimate(32, plan->run_len) >= estimate(KV_TILE, plan->run_len_128)) {
            plan->split_keys = false;
            plan->run_len = plan->run_len_128;
        }
    }
}

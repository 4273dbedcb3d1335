"""Shared helpers of the GPU parity tests: tolerances and oracle-side evaluation of a workload."""
import numpy as np
import torch

import oracle
from paper_2605_07569_amd import workloads as wl

# Per output tensor.  bf16 inputs: max-abs <= 2e-2 and relative L2 <= 5e-3.  fp32 inputs: relative
# L2 <= 1e-5 and max-abs <= 1e-5 * max(1, max|ref|).
TOL = {"bf16": dict(max_abs=2e-2, rel_l2=5e-3), "f32": dict(max_abs=1e-5, rel_l2=1e-5)}


def check(name, got, ref, dtype, log=None, abs_factor=1.0):
    """abs_factor widens the max-abs bound for intermediates that are sums of d products of an output
    (Delta = <dO, O> inherits up to sqrt(d) * |dO| times the per-element error allowed for O)."""
    got = np.asarray(got, dtype=np.float64)
    ref = np.asarray(ref, dtype=np.float64)
    assert got.shape == ref.shape, (name, got.shape, ref.shape)
    fin = np.isfinite(ref)
    assert np.array_equal(np.isfinite(got), fin), f"{name}: finiteness pattern differs"
    assert np.array_equal(got[~fin], ref[~fin]), f"{name}: infinities differ"
    g, r = got[fin], ref[fin]
    max_abs = float(np.max(np.abs(g - r))) if g.size else 0.0
    rel_l2 = float(np.linalg.norm(g - r) / max(np.linalg.norm(r), 1e-300)) if g.size else 0.0
    tol = TOL[dtype]
    lim_abs = abs_factor * tol["max_abs"] * (max(1.0, float(np.max(np.abs(r)))) if (dtype == "f32" and r.size) else 1.0)
    msg = f"{name}: max_abs={max_abs:.3e} (<= {lim_abs:.1e})  rel_l2={rel_l2:.3e} (<= {tol['rel_l2']:.1e})"
    if log is not None:
        log.append(msg)
    print("   ", msg, flush=True)
    assert max_abs <= lim_abs and rel_l2 <= tol["rel_l2"], msg
    return max_abs, rel_l2


def to64(t):
    return t.to(torch.float64).numpy()


def oracle_full(w, inputs, q_rows=None):
    """Exact results for the workload's shard (optionally a subset of its packed rows): o, lse, dq for
    those rows; dk, dv over the WHOLE global key range from those rows only."""
    q_pos = wl.seg_positions(w.q_segs).numpy()
    q, d_o = to64(inputs["q"]), to64(inputs["d_o"])
    if q_rows is not None:
        q, d_o, q_pos = q[q_rows], d_o[q_rows], q_pos[q_rows]
    # keys beyond the last query position are invisible to every row: leave them out
    n_keys = int(q_pos.max()) + 1
    k, v = to64(inputs["k"][:n_keys]), to64(inputs["v"][:n_keys])
    kv_pos = np.arange(n_keys, dtype=np.int64)
    r = oracle.attn_bwd(q, q_pos, k, v, kv_pos, d_o, w.scale, w.kv_of_q)
    o, lse = oracle.attn_fwd(q, q_pos, k, v, kv_pos, w.scale, w.kv_of_q)
    r["o"] = o
    assert np.array_equal(lse, r["lse"])
    r["n_keys"] = n_keys
    return r


def chunk_slices(w, j, x_global, n_keys):
    """Rows of a global-order [l_tot or n_keys, ...] oracle array for chunk j (zeros beyond n_keys)."""
    parts = []
    for s, n in w.chunks[j]:
        seg = np.zeros((n,) + x_global.shape[1:], dtype=x_global.dtype)
        hi = min(s + n, n_keys)
        if hi > s:
            seg[:hi - s] = x_global[s:hi]
        parts.append(seg)
    return np.concatenate(parts, axis=0)


# Ring steps (rows, keys, q heads, kv heads, head_dim) that the launchers give to the 256-row forward and dQ workgroups (dQ in a call
# for it alone): 256 units, one round of the chip.  The smaller sizes of the other tests go to the kernels for small launches.
# Row counts one past a tile, one short of it and whole tiles; key counts around the 64-key tiles, up to more than four of them, from
# two (with a single key dS is zero, and dq nothing to be relative to).
LARGE_STEPS = [(769, 2, 64, 8, 128), (800, 65, 64, 16, 128), (1023, 129, 64, 4, 128), (1024, 320, 64, 64, 128), (1793, 257, 32, 8, 128),
               (769, 64, 64, 8, 64), (1000, 193, 64, 16, 64), (1024, 385, 64, 4, 64), (511, 577, 128, 16, 64)]


# A shard (128 heads of 1800 rows: at 1024 units every step is large) and chunks in several segments, with holes, diagonal parts and
# keys that only the last rows see; a kv head's q heads are not adjacent.
LARGE_SHARD = dict(nq=128, nkv=8, q_segs=[(300, 400), (900, 1), (1000, 1399)],
                   chunks=[[(0, 180), (290, 110)], [(500, 1), (890, 130)], [(2300, 150)]], kv_of_q=[(5 * h + h // 8) % 8 for h in range(128)])

# Steps that the launch rules send to workgroups of 64 rows or keys: (lq, lc, nq, nkv, d, halves of the step that go there).  Blocks of 32
# rows and tiles of 64 by one more and one less, fewer rows than a block, runs of heads with and without atomics, chains of one
# block and of the unrolled loop and its remainder.
QUAD_STEPS = [(33, 65, 64, 64, 128, "b"), (33, 65, 64, 64, 64, "b"), (17, 129, 64, 64, 128, "b"), (17, 129, 64, 64, 64, "b"), (65, 33, 64, 64, 64, "b"),
              (130, 700, 64, 16, 128, "fb"), (130, 1000, 64, 16, 128, "fb"), (129, 33, 128, 8, 128, "f"), (129, 33, 128, 4, 128, "fb"),
              (200, 65, 64, 64, 128, "fb"), (200, 33, 128, 8, 64, "f"), (200, 33, 128, 4, 64, "fb"), (260, 700, 64, 16, 64, "b"), (257, 65, 64, 64, 64, "fb"), (520, 600, 64, 16, 64, "fb")]

# Single steps of the 64-row forward kernel, all keys visible or half of them at the start (off = lc / 2), and of dQ in 64-row workgroups in a call
# of its own (off = lc / 2).
QUAD_FWD_STEPS = [(130, 1000, 64, 16, 128), (520, 600, 64, 16, 64)]
QUAD_DQ_STEPS = [(130, 700, 64, 16, 128), (315, 132, 32, 32, 64)]

# A step whose dK / dV are cut into workgroups of 64 keys beside dQ in 256-row ones: (lq, lc, nq, nkv, head_dim, off), with one head to a group and,
# with atomics, three.
WIDE_DQ_STEPS = [(1998, 193, 64, 64, 64, 96), (2938, 83, 96, 32, 128, 83)]

# A shard of three segments whose steps all go to workgroups of 64 rows and keys: chunks with holes, wholly and partly visible; a kv
# head's q heads are not adjacent.
QUAD_SHARD = dict(nq=64, nkv=16, q_segs=[(1000, 180), (1230, 1), (1451, 210)], chunks=[[(0, 200), (500, 400)], [(200, 255), (1100, 346)], [(900, 200), (1460, 401)]],
                  kv_of_q=[(5 * h) % 16 for h in range(64)])

# fp32 steps at head_dim 64, all keys visible (off = lc) or diagonal (off = 0): (lq, lc, nq, nkv, off), shape of the forward, of dQ, of dK/dV
# and of dQ in a call of its own (0: 64 rows, shared; 1: 16 rows, split; 2: split, two workgroups a CU); rows and keys around the 16-row
# blocks, the 64-row tiles and the 128-row tiles of the split shapes, chunks shorter than a split tile.
F32_STEPS = [((33, 16, 2, 1, 16), (1, 1, 1, 1)), ((145, 257, 40, 40, 257), (2, 2, 0, 2)), ((1025, 17, 5, 1, 17), (0, 1, 1, 2)),
             ((273, 300, 24, 8, 300), (2, 2, 2, 2)), ((1000, 129, 48, 8, 129), (0, 1, 1, 0)), ((1000, 129, 24, 24, 129), (0, 0, 1, 0)), ((1039, 1039, 16, 4, 0), (2, 1, 1, 2)),
             ((497, 497, 12, 3, 0), (1, 1, 1, 1)), ((65, 1030, 24, 24, 1030), (1, 1, 0, 1)), ((128, 127, 128, 128, 127), (0, 0, 0, 0)),
             ((77, 1020, 16, 16, 0), (1, 0, 0, 1)), ((53, 865, 64, 16, 455), (1, 1, 0, 1))]      # (the last two: most keys are seen by no row)


# Forward steps of one round of 256-row workgroups (256 units of about the same length) and part of a second one; last tiles of 1, 188 and
# 76 rows.
PART_ROUND_STEPS = [(1025, 200, 64, 8, 128), (700, 200, 100, 20, 128), (1100, 257, 60, 60, 128)]


# Forward steps shared between whole rounds of 256-row workgroups and 64-row ones for the rest of the rows, (lq, lc, nq, nkv, head_dim, off): tiles
# of every head and of some, last tiles of 152, 213, 5 and 162 rows, the first rows without the last keys.
SHARED_STEPS = [(2712, 392, 24, 3, 128, 392), (5589, 388, 12, 3, 128, 388), (11269, 397, 6, 3, 128, 397), (4258, 420, 16, 8, 128, 399)]
SHARED_SHARD = dict(nq=24, nkv=3, d=128, q_segs=[(500, 1000), (1600, 1), (1650, 1711)], kv_segs=[(0, 300), (480, 120)])

# Backward steps whose dk / dv are summed in a fixed order, though runs of fewer heads are expected to be a little faster: (lq, lc, nq, nkv,
# head_dim, off), q heads per dK / dV workgroup in the step, and in a call for dK / dV alone: whole groups, and half groups, two of which add into
# a cleared element; the last two have more than two runs where dK / dV alone is expected to gain 15 %.
ORDER_STEPS = [((100, 123, 32, 4, 128, 0), 4, 4), ((364, 126, 16, 4, 64, 126), 2, 2), ((358, 535, 6, 2, 128, 0), 3, 3), ((3476, 3476, 12, 3, 128, 0), 2, 2),
               ((9087, 501, 24, 8, 128, 501), 3, 1), ((6280, 1109, 16, 4, 64, 1109), 2, 1)]

# Backward steps of 32-key and 64-key workgroups that add with atomics, in chunks whose last keys no row sees: (head_dim, nq, nkv, q_segs, kv_segs),
# keys per workgroup, keys seen (one less, as many and one more than whole workgroups).
UNSEEN_STEPS = [((128, 8, 1, [(0, 127)], [(0, 197)]), 32, 127), ((128, 8, 1, [(0, 128)], [(0, 428)]), 32, 128), ((64, 32, 4, [(0, 129)], [(0, 199)]), 32, 129),
                ((64, 8, 1, [(100, 60), (400, 90)], [(0, 150), (480, 200)]), 32, 160), ((128, 64, 8, [(0, 895)], [(0, 965)]), 64, 895),
                ((64, 64, 8, [(0, 1024)], [(0, 1094)]), 64, 1024), ((128, 64, 8, [(0, 1025)], [(0, 1095)]), 64, 1025)]


# fp32 steps of the split-operand kernels: (lq, lc, nq, nkv, head_dim), all keys visible, then what the rules deal out: the forward's tiles (32: all
# as 32-row units, 64: all as 64-row ones, 96: both, 0: another kernel), keys of a dK / dV unit (0: another kernel), rows of a dQ unit,
# units that the heads of a group are dealt to.
F32X3_STEPS = [((1079, 162, 4, 1, 128), (32, 32, 32, 2)), ((868, 112, 16, 8, 128), (64, 32, 64, 2)), ((691, 119, 32, 8, 128), (96, 32, 64, 2)),
               ((516, 93, 24, 8, 128), (64, 0, 0, 0)), ((523, 882, 9, 3, 128), (32, 32, 64, 2)), ((172, 196, 48, 16, 128), (64, 32, 64, 1)),
               ((726, 224, 24, 24, 128), (96, 32, 64, 1)), ((327, 161, 4, 1, 128), (0, 32, 32, 2)), ((625, 231, 24, 24, 128), (64, 32, 64, 1)),
               ((651, 577, 8, 8, 64), (32, 32, 64, 1)), ((91, 611, 48, 16, 64), (32, 64, 64, 1)), ((113, 814, 96, 24, 64), (64, 64, 64, 1)),
               ((693, 755, 24, 24, 64), (96, 64, 64, 1)), ((1196, 203, 32, 32, 64), (0, 0, 0, 0)),
               ((68, 151, 32, 32, 128), (0, 32, 32, 1)), ((53, 171, 48, 24, 128), (0, 32, 32, 1)), ((753, 16, 32, 32, 128), (0, 0, 0, 0)),
               ((820, 434, 32, 32, 128), (64, 32, 64, 1))]
# Those whose dk / dv are added to running sums by these kernels at head_dim 128: with all keys visible, in the diagonal chunk.
F32X3_ADDED = [(68, 151, 32, 32, 128), (53, 171, 48, 24, 128), (820, 434, 32, 32, 128)], [(753, 16, 32, 32, 128), (820, 434, 32, 32, 128)]

# fp32 steps that stay with the 16-row kernels at head_dim 128, rows from the middle of the keys: (lq, lc, nq, nkv), shapes of dQ and of dK / dV (0: 64 rows, shared;
# 1: 16 rows, split), chains of a score.
F32_128_STEPS = [((196, 199, 64, 64), (0, 0), 4), ((199, 16, 64, 32), (0, 1), 1), ((400, 43, 32, 16), (0, 1), 4), ((16, 266, 96, 48), (1, 0), 1), ((49, 256, 128, 64), (1, 0), 4),
                 ((70, 100, 2, 1), (1, 1), 1), ((513, 174, 8, 4), (1, 1), 4)]
# Others that are cut, forward and backward, rows from the middle of the keys: keys of a dK / dV unit, rows of a dQ unit, units to a group.
F32X3_MIDDLE_STEPS = [((685, 178, 6, 3, 128), (32, 32, 2)), ((347, 270, 16, 16, 128), (32, 64, 1)), ((871, 1364, 16, 16, 64), (64, 64, 1))]


def f32x3_diagonal(lq, lc):
    """The shard's own keys after a chunk of lc, in two segments with a gap, the first keys of which are not the shard's."""
    a = lq // 2
    return [(lc, a), (lc + a + 7, lq - a)], [(lc, a + 7), (lc + a + 7, lq - a)]

"""The launch rules (which workgroup shapes a bf16 ring step takes), compiled for the host alone."""
import os
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _compile(tmp_path_factory, name):
    hipcc = "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("shapes") / name)
    subprocess.check_call([hipcc, "-O1", "-std=c++17", "-x", "c++", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                           "-I", os.path.join(ROOT, "include"),
                           "-I", os.path.join(ROOT, "paper_2605_07569_amd", "csrc"),
                           os.path.join(ROOT, "tests", "host", name + ".cpp"), "-o", exe])
    return exe


@pytest.fixture(scope="module")
def shapes(tmp_path_factory):
    exe = _compile(tmp_path_factory, "shape_check")

    def ask(steps):
        """steps: (head_dim, nq, nkv, q_segs, kv_segs[, kv_of_q[, forced run length]]) -> dicts"""
        lines = []
        for d, nq, nkv, qs, ks, *more in steps:
            segs = lambda x: f"{len(x)} " + " ".join(f"{s} {n}" for s, n in x)
            m = " ".join(map(str, more[0])) if more and more[0] else ""
            lines.append(f"{d} {nq} {nkv} {more[1] if len(more) > 1 else 0} {segs(qs)} {segs(ks)} {m}")
        out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True).stdout.split("\n")
        names = ("fwd_rows", "dq_rows", "keys", "run_len", "atomic", "atomic_128", "dq_alone", "keys_alone",
                 "f32_fwd", "f32_dq", "f32_dkdv", "f32_dq_alone", "run_len_alone", "run_len_accumulate", "fwd_tiles", "rest_tiles")
        return [dict(zip(names, map(int, line.split()))) for line in out if line]

    return ask


def _step(lq, lc, nq, nkv, d, off):
    """rows [off, off + lq) against keys [0, lc)"""
    return d, nq, nkv, [(off, lq)], [(0, lc)]


def test_smallest_and_largest_launches(shapes):
    small, large, forced = shapes([_step(300, 700, 4, 2, 128, 700), _step(16384, 16384, 24, 8, 128, 16384),
                                   (128, 8, 1, [(1024, 512)], [(0, 512)], None, 3)])
    assert small["fwd_rows"] == 32 and small["dq_rows"] == 32 and small["keys"] == 32
    assert large["fwd_rows"] == 0 and large["dq_rows"] == 0 and large["keys"] == 128
    assert forced["keys"] == 128 and forced["run_len"] == 3        # a forced run length keeps the 128-key workgroups


@pytest.mark.parametrize("lq,lc,nq,nkv,d,off,rows", [
    # us measured in 256 / 64 / 32 rows per workgroup: 19.4 / 23.0 / 30.5, 20.0 / 23.7 / 31.5, 15.3 / 17.7 / 22.5,
    # 14.1 / 16.2 / 21.4, 150 / 212 / 243: the 256-row kernel
    (1091, 118, 32, 16, 128, 102, 0), (2450, 97, 16, 2, 128, 0, 0), (6523, 181, 8, 4, 64, 181, 0), (3254, 125, 16, 4, 64, 125, 0),
    (666, 6831, 48, 16, 128, 6831, 0),
    # 27.5 / 12.3 / 9.7, 32.0 / 16.3 / 20.8, 151 / 139 / 159, 60.6 / 78 / 99
    (300, 700, 4, 2, 128, 700, 32), (512, 1024, 24, 8, 128, 1024, 64), (4096, 4096, 24, 8, 64, 4096, 64),
    (2048, 2048, 24, 8, 128, 2048, 0)])
def test_forward_takes_the_shape_measured_faster(shapes, lq, lc, nq, nkv, d, off, rows):
    assert shapes([_step(lq, lc, nq, nkv, d, off)])[0]["fwd_rows"] == rows


@pytest.mark.parametrize("lq,lc,nq,nkv,d,off,keys,dq_alone,keys_alone", [
    # a step in joint launches of 64 or 32 rows and keys whose halves are faster in other shapes by themselves; us of the step in 128 keys and 256 rows /
    # in its own shape; of dQ alone in 256 rows / as many as in the step; of dK / dV alone in 128 keys / as in the step / in the shape taken:
    # 290 / 166, 93 / 98, 206 / 129 / 116; 266 / 204, 92 / 120, 177 / 178 / 137; 261 / 241, 114 / 127, 152 / 217 / 146; 60 / 58, 24 / 36, 36 / 49 / 30
    (7496, 634, 16, 4, 128, 634, 64, 0, 32), (7696, 530, 32, 4, 64, 430, 64, 0, 32), (7599, 1171, 24, 8, 64, 0, 64, 0, 64),
    (1016, 390, 64, 8, 64, 390, 32, 0, 32),
    # dQ 49 / 18 (64 rows), dK / dV 44 / 27 / 21 (32 keys); 36 / 9.3, 23 / 12 (32)
    (512, 1024, 24, 8, 128, 1024, 64, 64, 32), (300, 700, 4, 2, 128, 700, 32, 32, 32),
    # few keys and many rows, few rows and many keys: dQ 21.9 / 11.1 (32 rows; 11.4 in 64); 236 / 39 (32; 65.9 in 64)
    (8245, 74, 2, 2, 64, 0, 32, 32, 32), (582, 9338, 8, 1, 128, 6538, 64, 32, 32)])
def test_a_half_by_itself_is_not_sent_to_a_slower_shape(shapes, lq, lc, nq, nkv, d, off, keys, dq_alone, keys_alone):
    got = shapes([_step(lq, lc, nq, nkv, d, off)])[0]
    assert (got["keys"], got["dq_alone"], got["keys_alone"]) == (keys, dq_alone, keys_alone)


def test_64_keys_or_32(shapes):
    # us measured in 64 / 32 keys and rows: 31.5 / 39.5, 178 / 212, 384 / 459; 18.5 / 12.0, 96 / 58; 64-key workgroups beside 256-row dQ ones, in two launches
    steps = [_step(512, 1024, 24, 8, 128, 1024), _step(2048, 2048, 24, 8, 128, 2048), _step(4096, 4096, 24, 8, 64, 4096),
             _step(300, 700, 4, 2, 128, 700), _step(1016, 390, 64, 8, 64, 390), _step(5287, 902, 64, 16, 128, 0), _step(1998, 193, 64, 64, 64, 96)]
    assert [(got["keys"], got["dq_rows"]) for got in shapes(steps)] == [(64, 64), (64, 64), (64, 64), (32, 32), (32, 32), (64, 0), (64, 0)]


def test_no_step_gets_atomics_that_its_128_key_launch_would_not_have(shapes):
    import random
    rng = random.Random(11)
    log_int = lambda lo, hi: round(2.0 ** rng.uniform(lo, hi))
    steps = []
    for _ in range(3000):
        nkv = rng.choice([1, 2, 3, 8, 16])
        nq = nkv * rng.choice([1, 2, 3, 4, 8])
        if nq <= 128:
            lq, lc = log_int(0, 14), log_int(0, 16)
            steps.append(_step(lq, lc, nq, nkv, rng.choice([64, 128]), rng.choice([0, lc, rng.randrange(lc)])))
    assert all(got["atomic"] <= got["atomic_128"] for got in shapes(steps))


def test_sums_keep_a_fixed_order_for_a_small_gain(shapes):
    from parity_util import ORDER_STEPS
    got = shapes([_step(*s) for s, *_ in ORDER_STEPS])
    assert [(g["run_len"], g["run_len_alone"]) for g in got] == [(n, alone) for _, n, alone in ORDER_STEPS]
    # added to what dk and dv hold already, two runs have no fixed order: whole groups, unless two are expected to be 15 % faster
    assert [g["run_len_accumulate"] for g in got] == [8, 4, 3, 2, 3, 2]


def test_the_unseen_keys_tests_reach_atomics(shapes):
    from parity_util import UNSEEN_STEPS
    assert [(g["keys"], g["atomic"]) for g in shapes([s for s, *_ in UNSEEN_STEPS])] == [(keys, 1) for _, keys, _ in UNSEEN_STEPS]


def test_the_large_workgroups_tests_reach_them(shapes):
    from parity_util import LARGE_SHARD as s, LARGE_STEPS
    steps = [_step(lq, lc, nq, nkv, d, off) for lq, lc, nq, nkv, d in LARGE_STEPS for off in (lc, lc // 2)]
    steps += [(d, s["nq"], s["nkv"], s["q_segs"], ch, s["kv_of_q"]) for d in (64, 128) for ch in s["chunks"]]
    assert [(got["fwd_rows"], got["dq_alone"]) for got in shapes(steps)] == [(0, 0)] * len(steps)


def test_the_64_wide_workgroups_tests_reach_them(shapes):
    from parity_util import QUAD_STEPS
    steps = [(_step(lq, lc, nq, nkv, d, off), halves) for lq, lc, nq, nkv, d, halves in QUAD_STEPS for off in (lc, lc // 2)]
    for (step, halves), got in zip(steps, shapes([s for s, _ in steps])):
        assert "f" not in halves or got["fwd_rows"] == 64, step
        assert "b" not in halves or (got["dq_rows"] == 64 and got["keys"] == 64), step


def test_the_single_steps_of_64_wide_workgroups_reach_them(shapes):
    from parity_util import QUAD_DQ_STEPS, QUAD_FWD_STEPS, QUAD_SHARD as s, WIDE_DQ_STEPS
    assert [got["fwd_rows"] for got in shapes([_step(*x, off) for x in QUAD_FWD_STEPS for off in (x[1], x[1] // 2)])] == [64] * 4
    assert [got["dq_alone"] for got in shapes([_step(*x, x[1] // 2) for x in QUAD_DQ_STEPS])] == [64] * 2
    assert [(got["dq_rows"], got["keys"], got["atomic"]) for got in shapes([_step(*x) for x in WIDE_DQ_STEPS])] == [(0, 64, 0), (0, 64, 1)]
    for got in shapes([(d, s["nq"], s["nkv"], s["q_segs"], ch, s["kv_of_q"]) for d in (64, 128) for ch in s["chunks"]]):
        assert (got["fwd_rows"], got["dq_rows"], got["keys"], got["dq_alone"]) == (64, 64, 64, 64)


def test_a_round_and_a_part_of_large_forward_workgroups(shapes):
    # more than 64 units over whole rounds: one kernel for all rows.  384, 384, 380 units of 256 rows; us measured in 256 / 64 rows: 226 / 232, 127.5 /
    # 133.1; whole passes of eight such steps, some of 2048 visible keys, in 256 rows / shared 1144 / 1169; of four 1425 / 1486, 1858 / 1956
    steps = [_step(4096, 4096, 24, 8, 128, 4096), _step(4096, 2048, 24, 8, 128, 2048), _step(5705, 5705, 16, 4, 128, 5705), _step(7769, 7769, 12, 4, 128, 7769)]
    zigzag = lambda r: [(2048 * r, 2048), (2048 * (15 - r), 2048)]
    steps += [(128, 24, 8, zigzag(5), zigzag(j)) for j in range(8)]
    got = shapes(steps)
    assert [g["fwd_rows"] for g in got] == [0] * len(steps) and not any(g["rest_tiles"] for g in got)
    # head_dim 64, and rows with so few keys that a second launch takes what it saves
    from parity_util import PART_ROUND_STEPS
    got = shapes([_step(9000, 9000, 8, 2, 64, 9000)] + [_step(*s, s[1]) for s in PART_ROUND_STEPS])
    assert not any(g["rest_tiles"] for g in got)


def test_whole_rounds_of_large_forward_workgroups_and_the_rest_in_small_ones(shapes):
    from parity_util import SHARED_SHARD as w, SHARED_STEPS
    got = shapes([_step(*s) for s in SHARED_STEPS] + [(w["d"], w["nq"], w["nkv"], w["q_segs"], w["kv_segs"])])
    assert [(g["fwd_rows"], g["fwd_tiles"], g["rest_tiles"]) for g in got] == [(0, 256, 8), (0, 256, 8), (0, 256, 14), (0, 256, 16), (0, 256, 8)]
    # us of whole passes measured in one kernel / shared: 2172 / 1891, 4193 / 3635, 2254 / 2001, 1019 / 912, 3250 / 2947
    steps = [_step(lq, lq, nq, nkv, 128, lq) for lq, nq, nkv in ((5612, 24, 3), (11725, 12, 4), (6128, 24, 8), (4862, 16, 2), (6325, 32, 8))]
    assert [g["rest_tiles"] for g in shapes(steps)] == [16, 40, 64, 48, 32]


def test_a_shared_forward_step_covers_every_row_once(tmp_path_factory):
    import random
    exe, rng, lines = _compile(tmp_path_factory, "share_check"), random.Random(5), []
    for _ in range(3000):
        nq, n_q_tiles = rng.randint(1, 128), rng.randint(1, 40)
        if nq * n_q_tiles > nq:
            lines.append(f"{nq} {n_q_tiles} {rng.choice([nq, nq * n_q_tiles - 1, rng.randint(nq, nq * n_q_tiles - 1)])}")
    out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True).stdout.split()
    assert len(out) == len(lines) and set(out) == {"0"}


def test_f32_steps_take_the_shapes_they_are_meant_for(shapes):
    # (the rule of the 16-row kernels, which a step that goes to the split-operand ones does not come to)
    from parity_util import F32_STEPS
    got = shapes([_step(lq, lc, nq, nkv, 64, off) for (lq, lc, nq, nkv, off), _ in F32_STEPS])
    assert [(g["f32_fwd"], g["f32_dq"], g["f32_dkdv"], g["f32_dq_alone"]) for g in got] == [s for _, s in F32_STEPS]
    # us measured, shared / split / two a CU: forward 859 / 1106 / 902, 161 / 199 / 162, 55 / 61 / 50, diagonal 191 / 55 / 62, 155 / 179 / 135
    steps = [_step(4096, 4096, 24, 8, 64, 4096), _step(2048, 2048, 16, 4, 64, 2048), _step(1024, 1024, 16, 4, 64, 1024), _step(4096, 4096, 2, 2, 64, 0),
             _step(2048, 2048, 24, 8, 64, 0)]
    assert [g["f32_fwd"] for g in shapes(steps)] == [0, 0, 2, 1, 2]
    # keys that no row sees are units as well; us of the whole backward shared / split / two a CU 34 / 174 / 114; 26 / 24 / 19 (35 as two launches);
    # dQ split beside shared dK / dV 93, as one launch 148 / 285 / 182
    steps = [_step(lq, lc, nq, nkv, 64, off) for lq, lc, nq, nkv, off in ((117, 4743, 16, 16, 0), (209, 2390, 4, 4, 0), (53, 3065, 64, 16, 1555))]
    assert [(min(g["f32_dq"], 1), g["f32_dkdv"]) for g in shapes(steps)] == [(0, 0), (0, 0), (1, 0)]
    # backward 2781 / 3302 / 2769, 340 / 90 / 108, 203 / 47 / 50 for split / two a CU; head_dim 128 keeps one workgroup a CU
    steps = [_step(4096, 4096, 24, 8, 64, 4096), _step(1024, 2048, 4, 1, 64, 2048), _step(512, 512, 8, 2, 64, 512), _step(1000, 1010, 16, 16, 128, 1010),
             _step(300, 300, 4, 2, 128, 300)]
    assert [(g["f32_dq"], g["f32_dkdv"]) for g in shapes(steps)] == [(2, 2), (1, 1), (1, 1), (0, 0), (1, 1)]


@pytest.fixture(scope="module")
def split_operand_shapes(tmp_path_factory):
    exe = _compile(tmp_path_factory, "f32x3_check")

    def ask(steps, accumulate=False, chains=False, halves=False, forced=False):
        segs = lambda x: f"{len(x)} " + " ".join(f"{s} {n}" for s, n in x)
        lines = [f"{nq} {nkv} {d} {segs(qs)} {segs(ks)}" for d, nq, nkv, qs, ks in steps]
        out = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, check=True).stdout.split("\n")
        got = []
        for line in filter(None, out):
            use, n64, tiles, *bwds, n_chains, q, q64, kv, kv_runs, added, added_runs, runs_of_one, runs_of_all = map(int, line.split())
            if forced:
                got.append((runs_of_one, runs_of_all))
                continue
            bwd, keys, rows64, runs = bwds[4:] if accumulate else bwds[:4]
            got.append((q * (64 if q64 else 32), kv * kv_runs, added * added_runs) if halves else n_chains if chains else ((32 if n64 == 0 else 64 if n64 == tiles else 96) if use else 0, keys if bwd else 0,
                                                (64 if rows64 else 32) if bwd else 0, runs if bwd else 0))
        return got

    return ask


def test_scores_are_summed_in_one_chain_unless_a_part_of_the_step_is_cut(split_operand_shapes):
    # us of a backward with one chain / four: 664 / 729, 182 / 200; forward, backward or a backward under HEXI_ACCUMULATE cut: four
    steps = [_step(*s) for s in ((5761, 130, 32, 16, 128, 130), (1264, 108, 48, 24, 128, 0), (300, 300, 4, 2, 128, 300), (1079, 162, 4, 1, 128, 162),
                                 (516, 93, 24, 8, 128, 93), (327, 161, 4, 1, 128, 161), (4096, 4096, 16, 4, 128, 4096), (4096, 4096, 24, 8, 64, 4096))]
    assert split_operand_shapes(steps, chains=True) == [1, 1, 1, 4, 4, 4, 4, 1]


def test_a_forced_run_of_a_whole_group_holds_for_fp32_steps(split_operand_shapes):
    from parity_util import F32X3_STEPS
    two = [s for s, (*_, runs) in F32X3_STEPS if runs == 2]
    assert len(two) > 3 and set(split_operand_shapes([_step(lq, lc, nq, nkv, d, lc) for lq, lc, nq, nkv, d in two], forced=True)) == {(2, 1)}


def test_fp32_steps_that_stay_with_the_16_row_kernels_at_head_dim_128(shapes, split_operand_shapes):
    from parity_util import F32_128_STEPS
    steps = [_step(lq, lc, nq, nkv, 128, lc // 2) for (lq, lc, nq, nkv), *_ in F32_128_STEPS]
    assert [(g["f32_dq"], g["f32_dkdv"]) for g in shapes(steps)] == [s for _, s, _ in F32_128_STEPS]
    assert [b for _, b, *_ in split_operand_shapes(steps)] == [0] * len(steps) and split_operand_shapes(steps, chains=True) == [n for *_, n in F32_128_STEPS]
    # the forward of all visible keys: 64-row workgroups, split operands, 64-row ones beside a cut backward, 16-row ones
    steps = [_step(lq, lc, nq, nkv, 128, lc) for lq, lc, nq, nkv in ((199, 16, 64, 32), (1000, 1010, 16, 16), (404, 16, 32, 8), (100, 1010, 16, 16))]
    assert [f[0] and "cut" or g["f32_fwd"] for f, g in zip(split_operand_shapes(steps), shapes(steps))] == [0, "cut", 0, 1]
    assert split_operand_shapes(steps, chains=True) == [1, 4, 4, 1]


def test_an_fp32_half_by_itself_is_not_cut_where_that_is_slower(split_operand_shapes):
    # rows of a dQ unit, units of a group of heads for dK / dV alone, and for dK / dV added to running sums (0: 16-row kernels).  us of dQ in 16-row kernels / as in
    # the whole step: 92 / 126, 14 / 18, 13 / 19, 98 / 46, 283 / 192; of dK / dV 66 / 97, 118 / 164
    steps = [_step(*s) for s in ((329, 1509, 24, 8, 128, 1509), (332, 138, 8, 1, 128, 138), (124, 1995, 16, 8, 128, 0), (821, 2097, 16, 2, 128, 0), (1081, 5315, 6, 2, 128, 5315),
                                 (93, 2465, 24, 24, 128, 1232), (88, 4729, 32, 16, 128, 2364), (1000, 1000, 16, 2, 128, 0))]
    got = split_operand_shapes(steps, halves=True)
    assert [q for q, *_ in got[:5]] == [0, 0, 0, 32, 32] and [kv for _, kv, _ in got[5:7]] == [0, 0] and got[7] == (32, 2, 0)
    # whole steps, us in 16-row kernels / cut: 318 / 496, 108 / 146, 664 / 620
    assert [s[1] for s in split_operand_shapes([_step(135, 4439, 24, 24, 128, 4439), _step(93, 2465, 24, 24, 128, 1232), _step(1081, 5315, 6, 2, 128, 5315)])] == [0, 0, 32]


def test_split_operand_fp32_steps_take_the_shapes_they_are_meant_for(split_operand_shapes):
    from parity_util import F32X3_ADDED, F32X3_MIDDLE_STEPS, F32X3_STEPS, f32x3_diagonal
    ask = split_operand_shapes
    assert ask([_step(lq, lc, nq, nkv, d, lc) for (lq, lc, nq, nkv, d), _ in F32X3_STEPS]) == [s for _, s in F32X3_STEPS]
    # sums added to
    visible, diagonal = F32X3_ADDED
    assert all(b > 0 for _, b, *_ in ask([_step(lq, lc, nq, nkv, d, lc) for lq, lc, nq, nkv, d in visible], accumulate=True))
    assert all(b > 0 for _, b, *_ in ask([(d, nq, nkv) + f32x3_diagonal(lq, lc) for lq, lc, nq, nkv, d in diagonal], accumulate=True))
    # masked blocks: diagonal chunks as well, forward and backward, with units of 32 and of 64
    diagonal = ask([(d, nq, nkv) + f32x3_diagonal(lq, lc) for (lq, lc, nq, nkv, d), _ in F32X3_STEPS])
    assert [diagonal[i] for i in (0, 7, 8, 13)] == [(0, 32, 32, 2), (0, 32, 32, 2), (64, 32, 64, 1), (64, 64, 64, 1)]
    middle = ask([_step(lq, lc, nq, nkv, d, lc // 2) for (lq, lc, nq, nkv, d), _ in F32X3_MIDDLE_STEPS])
    assert all(f > 0 for f, *_ in middle) and [tuple(b) for _, *b in middle] == [s for _, s in F32X3_MIDDLE_STEPS]
    # us measured before / with the split-operand kernels: forward 1139 / 759, 295 / 215, 168 / 121; backward 3634 / 3049, 865 / 740, 496 / 404; 79 / 100
    # forward of 100 rows; 17 / 23 and 43 / 48 of 1024 at head_dim 64
    taken = ask([_step(4096, 4096, 16, 4, 128, 4096), _step(3056, 3000, 6, 2, 128, 3000), _step(4096, 4096, 8, 8, 64, 0),
                 _step(100, 4000, 8, 2, 128, 4000), _step(1024, 1024, 4, 4, 64, 1024)])
    assert [t[0] for t in taken] == [64, 96, 64, 0, 0] and [t[1] > 0 for t in taken] == [True, True, True, False, False]

"""GPU parity: the HIP library, called through the C ABI, against the fp64 CPU oracle.

Tier 0: configuration 1 (fp32) in full.  Tier 1: shape-preserving minis of configurations 2-5
(all token counts divided, heads / head_dim / chunk structure kept), every output element.  Edge
cases: ragged lengths, many segments, strided inputs, explicit head maps, chunks in the future,
rows that see nothing, the unfused fwd + merge path, accumulate flags.
"""
import numpy as np
import pytest
import torch

import oracle
from paper_2605_07569_amd import hexi, replay
from paper_2605_07569_amd import workloads as wl
from parity_util import (F32_128_STEPS, F32_STEPS, F32X3_MIDDLE_STEPS, F32X3_STEPS, LARGE_SHARD, LARGE_STEPS, ORDER_STEPS, PART_ROUND_STEPS, QUAD_DQ_STEPS, QUAD_FWD_STEPS, QUAD_SHARD, QUAD_STEPS,
                         SHARED_SHARD, SHARED_STEPS, UNSEEN_STEPS, WIDE_DQ_STEPS, check, chunk_slices, f32x3_diagonal, oracle_full, to64)

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


@pytest.fixture
def force_run_len():
    """Sets the dK/dV launcher's forced head-run length for the test and restores the automatic choice after it."""
    yield hexi.hexi_set_dkdv_run_len
    hexi.hexi_set_dkdv_run_len(0)


def _run_and_compare(w, seed=20260507, fused=True):
    """Runs the whole replay on the GPU and compares every element of every output with the oracle at the flat
    tolerances.  (Delta, an intermediate and not one of the five outputs, is a sum of d products of dO with o: its
    max-abs bound is that of o times sqrt(d); its effect on the outputs is covered by the flat bounds on dq / dk.)"""
    print(f"\n[{w.name}] lq={w.lq} heads={w.n_q_heads}/{w.n_kv_heads} d={w.head_dim} chunks={len(w.chunks)} fused={fused}", flush=True)
    inputs = wl.make_inputs(w, seed)
    run = replay.ShardRun(w, inputs, DEV, fused_merge=fused)
    run.step()
    torch.cuda.synchronize()
    ref = oracle_full(w, inputs)
    dk = np.concatenate([run.dk[j].cpu().numpy() for j in range(len(w.chunks))])
    dv = np.concatenate([run.dv[j].cpu().numpy() for j in range(len(w.chunks))])
    dk_ref = np.concatenate([chunk_slices(w, j, ref["dk"], ref["n_keys"]) for j in range(len(w.chunks))])
    dv_ref = np.concatenate([chunk_slices(w, j, ref["dv"], ref["n_keys"]) for j in range(len(w.chunks))])
    failures = []
    for name, got, want, fac in (("o", run.o.cpu(), ref["o"], 1.0), ("lse", run.lse.cpu(), ref["lse"], 1.0),
                                 ("delta", run.delta.cpu(), ref["delta"], float(w.head_dim) ** 0.5),
                                 ("dq", run.dq.cpu(), ref["dq"], 1.0), ("dk", dk, dk_ref, 1.0),
                                 ("dv", dv, dv_ref, 1.0)):
        try:
            check(name, got, want, w.dtype, abs_factor=fac)
        except AssertionError as e:
            failures.append(str(e))
    assert not failures, failures
    return run, inputs, ref


def test_tier0_cfg1_fp32_full():
    run, inputs, ref = _run_and_compare(wl.config(1))
    # bookkeeping: counted pairs of the replay equal the closed form
    n = sum(hexi.hexi_shard_mask(run.w.q_segs, ch, want_pos=False)["n_pairs"] for ch in run.w.chunks)
    assert n == 1573376


def test_cfg1_unfused_partials_and_merge():
    w = wl.config(1)
    inputs = wl.make_inputs(w)
    run = replay.ShardRun(w, inputs, DEV, fused_merge=False, keep_partials=True)
    run.forward()
    torch.cuda.synchronize()
    q_pos = wl.seg_positions(w.q_segs).numpy()
    q = to64(inputs["q"])
    o_acc = np.zeros_like(q)
    lse_acc = np.full((w.n_q_heads, w.lq), -np.inf)
    for j, ch in enumerate(w.chunks):
        kc, vc = to64(wl.gather_rows(inputs["k"], ch)), to64(wl.gather_rows(inputs["v"], ch))
        o_p, lse_p = oracle.attn_fwd(q, q_pos, kc, vc, wl.seg_positions(ch).numpy(), w.scale)
        check(f"o_part[{j}]", run.partials[j][0].cpu(), o_p, "f32")
        check(f"lse_part[{j}]", run.partials[j][1].cpu(), lse_p, "f32")
        o_acc, lse_acc = oracle.merge(o_acc, lse_acc, o_p, lse_p)
    check("o_merged", run.o.cpu(), o_acc, "f32")
    check("lse_merged", run.lse.cpu(), lse_acc, "f32")


@pytest.mark.parametrize("idx,shrink", [(2, 16), (3, 16), (4, 32), (5, 32)])
def test_tier1_minis_full_tensor(idx, shrink):
    # (configuration 4 scales K by 3: sharply peaked rows, whose few large dS values the dQ kernel carries with
    # their rounding residuals; every configuration is held to the same flat bounds)
    _run_and_compare(wl.config(idx, shrink=shrink))


def test_cfg2_mini_unfused_and_contiguous_chunking_agree():
    w = wl.config(2, shrink=32)
    _run_and_compare(w, fused=False)
    _run_and_compare(wl.contiguous_chunks(w, 8))


def _custom(name, dtype, nq, nkv, d, l_tot, q_segs, chunks, kv_of_q=None, k_scale=1.0):
    return wl.Workload(name, dtype, nq, nkv, d, l_tot, q_segs, chunks, k_scale=k_scale, kv_of_q=kv_of_q)


@pytest.mark.parametrize("dtype,d", [("bf16", 128), ("bf16", 64), ("f32", 64), ("f32", 128)])
def test_ragged_lengths_and_many_segments(dtype, d):
    # unaligned shard / chunk lengths (1000, 777, 1, 130), a shard of 4 segments, chunks of 1-3
    # segments, one chunk wholly in the future, rows that see nothing of some chunk
    q_segs = [(37, 1), (100, 130), (400, 777), (1500, 92)]
    chunks = [[(0, 777)], [(777, 1), (778, 222)], [(1000, 130), (1130, 370), (1500, 92)], [(1592, 408)]]
    w = _custom(f"ragged_{dtype}_{d}", dtype, 4, 2, d, 2000, q_segs, chunks)
    _run_and_compare(w, seed=7)


def test_explicit_head_map_and_single_rows():
    # a kv head shared by non-adjacent q heads (an HP cut through GQA groups), 1-row shard and 1-key chunk
    w = _custom("headmap", "bf16", 6, 3, 128, 600, [(0, 1), (299, 301)], [[(0, 1)], [(1, 299)], [(300, 300)]],
                kv_of_q=[2, 0, 1, 0, 2, 2])
    _run_and_compare(w, seed=11)
    w = _custom("headmap_f32", "f32", 3, 2, 64, 200, [(150, 50)], [[(0, 200)]], kv_of_q=[1, 0, 1])
    _run_and_compare(w, seed=12)


@pytest.mark.parametrize("run_len", [1, 2, 3, 8])
def test_dkdv_head_runs(run_len, force_run_len):
    # The dK/dV kernel walks runs of q heads that share a kv head in one workgroup; the launcher picks the
    # run length from the launch size, so small shapes would only ever see runs of one head.  Force the
    # length: whole groups (no atomics), runs with a remainder (3 of 5), non-adjacent heads of a group,
    # groups of unequal size, masked + full + ragged tiles in every head of a run.
    force_run_len(run_len)
    w = _custom(f"runs{run_len}", "bf16", 8, 3, 128, 700, [(150, 70), (400, 300)], [[(0, 333)], [(333, 367)]],
                kv_of_q=[0, 1, 0, 0, 2, 0, 1, 0])
    _run_and_compare(w, seed=21)
    # one group of 8 heads over several key tiles, unfused path
    w = _custom(f"runs{run_len}_hp", "bf16", 8, 1, 128, 1024, [(512, 512)], [[(0, 512)], [(512, 512)]])
    _run_and_compare(w, seed=22, fused=False)


def _random_case(rng, i, l_range=(200, 1400), max_heads=8, d_bf16=128):
    """A seeded random shard: the sequence [0, L) cut into pieces, each piece dealt to one of 1-4 chunks, the q
    shard takes 1-3 pieces; random head counts and kv map."""
    dtype = "bf16" if i % 3 else "f32"
    d = d_bf16 if dtype == "bf16" else int(rng.choice([64, 128]))
    L = int(rng.integers(*l_range))
    n_pieces = int(rng.integers(2, 9))
    cuts = sorted(set(int(c) for c in rng.integers(1, L, size=n_pieces - 1)))
    edges = [0] + cuts + [L]
    pieces = [(a, b - a) for a, b in zip(edges[:-1], edges[1:])]
    # every piece goes to exactly one chunk (the chunks together hold every key the shard can see); a chunk's
    # pieces need not be adjacent, so its segment list has holes, as a zigzag pair does
    n_chunks = int(rng.integers(1, min(4, len(pieces)) + 1))
    owner = rng.integers(0, n_chunks, size=len(pieces))
    chunks = [[p for p, o in zip(pieces, owner) if o == c] for c in range(n_chunks)]
    chunks = [c for c in chunks if c]
    rng.shuffle(chunks)                       # the ring may deliver them in any order
    own = sorted(rng.choice(len(pieces), size=min(len(pieces), int(rng.integers(1, 4))), replace=False).tolist())
    q_segs = [pieces[k] for k in own]
    nkv = int(rng.integers(1, 4))
    nq = int(rng.integers(nkv, max(nkv, max_heads) + 1))
    kv_of_q = sorted(int(x) for x in rng.integers(0, nkv, size=nq)) if rng.random() < 0.5 else [int(x) for x in rng.integers(0, nkv, size=nq)]
    return _custom(f"rand{i}_{dtype}", dtype, nq, nkv, d, L, q_segs, chunks, kv_of_q=kv_of_q)


def test_randomized_small_shards():
    rng = np.random.default_rng(20260507)
    for i in range(16):
        w = _random_case(rng, i)
        _run_and_compare(w, seed=100 + i, fused=bool(i % 2))


def test_randomized_longer_shards():
    # the same generator at lengths that span many q tiles (256 rows) and key tiles (64 / 128 keys) per workgroup
    rng = np.random.default_rng(7569)
    for i in range(8):
        w = _random_case(rng, 3 * i + 1, l_range=(2500, 6000), max_heads=4)     # bf16 cases
        _run_and_compare(w, seed=200 + i, fused=bool(i % 2))


def test_bf16_head_dim_64_minis_and_head_runs(force_run_len):
    # the bf16 kernels at head_dim 64 (the smaller models' heads): configurations 2 and 5 shrunk, heads halved to
    # 64 columns (zigzag pairs, one GQA group of 8, FULL + diagonal + EMPTY chunks), fused and unfused
    import dataclasses
    for idx, shrink in ((2, 32), (5, 64)):
        w = dataclasses.replace(wl.config(idx, shrink=shrink), head_dim=64, name=f"cfg{idx}_mini_d64")
        _run_and_compare(w, fused=(idx == 2))
    # forced dK/dV head runs: whole groups, runs with a remainder, non-adjacent heads of a group
    for run_len in (1, 3, 8):
        force_run_len(run_len)
        w = _custom(f"runs{run_len}_d64", "bf16", 8, 3, 64, 700, [(150, 70), (400, 300)], [[(0, 333)], [(333, 367)]],
                    kv_of_q=[0, 1, 0, 0, 2, 0, 1, 0])
        _run_and_compare(w, seed=31)


def test_bf16_head_dim_64_randomized_shards():
    rng = np.random.default_rng(64)
    for i in range(12):
        long_case = i >= 8     # the last four span many tiles per workgroup
        w = _random_case(rng, 3 * i + 1, l_range=(2500, 6000) if long_case else (200, 1400),
                         max_heads=4 if long_case else 8, d_bf16=64)
        _run_and_compare(w, seed=300 + i, fused=bool(i % 2))


@pytest.mark.parametrize("lq,lc", [(1, 1), (63, 65), (256, 129), (257, 300), (513, 1)])
def test_bf16_head_dim_64_workgroup_boundary_sizes(lq, lc):
    w = _custom(f"edge64_{lq}_{lc}", "bf16", 2, 1, 64, lc + lq, [(lc, lq)], [[(0, lc)], [(lc, lq)]])
    _run_and_compare(w, seed=lq * 1000 + lc + 64)


@pytest.mark.parametrize("run_len", [0, 1, 2])
def test_strided_inputs_and_accumulate_flags(run_len, force_run_len):
    # (also with forced dK/dV head runs: whole groups in one workgroup add to the running dk/dv without
    # atomics, split groups with them)
    force_run_len(run_len)
    # q/dO and k/v are slices of wider buffers (token and head strides larger than dense)
    w = _custom("strided", "bf16", 4, 2, 128, 512, [(128, 384)], [[(0, 256)], [(256, 256)]])
    inputs = wl.make_inputs(w, 5)
    dev = torch.device(DEV)
    lq, nq, nkv, d = w.lq, 4, 2, 128
    qbig = torch.zeros((lq, nq + 2, d + 64), dtype=torch.bfloat16, device=dev)
    gbig = torch.zeros_like(qbig)
    q, d_o = qbig[:, 1:1 + nq, 8:8 + d], gbig[:, 1:1 + nq, 8:8 + d]
    q.copy_(inputs["q"]); d_o.copy_(inputs["d_o"])
    o = torch.zeros((lq, nq, d), dtype=torch.float32, device=dev)
    lse = torch.full((nq, lq), float("-inf"), dtype=torch.float32, device=dev)
    delta = torch.empty_like(lse)
    dq = torch.zeros_like(o)
    ks, vs, descs = [], [], []
    for ch in w.chunks:
        kbig = torch.zeros((256, nkv + 1, d + 8), dtype=torch.bfloat16, device=dev)
        vbig = torch.zeros_like(kbig)
        kc, vc = kbig[:, :nkv, 8:], vbig[:, :nkv, 8:]
        kc.copy_(wl.gather_rows(inputs["k"], ch)); vc.copy_(wl.gather_rows(inputs["v"], ch))
        ks.append(kc); vs.append(vc)
        desc = hexi.desc_for(q, kc, w.scale)
        descs.append(desc)
        hexi.hexi_attn_fwd_chunk(desc, w.q_segs, ch, q, kc, vc, o, lse, flags=hexi.HEXI_ACCUMULATE)
    # dk/dv with HEXI_ACCUMULATE on pre-filled buffers: result = prefill + gradient
    dks = [torch.full((256, nkv, d), 0.5, dtype=torch.float32, device=dev) for _ in w.chunks]
    dvs = [torch.full((256, nkv, d), -0.25, dtype=torch.float32, device=dev) for _ in w.chunks]
    for j, ch in enumerate(w.chunks):
        flags = hexi.HEXI_ACCUMULATE | (hexi.HEXI_COMPUTE_DELTA if j == 0 else 0)
        hexi.hexi_attn_bwd_chunk(descs[j], w.q_segs, ch, q, ks[j], vs[j], o, d_o, lse, delta, dq, dks[j], dvs[j], flags=flags)
    torch.cuda.synchronize()
    ref = oracle_full(w, inputs)
    check("o", o.cpu(), ref["o"], "bf16")
    check("lse", lse.cpu(), ref["lse"], "bf16")
    check("dq", dq.cpu(), ref["dq"], "bf16")
    check("dk", torch.cat(dks).cpu().numpy() - 0.5, ref["dk"], "bf16")
    check("dv", torch.cat(dvs).cpu().numpy() + 0.25, ref["dv"], "bf16")


@pytest.mark.parametrize("d", [128, 64])
def test_dq_residuals_of_large_ds(d):
    # The dQ kernels add the rounding residuals of a 32-key block's dS when some |dS| >= 2.  With dO scaled by 64 (exact
    # in bf16; every gradient is linear in dO) nearly every block takes that path -- masked and unmasked tiles, ragged
    # tails -- here in the 32-row kernel; test_64_row_dq_residuals and
    # test_large_workgroups_residuals have the others -- and dq / 64 must still match the oracle, more closely than without the scaling
    # (dS carried to fp32 accuracy instead of bf16); dk and dv, which have no such path, must come out as exactly 64 x
    # their unscaled values.
    w = _custom(f"residual_{d}", "bf16", 4, 2, d, 1500, [(60, 200), (700, 777)], [[(0, 333)], [(333, 617), (950, 27)], [(977, 523)]],
                k_scale=2.0)
    inputs = wl.make_inputs(w, 41)
    ref = oracle_full(w, inputs)
    plain = replay.ShardRun(w, inputs, DEV)
    plain.step()
    scaled_inputs = dict(inputs, d_o=inputs["d_o"] * 64)
    assert torch.equal((scaled_inputs["d_o"].float() / 64).to(torch.bfloat16), inputs["d_o"])
    big = replay.ShardRun(w, scaled_inputs, DEV)
    big.step()
    torch.cuda.synchronize()
    for j in range(len(w.chunks)):
        assert torch.equal(big.dk[j], plain.dk[j] * 64) and torch.equal(big.dv[j], plain.dv[j] * 64)
    assert torch.equal(big.o, plain.o) and torch.equal(big.lse, plain.lse)
    e_plain, _ = check("dq", plain.dq.cpu(), ref["dq"], "bf16")
    e_big, _ = check("dq with residuals everywhere", (big.dq / 64).cpu(), ref["dq"], "bf16")
    frac = float((big.dq / 64 != plain.dq).float().mean())
    print(f"    dq elements changed by the residual path: {100 * frac:.1f} %", flush=True)
    assert frac > 0.5 and e_big <= e_plain


def test_future_chunk_and_merge_outputs():
    dev = torch.device(DEV)
    w = _custom("future", "bf16", 2, 1, 128, 512, [(0, 128)], [[(256, 256)]])
    inputs = wl.make_inputs(w, 3)
    q, d_o = inputs["q"].to(dev), inputs["d_o"].to(dev)
    kc = wl.gather_rows(inputs["k"], w.chunks[0]).to(dev)
    vc = wl.gather_rows(inputs["v"], w.chunks[0]).to(dev)
    desc = hexi.desc_for(q, kc, w.scale)
    o = torch.full((128, 2, 128), 9.0, dtype=torch.float32, device=dev)
    lse = torch.full((2, 128), 9.0, dtype=torch.float32, device=dev)
    hexi.hexi_attn_fwd_chunk(desc, w.q_segs, w.chunks[0], q, kc, vc, o, lse)
    assert torch.all(o == 0) and torch.all(lse == float("-inf"))
    o.fill_(1.5); lse.fill_(0.25)
    hexi.hexi_attn_fwd_chunk(desc, w.q_segs, w.chunks[0], q, kc, vc, o, lse, flags=hexi.HEXI_ACCUMULATE)
    assert torch.all(o == 1.5) and torch.all(lse == 0.25)
    dq = torch.zeros_like(o)
    dk = torch.full((256, 1, 128), 3.0, dtype=torch.float32, device=dev)
    dv = torch.full_like(dk, 3.0)
    delta = torch.zeros_like(lse)
    hexi.hexi_attn_bwd_chunk(desc, w.q_segs, w.chunks[0], q, kc, vc, o, d_o, lse, delta, dq, dk, dv)
    assert torch.all(dk == 0) and torch.all(dv == 0) and torch.all(dq == 0)
    # merge: -inf identities, bf16 and fp32 o_final, against the oracle's merge
    g = torch.Generator().manual_seed(1)
    o_a = torch.randn((300, 3, 128), generator=g); o_b = torch.randn((300, 3, 128), generator=g)
    l_a = torch.randn((3, 300), generator=g) * 4; l_b = torch.randn((3, 300), generator=g) * 4
    l_a[0, :10] = float("-inf"); l_b[1, 5:20] = float("-inf"); l_b[0, :5] = float("-inf")
    o_a[0:10, 0] = 0; o_b[5:20, 1] = 0; o_b[0:5, 0] = 0
    o_ref, l_ref = oracle.merge(to64(o_a), to64(l_a), to64(o_b), to64(l_b))
    for fdt in (None, torch.float32, torch.bfloat16):
        oa, la = o_a.to(dev), l_a.to(dev)
        fin = None if fdt is None else torch.empty((300, 3, 128), dtype=fdt, device=dev)
        hexi.hexi_attn_merge_lse(oa, la, o_b.to(dev), l_b.to(dev), o_final=fin)
        check("merge.o", oa.cpu(), o_ref, "f32")
        check("merge.lse", la.cpu(), l_ref, "f32")
        if fdt is torch.float32:
            assert torch.equal(fin, oa)
        if fdt is torch.bfloat16:
            assert torch.equal(fin, oa.to(torch.bfloat16))


def test_backward_halves_and_dq_reproducible():
    # HEXI_SKIP_DQ / HEXI_SKIP_DKDV run the two halves of the step separately; together they equal the full
    # call.  dq (bf16 path) has a fixed summation order: bit-identical between runs.
    w = wl.config(3, shrink=32)
    inputs = wl.make_inputs(w)
    run = replay.ShardRun(w, inputs, DEV)
    run.step(); torch.cuda.synchronize()
    dq_full = run.dq.clone()
    dk_full = [x.clone() for x in run.dk]
    run.dq.zero_()
    for j, ch in enumerate(w.chunks):
        run.dk[j].fill_(7.0); run.dv[j].fill_(7.0)
        hexi.hexi_attn_bwd_chunk(run.desc[j], w.q_segs, ch, run.q, run.k[j], run.v[j], run.o, run.d_o, run.lse, run.delta,
                                 run.dq, None, None, flags=hexi.HEXI_SKIP_DKDV)
    torch.cuda.synchronize()
    assert torch.equal(run.dq, dq_full)
    assert all(torch.all(x == 7.0) for x in run.dk)
    dq_before = run.dq.clone()
    for j, ch in enumerate(w.chunks):
        hexi.hexi_attn_bwd_chunk(run.desc[j], w.q_segs, ch, run.q, run.k[j], run.v[j], run.o, run.d_o, run.lse, run.delta,
                                 None, run.dk[j], run.dv[j], flags=hexi.HEXI_SKIP_DQ)
    torch.cuda.synchronize()
    assert torch.equal(run.dq, dq_before)
    for a, b in zip(run.dk, dk_full):
        assert torch.allclose(a, b, rtol=1e-4, atol=1e-5)
    with pytest.raises(hexi.HexiError) as e:
        hexi.hexi_attn_bwd_chunk(run.desc[0], w.q_segs, w.chunks[0], run.q, run.k[0], run.v[0], run.o, run.d_o, run.lse,
                                 run.delta, run.dq, run.dk[0], run.dv[0], flags=hexi.HEXI_SKIP_DQ | hexi.HEXI_SKIP_DKDV)
    assert e.value.code == hexi.HEXI_EINVAL


def test_dkdv_reproducible_when_a_workgroup_sums_the_whole_group(force_run_len):
    # whole-group head runs use plain stores and a fixed summation order: dk / dv are bit-identical between runs
    # (runs that split a group add with floating-point atomics, whose order may vary)
    w = wl.config(2, shrink=16)
    inputs = wl.make_inputs(w)
    run = replay.ShardRun(w, inputs, DEV)
    run.forward()
    force_run_len(w.n_q_heads // w.n_kv_heads)
    run.backward(); torch.cuda.synchronize()
    first = [(a.clone(), b.clone()) for a, b in zip(run.dk, run.dv)]
    for a, b in zip(run.dk, run.dv):
        a.fill_(float("nan")); b.fill_(float("nan"))
    run.backward(); torch.cuda.synchronize()
    for (a0, b0), a1, b1 in zip(first, run.dk, run.dv):
        assert torch.equal(a0, a1) and torch.equal(b0, b1)


@pytest.mark.parametrize("step,run_len,run_len_alone", ORDER_STEPS)
def test_dkdv_reproducible_in_whole_and_in_half_groups(step, run_len, run_len_alone):
    # the shapes that the library chooses by itself (asserted on the CPU): the same bits in every call for the step, and in every one for dK / dV
    # alone where its sums have a fixed order
    lq, lc, nq, nkv, d, off = step
    q, d_o, k, v = _large_step_inputs(lq, lc, nq, nkv, d, lq + lc)
    qd, gd, kd, vd = (t.to(DEV) for t in (q, d_o, k, v))
    desc, args = hexi.desc_for(qd, kd, d ** -0.5), ([(off, lq)], [(0, lc)], qd, kd, vd)
    o, lse, delta, dq = (torch.zeros(s, device=DEV) for s in (q.shape, (nq, lq), (nq, lq), q.shape))
    hexi.hexi_attn_fwd_chunk(desc, *args, o, lse)
    outs = {0: [], hexi.HEXI_SKIP_DQ: []}
    for flags in (hexi.HEXI_COMPUTE_DELTA, 0, hexi.HEXI_SKIP_DQ, hexi.HEXI_SKIP_DQ, 0, hexi.HEXI_SKIP_DQ):
        dk, dv = torch.full(k.shape, float("nan"), device=DEV), torch.full(v.shape, float("nan"), device=DEV)
        hexi.hexi_attn_bwd_chunk(desc, *args, o, gd, lse, delta, dq, dk, dv, flags=flags)
        outs[flags & hexi.HEXI_SKIP_DQ].append((dk, dv))
    for alone, calls in outs.items():
        assert all(bool(torch.isfinite(t).all()) for c in calls for t in c)
        if 2 * (run_len_alone if alone else run_len) >= nq // nkv:
            assert all(torch.equal(dk, calls[0][0]) and torch.equal(dv, calls[0][1]) for dk, dv in calls)


def test_forward_is_deterministic():
    w = wl.config(3, shrink=32)
    inputs = wl.make_inputs(w)
    run = replay.ShardRun(w, inputs, DEV)
    run.forward(); torch.cuda.synchronize()
    o1, l1 = run.o.clone(), run.lse.clone()
    run.forward(); torch.cuda.synchronize()
    assert torch.equal(o1, run.o) and torch.equal(l1, run.lse)


@pytest.mark.parametrize("lq,lc", [(1, 1), (63, 65), (255, 64), (256, 129), (257, 300), (600, 192), (513, 1)])
def test_workgroup_boundary_sizes(lq, lc):
    # shard / chunk lengths just below, at and above multiples of 32, 64, 128 and 256 rows and keys, a single row, a single
    # key; two chunks so that the second is diagonal (launches this small take 32- and 64-row workgroups; the 256-row
    # ones: test_large_workgroups_boundary_sizes)
    l_tot = lc + lq
    q_segs = [(lc, lq)]
    chunks = [[(0, lc)], [(lc, lq)]]
    w = _custom(f"edge_{lq}_{lc}", "bf16", 2, 1, 128, l_tot, q_segs, chunks)
    _run_and_compare(w, seed=lq * 1000 + lc)


@pytest.mark.parametrize("d", [128, 64])
def test_forward_exact_softmax_fallback(d):
    # Scores that leave the range of a fixed softmax reference: keys beyond the first 64 are scaled so that later scores
    # exceed the earlier maximum by far more than 2^100, and a second shard does the reverse (the first keys huge, the rest
    # tiny).  A launch this small runs the kernel with a running maximum per wavefront, whose parts differ by those
    # factors when they are combined; the 256-row kernel's fallback: test_large_workgroups_softmax_fallback.
    dev = torch.device(DEV)
    g = torch.Generator().manual_seed(99)
    lq, lc, nq = 300, 640, 2
    for first_scale, later_scale in ((1.0, 60.0), (60.0, 0.02)):
        q = (torch.randn((lq, nq, d), generator=g) * 3).to(torch.bfloat16)
        k = torch.randn((lc, 1, d), generator=g)
        k[:64] *= first_scale
        k[64:] *= later_scale
        k = k.to(torch.bfloat16)
        v = torch.randn((lc, 1, d), generator=g).to(torch.bfloat16)
        scale = d ** -0.5
        qd, kd, vd = q.to(dev), k.to(dev), v.to(dev)
        o = torch.zeros((lq, nq, d), dtype=torch.float32, device=dev)
        lse = torch.full((nq, lq), float("-inf"), dtype=torch.float32, device=dev)
        q_segs, kv_segs = [(lc, lq)], [(0, lc)]
        hexi.hexi_attn_fwd_chunk(hexi.desc_for(qd, kd, scale), q_segs, kv_segs, qd, kd, vd, o, lse)
        torch.cuda.synchronize()
        o_ref, lse_ref = oracle.attn_fwd(to64(q), np.arange(lc, lc + lq), to64(k), to64(v), np.arange(lc), scale)
        spread = float(np.max(lse_ref) - np.min(lse_ref))
        print(f"  scales {first_scale}/{later_scale}: lse range {np.min(lse_ref):.1f} .. {np.max(lse_ref):.1f}", flush=True)
        assert spread > 50.0     # the case really spans a wide range
        check("o", o.cpu(), o_ref, "bf16")
        check("lse", lse.cpu(), lse_ref, "bf16")     # values in the hundreds, still inside the flat bound


def test_device_share_of_a_scheduled_plan():
    # host scheduler -> shard descriptor -> attention kernels: with 3 heads on two fast + two slow devices the
    # plan is two node groups of uneven length with uneven head counts; one device per group runs its share
    # (its group's block, its head range, which cuts through a GQA group; the ring's blocks in order, the
    # later group's block lying in the first group's future) against the oracle
    import sys, os
    sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
    from sched_util import cluster_arrays, model_args
    arr = cluster_arrays([("h100", 2), ("a800", 2)])
    plan = hexi.hexi_sched_solve(arr, model_args(l_tot=4096, n_heads=3, hidden=384), token_quantum=64, m2=4, i_max=20)
    print("\nplan:", plan)
    assert plan["groups"] == [[0, 1], [2, 3]] and sum(plan["l_group"]) == 4096 and plan["l_group"][0] != plan["l_group"][1]
    for dev in (1, 2):
        w = wl.from_schedule(plan["groups"], plan["l_group"], plan["n_heads"], dev, head_dim=128, q_per_kv=2)
        assert w.n_q_heads == plan["n_heads"][dev] and len(w.chunks) == 2
        _run_and_compare(w, seed=31 + dev)


def test_measured_compute_rate_feeds_the_scheduler():
    # c_d of the cost model (Eq. 11 convention: 16 * Lq * Lc * n_d * d_h flop per fully visible step) measured on
    # this GPU through the library's own kernels, then used as the compute rate of a homogeneous 8-device plan
    import sys, os
    sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
    from sched_util import cluster_arrays, model_args
    from paper_2605_07569_amd import calibrate
    c_d = calibrate.measure_c_d(lq=4096, lc=4096, reps=3)
    print(f"\n  measured c_d = {c_d / 1e12:.0f} TFLOP/s (Eq. 11 convention)", flush=True)
    # 14/16 of it is the counted rate on unmasked pairs: between a tenth of and the whole bf16 MFMA roof
    assert 0.25e15 < c_d < 2.9e15
    arr = cluster_arrays([("h100", 8)])
    arr["c"] = np.full(8, c_d)
    model = model_args(l_tot=65536, n_heads=32, hidden=4096)
    plan = hexi.hexi_sched_solve(arr, model, m2=4, i_max=10)
    assert sum(plan["l_group"]) == 65536 and all(sum(plan["n_heads"][d] for d in g) == 32 for g in plan["groups"])
    t_blk, t_non, t_a2a, t_ring, feasible = hexi.hexi_sched_cost(arr, model, plan["groups"], plan["l_group"], plan["s_pre"], plan["n_heads"])
    assert feasible and abs(t_blk - plan["cost"]) <= 1e-12 * t_blk
    # a slower device rate can only raise the modelled ring time
    arr_slow = dict(arr, c=np.full(8, c_d / 4))
    assert hexi.hexi_sched_cost(arr_slow, model, plan["groups"], plan["l_group"], plan["s_pre"], plan["n_heads"])[3] >= t_ring


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("nq,nkv,lq,lc", [(2, 1, 1, 1), (2, 2, 15, 17), (3, 1, 16, 128), (2, 1, 17, 129), (2, 1, 129, 15), (4, 2, 300, 257), (16, 16, 1000, 1010), (64, 32, 199, 16), (96, 48, 16, 266)])
def test_f32_workgroup_shapes(nq, nkv, lq, lc, d):
    # lengths at the edges of the fp32 kernels' 16-row blocks and 128-row (split) / 32-row (shared) tiles; 1000 rows are dealt to the split-operand
    # kernels at head_dim 128 and to two split workgroups a CU at 64, at 128 the forward and dQ of 199 rows and dK / dV of 266 keys are shared, the others
    # split.  The second chunk is diagonal.
    w = _custom(f"f32_{nq}_{lq}_{lc}_{d}", "f32", nq, nkv, d, lc + lq, [(lc, lq)], [[(0, lc)], [(lc, lq)]])
    run, inputs, ref = _run_and_compare(w, seed=lq * 1000 + lc + d)
    # dk / dv under HEXI_ACCUMULATE: the running value plus the gradient; dq_acc adds up over calls
    for j, ch in enumerate(w.chunks):
        dk, dv, dq = torch.full_like(run.dk[j], 0.5), torch.full_like(run.dv[j], -0.25), torch.full_like(run.dq, 1.0)
        hexi.hexi_attn_bwd_chunk(run.desc[j], w.q_segs, ch, run.q, run.k[j], run.v[j], None, run.d_o, run.lse, run.delta, dq, dk, dv,
                                 flags=hexi.HEXI_ACCUMULATE)
        check("dk acc", dk.cpu(), chunk_slices(w, j, ref["dk"], ref["n_keys"]) + 0.5, "f32")
        check("dv acc", dv.cpu(), chunk_slices(w, j, ref["dv"], ref["n_keys"]) - 0.25, "f32")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("nq,nkv,lq,lc", [(2, 2, 31, 33), (3, 1, 32, 64), (2, 1, 95, 257), (24, 8, 500, 1000), (8, 1, 600, 600)])
def test_bf16_split_workgroup_shapes(nq, nkv, lq, lc, d):
    # lengths around the 32-row blocks of the kernels for small launches, fewer and more of them than a workgroup has
    # wavefronts; at head_dim 128 the fourth size takes 64-row workgroups instead, the last one cuts its group of
    # heads into runs that add their dk / dv.  The second chunk is diagonal and in two segments.
    w = _custom(f"split_{nq}_{lq}_{lc}_{d}", "bf16", nq, nkv, d, lc + lq + 7, [(lc, lq // 2), (lc + lq // 2 + 7, lq - lq // 2)],
                [[(0, lc)], [(lc, lq // 2 + 7), (lc + lq // 2 + 7, lq - lq // 2)]])
    run, inputs, ref = _run_and_compare(w, seed=lq * 1000 + lc + d)
    # dk / dv under HEXI_ACCUMULATE: the running value plus the gradient
    for j, ch in enumerate(w.chunks):
        dk, dv, dq = torch.full_like(run.dk[j], 0.5), torch.full_like(run.dv[j], -0.25), torch.zeros_like(run.dq)
        hexi.hexi_attn_bwd_chunk(run.desc[j], w.q_segs, ch, run.q, run.k[j], run.v[j], None, run.d_o, run.lse, run.delta, dq, dk, dv,
                                 flags=hexi.HEXI_ACCUMULATE)
        check("dk acc", dk.cpu(), chunk_slices(w, j, ref["dk"], ref["n_keys"]) + 0.5, "bf16")
        check("dv acc", dv.cpu(), chunk_slices(w, j, ref["dv"], ref["n_keys"]) - 0.25, "bf16")


def _exact_ds_case(lq, lc, nq, nkv, d, seed):
    """Inputs whose every step is exact in fp32: Q = 0 and LSE = 0 make P = 1, Delta = 0, and dP is an integer of up to 24
    bits (dO holds its bytes, V picks three of them; 16 columns apart, so that each is the only product of its matrix
    instruction), so dS = dP; key j < d is the unit vector e_j: column j of dq is scale * dS_ij, with scale a power of two."""
    g = torch.Generator().manual_seed(seed)
    q = torch.zeros((lq, nq, d))
    byte = torch.randint(0, 256, (lq, nq, 3, 3), generator=g).double()      # [..., byte, choice]
    byte[..., 0, :] = byte[..., 0, :].clamp(min=1.0)
    sign = (1 - 2 * torch.randint(0, 2, (lq, nq, 1, 1), generator=g)).double()
    byte = byte * sign * torch.tensor([65536.0, 256.0, 1.0], dtype=torch.float64)[:, None]
    d_o = torch.zeros((lq, nq, d), dtype=torch.float64)
    for n in range(3):
        d_o[..., 16 * n:16 * n + 3] = byte[..., n, :]
    k, v = torch.zeros((lc, nkv, d)), torch.zeros((lc, nkv, d))
    n = min(lc, d)
    k[torch.arange(n), :, torch.arange(n)] = 1.0
    for j in range(lc):
        v[j, :, j % 3:48:16] = 1.0
    q_segs = [(lc // 2, lq)]
    visible = torch.arange(n)[None, :] <= torch.arange(lc // 2, lc // 2 + lq)[:, None]
    want = torch.zeros((lq, nq, d), dtype=torch.float64)
    want[..., :n] = 0.125 * byte.sum(2)[..., torch.arange(n) % 3] * visible[:, None, :]
    b16 = lambda t: t.to(torch.bfloat16).to(DEV)
    return b16(q), b16(d_o), b16(k), b16(v), q_segs, want


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("lq,lc,nq,nkv", [(1, 1, 1, 1), (40, 100, 2, 1), (300, 700, 4, 2), (512, 1000, 24, 8), (300, 2100, 128, 8),
                                          (1024, 320, 64, 64), (1024, 385, 64, 4),      # 256-row workgroups
                                          (130, 700, 64, 16), (315, 132, 32, 32)])      # 64-row ones at head_dim 128 and 64
def test_large_ds_reaches_dq_unrounded(lq, lc, nq, nkv, d):
    # a dS of 24 significant bits must come out of the dQ kernels bit for bit (a residual rounded to bf16 loses up to
    # 2^-18 of it)
    q, d_o, k, v, q_segs, want = _exact_ds_case(lq, lc, nq, nkv, d, lq + lc + d)
    kv_segs = [(0, lc)]
    lse, delta = torch.zeros((nq, lq), device=DEV), torch.zeros((nq, lq), device=DEV)
    dq = torch.zeros((lq, nq, d), device=DEV)
    print(f"\n  exact dS: {lq} x {lc} x {nq}/{nkv} x {d}", flush=True)
    hexi.hexi_attn_bwd_chunk(hexi.desc_for(q, k, 0.125), q_segs, kv_segs, q, k, v, None, d_o, lse, delta, dq, None, None,
                             flags=hexi.HEXI_SKIP_DKDV)
    torch.cuda.synchronize()
    got = dq.cpu().double()
    wrong = int((got != want).sum())
    assert wrong == 0, (wrong, float(((got - want).abs() / want.abs().clamp(min=1.0)).max()))


def _bwd_reference(q, k, v, d_o, q_pos, kv_pos, lse, delta, scale, group):
    """dq, dk, dv in float64 from the given LSE [nq, lq] and Delta; P = 0 where the LSE is infinite.  Heads h read kv head h // group."""
    q, k, v, d_o = (t.double() for t in (q, k, v, d_o))
    nkv = k.shape[1]
    kk, vv = k.repeat_interleave(group, 1), v.repeat_interleave(group, 1)
    s = torch.matmul(q.permute(1, 0, 2), kk.permute(1, 2, 0).contiguous()) * scale
    dead = ~torch.isfinite(lse)
    p = torch.exp(s - torch.where(dead, torch.zeros_like(lse), lse).double()[..., None])
    p = torch.where(dead[..., None] | (kv_pos[None, None, :] > q_pos[None, :, None]), torch.zeros_like(p), p)
    dp = torch.matmul(d_o.permute(1, 0, 2), vv.permute(1, 2, 0).contiguous())
    ds = p * (dp - delta.double()[..., None])
    dq = scale * torch.matmul(ds, kk.permute(1, 0, 2).contiguous()).permute(1, 0, 2)
    per_kv = lambda t: t.permute(1, 0, 2).reshape(k.shape[0], nkv, group, -1).sum(2)
    dk = scale * per_kv(torch.matmul(ds.transpose(1, 2).contiguous(), q.permute(1, 0, 2).contiguous()))
    return dq, dk, per_kv(torch.matmul(p.transpose(1, 2).contiguous(), d_o.permute(1, 0, 2).contiguous()))


def _infinite_lse_case(dtype, lq, lc, nq, nkv, d, dead):
    """One chunk, every row of which sees keys; LSE is `dead` on a third of the rows, on whole and on partial row blocks."""
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    g = torch.Generator().manual_seed(lq + 31 * lc + d)
    rnd = lambda *s: torch.randn(s, generator=g).to(dt)
    q, d_o, k, v = rnd(lq, nq, d), rnd(lq, nq, d), rnd(lc, nkv, d), rnd(lc, nkv, d)
    q_pos, kv_pos = torch.arange(lc // 2, lc // 2 + lq), torch.arange(lc)
    scale = d ** -0.5
    s = torch.matmul(q.double().permute(1, 0, 2), k.double().repeat_interleave(nq // nkv, 1).permute(1, 2, 0).contiguous()) * scale
    lse = torch.logsumexp(torch.where(kv_pos[None, None, :] > q_pos[None, :, None], torch.full_like(s, -float("inf")), s), 2).float()
    delta = torch.randn((nq, lq), generator=g) * 0.1
    lse[:, ::7] = dead
    lse[:, lq // 2:lq // 2 + lq // 5 + 1] = dead
    ref = _bwd_reference(q, k, v, d_o, q_pos, kv_pos, lse, delta, scale, nq // nkv)
    dev = [t.to(DEV) for t in (q, k, v, d_o, lse, delta)]
    return dev, [(lc // 2, lq)], [(0, lc)], scale, ref


@pytest.mark.parametrize("dead", [-float("inf"), float("inf")])
@pytest.mark.parametrize("lq,lc,nq,nkv,d", [(70, 100, 2, 1, 128), (70, 100, 2, 1, 64), (512, 1000, 24, 8, 128), (512, 1000, 24, 8, 64)] + QUAD_DQ_STEPS)
def test_bf16_dq_of_rows_with_an_infinite_lse(lq, lc, nq, nkv, d, dead):
    # a row switched off through its LSE contributes nothing, whether or not it sees keys
    (q, k, v, d_o, lse, delta), qs, ks, scale, ref = _infinite_lse_case("bf16", lq, lc, nq, nkv, d, dead)
    dq = torch.zeros((lq, nq, d), device=DEV)
    print(f"\n  infinite LSE: bf16 {lq} x {lc} x {nq}/{nkv} x {d}", flush=True)
    hexi.hexi_attn_bwd_chunk(hexi.desc_for(q, k, scale), qs, ks, q, k, v, None, d_o, lse, delta, dq, None, None, flags=hexi.HEXI_SKIP_DKDV)
    check("dq", dq.cpu(), ref[0], "bf16")
    assert torch.all(dq.permute(1, 0, 2)[~torch.isfinite(lse)] == 0)


# fp32 steps in every shape at head_dim 128 and in the split-operand kernels (asserted on the CPU), rows from the middle of the keys
F32_MIDDLE_SIZES = [s + (128,) for s, *_ in F32_128_STEPS[:5]] + [s for s, _ in F32X3_MIDDLE_STEPS]


@pytest.mark.parametrize("dead", [-float("inf"), float("inf")])
@pytest.mark.parametrize("lq,lc,nq,nkv,d", [(70, 100, 2, 1, 128), (70, 100, 2, 1, 64), (1000, 1010, 16, 16, 128), (1000, 1010, 16, 16, 64)] + F32_MIDDLE_SIZES)
def test_f32_backward_of_rows_with_an_infinite_lse(lq, lc, nq, nkv, d, dead):
    # the same in fp32, in every workgroup shape of the 16-row kernels and in the split-operand ones, dk and dv included
    (q, k, v, d_o, lse, delta), qs, ks, scale, ref = _infinite_lse_case("f32", lq, lc, nq, nkv, d, dead)
    dq, dk, dv = torch.zeros((lq, nq, d), device=DEV), torch.empty((lc, nkv, d), device=DEV), torch.empty((lc, nkv, d), device=DEV)
    print(f"\n  infinite LSE: f32 {lq} x {lc} x {nq}/{nkv} x {d}", flush=True)
    hexi.hexi_attn_bwd_chunk(hexi.desc_for(q, k, scale), qs, ks, q, k, v, None, d_o, lse, delta, dq, dk, dv)
    for name, got, want in zip(("dq", "dk", "dv"), (dq, dk, dv), ref):
        check(name, got.cpu(), want, "f32")
    assert torch.all(dq.permute(1, 0, 2)[~torch.isfinite(lse)] == 0)


@pytest.mark.parametrize("scale", [64 ** -0.5, 128 ** -0.5, 0.1, 0.05, 1.0])
@pytest.mark.parametrize("lq,lc,nq,nkv,d", [(70, 100, 2, 1, 128), (70, 100, 2, 1, 64), (1000, 1010, 16, 16, 128), (1000, 1010, 16, 16, 64)] + F32_MIDDLE_SIZES)
def test_f32_scores_that_overflow_downwards(lq, lc, nq, nkv, d, scale):
    # every seventh key's score is -1e40, i.e. -inf in fp32: the key weighs nothing, forward and backward, whatever the sign of
    # the low half of scale * log2(e)
    g = torch.Generator().manual_seed(lq + d)
    q, d_o = torch.randn((lq, nq, d), generator=g), torch.randn((lq, nq, d), generator=g)
    k, v = torch.randn((lc, nkv, d), generator=g), torch.randn((lc, nkv, d), generator=g)
    q[..., 0] = 1e20
    k[..., 0] = 0.0
    k[3::7, :, 0] = -1e20
    qs, ks = [(lc // 2, lq)], [(0, lc)]
    run = {n: t.to(DEV) for n, t in dict(q=q, k=k, v=v, d_o=d_o).items()}
    o, lse, delta = torch.empty((lq, nq, d), device=DEV), torch.empty((nq, lq), device=DEV), torch.empty((nq, lq), device=DEV)
    dq, dk, dv = torch.zeros((lq, nq, d), device=DEV), torch.empty((lc, nkv, d), device=DEV), torch.empty((lc, nkv, d), device=DEV)
    desc = hexi.desc_for(run["q"], run["k"], scale)
    hexi.hexi_attn_fwd_chunk(desc, qs, ks, run["q"], run["k"], run["v"], o, lse)
    hexi.hexi_attn_bwd_chunk(desc, qs, ks, run["q"], run["k"], run["v"], o, run["d_o"], lse, delta, dq, dk, dv, flags=hexi.HEXI_COMPUTE_DELTA)
    got = [t.cpu() for t in (o, lse, dq, dk, dv)]
    # the reference: without those keys (Q's first column meets zeros only)
    keep = torch.tensor([j for j in range(lc) if j % 7 != 3])
    s32 = float(np.float32(scale))
    o_ref, lse_ref = oracle.attn_fwd(to64(q), np.arange(lc // 2, lc // 2 + lq), to64(k[keep]), to64(v[keep]), keep.numpy(), s32)
    ref = oracle.attn_bwd(to64(q), np.arange(lc // 2, lc // 2 + lq), to64(k[keep]), to64(v[keep]), keep.numpy(), to64(d_o), s32)
    check("o", got[0], o_ref, "f32")
    check("lse", got[1], lse_ref, "f32")
    check("dq", got[2], ref["dq"], "f32")
    # (column 0 of dk holds sums of 1e20-sized terms; the others are ordinary)
    check("dk", got[3][keep][..., 1:], ref["dk"][..., 1:], "f32")
    check("dv", got[4][keep], ref["dv"], "f32")
    drop = torch.tensor([j for j in range(lc) if j % 7 == 3])
    assert torch.all(got[3][drop] == 0) and torch.all(got[4][drop] == 0)


@pytest.mark.parametrize("nq,nkv,lq,d", [(4, 2, 200, 128), (4, 4, 333, 64), (16, 16, 1000, 64)])
def test_f32_dq_of_chunks_on_two_streams(nq, nkv, lq, d):
    # chunks of one shard may add to the same dq from several streams in fp32, in both workgroup shapes
    n_chunks, lc = 8, 150
    w = _custom(f"streams_{nq}_{lq}_{d}", "f32", nq, nkv, d, n_chunks * lc + lq, [(n_chunks * lc, lq)],
                [[(j * lc, lc)] for j in range(n_chunks)] + [[(n_chunks * lc, lq)]])
    run, inputs, ref = _run_and_compare(w, seed=lq + d)
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    run.dq.zero_()
    torch.cuda.synchronize()
    for j, ch in enumerate(w.chunks):
        hexi.hexi_attn_bwd_chunk(run.desc[j], w.q_segs, ch, run.q, run.k[j], run.v[j], None, run.d_o, run.lse, run.delta, run.dq,
                                 run.dk[j], run.dv[j], stream=streams[j % 2].cuda_stream)
    torch.cuda.synchronize()
    check("dq", run.dq.cpu(), ref["dq"], "f32")


def _large_step_inputs(lq, lc, nq, nkv, d, seed, k_scale=1.0):
    g = torch.Generator().manual_seed(seed)
    rnd = lambda *s: torch.randn(s, generator=g)
    q, d_o, v = rnd(lq, nq, d), rnd(lq, nq, d), rnd(lc, nkv, d)
    return [t.to(torch.bfloat16) for t in (q, d_o, rnd(lc, nkv, d) * k_scale, v)]


def _large_backward(q, k, v, d_o, o, lse, q_segs, kv_segs, scale, kv_of_q=None, delta=None):
    """dq, dk, dv of one step, the halves in calls of their own (dq in 256-row workgroups)."""
    desc = hexi.desc_for(q, k, scale, kv_of_q)
    flags = hexi.HEXI_COMPUTE_DELTA if delta is None else 0
    delta = torch.empty_like(lse) if delta is None else delta
    dq = torch.zeros(q.shape, dtype=torch.float32, device=DEV)
    dk, dv = torch.empty(k.shape, dtype=torch.float32, device=DEV), torch.empty(k.shape, dtype=torch.float32, device=DEV)
    hexi.hexi_attn_bwd_chunk(desc, q_segs, kv_segs, q, k, v, o, d_o, lse, delta, dq, None, None, flags=flags | hexi.HEXI_SKIP_DKDV)
    hexi.hexi_attn_bwd_chunk(desc, q_segs, kv_segs, q, k, v, None, d_o, lse, delta, None, dk, dv, flags=hexi.HEXI_SKIP_DQ)
    return dq, dk, dv


@pytest.mark.parametrize("lq,lc,nq,nkv,d", LARGE_STEPS)
@pytest.mark.parametrize("diagonal", [False, True])
def test_large_workgroups_boundary_sizes(lq, lc, nq, nkv, d, diagonal):
    # 256-row workgroups: last q tiles of 1, 32 and 255 rows and whole ones; 1, 64, 65, ... keys; fully and partly visible
    off = lc // 2 if diagonal else lc
    print(f"\n  large step: {lq} x {lc} x {nq}/{nkv} x {d} at {off}", flush=True)
    q, d_o, k, v = _large_step_inputs(lq, lc, nq, nkv, d, lq + lc)
    qd, gd, kd, vd = (t.to(DEV) for t in (q, d_o, k, v))
    o, lse = torch.empty(q.shape, dtype=torch.float32, device=DEV), torch.empty((nq, lq), device=DEV)
    q_segs, kv_segs, scale = [(off, lq)], [(0, lc)], d ** -0.5
    hexi.hexi_attn_fwd_chunk(hexi.desc_for(qd, kd, scale), q_segs, kv_segs, qd, kd, vd, o, lse)
    dq, dk, dv = _large_backward(qd, kd, vd, gd, o, lse, q_segs, kv_segs, scale)
    q_pos = np.arange(off, off + lq)
    o_ref, lse_ref = oracle.attn_fwd(to64(q), q_pos, to64(k), to64(v), np.arange(lc), scale)
    ref = oracle.attn_bwd(to64(q), q_pos, to64(k), to64(v), np.arange(lc), to64(d_o), scale)
    for name, got, want in (("o", o, o_ref), ("lse", lse, lse_ref), ("dq", dq, ref["dq"]), ("dk", dk, ref["dk"]), ("dv", dv, ref["dv"])):
        # (a key seen by few rows among 64 heads has gradients of several units: the bf16 bound on a single element is relative there)
        check(name, got.cpu(), want, "bf16", abs_factor=max(1.0, float(np.max(np.abs(want))) / 8) if name in ("dk", "dv") else 1.0)


@pytest.mark.parametrize("d,run_len", [(64, 0), (64, 3), (128, 0), (128, 16)])
def test_large_workgroups_segments_strides_and_head_map(d, run_len, force_run_len):
    # strided q / dO and k / v, three-segment shard, chunks with holes and diagonal parts, accumulated o / lse / dq, dk / dv
    # under HEXI_ACCUMULATE; dK / dV in the launcher's shape and in 128-key workgroups walking whole groups or runs with a remainder
    force_run_len(run_len)
    _segments_strides_and_head_map(LARGE_SHARD, d, run_len, together=False)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("together", [False, True])
def test_64_wide_workgroups_segments_strides_and_head_map(d, together):
    # the same in workgroups of 64 rows and keys, the halves of a backward step in one launch too
    _segments_strides_and_head_map(QUAD_SHARD, d, 0, together)


def _segments_strides_and_head_map(s, d, run_len, together):
    nq, nkv, q_segs, kv_of_q, scale = s["nq"], s["nkv"], s["q_segs"], s["kv_of_q"], d ** -0.5
    print(f"\n  shard of {nq}/{nkv} heads: d={d} run_len={run_len} together={together}", flush=True)
    g = torch.Generator().manual_seed(d + run_len)
    rnd = lambda *x: torch.randn(x, generator=g).to(torch.bfloat16)
    q_pos = np.concatenate([np.arange(a, a + n) for a, n in q_segs])
    kv_pos = [np.concatenate([np.arange(a, a + n) for a, n in ch]) for ch in s["chunks"]]
    lq = len(q_pos)
    q, d_o = rnd(lq, nq, d), rnd(lq, nq, d)
    ks, vs = [rnd(len(p), nkv, d) for p in kv_pos], [rnd(len(p), nkv, d) for p in kv_pos]

    def strided(t):
        big = torch.zeros((t.shape[0], t.shape[1] + 1, t.shape[2] + 8), dtype=t.dtype, device=DEV)
        big[:, :-1, 8:] = t.to(DEV)
        return big[:, :-1, 8:]

    qd, gd, kd, vd = strided(q), strided(d_o), [strided(t) for t in ks], [strided(t) for t in vs]
    o, lse = torch.zeros((lq, nq, d), device=DEV), torch.full((nq, lq), -float("inf"), device=DEV)
    delta, dq = torch.empty((nq, lq), device=DEV), torch.zeros((lq, nq, d), device=DEV)
    desc = [hexi.desc_for(qd, t, scale, kv_of_q) for t in kd]
    for j, ch in enumerate(s["chunks"]):
        hexi.hexi_attn_fwd_chunk(desc[j], q_segs, ch, qd, kd[j], vd[j], o, lse, flags=hexi.HEXI_ACCUMULATE)
    dk, dv = [torch.full(t.shape, 0.5, device=DEV) for t in ks], [torch.full(t.shape, -0.25, device=DEV) for t in ks]
    for j, ch in enumerate(s["chunks"]):
        if together:
            hexi.hexi_attn_bwd_chunk(desc[j], q_segs, ch, qd, kd[j], vd[j], o, gd, lse, delta, dq, dk[j], dv[j],
                                     flags=hexi.HEXI_ACCUMULATE | (hexi.HEXI_COMPUTE_DELTA if j == 0 else 0))
            continue
        hexi.hexi_attn_bwd_chunk(desc[j], q_segs, ch, qd, kd[j], vd[j], o, gd, lse, delta, dq, None, None,
                                 flags=hexi.HEXI_SKIP_DKDV | (hexi.HEXI_COMPUTE_DELTA if j == 0 else 0))
        hexi.hexi_attn_bwd_chunk(desc[j], q_segs, ch, qd, kd[j], vd[j], None, gd, lse, delta, None, dk[j], dv[j],
                                 flags=hexi.HEXI_SKIP_DQ | hexi.HEXI_ACCUMULATE)
    k64, v64, p64 = np.concatenate([to64(t) for t in ks]), np.concatenate([to64(t) for t in vs]), np.concatenate(kv_pos)
    o_ref, lse_ref = oracle.attn_fwd(to64(q), q_pos, k64, v64, p64, scale, kv_of_q)
    ref = oracle.attn_bwd(to64(q), q_pos, k64, v64, p64, to64(d_o), scale, kv_of_q)
    check("o", o.cpu(), o_ref, "bf16")
    check("lse", lse.cpu(), lse_ref, "bf16")
    check("dq", dq.cpu(), ref["dq"], "bf16")
    for name, got, want in (("dk", torch.cat(dk).cpu().numpy() - 0.5, ref["dk"]), ("dv", torch.cat(dv).cpu().numpy() + 0.25, ref["dv"])):
        check(name, got, want, "bf16", abs_factor=max(1.0, float(np.max(np.abs(want))) / 8))


@pytest.mark.parametrize("lq,lc,nq,nkv,d", [(1024, 320, 64, 64, 128), (1024, 385, 64, 4, 64)] + QUAD_FWD_STEPS)
def test_large_workgroups_softmax_fallback(lq, lc, nq, nkv, d):
    # The 256-row forward kernel fixes each row's softmax reference at its first key tile and repeats the workgroup with the
    # exact online softmax when a row's sum leaves [2^-60, 2^60]; the 64-row one (the last two sizes) raises its reference as it goes, and the parts
    # of its four wavefronts differ by such factors when they are combined.  Every second kv head scales the keys beyond the first
    # tile so that later scores exceed the first tile's maximum by far more than 2^100; the others do the reverse.
    q, _, k, v = _large_step_inputs(lq, lc, nq, nkv, d, 99)
    q = (q.float() * 3).to(torch.bfloat16)
    k = k.float()
    k[64:, ::2] *= 60.0
    k[:64, 1::2] *= 60.0
    k[64:, 1::2] *= 0.02
    k = k.to(torch.bfloat16)
    print(f"\n  large fallback: {lq} x {lc} x {nq}/{nkv} x {d}", flush=True)
    qd, kd, vd = q.to(DEV), k.to(DEV), v.to(DEV)
    o, lse = torch.empty(q.shape, dtype=torch.float32, device=DEV), torch.empty((nq, lq), device=DEV)
    for off in (lc, lc // 2):
        hexi.hexi_attn_fwd_chunk(hexi.desc_for(qd, kd, d ** -0.5), [(off, lq)], [(0, lc)], qd, kd, vd, o, lse)
        o_ref, lse_ref = oracle.attn_fwd(to64(q), np.arange(off, off + lq), to64(k), to64(v), np.arange(lc), d ** -0.5)
        assert float(np.max(lse_ref) - np.min(lse_ref)) > 50.0
        check("o", o.cpu(), o_ref, "bf16")
        check("lse", lse.cpu(), lse_ref, "bf16")


@pytest.mark.parametrize("lq,lc,nq,nkv,d", [(1024, 320, 64, 64, 128), (1024, 385, 64, 4, 64)])
def test_large_workgroups_residuals(lq, lc, nq, nkv, d):
    # test_dq_residuals_of_large_ds in the 256-row dQ kernel, whose residuals are fp32 products
    _dq_residuals(lq, lc, nq, nkv, d)


@pytest.mark.parametrize("lq,lc,nq,nkv,d", QUAD_DQ_STEPS)
def test_64_row_dq_residuals(lq, lc, nq, nkv, d):
    # the same in the 64-row one, whose residuals are two more bf16 operands on the fragments of the product before
    _dq_residuals(lq, lc, nq, nkv, d)


def _dq_residuals(lq, lc, nq, nkv, d):
    q, d_o, k, v = _large_step_inputs(lq, lc, nq, nkv, d, 41, k_scale=2.0)
    off, scale = lc // 2, d ** -0.5
    print(f"\n  large residuals: {lq} x {lc} x {nq}/{nkv} x {d}", flush=True)
    qd, gd, kd, vd = (t.to(DEV) for t in (q, d_o, k, v))
    o, lse = torch.empty(q.shape, dtype=torch.float32, device=DEV), torch.empty((nq, lq), device=DEV)
    hexi.hexi_attn_fwd_chunk(hexi.desc_for(qd, kd, scale), [(off, lq)], [(0, lc)], qd, kd, vd, o, lse)
    plain = _large_backward(qd, kd, vd, gd, o, lse, [(off, lq)], [(0, lc)], scale)[0]
    big = _large_backward(qd, kd, vd, gd * 64, o, lse, [(off, lq)], [(0, lc)], scale)[0]
    ref = oracle.attn_bwd(to64(q), np.arange(off, off + lq), to64(k), to64(v), np.arange(lc), to64(d_o), scale)
    e_plain, _ = check("dq", plain.cpu(), ref["dq"], "bf16")
    e_big, _ = check("dq with residuals everywhere", (big / 64).cpu(), ref["dq"], "bf16")
    assert float((big / 64 != plain).float().mean()) > 0.5 and e_big <= e_plain


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("nq,nkv,lq,lc", [(16, 2, 1000, 1010), (32, 16, 1000, 1010), (16, 16, 100, 1010), (6, 3, 77, 90), (64, 32, 199, 16), (96, 48, 16, 266)])
def test_f32_grouped_heads_in_both_shapes(nq, nkv, lq, lc, d):
    # fp32 with several q heads per kv head: at head_dim 128 operands cut in the diagonal chunk of the first size, heads in two runs, and in both of the
    # second, dK / dV shared in 64-key workgroups in the third's and the last's first chunk, dQ in 64-row ones in 199 rows, the rest split; at 64 split, two of
    # them a CU in the second size, and dK / dV shared in the first chunk of the third (test_f32_shapes_at_head_dim_64 has the others).  The halves
    # together and in calls of their own, with the same bits: no sum is spread over more than two workgroups
    w = _custom(f"f32_gqa_{nq}_{lq}_{lc}_{d}", "f32", nq, nkv, d, lc + lq, [(lc, lq)], [[(0, lc)], [(lc, lq)]])
    run, inputs, ref = _run_and_compare(w, seed=lq + lc + d)
    dq = torch.zeros_like(run.dq)
    for j, ch in enumerate(w.chunks):
        dk, dv = torch.full_like(run.dk[j], 7.0), torch.full_like(run.dv[j], 7.0)
        args = (run.desc[j], w.q_segs, ch, run.q, run.k[j], run.v[j], None, run.d_o, run.lse, run.delta)
        hexi.hexi_attn_bwd_chunk(*args, dq, None, None, flags=hexi.HEXI_SKIP_DKDV)
        hexi.hexi_attn_bwd_chunk(*args, None, dk, dv, flags=hexi.HEXI_SKIP_DQ)
        assert torch.equal(dk, run.dk[j]) and torch.equal(dv, run.dv[j])
    assert torch.equal(dq, run.dq)


@pytest.mark.parametrize("lq,lc,nq,nkv,d", [s[:5] for s in QUAD_STEPS])
def test_64_wide_workgroup_shapes(lq, lc, nq, nkv, d):
    # one chunk fully visible and one diagonal in two segments, K scaled by 3 (scores that raise the running maximum, large dS), through
    # the whole replay: the second chunk merges into the first one's o / lse and adds to its dq
    w = _custom(f"quad_{nq}_{lq}_{lc}_{d}", "bf16", nq, nkv, d, lc + lq + 7, [(lc, lq // 2), (lc + lq // 2 + 7, lq - lq // 2)],
                [[(0, lc)], [(lc, lq // 2 + 7), (lc + lq // 2 + 7, lq - lq // 2)]], k_scale=3.0)
    print(f"\n[{w.name}]", flush=True)
    inputs = wl.make_inputs(w, lq * 1000 + lc + d)
    run = replay.ShardRun(w, inputs, DEV)
    run.step()
    torch.cuda.synchronize()
    ref = oracle_full(w, inputs)
    for name, got, want in (("o", run.o, ref["o"]), ("lse", run.lse, ref["lse"]), ("dq", run.dq, ref["dq"])):
        check(name, got.cpu(), want, "bf16")
    for j in range(2):
        for name, got in (("dk", run.dk[j]), ("dv", run.dv[j])):
            want = chunk_slices(w, j, ref[name], ref["n_keys"])
            # P and dS are rounded to bf16, 2^-9 of each product: an element of dv is off by up to 2^-9 sum P |dO| over the rows and heads
            # that see the key, 2e-2 where that sum is 10; with 16 heads to a group and peaked rows it reaches twice the largest |dv|
            check(f"{name}[{j}]", got.cpu(), want, "bf16", abs_factor=max(1.0, float(np.max(np.abs(want))) / 5.0))


def test_64_wide_workgroups_accumulate():
    # dk / dv under HEXI_ACCUMULATE (plain stores and atomics): the running value plus the gradient
    for lq, lc, nq, nkv, d, _ in (s for s in QUAD_STEPS if s[0] in (129, 260)):
        q, d_o, k, v = _large_step_inputs(lq, lc, nq, nkv, d, lq)
        qd, gd, kd, vd = (t.to(DEV) for t in (q, d_o, k, v))
        q_segs, kv_segs, scale = [(lc // 2, lq)], [(0, lc)], d ** -0.5
        o, lse, delta = torch.empty(q.shape, device=DEV), torch.empty((nq, lq), device=DEV), torch.empty((nq, lq), device=DEV)
        desc = hexi.desc_for(qd, kd, scale)
        hexi.hexi_attn_fwd_chunk(desc, q_segs, kv_segs, qd, kd, vd, o, lse)
        outs = []
        for flags in (0, hexi.HEXI_ACCUMULATE):
            dq = torch.zeros(q.shape, device=DEV)
            dk, dv = torch.full(k.shape, 0.5, device=DEV), torch.full(v.shape, -0.25, device=DEV)
            hexi.hexi_attn_bwd_chunk(desc, q_segs, kv_segs, qd, kd, vd, o, gd, lse, delta, dq, dk, dv, flags=flags | hexi.HEXI_COMPUTE_DELTA)
            outs.append((dk, dv))
        # (the same sums, in another order where they are atomic)
        bound = 1e-5 * float(outs[0][0].abs().max() + outs[0][1].abs().max() + 1.0)
        assert float((outs[1][0] - outs[0][0] - 0.5).abs().max()) <= bound and float((outs[1][1] - outs[0][1] + 0.25).abs().max()) <= bound


@pytest.mark.parametrize("step,keys,seen", UNSEEN_STEPS)
def test_atomic_sums_of_a_chunk_with_keys_that_no_row_sees(step, keys, seen):
    # zeros where nothing is seen, over NaN and over what is to be added to
    d, nq, nkv, q_segs, kv_segs = step
    print(f"\n  {keys} keys, {step}, {seen} seen", flush=True)
    lq, lc = sum(n for _, n in q_segs), sum(n for _, n in kv_segs)
    q_pos, k_pos = (np.concatenate([np.arange(a, a + n) for a, n in segs]) for segs in (q_segs, kv_segs))
    assert int(np.sum(k_pos <= q_pos[-1])) == seen
    q, d_o, k, v = _large_step_inputs(lq, lc, nq, nkv, d, lq + lc)
    qd, gd, kd, vd = (t.to(DEV) for t in (q, d_o, k, v))
    desc, args = hexi.desc_for(qd, kd, d ** -0.5), (q_segs, kv_segs, qd, kd, vd)
    o, lse, delta, dq = (torch.zeros(s, device=DEV) for s in (q.shape, (nq, lq), (nq, lq), q.shape))
    hexi.hexi_attn_fwd_chunk(desc, *args, o, lse)
    ref = oracle.attn_bwd(to64(q), q_pos, to64(k), to64(v), k_pos, to64(d_o), d ** -0.5)
    for flags, fill in ((0, float("nan")), (hexi.HEXI_ACCUMULATE, 0.5)):
        dq.zero_()
        dk, dv = torch.full(k.shape, fill, device=DEV), torch.full(v.shape, fill, device=DEV)
        hexi.hexi_attn_bwd_chunk(desc, *args, o, gd, lse, delta, dq, dk, dv, flags=flags | hexi.HEXI_COMPUTE_DELTA)
        held = fill if flags else 0.0
        check("dq", dq.cpu(), ref["dq"], "bf16")
        for name, got in (("dk", dk), ("dv", dv)):      # (the bound on a single element as in test_large_workgroups_boundary_sizes)
            assert bool((got[seen:] == held).all())
            check(name, got.cpu() - held, ref[name], "bf16", abs_factor=max(1.0, float(np.max(np.abs(ref[name]))) / 8))


@pytest.mark.parametrize("lq,lc,nq,nkv,d,off", WIDE_DQ_STEPS)
def test_64_key_workgroups_beside_256_row_dq(lq, lc, nq, nkv, d, off):
    print(f"\n  64 keys, 256 rows: {lq} x {lc} x {nq}/{nkv} x {d} at {off}", flush=True)
    q, d_o, k, v = _large_step_inputs(lq, lc, nq, nkv, d, lq + lc)
    qd, gd, kd, vd = (t.to(DEV) for t in (q, d_o, k, v))
    desc, args = hexi.desc_for(qd, kd, d ** -0.5), ([(off, lq)], [(0, lc)], qd, kd, vd)
    o, lse, delta, dq = torch.empty(q.shape, device=DEV), torch.empty((nq, lq), device=DEV), torch.empty((nq, lq), device=DEV), torch.zeros(q.shape, device=DEV)
    dk, dv = torch.full(k.shape, 7.0, device=DEV), torch.full(v.shape, 7.0, device=DEV)
    hexi.hexi_attn_fwd_chunk(desc, *args, o, lse)
    hexi.hexi_attn_bwd_chunk(desc, *args, o, gd, lse, delta, dq, dk, dv, flags=hexi.HEXI_COMPUTE_DELTA)
    ref = oracle.attn_bwd(to64(q), np.arange(off, off + lq), to64(k), to64(v), np.arange(lc), to64(d_o), d ** -0.5)
    check("dq", dq.cpu(), ref["dq"], "bf16")
    for name, got in (("dk", dk), ("dv", dv)):      # (the bound on a single element as in test_large_workgroups_boundary_sizes)
        check(name, got.cpu(), ref[name], "bf16", abs_factor=max(1.0, float(np.max(np.abs(ref[name]))) / 8))


def _forward_alone_and_merged(q_segs, kv_segs, lq, lc, nq, nkv, d):
    # every row exactly once, first alone, then merged into a running (o, lse)
    print(f"\n  forward: {q_segs} x {kv_segs} x {nq}/{nkv} x {d}", flush=True)
    q, _, k, v = _large_step_inputs(lq, lc, nq, nkv, d, lq + lc)
    qd, kd, vd = (t.to(DEV) for t in (q, k, v))
    desc = hexi.desc_for(qd, kd, d ** -0.5)
    q_pos, kv_pos = (np.concatenate([np.arange(a, a + n) for a, n in segs]) for segs in (q_segs, kv_segs))
    o_ref, lse_ref = oracle.attn_fwd(to64(q), q_pos, to64(k), to64(v), kv_pos, d ** -0.5)
    o, lse = torch.full(q.shape, float("nan"), device=DEV), torch.full((nq, lq), float("nan"), device=DEV)
    hexi.hexi_attn_fwd_chunk(desc, q_segs, kv_segs, qd, kd, vd, o, lse)
    check("o", o.cpu(), o_ref, "bf16")
    check("lse", lse.cpu(), lse_ref, "bf16")
    g = torch.Generator().manual_seed(lq)
    o0, lse0 = torch.randn(q.shape, generator=g), torch.randn((nq, lq), generator=g)
    o, lse = o0.to(DEV), lse0.to(DEV)
    hexi.hexi_attn_fwd_chunk(desc, q_segs, kv_segs, qd, kd, vd, o, lse, flags=hexi.HEXI_ACCUMULATE)
    o_ref, lse_ref = oracle.merge(to64(o0), to64(lse0), o_ref, lse_ref)
    check("o merged", o.cpu(), o_ref, "bf16")
    check("lse merged", lse.cpu(), lse_ref, "bf16")


@pytest.mark.parametrize("lq,lc,nq,nkv,d", PART_ROUND_STEPS)
def test_forward_of_a_round_and_a_part(lq, lc, nq, nkv, d):
    _forward_alone_and_merged([(lc, lq)], [(0, lc)], lq, lc, nq, nkv, d)


@pytest.mark.parametrize("lq,lc,nq,nkv,d,off", SHARED_STEPS)
def test_forward_shared_by_large_and_64_row_workgroups(lq, lc, nq, nkv, d, off):
    _forward_alone_and_merged([(off, lq)], [(0, lc)], lq, lc, nq, nkv, d)


def test_forward_shared_by_large_and_64_row_workgroups_in_segments():
    w = SHARED_SHARD
    _forward_alone_and_merged(w["q_segs"], w["kv_segs"], sum(n for _, n in w["q_segs"]), sum(n for _, n in w["kv_segs"]), w["nq"], w["nkv"], w["d"])


@pytest.mark.parametrize("lq,lc,nq,nkv,d", PART_ROUND_STEPS + [(4096, 4096, 24, 8, 128), (15773, 21188, 9, 3, 64)])
def test_rows_and_heads_of_a_forward_step_are_summed_alike(lq, lc, nq, nkv, d):
    # one row and one set of keys, repeated over all rows and heads, all keys visible: results with the same bits everywhere, as all rows of such a
    # step go to one kernel (whose rest over whole rounds of workgroups is too large for a second one)
    g = torch.Generator().manual_seed(lq + nq)
    q = torch.randn((1, 1, d), generator=g).to(torch.bfloat16).expand(lq, nq, d).contiguous().to(DEV)
    k, v = (torch.randn((lc, 1, d), generator=g).to(torch.bfloat16).expand(lc, nkv, d).contiguous().to(DEV) for _ in range(2))
    o, lse = torch.full(q.shape, float("nan"), device=DEV), torch.full((nq, lq), float("nan"), device=DEV)
    hexi.hexi_attn_fwd_chunk(hexi.desc_for(q, k, d ** -0.5), [(lc, lq)], [(0, lc)], q, k, v, o, lse)
    assert torch.equal(o, o[:1, :1].expand_as(o)) and torch.equal(lse, lse[:1, :1].expand_as(lse))


@pytest.mark.parametrize("step,shapes", F32_STEPS)
def test_f32_shapes_at_head_dim_64(step, shapes):
    # forward alone and merged, backward added to running dq / dk / dv, in every shape the rules deal out (the shapes are asserted on the CPU);
    # the halves in calls of their own as well: with the same bits, one workgroup a CU or two, unless dQ is split in one of the calls only
    lq, lc, nq, nkv, off = step
    d, g = 64, torch.Generator().manual_seed(lq + lc)
    q, k, v, d_o = (torch.randn(n, h, d, generator=g) for n, h in ((lq, nq), (lc, nkv), (lc, nkv), (lq, nq)))
    scale, pos = d ** -0.5, np.arange(off, off + lq)
    o_ref, lse_ref = oracle.attn_fwd(to64(q), pos, to64(k), to64(v), np.arange(lc), scale)
    ref = oracle.attn_bwd(to64(q), pos, to64(k), to64(v), np.arange(lc), to64(d_o), scale)
    qd, kd, vd, gd = (t.to(DEV) for t in (q, k, v, d_o))
    desc, args = hexi.desc_for(qd, kd, scale), ([(off, lq)], [(0, lc)], qd, kd, vd)
    o, lse = torch.full(q.shape, float("nan"), device=DEV), torch.full((nq, lq), float("nan"), device=DEV)
    hexi.hexi_attn_fwd_chunk(desc, *args, o, lse)
    check("o", o.cpu(), o_ref, "f32")
    check("lse", lse.cpu(), lse_ref, "f32")
    o0, lse0 = torch.randn(q.shape, generator=g), torch.randn((nq, lq), generator=g)
    om, lsem = o0.to(DEV), lse0.to(DEV)
    hexi.hexi_attn_fwd_chunk(desc, *args, om, lsem, flags=hexi.HEXI_ACCUMULATE)
    om_ref, lsem_ref = oracle.merge(to64(o0), to64(lse0), o_ref, lse_ref)
    check("o merged", om.cpu(), om_ref, "f32")
    check("lse merged", lsem.cpu(), lsem_ref, "f32")
    delta = torch.empty((nq, lq), device=DEV)
    dq, dk, dv = torch.zeros(q.shape, device=DEV), torch.full(k.shape, 7.0, device=DEV), torch.full(v.shape, 7.0, device=DEV)
    hexi.hexi_attn_bwd_chunk(desc, *args, o, gd, lse, delta, dq, dk, dv, flags=hexi.HEXI_COMPUTE_DELTA)
    for name, got in (("dq", dq), ("dk", dk), ("dv", dv)):
        check(name, got.cpu(), ref[name], "f32")
    dq2, dk2, dv2 = torch.zeros_like(dq), torch.zeros_like(dk), torch.zeros_like(dv)
    hexi.hexi_attn_bwd_chunk(desc, *args, None, gd, lse, delta, dq2, None, None, flags=hexi.HEXI_SKIP_DKDV)
    hexi.hexi_attn_bwd_chunk(desc, *args, None, gd, lse, delta, None, dk2, dv2, flags=hexi.HEXI_SKIP_DQ)
    check("dq alone", dq2.cpu(), ref["dq"], "f32")
    assert torch.equal(dk, dk2) and torch.equal(dv, dv2) and ((shapes[1] == 0) != (shapes[3] == 0) or torch.equal(dq, dq2))


@pytest.mark.parametrize("step,_", F32X3_STEPS)
def test_f32_split_operand_shapes(step, _):
    # the kernels that cut fp32 operands into three bf16 ones, in every shape the rules deal out (asserted on the CPU): one chunk fully visible and
    # a diagonal one in two segments that merges into its o / lse, K scaled by 3; strided tensors with the same bits; dk / dv under
    # HEXI_ACCUMULATE; the halves in calls of their own, which may take other kernels
    lq, lc, nq, nkv, d = step
    q_segs, own = f32x3_diagonal(lq, lc)
    w = _custom(f"f32x3_{nq}_{lq}_{lc}_{d}", "f32", nq, nkv, d, own[-1][0] + own[-1][1], q_segs, [[(0, lc)], own], k_scale=3.0)
    run, inputs, ref = _run_and_compare(w, seed=lq + lc + d)
    wide = lambda t: torch.cat([t, torch.zeros_like(t[:, :1])], 1)[:, :t.shape[1]]
    for j, ch in enumerate(w.chunks):
        dk, dv, dq = torch.full_like(run.dk[j], 0.5), torch.full_like(run.dv[j], -0.25), torch.zeros_like(run.dq)
        args = (run.desc[j], w.q_segs, ch, run.q, run.k[j], run.v[j], None, run.d_o, run.lse, run.delta)
        hexi.hexi_attn_bwd_chunk(*args, dq, dk, dv, flags=hexi.HEXI_ACCUMULATE)
        check("dk acc", dk.cpu(), chunk_slices(w, j, ref["dk"], ref["n_keys"]) + 0.5, "f32")
        check("dv acc", dv.cpu(), chunk_slices(w, j, ref["dv"], ref["n_keys"]) - 0.25, "f32")
        q, d_o, k, v = wide(run.q), wide(run.d_o), wide(run.k[j]), wide(run.v[j])
        wide_args = (hexi.desc_for(q, k, w.scale), w.q_segs, ch, q, k, v, None, d_o, run.lse, run.delta)
        out = []
        for a in (args, wide_args):
            dq, dk, dv = torch.zeros_like(dq), torch.full_like(dk, 7.0), torch.full_like(dv, 7.0)
            dq_half, dk_half, dv_half = torch.zeros_like(dq), torch.full_like(dk, 7.0), torch.full_like(dv, 7.0)
            hexi.hexi_attn_bwd_chunk(*a, dq, dk, dv)
            hexi.hexi_attn_bwd_chunk(*a, dq_half, None, None, flags=hexi.HEXI_SKIP_DKDV)
            hexi.hexi_attn_bwd_chunk(*a, None, dk_half, dv_half, flags=hexi.HEXI_SKIP_DQ)
            out.append((dq, dk, dv, dq_half, dk_half, dv_half))
        assert all(torch.equal(x, y) for x, y in zip(*out)) and torch.equal(out[0][1], run.dk[j]) and torch.equal(out[0][2], run.dv[j])
        check("dk alone", out[0][4].cpu(), chunk_slices(w, j, ref["dk"], ref["n_keys"]), "f32")
        check("dv alone", out[0][5].cpu(), chunk_slices(w, j, ref["dv"], ref["n_keys"]), "f32")
        check("dq alone", out[0][3].cpu(), to64(out[0][0].cpu()), "f32")
    o, lse = torch.full_like(run.o, float("nan")), torch.full_like(run.lse, float("nan"))
    for j, ch in enumerate(w.chunks):
        k, v = wide(run.k[j]), wide(run.v[j])
        hexi.hexi_attn_fwd_chunk(hexi.desc_for(wide(run.q), k, w.scale), w.q_segs, ch, wide(run.q), k, v, o, lse, flags=hexi.HEXI_ACCUMULATE if j else 0)
    assert torch.equal(o, run.o) and torch.equal(lse, run.lse)


@pytest.mark.parametrize("lq,lc,nq,nkv,d", [(172, 196, 48, 16, 128), (868, 112, 16, 8, 128), (651, 577, 8, 8, 64)])
def test_f32_split_operands_at_the_ends_of_the_range(lq, lc, nq, nkv, d):
    # q near the largest fp32 value, columns of v of 1e33 and 1e-30, scores of -inf: left to the units on the fp32 instruction
    g = torch.Generator().manual_seed(lq)
    q, k, v, d_o = (torch.randn((n, h, d), generator=g) for n, h in ((lq, nq), (lc, nkv), (lc, nkv), (lq, nq)))
    v[..., 0] *= 1e33
    v[..., 1] *= 1e-30
    k[:, :, 0] = 0.0
    q[..., 0] = 3.4e38
    k[3::7, :, 0] = -1e20
    qs, ks = [(lc, lq)], [(0, lc)]
    t = {n: x.to(DEV) for n, x in dict(q=q, k=k, v=v).items()}
    o, lse = torch.empty((lq, nq, d), device=DEV), torch.empty((nq, lq), device=DEV)
    hexi.hexi_attn_fwd_chunk(hexi.desc_for(t["q"], t["k"], 0.1), qs, ks, t["q"], t["k"], t["v"], o, lse)
    keep = torch.tensor([j for j in range(lc) if j % 7 != 3])
    o_ref, lse_ref = oracle.attn_fwd(to64(q), np.arange(lc, lc + lq), to64(k[keep]), to64(v[keep]), keep.numpy(), float(np.float32(0.1)))
    check("lse", lse.cpu(), lse_ref, "f32")
    for col, unit in ((0, 1e33), (1, 1e-30), (slice(2, None), 1.0)):
        check(f"o[{col}]", (o.cpu().double() / unit)[..., col].float(), o_ref[..., col] / unit, "f32")


@pytest.mark.parametrize("lq,lc,nq,nkv,d", [(691, 119, 32, 8, 128), (651, 577, 8, 8, 64)])
def test_f32_split_operands_with_infinite_values(lq, lc, nq, nkv, d):
    # infinite values of v, whose rests after the cut are NaN: columns of one sign, of both and with a NaN, the others untouched; q with a NaN in one row
    g = torch.Generator().manual_seed(lc)
    q, k, v = (torch.randn((n, h, d), generator=g) for n, h in ((lq, nq), (lc, nkv), (lc, nkv)))
    inf, nan = float("inf"), float("nan")
    o_ref, lse_ref = oracle.attn_fwd(to64(q), np.arange(lc, lc + lq), to64(k), to64(v), np.arange(lc), float(np.float32(0.1)))
    v[5, :, 0], v[lc - 1, :, 1], v[5, :, 2], v[40, :, 2], v[9, :, 3] = inf, -inf, inf, -inf, nan
    q[7] = nan
    t = {n: x.to(DEV) for n, x in dict(q=q, k=k, v=v).items()}
    o, lse = torch.empty((lq, nq, d), device=DEV), torch.empty((nq, lq), device=DEV)
    hexi.hexi_attn_fwd_chunk(hexi.desc_for(t["q"], t["k"], 0.1), [(lc, lq)], [(0, lc)], t["q"], t["k"], t["v"], o, lse)
    rows = [r for r in range(lq) if r != 7]
    check("o", o.cpu()[rows][..., 4:], o_ref[rows][..., 4:], "f32")
    check("lse", lse.cpu()[:, rows], lse_ref[:, rows], "f32")
    o = o.cpu()
    assert (o[rows][..., 0] == inf).all() and (o[rows][..., 1] == -inf).all() and o[rows][..., 2:4].isnan().all() and o[7].isnan().all()


@pytest.mark.parametrize("lq,lc,nq,nkv,d,limit", [(579, 5000, 8, 2, 64, 5.2e-7), (338, 12000, 12, 3, 128, 7.8e-7)])
def test_f32_long_rows_are_no_further_from_float64_where_operands_are_cut(lq, lc, nq, nkv, d, limit):
    # o of rows that see many keys: relative errors on the fp32 instruction 5.3e-7 and 8.0e-7 (1.5 % between seeds), cut with one chain of sums 5.7e-7 and 9.1e-7
    g = torch.Generator().manual_seed(lc)
    q, k, v = (torch.randn((n, h, d), generator=g) for n, h in ((lq, nq), (lc, nkv), (lc, nkv)))
    scale = float(np.float32(d ** -0.5))
    o, lse = torch.empty((lq, nq, d), device=DEV), torch.empty((nq, lq), device=DEV)
    t = [x.to(DEV) for x in (q, k, v)]
    hexi.hexi_attn_fwd_chunk(hexi.desc_for(t[0], t[1], scale), [(lc, lq)], [(0, lc)], *t, o, lse)
    rows = slice(0, lq, 8)
    o_ref, lse_ref = oracle.attn_fwd(to64(q[rows]), np.arange(lc, lc + lq)[rows], to64(k), to64(v), np.arange(lc), scale)
    _, rel = check("o", o[rows].cpu(), o_ref, "f32")
    check("lse", lse[:, rows].cpu(), lse_ref, "f32")
    assert rel < limit


def _f32_step(q, k, v, d_o, off, scale, merged=False):
    """o, lse, dq, dk, dv of one fp32 step, rows from `off` against keys from 0; merged: o / lse into an empty running result, dk / dv added to zeros."""
    lq, lc = q.shape[0], k.shape[0]
    t = [x.to(DEV) for x in (q, k, v, d_o)]
    desc, args, add = hexi.desc_for(t[0], t[1], scale), ([(off, lq)], [(0, lc)], *t[:3]), hexi.HEXI_ACCUMULATE if merged else 0
    o, lse, delta, dq = torch.zeros_like(t[0]), torch.full((q.shape[1], lq), -float("inf"), device=DEV), torch.empty((q.shape[1], lq), device=DEV), torch.zeros_like(t[0])
    dk, dv = torch.zeros_like(t[1]), torch.zeros_like(t[1])
    hexi.hexi_attn_fwd_chunk(desc, *args, o, lse, flags=add)
    hexi.hexi_attn_bwd_chunk(desc, *args, o, t[3], lse, delta, dq, dk, dv, flags=hexi.HEXI_COMPUTE_DELTA | add)
    return [x.cpu() for x in (o, lse, dq, dk, dv)]


# (the kernels that cut operands, forward and backward: with heads in two runs, with 64-row units, at head_dim 64 with 32 and 64 keys)
F32X3_VALUE_STEPS = [(523, 882, 9, 3, 128), (172, 196, 48, 16, 128), (651, 577, 8, 8, 64), (693, 755, 24, 24, 64)]
F32X3_MASKED_STEPS = [(568, 167, 8, 2, 128), (347, 270, 16, 16, 128), (625, 231, 24, 24, 128), (635, 1158, 24, 24, 64)]      # (rows from the middle of the keys)


@pytest.mark.parametrize("lq,lc,nq,nkv,d", F32X3_VALUE_STEPS)
@pytest.mark.parametrize("units", [dict(v=1e-36), dict(d_o=1e-36), dict(d_o=1e-32), dict(q=1e36, k=1e-36), dict(q=1e-36, k=1e36), dict(v=1e-25, d_o=1e-10),
                                   dict(d_o=3e30), dict(d_o=1e20, v=1e10), dict(q=1e10, k=1e10, scale=1e-21), dict(q=1e-5, k=1e-5, scale=1e9),
                                   dict(q=1e-36, k=1e36, d_o=1e-30, v=1e30)], ids=str)
def test_f32_keeps_its_range_where_operands_are_cut(lq, lc, nq, nkv, d, units):
    # operands with magnitudes near the ends of fp32's range: every output keeps its relative accuracy
    g = torch.Generator().manual_seed(lq)
    x = {n: torch.randn((rows, h, d), generator=g) for n, rows, h in (("q", lq, nq), ("k", lc, nkv), ("v", lc, nkv), ("d_o", lq, nq))}
    u = {n: units.get(n, 1.0) for n in x}
    for name, unit in u.items():
        x[name] *= unit
    scale = float(np.float32(units.get("scale", 0.1)))
    got = _f32_step(*x.values(), lc, scale)
    in_units = {n: to64(x[n]) / u[n] for n in x}
    qk = u["q"] * u["k"]
    ref = oracle.attn_bwd(in_units["q"], np.arange(lc, lc + lq), in_units["k"], in_units["v"], np.arange(lc), in_units["d_o"], scale * qk)
    o_ref, lse_ref = oracle.attn_fwd(in_units["q"], np.arange(lc, lc + lq), in_units["k"], in_units["v"], np.arange(lc), scale * qk)
    g_v = u["v"] * u["d_o"]
    for name, t, want, unit in (("o", got[0], o_ref, u["v"]), ("lse", got[1], lse_ref, 1.0), ("dq", got[2], ref["dq"], g_v / u["q"]),
                                ("dk", got[3], ref["dk"], g_v / u["k"]), ("dv", got[4], ref["dv"], u["d_o"])):
        if unit > (1e-33 if name in ("dq", "dk") else 1e-37):      # (dS, and below 1e-38 everything, has fewer than 24 bits in fp32)
            check(name, t.double() / unit, want, "f32")


@pytest.mark.parametrize("lq,lc,nq,nkv,d", F32X3_VALUE_STEPS)
def test_f32_large_values_whose_weighted_sum_is_finite(lq, lc, nq, nkv, d):
    # positive values of v up to 1e37, scores that rise after the first keys: the sum of v with weights of at most 1 is finite
    g = torch.Generator().manual_seed(lq)
    q, k, v = (torch.randn((n, h, d), generator=g) for n, h in ((lq, nq), (lc, nkv), (lc, nkv)))
    k[:128] *= 0.02
    v = 2.0 + torch.tanh(v)
    scale = float(np.float32(1.2 * d ** -0.5))
    o, lse = torch.empty((lq, nq, d), device=DEV), torch.empty((nq, lq), device=DEV)
    t = [x.to(DEV) for x in (q, k, v * 3e36)]
    hexi.hexi_attn_fwd_chunk(hexi.desc_for(t[0], t[1], scale), [(lc, lq)], [(0, lc)], *t, o, lse)
    o_ref, lse_ref = oracle.attn_fwd(to64(q), np.arange(lc, lc + lq), to64(k), to64(v * 3e36) / 3e36, np.arange(lc), scale)
    check("o", o.cpu().double() / 3e36, o_ref, "f32")
    check("lse", lse.cpu(), lse_ref, "f32")


@pytest.mark.parametrize("lq,lc,nq,nkv,d", F32X3_VALUE_STEPS)
def test_f32_nan_with_a_payload_in_its_lower_bits(lq, lc, nq, nkv, d):
    # cut to its upper 16 bits it is an infinity, here one whose scores are -inf: the rows that see it are NaN all the same
    g = torch.Generator().manual_seed(lc)
    q, k, v, d_o = (torch.randn((n, h, d), generator=g) for n, h in ((lq, nq), (lc, nkv), (lc, nkv), (lq, nq)))
    q[..., 0] = -q[..., 0].abs() - 0.1
    k[lc - 7, 0, 0] = torch.tensor(0x7f800001, dtype=torch.int32).view(torch.float32)
    o, lse, dq, dk, dv = _f32_step(q, k, v, d_o, lc, 0.1)
    group = nq // nkv
    assert o[:, :group].isnan().all() and not o[:, group:].isnan().any()
    assert dq[:, :group].isnan().all() and dk[:, 0].isnan().all() and not dq[:, group:].isnan().any() and not dk[:, 1:].isnan().any()


@pytest.mark.parametrize("merged", [False, True])
@pytest.mark.parametrize("lq,lc,nq,nkv,d,off", [s + (s[1],) for s in F32X3_VALUE_STEPS] + [s + (s[1] // 2,) for s in F32X3_MASKED_STEPS])
def test_f32_infinite_gradients_of_the_output(lq, lc, nq, nkv, d, off, merged):
    # one infinite dO: dv of the keys that its row sees is infinite in that column, and dk has the signs of P x v x q there; nothing else is touched
    g = torch.Generator().manual_seed(lc + 1)
    q, k, v, d_o = (torch.randn((n, h, d), generator=g) for n, h in ((lq, nq), (lc, nkv), (lc, nkv), (lq, nq)))
    row, head, col = 61, nkv - 1, 5
    t = [x.to(DEV) for x in (q, k, v, d_o)]
    desc, args = hexi.desc_for(t[0], t[1], 0.1), ([(off, lq)], [(0, lc)], *t[:3])
    o, lse, delta = torch.zeros_like(t[0]), torch.full((nq, lq), -float("inf"), device=DEV), torch.empty((nq, lq), device=DEV)
    hexi.hexi_attn_fwd_chunk(desc, *args, o, lse)
    run = lambda: [torch.zeros_like(t[0]), torch.zeros_like(t[1]), torch.zeros_like(t[1])]
    want, got = run(), run()
    flags = hexi.HEXI_ACCUMULATE if merged else 0
    hexi.hexi_attn_bwd_chunk(desc, *args, o, t[3], lse, delta, *want, flags=flags | hexi.HEXI_COMPUTE_DELTA)
    t[3][row, head * (nq // nkv), col] = float("inf")
    hexi.hexi_attn_bwd_chunk(desc, *args, None, t[3], lse, delta, *got, flags=flags)
    (dq, dk, dv), (_, dk0, dv0) = [x.cpu() for x in got], [x.cpu() for x in want]
    seen = off + row + 1
    h = head * (nq // nkv)
    assert (dv[:seen, head, col] == float("inf")).all() and (dk[:seen, head] == float("inf") * torch.sign(v[:seen, head, col, None] * q[row, h])).all()
    rest = lambda x: torch.cat([x[seen + 127:, head].flatten(), x[:, :head].flatten()])      # (0 x inf: keys just behind the row's may be NaN)
    for name, x, x0 in (("dk", dk, dk0), ("dv", dv, dv0)):
        check(name, rest(x), rest(x0), "f32")
    others = torch.ones((lq, nq), dtype=torch.bool)
    others[row - row % 16:row - row % 16 + 16, h] = False
    check("dq", dq[others], want[0].cpu()[others], "f32")


@pytest.mark.parametrize("lq,lc,nq,nkv,d", F32X3_MASKED_STEPS)
def test_f32_infinite_value_at_a_key_that_some_rows_do_not_see(lq, lc, nq, nkv, d):
    # rows of blocks before the key are as if it were not there, rows that see it are infinite in its column
    g = torch.Generator().manual_seed(lc + 2)
    q, k, v, d_o = (torch.randn((n, h, d), generator=g) for n, h in ((lq, nq), (lc, nkv), (lc, nkv), (lq, nq)))
    off, key, col = lc // 2, lc // 2 + 83, 9
    o_ref, lse_ref = oracle.attn_fwd(to64(q), np.arange(off, off + lq), to64(k), to64(v), np.arange(lc), float(np.float32(0.1)))
    v[key, 0, col] = float("inf")
    o, lse, *_ = _f32_step(q, k, v, d_o, off, 0.1)
    group = nq // nkv
    assert (o[83:, :group, col] == float("inf")).all()
    check("lse", lse, lse_ref, "f32")
    before = 16 * max(b for b in range(6) if off + 16 * b <= key // 16 * 16)      # (0 x inf: a 16-row block that sees other keys of the key's block is NaN)
    assert before >= 64
    check("o of the rows before", o[:before], o_ref[:before], "f32")
    others = [j for j in range(d) if j != col]
    check("other columns", o[:, :, others], o_ref[:, :, others], "f32")


@pytest.mark.parametrize("d", [64, 128, 12])
@pytest.mark.parametrize("final", [None, torch.float32, torch.bfloat16])
def test_merge_of_partials_that_saw_nothing(d, final):
    # rows whose partial has LSE -inf are the identity, whatever finite values its o holds; both sides -inf: o = 0; the other rows as ever
    g = torch.Generator().manual_seed(d)
    rows, nq = 37, 3
    oa, ob = torch.randn((rows, nq, d), generator=g), torch.randn((rows, nq, d), generator=g)
    la, lb = torch.randn((nq, rows), generator=g), torch.randn((nq, rows), generator=g)
    lb[:, 5:20] = -float("inf")
    la[1, 10:25] = -float("inf")
    ob[5:20] = 3e38
    og, lg = oa.clone().to(DEV), la.clone().to(DEV)
    out = None if final is None else torch.empty((rows, nq, d), dtype=final, device=DEV)
    hexi.hexi_attn_merge_lse(og, lg, ob.to(DEV), lb.to(DEV), out)
    o_ref, l_ref = oracle.merge(to64(oa), to64(la), to64(ob), to64(lb))
    check("o", og.cpu(), o_ref, "f32")
    check("lse", lg.cpu(), l_ref, "f32")
    same = (torch.isinf(lb) & ~torch.isinf(la)).T
    assert torch.equal(og.cpu()[same], oa[same]) and torch.equal(lg.cpu().T[same], la.T[same])
    if final is not None:
        assert torch.equal(out, og.to(final))


@pytest.mark.parametrize("d", [64, 128, 12])
@pytest.mark.parametrize("final", [None, torch.float32, torch.bfloat16])
def test_merge_keeps_what_is_not_finite_in_a_weightless_partial(d, final):
    # a partial whose sum is NaN has LSE -inf as well (0 x NaN and 0 x inf are NaN); the other columns of its rows and both rows' LSE stay; a running LSE of
    # +inf leaves no weights at all
    g = torch.Generator().manual_seed(d + 1)
    rows, nq = 37, 3
    oa, ob, la = torch.randn((rows, nq, d), generator=g), torch.randn((rows, nq, d), generator=g), torch.randn((nq, rows), generator=g)
    lb = torch.full((nq, rows), -float("inf"))
    ob[3, :, :], ob[8, 1, d - 1], ob[9, 2, 0], la[0, 30] = float("nan"), float("nan"), float("inf"), float("inf")
    og, lg = oa.clone().to(DEV), la.clone().to(DEV)
    out = None if final is None else torch.empty((rows, nq, d), dtype=final, device=DEV)
    hexi.hexi_attn_merge_lse(og, lg, ob.to(DEV), lb.to(DEV), out)
    want, lse = oa + 0.0 * ob, la.clone()
    want[30, 0], lse[0, 30] = float("nan"), float("nan")
    assert torch.equal(torch.isnan(og.cpu()), torch.isnan(want)) and torch.equal(og.cpu().nan_to_num(), want.nan_to_num())
    assert torch.equal(lg.cpu().isnan(), lse.isnan()) and torch.equal(lg.cpu().nan_to_num(), lse.nan_to_num())
    if final is not None:
        assert torch.equal(out.isnan(), og.isnan()) and torch.equal(out.nan_to_num(), og.to(final).nan_to_num())


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("chunk", [0, 2])
def test_a_poisoned_chunk_is_not_left_out_of_an_unfused_replay(dtype, chunk):
    # NaN in one key, and finite q and k whose score overflows to +inf: the rows that see them are NaN in o, with the merges apart as with the fused ones
    w = _custom(f"poison_{dtype}", dtype, 4, 2, 128, 1200, [(700, 500)], [[(300 * j, 300)] for j in range(4)])
    inputs = wl.make_inputs(w, 5)
    inputs["k"][300 * chunk + 17, 0] = float("nan")
    inputs["k"][300 * chunk + 100, 1, 0] = 3e38
    inputs["q"][:, 2:, 0] = 0.0
    inputs["q"][::5, 2, 0] = 100.0
    got = []
    for fused in (True, False):
        run = replay.ShardRun(w, inputs, DEV, fused_merge=fused)
        run.forward()
        got.append(run.o.cpu())
    sees = (torch.arange(700, 1200) >= 300 * chunk + 100)
    assert all(o[sees][:, :2].isnan().all() and o[sees][::5, 2].isnan().all() and not o[:, 3].isnan().any() for o in got)
    assert torch.equal(got[0].isnan(), got[1].isnan())


@pytest.mark.parametrize("lq,nq,d", [(1, 1, 64), (33, 3, 128), (1000, 5, 64)])
def test_partial_of_a_chunk_in_the_future(lq, nq, d):
    # o = 0 and lse = -inf, whatever was there
    q = torch.ones((lq, nq, d), dtype=torch.bfloat16, device=DEV)
    o, lse = torch.full((lq * nq * d + 8,), float("nan"), device=DEV), torch.full((nq * lq + 8,), 7.0, device=DEV)
    hexi.hexi_attn_fwd_chunk(hexi.desc_for(q, q, 1.0), [(0, lq)], [(lq, lq)], q, q, q, o[:lq * nq * d].view(lq, nq, d), lse[:nq * lq].view(nq, lq))
    assert torch.all(o[:lq * nq * d] == 0) and torch.all(torch.isnan(o[lq * nq * d:]))
    assert torch.all(lse[:nq * lq] == -float("inf")) and torch.all(lse[nq * lq:] == 7.0)

"""The work that users of the library have it do, as cases that can be timed and compared.

A case is one device's share of ring attention (its whole replay over the KV chunks it is sent, forward and backward or
forward alone), or the head redistribution either side of the ring, at sizes from a two-thousand-token debugging run
to the 512K-token shard of an 8B-like model.  Every pass goes through the package's public entry points: the replay
(`replay.ShardRun`, one library call per ring step) or the `hexi_a2a_*` calls of the binding.

Fields of a case
  kind      "train": forward and backward of the whole replay; "forward": forward replay with the fused merge (evaluation,
            or the recomputation of a checkpointed layer); "unfused": forward replay with a partial per ring step and a
            separate log-sum-exp merge; "exchange": pack of the fused q / k / v heads for the ragged all-to-all and
            unpack of the heads that come back.
  dtype, head_dim, nq, nkv   element type, columns, local q and kv heads
  layout, l_tot, ranks, rank, cut_seed
            how the sequence lies over the ring: "zigzag" (2 x ranks equal blocks, a pair per rank), "even" (equal
            contiguous shards) or "uneven" (contiguous shards of seeded uneven lengths; asymmetric groups)
  k_scale   K is multiplied by it (above 1: sharply peaked rows)
  tokens, head_seed          "exchange": tokens of the shard; seed of the per-rank head counts and of the head order
"""
import math
import random

import torch

from paper_2605_07569_amd import hexi, replay
from paper_2605_07569_amd import workloads as wl

DEV = "cuda:0"


def _attn(name, kind, dtype, d, nq, nkv, layout, l_tot, ranks, rank, cut_seed=0, k_scale=1.0):
    c = dict(kind=kind, dtype=dtype, head_dim=d, nq=nq, nkv=nkv, layout=layout, l_tot=l_tot, ranks=ranks, rank=rank,
             cut_seed=cut_seed, k_scale=k_scale)
    return dict(name=name, **c) if name else c


def _exchange(name, dtype, d, nq, nkv, tokens, ranks, head_seed):
    c = dict(kind="exchange", dtype=dtype, head_dim=d, nq=nq, nkv=nkv, tokens=tokens, ranks=ranks, head_seed=head_seed)
    return dict(name=name, **c) if name else c


def listed():
    return [
        # a smoke run: the smallest zigzag shard that a developer starts to see that everything works; launches and host time
        _attn("smoke_zigzag", "train", "bf16", 128, 4, 2, "zigzag", 2048, 4, 1),
        # the fp32 parity configuration: 1024 of 2048 tokens, numerics debugging without reduced precision
        _attn("fp32_tiny", "train", "f32", 64, 4, 4, "even", 2048, 2, 1),
        # the same check on a longer, asymmetric, odd-sized shard with 128-column GQA heads
        _attn("fp32_uneven", "train", "f32", 128, 6, 2, "uneven", 12011, 4, 2, cut_seed=5),
        # evaluation of a short context: one head group of a large model, 1024 rows per device
        _attn("short_forward", "forward", "bf16", 128, 8, 1, "even", 4096, 4, 3),
        # a 3B-like layer at an 8K context over 8 devices (zigzag): the common short training context
        _attn("short_zigzag", "train", "bf16", 128, 24, 8, "zigzag", 8192, 8, 0),
        # asymmetric groups at a 20K context: odd shard lengths, 12 of an 8B-like model's heads
        _attn("uneven_20k", "train", "bf16", 128, 12, 3, "uneven", 20011, 5, 2, cut_seed=3),
        # 64-column heads (smaller models) at a 32K context, 4096 rows per device
        _attn("heads64_32k", "train", "bf16", 64, 24, 8, "zigzag", 32768, 8, 3),
        # forward with one partial per ring step and the separate merge, 32K context
        _attn("unfused_32k", "unfused", "bf16", 128, 24, 8, "zigzag", 32768, 8, 5),
        # the 3B-like 128K context over 8 devices
        _attn("zigzag_128k", "train", "bf16", 128, 24, 8, "zigzag", 131072, 8, 0),
        # forward of one head group (8 q / 1 kv) of a 70B-like model at 1M tokens: 32 ring steps, half of them in the future
        _attn("forward_1m", "forward", "bf16", 128, 8, 1, "even", 1048576, 32, 15),
        # the largest single-device shard: 8B-like, 512K tokens over 16 devices, peaked rows
        _attn("zigzag_512k", "train", "bf16", 128, 32, 8, "zigzag", 524288, 16, 3, k_scale=3.0),
        # head redistribution of a 16K-token shard, 3B-like heads, eight ranks with uneven head counts
        _exchange("exchange_16k", "bf16", 128, 24, 8, 16384, 8, 1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    while True:
        kind = rng.choice(["train", "train", "train", "forward", "unfused", "exchange"])
        d = rng.choice([128, 128, 64])
        nkv = rng.choice([1, 2, 3, 4, 8])
        nq = nkv * rng.choice([1, 2, 3, 4, 8])
        if kind == "exchange":
            ranks = rng.randint(2, 8)
            c = _exchange(None, rng.choice(["bf16", "bf16", "f32"]), d, nq, nkv, _log_int(rng, 300, 40000), ranks, rng.randint(1, 999))
            if nq + 2 * nkv * ranks > 250 or nq < ranks:
                continue
            return c
        dtype = "f32" if kind != "unfused" and rng.random() < 0.25 else "bf16"
        layout = rng.choice(["zigzag", "even", "uneven", "uneven"])
        ranks = rng.randint(2, 16)
        l_tot = _log_int(rng, 1500, 16000 if dtype == "f32" else 300000)
        if layout == "uneven":
            if l_tot < 200 * ranks:
                continue
        else:
            parts = 2 * ranks if layout == "zigzag" else ranks
            l_tot = max(1, l_tot // parts) * parts
        c = _attn(None, kind, dtype, d, nq, nkv, layout, l_tot, ranks, rng.randrange(ranks),
                  cut_seed=rng.randint(1, 999) if layout == "uneven" else 0, k_scale=rng.choice([1.0, 1.0, 3.0]))
        if nq > 32 or _flops(c) > (4e11 if dtype == "f32" else 1.5e14) or l_tot * nkv * d > 1 << 30:
            continue
        return c


def _workload(c):
    lt, r = c["l_tot"], c["ranks"]
    if c["layout"] == "zigzag":
        shards = [wl.zigzag_segs(j, r, lt) for j in range(r)]
    elif c["layout"] == "even":
        shards = [[(j * (lt // r), lt // r)] for j in range(r)]
    else:       # parts between about half and twice the mean, any token counts
        rng = random.Random(c["cut_seed"])
        w = [rng.uniform(0.5, 2.0) for _ in range(r)]
        edges = [round(lt * sum(w[:j]) / sum(w)) for j in range(r)] + [lt]
        shards = [[(a, b - a)] for a, b in zip(edges[:-1], edges[1:])]
    return wl.Workload("perf", c["dtype"], c["nq"], c["nkv"], c["head_dim"], lt, shards[c["rank"]], shards, k_scale=c["k_scale"])


def _pairs(c):
    w = _workload(c)
    total = 0
    for q0, qn in w.q_segs:
        for ch in w.chunks:
            for k0, kn in ch:      # row at position p sees min(kn, p - k0 + 1) keys of the segment
                lo, hi = max(q0, k0), min(q0 + qn, k0 + kn)
                if hi > lo:
                    total += (lo - k0 + 1 + hi - k0) * (hi - lo) // 2
                total += kn * max(0, q0 + qn - max(q0, k0 + kn))
    return total


def _flops(c):
    per_pair = 14 if c["kind"] == "train" else 4
    return per_pair * c["head_dim"] * c["nq"] * _pairs(c)


def _normal(seed, shape, dtype, scale=1.0):
    g = torch.Generator(device=DEV).manual_seed(seed)
    x = torch.randn(shape, generator=g, device=DEV, dtype=torch.float32)
    if scale != 1.0:
        x *= scale
    return x.to(dtype)


def _head_lists(c):
    """Per-rank head lists over the fused [q heads | k heads | v heads] axis: uneven q head counts, each rank with the
    kv heads that its q heads read (replicated where a group is split)."""
    rng = random.Random(c["head_seed"])
    nq, nkv, ranks = c["nq"], c["nkv"], c["ranks"]
    cuts = sorted(rng.sample(range(1, nq), ranks - 1))
    q_parts = [list(range(a, b)) for a, b in zip([0] + cuts, cuts + [nq])]
    lists = []
    for q in q_parts:
        kv = sorted({h // (nq // nkv) for h in q})
        lists.append(q + [nq + h for h in kv] + [nq + nkv + h for h in kv])
    return q_parts, lists


def prepare(case, seed):
    c = case
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    d = c["head_dim"]
    if c["kind"] == "exchange":
        q_parts, lists = _head_lists(c)
        n = c["nq"] + 2 * c["nkv"]
        s = c["tokens"]
        return dict(case=c, lists=lists, q_parts=q_parts,
                    qkv=_normal(seed * 8 + 1, (s, n, d), dt),
                    packed=torch.empty(sum(len(x) for x in lists) * s * d, dtype=dt, device=DEV),
                    o_packed=_normal(seed * 8 + 2, (s * c["nq"] * d,), dt),
                    o=torch.empty((s, c["nq"], d), dtype=dt, device=DEV))
    w = _workload(c)
    inputs = dict(q=_normal(seed * 8 + 1, (w.lq, c["nq"], d), dt), d_o=_normal(seed * 8 + 2, (w.lq, c["nq"], d), dt),
                  k=_normal(seed * 8 + 3, (w.l_tot, c["nkv"], d), dt, w.k_scale), v=_normal(seed * 8 + 4, (w.l_tot, c["nkv"], d), dt))
    return dict(case=c, run=replay.ShardRun(w, inputs, DEV, fused_merge=c["kind"] != "unfused"))


def run(state):
    c = state["case"]
    if c["kind"] == "exchange":
        hexi.hexi_a2a_pack(state["qkv"], state["packed"], state["lists"])
        hexi.hexi_a2a_unpack(state["o_packed"], state["o"], state["q_parts"])
        return dict(packed=state["packed"], o=state["o"])
    r = state["run"]
    if c["kind"] == "train":
        r.step()
        return dict(o=r.o, lse=r.lse, dq=r.dq, dk=r.dk, dv=r.dv)
    r.forward()
    return dict(o=r.o, lse=r.lse)


def work(case):
    c = case
    e, d, nq, nkv = (2 if c["dtype"] == "bf16" else 4), c["head_dim"], c["nq"], c["nkv"]
    if c["kind"] == "exchange":
        listed_heads = sum(len(x) for x in _head_lists(c)[1])
        # the fused tensor once, every listed head written; the returned heads read and written
        return dict(bytes=c["tokens"] * d * e * (nq + 2 * nkv + listed_heads + 2 * nq), flops=0)
    w = _workload(c)
    seen = sum(n for ch in w.chunks for s, n in ch if s <= max(q0 + qn - 1 for q0, qn in w.q_segs))
    q_elems, kv_elems = w.lq * nq * d, seen * nkv * d
    b = e * (q_elems + 2 * kv_elems) + 4 * (q_elems + w.lq * nq)                  # q, k, v read; o, lse written
    if c["kind"] == "train":
        b += e * q_elems + 4 * q_elems + 4 * 2 * w.l_tot * nkv * d                # dO read; dq, dk, dv written
    return dict(bytes=b, flops=_flops(c))


def tolerance(case):
    """About four times the largest error of any output against a float64 evaluation of the same inputs (the cases up to a
    32K context, K scaled by 1 and by 3): bf16 1.9e-3 (P and dS are rounded to bf16 as matrix operands) and 1.0e-1 for a
    single element, the dv of keys that few rows weigh; fp32 2.3e-6 and 3.8e-5."""
    if case["kind"] == "exchange":
        return "exact"
    return {"rel": 7e-3, "max": 0.4} if case["dtype"] == "bf16" else {"rel": 1e-5, "max": 1.5e-4}

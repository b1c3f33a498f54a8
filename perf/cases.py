"""The work that a serving program has this library do, as cases that can be
timed and checked: the adapter delta of decode and prompt steps, planned once
or re-planned per iteration, one projection or a whole layer, the two halves
apart, and the base projection fused with the delta.

A case is a dict of plain values:

  path     "plan"   lora_plan_apply / lora_plan_apply_multi on plans made beforehand
           "graph"  the same launches recorded in a HIP graph, replayed
           "replan" lora_plan_update with the iteration's batch, then "plan"
           "fused"  lora_apply_fused (plan uploaded by the call)
           "halves" lora_shrink into a float32 v, then lora_expand from it
           "base"   lora_base_apply (Eq. 1 whole, work list uploaded by the call)
           "base_plan"  lora_base_plan_apply on a plan made beforehand
  groups   the projections of one layer: "h_in:h_out,h_out;h_in:h_out"; those
           of one group read the same x and run as one launch
  layers   layers of those projections that one pass runs
  dtype    "f16" or "bf16"
  decode   single-token segments; plain: how many of all segments carry no adapter
  prompts, len_lo, len_hi   prompt segments and the range of their lengths
  adapters, ranks, law      registered adapters, their ranks ("8,16"), and which
           segment uses which: "zipf" (1.1), "each" (segment s uses adapter s,
           round robin)
  scale    s_g of every adapter, 0 for 16 / r
  batch    seed of the batch's structure (ranks, adapters, lengths)

Inputs are normal: x ~ N(0, 1), A ~ N(0, 1/h_in), B ~ N(0, 1/r), y ~ N(0, 1),
W ~ N(0, 1/h_in), rounded to the storage type, as in the repository's
workloads.
"""
from __future__ import annotations

import random

import numpy as np
import torch

from paper_2401_11240_amd import lora as L

TORCH_DTYPE = {"f16": torch.float16, "bf16": torch.bfloat16}
LORA_DTYPE = {"f16": L.LORA_F16, "bf16": L.LORA_BF16}


def _case(path, groups, dtype, *, layers=1, decode=0, plain=0, prompts=0, len_lo=0, len_hi=0, adapters=1, ranks="16",
          law="zipf", scale=0.0, batch=0, **more):
    return dict(path=path, groups=groups, layers=layers, dtype=dtype, decode=decode, plain=plain, prompts=prompts,
                len_lo=len_lo, len_hi=len_hi, adapters=adapters, ranks=ranks, law=law, scale=scale, batch=batch, **more)


def listed():
    return [
        # The smallest call: a handful of tokens on one projection, rank 8,
        # called eagerly (the repository's 8-token decode workload).
        _case("plan", "4096:4096", "f16", decode=8, adapters=4, ranks="8", law="each", scale=2.0, name="decode_t8_r8"),
        # An ordinary decode step, mixed ranks, recorded in a graph as a
        # decode loop records it: one projection of eight layers.
        _case("graph", "4096:4096", "f16", layers=8, decode=64, adapters=32, ranks="8,16,32,64", batch=1,
              name="decode_t64_graph"),
        # Continuous batching: the batch changes, the plan is updated, then
        # the q, k, v and o projections of two layers run it.
        _case("replan", "4096:4096;4096:4096;4096:4096;4096:4096", "f16", layers=2, decode=48, adapters=64,
              ranks="8,16,32,64", batch=6, name="decode_t48_replan"),
        # Every adapted projection of a 13B-shaped layer at 128 decode tokens,
        # projections that share their input in one launch.
        _case("plan", "5120:5120,5120,5120;5120:5120;5120:13824,13824;13824:5120", "bf16", decode=128, adapters=64,
              ranks="8,16,32,64", batch=3, name="decode_13b_layer"),
        # A prompt step: 16 prompts, each with its own adapter.
        _case("plan", "4096:4096", "bf16", prompts=16, len_lo=64, len_hi=1024, adapters=16, ranks="8,16,32,64",
              law="each", batch=2, name="prefill_16seg"),
        # One short prompt with a rank-16 adapter, planned by the call itself.
        _case("fused", "4096:4096", "f16", prompts=1, len_lo=203, len_hi=203, adapters=1, ranks="16", law="each",
              name="prefill_l203_fused"),
        # A mixed step of 70B-shaped projections: decode tokens and prompts
        # together, q and gate in one launch.
        _case("plan", "8192:8192,28672", "bf16", decode=256, prompts=4, len_lo=512, len_hi=512, adapters=128,
              ranks="8,16,32,64,128", batch=4, name="mixed_70b"),
        # Ragged: widths that no tile divides, small and odd ranks, rows
        # without an adapter, decode tokens beside two prompts.
        _case("plan", "2056:5640", "f16", decode=37, plain=9, prompts=2, len_lo=75, len_hi=301, adapters=12,
              ranks="4,12,20,40", batch=8, name="mixed_ragged"),
        # The two halves apart, as a row-parallel shard uses them (v can be
        # summed over ranks in between).
        _case("halves", "3456:5120", "bf16", decode=32, prompts=3, len_lo=100, len_hi=600, adapters=20,
              ranks="16,64", batch=9, name="halves_shard"),
        # Eq. 1 whole for one 1024-token prompt.
        _case("base_plan", "4096:4096", "bf16", prompts=1, len_lo=1024, len_hi=1024, adapters=1, ranks="64", law="each",
              batch=5, name="base_l1024"),
        # Eq. 1 whole for the prompt step of 16 prompts.
        _case("base_plan", "4096:4096", "bf16", prompts=16, len_lo=64, len_hi=1024, adapters=16, ranks="8,16,32,64",
              law="each", batch=2, name="base_16seg"),
        # Eq. 1 whole for a few ragged prompts on a wide projection, planned
        # by the call itself.
        _case("base", "5120:13824", "f16", plain=1, prompts=4, len_lo=33, len_hi=260, adapters=4, ranks="8,32",
              law="each", batch=11, name="base_ragged_f16"),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(lo * (hi / lo) ** rng.random()))))


def _width(rng, lo=1024, hi=14336):
    return 8 * _log_int(rng, lo // 8, hi // 8)


def draw(rng: random.Random):
    """One more case of the listed ones' ranges."""
    while True:
        path = rng.choice(("plan", "plan", "plan", "graph", "replan", "fused", "halves", "base_plan", "base"))
        dtype = rng.choice(("f16", "bf16"))
        base = path in ("base", "base_plan")
        kind = "prompt" if base else rng.choice(("decode", "prompt", "mixed"))
        c = dict(decode=0, prompts=0, len_lo=0, len_hi=0)
        if kind != "prompt":
            c["decode"] = _log_int(rng, 1, 256)
        if kind != "decode":
            c["prompts"] = _log_int(rng, 1, 16)
            c["len_lo"] = _log_int(rng, 17, 512)
            c["len_hi"] = min(1024, c["len_lo"] + _log_int(rng, 1, 512))
        n_seg = c["decode"] + c["prompts"]
        c["plain"] = rng.choice((0, 0, n_seg // 5))
        c["adapters"] = _log_int(rng, 1, 128)
        c["ranks"] = rng.choice(("8", "16", "64", "8,16,32,64", "8,16,32,64,128", "16,64", "4,12,20,40"))
        c["law"] = rng.choice(("zipf", "each"))
        c["scale"] = rng.choice((0.0, 2.0))
        c["batch"] = rng.randrange(1 << 20)
        h_in = rng.choice((4096, 5120, 8192, _width(rng), _width(rng)))
        outs = [rng.choice((4096, 5120, 8192, 13824, _width(rng), _width(rng)))]
        if path in ("plan", "graph") and rng.random() < 0.4:
            outs += [rng.choice((outs[0], _width(rng))) for _ in range(rng.choice((1, 2)))]
        layers = rng.choice((1, 2, 4)) if path in ("plan", "graph", "replan") else 1
        case = _case(path, "%d:%s" % (h_in, ",".join(map(str, outs))), dtype, layers=layers, **c)
        w = work(case)
        if w["bytes"] <= 0.55e9 and w["flops"] <= 2.8e11:
            return case


# ---------------------------------------------------------------------------
# the batch and the shapes of a case
# ---------------------------------------------------------------------------

def _groups(case):
    out = []
    for g in case["groups"].split(";"):
        h_in, outs = g.split(":")
        out.append((int(h_in), [int(v) for v in outs.split(",")]))
    return out


def _batch(case):
    """(seg_offset, seg_adapter, ranks, scales) of the case: the same for every seed."""
    rng = np.random.default_rng(case["batch"])
    n = case["adapters"]
    choices = np.array([int(v) for v in case["ranks"].split(",")], dtype=np.int32)
    ranks = rng.choice(choices, size=n).astype(np.int32)
    n_seg = case["decode"] + case["prompts"]
    if case["law"] == "zipf":
        p = np.arange(1, n + 1, dtype=np.float64) ** -1.1
        seg = rng.choice(n, size=n_seg, p=p / p.sum()).astype(np.int32)
    else:
        seg = (np.arange(n_seg) % n).astype(np.int32)
    if case["plain"]:
        seg[rng.choice(n_seg, size=min(case["plain"], n_seg - 1), replace=False)] = -1
    lens = np.ones(n_seg, dtype=np.int64)
    if case["prompts"]:
        lens[case["decode"]:] = rng.integers(case["len_lo"], case["len_hi"] + 1, size=case["prompts"])
    off = np.zeros(n_seg + 1, dtype=np.int32)
    off[1:] = np.cumsum(lens)
    scales = (16.0 / ranks if case["scale"] == 0 else np.full(n, case["scale"])).astype(np.float32)
    return off, seg, ranks, scales


def work(case):
    """Factors of every adapter in use, x of adapted rows and y (read and
    written) once; with the base weight: all of x and W read, y written."""
    off, seg, ranks, _ = _batch(case)
    lens = np.diff(off)
    used = np.unique(seg[seg >= 0])
    rows = int(lens[seg >= 0].sum())
    rank_sum = int(ranks[used].sum())
    rank_rows = int((ranks[seg[seg >= 0]].astype(np.int64) * lens[seg >= 0]).sum())
    base = case["path"] in ("base", "base_plan")
    nbytes = flops = 0
    for h_in, outs in _groups(case):
        nbytes += 2 * (int(off[-1]) if base else rows) * h_in
        for h_out in outs:
            nbytes += 2 * rank_sum * (h_in + h_out)
            flops += 2 * rank_rows * (h_in + h_out)
            if base:
                nbytes += 2 * (h_in * h_out + int(off[-1]) * h_out)
                flops += 2 * int(off[-1]) * h_in * h_out
            else:
                nbytes += 4 * rows * h_out
            if case["path"] == "halves":
                nbytes += 4 * 2 * rank_rows
    return {"bytes": nbytes * case["layers"], "flops": flops * case["layers"]}


def tolerance(case):
    # Against 64 bits the path is off by the one rounding of y: 1.7e-3 in
    # bfloat16, 2.1e-4 in binary16 (relative 2-norm); the float32 v of the two
    # halves by about 2e-7, far inside either.  A result may fall on the other
    # side of a rounding boundary, one unit of the last place: 2^-7 of the value
    # in bfloat16, 2^-10 in binary16.
    if case["dtype"] == "bf16":
        return {"rel": 6e-3, "max": 2.0 ** -6}
    return {"rel": 8e-4, "max": 2.0 ** -9}


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _inputs(case, seed):
    """Per layer and group: x, and per projection A and B of every adapter (two
    packed buffers), y or W."""
    off, _, ranks, _ = _batch(case)
    n_rows = int(off[-1])
    dtype = TORCH_DTYPE[case["dtype"]]
    dev = torch.device("cuda:0")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)

    def normal(shape, std=1.0):
        t = torch.randn(shape, generator=gen, device=dev, dtype=torch.float32)
        return (t if std == 1.0 else t.mul_(std)).to(dtype)

    rank_std = torch.from_numpy(np.repeat(1.0 / np.sqrt(ranks.astype(np.float32)), ranks)).to(dev)
    base = case["path"] in ("base", "base_plan")
    total = int(ranks.sum())
    out = []
    for _ in range(case["layers"]):
        for h_in, outs in _groups(case):
            projs = []
            x = normal((n_rows, h_in))
            for h_out in outs:
                A = normal((total * h_in,), h_in ** -0.5)     # adapter after adapter, each [h_in, r]
                B = torch.randn((total, h_out), generator=gen, device=dev, dtype=torch.float32)
                B = B.mul_(rank_std[:, None]).to(dtype)       # adapter after adapter, each [r, h_out]
                p = dict(h_in=h_in, h_out=h_out, A=A, B=B)
                if base:
                    p["wt"] = normal((h_out, h_in), h_in ** -0.5)
                    p["y"] = torch.zeros((n_rows, h_out), dtype=dtype, device=dev)
                else:
                    p["y"] = normal((n_rows, h_out))
                projs.append(p)
            out.append((x, projs))
    return out


class _State:
    """Inputs on the GPU, adapter tables, plans, and what else a program keeps."""

    def __init__(self, case, seed):
        off, seg, ranks, scales = _batch(case)
        self.path = case["path"]
        self.inputs = _inputs(case, seed)
        self.batch = L.Batch(off, seg)
        self.stream = torch.cuda.current_stream()
        self.tables = []                 # per layer and group: a table per projection
        self.plans = {}                  # per shape
        self.base_plan = 0
        starts = np.concatenate([[0], np.cumsum(ranks)])[:-1].astype(np.int64)
        for x, projs in self.inputs:
            row = []
            for p in projs:
                a, b = p["A"].data_ptr(), p["B"].data_ptr()
                row.append(L.lora_register_adapters(
                    0, p["h_in"], p["h_out"], LORA_DTYPE[case["dtype"]],
                    [a + 2 * int(s) * p["h_in"] for s in starts], [b + 2 * int(s) * p["h_out"] for s in starts],
                    ranks, scales, self.stream))
            self.tables.append(row)
        t0, p0 = self.tables[0][0], self.inputs[0][1][0]
        if self.path in ("plan", "graph", "replan"):
            self.keys = []
            for (x, projs), row in zip(self.inputs, self.tables):
                key = (projs[0]["h_in"],) + tuple(p["h_out"] for p in projs)
                self.keys.append(key)
                if key not in self.plans:
                    self.plans[key] = (L.lora_plan_create(row[0], self.batch, self.stream) if len(row) == 1 else
                                       L.lora_plan_create_multi(row, self.batch, self.stream))
        elif self.path == "base_plan":
            self.base_plan = L.lora_base_plan_create(t0, self.batch, self.stream)
        else:
            n = L.lora_base_workspace_bytes(t0, self.batch) if self.path == "base" else L.lora_workspace_bytes(t0, self.batch)
            self.ws = torch.empty(n, dtype=torch.uint8, device="cuda:0")
            if self.path == "halves":
                self.v = torch.zeros((self.batch.n_rows, (int(ranks.max()) + 7) // 8 * 8), dtype=torch.float32,
                                     device="cuda:0")
        self.ys = [p["y"] for _, projs in self.inputs for p in projs]
        if self.path == "graph":
            self.graph = torch.cuda.CUDAGraph()
            torch.cuda.synchronize()
            with torch.cuda.graph(self.graph):
                self.apply(torch.cuda.current_stream())

    def apply(self, stream):
        for (x, projs), row, key in zip(self.inputs, self.tables, self.keys):
            plan = self.plans[key]
            if len(row) == 1:
                L.lora_plan_apply(plan, row[0], x, x.shape[1], projs[0]["y"], projs[0]["h_out"], stream)
            else:
                L.lora_plan_apply_multi(plan, row, x, x.shape[1], [p["y"] for p in projs],
                                        [p["h_out"] for p in projs], stream)

    def __del__(self):
        try:
            torch.cuda.synchronize()
            if self.path == "graph":
                del self.graph
            for plan in self.plans.values():
                L.lora_plan_destroy(plan)
            if self.base_plan:
                L.lora_base_plan_destroy(self.base_plan)
            for row in self.tables:
                for t in row:
                    L.lora_release_adapters(t)
        except Exception:
            pass


def prepare(case, seed):
    return _State(case, seed)


def run(state):
    s = state
    path = s.path
    if path == "graph":
        s.graph.replay()
        return s.ys
    stream = s.stream
    if path == "plan":
        s.apply(stream)
        return s.ys
    if path == "replan":
        for plan in s.plans.values():
            L.lora_plan_update(plan, None, s.batch, stream)
        s.apply(stream)
        return s.ys
    x, projs = s.inputs[0]
    p, t = projs[0], s.tables[0][0]
    if path == "fused":
        L.lora_apply_fused(t, s.batch, x, p["h_in"], p["y"], p["h_out"], s.ws, s.ws.numel(), stream)
    elif path == "halves":
        ldv = s.v.shape[1]
        L.lora_shrink(t, s.batch, x, p["h_in"], s.v, ldv, s.ws, s.ws.numel(), stream)
        L.lora_expand(t, s.batch, s.v, ldv, p["y"], p["h_out"], s.ws, s.ws.numel(), stream)
        return [s.v, p["y"]]
    elif path == "base":
        L.lora_base_apply(t, s.batch, x, p["h_in"], p["wt"], p["h_in"], p["y"], p["h_out"], s.ws, s.ws.numel(), stream)
    else:
        L.lora_base_plan_apply(s.base_plan, t, x, p["h_in"], p["wt"], p["h_in"], p["y"], p["h_out"], stream)
    return s.ys


def exact(case, seed):
    off, seg, ranks, scales = _batch(case)
    row_adapter = np.repeat(seg, np.diff(off))
    starts = np.concatenate([[0], np.cumsum(ranks)]).astype(np.int64)
    v_all = None
    ys = []
    for x, projs in _inputs(case, seed):
        xd = x.double()
        for p in projs:
            h_in, h_out = p["h_in"], p["h_out"]
            y = xd @ p["wt"].double().t().contiguous() if "wt" in p else p["y"].double()
            if case["path"] == "halves":
                v_all = torch.zeros((x.shape[0], (int(ranks.max()) + 7) // 8 * 8), dtype=torch.float64, device=x.device)
            for g in np.unique(seg[seg >= 0]):
                r = int(ranks[g])
                rows = torch.from_numpy(np.flatnonzero(row_adapter == g)).to(x.device)
                A = p["A"][int(starts[g]) * h_in:int(starts[g + 1]) * h_in].view(h_in, r).double()
                B = p["B"][int(starts[g]):int(starts[g + 1])].double()
                v = xd[rows] @ A
                y[rows] += float(scales[g]) * (v @ B)
                if v_all is not None:
                    v_all[rows, :r] = v
            ys.append(y)
    return [v_all] + ys if v_all is not None else ys

"""Decode row blocks whose shrink items stream K ranges of several passes (steps
with at least a round of one-pass items): blocks of 1 to 16 rows, ranks with one
to fifteen 16-rank tiles (waves splitting K four, two and one ways), ranks that
are not a multiple of 8 and one too wide to stream beside them, h_in that no
pass divides, prompt blocks cut by bytes in the same step.  Every row against the oracle; the step launch, the separate
launches and a launch of two projections bit for bit.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():   # collected on CPU-only hosts, never run there
    pytest.skip("no GPU", allow_module_level=True)

import oracle  # noqa: E402
from paper_2401_11240_amd import device as D  # noqa: E402
from paper_2401_11240_amd import lora as L  # noqa: E402
from paper_2401_11240_amd import workloads as W  # noqa: E402

from parity import compare, magnitude  # noqa: E402

DEV = torch.device("cuda:0")

# ranks repeat over the adapters; rows per adapter likewise
RANKS = [24, 64, 128, 16, 40, 240, 32, 12, 8, 256, 96, 48]


def workload(dtype, h_in, rows, prompts=()):
    n = 4 * len(RANKS)
    lens, sa = [], []
    for g in range(n):
        for _ in range(rows[g % len(rows)]):   # single tokens, dealt out so that rows of a block are scattered
            lens.append(1)
            sa.append(g)
    order = np.random.default_rng(3).permutation(len(sa))
    sa = [sa[i] for i in order] + [3 * i % n for i in range(len(prompts))]
    lens += prompts
    return W.build_workload(name="stream", seed=31, dtype=dtype, n_adapters=n, fixed_ranks=RANKS * 4,
                            seg_adapter=sa, seg_lens=lens,
                            projections=(("a", h_in, 264, "x"), ("b", h_in, 520, "x")))


# prompt segments beside: blocks of two and four 16-row subtiles, ranks that stream and that do not
PROMPTS = [17, 64, 33, 130, 40]


@pytest.mark.parametrize("dtype,h_in,rows,prompts", [(W.F16, 8200, [1], []), (W.BF16, 6152, [1, 3, 16, 2], []),
                                                     (W.BF16, 8192, [16], []), (W.F16, 6152, [1], PROMPTS),
                                                     (W.BF16, 8200, [1, 2], PROMPTS)])
def test_streamed_ranges(dtype, h_in, rows, prompts):
    print("stream", dtype, h_in, rows, prompts, flush=True)
    w = workload(dtype, h_in, rows, prompts)
    items = L.lora_plan_inspect(L.Batch(w.seg_offset, w.seg_adapter), h_in, 264, w.ranks, 8)
    sh = items[(items["kind"] == 1) & (items["nrows"] <= 16)]
    assert (sh["len"] > sh["sub"]).any()       # the batch takes the streamed path
    if prompts:                                # its larger blocks cut by bytes too: not all into as many ranges
        assert np.unique(items["nsplit"][(items["kind"] == 1) & (items["nrows"] > 16)]).size > 1
    dw = D.upload(w, DEV)
    s = torch.cuda.current_stream(DEV)
    x = dw.xs["x"]
    single = []
    for p, pr in zip(dw.projections, w.projections):
        y = p.y.clone()
        plan = L.lora_plan_create(p.table, dw.batch, s)
        L.lora_plan_apply(plan, p.table, x, h_in, y, p.h_out, s)
        L.lora_plan_status(plan, s)
        got = D.from_device_bits(y)
        ref = oracle.lora_apply(w.seg_offset, w.seg_adapter, w.xs["x"], pr.A, pr.B, w.ranks, w.scales, pr.y, w.dtype)
        compare(got, ref, w.dtype, pr.name, mag=magnitude(w, pr.name))
        y2 = p.y.clone()
        L.lora_plan_shrink(plan, p.table, x, h_in, s)
        L.lora_plan_expand(plan, p.table, y2, p.h_out, s)
        torch.cuda.synchronize()
        assert np.array_equal(D.from_device_bits(y2), got)
        L.lora_plan_destroy(plan)
        single.append(got)
    tables = [p.table for p in dw.projections]
    plan = L.lora_plan_create_multi(tables, dw.batch, s)
    for _ in range(3):                         # both step buffers, and the first again
        ys = [p.y.clone() for p in dw.projections]
        L.lora_plan_apply_multi(plan, tables, x, h_in, ys, [p.h_out for p in dw.projections], s)
        L.lora_plan_status(plan, s)
        for y, ref in zip(ys, single):
            assert np.array_equal(D.from_device_bits(y), ref)
    L.lora_plan_destroy(plan)
    dw.release()


@pytest.mark.parametrize("dtype,ranks", [(W.F16, [8, 12, 8]), (W.BF16, [32, 12, 24])])
def test_long_contraction(dtype, ranks):
    """h_in past what 4096 one-pass K ranges cover: ranges of several passes in
    every body (the token of rank 32 streams, those of rank 8 and 12 go through
    registers)."""
    h_in = 4096 * 512 + 8
    print("long contraction", dtype, ranks, flush=True)
    w = W.build_workload(name="long", seed=5, dtype=dtype, n_adapters=3, fixed_ranks=ranks, seg_adapter=[0, 1, 2],
                         seg_lens=[1, 1, 18], projections=(("proj", h_in, 264, "x"),))
    items = L.lora_plan_inspect(L.Batch(w.seg_offset, w.seg_adapter), h_in, 264, w.ranks, 8)
    sh = items[(items["kind"] == 1) & (items["nrows"] == 1)]
    assert items["nsplit"].max() <= 4096 and np.unique(sh["rank"][sh["len"] > 512]).size == 2
    dw = D.upload(w, DEV)
    p, pr = dw.projections[0], w.projections[0]
    s = torch.cuda.current_stream(DEV)
    plan = L.lora_plan_create(p.table, dw.batch, s)
    y = p.y.clone()
    L.lora_plan_apply(plan, p.table, dw.xs["x"], h_in, y, p.h_out, s)
    L.lora_plan_status(plan, s)
    got = D.from_device_bits(y)
    ref = oracle.lora_apply(w.seg_offset, w.seg_adapter, w.xs["x"], pr.A, pr.B, w.ranks, w.scales, pr.y, w.dtype)
    compare(got, ref, w.dtype, "long contraction", mag=magnitude(w, pr.name))
    y2 = p.y.clone()
    L.lora_plan_shrink(plan, p.table, dw.xs["x"], h_in, s)
    L.lora_plan_expand(plan, p.table, y2, p.h_out, s)
    torch.cuda.synchronize()
    assert np.array_equal(D.from_device_bits(y2), got)
    L.lora_plan_destroy(plan)
    dw.release()


def test_recorded_launch_outlives_the_table():
    """A recorded streamed step of up to 128 adapters carries their pointers and
    scales, as every other step does: it replays after the table is released."""
    print("recorded, table released", flush=True)
    w = workload(W.BF16, 6152, [1])
    dw = D.upload(w, DEV)
    p, pr, x = dw.projections[0], w.projections[0], dw.xs["x"]
    s = torch.cuda.current_stream(DEV)
    plan = L.lora_plan_create(p.table, dw.batch, s)
    y = p.y.clone()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        L.lora_plan_apply(plan, p.table, x, x.shape[1], y, p.h_out, torch.cuda.current_stream(DEV))
    dw.release()
    ref = oracle.lora_apply(w.seg_offset, w.seg_adapter, w.xs["x"], pr.A, pr.B, w.ranks, w.scales, pr.y, w.dtype)
    for _ in range(3):
        y.copy_(p.y)
        g.replay()
        L.lora_plan_status(plan, s)
        compare(D.from_device_bits(y), ref, w.dtype, pr.name, mag=magnitude(w, pr.name))
    del g
    L.lora_plan_destroy(plan)

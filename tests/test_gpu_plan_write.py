"""The kernel that writes a work list into device memory, at the edges of what
one launch of it carries (896 words: 64 row blocks of consecutive rows, fewer
when their rows are listed): batches of 64, 65, 66 and 131 row blocks, blocks of
1 to 64 scattered rows, so many of them that the list is read from pinned memory,
a batch of one row and a plan updated from one to the other, through the one-shot
call, the plan and the base projection (whose tile list rides in the same
launches).  Every row against the oracle; the two delta forms bit for bit.
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
from test_gpu_base import oracle_rows, run_base, allowance  # noqa: E402

DEV = torch.device("cuda:0")


def interleaved(n_ad, per):
    """per rows of each of n_ad adapters, dealt out in turn: no two consecutive."""
    return [1] * (n_ad * per), [i % n_ad for i in range(n_ad * per)]


CASES = {
    "one": ([1], [0], 1),
    "64": ([1] * 64, list(range(64)), 64),
    "65": ([1] * 65, list(range(65)), 65),
    "66": ([1] * 66, list(range(66)), 66),
    "131": ([2] * 131, list(range(131)), 131),
    "scattered16": interleaved(40, 16) + (40,),
    "scattered64": interleaved(15, 64) + (15,),
    "scattered70": interleaved(14, 70) + (14,),
    "scattered5000": interleaved(10, 500) + (10,),
    "mixed": ([1, 200, 1, 1, 64, 1, 65, 3], [0, 1, 2, 0, 3, -1, 1, 0], 4),
}


def workload(name, base=False):
    lens, sa, n_ad = CASES[name]
    return W.build_workload(name=name, seed=77, dtype=W.BF16, n_adapters=n_ad, rank_set=[4, 8, 16, 24],
                            seg_adapter=sa, seg_lens=lens, projections=(("proj", 136, 264, "x"),), base_weight=base)


def run(dw, plan):
    p, x = dw.projection("proj"), dw.xs["x"]
    s = torch.cuda.current_stream(DEV)
    y = p.y.clone()
    if plan:
        L.lora_plan_apply(plan, p.table, x, x.shape[1], y, y.shape[1], s)
        L.lora_plan_status(plan, s)
    else:
        n = L.lora_workspace_bytes(p.table, dw.batch)
        ws = torch.full((n,), 0xAB, dtype=torch.uint8, device=DEV)   # any contents
        L.lora_apply_fused(p.table, dw.batch, x, x.shape[1], y, y.shape[1], ws, n, s)
    torch.cuda.synchronize()
    return D.from_device_bits(y)


@pytest.mark.parametrize("name", list(CASES))
def test_written_lists(name):
    print("plan write", name, flush=True)
    w = workload(name)
    dw = D.upload(w, DEV)
    t = dw.projection("proj").table
    pr = w.projections[0]
    ref = oracle.lora_apply(w.seg_offset, w.seg_adapter, w.xs["x"], pr.A, pr.B, w.ranks, w.scales, pr.y, w.dtype)
    got = run(dw, 0)
    compare(got, ref, w.dtype, name, mag=magnitude(w, "proj"))
    plan = L.lora_plan_create(t, dw.batch)
    assert np.array_equal(run(dw, plan), got)
    assert np.array_equal(run(dw, plan), got)          # the other step buffer
    # through a plan that held another batch before
    other = workload("scattered16" if name != "scattered16" else "66")
    do = D.upload(other, DEV)
    to = do.projection("proj").table
    room = max(L.lora_plan_bytes(t, dw.batch), L.lora_plan_bytes(to, do.batch))
    p2 = L.lora_plan_create_reserved(to, do.batch, room)
    first = run(do, p2)
    L.lora_plan_update(p2, t, dw.batch)
    assert np.array_equal(run(dw, p2), got)
    L.lora_plan_update(p2, to, do.batch)
    assert np.array_equal(run(do, p2), first)
    for q in (plan, p2):
        L.lora_plan_destroy(q)
    dw.release()
    do.release()


@pytest.mark.parametrize("name", ["one", "65", "scattered64", "scattered5000", "mixed"])
def test_written_base_tiles(name):
    print("base tiles", name, flush=True)
    w = workload(name, base=True)
    dw = D.upload(w, DEV)
    rows = np.arange(w.n_rows)
    compare(run_base(dw, w), oracle_rows(w, rows), w.dtype, name, mag=allowance(w, rows))
    dw.release()


def test_pinned_slots_in_turn():
    """Lists read from pinned memory, call after call with no wait between, past the
    number of slots: two batches in turn, each call with its own rows."""
    print("pinned slots", flush=True)
    lens, sa, n_ad = CASES["scattered5000"]
    w = workload("scattered5000")
    dw = D.upload(w, DEV)
    p, x = dw.projection("proj"), dw.xs["x"]
    s = torch.cuda.current_stream(DEV)
    batches = [dw.batch, L.Batch(w.seg_offset, [(7 * a + 3) % n_ad for a in sa])]
    room = max(L.lora_workspace_bytes(p.table, b) for b in batches)
    ws = torch.empty(room, dtype=torch.uint8, device=DEV)
    ys = [p.y.clone() for _ in range(24)]
    for i, y in enumerate(ys):
        L.lora_apply_fused(p.table, batches[i % 2], x, x.shape[1], y, y.shape[1], ws, room, s)
    torch.cuda.synchronize()
    pr = w.projections[0]
    for k in (0, 1):
        ref = oracle.lora_apply(w.seg_offset, np.asarray(batches[k].seg_adapter), w.xs["x"], pr.A, pr.B, w.ranks, w.scales,
                                pr.y, w.dtype)
        got = D.from_device_bits(ys[k])
        compare(got, ref, w.dtype, f"batch {k}")
        for y in ys[k::2]:
            assert np.array_equal(D.from_device_bits(y), got)
    dw.release()

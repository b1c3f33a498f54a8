"""The fused base GEMM's step ring at its edges, against the oracle: h_in of
one 16-byte chunk, around one K-64 step, and shorter than, as long as and just
past the ring (2 steps in tiles of 256, 4 in tiles of 128); rows and columns one
past a tile; ranks around the 4, 8 and 64 that the staged factors come in; and
a binary16 intermediate past 2^15 in tiles of 256.  Tolerance as in
test_gpu_base.py (the oracle's rounding plus the float32 sums of h_in products).
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu

if not torch.cuda.is_available():   # collected on CPU-only hosts, never run there
    pytest.skip("no GPU", allow_module_level=True)

from paper_2401_11240_amd import device as D  # noqa: E402
from paper_2401_11240_amd import workloads as W  # noqa: E402

from parity import compare  # noqa: E402
from test_gpu_base import DEV, allowance, oracle_rows, run_base, say, small_case  # noqa: E402

KS = [8, 56, 64, 72, 128, 136, 248, 256, 264, 320]


@pytest.mark.parametrize("dtype", [W.F16, W.BF16])
@pytest.mark.parametrize("h_in", KS)
def test_small_tile_steps(h_in, dtype):
    say(f"ring, tiles of 128: h_in={h_in} dtype={dtype}")
    ranks = [1 + h_in % 7, 63, 65, 12]
    w = small_case(400 + h_in, dtype, h_in, 136, ranks, [1, 70, 58, 128, 3], [0, 1, 2, 3, -1])
    dw = D.upload(w, DEV)
    rows = np.arange(w.n_rows)
    st = compare(run_base(dw, w), oracle_rows(w, rows), w.dtype, f"h_in {h_in}", mag=allowance(w, rows))
    say("  ", st)
    dw.release()


@pytest.mark.parametrize("dtype", [W.F16, W.BF16])
@pytest.mark.parametrize("h_in", [8, 64, 120, 136, 200])
def test_big_tile_steps(h_in, dtype):
    """4097 x 4104: 289 tiles of 256, the last of one row and of eight columns;
    the oracle on the rows at the edges of tiles and segments."""
    say(f"ring, tiles of 256: h_in={h_in} dtype={dtype}")
    lens = [255, 3, 1790, 2049]
    w = small_case(500 + h_in, dtype, h_in, 4104, [5, 64, 72], lens, [0, 1, -1, 2])
    if dtype == W.F16:
        w.scales[1] = 3e4                     # s_g v past 2^15 beside runs that stay below; the delta within range
        B = w.projections[0].B
        B[1] = W.normal_bits(np.random.default_rng(1), B[1].shape, 0.005, dtype)
    dw = D.upload(w, DEV)
    got = run_base(dw, w)
    off = w.seg_offset
    rows = np.unique(np.concatenate([off[:-1], off[1:] - 1, np.arange(0, 4097, 256), np.arange(255, 4097, 256)]))
    ref = oracle_rows(w, rows)
    assert np.all(np.abs(ref) < 65000)
    st = compare(got[rows], ref, w.dtype, f"h_in {h_in}", mag=allowance(w, rows))
    say("  ", st)
    dw.release()

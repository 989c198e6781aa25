"""GPU parity of Algorithm 3 (turbo_sas_softmax) against the oracle's
sas_softmax_rows.

The SAS values are the same binary32 operations on both sides; the row sum is
fp32 on the GPU (at most 64 sequential additions per lane, then a tree) and
double in the oracle, and the GPU divides in fp32.  Each output is therefore
within (64 + 16 + 2) * 2^-24 < 1e-5 of the oracle's, relative to itself; zeros
(scores more than 6 below the row maximum, -inf) are exact.
"""
import sys

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

REL_TOL = 1e-5


def _log(msg):
    print(msg, flush=True)
    sys.stdout.flush()


@pytest.fixture(scope="module")
def dev():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    return torch.device("cuda:0")


@pytest.fixture(scope="module")
def ta(dev):
    import paper_2412_08585_amd as ta
    ta.lib()
    return ta


def _scores(rows, cols, seed, std=2.0):
    g = torch.Generator().manual_seed(seed)
    return torch.randn(rows, cols, generator=g) * std


def _check(got: torch.Tensor, ref: np.ndarray, what: str):
    g = got.cpu().numpy().astype(np.float64)
    assert np.array_equal(g == 0, ref == 0), f"{what}: zero pattern"
    nz = ref != 0
    if nz.any():
        worst = float(np.max(np.abs(g[nz] - ref[nz]) / ref[nz]))
        assert worst < REL_TOL, f"{what}: max relative error {worst:.3e}"
    np.testing.assert_allclose(g.sum(axis=1), 1.0, rtol=1e-5)


SHAPES = [(7, 1), (5, 3), (33, 64), (9, 250), (4, 257), (6, 1000), (5, 2048), (3, 2049),
          (3, 4096), (2, 5000), (2, 8192), (2, 16384), (1, 16385), (2, 40000)]


@pytest.mark.parametrize("rows,cols", SHAPES)
@pytest.mark.parametrize("aligned", [True, False])
def test_sas_softmax_parity(orc, ta, dev, rows, cols, aligned):
    _log(f"sas_softmax rows={rows} cols={cols} aligned={aligned}")
    x = _scores(rows, cols, rows * 100003 + cols)
    x[0, cols // 2] = 9.0                 # a clear maximum in row 0
    if rows > 2 and cols > 3:
        x[1, ::3] = -float("inf")         # masked entries
        x[2, :] = x[2, 0]                 # a constant row
    ref = orc.sas_softmax_rows(x.numpy())
    if aligned:
        xd = x.to(dev)
    else:  # 4-byte offset: rows that start inside a 16-byte unit
        buf = torch.empty(rows * cols + 1, dtype=torch.float32, device=dev)
        xd = buf[1:].view(rows, cols)
        xd.copy_(x)
    y = ta.turbo_sas_softmax(xd)
    torch.cuda.synchronize()
    _check(y, ref, f"rows={rows} cols={cols}")


@pytest.mark.parametrize("cols", [1, 2, 3, 5, 253, 254, 257, 509, 1021, 1022, 2045, 2047, 4093, 4095,
                                  8189, 16381, 16383, 17405, 17407])
@pytest.mark.parametrize("xo,yo", [(0, 0), (1, 1), (3, 3), (0, 2), (2, 1)])
def test_sas_softmax_rows_that_start_anywhere(orc, ta, dev, cols, xo, yo):
    """Ragged rows (each starts 0 to 3 values into a 16-byte unit), with input
    and output lying alike or not, at the edges of the register sizes; nothing
    around the output is written."""
    rows = 6
    _log(f"sas_softmax rows={rows} cols={cols} x offset={xo} y offset={yo}")
    x = _scores(rows, cols, cols * 8 + xo)
    xb = torch.full((rows * cols + 8,), float("nan"), device=dev)
    yb = torch.full((rows * cols + 8,), -7.0, device=dev)
    xd, yd = (b[o:o + rows * cols].view(rows, cols) for b, o in ((xb, xo), (yb, yo)))
    xd.copy_(x)
    ta.turbo_sas_softmax(xd, out=yd)
    torch.cuda.synchronize()
    _check(yd, orc.sas_softmax_rows(x.numpy()), f"cols={cols}")
    assert bool((yb[:yo] == -7.0).all()) and bool((yb[yo + rows * cols:] == -7.0).all())


# below and past the width that takes vector accesses; one and several chunks a lane;
# one work-group per row, in registers and in passes over memory
@pytest.mark.parametrize("cols", [1, 3, 97, 135, 137, 138, 139, 1001, 2047, 3001, 8190, 16383, 16386])
def test_sas_softmax_bits_do_not_depend_on_where_a_row_lies(ta, dev, cols):
    """Equal rows give equal bits in every row of a matrix and wherever it starts."""
    rows = 9
    _log(f"sas_softmax equal rows cols={cols}")
    row = _scores(1, cols, cols)
    want = None
    for off in range(4):
        buf = torch.empty(rows * cols + 4, dtype=torch.float32, device=dev)
        x = buf[off:off + rows * cols].view(rows, cols)
        x.copy_(row.expand(rows, cols))
        y = ta.turbo_sas_softmax(x).view(torch.int32)
        want = y[:1].clone() if want is None else want
        assert torch.equal(y, want.expand(rows, cols)), off


def test_sas_softmax_in_place_and_single_survivor(orc, ta, dev):
    """In place (y aliases x); a row whose other entries all lie more than 6
    below its maximum is exactly one-hot."""
    x = _scores(64, 3000, 17)
    x[5] = -100.0
    x[5, 1234] = 3.0
    ref = orc.sas_softmax_rows(x.numpy())
    xd = x.to(dev)
    y = ta.turbo_sas_softmax(xd, out=xd)
    torch.cuda.synchronize()
    assert y.data_ptr() == xd.data_ptr()
    _check(xd, ref, "in place")
    row = xd[5].cpu()
    assert row[1234].item() == 1.0 and int((row != 0).sum()) == 1


def test_sas_softmax_full_size_sampled(orc, ta, dev):
    """The 40 x 4096 score rows of the benchmark workload, computed in full on
    the GPU; 512 rows compared with the oracle."""
    from paper_2412_08585_amd import workloads as W
    w = W.WORKLOADS["phi3m-sas-softmax-4k"]
    x = W.softmax_scores(w, device=dev)
    y = ta.turbo_sas_softmax(x)
    torch.cuda.synchronize()
    rows = np.random.default_rng(0).choice(x.shape[0], 512, replace=False)
    idx = torch.from_numpy(rows).to(dev)
    ref = orc.sas_softmax_rows(x[idx].cpu().numpy())
    _check(y[idx], ref, "full size")
    del x, y
    torch.cuda.empty_cache()

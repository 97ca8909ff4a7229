"""GPU parity of the log outputs on the kernels that they share with the
probabilities: grouped rows (whole strips up to 256 columns), packed tiles of
65 to 256 columns and the 32-bit rows that replace them for few rows, and rows
with a start phase once the rows fill the device.  Also the probabilities on
that 32-bit route.  Row counts sit on both sides of each change (taken from
the device's compute units); bars are the header's.
"""
import math

import numpy as np
import pytest
import torch

import oracle
import paper_1904_12380_amd as sm
import workloads

pytestmark = pytest.mark.gpu
NEG_INF = float("-inf")


def _cus():
    return torch.cuda.get_device_properties(0).multi_processor_count


def _check(rows, cols, lo, off):
    x = workloads.random_logits(rows, cols, seed=rows + cols, kind="clip_heavy", scale=30.0)
    x[0, cols - 1] = -np.inf
    x[rows // 2, 0] = np.nan
    n = rows * cols
    buf = torch.full((n + 8,), float("nan"), device="cuda:0")
    buf[off:off + n] = torch.from_numpy(x.reshape(-1)).to("cuda:0")
    xt = buf[off:off + n].view(rows, cols)
    out = torch.full((n + 8,), 777.0, device="cuda:0")
    yt = out[off:off + n].view(rows, cols)
    sm.softmax_log_fwd(xt, lo, out=yt)
    torch.cuda.synchronize()
    got = yt.cpu().numpy().astype(np.float64)
    want = oracle.log_softmax_clipped(x, lo)
    assert np.array_equal(np.isnan(got), np.isnan(want))
    assert np.array_equal(np.isneginf(got), np.isneginf(want))
    fin = np.isfinite(want)
    bound = 2e-6 + 2.5e-7 * (np.abs(want[fin]) + math.log(cols))
    assert np.all(np.abs(got[fin] - want[fin]) <= bound), (rows, cols, lo, off)
    edge = torch.cat([out[:off], out[off + n:]]).cpu().numpy()
    assert np.all(edge == np.float32(777.0)), "written outside the output"
    sm.softmax_fwd_clip(xt, lo, out=yt)
    torch.cuda.synchronize()
    got = yt.cpu().numpy().astype(np.float64)
    want = oracle.softmax_clipped(x, lo)
    fin = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), fin)
    assert np.all(np.abs(got[fin] - want[fin]) <= 4e-6 * want[fin] + 2.0 ** -148)


@pytest.mark.parametrize("cols", [4, 8, 60, 64, 68, 128, 132, 192, 252, 256, 65, 66, 127, 129,
                                  190, 192, 193, 223, 225, 255])
def test_short(cols):
    print(f"[log-rows] {cols}", flush=True)
    cus = _cus()
    for rows in (5, 4 * cus, 4 * cus + 1, 32 * cus + 3):
        if rows * cols > 1 << 21:
            rows = 4 * cus + 1
        _check(rows, cols, NEG_INF if rows % 2 else -64.0, 4)
    _check(37, cols, -64.0, 1)


@pytest.mark.parametrize("cols", [2049, 2051, 4093, 4094, 8189, 8190, 12001, 16377])
def test_phase_rows(cols):
    print(f"[log-rows] phase {cols}", flush=True)
    cus = _cus()
    for rows in (3, 3 * cus - 1, 3 * cus):
        if rows * cols <= 1 << 23:
            _check(rows, cols, -64.0, 4)


@pytest.mark.parametrize("rows,cols", [(3, 16380), (3, 30003), (2, 65533), (9, 100003),
                                       (60, 300000), (2, 1048579), (40, 20000), (90, 17000)])
def test_split(rows, cols):
    print(f"[log-rows] split {rows}x{cols}", flush=True)
    _check(rows, cols, NEG_INF, 4)


# Rows per CU where log rows change from a wavefront each to packed tiles: by
# columns per lane (65 and 130: 9; 98 and 127: 13 and 16) and alignment.
@pytest.mark.parametrize("cols,per_cu,off", [(65, 12, 4), (130, 12, 4), (127, 32, 4), (224, 32, 4),
                                             (79, 32, 1), (98, 40, 3), (190, 40, 1)])
def test_packed_lines(cols, per_cu, off):
    for rows in (per_cu * _cus(), per_cu * _cus() + 1):
        print(f"[log-rows] {rows}x{cols}+{off}", flush=True)
        _check(rows, cols, NEG_INF, off)

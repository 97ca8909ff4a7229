"""GPU parity of the 256-thread row kernel at the edges of its ranges: each
count of strips per lane full, with one column more and with a start phase,
row counts on both sides of the changes to the other kernels (taken from the
device's compute units), every output, in place and between canaries.  Bars
are the header's, against the float64 oracle.
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


def _check(rows, cols):
    x = workloads.random_logits(rows, cols, seed=rows * 7 + cols, kind="clip_heavy", scale=30.0)
    x[0, cols - 1] = -np.inf
    x[rows - 1, cols // 2] = np.nan
    if rows > 2:
        x[1, :] = -np.inf
    n = rows * cols
    buf = torch.full((n + 8,), 9.0, device="cuda:0")
    yt = buf[4:4 + n].view(rows, cols)
    xt = torch.from_numpy(x).to("cuda:0")
    d = np.minimum(np.abs(x.astype(np.float64) - x.max(1, keepdims=True)), 64.0)
    for name, lo in (("fwd", -64.0), ("clip", NEG_INF), ("approx", -64.0), ("log", NEG_INF),
                     ("inplace", -64.0)):
        want = oracle.log_softmax_clipped(x, lo) if name == "log" else oracle.softmax_clipped(x, lo)
        if name == "approx":
            sm.softmax_fwd_approx(xt, lo, out=yt)
        elif name == "log":
            sm.softmax_log_fwd(xt, lo, out=yt)
        elif name == "inplace":
            yt.copy_(xt)
            sm.softmax_fwd(yt, out=yt)
        else:
            sm.softmax_fwd_clip(xt, lo, out=yt)
        torch.cuda.synchronize()
        got = yt.cpu().numpy().astype(np.float64)
        assert np.array_equal(np.isnan(got), np.isnan(want)), name
        assert np.array_equal(np.isneginf(got), np.isneginf(want)), name
        fin = np.isfinite(want)
        w = want[fin]
        tol = (2e-6 + 2.5e-7 * (np.abs(w) + math.log(cols)) if name == "log" else
               (2e-6 + 1.5e-7 * d[fin]) * w if name == "approx" else 4e-6 * w + 2.0 ** -148)
        assert np.all(np.abs(got[fin] - w) <= tol), (name, rows, cols)
        edge = torch.cat([buf[:4], buf[4 + n:]]).cpu().numpy()
        assert np.all(edge == np.float32(9.0)), (name, "written outside the output")


@pytest.mark.parametrize("cols", [1087, 1088, 2045, 2046, 2048, 2049, 3069, 3070, 3072, 3073,
                                  4093, 4094, 4096, 4097, 5117, 5118, 5120, 5121, 6142, 8189,
                                  8192, 8193, 10237, 10240, 10241])
def test_strips(cols):
    print(f"[row-blocks] {cols}", flush=True)
    _check(5, cols)
    _check(2, cols)


@pytest.mark.parametrize("cols,num,den", [(1500, 8, 1), (2051, 11, 1), (2060, 6, 1),
                                          (4000, 5, 1), (2049, 13, 1), (16384, 1, 1),
                                          (20480, 1, 1), (20481, 1, 3), (24573, 1, 3),
                                          (24572, 1, 1), (16385, 1, 3)])
def test_row_counts(cols, num, den):
    rows = _cus() * num // den
    for r in (rows, rows + 1):
        print(f"[row-blocks] {r}x{cols}", flush=True)
        _check(r, cols)


@pytest.mark.parametrize("rows,cols", [(300, 1501), (300, 1500), (300, 3001), (700, 5000),
                                       (9, 10237), (600, 18001), (400, 17000), (300, 24573),
                                       (9, 12001), (300, 1087), (5000, 130)])
def test_a_plan_runs_as_planned(rows, cols):
    """softmax_fwd_planned takes what softmax_plan reports and runs the same
    kernel: the same bits."""
    print(f"[row-blocks] plan {rows}x{cols}", flush=True)
    x = torch.randn(rows, cols, device="cuda:0")
    y = torch.empty_like(x)
    plan = sm.softmax_plan(rows, cols, x.data_ptr(), y.data_ptr())
    sm.softmax_fwd_planned(x, plan, out=y)
    assert torch.equal(y, sm.softmax_fwd(x))


@pytest.mark.parametrize("cols,threads", [(5117, 256), (10236, 256), (10237, 256), (10238, 1024),
                                          (10239, 1024), (10240, 256), (10241, 1024)])
def test_ten_strips_at_most(cols, threads):
    """256 threads take rows of up to ten strips per lane, the columns that a
    row's start phase adds among them; the next instance has twenty."""
    print(f"[row-blocks] {cols}", flush=True)
    for rows in (1, 5, 3000):
        p = sm.softmax_plan(rows, cols)
        assert (p["kernel_name"], p["block_threads"]) == ("block_row", threads), p
        assert p["elems_per_lane"] * threads < 2 * cols
    _check(5, cols)


# columns, rows per CU (num / den, +1 row), kernel, threads: both sides of the
# lines between the 256-thread kernel and the others.
LINES = [(1100, 8, 1, 0, "block_row", 256), (1100, 8, 1, 1, "wave_row", 256),
         (1120, 30, 1, 0, "wave_row", 256), (1124, 30, 1, 0, "block_row", 256),
         (1117, 40, 1, 0, "block_row", 256), (1117, 40, 1, 1, "wave_row", 256),
         (1121, 40, 1, 1, "block_row", 256), (1201, 11, 1, 1, "wave_row", 256),
         (3073, 8, 1, 0, "block_row", 256), (3073, 8, 1, 1, "wave_row", 256),
         (3585, 6, 1, 1, "wave_row", 256), (3585, 13, 1, 1, "block_row", 256),
         (6141, 1, 1, 0, "block_row", 256), (6142, 2, 1, 0, "block_row", 1024),
         (6142, 2, 1, 1, "block_row", 256), (8189, 2, 1, 0, "block_row", 1024),
         (8190, 2, 1, 0, "block_row", 256), (6144, 1, 1, 0, "block_row", 256),
         (16384, 2, 1, 0, "block_row", 256), (16384, 2, 1, 1, "split_row", 256),
         (16384, 4, 1, 0, "split_row", 256), (16388, 4, 1, 0, "block_row", 256),
         (20480, 5, 2, 0, "split_row", 256), (20480, 6, 1, 1, "split_row", 256),
         (24572, 2, 1, 0, "block_row", 256), (24572, 4, 1, 0, "split_row", 256),
         (24576, 2, 1, 0, "split_row", 256), (20477, 1, 2, -1, "block_row", 256),
         (20478, 1, 2, -1, "split_row", 256), (20478, 1, 2, 0, "block_row", 256),
         (24573, 7, 8, 0, "block_row", 256), (24573, 7, 8, 1, "split_row", 256),
         (24573, 4, 1, 0, "split_row", 256), (24573, 4, 1, 1, "block_row", 256),
         (24573, 8, 1, 0, "split_row", 256), (24573, 8, 1, 1, "block_row", 256)]


@pytest.mark.parametrize("cols,num,den,more,kernel,threads", LINES)
def test_lines(cols, num, den, more, kernel, threads):
    rows = _cus() * num // den + more
    p = sm.softmax_plan(rows, cols)
    print(f"[row-blocks] {rows}x{cols} {p['kernel_name']} {p['block_threads']}", flush=True)
    assert (p["kernel_name"], p["block_threads"]) == (kernel, threads), p


@pytest.mark.parametrize("cols", [2047, 16388, 20477, 20478, 24573])
def test_rows_over_the_split_kernel(cols):
    """Row counts past two and three per CU, where log rows and probability rows
    go different ways."""
    for rows in (2 * _cus(), 3 * _cus() + 1):
        print(f"[row-blocks] {rows}x{cols}", flush=True)
        _check(rows, cols)


def test_a_plan_of_24_strips_still_runs():
    """A caller's plan may ask for 256 threads on rows of 21 to 24 strips whose
    number the library itself gives to the split kernel."""
    for cols in (20484, 24000, 24570):
        print(f"[row-blocks] planned {cols}", flush=True)
        x = torch.randn(40, cols, device="cuda:0")
        y = sm.softmax_fwd_planned(x, dict(kernel_name="block_row", vec_width=4,
                                           block_threads=256))
        want = oracle.softmax_clipped(x.cpu().numpy())
        assert np.all(np.abs(y.cpu().numpy() - want) <= 4e-6 * want)

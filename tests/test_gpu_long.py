"""GPU parity of the two streaming passes over rows too long for one pass:
one row and several, rows of one to 16 exchange entries, more rows than one
group of launches takes, ragged ends, x and y at the same and at different
phases, in place, every output, and non-finite rows.  Bars are the header's,
against the float64 oracle.
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
TWO_PASS = dict(kernel_name="split_row", vec_width=1, block_threads=512, elems_per_lane=32)


def _at(n, off, fill):
    buf = torch.full((n + 8,), fill, device="cuda:0")
    return buf, buf[off:off + n]


def _rest(buf, off, n, fill):
    edge = torch.cat([buf[:off], buf[off + n:]]).cpu().numpy()
    assert np.all(edge == np.float32(fill)), "written outside the output"


@pytest.mark.parametrize("rows,cols,xo,yo", [(1, 2097153, 4, 4), (1, 2097160, 4, 4),
                                             (3, 2097155, 1, 1), (2, 2500003, 1, 4),
                                             (2, 2100000, 3, 1), (5, 2097156, 0, 2),
                                             (1, 4194304, 0, 0), (1, 8388611, 1, 1),
                                             (1, 8388611, 4, 3)])
def test_rows(rows, cols, xo, yo):
    print(f"[long] {rows}x{cols}+{xo}+{yo}", flush=True)
    x = workloads.random_logits(rows, cols, seed=cols + rows, kind="clip_heavy")
    n = rows * cols
    xb, xf = _at(n, xo, float("nan"))
    xf.copy_(torch.from_numpy(x.reshape(-1)))
    xt = xf.view(rows, cols)
    for lo in (-64.0, NEG_INF):
        want = oracle.softmax_clipped(x, lo)
        yb, yf = _at(n, yo, 5.0)
        yt = yf.view(rows, cols)
        sm.softmax_fwd_clip(xt, lo, out=yt)
        torch.cuda.synchronize()
        got = yt.cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - want) <= 4e-6 * want + 2.0 ** -148), lo
        _rest(yb, yo, n, 5.0)
    lw = oracle.log_softmax_clipped(x, -64.0)
    sm.softmax_log_fwd(xt, out=yt)
    torch.cuda.synchronize()
    err = np.abs(yt.cpu().numpy() - lw)
    assert np.all(err <= 2e-6 + 2.5e-7 * (np.abs(lw) + math.log(cols)))
    want = oracle.softmax_clipped(x, -64.0)
    sm.softmax_fwd_approx(xt, out=yt)
    torch.cuda.synchronize()
    d = np.minimum(np.abs(x.astype(np.float64) - x.max(1, keepdims=True)), 64.0)
    assert np.all(np.abs(yt.cpu().numpy() - want) <= (2e-6 + 1.5e-7 * d) * want)
    _rest(yb, yo, n, 5.0)
    sm.softmax_fwd(xt, out=xt)  # in place
    torch.cuda.synchronize()
    assert np.all(np.abs(xt.cpu().numpy() - want) <= 4e-6 * want)
    assert sm.softmax_exchange_status() == {"join_give_ups": 0, "wait_give_ups": 0,
                                            "entries_in_use": 0}


def test_more_rows_than_a_group():
    """70 rows of 1048577 columns: a group of launches holds 256 MiB of x, 63
    rows, so a second one follows, of other workgroup and entry counts."""
    rows, cols = 70, (1 << 20) + 1
    print(f"[long] {rows}x{cols}", flush=True)
    p = sm.softmax_plan(rows, cols)
    assert p["kernel_name"] == "split_row" and p["launches"] == 4, p
    x = workloads.random_logits(rows, cols, seed=70, kind="offset")
    xt = torch.from_numpy(x).to("cuda:0")
    y, lg = sm.softmax_fwd(xt), sm.softmax_log_fwd(xt)
    again = sm.softmax_fwd(xt)
    torch.cuda.synchronize()
    assert torch.equal(y, again)
    for a in range(0, rows, 7):
        want = oracle.softmax_clipped(x[a:a + 7])
        got = y[a:a + 7].cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - want) <= 4e-6 * want), a
        lw = oracle.log_softmax_clipped(x[a:a + 7], -64.0)
        err = np.abs(lg[a:a + 7].cpu().numpy() - lw)
        assert np.all(err <= 2e-6 + 2.5e-7 * (np.abs(lw) + math.log(cols))), a
    assert sm.softmax_exchange_status() == {"join_give_ups": 0, "wait_give_ups": 0,
                                            "entries_in_use": 0}


def test_nonfinite_rows():
    print("[long] nonfinite", flush=True)
    cols = 2097155
    x = np.random.default_rng(3).standard_normal((5, cols)).astype(np.float32)
    x[0, cols - 1] = np.nan
    x[1, 7] = np.inf
    x[2, :] = -np.inf
    x[3, : cols - 5] = -np.inf
    xt = torch.from_numpy(x).to("cuda:0")
    for lo in (-64.0, NEG_INF):
        want = oracle.softmax_clipped(x, lo)
        got = sm.softmax_fwd_clip(xt, lo).cpu().numpy().astype(np.float64)
        assert np.array_equal(np.isnan(got), np.isnan(want))
        fin = np.isfinite(want)
        assert np.all(np.abs(got[fin] - want[fin]) <= 4e-6 * want[fin] + 2.0 ** -148)


def test_planned_and_replayed():
    """The caller's two-pass plan, and replays of a captured call beside eager
    ones: the same bits every time, and the entries back at rest."""
    print("[long] planned, graph", flush=True)
    x = torch.from_numpy(workloads.random_logits(2, 1048580, seed=9, kind="offset")).to("cuda:0")
    want = oracle.softmax_clipped(x.cpu().numpy())
    y = sm.softmax_fwd_planned(x, TWO_PASS)
    torch.cuda.synchronize()
    assert np.all(np.abs(y.cpu().numpy() - want) <= 4e-6 * want)
    x = torch.from_numpy(workloads.random_logits(3, 2200000, seed=9, kind="offset")).to("cuda:0")
    ref = sm.softmax_fwd(x)
    s, g = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    out = torch.empty_like(x)
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.graph(g, stream=s):
        sm.softmax_fwd(x, out=out, stream=s)
    for rep in range(3):
        out.zero_()
        again = sm.softmax_fwd(x)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, ref) and torch.equal(again, ref), rep
    assert sm.softmax_exchange_status()["entries_in_use"] == 0

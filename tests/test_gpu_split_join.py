"""One-pass split rows in calls that hold more rows than are resident at once,
with a short or a long rest (whole strips, ragged rows and rows with 32-bit
access), the row counts taken from softmax_plan.  Every row against the float64
oracle at the header's bar, repeated bit for bit, with the exchange back at
rest; every launch's workgroups resident together; and two such calls at a time
on two streams.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_1904_12380_amd as sm
import workloads

pytestmark = pytest.mark.gpu


def _resident_rows(cols, x_ptr):
    p = sm.softmax_plan(1, cols, x_ptr)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    return 2048 // p["block_threads"] * cus // p["chunks_per_row"]


# cols, offset of x in floats, share of a launch over
@pytest.mark.parametrize("cols,off,over", [(40000, 0, 0.02), (40000, 0, 0.19), (40000, 0, 0.3),
                                           (50001, 0, 0.34), (50001, 0, 0.4), (65536, 0, 1.1),
                                           (49999, 1, 0.3)])
def test_rest(cols, off, over):
    rows = int(_resident_rows(cols, (1 << 44) + 4 * off) * (1.0 + over)) + 1
    print(f"[split-join] {rows}x{cols}+{off}", flush=True)
    x = workloads.random_logits(rows, cols, seed=rows + cols, kind="offset")
    n = rows * cols
    buf = torch.empty(n + 4, device="cuda:0")
    xt = buf[off:off + n].view(rows, cols)
    xt.copy_(torch.from_numpy(x))
    y = sm.softmax_fwd(xt)
    again = sm.softmax_fwd(xt)
    lg = sm.softmax_log_fwd(xt)
    torch.cuda.synchronize()
    assert torch.equal(y, again)
    for a in range(0, rows, 64):
        want = oracle.softmax_clipped(x[a:a + 64])
        got = y[a:a + 64].cpu().numpy().astype(np.float64)
        assert np.all(np.abs(got - want) <= 4e-6 * want), a
        lw = oracle.log_softmax_clipped(x[a:a + 64], -64.0)
        err = np.abs(lg[a:a + 64].cpu().numpy() - lw)
        assert np.all(err <= 2e-6 + 2.5e-7 * (np.abs(lw) + np.log(cols))), a
    assert sm.softmax_exchange_status() == {"join_give_ups": 0, "wait_give_ups": 0,
                                            "entries_in_use": 0}


@pytest.mark.parametrize("cols,off", [(40000, 0), (50001, 0), (65536, 0), (131071, 0),
                                      (28001, 0), (17361, 1), (400001, 2), (300000, 0)])
def test_no_launch_exceeds_what_is_resident(cols, off):
    """The workgroups of a split row wait for each other while they hold their
    places, so a launch holds no more of them than run at once (2048 threads per
    CU), also where a rest of a few rows is left."""
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    ptr = (1 << 44) + 4 * off
    full = _resident_rows(cols, ptr)
    for rows in (1, full, full + 1, full * 11 // 10, full * 4 // 3, 2 * full + 1, 1024, 5000):
        p = sm.softmax_plan(rows, cols, ptr, ptr + (1 << 43))
        print(f"[split-join] plan {rows}x{cols}+{off}: {p['kernel_name']} {p['grid']}",
              flush=True)
        if p["kernel_name"] == "split_row":
            assert p["grid"] * p["block_threads"] <= 2048 * cus, (rows, p)


def test_two_streams_with_rests():
    """Calls of several launches each, queued on two streams: every output
    bitwise that of the same call alone, and no wait gave up."""
    calls = [("log", 300, 131071, 0), ("softmax", 335, 50001, 0), ("softmax", 600, 17361, 1),
             ("log", 83, 400001, 0), ("softmax", 471, 40000, 0)]
    cases = []
    for op, rows, cols, off in calls:
        n = rows * cols
        buf = torch.randn(n + 4, device="cuda:0")
        x = buf[off:off + n].view(rows, cols)
        fn = sm.softmax_log_fwd if op == "log" else sm.softmax_fwd
        cases.append((fn, x, fn(x), torch.empty_like(buf)[off:off + n].view(rows, cols)))
    torch.cuda.synchronize()
    at_rest = {"join_give_ups": 0, "wait_give_ups": 0, "entries_in_use": 0}
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    for i in range(len(cases)):
        pair = (cases[i], cases[(i + 1) % len(cases)])
        print(f"[split-join] streams {calls[i]} {calls[(i + 1) % len(cases)]}", flush=True)
        for _, _, _, y in pair:
            y.zero_()
        torch.cuda.synchronize()
        for _ in range(3):
            for (fn, x, _, y), s in zip(pair, streams):
                fn(x, out=y, stream=s)
        torch.cuda.synchronize()
        for fn, x, ref, y in pair:
            assert torch.equal(y, ref), calls[i]
        assert sm.softmax_exchange_status() == at_rest

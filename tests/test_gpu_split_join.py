"""GPU parity of one-pass split launches that hold more rows than are resident
at once: a short rest joined to a full launch (whole strips and ragged rows)
and 32-bit rows in one launch, the row counts taken from softmax_plan.  Every
row against the float64 oracle at the header's bar, repeated bit for bit, with
the exchange back at rest.
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

"""Row sums of the streaming kernels (losses, rows in two passes) on structured
logits, where every step of a lane's running sum would round the same way:
values that repeat with the step, rows that rise steadily, and one maximum far
above a mass of equal logits.  Random logits hide these errors; the reference
is binary64.
"""
import math

import pytest
import torch

import paper_1904_12380_amd as sm

pytestmark = pytest.mark.gpu
NEG_INF = float("-inf")


def _loss_bound(loss, cols):
    return 2e-6 + 2.5e-7 * (loss.abs() + math.log(cols))


def _check_losses(x, labels):
    """Every loss within the header's bound of binary64."""
    rows, cols = x.shape
    got = sm.softmax_nll_fwd(x, labels, NEG_INF).double()
    want = torch.empty_like(got)
    for a in range(0, rows, 8):
        c = x[a:a + 8].double()
        c -= c.amax(1, keepdim=True)
        picked = c.gather(1, labels[a:a + 8, None])[:, 0]
        want[a:a + 8] = c.exp_().sum(1).log() - picked
    err = (got - want).abs()
    worst = int((err / _loss_bound(want, cols)).argmax())
    print(f"[sums] worst row {worst}: {err[worst].item():.3e} of "
          f"{_loss_bound(want, cols)[worst].item():.3e}", flush=True)
    assert bool((err <= _loss_bound(want, cols)).all()), (worst, err[worst].item())


# Rows for 256 threads each (enough of them to fill the device with fewer
# threads than a workgroup may have): 4096 columns per step.
@pytest.mark.parametrize("kind", ["alternating", "rising"])
def test_losses_of_long_structured_rows(kind):
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    rows, cols = 3 * cus // 2, 1 << 22
    print(f"[sums] loss {kind} {rows}x{cols}", flush=True)
    x = torch.empty(rows, cols, device="cuda:0")
    par = torch.linspace(0.0, 1.0, rows, device="cuda:0")
    if kind == "alternating":  # (0, v): S = cols / 2 (1 + e^v)
        x.view(rows, cols // 2, 2)[:, :, 0] = 0.0
        x.view(rows, cols // 2, 2)[:, :, 1] = (-12.0 * par)[:, None]
    else:  # 1e-4 to 3e-2 more with every 4096 columns
        slope = 1e-4 + 2.99e-2 * par
        step = torch.arange(cols // 4096, device="cuda:0")
        x.view(rows, cols // 4096, 4096).copy_((slope[:, None] * step)[:, :, None].expand(
            rows, cols // 4096, 4096))
    _check_losses(x, torch.full((rows,), 5, dtype=torch.int64, device="cuda:0"))


def test_two_pass_probabilities_of_a_repeating_row():
    """2^31 columns of alternating (0, v): 256 steps per workgroup.  Tolerance:
    half of the row's terms within 1.5 ulp (0.9e-7), 4 roundings of a step's tree
    sum, one of the lane's sum and of its pair (equal values double exactly over
    lanes, and the pairs merge in binary64), 1 / S, the exponential of the output
    (1.8e-7) and the product: 8e-7."""
    cols = 1 << 31
    x = torch.empty(1, cols, device="cuda:0")
    y = torch.empty_like(x)
    for v in (-3.8361797, -9.69764, -0.7, -1.9, -5.3):
        print(f"[sums] softmax 1x{cols} {v}", flush=True)
        x.view(cols // 2, 2)[:, 0] = 0.0
        x.view(cols // 2, 2)[:, 1] = v
        sm.softmax_fwd(x, out=y)
        v32 = float(x[0, 1].double())
        s = cols // 2 * (1.0 + math.exp(v32))
        for c, want in ((0, 1.0 / s), (cols - 1, math.exp(v32) / s), (cols // 2, 1.0 / s)):
            err = abs(float(y[0, c].double()) / want - 1.0)
            print(f"[sums]   column {c}: {err:.3e}", flush=True)
            assert err <= 8e-7, (v, c, err)


# M - x is not an fp32 number: rounded to fp32 it is off by almost half an ulp
# of 16 (9.5e-7), which would scale the whole mass below the maximum.
@pytest.mark.parametrize("top,low", [(16.0625, 9.3e-7), (16.25, -9.3e-7), (16.125, 9.4e-7),
                                     (16.1875, -9.4e-7)])
def test_partial_sums_are_rescaled_exactly(top, low):
    """2^27 columns at `low` and one at `top`: S is 12 to 15.  Sums of equal
    terms are exact, so what is left is one rescaling of the mass within 1.5 ulp
    (1.8e-7); the roundings on the maximum's way through the sums, up to 22 of
    6e-8 absolute while its partial sum is below 2 (9e-8 of S) and then halves
    of an ulp of partials that double (1.2e-7 of S); and two roundings of the
    output (a loss: 1 ulp of log2 S and the product, 2.9e-7)."""
    cols = 1 << 27
    print(f"[sums] rescale {top} {low}", flush=True)
    x = torch.full((1, cols), low, device="cuda:0")
    at = 12345677
    x[0, at] = top
    low32 = float(x[0, 0].double())
    s = 1.0 + (cols - 1) * math.exp(low32 - top)
    y = sm.softmax_fwd(x)
    err = abs(float(y[0, at].double()) * s - 1.0)
    label = torch.full((1,), at, dtype=torch.int64, device="cuda:0")
    loss = sm.softmax_nll_fwd(x, label, NEG_INF)
    loss_err = abs(float(loss[0].double()) - math.log(s))
    print(f"[sums]   {err:.3e} {loss_err:.3e}", flush=True)
    assert err <= 5.1e-7 and loss_err <= 6.8e-7, (err, loss_err)

"""Row sums of the streaming kernels (losses, rows in two passes) on structured
logits, whose rounding errors random logits hide: one maximum far above a mass
of equal logits.  The reference is binary64.
"""
import math

import pytest
import torch

import paper_1904_12380_amd as sm

pytestmark = pytest.mark.gpu
NEG_INF = float("-inf")


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

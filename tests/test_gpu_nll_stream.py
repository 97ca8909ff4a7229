"""GPU parity of the streamed loss kernels (rows of more than 64 columns) at
the edges of their ranges: the last lane strip full or holding one column,
each start phase of a row against 16 bytes, a step of the stream exactly
full or one column over, one row and several, chunks of a split row, labels
in the columns outside the aligned strips.  Bar as in test_gpu_nll.py (the
header's bound), against the float64 oracle.
"""
import numpy as np
import pytest
import torch

import paper_1904_12380_amd as sm
import workloads
from tests.test_gpu_nll import check_nll

pytestmark = pytest.mark.gpu
NEG_INF = float("-inf")

# Row lengths around every change of kernel: lanes per row and strips per
# lane (65 ... 2048), one wavefront per row with 1024 columns per step, 256,
# 512 and 1024 threads per row; with few rows, split rows.
SHAPES = [(37, c) for c in (65, 93, 94, 96, 97, 125, 126, 128, 129, 221, 222, 224, 225, 381,
                            382, 384, 385, 797, 798, 800, 801, 1024, 2044, 2045, 2046, 2048)]
SHAPES += [(5, c) for c in (2049, 2052, 3071, 3075, 4099, 8189, 8192, 8197)]
SHAPES += [(1100, 2051), (600, 4097), (1030, 32771), (260, 9001), (129, 32800)]
SHAPES += [(1, 32969), (1, 65536), (3, 40963), (2, 1000003), (1, 2097153), (128, 58372)]


@pytest.mark.parametrize("rows,cols", SHAPES)
def test_edges(rows, cols):
    print(f"[nll-stream] {rows}x{cols}", flush=True)
    rng = np.random.default_rng(rows * 31 + cols)
    x = workloads.random_logits(rows, cols, seed=rows + cols, kind="clip_heavy", scale=30.0)
    t = rng.integers(0, cols, size=rows, dtype=np.int64)
    t[0], t[-1] = cols - 1, 0
    tt = torch.from_numpy(t).to("cuda:0")
    n = rows * cols
    buf = torch.full((n + 8,), float("nan"), device="cuda:0")
    for off in (0, 1, 3):  # NaN on both sides: a column read from outside shows
        buf.fill_(float("nan"))
        buf[off + 1:off + 1 + n] = torch.from_numpy(x.reshape(-1)).to("cuda:0")
        xv = buf[off + 1:off + 1 + n].view(rows, cols)
        loss = sm.softmax_nll_fwd(xv, tt, NEG_INF if off else -64.0)
        torch.cuda.synchronize()
        check_nll(x, t, loss.cpu().numpy(), NEG_INF if off else -64.0, f"{rows}x{cols}+{off}")
    assert sm.softmax_exchange_status()["entries_in_use"] == 0


@pytest.mark.parametrize("cols", [65, 200, 777, 3000, 9000, 50001, 400003])
def test_nonfinite(cols):
    print(f"[nll-stream] nonfinite {cols}", flush=True)
    rng = np.random.default_rng(cols)
    x = rng.standard_normal((9, cols)).astype(np.float32)
    x[0, cols - 1] = np.nan
    x[1, 0] = np.inf
    x[2, :] = -np.inf
    x[3, : cols // 2] = -np.inf
    x[4, 1:] = -np.inf
    x[5, 0] = np.finfo(np.float32).min
    t = np.array([0, 0, 0, 1, 0, cols - 1, -1, cols, cols // 2], dtype=np.int64)
    xt, tt = torch.from_numpy(x).to("cuda:0"), torch.from_numpy(t).to("cuda:0")
    for lo in (-64.0, NEG_INF):
        loss = sm.softmax_nll_fwd(xt, tt, lo)
        torch.cuda.synchronize()
        check_nll(x, t, loss.cpu().numpy(), lo, f"nonfinite {cols}")

"""GPU parity of the one-wavefront attention kernel at the edges of its
tiles: every count of query and key tiles, key tiles with one key and full
ones, d and dv around multiples of 4, 16, 32 and 64 (one block, a pair, the
last block or column tile holding one column), d below 4, several column
blocks, more items than resident wavefronts, operands 4 bytes past a 16-byte
boundary inside NaN, an output between canaries, and clip bounds below -87.
Bar as in test_gpu_attention.py, against the float64 oracle.
"""
import numpy as np
import pytest
import torch

import paper_1904_12380_amd as sm
import workloads
from tests.test_gpu_attention import bound

pytestmark = pytest.mark.gpu
NEG_INF = float("-inf")
CANARY = 12345.0

SHAPES = [
    # query and key tiles
    (3, 1, 1, 8, 8), (3, 16, 16, 16, 16), (3, 17, 17, 16, 64), (3, 32, 33, 32, 64),
    (2, 33, 48, 64, 128), (2, 48, 49, 64, 200), (2, 64, 64, 48, 132), (2, 65, 47, 36, 192),
    (2, 130, 31, 20, 260), (1100, 33, 40, 12, 20), (600, 18, 64, 32, 32),
    # d: below 4, one past a block, a pair, two pairs
    (5, 9, 20, 1, 3), (5, 9, 20, 2, 2), (5, 9, 20, 3, 1), (5, 9, 20, 5, 5), (4, 20, 40, 15, 15),
    (4, 20, 40, 17, 17), (4, 20, 40, 31, 33), (4, 20, 40, 33, 31), (4, 20, 40, 63, 65),
    (4, 20, 40, 65, 63), (4, 20, 40, 97, 49), (3, 20, 40, 130, 47), (3, 40, 60, 202, 113),
    (2, 5, 5, 0, 9),
    # dv: every width of the last column block, several full ones, three key tiles
    (3, 7, 45, 32, 200), (3, 7, 45, 32, 150), (3, 7, 45, 32, 170), (3, 7, 45, 32, 187),
    (3, 50, 35, 32, 257), (3, 50, 20, 32, 321), (3, 7, 64, 32, 1),
    # more items than resident wavefronts; one item per CU
    (9000, 4, 12, 9, 10), (256, 16, 50, 40, 40), (257, 16, 50, 40, 40), (5000, 20, 37, 32, 64),
    # the DAM tile with one query tile and many batch elements
    (1024, 3, 50, 200, 200),
]


def _place(a, off):
    """a on the GPU, `off` floats into a NaN-filled buffer."""
    n = a.size
    buf = torch.full((n + 8,), float("nan"), device="cuda:0")
    buf[off:off + n] = torch.from_numpy(a.reshape(-1)).to("cuda:0")
    return buf[off:off + n].view(a.shape)


@pytest.mark.parametrize("b,lq,lk,d,dv", SHAPES)
def test_edges(b, lq, lk, d, dv):
    print(f"[attn-wave] {b}x{lq}x{lk}x{d}x{dv}", flush=True)
    q, k, v = workloads.random_qkv(b, lq, lk, d, dv, seed=b + lq * 3 + lk * 5 + d * 7 + dv)
    scale = float(np.float32(1.0 / np.sqrt(max(d, 1))))
    n = b * lq * dv
    for off, lo, s in ((4, -64.0, scale), (1, NEG_INF, 8.0 * scale), (3, -100.0, 8.0 * scale)):
        buf = torch.full((n + 8,), CANARY, device="cuda:0")
        out = buf[off:off + n].view(b, lq, dv)
        sm.softmax_attention_fwd(_place(q, off), _place(k, off), _place(v, off), scale=s,
                                 clip_lo=lo, out=out)
        torch.cuda.synchronize()
        want, tol = bound(q, k, v, s, lo)
        err = np.abs(out.cpu().numpy().astype(np.float64) - want)
        assert np.all(err <= tol), (off, lo, float((err / tol).max()))
        edge = torch.cat([buf[:off], buf[off + n:]]).cpu().numpy()
        assert np.all(edge == np.float32(CANARY)), (off, "written outside the output")


def test_nan_and_inf_stay_in_their_rows():
    """A NaN query row, a query of infinities and a NaN value reach only the
    outputs that depend on them."""
    print("[attn-wave] nonfinite", flush=True)
    q, k, v = workloads.random_qkv(3, 20, 21, 30, 70, seed=5)
    q[0, 3, 29] = np.nan
    v[1, 20, 69] = np.nan
    q[2, 5, :] = np.inf
    want, _ = bound(q, k, v, 0.2, -64.0)
    out = sm.softmax_attention_fwd(_place(q, 1), _place(k, 1), _place(v, 1), scale=0.2)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.array_equal(np.isnan(got), np.isnan(want))
    fin = ~np.isnan(want)
    assert np.all(np.abs(got[fin] - want[fin]) <= 1e-4)


# Outputs of 64 MiB and more in rows that are not whole 32-byte sectors: one,
# two and three query tiles against one to three key tiles, d and dv whole
# 16-byte strips and not, the last column block of every width.
@pytest.mark.parametrize("lq,lk,d,dv", [(10, 5, 8, 100), (20, 16, 9, 94), (40, 15, 8, 188),
                                        (16, 20, 9, 67), (32, 32, 12, 604), (33, 17, 5, 89),
                                        (7, 48, 16, 76), (100, 37, 7, 113), (48, 33, 8, 132)])
def test_large_outputs_of_partial_sectors(lq, lk, d, dv):
    """The whole output bit for bit against the same batch elements in calls of
    smaller outputs, and its ends against the oracle."""
    b = -(-(1 << 24) // (lq * dv)) + 1
    print(f"[attn-wave] large {b}x{lq}x{lk}x{d}x{dv}", flush=True)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(lq + dv)
    q, k, v = (torch.randn(b, n, w, device="cuda:0", generator=g)
               for n, w in ((lq, d), (lk, d), (lk, dv)))
    n = b * lq * dv
    buf = torch.full((n + 8,), CANARY, device="cuda:0")
    out = buf[4:4 + n].view(b, lq, dv)
    sm.softmax_attention_fwd(q, k, v, scale=0.3, out=out)
    step = -(-b // 3)
    for a in range(0, b, step):
        part = sm.softmax_attention_fwd(q[a:a + step], k[a:a + step], v[a:a + step], scale=0.3)
        assert torch.equal(out[a:a + step], part), a
    edge = torch.cat([buf[:4], buf[4 + n:]]).cpu().numpy()
    assert np.all(edge == np.float32(CANARY)), "written outside the output"
    for a in (0, b - 3):
        qa, ka, va = (t[a:a + 3].cpu().numpy() for t in (q, k, v))
        want, tol = bound(qa, ka, va, float(np.float32(0.3)), -64.0)
        assert np.all(np.abs(out[a:a + 3].cpu().numpy().astype(np.float64) - want) <= tol)

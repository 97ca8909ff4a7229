"""Rows in two passes that cannot get one of their exchange entries: a row takes
up to 16 entries, and one of them is held for longer than the row may wait.  The
row is NaN, the other rows are right, and no entry keeps what the row had
claimed: the kernels run on a table of the test's own (tests/native), where the
test holds the entry and the wait limit is short.
"""
import ctypes
import os

import numpy as np
import pytest
import torch

import oracle
import workloads
from paper_1904_12380_amd import build

pytestmark = pytest.mark.gpu


def _probe():
    if not os.path.exists(build.PROBE_LIB):
        build.build()
    lib = ctypes.CDLL(build.PROBE_LIB)
    for name in ("probe_scratch_words", "probe_entry_words", "probe_entries"):
        getattr(lib, name).restype = ctypes.c_int64
    p, i64, u32 = ctypes.c_void_p, ctypes.c_int64, ctypes.c_uint32
    lib.probe_long_rows.argtypes = [p, p, p, ctypes.c_uint64, u32, i64, i64, ctypes.c_int, i64,
                                    u32, p]
    return lib


# workgroups per row, entry of row 1 that is held, first entry (the table wraps)
@pytest.mark.parametrize("wpr,held,base", [(512, 5, 100), (130, 0, 4094), (1024, 15, 4080),
                                           (40, 0, 7)])
def test_a_row_without_one_of_its_entries_leaves_none_claimed(wpr, held, base):
    print(f"[long-entries] {wpr} workgroups, entry {held} held", flush=True)
    lib = _probe()
    rows, chunk = 3, 2048
    cols = wpr * chunk - 3
    entries = -(-wpr // 64)
    words, n_entries = lib.probe_entry_words(), lib.probe_entries()
    table = torch.zeros(lib.probe_scratch_words(), dtype=torch.int64, device="cuda:0")
    per_entry = table[:n_entries * words].view(n_entries, words)
    x = workloads.random_logits(rows, cols, seed=wpr, kind="offset")
    want = oracle.softmax_clipped(x)
    xt = torch.from_numpy(x).to("cuda:0")
    y = torch.empty_like(xt)

    def run(key):
        y.fill_(7.0)
        # 2000 ticks: 20 us of the 100 MHz wall clock
        assert lib.probe_long_rows(xt.data_ptr(), y.data_ptr(), table.data_ptr(), key, base, rows,
                                   cols, wpr, chunk, 2000,
                                   torch.cuda.current_stream().cuda_stream) == 0
        torch.cuda.synchronize()
        return y.cpu().numpy().astype(np.float64)

    at = (base + entries + held) % n_entries
    per_entry[at, 0] = 12345
    got = run(1)
    assert np.all(np.isnan(got[1]))
    for r in (0, 2):
        assert np.all(np.abs(got[r] - want[r]) <= 4e-6 * want[r]), r
    per_entry[at, 0] -= 12345
    assert int(torch.count_nonzero(per_entry)) == 0, "entries still claimed"
    got = run(2)  # the same entries again
    assert np.all(np.abs(got - want) <= 4e-6 * want)
    assert int(torch.count_nonzero(per_entry)) == 0

"""How the rows that survive are numbered and gathered at the end: in one launch for small results, in two for larger ones
(finish_rows_kernel; compact_kernel and gather_rows_kernel).  Batches on both sides of its limits, in rows and in bytes, give the
survivors, numbers and bits that the same rows give in small batches."""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,batch,window", [
    (64, 8192, 64), (64, 8193, 64), (64, 16385, 64),                       # rows
    (4096, 4096, 4096), (4096, 4097, 4096),                                # 64 MB, and a row more
    (65536, 256, 4096), (65536, 257, 4096),
    (32, 1025, 32),                                                        # more rows than workgroups
])
def test_both_sides_of_the_limits(N, batch, window):
    import torch
    import paper_2007_14152_amd as sp
    rng = np.random.default_rng(N + batch)
    idx = [np.sort(rng.integers(0, window, size=(N, 32)) + np.arange(N)[:, None] // window * window, axis=1).astype(np.int32) for _ in range(2)]
    m = sp.Model(idx, [np.full((N, 32), 0.0625, np.float32)] * 2, np.full(N, -0.3, np.float32))
    Y0 = torch.from_numpy(synth.gen_y0(batch, N, 71, density="mixed")).to("cuda:0")
    n, rows, Y = m.infer(Y0)
    assert 0 < n < batch and m.infer(Y0, want_Y=False)[0] == n
    assert torch.equal(m.infer(Y0, want_Y=False)[1], rows)
    step = max(1, batch // 5)
    parts = [(lo, m.infer(Y0[lo:lo + step].contiguous())) for lo in range(0, batch, step)]
    m.close()
    assert sum(p[0] for _, p in parts) == n
    assert torch.equal(torch.cat([p[1] + lo for lo, p in parts]), rows) and torch.equal(torch.cat([p[2] for _, p in parts]), Y)

"""Networks of strided sums -- neuron j reads the columns (j + off + k S) mod N with one weight -- which strided_kernel runs
with the rows in LDS and sums shared along the orbits of "+S".  Orbits of 32, of lengths that 33 does and does not divide,
strides that wrap around the row end inside a lane's span, one and several pairs of rows per pass, odd batches, several
passes and launches, rows of fewer columns than it takes; against the oracle, and the same bits whatever the batch and wherever the weights live."""
import numpy as np
import pytest

import oracle
import synth
from parity_util import check_against_oracle

pytestmark = pytest.mark.gpu


def layer(N, S, off):
    return np.sort((np.arange(N)[:, None] + off + S * np.arange(32)[None, :]) % N, axis=1).astype(np.int32)


def network(N, strides, weight, offs=(0,)):
    idx = [layer(N, s, offs[l % len(offs)]) for l, s in enumerate(strides)]
    val = [np.full((N, 32), weight, np.float32)] * len(strides)
    return idx, val


@pytest.mark.parametrize("N,strides,batch,weight,offs", [
    (32, (1, 1), 5, 0.0625, (0, 31)),                  # one orbit of 32 for the whole row
    (36, (1, 1, 1), 400, 0.0625, (0, 5)),              # orbits of 36, two lanes with 30 neurons in common
    (100, (3, 1, 2), 1000, 0.07, (0, 99)),             # 16 pairs of rows per pass
    (1024, (1, 32, 8, 32), 4001, 0.0625, (0,)),        # several passes, the last of one row
    (1056, (32, 1), 77, 0.0625, (0,)),                 # orbits of 33
    (1088, (32, 1, 2), 2000, 0.0625, (7, 0)),          # orbits of 34
    (4096, (1, 32, 128, 1, 32, 128), 3000, 0.0625, (0,)),  # compacted between two launches
    (8188, (1, 4, 92), 301, 0.0625, (8187, 3)),
    (16384, (1, 32, 512, 2, 264, 3), 301, 0.0625, (0, 1, 16383)),
    (16384, (512, 1), 1, 0.0625, (0,)),
    # (the sizes below 1152 go to the kernels for any columns; from here on the same edges in strided_kernel)
    (1148, (1, 3), 70, 0.0625, (0,)),                  # one size below: as before
    (1152, (36, 1, 36), 8001, 0.0625, (0, 1151)),      # orbits of 32 and the whole row, seven pairs of rows per pass, the last row alone
    (1152, (1, 36), 5, 0.07, (0,)),
    (1188, (36, 1, 1), 400, 0.0625, (0, 5)),           # orbits of 33
    (1224, (36, 3), 2000, 0.0625, (7, 0)),             # orbits of 34 and 408
    (1320, (40, 37, 2), 77, 0.0625, (0,)),             # a stride that has no divisor in common with the row
    (2048, (3,), 50, 0.0625, (0,)),                    # one layer
])
def test_strided_networks(N, strides, batch, weight, offs):
    import torch
    import paper_2007_14152_amd as sp
    L = len(strides)
    idx, val = network(N, strides, weight, offs)
    bias = synth.gen_bias(N, -0.3)
    Y0 = synth.gen_y0(batch, N, 41, density="mixed")
    if batch > 8:
        Y0[5] = 0
    ids = np.arange(batch) if batch * N <= 1 << 23 else np.r_[0:batch // 8, batch - batch // 8:batch]
    ref = oracle.infer(idx, val, bias, Y0[ids])
    m = sp.Model(idx, val, bias)
    m.set_profiling(True)
    y0 = torch.from_numpy(Y0).to("cuda:0")
    n, rows, Y = m.infer(y0)
    launches, resident = m.launches()
    assert resident == launches and (L <= 4) <= (launches == 1)   # no layer of its own
    assert (m.row_kernel() == sp.SPDNN_ROWS_STRIDED) == (N >= 1152)
    run, rows_in, _ = m.profile()
    rows_h, Y_h = rows.cpu().numpy(), Y.cpu().numpy()
    mine = np.isin(rows_h, ids)
    check_against_oracle(ref, int(mine.sum()), rows_h[mine], Y_h[mine], row_ids=ids, what="strided N=%d %s" % (N, strides))
    if len(ids) == batch and not (ref.fragile_layer >= 0).any():
        assert [int(x) for x in rows_in[:run]] == [int(x) for x in ref.active_per_layer[:run]]
    # fewer rows, another split into launches: the same rows' bits
    few = max(1, batch // 3)
    m.set_profiling(False)
    n2, rows2, Y2 = m.infer(y0[:few].contiguous())
    keep = rows < few
    assert n2 == int(keep.sum()) and torch.equal(rows2, rows[keep]) and torch.equal(Y2, Y[keep])
    m.close()
    ooc = sp.Model(idx, val, bias, out_of_core=True)
    n3, rows3, Y3 = ooc.infer(y0)
    assert n3 == n and torch.equal(rows3, rows) and torch.equal(Y3, Y)
    ooc.close()


@pytest.mark.parametrize("change", ["column", "weight", "infinite weight", "bias", "two strides", "duplicate", "too many lanes"])
def test_what_is_no_strided_network_runs_as_before(change):
    """One connection, weight or bias out of line, a pattern that is not one sequence, a weight whose products cannot be
    summed first, or orbits that take more lanes than a workgroup has: the general kernels, with the oracle's result."""
    import paper_2007_14152_amd as sp
    N, L, batch = (16320, 2, 9) if change == "too many lanes" else (8192, 2, 9)
    idx, val = network(N, (480, 480) if change == "too many lanes" else (1, 32), 0.0625)
    val = [v.copy() for v in val]
    bias = synth.gen_bias(N, -0.3)
    if change == "column":
        idx[1][N - 1][7] = (idx[1][N - 1][7] + 1) % N
    elif change == "weight":
        val[1][N - 1][31] = np.nextafter(np.float32(0.0625), np.float32(1))
    elif change == "infinite weight":
        val[1][:] = np.inf
    elif change == "bias":
        bias[N - 1] = -0.31
    elif change == "two strides":
        idx[1] = np.sort(np.concatenate([layer(N, 1, 0)[:, :16], layer(N, 2, 100)[:, :16]], axis=1), axis=1)
    elif change == "duplicate":
        idx[1][5][3] = idx[1][5][4]
    Y0 = synth.gen_y0(batch, N, 43, density="mixed")
    ref = oracle.infer(idx, val, bias, Y0)
    m = sp.Model(idx, val, bias)
    from parity_util import gpu_infer
    n, rows, Y = gpu_infer(idx, val, bias, Y0, model=m)
    assert m.launches()[1] == 0 and m.row_kernel() == sp.SPDNN_ROWS_NONE
    m.close()
    if change == "infinite weight":  # infinity times 0 is NaN, which the kernels' maximum with 0 turns into 0: an output is 0 or 32
        ref.Y = np.nan_to_num(ref.Y, nan=0.0)
    check_against_oracle(ref, n, rows, Y, what=change)


@pytest.mark.parametrize("N,strides,batch", [
    (1152, (1, 36, 5), 3001),       # several pairs of rows per pass
    (8192, (256, 1, 3), 30),        # orbits of 32 first
    (16384, (1, 512), 9),
])
@pytest.mark.parametrize("weights", [(0.07,), (0.0613, -0.04, 0.09), (0.05, 0.0, 0.07), (-0.03, 0.1)])
def test_inputs_and_weights_of_any_sign(N, strides, batch, weights):
    """Real inputs between -5 and 40, blank rows, and rows of a few values; weights that are no power of two, negative and zero:
    against the oracle, and against 64 bits.  Layer 0 rounds the products before it adds them up (inputs may be of any size), later layers the sum:
    32 products and 31 additions of relative error u = 2^-24 each at most, then weight and bias in one, so an output differs from the exact one
    by at most 33 u (sum of the magnitudes), layer by layer."""
    import torch
    import paper_2007_14152_amd as sp
    L = len(strides)
    rng = np.random.default_rng(N + len(weights))
    idx, _ = network(N, strides, 0.0, (3, 0))
    w = [np.float32(weights[l % len(weights)]) for l in range(L)]
    val = [np.full((N, 32), x, np.float32) for x in w]
    bias = synth.gen_bias(N, -0.02)
    Y0 = rng.uniform(-5, 40, size=(batch, N)).astype(np.float32)
    Y0[1::4] *= rng.uniform(size=Y0[1::4].shape) < 0.05
    Y0[2] = 0
    ids = np.unique(np.r_[0:min(batch, 12), batch - 5:batch])
    ref = oracle.infer(idx, val, bias, Y0[ids])
    m = sp.Model(idx, val, bias)
    n, rows, Y = m.infer(torch.from_numpy(Y0).to("cuda:0"))
    assert m.row_kernel() == sp.SPDNN_ROWS_STRIDED
    m.close()
    rows, Y = rows.cpu().numpy(), Y.cpu().numpy()
    mine = np.isin(rows, ids)
    check_against_oracle(ref, int(mine.sum()), rows[mine], Y[mine], row_ids=ids, what="strided N=%d %s" % (N, weights))
    y, bound = Y0[ids].astype(np.float64), np.zeros((len(ids), N))
    for c, x in zip(idx, w.copy()):
        a = abs(np.float64(x))
        bound = a * sum(bound[:, c[:, k]] for k in range(32)) + 33 * 2.0 ** -24 * (a * sum(np.abs(y[:, c[:, k]]) for k in range(32)) + 0.02)
        y = np.clip(np.float64(x) * sum(y[:, c[:, k]] for k in range(32)) + np.float64(bias[0]), 0, 32)
    full = np.zeros_like(y)
    full[np.searchsorted(ids, rows[mine])] = Y[mine]
    assert (np.abs(full - y) <= bound * 1.001).all()


@pytest.mark.parametrize("N,strides,batch,weight,offs", [
    (2048, (1, 2, 4, 8, 16, 32, 64), 300, 0.0625, (0, 2047, 33)),       # all that leave orbits of 32 or of 64 and more; several pairs of rows
    (4096, (16, 32, 64, 128), 41, 0.07, (4095, 0, 31)),                 # orbits of 256 down to 32
    (8192, (256, 128, 1, 64), 30, 0.0625, (0, 127, 8191)),
    (16384, (1, 2, 4, 8, 16, 32, 64, 128, 256, 512), 9, 0.0625, (0, 16383, 5)),  # a pair of rows per pass
    (16384, (512, 256, 512), 600, 0.0625, (511, 512, 8000)),
    (12288, (1, 64, 128), 21, 0.0625, (0, 12287)),                      # rows that are no power of two
    (12288, (128, 256), 21, 0.0625, (12000, 12287)),                    # orbits of 48: a lane's 64 entries go past the row end twice
    (1280, (4, 16, 20), 500, 0.0625, (1279, 0)),                        # orbits of 320, 80 and 64, the last stride no power of two
])
def test_strides_that_are_known_beforehand(N, strides, batch, weight, offs):
    test_strided_networks(N, strides, batch, weight, offs)


@pytest.mark.parametrize("N,strides", [(2048, (1, 64)), (16384, (32, 1)), (12288, (3, 256))])
def test_infinite_inputs(N, strides):
    """Infinity is clipped to 32, infinity less infinity and NaN give 0, in the neurons that read them."""
    import torch
    import paper_2007_14152_amd as sp
    idx, val = network(N, strides, 0.0625, (N - 1,))
    bias = synth.gen_bias(N, -0.3)
    Y0 = synth.gen_y0(6, N, 7, density="mixed")
    Y0[0, 17], Y0[1, N - 1], Y0[2, 100], Y0[2, 101], Y0[3, 0] = np.inf, -np.inf, np.inf, -np.inf, np.nan
    y = Y0.astype(np.float64)
    with np.errstate(invalid="ignore"):
        for i, v in zip(idx, val):
            s = y[:, i].sum(2) * np.float64(v[0, 0]) + np.float64(np.float32(-0.3))
            y = np.clip(np.nan_to_num(s, nan=0.0, posinf=np.inf, neginf=-np.inf), 0.0, 32.0)
    m = sp.Model(idx, val, bias)
    n, rows, Y = m.infer(torch.from_numpy(Y0).to("cuda:0"))
    assert m.row_kernel() == sp.SPDNN_ROWS_STRIDED
    alive = np.flatnonzero((y > 0).any(1))
    assert [int(r) for r in rows] == [int(r) for r in alive]
    # weights are 1/16, inputs 0 and 1: 31 additions and one rounding per layer, 34 u of at most 32 * 32 / 16 + 0.3
    np.testing.assert_allclose(Y.cpu().numpy(), y[alive], rtol=0, atol=2 * 34 * 2.0**-24 * 64.3)
    m.close()


@pytest.mark.parametrize("N,strides", [(2048, (1, 64)), (16384, (32, 1)), (12288, (3, 256))])  # several pairs of rows, one, a stride like any other
@pytest.mark.parametrize("weight", [1e-38, 1e-40, 1e-43, 1e-44])
@pytest.mark.parametrize("bias", [-0.01, -1e-6, 0.0])
def test_small_weights_on_large_inputs(N, strides, weight, bias):
    """A first layer whose weight is near the end of the 32-bit range or below its normal part, and inputs that make up for it: the products
    are ordinary numbers with all their bits.  Against 64 bits, the bound of test_inputs_and_weights_of_any_sign."""
    rng = np.random.default_rng(N)
    Y0 = rng.uniform(0.5e38, 1e38, size=(7, N)).astype(np.float32)
    Y0[2:] *= rng.uniform(size=(5, N)) < 0.1
    against_64_bits(N, strides, (weight, 0.0625), bias, Y0)


@pytest.mark.parametrize("N,strides", [(2048, (1, 64)), (16384, (32, 1)), (12288, (3, 256))])
@pytest.mark.parametrize("weights", [(1.0, 1.0), (0.07, 0.0613)])
@pytest.mark.parametrize("bias", [0.0, -2.0 ** -149, -2.0 ** -140, -2.0 ** -61, -2.0 ** -60])
def test_small_values(N, strides, weights, bias):
    """Rows of the smallest numbers, whose outputs are as small where the bias is, and still count as outputs."""
    rng = np.random.default_rng(N + 1)
    Y0 = np.zeros((6, N), np.float32)
    for b, e in enumerate((-149, -146, -130, -120, -62, -58)):
        Y0[b] = np.ldexp(rng.uniform(1, 2, size=N), e) * (rng.uniform(size=N) < 0.2)
    against_64_bits(N, strides, weights, bias, Y0)


def against_64_bits(N, strides, weights, bias, Y0):
    """33 roundings of relative error 2^-24 per layer (32 products or one, 31 additions, one multiply-add), or half of 2^-149 where that is more."""
    import torch
    import paper_2007_14152_amd as sp
    idx, _ = network(N, strides, 0.0, (N - 1,))
    w = [np.float32(x) for x in weights]
    b = np.float32(bias)
    m = sp.Model(idx, [np.full((N, 32), x, np.float32) for x in w], np.full(N, b, np.float32))
    n, rows, Y = m.infer(torch.from_numpy(Y0).to("cuda:0"))
    assert m.row_kernel() == sp.SPDNN_ROWS_STRIDED
    m.close()
    y, bound = Y0.astype(np.float64), np.zeros(Y0.shape)
    for i, x in zip(idx, w):
        s, x = y[:, i].sum(2), np.float64(x)
        bound = x * bound[:, i].sum(2) + 33 * (2.0 ** -24 * (x * s + abs(np.float64(b))) + 2.0 ** -150)
        y = np.clip(x * s + np.float64(b), 0.0, 32.0)
    full = np.zeros_like(y)
    full[rows.cpu().numpy()] = Y.cpu().numpy()
    assert (np.abs(full - y) <= bound * 1.001).all()
    assert not ((y > bound * 1.001).any(1) & ~np.isin(np.arange(len(y)), rows.cpu().numpy())).any()

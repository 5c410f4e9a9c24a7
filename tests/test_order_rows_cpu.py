"""Which order of connections rows of which length get (csrc/spdnn_order.h): steps that read a quad twice come first for rows of one
stage, 4096 columns; for longer ones every step is a matching that reads as many different quads as can be."""
import ctypes

import numpy as np
import pytest
import synth
from scipy.sparse import csr_matrix
from scipy.sparse.csgraph import maximum_bipartite_matching

from paper_2007_14152_amd import build as hip_build
from test_order_cpu import brute_cost, lib, order  # noqa: F401 (lib is a fixture)


def order_row(lib, quads, nsteps, N):  # noqa: F811
    lib.spdnn_order_row_host.argtypes = [ctypes.c_void_p, ctypes.c_void_p, ctypes.c_int, ctypes.c_int]
    quads = np.ascontiguousarray(quads, dtype=np.uint8)
    step_of = np.zeros((16, 32), dtype=np.uint8)
    return lib.spdnn_order_row_host(quads.ctypes.data, step_of.ctypes.data, nsteps, N), step_of


def most_quads(quads, left):
    """The most lanes that can read different quads, of the connections `left` (bool [16, 32])."""
    graph = np.zeros((16, 16), np.int8)
    l, k = np.nonzero(left)
    graph[l, quads[l, k]] = 1
    return int((maximum_bipartite_matching(csr_matrix(graph)) >= 0).sum())


@pytest.mark.parametrize("nsteps", [8, 16, 32])
@pytest.mark.parametrize("N", [4097, 65536])
def test_long_rows_read_as_many_quads_as_can_be_in_every_step(lib, nsteps, N):  # noqa: F811
    rng = np.random.default_rng(nsteps)
    for trial in range(20):
        quads = np.full((16, 32), 255, dtype=np.uint8)
        for l in range(16):  # stages hold up to nsteps connections of a neuron; in half of the trials all lanes hold as many
            n = nsteps if trial % 2 else rng.integers(0, nsteps + 1)
            quads[l, :n] = rng.integers(0, 16, size=n)
        cost, step_of = order_row(lib, quads, nsteps, N)
        assert cost == brute_cost(quads, step_of)
        left = quads != 255
        assert np.array_equal(step_of != 255, left)
        for step in range(nsteps):
            l, k = np.nonzero((step_of == step) & left)
            assert len(set(l)) == len(l)
            assert len(set(quads[l, k])) == most_quads(quads, left), (trial, step)
            left[l, k] = False


def test_short_rows_have_the_double_steps(lib):  # noqa: F811
    rng = np.random.default_rng(7)
    fewer = 0
    for _ in range(20):
        quads = rng.integers(0, 16, size=(16, 32)).astype(np.uint8)
        cost, step_of = order_row(lib, quads, 32, 4096)
        assert (cost, step_of.tolist()) == (lambda c, s: (c, s.tolist()))(*order(lib, quads))
        fewer += order_row(lib, quads, 32, 65536)[0] - cost
    assert fewer > 0


@pytest.mark.parametrize("config,limit", [(0, 1.05), (2, 1.05), (3, 1.12), (4, 1.12)])
def test_benchmark_patterns_at_their_own_length(lib, config, limit):  # noqa: F811
    """1024 and 4096 columns with double steps, 16384 and 65536 with single matchings."""
    c = synth.config(config)
    idx = synth.gen_layer(c["N"], 0, c["seed"], c["window"])[:1024]
    cost = bound = 0
    for g in ((idx - (idx.min() // 4) * 4) % 16).astype(np.uint8).reshape(-1, 16, 32):
        cost += order_row(lib, g, 32, c["N"])[0]
        bound += max(32, int(np.bincount(g.ravel(), minlength=16).max()))
    assert cost < limit * bound


@pytest.mark.parametrize("nsteps", [8, 16, 24, 32])  # a layer's steps come in eights
@pytest.mark.parametrize("half", [0, 1])
def test_spread_steps_are_a_permutation(lib, nsteps, half):  # noqa: F811
    at = [lib.spdnn_spread_step_host(step, nsteps, half) for step in range(nsteps)]
    assert sorted(at) == list(range(nsteps))
    # the first half, where the double steps are, leaves no four reads in a row without one of its own
    assert max(np.diff([-1] + sorted(at[:nsteps // 2]) + [nsteps])) <= 4

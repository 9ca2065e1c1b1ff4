"""How a sweep() call is split into launches, at the sizes where the split
changes, against the oracle: a run of four sweeps of 4-bit lattices from L =
4096 on (a vector a thread, 16-row tiles and more) and of 1-bit ones up to the
largest, runs of three and four on both sides of the sizes between them, calls
of two sweeps at sizes that take a launch per half-sweep for them, and
1-bit sizes that take no runs at all."""
import math

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

BETA_C = math.log(1 + math.sqrt(2)) / 2


@pytest.fixture(scope="module")
def mcl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_18624_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("model,L,ns", [
    (0, 4096, (4,)), (1, 4160, (4,)), (0, 5120, (8,)), (1, 7168, (4,)), (0, 7168, (4,)),        # four, by vectors
    (2, 4352, (4,)), (2, 8192, (4,)), (2, 12288, (4,)),                                         # four, 1-bit
    (0, 1472, (4, 7)), (1, 1536, (3, 4, 7)), (0, 3584, (3, 4)), (1, 3648, (4,)),                # three, or four
    (0, 3840, (2,)), (1, 3904, (2, 3)), (0, 4096, (2, 3)), (1, 4096, (2,)), (0, 4160, (2,)),    # two sweeps
    (2, 11008, (2,)), (2, 11264, (2,)), (2, 11520, (2, 3))])
def test_runs(mcl, model, L, ns):
    print("runs", model, L, ns, flush=True)
    beta, D = (1 / 1.4, 1.0) if model == 1 else (BETA_C, 0.0)
    lat = mcl.Lattice(model, L, 6500 + L)
    want = oracle.init(model, L, 6500 + L)
    t = 0
    for n in ns:
        lat.sweep(n, beta, D)
        oracle.sweep(want, model, 6500 + L, t, n, beta, D, nthreads=16)
        t += n
        assert lat.t == t
        assert np.array_equal(lat.read(), want), n
    lat.free()


@pytest.mark.parametrize("model,sizes", [(0, (64, 192, 1024, 2112)), (1, (64, 256, 1088)), (2, (256, 768, 2048))])
def test_a_launch_per_half_sweep_at_small_sizes(mcl, monkeypatch, model, sizes):
    """The band kernels where other forms run by default."""
    monkeypatch.setenv("MCL_SWEEP_GRAPH", "0")
    beta, D = (1 / 1.4, 1.0) if model == 1 else (BETA_C, 0.0)
    for L in sizes:
        print("half-sweeps", model, L, flush=True)
        lat = mcl.Lattice(model, L, 6600 + L)
        want = oracle.init(model, L, 6600 + L)
        for t, n in ((0, 1), (1, 5)):
            lat.sweep(n, beta, D)
            oracle.sweep(want, model, 6600 + L, t, n, beta, D, nthreads=8)
            assert np.array_equal(lat.read(), want), (L, n)
        lat.free()

"""B, M, Q, counts and the sigma-h histogram of states in which threads of the
B/M/Q pass see more opposite than equal neighbours, so that their shares of
the bond sum are negative: the random start before its first sweep, the
antiferromagnetic checkerboard (every bond -1), and stripes of two of its
kind.  Without correlations (the B/M/Q pass) and with them, against the
oracle: whole numbers, equality."""
import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mcl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_18624_amd as m
    m.lib()
    return m


def _states(model, L):
    y, x = np.indices((L, L))
    checker = np.where((x + y) & 1, 1, -1).astype(np.int8)
    stripes = checker.copy()
    stripes[L // 4:L // 2] = 1                                  # ordered rows between
    yield "random", oracle.init(model, L, 61 + L)
    yield "checkerboard", checker
    yield "stripes", stripes


@pytest.mark.parametrize("model,L", [(0, 64), (0, 256), (0, 576), (0, 4096), (1, 64), (1, 576), (2, 256), (2, 1024)])
def test_negative_shares_of_the_bond_sum(mcl, model, L):
    lat = mcl.Lattice(model, L, 3)
    for name, s in _states(model, L):
        print("bond sum", model, L, name, flush=True)
        lat.write(s, 0)
        want = oracle.measure(s, 8)
        sd = [int(v) for v in oracle.sd_hist(s, 8)]
        for mode in (mcl.CORR_NONE, mcl.CORR_FULL) if L <= 576 else (mcl.CORR_NONE, mcl.CORR_PROTOCOL):
            m = lat.measure(mode)
            assert (m["B"], m["M"], m["Q"], m["counts"], m["invalid"]) == (
                want["B"], want["M"], want["Q"], want["counts"], 0), (name, mode)
            assert m["sd"] == sd, (name, mode)
    lat.free()

"""1-bit lattices well below T_c, where buckets of the draw table hold several
thresholds and words take the exact search (at T_c / 2 three of the 4096, so
31% of a wave's words per stream; at T_c none): the kernels that take a row
band per thread against the oracle, alone and in a batch, and what the search
may cost them."""
import math
import time

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

BETA_C = math.log(1 + math.sqrt(2)) / 2
LUT = 2


@pytest.fixture(scope="module")
def mcl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_18624_amd as m
    m.lib()
    return m


@pytest.mark.parametrize("group", [False, True])
@pytest.mark.parametrize("fraction", [0.6, 0.5, 0.2])
def test_cold_bands(mcl, fraction, group):
    print("cold bands", fraction, group, flush=True)
    L, seed, beta, n = 8192, 6100, BETA_C / fraction, 1
    lats = [mcl.Lattice(LUT, L, seed + i) for i in range(2 if group else 1)]
    for _ in range(2):                                          # (one sweep at a time: a launch per half-sweep)
        if group:
            mcl.group_sweep(lats, n, beta, 0.0)
        else:
            lats[0].sweep(n, beta)
    W, pad = 64, 4
    for i, lat in enumerate(lats):
        for x0, y0 in ((0, 0), (L - 16, L // 2 - 32), (L // 3, L - 24)):
            got = lat.read_window(x0, y0, W, W)
            patch = oracle.window_run(LUT, L, seed + i, (x0 - pad) % L, (y0 - pad) % L, W + 2 * pad, 2, beta)
            assert np.array_equal(got, patch[pad:pad + W, pad:pad + W]), (i, x0, y0)
        lat.free()


@pytest.mark.parametrize("L,ns", [(256, (1, 5)), (512, (4, 7)), (1536, (1, 6)), (4352, (4,))])
def test_cold_rows_in_lds(mcl, L, ns):
    """A word per thread, a whole lattice and tiles of rows in LDS."""
    print("cold rows in LDS", L, flush=True)
    beta, t = 2 * BETA_C, 0
    lat = mcl.Lattice(LUT, L, 6150 + L)
    want = oracle.init(LUT, L, 6150 + L)
    for n in ns:
        lat.sweep(n, beta)
        oracle.sweep(want, LUT, 6150 + L, t, n, beta, 0.0, nthreads=16)
        t += n
        assert np.array_equal(lat.read(), want), n
    lat.free()


def test_what_the_exact_search_costs(mcl):
    """A word of 32 cells is about 242 VALU instructions; the search, 8 x 16
    instructions in eight independent chains, by 31% of them in each of two
    streams adds 79: a third.  As one serial chain of 8 x 26 it would be 129
    and the latency of 24 table reads in a row.  Both temperatures in turn, in
    one process; the bound is half as much again.  A launch per half-sweep (one
    sweep of L = 8192) and several sweeps of rows in LDS (32 of L = 4096)."""
    import torch
    print("cost of the exact search", flush=True)
    for L, n, calls in ((8192, 1, 100), (4096, 32, 10)):
        lat = mcl.Lattice(LUT, L, 6200)

        def once(beta):
            torch.cuda.synchronize()
            a = time.perf_counter()
            for _ in range(calls):
                lat.sweep(n, beta)
            torch.cuda.synchronize()
            return (time.perf_counter() - a) / calls * 1e6

        once(BETA_C)
        warm, cold = [], []
        for _ in range(8):
            warm.append(once(BETA_C))
            cold.append(once(2 * BETA_C))
        lat.free()
        print(L, n, "us a call at T_c", min(warm), "at T_c / 2", min(cold), flush=True)
        assert min(cold) < 1.5 * min(warm)

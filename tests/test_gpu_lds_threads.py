"""Two threads that launch the same kernels for lattices of different sizes at
the same time, each on a stream of its own: the dynamic LDS that a kernel may
take is a property of the kernel, not of the launch, so no thread's launch may
leave less than another's needs.  Sweeps of several launches and measurements
at every distance and in the protocol, against the same calls one after the
other."""
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def mcl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_18624_amd as m
    m.lib()
    return m


def _work(mcl, lat, calls, mode, out):
    try:
        for _ in range(calls):
            lat.sweep(2, 0.5, 1.0)
            m = lat.measure(mode)
            out.append((m["B"], m["M"], m["Cx"].tobytes(), m["Cy"].tobytes()))
    except Exception as e:                                      # (to the test's thread)
        out.append(e)


@pytest.mark.parametrize("model,sizes,mode", [(0, (4096, 7168), 0), (1, (640, 3008), 0), (2, (2304, 12288), 0),
                                              (0, (576, 2112), 1), (2, (2304, 4352), 1), (2, (4096, 65536), 2)])
def test_one_kernel_two_sizes(mcl, model, sizes, mode):
    import torch
    print("lds and threads", model, sizes, mode, flush=True)
    results = []
    for together in (False, True):
        lats = [mcl.Lattice(model, L, 6400 + L, stream=torch.cuda.Stream()) for L in sizes]
        outs = [[], []]
        calls = [60, 20] if mode != 2 else [30, 10]
        threads = [threading.Thread(target=_work, args=(mcl, lat, c, mode, out))
                   for lat, c, out in zip(lats, calls, outs)]
        for th in threads:
            th.start()
            if not together:
                th.join()
        for th in threads:
            th.join()
        for o in outs:
            assert not isinstance(o[-1], Exception), o[-1]
        results.append((outs, [lat.read_packed() for lat in lats]))
        for lat in lats:
            lat.free()
    assert results[0][0] == results[1][0]
    assert all(np.array_equal(a, b) for a, b in zip(results[0][1], results[1][1]))

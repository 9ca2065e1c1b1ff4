"""Spins to the host and back (read, write, read_window): one chunk, two and
several of the pinned buffers' rows, with a last one of fewer rows; windows
that wrap on both axes, of one site, and larger than a chunk.  A write that is
refused leaves the lattice as it was.  Whole numbers: equality."""
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


@pytest.mark.parametrize("model,L", [(0, 64), (0, 2048), (0, 2112), (0, 4352), (1, 192), (1, 2304), (2, 256), (2, 2304),
                                     (2, 4352)])
def test_spins_to_the_host_and_back(mcl, model, L):
    print("io", model, L, flush=True)
    lat = mcl.Lattice(model, L, 5400 + L)
    s = lat.read()
    assert np.array_equal(s, oracle.init(model, L, 5400 + L))
    packed = lat.read_packed()
    turned = s[::-1, ::-1].copy()
    lat.write(turned, 17)
    assert np.array_equal(lat.read(), turned) and lat.t == 17
    lat.write(s, 3)
    assert np.array_equal(lat.read_packed(), packed) and lat.t == 3
    for x0, y0, w, h in ((0, 0, 1, 1), (L - 3, L - 2, 40, 9), (5, L - 1, L, L), (17, 3, 33, min(L, 200))):
        want = np.roll(np.roll(s, -y0, 0), -x0, 1)[:h, :w]
        assert np.array_equal(lat.read_window(x0, y0, w, h), want), (x0, y0, w, h)
    for value in (5, -2, 0) if model != 1 else (5, -2):
        bad = s.copy()
        bad[L - 1, L - 1] = value
        with pytest.raises(mcl.MclError) as e:
            lat.write(bad, 0)
        assert e.value.code == -11
        assert lat.t == 3 and np.array_equal(lat.read_packed(), packed)
    lat.free()

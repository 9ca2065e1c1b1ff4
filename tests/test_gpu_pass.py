"""The measurement pass (every-source correlations r = 0 .. 32 on the matrix
cores, B, M, Q, counts and the sigma-h histogram, and the bits that the
sampled passes read) against the oracle, at the edges of its split: less than
one 32-cell vector's neighbours (L = 64), a last strip and a last workgroup
with fewer columns, a workgroup whose waves have no columns at all, runs of
one, two and many tiles, and the smallest lattices with packed T bits.
Whole numbers: equality."""
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


@pytest.mark.parametrize("grid", [0, 3])
@pytest.mark.parametrize("model,L,mode", [
    (model, L, mode) for model in (0, 1, 2) for L, mode in
    ((64, 1), (64, 2), (128, 1), (192, 1), (256, 2), (512, 2), (576, 1), (768, 1), (1024, 2), (1088, 1), (2048, 2),
     (2304, 1)) if model != 2 or L % 256 == 0])
def test_measurement_pass(mcl, monkeypatch, model, L, mode, grid):
    print("measurement pass", model, L, mode, grid, flush=True)
    if grid:
        monkeypatch.setenv("MCL_MEASURE_GRID", str(grid))       # several units per workgroup
    beta, D = (1 / 1.4, 1.0) if model == 1 else (BETA_C, 0.0)
    lat = mcl.Lattice(model, L, 4900 + model)
    lat.sweep(2, beta, D)
    m = lat.measure(mode)
    s = lat.read()
    lat.free()
    om = oracle.measure(s, 16)
    assert (m["B"], m["M"], m["Q"], m["counts"], m["invalid"]) == (om["B"], om["M"], om["Q"], om["counts"], 0)
    assert m["sd"] == [int(v) for v in oracle.sd_hist(s, 16)]
    r = oracle.rset(mode, L, m["t"])
    Cx, Cy, ns = oracle.corr(s, mode, r, 16)
    assert np.array_equal(m["r"], r) and np.array_equal(m["nsrc"], ns)
    assert np.array_equal(m["Cx"], Cx)
    assert np.array_equal(m["Cy"], Cy)


@pytest.mark.parametrize("model", [0, 1])
def test_correlations_of_cells_that_hold_no_spin(mcl, model):
    """A cell that holds no spin counts in the correlations by the bits that
    define one: Ising +1 where bit 1 is set, else -1; Blume-Capel 0 where
    bit 0 is set, else as Ising."""
    print("correlations with invalid cells", model, flush=True)
    L = 512
    lat = mcl.Lattice(model, L, 4950 + model)
    buf = lat.read_packed().copy()
    rng = np.random.default_rng(6 + model)
    for p in rng.choice(buf.size, size=500, replace=False):
        buf[p] = rng.integers(0, 256)
    lat.write_packed(buf, 0)
    m = lat.measure(mcl.CORR_PROTOCOL)
    lat.free()
    cells = np.stack([buf & 15, buf >> 4], axis=-1).reshape(2, L, L // 2).astype(np.int8)
    spins = np.where(cells & 2, 1, -1)
    if model == 1:
        spins = np.where(cells & 1, 0, spins)
    s = np.empty((L, L), dtype=np.int8)
    y = np.arange(L)[:, None]
    for c in (0, 1):
        s[y, 2 * np.arange(L // 2)[None, :] + ((y + c) & 1)] = spins[c]
    Cx, Cy, _ = oracle.corr(s, oracle.CORR_PROTOCOL, m["r"])
    assert np.array_equal(m["Cx"], Cx) and np.array_equal(m["Cy"], Cy)


@pytest.mark.parametrize("model,L", [(0, 8960), (1, 9024), (2, 8960), (2, 9216)])
def test_every_distance_at_the_limit_of_lds(mcl, model, L):
    """FULL on both sides of the largest lattice whose rows fit LDS, a
    distance list's ends and a few between against the oracle."""
    print("full mode", model, L, flush=True)
    lat = mcl.Lattice(model, L, 4960 + model)
    m = lat.measure(mcl.CORR_FULL)
    s = lat.read()
    lat.free()
    assert np.array_equal(m["r"], np.arange(L // 2 + 1))
    r = np.array([0, 1, 32, 33, 34, 47, 48, 1000, 2049, L // 2 - 1, L // 2], dtype=np.int32)
    Cx, Cy, _ = oracle.corr(s, oracle.CORR_FULL, r, 16)
    assert np.array_equal(m["Cx"][r], Cx) and np.array_equal(m["Cy"][r], Cy)

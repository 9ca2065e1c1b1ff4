"""Every band height of the batched launches (2 .. 64 rows a thread) against
the oracle, bit for bit: small calls plan short bands, so the heights of large
calls are set by MCL_GROUP_ROWS, and the planned ones are asserted.  Rows of
whole waves of vectors (L = 4096) and of a number that fills no tile, a
band at either end, plain launches and replayed ones, one workgroup per tile
and fewer."""
import math

import numpy as np
import pytest

import oracle

pytestmark = pytest.mark.gpu

BETA_C = math.log(1 + math.sqrt(2)) / 2
REPS = [(0, 1088, 3), (1, 1024, 3), (2, 2304, 2), (1, 1152, 2), (0, 4096, 1), (2, 2048, 3), (1, 4096, 1)]


@pytest.fixture(scope="module")
def mcl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2502_18624_amd as m
    m.lib()
    return m


def _params(model, i):
    return (1 / 1.4 + i / 50, 1.0) if model == 1 else (BETA_C * (0.8 + i / 10), 0.0)


@pytest.fixture(scope="module")
def wanted():
    out = []
    for i, (model, L, n) in enumerate(REPS):
        s = oracle.init(model, L, 6300 + i)
        oracle.sweep(s, model, 6300 + i, 0, 3 * n, *_params(model, i), nthreads=16)
        out.append(s)
    return out


@pytest.mark.parametrize("rows,wg_per_cu,split", [(2, 0, 0), (4, 0, 1), (8, 1, 0), (16, 0, 0), (16, 1, 1), (32, 0, 0),
                                                  (32, 1, 0), (64, 0, 0), (64, 1, 0), (64, 0, 1)])
def test_band_heights_of_a_batch(mcl, monkeypatch, wanted, rows, wg_per_cu, split):
    from paper_2502_18624_amd import autotune
    print("group rows", rows, wg_per_cu, split, flush=True)
    monkeypatch.setenv("MCL_GROUP_ROWS", str(rows))
    old, tuning = autotune.get_tuning(), autotune.get_tuning()
    for k in range(21):
        tuning.rows_log2L[k] = max(8, rows)
    tuning.wg_per_cu, tuning.split_models, tuning.use_graph = wg_per_cu, split, 1
    lats = [mcl.Lattice(m, L, 6300 + i) for i, (m, L, _) in enumerate(REPS)]
    params = [_params(m, i) for i, (m, _, _) in enumerate(REPS)]
    autotune.set_tuning(tuning)
    try:
        assert autotune.planned_rows([r[:2] for r in REPS]) == [rows] * len(REPS)
        for _ in range(3):                                       # plain, captured, replayed
            mcl.group_sweep(lats, [r[2] for r in REPS], [p[0] for p in params], [p[1] for p in params])
    finally:
        autotune.set_tuning(old)
    for lat, want, rep in zip(lats, wanted, REPS):
        assert np.array_equal(lat.read(), want), rep
        lat.free()

"""Small lattices swept in one launch, both planes in a workgroup's LDS:
sweep() of one lattice and group_sweep() / group_sweep_noalloc() of many,
against the oracle, bit for bit.  Sizes at the edges of the rule: a wave with
rows of both parities (L = 64), rows of a number of vectors that is no power
of two, the largest that goes this way alone and the next; one sweep, the
fewest that go this way, and more than one launch's; the end of the counter;
batches above and below the count from which they go resident, with large
replicas beside them, replicas that end early and ones that do nothing."""
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


def _params(model):
    return (1 / 1.4, 1.0) if model == 1 else (BETA_C, 0.0)


@pytest.mark.parametrize("model,L", [(0, 64), (0, 128), (0, 192), (0, 256), (0, 320), (1, 64), (1, 192), (1, 256),
                                     (2, 256), (2, 512), (2, 768)])
def test_small_lattice(mcl, model, L):
    print("resident sweep", model, L, flush=True)
    beta, D = _params(model)
    seed = 5000 + L + model
    lat = mcl.Lattice(model, L, seed)
    want = oracle.init(model, L, seed)
    t = 0
    for n in (1, 4, 3, 300):
        lat.sweep(n, beta, D)
        oracle.sweep(want, model, seed, t, n, beta, D, nthreads=8)
        t += n
        assert lat.t == t
        assert np.array_equal(lat.read(), want), n
    # hot, cold and frozen, and the last sweep indices
    for beta, t0, n in ((0.0, 5, 5), (math.inf, 7, 4), (1.3, 2**32 - 6, 6)):
        lat.write(want, t0)
        lat.sweep(n, beta, D)
        oracle.sweep(want, model, seed, t0, n, beta, D, nthreads=8)
        assert np.array_equal(lat.read(), want), (beta, t0)
    lat.free()


@pytest.mark.parametrize("noalloc", [False, True])
@pytest.mark.parametrize("count,sizes", [(3, (64, 256)), (5, (64, 128, 1024)), (140, (64, 128, 192, 256, 384)),
                                         (134, (64, 256, 512, 1088))])
def test_batch_of_small_lattices(mcl, noalloc, count, sizes):
    print("resident batch", count, sizes, noalloc, flush=True)
    rng = np.random.default_rng(count)
    reps = []
    for i in range(count):
        model = int(rng.integers(0, 3))
        L = int(sizes[i % len(sizes)]) if i % len(sizes) else int(sizes[0])
        if model == 2:
            L = 256 if L <= 384 else 512
        n = int(rng.choice([0, 1, 3, 6])) if i else 260 if count < 10 else 6
        reps.append((model, L, 5100 + i, float(BETA_C / rng.uniform(0.5, 1.5)), 0.5 if model == 1 else 0.0, n))
    lats = [mcl.Lattice(m, L, s) for m, L, s, *_ in reps]
    for _ in range(2):
        mcl.group_sweep(lats, [r[5] for r in reps], [r[3] for r in reps], [r[4] for r in reps], noalloc=noalloc)
    for lat, (model, L, seed, beta, D, n) in zip(lats, reps):
        want = oracle.init(model, L, seed)
        oracle.sweep(want, model, seed, 0, 2 * n, beta, D, nthreads=8)
        assert lat.t == 2 * n
        assert np.array_equal(lat.read(), want), (model, L, n)
        lat.free()


@pytest.mark.parametrize("model,L", [(0, 320), (0, 1088), (0, 1600), (0, 3008), (0, 3072), (0, 3136), (0, 4096), (0, 4160), (0, 7168), (1, 256),
                                     (1, 448), (1, 1536), (1, 2112), (1, 5120), (2, 512), (2, 768), (2, 2304), (2, 4096), (2, 4352),
                                     (2, 12288)])
def test_several_sweeps_in_two_launches(mcl, model, L):
    """A sweep alone (a word per thread), and the launches that run several
    sweeps of tiles of rows and then what is left around the cuts: every length of a run of sweeps (2, 3, 4), words and
    vectors, tile heights that differ by a row, rows that start within a
    generator block of proposals, the end of the counter."""
    print("several sweeps", model, L, flush=True)
    beta, D = _params(model)
    seed = 5200 + L + model
    lat = mcl.Lattice(model, L, seed)
    want = oracle.init(model, L, seed)
    t = 0
    for n in (2, 1, 3, 4, 11) if L <= 2304 else (5, 1):
        lat.sweep(n, beta, D)
        oracle.sweep(want, model, seed, t, n, beta, D, nthreads=16)
        t += n
        assert lat.t == t
        assert np.array_equal(lat.read(), want), n
    if L <= 2304:
        lat.write(want, 2**32 - 3)
        lat.sweep(3, beta, D)
        oracle.sweep(want, model, seed, 2**32 - 3, 3, beta, D, nthreads=16)
        assert np.array_equal(lat.read(), want)
    lat.free()


@pytest.mark.parametrize("model,L", [(0, 128), (1, 512), (2, 768)])
def test_caller_captures_several_sweeps(mcl, model, L):
    """A caller's graph of 7 sweeps, replayed with eager work between."""
    import torch
    print("capture", model, L, flush=True)
    beta, D = _params(model)
    st = torch.cuda.Stream()
    lat = mcl.Lattice(model, L, 5300 + model, stream=st)
    want = lat.read()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=st):
        lat.sweep(7, beta, D)
    for k in range(3):
        g.replay()
        torch.cuda.synchronize()
        oracle.sweep(want, model, 5300 + model, 0, 7, beta, D, nthreads=8)
        assert np.array_equal(lat.read(), want), k
        x = torch.ones(4096, device="cuda")
        assert float((x + 1.0).sum()) == 8192.0
    lat.free()


@pytest.mark.parametrize("wg_per_cu,split", [(0, 0), (2, 0), (0, 1)])
@pytest.mark.parametrize("reps", [
    [(2, 2048)] + [(0, 320)] * 9,                                # most of the cost at the front,
    [(0, 320)] * 9 + [(1, 1088), (2, 1536)],                     # at the back
    [(2, 768), (0, 64)],                                         # fewer tiles than XCDs
    [(0, 640), (1, 704), (2, 1024), (0, 1472), (1, 64), (2, 256), (0, 1024)],
])
def test_shares_of_a_mixed_batch(mcl, reps, wg_per_cu, split):
    """The XCDs' shares of a batched launch, divided by cost: replicas of very
    different cost, shares that begin inside a replica or are empty, one
    workgroup per tile and fewer; a call three times, the last a replay."""
    from paper_2502_18624_amd import autotune
    print("shares", reps, wg_per_cu, split, flush=True)
    old, tuning = autotune.get_tuning(), autotune.get_tuning()
    tuning.wg_per_cu, tuning.split_models, tuning.use_graph = wg_per_cu, split, 1
    n = [3 - i % 2 for i in range(len(reps))]
    lats = [mcl.Lattice(m, L, 5400 + i) for i, (m, L) in enumerate(reps)]
    autotune.set_tuning(tuning)
    try:
        for _ in range(3):
            mcl.group_sweep(lats, n, [_params(m)[0] for m, _ in reps], [_params(m)[1] for m, _ in reps])
    finally:
        autotune.set_tuning(old)
    for i, (lat, (model, L)) in enumerate(zip(lats, reps)):
        want = oracle.init(model, L, 5400 + i)
        oracle.sweep(want, model, 5400 + i, 0, 3 * n[i], *_params(model), nthreads=16)
        assert np.array_equal(lat.read(), want), (i, model, L)
        lat.free()

"""The band heights that group_sweep plans (mcl_group_rows), against the rule
written out again: the tuning's height of a size, capped so that the call's
batched replicas give 2^20 threads (1-bit replicas at half the cap), and low
enough to fill a tile of 256 threads; none for replicas held in LDS or swept
alone.  No GPU."""
import ctypes

import numpy as np
import pytest


@pytest.fixture()
def lib(monkeypatch):
    import paper_2502_18624_amd as m
    monkeypatch.delenv("MCL_GROUP_ROWS", raising=False)
    return m.lib()


def _rule(shapes, tuned, forced=0):
    fits = lambda m, L: (L * L // 8 + 32768 if m == 2 else L * L // 2) <= 76 * 1024
    batched = [(m, L) for m, L in shapes if L <= 2**17]
    if len(batched) < 2:
        return [0] * len(shapes)
    every = all(L <= (512 if m == 2 else 256) for m, L in batched)
    many = sum(fits(m, L) for m, L in batched) >= 128
    resident = lambda m, L: every or (many and fits(m, L))
    vectors = lambda m, L: L // (256 if m == 2 else 64)

    def rows(m, L, cap):
        cap = max(2, cap // 2) if m == 2 and not forced else cap
        r = min(cap, tuned[L.bit_length() - 1])
        while r > 2 and vectors(m, L) * (L // r) < 256:
            r //= 2
        return r

    caps = [forced] if forced else [64, 32, 16, 8, 4, 2]
    cap = next((c for c in caps if sum(vectors(m, L) * (L // rows(m, L, c)) for m, L in batched
                                       if not resident(m, L)) >= 2**20), caps[-1])
    return [0 if L > 2**17 or resident(m, L) else rows(m, L, cap) for m, L in shapes]


@pytest.mark.parametrize("forced", [0, 2, 16, 64])
def test_planned_rows(lib, monkeypatch, forced):
    from paper_2502_18624_amd import autotune
    if forced:
        monkeypatch.setenv("MCL_GROUP_ROWS", str(forced + (2 < forced < 64)))          # (rounded down)
    old = autotune.get_tuning()
    rng = np.random.default_rng(7 + forced)
    heights = set()
    try:
        for k in range(60):
            t = autotune.get_tuning()
            for i in range(21):
                t.rows_log2L[i] = int(rng.choice([8, 16, 32, 64]))
            autotune.set_tuning(t)
            hi = 2.0 ** rng.uniform(8.2, 16)
            shapes = []
            for _ in range(int(2 ** rng.uniform(0, 9))):
                m = int(rng.integers(0, 3))
                unit = 256 if m == 2 else 64
                shapes.append((m, max(1, int(2.0 ** rng.uniform(6, np.log2(hi)) / unit)) * unit))
            if k % 10 == 0:
                shapes.append((2, 2**17 + 256))
            got = autotune.planned_rows(shapes)
            assert got == _rule(shapes, list(t.rows_log2L), forced), shapes
            heights.update(got)
    finally:
        autotune.set_tuning(old)
    assert heights >= ({0, 2, 4, 8, 16, 32, 64} if not forced else {0, 2} | {forced})


def test_planned_rows_arguments(lib):
    one = (ctypes.c_int * 1)
    L, rows = (ctypes.c_int64 * 1)(128), (ctypes.c_int32 * 1)()
    assert lib.mcl_group_rows(0, None, None, None) == 0
    assert lib.mcl_group_rows(-1, one(0), L, rows) == -9
    assert lib.mcl_group_rows(1, one(0), L, None) == -9
    assert lib.mcl_group_rows(1, one(3), L, rows) == -1
    assert lib.mcl_group_rows(1, one(2), L, rows) == -2
    assert lib.mcl_group_rows(1, one(0), L, rows) == 0 and rows[0] == 0

"""The autotuner's search, with the GPU work replaced by a clock that calls
every later candidate faster: settings that plan the same launches are not
searched, so noise installs none of them."""
import pytest


@pytest.fixture()
def tuner(monkeypatch):
    import torch

    from paper_2502_18624_amd import autotune, lattice
    monkeypatch.delenv("MCL_GROUP_ROWS", raising=False)
    monkeypatch.setattr(autotune, "_cache", {})
    monkeypatch.setattr(torch.cuda, "get_device_name", lambda *a: "none")

    class Nothing:
        def __init__(self, *a):
            pass

        def free(self):
            pass

    tried = []

    def clock(lats, *a):
        tried.append(autotune.tuning_dict(autotune.get_tuning()))
        return 1.0 / len(tried)

    monkeypatch.setattr(lattice, "Lattice", Nothing)
    monkeypatch.setattr(autotune, "_time_group", clock)
    old = autotune.get_tuning()
    yield autotune, tried
    autotune.set_tuning(old)


# calls whose bands the cap takes to 2 rows, ones held in LDS, and one replica
@pytest.mark.parametrize("shapes", [[(0, 512), (1, 768), (2, 1024)] * 3, [(0, 128)] * 4, [(1, 4096)], [(0, 64)] * 200])
def test_heights_without_effect_stay(tuner, shapes):
    autotune, tried = tuner
    before = list(autotune.get_tuning().rows_log2L)
    res = autotune.autotune_group(shapes)
    assert res["rows_log2L"] == before
    assert list(autotune.get_tuning().rows_log2L) == before
    if not any(autotune.planned_rows(shapes)):
        assert len(tried) == 1                                  # the present setting's time only


def test_every_plan_is_timed_once(tuner):
    """256 Blume-Capel replicas of L = 4096: the cap is 64 rows, all four heights differ."""
    autotune, tried = tuner
    shapes = [(1, 4096)] * 256 + [(0, 512)] * 2
    res = autotune.autotune_group(shapes)
    assert {t["rows_log2L"][12] for t in tried} == {8, 16, 32, 64}
    assert res["rows_log2L"][12] == 64                          # (each later one is "faster")
    assert res["rows_log2L"][9] == 8                            # (L = 512 fills a tile with 16 rows at most: 8 is the only other)
    plans = []
    for t in tried:
        if all(t[f] == tried[0][f] for f in autotune.FIELDS):   # the search of the heights
            autotune.set_tuning(autotune.tuning_from_dict(t))
            plans.append(tuple(autotune.planned_rows(shapes)))
    assert len(plans) == 5 and len(set(plans)) == 5

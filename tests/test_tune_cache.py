"""Which entries of a tune cache a plan takes, on the host: those of this
library's table of shapes and of the plan's boundaries."""
import json

import pytest

from paper_2502_06296_amd import autotune

GRID = (256, 128, 64)


class _Plan:
    def __init__(self, ybc, xbc):
        self.ybc, self.xbc, self.shape, self.set = ybc, xbc, (64, 128, 256), {}


@pytest.fixture
def cache(tmp_path, monkeypatch):
    table = autotune.SHAPE_TABLE
    monkeypatch.setattr(autotune, "_arch_key", lambda: f"gfx950|hip7|shapes{table}")
    monkeypatch.setattr(autotune, "set_variant", lambda plan, stage, v: plan.set.update({stage: v}) or True)
    path = tmp_path / "tune.json"
    entry = {"zsolve_variant": 41, "xshape": 1, "yshape": 2}
    path.write_text(json.dumps({autotune.poisson_key(*GRID, "fp64"): entry}))
    return str(path), entry


def test_a_plan_takes_the_entry_of_its_own_boundaries(cache):
    path, entry = cache
    assert autotune.apply_cached_poisson(_Plan(0, 0), *GRID, "fp64", path) == entry
    for ybc, xbc in ((1, 0), (2, 0), (0, 1), (0, 2), (1, 1)):
        assert autotune.apply_cached_poisson(_Plan(ybc, xbc), *GRID, "fp64", path) is None
    keys = {autotune.poisson_key(*GRID, "fp64", y, x) for y in range(3) for x in range(3)}
    assert len(keys) == 9


def test_entries_of_another_table_of_shapes_are_not_taken(tmp_path, cache):
    path, entry = cache
    old = autotune.poisson_key(*GRID, "fp64").replace(f"|shapes{autotune.SHAPE_TABLE}", "")
    other = tmp_path / "old.json"
    other.write_text(json.dumps({old: entry}))
    plan = _Plan(0, 0)
    assert autotune.apply_cached_poisson(plan, *GRID, "fp64", str(other)) is None
    assert plan.set == {}


def test_the_key_names_the_table_of_shapes(monkeypatch):
    torch = pytest.importorskip("torch")
    props = type("P", (), {"gcnArchName": "gfx950", "name": "x"})()
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "get_device_properties", lambda d: props)
    first = autotune._arch_key()
    monkeypatch.setattr(autotune, "SHAPE_TABLE", autotune.SHAPE_TABLE + 1)
    assert autotune._arch_key() != first

"""Which kernel the tuner keeps, with the timing replaced (no GPU)."""
import json

import pytest

from paper_2405_00698_amd import tune as tuner

SLOT_PLAN, PAIRED = (768, 1983233), (768, 1)  # two equivalent kernels of a side


class Fake:
    """What tune() uses of a population: the default depends on whether there
    are more robots than CUs, as the library's does at 8^3."""
    dashpots = False
    device = None
    steps_per_launch = 0

    def __init__(self, sides):
        self.sides = sides
        self.chosen = {n: SLOT_PLAN if len(sides) <= 256 else PAIRED for n in sides}

    def persist_variant(self, n):
        return self.chosen[n]

    def set_persist_variant(self, n, block, variant):
        self.chosen[n] = (block, variant)

    def set_schedule(self, sides, lanes):
        pass

    def set_step_config(self, mode, block, steps_per_launch):
        pass

    def reset(self):
        pass

    def close(self):
        pass


@pytest.fixture
def timed(monkeypatch):
    calls = []

    def time_of(p, steps, reps=2):
        calls.append(len(p.sides))
        return 1.0  # equal: the default must win

    monkeypatch.setattr(tuner, "_time", time_of)
    monkeypatch.setattr(tuner, "_sub_population", lambda pop, n: Fake([m for m in pop.sides if m == n]))
    monkeypatch.setattr(tuner.api, "persist_configs", lambda n: [SLOT_PLAN, PAIRED])
    monkeypatch.setattr(tuner.torch.cuda, "get_device_name", lambda device=None: "gpu")
    return calls


def test_default_is_the_whole_populations(timed):
    """100 robots of 8^3 among 900 share their CUs: the kernel for a CU per
    robot, default of the 100 alone, is not favoured."""
    pop = Fake([8] * 100 + [5] * 800)
    tuner.tune(pop)
    assert pop.persist_variant(8) == PAIRED
    alone = Fake([8] * 100 + [5] * 20)
    tuner.tune(alone)
    assert alone.persist_variant(8) == SLOT_PLAN


def test_cached_choice_is_not_carried_between_the_two(timed, tmp_path):
    cache = str(tmp_path / "tuned.json")
    tuner.tune(Fake([8] * 100 + [5] * 20), cache_path=cache)
    before = len(timed)
    pop = Fake([8] * 100 + [5] * 800)
    tuner.tune(pop, cache_path=cache)
    assert pop.persist_variant(8) == PAIRED and len(timed) > before
    kept = json.load(open(cache))
    before = len(timed)
    again = Fake([8] * 100 + [5] * 800)
    tuner.tune(again, cache_path=cache)
    assert again.chosen == pop.chosen and len(timed) == before and json.load(open(cache)) == kept

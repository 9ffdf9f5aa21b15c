"""Cached launch shapes of small meshes, which the default shape may run as one launch of many half-steps."""
import types

import pytest

from paper_2104_04347_amd import autotune


class Small:
    """Stands in for binding.Solver: scripted times per shape, no GPU."""
    equation, P = "euler", 3

    class params:
        precision, limiter = 0, 1

    def __init__(self, N, times):
        self.N, self.times, self.shape = N, times, {"threads": 256, "blocks": 0, "variant": 1}
        self.set = 0

    def get_launch(self):
        return dict(self.shape)

    def set_launch(self, threads=0, blocks=0, variant=-1):
        self.shape = {"threads": threads or 256, "blocks": blocks,
                      "variant": self.shape["variant"] if variant < 0 else variant}
        self.set += 1

    def write(self, q0):
        pass

    def run(self, steps, cfl):
        self.steps = steps

    def last_run_ms(self):
        s = self.shape
        return self.times.get((s["variant"], s["threads"], s["blocks"]), 1.0) * self.steps


@pytest.fixture
def cache(tmp_path, monkeypatch):
    monkeypatch.setenv("WCC_AUTOTUNE_CACHE", str(tmp_path / "c.json"))
    fake = types.SimpleNamespace(cuda=types.SimpleNamespace(
        get_device_properties=lambda i: types.SimpleNamespace(multi_processor_count=256), synchronize=lambda: None))
    monkeypatch.setitem(__import__("sys").modules, "torch", fake)


def test_a_shape_tuned_beyond_the_one_launch_form_is_not_applied_within_it(cache):
    """Euler P = 3: 510 intervals (9 tiles) are a launch per half-step, 300 (5 tiles) one launch; both lie in 2^8."""
    big = Small(510, {(0, 256, 512): 0.5})
    best = autotune.tune_single(big, None, 0.25, steps=10, threads=(256,), block_factors=(0, 2), variants=(0, 1))
    assert (best["variant"], best["blocks"]) == (0, 512)
    assert autotune.apply_single(Small(510, {}))
    small = Small(300, {})
    assert not autotune.apply_single(small) and small.set == 0
    assert autotune.cached_single(small) is None


def test_keys_on_both_sides_of_the_largest_one_launch_mesh():
    key = lambda n: autotune.key_single("burgers", 1, n, "fp64", True)   # noqa: E731
    assert key(1008) != key(1007) and key(1009) == key(1023) and key(1024) == key(2047)


def test_the_one_launch_time_is_no_variant_s_time(cache):
    s = Small(300, {(1, 256, 0): 0.1, (1, 256, 512): 0.8, (0, 256, 0): 0.7})
    best = autotune.tune_single(s, None, 0.25, steps=10, threads=(256,), block_factors=(0, 2), variants=(0, 1))
    assert best["per_variant_ms"] == {0: 0.7, 1: 0.8}
    assert (best["variant"], best["threads"], best["blocks"]) == (1, 256, 0)   # and yet it is chosen
    assert s.get_launch() == {"threads": 256, "blocks": 0, "variant": 1}

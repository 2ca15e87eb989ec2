"""The autotuner's search on a stand-in context with made-up times: the
library's own choice is among what it tries, and stays in force when it wins."""
import types

import pytest

from paper_2407_19396_amd import autotune
from paper_2407_19396_amd import workloads as wl


class Context:
    """The launch settings of a context; blocks 0: the library's own."""

    obs_mode = reward_mode = 0

    def __init__(self, n):
        self.table, self.n = wl.uniform_table(n, wl.FAMILY_EMPTY, 8), n
        self.tile_envs, self.K, self.blocks = 64, 64, 0

    def set_tiling(self, tile_envs):
        self.tile_envs, self.blocks = tile_envs, 0

    def set_launch(self, K, blocks=0):
        self.K, self.blocks = K, blocks or self.blocks

    def info(self):
        n_tiles = -(-self.n // self.tile_envs)
        return {"n_tiles": n_tiles, "blocks": self.blocks or n_tiles, "lds_bytes": 6000 + 64 * self.tile_envs}


@pytest.fixture
def tune(monkeypatch):
    import torch
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: None)
    monkeypatch.setattr(torch.cuda, "get_device_properties",
                        lambda dev: types.SimpleNamespace(name="none", multi_processor_count=256))

    def run(n, ms, **kw):
        env = Context(n)
        monkeypatch.setattr(autotune, "_time_rollout",
                            lambda env, traj, steps, K, stream: steps * ms(env.tile_envs, env.blocks))
        best = autotune.tune(env, types.SimpleNamespace(rows=1024), use_cache=False, **kw)
        return env, best

    return run


@pytest.mark.parametrize("n,own", [(16, 4), (4096, 4), (4097, 8), (8192, 8), (8193, 16), (30000, 32), (262144, 64)])
def test_the_librarys_own_tiles_are_tried(tune, n, own):
    env, best = tune(n, lambda tile_envs, blocks: 1.0 if tile_envs == own else 2.0)
    assert env.tile_envs == best["tile_envs"] == own


def test_the_librarys_own_workgroups_stay_in_force(tune):
    env, best = tune(262144, lambda tile_envs, blocks: 2.0 if blocks else 1.0)
    assert best["blocks"] == env.blocks == 0 and env.K == best["K"]


def test_chosen_workgroups_and_tiles_still_win(tune):
    env, best = tune(262144, lambda tile_envs, blocks: 1.0 if (tile_envs, blocks) == (32, 4096) else 2.0)
    assert (env.tile_envs, env.blocks) == (best["tile_envs"], best["blocks"]) == (32, 4096)


def test_a_callers_tiles_alone_are_tried(tune):
    env, best = tune(16, lambda tile_envs, blocks: float(tile_envs), tile_envs=(32, 16))
    assert env.tile_envs == 16 and {r["tile_envs"] for r in best["trials"]} == {16, 32}

"""Which kernel, tiles and workgroups a call launches: the host runtime built
with recording stubs in place of HIP and the kernels (launch_recorder.cpp), so
that rules on batch size, grid sides and families are checked without a GPU."""
import ctypes
import os
import subprocess

import numpy as np
import pytest

from paper_2407_19396_amd import gridenv as ge
from paper_2407_19396_amd import workloads as wl

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2407_19396_amd", "csrc")
KINDS = ("plain", "fused", "reset")


class Launch(ctypes.Structure):
    _fields_ = [(f, ctypes.c_int32) for f in ("kind", "tile_envs", "n_tiles", "blocks", "max_cells", "steps",
                                              "balls", "corridors")]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("routes") / "recorder.so")
    src = [os.path.join(HERE, "launch_recorder.cpp")] + [os.path.join(CSRC, f) for f in (
        "runtime.cpp", "server.cpp", "static_rollout.cpp")]
    subprocess.run(["g++", "-std=c++17", "-O1", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__",
                    "-D__align__(n)=__attribute__((aligned(n)))", "-DHIP_SYMBOL(x)=x", "-I/opt/rocm/include",
                    "-I", CSRC, *src, "-o", out], check=True)
    return ctypes.CDLL(out)


class Batch:
    """A context of the recorded runtime; its calls return what they launched."""

    def __init__(self, lib, table, obs_mode=0):
        self.lib, self.n = lib, table.n
        self.keep = [np.ascontiguousarray(a) for a in (table.family, table.side, table.param, table.max_steps)]
        fam, side, par, ms = (a.ctypes.data for a in self.keep)
        self.cfg = ge.GxConfig(table.n, 0, obs_mode, fam, side, par, ms, None, 0, None, None)
        self.ctx = ctypes.c_void_p()
        assert lib.env_create(ctypes.byref(self.cfg), ctypes.byref(self.ctx)) == ge.GX_OK
        self.st = ge.GxState(*([16] * len(ge.STATE_FIELDS)))
        self.reset()

    def _took(self, rc):
        assert rc == ge.GX_OK
        buf = (Launch * 64)()
        n = self.lib.rec_take(buf, 64)
        return [{f: getattr(buf[i], f) for f, _ in Launch._fields_} | {"kind": KINDS[buf[i].kind]} for i in range(n)]

    def _out(self, obs, rows=1):
        return ctypes.byref(ge.GxTraj(16 if obs else None, 16, 16, 16, rows, None))

    def reset(self):
        return self._took(self.lib.env_reset(self.ctx, ctypes.byref(self.st), None, None))

    def step(self, obs=True):
        return self._took(self.lib.env_step(self.ctx, ctypes.byref(self.st), None, self._out(obs), None))

    def rollout(self, steps, K=0, obs=True, actions=None):
        return self._took(self.lib.env_rollout(self.ctx, ctypes.byref(self.st), steps, actions,
                                               self._out(obs, steps), K, None))

    def set_tiling(self, tile_envs):
        assert self.lib.env_set_tiling(self.ctx, tile_envs) == ge.GX_OK

    def set_launch(self, K, blocks=0):
        assert self.lib.env_set_launch(self.ctx, K, blocks) == ge.GX_OK

    def info(self):
        i = ge.GxInfo()
        assert self.lib.env_info(self.ctx, ctypes.byref(i)) == ge.GX_OK
        return i

    def close(self):
        assert self.lib.env_destroy(self.ctx) == ge.GX_OK


def some_balls(n, side, every, balls):
    t = wl.uniform_table(n, wl.FAMILY_EMPTY, side)
    t.family[::every] = wl.FAMILY_DYNOBS
    t.param[::every] = balls
    return t


@pytest.mark.parametrize("n,side,every,balls,obs,kind", [
    (262144, 31, 101, 4, True, "plain"), (262144, 16, 101, 4, True, "plain"), (65536, 19, 101, 4, True, "plain"),
    (262144, 8, 101, 4, False, "plain"), (4096, 31, 101, 4, False, "plain"), (16, 8, 101, 4, False, "plain"),
    (262144, 24, 1, 8, True, "plain"), (262144, 8, 1, 8, True, "fused"), (65536, 8, 1, 4, True, "fused"),
    (4096, 16, 101, 4, True, "fused"), (16, 8, 1, 2, True, "fused"), (262144, 8, 1, 8, False, "fused")])
def test_steps_with_moving_balls(lib, n, side, every, balls, obs, kind):
    """A few moving balls must not make a step read every grid of the batch."""
    b = Batch(lib, some_balls(n, side, every, balls))
    (step,) = b.step(obs)
    assert step["kind"] == kind and step["steps"] == 1
    assert kind == "fused" or step["balls"] == 1
    b.close()


@pytest.mark.parametrize("obs_mode", [0, 1, 2, 3])
def test_steps_without_balls(lib, obs_mode):
    b = Batch(lib, wl.mixed_table(5000), obs_mode)
    (step,) = b.step()
    assert step["kind"] == ("plain" if obs_mode < 2 else "fused") and step["balls"] == 0
    (step,) = b.step(obs=False)
    assert step["kind"] == "plain"
    b.close()


@pytest.mark.parametrize("obs_mode", [0, 2])
@pytest.mark.parametrize("tile_envs,launch", [(0, (64, 16)), (1, None), (64, None), (16, (128, 4096))])
def test_chosen_shapes_are_the_rollouts_alone(lib, tile_envs, launch, obs_mode):
    """Tiles and workgroups chosen for rollouts change neither steps nor resets."""
    b = Batch(lib, wl.uniform_table(65536, wl.FAMILY_DYNOBS, 8, param=4), obs_mode)
    step, reset, rollout = b.step(), b.reset(), b.rollout(4)
    assert step[0]["kind"] == "fused"
    if tile_envs:
        b.set_tiling(tile_envs)
    if launch:
        b.set_launch(*launch)
    assert b.step() == step and b.reset() == reset
    (chosen,) = b.rollout(4)
    if tile_envs not in (0, 64):
        assert chosen["tile_envs"] == tile_envs
    if launch:
        assert chosen["blocks"] == launch[1]
    assert rollout[0]["blocks"] == 1024
    b.close()


@pytest.mark.parametrize("n", [262144, 40000, 9000, 100])
@pytest.mark.parametrize("side", [4, 8, 16, 17, 24, 31, 32])
def test_one_pass_launches_of_large_grids(lib, n, side):
    """A reset or a whole-grid step reads or writes each grid once: its tiles
    hold at most 16 384 cells, and are not cut without need."""
    table = wl.uniform_table(n, wl.FAMILY_EMPTY, side)
    b = Batch(lib, table, 2)
    (step,), (reset,), (rollout,) = b.step(), b.reset(), b.rollout(2)
    assert reset["tile_envs"] <= 32
    for launch, most in ((step, 64), (reset, 32), (rollout, 64)):
        E = launch["tile_envs"]
        assert launch["n_tiles"] == launch["blocks"] == -(-n // E)
        assert launch["max_cells"] == min(E, n) * side * side
        if launch is not rollout:
            assert launch["max_cells"] <= 16384
            assert E == min(rollout["tile_envs"], most) or 2 * E * side * side > 16384
    b.close()


def test_static_rollout_runs_a_contexts_launches(lib):
    table = wl.uniform_table(70000, wl.FAMILY_TWOROOM, 31)
    b = Batch(lib, table)
    tr, n = b._out(True, 200), table.n
    rc = lib.env_rollout_static(ctypes.byref(b.cfg), ctypes.byref(b.st), 1, tr, 100, None, tr, 0, None)
    assert b._took(rc) == b.reset() + b.rollout(100)
    b.close()


def steps_and_blocks(launches):
    return [(r["steps"], r["blocks"]) for r in launches]


def test_long_rollouts_take_tiles_in_turn(lib):
    """Unless the caller has chosen otherwise, whatever way it leaves the choice
    to the library: no K, tiles of 64 set, or a K of its own."""
    b = Batch(lib, wl.mixed_table(262144))
    assert steps_and_blocks(b.rollout(256)) == [(256, 1024)]
    assert steps_and_blocks(b.rollout(2100)) == [(1024, 1024), (1024, 1024), (52, 4096)]
    assert steps_and_blocks(b.rollout(127)) == [(64, 4096), (63, 4096)]
    assert steps_and_blocks(b.rollout(256, K=128)) == [(128, 1024)] * 2
    assert steps_and_blocks(b.rollout(256, obs=False)) == [(64, 4096)] * 4
    assert steps_and_blocks(b.rollout(256, actions=16)) == [(64, 4096)] * 4
    assert steps_and_blocks(b.rollout(256, K=256, actions=16)) == [(256, 4096)]
    b.set_tiling(64)
    assert steps_and_blocks(b.rollout(256)) == [(256, 1024)]
    b.set_launch(64)
    assert steps_and_blocks(b.rollout(256)) == [(64, 4096)] * 4
    assert steps_and_blocks(b.rollout(256, K=200)) == [(200, 1024), (56, 4096)]
    b.set_launch(256, 4096)
    assert steps_and_blocks(b.rollout(256)) == [(256, 4096)]
    b.set_tiling(32)
    assert steps_and_blocks(b.rollout(256)) == [(256, 8192)]
    b.close()


@pytest.mark.parametrize("table,obs_mode", [(wl.mixed_table(90000), 0), (wl.mixed_table(65536), 0),
                                            (wl.lava_table(262144), 0), (wl.mixed_table(262144), 1)],
                         ids=["uneven turns", "one tile per SIMD", "frequent resets", "type ids"])
def test_other_rollouts_run_64_steps_a_launch(lib, table, obs_mode):
    b = Batch(lib, table, obs_mode)
    assert steps_and_blocks(b.rollout(256)) == [(64, -(-table.n // 64))] * 4
    b.close()


@pytest.mark.parametrize("table", [wl.mixed_table(122880), wl.mixed_table(90000), wl.lava_table(122880),
                                   wl.uniform_table(100, wl.FAMILY_KEYCORRIDOR, 7, param=1)],
                         ids=["in turn", "uneven turns", "lava", "corridors"])
@pytest.mark.parametrize("steps,K,actions", [(300, 0, None), (300, 200, None), (40, 0, None), (300, 0, 16)])
def test_static_rollout_follows_the_context(lib, table, steps, K, actions):
    b = Batch(lib, table)
    tr = b._out(True, steps)
    rc = lib.env_rollout_static(ctypes.byref(b.cfg), ctypes.byref(b.st), 1, tr, steps, actions, tr, K, None)
    assert b._took(rc) == b.reset() + b.rollout(steps, K, actions=actions)
    b.close()


@pytest.mark.parametrize("obs_mode", [0, 1, 2])
def test_lds_bytes_of_pairs(lib, obs_mode):
    """The reported LDS of a workgroup holds the second wave's share wherever the
    reported shape runs in pairs (the recorder's stub: one byte more)."""
    b = Batch(lib, wl.uniform_table(70000, wl.FAMILY_EMPTY, 8), obs_mode)
    cells = 64 * 64
    assert b.info().lds_bytes == cells                 # 1094 workgroups
    b.set_launch(128, 1024)
    assert b.info().lds_bytes == cells + (obs_mode < 2)
    b.set_tiling(32)
    assert b.info().lds_bytes == cells // 2
    b.close()
    b = Batch(lib, wl.uniform_table(65536, wl.FAMILY_EMPTY, 8), obs_mode)
    assert b.info().lds_bytes == cells + (obs_mode < 2)
    b.close()

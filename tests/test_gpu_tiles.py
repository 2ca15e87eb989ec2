"""Launch shapes and lengths that small tables do not reach by themselves."""
import numpy as np
import pytest

import oracle as ox
import parity as P
from paper_2407_19396_amd import workloads as wl

pytestmark = pytest.mark.gpu


def check_rollout(table, steps, K, obs_mode=0, tile_envs=0, actions=None, what=""):
    import torch
    from paper_2407_19396_amd import gridenv as ge
    b, s, first = P.oracle_reset(table, 0, obs_mode)
    env = ge.GridEnv(table, obs_mode=obs_mode)
    if tile_envs:
        env.set_tiling(tile_envs)
    row = env.traj(1)
    env.reset(row)
    P.assert_rows_equal(row, first, what=f"{what}: first timestep")
    ref = ox.rollout(b, s, steps, actions, nthreads=8)
    traj = env.traj(steps)
    env.rollout(steps, traj, None if actions is None else torch.from_numpy(actions).cuda(), K=K)
    torch.cuda.synchronize()
    P.assert_rows_equal(traj, ref, what=what)
    P.assert_state_equal(env, s, what)
    env.close()


@pytest.mark.parametrize("obs_mode", [0, 2, 3])
@pytest.mark.parametrize("K", [2, 15, 16, 17, 40])
def test_corridors_drawn_ahead_or_not(K, obs_mode):
    """KeyCorridor layouts are drawn for the lanes that reset until 16 steps are
    left, then ahead; other families in the same waves from 2 on."""
    n = 700
    rng = np.random.default_rng(K)
    table = wl.keycorridor_table(n, seed=K)
    other = rng.random(n) < 0.3
    table.family[other], table.side[other], table.param[other] = wl.FAMILY_CROSSINGS, 9, 2
    table.max_steps[:] = rng.integers(1, 25, n)
    check_rollout(table, 40, K, obs_mode, what=f"corridors, K = {K}, mode {obs_mode}")

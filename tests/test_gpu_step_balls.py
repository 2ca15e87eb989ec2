"""One-step calls of batches with Dynamic-Obstacles envs that move their balls
in HBM (step_in_hbm): large grids, few balls, or no records."""
import numpy as np
import pytest

import oracle as ox
import parity as P
from paper_2407_19396_amd import workloads as wl

pytestmark = pytest.mark.gpu


def table_of(n, side, share):
    """share of the envs Dynamic-Obstacles with 1 to 8 balls, the others of
    every family that `side` allows; short episodes."""
    rng = np.random.default_rng(n + side)
    fam = rng.choice([wl.FAMILY_EMPTY, wl.FAMILY_TWOROOM, wl.FAMILY_LAVAGAP, wl.FAMILY_GOTODOOR], n)
    fam = np.where(rng.random(n) < share, wl.FAMILY_DYNOBS, fam).astype(np.uint8)
    par = np.where(fam == wl.FAMILY_DYNOBS, rng.integers(1, 9 if side > 5 else 8, n), 0).astype(np.uint8)
    return wl.EnvTable(fam, np.full(n, side, np.uint8), rng.integers(4, 40, n).astype(np.int32),
                       np.full(n, 5 + n, np.uint64), np.arange(n, dtype=np.uint32), "balls", par)


def run(table, obs_mode, steps, with_obs, spoil=0):
    import torch
    from paper_2407_19396_amd import gridenv as ge
    acts = np.random.default_rng(table.n).choice(np.array([0, 1, 2, 2, 2, 3, 5, 6, 200], np.uint8), (steps, table.n))
    b, s, _ = P.oracle_reset(table, 0, obs_mode)
    env = ge.GridEnv(table, obs_mode=obs_mode)
    env.reset()
    if spoil:   # list entries off the interior do not move
        rng = np.random.default_rng(spoil)
        obst = s.obst.reshape(table.n, 16)
        for i in np.flatnonzero((table.family == wl.FAMILY_DYNOBS) & (rng.random(table.n) < 0.5)):
            obst[i, 2 * rng.integers(0, table.param[i]) + rng.integers(0, 2)] = rng.choice([0, table.side[i] - 1, 200])
        env.obst.copy_(torch.from_numpy(s.obst.reshape(-1).copy()).cuda())
    ref = ox.rollout(b, s, steps, acts, nthreads=8)
    traj = env.traj(steps, with_obs=with_obs)
    dacts = torch.from_numpy(acts).cuda()
    for k in range(steps):
        env.step(traj.row(k), dacts[k])
    torch.cuda.synchronize()
    P.assert_rows_equal(traj, ref, what=f"{table.n} envs of side {table.side[0]}")
    P.assert_state_equal(env, s, f"{table.n} envs of side {table.side[0]}")
    env.close()


@pytest.mark.parametrize("n,side,spoil", [(1, 32, 0), (3, 32, 0), (64, 32, 1), (65, 19, 2), (300, 32, 3), (17, 9, 0)])
def test_balls_without_records(n, side, spoil):
    run(table_of(n, side, 0.1 if side == 9 else 0.6), 0, 50, False, spoil)


@pytest.mark.parametrize("obs_mode", [0, 1])
@pytest.mark.parametrize("n,side,share,steps", [(4099, 32, 0.5, 24), (16390, 31, 0.2, 10), (65601, 12, 0.05, 10)])
def test_balls_with_records(n, side, share, steps, obs_mode):
    run(table_of(n, side, share), obs_mode, steps, True)

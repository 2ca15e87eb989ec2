"""The fused kernel's records from cell codes: every cut of the last group of
four cells, passes that start at any byte of the output, and nothing written
outside the rows."""
import numpy as np
import pytest

import oracle as ox
import parity as P
from paper_2407_19396_amd import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("obs_mode", [0, 1, 2, 3])
@pytest.mark.parametrize("n,offset", [(1, 0), (1, 1), (2, 3), (3, 16), (5, 4), (6, 63), (13, 2), (21, 64), (22, 37),
                                      (63, 1), (64, 0), (65, 48), (130, 5)])
def test_records_at_any_alignment(n, offset, obs_mode):
    import torch
    from paper_2407_19396_amd import gridenv as ge
    table = wl.families_table(n, seed=n, mix_seed=n + offset)
    steps = 9
    b, s, _ = P.oracle_reset(table, 0, obs_mode)
    ref = ox.rollout(b, s, steps, None)
    env = ge.GridEnv(table, obs_mode=obs_mode)
    env.reset()
    traj = env.traj(steps)
    whole = traj.obs
    guard = 256
    raw = torch.full((whole.numel() + 2 * guard,), 0xA5, dtype=torch.uint8, device="cuda")
    at = guard + offset - raw.data_ptr() % 64
    traj.obs = raw[at:at + whole.numel()].view(whole.shape)
    env.rollout(steps, traj, K=4)
    torch.cuda.synchronize()
    P.assert_rows_equal(traj, ref, what=f"{n} envs at byte {offset}, mode {obs_mode}")
    P.assert_state_equal(env, s, f"{n} envs at byte {offset}, mode {obs_mode}")
    assert bool((raw[:at] == 0xA5).all()) and bool((raw[at + whole.numel():] == 0xA5).all())
    env.close()

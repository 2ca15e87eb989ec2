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


# families at their smallest, odd, even and largest sides, with every parameter
RESET_CASES = ([(wl.FAMILY_EMPTY, s, 0) for s in (4, 5, 32)] + [(wl.FAMILY_TWOROOM, s, 0) for s in (5, 8, 32)] +
               [(wl.FAMILY_FOURROOMS, s, 0) for s in (7, 9, 31)] + [(wl.FAMILY_LAVAGAP, s, 0) for s in (5, 6, 32)] +
               [(wl.FAMILY_CROSSINGS, 5, 1), (wl.FAMILY_CROSSINGS, 9, 3), (wl.FAMILY_CROSSINGS, 31, 8)] +
               [(wl.FAMILY_DISTSHIFT, 6, 1), (wl.FAMILY_DISTSHIFT, 9, 2), (wl.FAMILY_DISTSHIFT, 32, 1)] +
               [(wl.FAMILY_DYNOBS, 5, 1), (wl.FAMILY_DYNOBS, 5, 7), (wl.FAMILY_DYNOBS, 32, 8)] +
               [(wl.FAMILY_GOTODOOR, s, 0) for s in (5, 11, 32)] +
               [(wl.FAMILY_KEYCORRIDOR, 7, 1), (wl.FAMILY_KEYCORRIDOR, 10, 2), (wl.FAMILY_KEYCORRIDOR, 31, 3)])


@pytest.mark.parametrize("case", [[c] for c in RESET_CASES] + [RESET_CASES],
                         ids=[f"{wl.FAMILY_NAMES[f]}-{s}-{p}" for f, s, p in RESET_CASES] + ["all"])
def test_resets_all_the_time(case):
    """Step limits of 1 to 3, so that layouts are drawn and filled on most
    steps, some lanes of a tile resetting while others do not."""
    import torch
    from paper_2407_19396_amd import gridenv as ge
    n, steps = 330, 24
    rng = np.random.default_rng(len(case))
    pick = np.array(case)[rng.integers(0, len(case), n)]
    table = wl.EnvTable(pick[:, 0].astype(np.uint8), pick[:, 1].astype(np.uint8),
                        rng.integers(1, 4, n).astype(np.int32), np.full(n, 99, np.uint64),
                        np.arange(n, dtype=np.uint32), "resets", pick[:, 2].astype(np.uint8))
    b, s, _ = P.oracle_reset(table, 0, 2)
    ref = ox.rollout(b, s, steps, None, nthreads=8)
    env = ge.GridEnv(table, obs_mode=2)
    env.reset()
    traj = env.traj(steps)
    env.rollout(steps, traj, K=11)
    torch.cuda.synchronize()
    P.assert_rows_equal(traj, ref, what="resets")
    P.assert_state_equal(env, s, "resets")
    env.close()


@pytest.mark.parametrize("obs_mode", [0, 1])
@pytest.mark.parametrize("n,offset", [(1, 0), (2, 3), (3, 16), (5, 33), (17, 2), (66, 1), (300, 48)])
def test_steps_at_any_alignment(n, offset, obs_mode):
    """The plain kernel: the first and the last grid of the buffer in every
    batch, resets on many steps, doors toggled often."""
    import torch
    from paper_2407_19396_amd import gridenv as ge
    table = wl.families_table(4 * n + 40, seed=n, mix_seed=3 * n + offset)
    table = table.subset(np.flatnonzero(table.family != wl.FAMILY_DYNOBS)[:n])
    table.max_steps[:] = np.random.default_rng(n).integers(2, 30, n)
    steps = 40
    acts = np.random.default_rng(n + 1).choice(np.array([0, 1, 2, 2, 2, 3, 4, 5, 5, 6, 200], np.uint8), (steps, n))
    b, s, _ = P.oracle_reset(table, 0, obs_mode)
    ref = ox.rollout(b, s, steps, acts)
    env = ge.GridEnv(table, obs_mode=obs_mode)
    env.reset()
    traj = env.traj(steps)
    raw = torch.full((traj.obs.numel() + 256,), 0xA5, dtype=torch.uint8, device="cuda")
    at = 64 + offset - raw.data_ptr() % 64
    shape, size = traj.obs.shape, traj.obs.numel()
    traj.obs = raw[at:at + size].view(shape)
    dacts = torch.from_numpy(acts).cuda()
    for k in range(steps):
        env.step(traj.row(k), dacts[k])
    torch.cuda.synchronize()
    P.assert_rows_equal(traj, ref, what=f"{n} envs at byte {offset}, mode {obs_mode}")
    P.assert_state_equal(env, s, f"{n} envs at byte {offset}, mode {obs_mode}")
    assert bool((raw[:at] == 0xA5).all()) and bool((raw[at + size:] == 0xA5).all())
    env.close()


@pytest.mark.parametrize("obs_mode", [0, 1])
@pytest.mark.parametrize("tile_envs,blocks", [(1, 1025), (1, 1024), (8, 40), (64, 17), (64, 3), (0, 0)])
def test_waves_alone_and_in_pairs(tile_envs, blocks, obs_mode):
    """More workgroups than run in pairs of waves, as many, and pairs that
    take several tiles one after another; resets and toggles on most steps."""
    import torch
    from paper_2407_19396_amd import gridenv as ge
    n, steps = 1025, 14
    table = wl.families_table(n, seed=3, mix_seed=8)
    table.max_steps[:] = np.random.default_rng(5).integers(1, 12, n)
    acts = np.random.default_rng(6).choice(np.array([0, 1, 2, 2, 3, 4, 5, 5, 6], np.uint8), (steps, n))
    for actions in (None, acts):
        b, s, _ = P.oracle_reset(table, 0, obs_mode)
        ref = ox.rollout(b, s, steps, actions, nthreads=8)
        env = ge.GridEnv(table, obs_mode=obs_mode)
        if tile_envs:
            env.set_tiling(tile_envs)
            env.set_launch(6, blocks)
        env.reset()
        traj = env.traj(steps)
        env.rollout(steps, traj, None if actions is None else torch.from_numpy(actions).cuda(), K=6)
        torch.cuda.synchronize()
        P.assert_rows_equal(traj, ref, what=f"{blocks} workgroups, mode {obs_mode}")
        P.assert_state_equal(env, s, f"{blocks} workgroups, mode {obs_mode}")
        env.close()


@pytest.mark.parametrize("n", [32769, 40000])
def test_reset_in_halves_of_a_launch_tile(n):
    """From 32 769 envs on resets run tiles of 32 and steps tiles of 64, ragged
    at both."""
    import torch
    from paper_2407_19396_amd import gridenv as ge
    table = wl.families_table(n, seed=4)
    b, s, first = P.oracle_reset(table, 0, 0)
    env = ge.GridEnv(table)
    row = env.traj(1)
    env.reset(row)
    P.assert_rows_equal(row, first, what=f"{n} envs, first timestep")
    ref = ox.rollout(b, s, 3, None, nthreads=8)
    traj = env.traj(3)
    env.rollout(3, traj)
    torch.cuda.synchronize()
    P.assert_rows_equal(traj, ref, what=f"{n} envs")
    P.assert_state_equal(env, s, f"{n} envs")
    env.close()


def test_current_stream_of_a_call():
    import torch
    from paper_2407_19396_amd import gridenv as ge
    torch.zeros(1, device="cuda")
    side = torch.cuda.Stream()
    assert ge._stream_ptr(None) is None and ge._stream_ptr(side) == side.cuda_stream
    with torch.cuda.stream(side):
        assert ge._stream_ptr(None) == side.cuda_stream
        assert ge._stream_ptr(torch.cuda.default_stream()) is None
    assert ge._stream_ptr(None) is None


@pytest.mark.parametrize("n,steps", [(61440 + 4, 128), (122880, 128), (122816, 128), (131072 + 1, 129)])
def test_long_rollouts_of_many_tiles(n, steps):
    """Batches at and beside the tile counts whose long launches take the tiles
    in turn; the ring keeps the last rows."""
    import torch
    from paper_2407_19396_amd import gridenv as ge
    table = wl.mixed_table(n, seed=9)
    b, s, _ = P.oracle_reset(table, 0, 0)
    ref = ox.rollout(b, s, steps, None, rows=3, nthreads=8)
    env = ge.GridEnv(table)
    env.reset()
    traj = env.traj(3)
    env.rollout(steps, traj, K=steps)
    torch.cuda.synchronize()
    P.assert_rows_equal(traj, ref, what=f"{n} envs")
    P.assert_state_equal(env, s, f"{n} envs")
    env.close()


@pytest.mark.parametrize("obs_mode", [0, 1, 2])
@pytest.mark.parametrize("n,together", [(7, 7), (64, 64), (320, 9), (320, 8), (3000, 40)])
def test_corridors_connected_by_few_lanes(n, together, obs_mode):
    """Waves with few, exactly eight, nine and only KeyCorridor envs: layouts
    whose last doors the wave looks for together."""
    import torch
    from paper_2407_19396_amd import gridenv as ge
    rng = np.random.default_rng(n + together)
    corridor = np.arange(n) % 64 < together
    side = np.where(corridor, rng.choice([7, 10, 13, 16, 19], n), 5).astype(np.uint8)
    table = wl.EnvTable(np.where(corridor, wl.FAMILY_KEYCORRIDOR, wl.FAMILY_EMPTY).astype(np.uint8), side,
                        rng.integers(1, 6, n).astype(np.int32), np.full(n, 77 + n, np.uint64),
                        np.arange(n, dtype=np.uint32), "corridors",
                        np.where(corridor, rng.integers(1, 4, n), 0).astype(np.uint8))
    steps = 30
    b, s, first = P.oracle_reset(table, 0, obs_mode)
    env = ge.GridEnv(table, obs_mode=obs_mode)
    env.set_tiling(64)
    row = env.traj(1)
    env.reset(row)
    P.assert_rows_equal(row, first, what="first timestep")
    ref = ox.rollout(b, s, steps, None, nthreads=8)
    traj = env.traj(steps)
    env.rollout(steps, traj, K=13)
    torch.cuda.synchronize()
    P.assert_rows_equal(traj, ref, what="corridors")
    P.assert_state_equal(env, s, "corridors")
    env.close()

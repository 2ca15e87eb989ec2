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


def busy_table(n, corridors, seed):
    """Every family at small sides (KeyCorridor or not), episodes of 1 to 11
    steps: layouts drawn and filled, balls moved and doors toggled on most steps."""
    table = wl.families_table(2 * n, seed=seed, mix_seed=seed + 1)
    table = table.subset(np.flatnonzero((table.family == wl.FAMILY_KEYCORRIDOR) <= corridors)[:n])
    table.rng_id[:] = np.arange(n)
    table.max_steps[:] = np.random.default_rng(seed).integers(1, 12, n)
    return table


@pytest.mark.parametrize("obs_mode", [0, 1])
@pytest.mark.parametrize("n,corridors,with_actions", [(65600, False, False), (65600, True, False),
                                                      (65600, False, True), (65600, True, True),
                                                      (65601, False, False), (65599, True, True)])
def test_full_tiles_of_single_waves(n, corridors, with_actions, obs_mode):
    """More than 1024 tiles of 64 envs: one wave takes the steps and writes the
    records, its stage holding layout words, views and the write-back's bitmap
    in turn; rows on 64-byte boundaries (65 600 envs) and off them."""
    table = busy_table(n, corridors, seed=n + corridors)
    steps = 17
    acts = None
    if with_actions:
        acts = np.random.default_rng(n).choice(np.array([0, 1, 2, 2, 2, 3, 4, 5, 5, 6, 99], np.uint8), (steps, n))
    check_rollout(table, steps, 9, obs_mode, actions=acts, what=f"{n} envs, mode {obs_mode}")


@pytest.mark.parametrize("offset", [0, 16, 64, 128, 147])
def test_single_waves_at_any_alignment(offset):
    import torch
    from paper_2407_19396_amd import gridenv as ge
    n, steps = 65600, 5
    table = wl.mixed_table(n, seed=offset)
    b, s, _ = P.oracle_reset(table)
    ref = ox.rollout(b, s, steps, None, nthreads=8)
    env = ge.GridEnv(table)
    env.reset()
    traj = env.traj(steps)
    shape, size = traj.obs.shape, traj.obs.numel()
    raw = torch.full((size + 1024,), 0xA5, dtype=torch.uint8, device="cuda")
    at = 256 + offset - raw.data_ptr() % 128
    traj.obs = raw[at:at + size].view(shape)
    env.rollout(steps, traj)
    torch.cuda.synchronize()
    P.assert_rows_equal(traj, ref, what=f"records at byte {offset}")
    P.assert_state_equal(env, s, f"records at byte {offset}")
    assert bool((raw[:at] == 0xA5).all()) and bool((raw[at + size:] == 0xA5).all())
    env.close()


@pytest.mark.parametrize("n,steps", [(61440 + 64, 200), (122880, 1030), (122880 - 64, 130)])
def test_default_calls_of_long_rollouts(n, steps):
    """No K and no shape: one launch of up to 1024 steps, tiles in turn, and what
    is left in another; through both entry points."""
    import torch
    import test_zz_no_alloc as static
    table = wl.mixed_table(n, seed=6)
    env, bufs = static.run_pair(table, steps, 3, 0)
    b, s, _ = P.oracle_reset(table)
    ref = ox.rollout(b, s, steps, None, rows=3, nthreads=8)
    P.assert_rows_equal(bufs.traj, ref, what=f"{n} envs")
    P.assert_state_equal(env, s, f"{n} envs")
    env.close()
    torch.cuda.empty_cache()


def test_long_rollouts_beside_other_kernels():
    """Pairs that take tiles in turn count their renderers per SIMD: two such
    launches on two streams at once, with other kernels before and between."""
    import torch
    from paper_2407_19396_amd import gridenv as ge
    n, steps = 122880, 128
    other = torch.zeros(1 << 26, dtype=torch.uint8, device="cuda")
    streams = [torch.cuda.Stream(), torch.cuda.Stream()]
    runs = []
    for k, stream in enumerate(streams):
        table = wl.mixed_table(n, seed=20 + k)
        env = ge.GridEnv(table)
        env.reset()
        runs.append((table, env, env.traj(3), stream))
    torch.cuda.synchronize()
    for _ in range(3):
        for _, env, traj, stream in runs:
            with torch.cuda.stream(stream):
                other.add_(1)
                env.rollout(steps, traj, K=steps)
    torch.cuda.synchronize()
    for table, env, traj, _ in runs:
        b, s, _ = P.oracle_reset(table)
        for _ in range(3):
            ref = ox.rollout(b, s, steps, None, rows=3, nthreads=8)
        P.assert_rows_equal(traj, ref, what="beside other kernels")
        P.assert_state_equal(env, s, "beside other kernels")
        env.close()


def largest_table(n_odd=64):
    """64 envs of side 32 (the most cells a tile can hold), 64 of side 31 of the
    families that need an odd side, 5 more of side 32; short episodes."""
    big = ([(wl.FAMILY_EMPTY, 32, 0), (wl.FAMILY_TWOROOM, 32, 0), (wl.FAMILY_LAVAGAP, 32, 0),
            (wl.FAMILY_DISTSHIFT, 32, 1), (wl.FAMILY_GOTODOOR, 32, 0)] +
           [(wl.FAMILY_DYNOBS, 32, k) for k in range(1, 9)])
    odd = ([(wl.FAMILY_FOURROOMS, 31, 0)] + [(wl.FAMILY_CROSSINGS, 31, k) for k in range(1, 9)] +
           [(wl.FAMILY_KEYCORRIDOR, 31, r) for r in (1, 2, 3)])
    tasks = [big[i % len(big)] for i in range(64)] + [odd[i % len(odd)] for i in range(n_odd)] + big[:5]
    fam, side, par = (np.array(c, np.uint8) for c in zip(*tasks))
    n = len(tasks)
    return wl.EnvTable(fam, side, np.random.default_rng(n).integers(3, 40, n).astype(np.int32),
                       np.full(n, 61, np.uint64), np.arange(n, dtype=np.uint32), "largest tiles", par)


@pytest.mark.parametrize("obs_mode", [0, 1, 2, 3])
@pytest.mark.parametrize("tile_envs", [64, 0])
def test_largest_tiles_as_launched(tile_envs, obs_mode):
    """64 grids of side 32 in one workgroup: 64 KB of codes and a table of blocks
    to write back that spans them, in pairs of waves and alone (whole grids);
    beside it the tiles the library chooses."""
    table = largest_table()
    assert int((table.side[:64].astype(int) ** 2).sum()) == 65536
    check_rollout(table, 45, 16, obs_mode, tile_envs, what=f"largest tiles of {tile_envs or 'any'}, mode {obs_mode}")


@pytest.mark.parametrize("obs_mode", [0, 2])
def test_largest_reset_and_step_tiles(obs_mode):
    """Resets and one-step launches of a large batch of the largest grids, in the
    tiles that 16 384 cells allow them (16 grids of side 32)."""
    import torch
    from paper_2407_19396_amd import gridenv as ge
    n = 16400
    some = largest_table(0).subset(np.arange(64))
    table = some.subset(np.arange(n) % 64)
    table.rng_id[:] = np.arange(n)
    table.max_steps[:] = 2
    b, s, first = P.oracle_reset(table, 0, obs_mode)
    env = ge.GridEnv(table, obs_mode=obs_mode)
    row = env.traj(1)
    env.reset(row)
    P.assert_rows_equal(row, first, what="first timestep")
    ref = ox.rollout(b, s, 4, None, nthreads=8)
    traj = env.traj(4)
    for k in range(4):
        env.step(traj.row(k))
    torch.cuda.synchronize()
    P.assert_rows_equal(traj, ref, what=f"{n} envs of side 32, mode {obs_mode}")
    P.assert_state_equal(env, s, f"{n} envs of side 32, mode {obs_mode}")
    env.close()


def test_serving_in_whole_tiles():
    """More than 1024 live tiles, most of them full: launches whose tiles run
    whole, in single waves; a second wave of requests is admitted between
    launches, so that fresh and running tiles share one, and every family with
    layouts that reset, draw or move balls is among them."""
    import torch
    from paper_2407_19396_amd import gridenv as ge
    steps, K = 24, 9
    sizes = [30000, 20001, 15000, 700, 64, 1, 4000]
    srv = ge.Server(sum(-(-n // 64) for n in sizes), 32)
    reqs, live = [], {}

    def admit(k):
        table = busy_table(sizes[k], corridors=True, seed=40 + k)
        table.seed[:] = 40 + k
        stride = ge.padded_stride(table.n)
        out = ge.Traj.alloc(steps, stride)
        live[srv.admit(table, steps, out, stride)] = len(reqs)
        reqs.append((table, out))

    for k in range(5):
        admit(k)
    fin = srv.step(K)
    assert not fin
    admit(5)
    admit(6)
    while live:
        for h in srv.step(K):
            torch.cuda.synchronize()
            srv.release(h)
            live.pop(h)
    torch.cuda.synchronize()
    srv.close()
    for table, out in reqs:
        b, s, _ = P.oracle_reset(table)
        ref = ox.rollout(b, s, steps, None, nthreads=8)
        n = table.n
        P.assert_rows_equal(ge.Traj(out.obs[:, :n], out.reward[:, :n], out.flags[:, :n], out.action[:, :n]), ref,
                            what=f"request of {n} envs")

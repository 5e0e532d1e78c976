"""Small batches are stepped by teams of wavefronts.  At the sizes where the number of boards per team changes, and in the last
team of a batch, their outputs and state are those of the kernel in which one wavefront does everything (set_boards_per_wavefront asks
for it), through skipped, illegal and passed plies, captures, endings and restarts in one team."""
import numpy as np
import pytest
import torch

import bench
import paper_2303_17503_amd as pg
import workloads
from gpu_common import Pair

pytestmark = pytest.mark.gpu


def bound(env, obs):
    B = env.B
    out = [env.new_mask(), env.new_obs() if obs else None, torch.zeros((B, 2), dtype=torch.float32, device="cuda"), torch.zeros(B, dtype=torch.uint8, device="cuda")]
    env.bind_outputs(*out)
    return [t for t in out if t is not None]


@pytest.mark.parametrize("N,B,obs,steps,slices,team", [   # on both sides of every line; steps = 0: a step call
    (9, 256, True, 0, 1, (1, 4)), (9, 384, True, 0, 1, (1, 4)), (9, 385, False, 0, 1, (2, 4)), (9, 4096, True, 0, 1, (4, 4)), (9, 4097, True, 0, 1, (0, 1)),
    (19, 512, True, 0, 1, (1, 4)), (19, 6144, True, 0, 1, (3, 4)), (19, 6145, True, 0, 1, (0, 1)), (19, 4098, False, 0, 1, (3, 4)), (19, 4099, False, 0, 1, (0, 1)),
    (9, 5001, True, 1, 1, (0, 1)), (9, 5001, False, 64, 64, (6, 2)), (9, 12288, True, 2, 1, (6, 3)), (9, 12289, True, 2, 1, (0, 1)), (9, 13312, True, 3, 1, (6, 3)),
    (9, 15360, True, 7, 1, (6, 3)), (9, 15361, True, 7, 1, (0, 1)), (9, 16384, True, 8, 1, (6, 3)), (9, 16385, True, 64, 1, (0, 1)), (9, 18432, True, 9, 1, (0, 1)),
    (9, 18433, True, 9, 1, (6, 3)), (9, 18433, True, 5, 1, (0, 1)), (9, 20480, True, 6, 1, (6, 3)), (9, 20481, True, 9, 1, (0, 1)),
    (9, 8192, False, 2, 1, (6, 2)), (9, 8193, False, 2, 1, (0, 1)), (9, 13313, False, 3, 1, (0, 1)), (9, 20480, False, 4, 1, (6, 2)), (9, 20481, False, 4, 1, (0, 1)),
    (19, 1024, False, 2, 1, (1, 2)), (19, 3072, False, 2, 1, (3, 2)), (19, 3073, False, 2, 1, (0, 1)), (19, 4097, False, 3, 1, (0, 1)), (19, 7168, False, 4, 1, (3, 2)),
    (19, 7169, False, 15, 1, (0, 1)), (19, 10752, False, 16, 1, (3, 2)), (19, 10753, False, 99, 1, (0, 1)),
    (19, 26624, True, 2, 1, (3, 3)), (19, 26625, True, 2, 1, (0, 1)), (19, 30720, True, 4, 1, (3, 3)), (19, 30721, True, 15, 1, (0, 1)), (19, 30721, True, 16, 1, (3, 3)),
    (19, 22528, True, 3, 2, (3, 3)), (19, 22529, True, 6, 2, (0, 1)), (19, 22529, True, 7, 2, (3, 3)), (19, 16384, True, 16, 1, (3, 3)), (19, 16384, True, 16, 16, (0, 1))])
def test_which_calls_go_by_teams(N, B, obs, steps, slices, team):
    env = pg.GoEnv(B, N)
    assert env.boards_per_team(steps, slices, obs=obs) == team
    env.set_boards_per_wavefront(2)
    assert env.boards_per_team(steps, slices, obs=obs) == (0, 1)
    env.set_boards_per_wavefront(0)
    assert env.boards_per_team(steps, slices, obs=obs) == team
    assert pg.GoEnv(B, N, mask_pitch=N * N + 2).boards_per_team(steps, slices, obs=obs) == (0, 1)


@pytest.mark.parametrize("config", [0, 2, 3])
def test_the_benchmark_compares_a_ply_with_one_group_of_the_same_kernel(config):
    cfg = workloads.CONFIGS[config]
    env = pg.GoEnv(cfg.batch, cfg.board_size)
    one = bench.one_group(cfg, env, True)
    kernel, waves = bench.go_kernel(env, cfg.batch, True)
    assert kernel.startswith("go_step_team_kernel" if config < 3 else "go_step_kernel")
    assert bench.go_kernel(one.env, one.B, True)[0] == kernel
    assert waves == {0: 256 * 4 / 1024, 2: 342 * 4 / 1024, 3: 5462 / 1024}[config]


@pytest.mark.parametrize("N,B,auto_reset,obs,line_padded", [
    (9, 1, True, True, False), (9, 384, True, True, False), (9, 385, False, True, True), (9, 1025, True, True, False), (9, 4095, True, False, False),
    (19, 1, True, True, True), (19, 512, True, True, False), (19, 513, False, True, False), (19, 4097, True, False, False), (19, 6143, True, True, False)])
def test_teams_and_single_wavefronts_agree(N, B, auto_reset, obs, line_padded):
    kw = dict(seed=9, auto_reset=auto_reset, line_padded=line_padded, max_steps=60 if auto_reset else 0)
    a, b = pg.GoEnv(B, N, **kw), pg.GoEnv(B, N, **kw)
    b.set_boards_per_wavefront(2)
    for e in (a, b):
        e.rollout(40 if auto_reset else 150, 9, 0)
    oa, ob = bound(a, obs), bound(b, obs)
    rng = np.random.default_rng(B)
    nxt = a.random_actions(9, 500)
    for t in range(24):
        odd = torch.as_tensor(rng.choice([-1, 0, N * N, N * N + 5], size=B).astype(np.int32), device="cuda")   # skip, a corner, pass, out of range
        use = torch.as_tensor(rng.random(B) < (0.1 if t % 2 else 0.0), device="cuda")                          # every other ply all boards play
        act = torch.where(use, odd, nxt).contiguous()
        if t % 3 == 0:
            a.step(act); b.step(act)
            nxt, nb = a.random_actions(9, 501 + t), b.random_actions(9, 501 + t)
        else:
            nxt, nb = a.step_sample(act, 9, 501 + t), b.step_sample(act, 9, 501 + t)
        assert torch.equal(nxt, nb), t
        for x, y in zip(oa, ob):
            assert torch.equal(x, y), t
    sa, sb = a.export_state(), b.export_state()
    for k in sa:
        assert torch.equal(sa[k], sb[k]), k


@pytest.mark.parametrize("N,B,steps,slices,obs,auto_reset", [
    (9, 1, 5, 1, True, True), (9, 385, 9, 4, True, True), (9, 1023, 2, 2, False, False), (9, 20480, 6, 3, True, True), (9, 4097, 11, 11, False, True),
    (19, 1, 4, 1, False, True), (19, 511, 7, 7, True, False), (19, 1025, 5, 2, False, True), (19, 9001, 3, 1, True, True), (19, 11000, 2, 1, False, True)])
def test_rollouts_by_teams_and_by_single_wavefronts_agree(N, B, steps, slices, obs, auto_reset):
    kw = dict(seed=4, auto_reset=auto_reset, max_steps=45 if auto_reset else 0)
    envs = [pg.GoEnv(B, N, **kw), pg.GoEnv(B, N, **kw)]
    envs[1].set_boards_per_wavefront(3)
    start = torch.as_tensor(np.random.default_rng(B).integers(0, 44, size=B).astype(np.int32), device="cuda")   # some wait through a whole launch
    got = []
    for e in envs:
        assert not e.rollout_in_time_slots(steps, slices, True, obs)[0]
        m, o = torch.full((slices, B, e.mask_pitch), 7, dtype=torch.uint8, device="cuda"), torch.full((slices, B, e.obs_pitch), 7, dtype=torch.uint8, device="cuda")
        r, t = torch.full((slices, B, 2), 7.0, dtype=torch.float32, device="cuda"), torch.full((slices, B), 7, dtype=torch.uint8, device="cuda")
        a = torch.full((slices, B), 7, dtype=torch.int32, device="cuda")
        seen = []
        for k in range(4):
            e.rollout(steps, 4, 36 + k * steps, start_t=start, slices=slices, actions=a, rewards=r, terminated=t, mask=m, obs=o if obs else None)
            seen += [x.clone() for x in (m, o, r, t, a)]
        seen += list(e.export_state().values())
        got.append(seen)
    for i, (x, y) in enumerate(zip(*got)):
        assert torch.equal(x, y), i


@pytest.mark.parametrize("B,steps,slices,team", [(30720, 5, 1, 3), (30720, 2, 1, 0), (30721, 15, 1, 0), (30721, 16, 1, 3), (40001, 17, 2, 3)])
def test_large_rollouts_by_teams_and_by_single_wavefronts_agree(B, steps, slices, team):
    assert pg.GoEnv(B, 19).boards_per_team(steps, slices)[0] == team
    test_rollouts_by_teams_and_by_single_wavefronts_agree(19, B, steps, slices, True, True)


def test_rollouts_by_teams_with_slices_beyond_four_gibibytes():
    """720001 games of 19x19, two slices of 4.4 GB, some 90 times the games that the machine holds at once: the oracle replays the first games,
    those on both sides of the 4 GiB offset and the last ones."""
    B, N, seed, before, plies = 720001, 19, 21, 60, 17
    cross = (1 << 32) // (N * N * 17)
    ids = np.concatenate([np.arange(384), np.arange(cross - 192, cross + 192), np.arange(B - 384, B)]).astype(np.int32)
    p = Pair(B, N, seed, True, ids=ids, bind=False)
    assert p.env.boards_per_team(plies, 2) == (3, 3) and not p.env.rollout_in_time_slots(plies, 2)[0]
    p.env.rollout(before, seed, 0)
    for t in range(before):
        p.orc.step(p.orc.random_actions(seed, t))
    new = lambda *shape, dtype=torch.uint8: torch.full(shape, 7, dtype=dtype, device="cuda")  # noqa: E731
    mask, obs = new(2, B, N * N + 1), new(2, B, N * N * 17)
    act, rew, term = new(2, B, dtype=torch.int32), new(2, B, 2, dtype=torch.float32), new(2, B)
    p.env.rollout(plies, seed, before, slices=2, actions=act, rewards=rew, terminated=term, mask=mask, obs=obs)
    for i in range(plies):
        a = p.orc.random_actions(seed, before + i)
        p.orc.step(a)
        if i >= plies - 2:
            k = i & 1
            for name, x, y in (("actions", act, a), ("mask", mask, p.orc.legal_mask()), ("obs", obs, p.orc.observe()), ("rewards", rew, p.orc.rewards()),
                               ("terminated", term, p.orc.terminated())):
                assert (p.pick(x[k]).reshape(y.shape) == y).all(), (name, i)
    g, c = p.env.export_state(), p.orc.export_state()
    for name in ("board", "history", "ko", "to_play", "steps", "passes", "episode"):
        assert (p.pick(g[name]).astype(np.int64) == getattr(c, name).astype(np.int64)).all(), name


@pytest.mark.parametrize("N,B,obs", [(9, 7, True), (9, 1500, False), (19, 2, False), (19, 517, True)])
def test_the_shortest_rollouts_by_teams_of_games_whose_rings_begin_anywhere(N, B, obs):
    """One wavefront of a team reads where a game's ring of positions begins, which the launch itself sets back to its start."""
    envs = [pg.GoEnv(B, N, seed=6, auto_reset=True, max_steps=30) for _ in range(2)]
    envs[1].set_boards_per_wavefront(2)
    outs = [bound(e, True) for e in envs]
    rng = np.random.default_rng(B)
    for t in range(0, 40, 4):
        for k in range(2):
            a = envs[0].random_actions(6, t + k)
            a[torch.as_tensor(rng.random(B) < 0.4, device="cuda")] = -1   # a game that sits out keeps its ring where it is
            for e in envs:
                e.step(a)
        got = []
        for e in envs:
            m, o = torch.full((2, B, e.mask_pitch), 7, dtype=torch.uint8, device="cuda"), torch.full((2, B, e.obs_pitch), 7, dtype=torch.uint8, device="cuda")
            e.rollout(2, 6, t + 2, slices=2, mask=m, obs=o if obs else None)
            got.append([m, o, *e.export_state().values()])
        for i, (x, y) in enumerate(zip(*got)):
            assert torch.equal(x, y), (t, i)
        a = envs[0].random_actions(6, t + 4)
        for e in envs:
            e.step(a)
        for i, (x, y) in enumerate(zip(*outs)):
            assert torch.equal(x, y), (t, i)


@pytest.mark.parametrize("N,n,auto_reset,obs,line_padded", [
    (9, 1, False, True, False), (9, 385, True, True, True), (9, 1023, False, False, False), (9, 1025, False, True, False), (9, 4095, False, True, False),
    (19, 2, False, True, True), (19, 512, True, True, False), (19, 514, False, False, False), (19, 4097, False, True, False)])
def test_search_entries_by_teams_and_by_single_wavefronts_agree(N, n, auto_reset, obs, line_padded):
    pool = 3 * n + 1
    kw = dict(seed=3, auto_reset=auto_reset, line_padded=line_padded, max_steps=50)
    envs = [pg.GoEnv(pool, N, **kw), pg.GoEnv(pool, N, **kw)]
    envs[1].set_boards_per_wavefront(3)
    for e in envs:
        e.rollout(46, 3, 0)
    rng = np.random.default_rng(n)
    dev = lambda x: torch.as_tensor(x.astype(np.int32), device="cuda")  # noqa: E731
    for t in range(8):
        order = rng.permutation(pool)
        src = rng.choice(order[:pool - n], size=n)                  # several entries may come from one slot
        dst = np.where(rng.random(n) < 0.2, -1, order[pool - n:])   # (-1: filled in below)
        own = np.unique(src, return_index=True)[1]                  # an entry whose source nobody else reads may go back to it
        alone = np.array([i for i in own if (src == src[i]).sum() == 1 and dst[i] < 0], dtype=int)
        dst[alone] = src[alone]
        dst[dst < 0] = order[pool - n:][dst < 0]
        act = envs[0].random_actions(3, 60 + t).cpu().numpy()[src]
        if t % 2:
            act = np.where(rng.random(n) < 0.15, rng.choice([-1, 0, N * N, N * N + 7], size=n), act)   # a copy, a corner, pass, out of range
            outside = rng.random(n) < 0.03
            src = np.where(outside, rng.choice([-1, pool], size=n), src)
        out = []
        for e in envs:
            m, r, z = torch.full((n, e.mask_pitch), 7, dtype=torch.uint8, device="cuda"), torch.full((n, 2), 7.0, device="cuda"), torch.full((n,), 7, dtype=torch.uint8, device="cuda")
            o = torch.full((n, e.obs_pitch), 7, dtype=torch.uint8, device="cuda")
            some = t != 6   # once without rewards and terminated
            e.step_slots(dev(src), dev(act), dev(dst), mask=m if t != 4 else None, obs=o if obs else None, rewards=r if some else None, terminated=z if some else None)
            out.append([m, o, r, z, *e.export_state().values()])
        for i, (x, y) in enumerate(zip(*out)):
            assert torch.equal(x, y), (t, i)

"""Plies with the repetition rule in the mask, and rollouts with the rule in either reading, are run by teams of wavefronts up to a line.  At the sizes where the boards per team change,
and in ragged last teams, outputs and state are those of the kernel in which one wavefront does everything; the oracle checks positions
with more forbidden plays than a game's record holds."""
import numpy as np
import pytest
import torch

import bench
import paper_2303_17503_amd as pg
from gpu_common import Pair, to_np
from test_gpu_superko import N9, a9, hand_history, import_both
from test_gpu_teams import bound

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B,obs,mode,team", [
    (9, 384, True, 2, (1, 3)), (9, 385, False, 2, (4, 2)), (9, 4097, True, 2, (6, 3)), (9, 16384, True, 2, (6, 3)), (9, 16385, True, 2, (0, 1)), (9, 256, True, 1, (0, 1)),
    (19, 384, True, 2, (1, 3)), (19, 385, True, 2, (3, 3)), (19, 10240, False, 2, (3, 2)), (19, 10241, True, 2, (0, 1)), (19, 256, True, 1, (0, 1))])
def test_which_plies_go_by_teams(N, B, obs, mode, team):
    env = pg.GoEnv(B, N)
    env.enable_superko(mode)
    assert env.boards_per_team(0, obs=obs) == team
    assert bench.go_kernel(env, B, obs, superko=mode)[0].startswith("go_step_superko_team" if team[0] else "go_step_superko_kernel")
    env.set_boards_per_wavefront(2)
    assert env.boards_per_team(0, obs=obs) == (0, 1)


@pytest.mark.parametrize("N,B,auto_reset,obs,line_padded", [
    (9, 1, True, True, False), (9, 384, True, False, False), (9, 387, False, True, True), (9, 4097, True, True, False), (9, 16383, True, False, False),
    (19, 1, False, True, True), (19, 385, True, True, False), (19, 1000, False, False, False), (19, 10240, True, True, False)])
def test_teams_and_single_wavefronts_agree(N, B, auto_reset, obs, line_padded):
    kw = dict(seed=9, auto_reset=auto_reset, line_padded=line_padded, max_steps=60 if auto_reset else 0)
    a, b = pg.GoEnv(B, N, **kw), pg.GoEnv(B, N, **kw)
    b.set_boards_per_wavefront(2)
    for e in (a, b):
        e.enable_superko(2)
        e.rollout(40 if auto_reset else 150, 9, 0)
    oa, ob = bound(a, obs), bound(b, obs)
    rng = np.random.default_rng(B)
    nxt = a.random_actions(9, 500)
    for t in range(40):
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


@pytest.mark.parametrize("forbidden", [1, 2, 3, 5])
def test_more_forbidden_plays_than_a_record_holds(forbidden):
    """Each earlier position is the current one plus a black stone: that many plays of Black's are forbidden, and found anew from the table if
    there are more than two.  Games that skip, pass, play one of them or another point, twice in a row."""
    points = [a9(4, 4), a9(0, 8), a9(8, 0), a9(1, 5), a9(7, 3)][:forbidden]
    cur = {a9(2, 2): 1, a9(6, 6): -1, a9(3, 7): -1}
    acts = np.array([-1, 81, points[0], points[-1], a9(5, 5), a9(2, 2), -1], np.int32)
    s = hand_history(len(acts), cur, {**cur, points[0]: 1}, 1)
    for i, p in enumerate(points[1:]):
        for q, v in {**cur, p: 1}.items():
            s.history[:, 2 + i, q] = v
    pair = Pair(len(acts), N9, seed=4, auto_reset=False, superko="mask")
    assert pair.env.boards_per_team(0)[0] > 0
    import_both(pair, s)
    pair.compare("after import", state=True)
    assert not to_np(pair.mask)[:, points].any()
    for turn in range(3):
        a = np.roll(acts, turn)
        pair.step(torch.as_tensor(a, device="cuda"), a)
        pair.compare(f"turn {turn}", state=True)


@pytest.mark.parametrize("N,B,obs,mode,steps,team", [
    (9, 9216, True, 1, 2, (6, 3)), (9, 9217, True, 1, 16, (0, 1)), (9, 6912, True, 2, 16, (6, 3)), (9, 6913, True, 2, 16, (0, 1)), (9, 12288, False, 1, 3, (6, 2)),
    (9, 12289, False, 1, 16, (0, 1)), (9, 1000, False, 1, 2, (0, 1)), (9, 6144, False, 2, 8, (6, 2)), (9, 6144, False, 2, 7, (0, 1)), (9, 6145, False, 2, 16, (0, 1)),
    (19, 4608, True, 1, 2, (3, 3)), (19, 4609, True, 1, 8, (0, 1)), (19, 3456, True, 2, 2, (3, 3)), (19, 3457, True, 2, 8, (0, 1)), (19, 4096, False, 1, 3, (3, 2)),
    (19, 4097, False, 1, 3, (0, 1)), (19, 6144, False, 1, 4, (3, 2)), (19, 6145, False, 1, 4, (0, 1)), (19, 512, True, 2, 2, (1, 3)), (19, 512, True, 2, 1, (0, 1))])
def test_which_rollouts_go_by_teams(N, B, obs, mode, steps, team):
    env = pg.GoEnv(B, N)
    env.enable_superko(mode)
    assert env.boards_per_team(steps, 1, obs=obs) == team
    assert env.boards_per_team(steps, 1, mask=False, obs=False) == (0, 1)
    env.set_boards_per_wavefront(3)
    assert env.boards_per_team(steps, 1, obs=obs) == (0, 1)


@pytest.mark.parametrize("mode", [1, 2])
@pytest.mark.parametrize("N,B,steps,slices,obs,auto_reset", [
    (9, 1, 9, 1, True, True), (9, 385, 9, 4, True, False), (9, 1023, 8, 8, False, True), (9, 6143, 8, 2, True, True), (9, 2, 2, 1, True, False),
    (19, 1, 8, 1, False, True), (19, 511, 7, 7, True, False), (19, 1025, 8, 2, False, True), (19, 3455, 3, 1, True, True)])
def test_rollouts_by_teams_and_by_single_wavefronts_agree(N, B, steps, slices, obs, auto_reset, mode):
    kw = dict(seed=4, auto_reset=auto_reset, max_steps=45 if auto_reset else 0)
    envs = [pg.GoEnv(B, N, **kw), pg.GoEnv(B, N, **kw)]
    envs[1].set_boards_per_wavefront(3)
    start = torch.as_tensor(np.random.default_rng(B).integers(0, 44, size=B).astype(np.int32), device="cuda")   # some wait through a whole launch
    got = []
    for e in envs:
        e.enable_superko(mode)
        assert (e.boards_per_team(steps, slices, obs=obs)[0] > 0) == (e is envs[0])
        m, o = torch.full((slices, B, e.mask_pitch), 7, dtype=torch.uint8, device="cuda"), torch.full((slices, B, e.obs_pitch), 7, dtype=torch.uint8, device="cuda")
        r, t = torch.full((slices, B, 2), 7.0, dtype=torch.float32, device="cuda"), torch.full((slices, B), 7, dtype=torch.uint8, device="cuda")
        a = torch.full((slices, B), 7, dtype=torch.int32, device="cuda")
        seen = []
        for k in range(20 if N == 9 else 6):
            e.rollout(steps, 4, 36 + k * steps, start_t=start, slices=slices, actions=a, rewards=r, terminated=t, mask=m, obs=o if obs else None)
            seen += [x.clone() for x in (m, o, r, t, a)]
        seen += [e.legal_mask().clone()] + list(e.export_state().values())   # the mask by the record that the launch leaves
        got.append(seen)
    for i, (x, y) in enumerate(zip(*got)):
        assert torch.equal(x, y), i

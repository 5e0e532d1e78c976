"""Hex rollouts of small batches are run by teams of wavefronts: their outputs and state are those of the kernel in which one wavefront does
everything (set_mapping(1) asks for it), at the lines, in ragged last teams, with games that wait, end, restart and swap."""
import numpy as np
import pytest
import torch

import bench
import paper_2303_17503_amd as pg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("B,steps,slices,mask,obs,auto_reset", [
    (1, 2, 1, True, True, True), (4, 9, 9, True, True, False), (6, 5, 2, True, False, True), (1281, 7, 3, True, True, True), (5119, 16, 1, True, True, True),
    (5120, 3, 1, True, False, True), (5121, 3, 1, True, False, True), (10240, 3, 2, True, True, True), (10241, 2, 1, True, True, True), (12288, 4, 1, True, False, False),
    (16384, 16, 2, True, True, True), (16384, 17, 1, True, False, True), (999, 40, 4, False, True, True)])
def test_rollouts_by_teams_and_by_single_wavefronts_agree(B, steps, slices, mask, obs, auto_reset):
    envs = [pg.HexEnv(B, seed=6, auto_reset=auto_reset) for _ in range(2)]
    envs[1].set_mapping(1)
    by_teams = (B, steps, obs) not in [(5121, 3, False), (10241, 2, True)]   # the other side of a line
    assert [e.boards_per_team(steps, slices, mask=mask, obs=obs) for e in envs] == [(5, 3 if obs else 2) if by_teams else (0, 1), (0, 1)]
    start = torch.as_tensor(np.random.default_rng(B).integers(-3, 40, size=B).astype(np.int32), device="cuda")   # some wait through a whole launch
    got = []
    for e in envs:
        new = lambda *shape, dtype=torch.uint8: torch.full((slices, B, *shape), 7, dtype=dtype, device="cuda")  # noqa: E731
        m, o, r, t, a = new(e.A), new(e.OBS), new(2, dtype=torch.float32), new(), new(dtype=torch.int32)
        seen, ply = [], 0
        while ply < 150:                       # past the end of the first games
            e.rollout(steps, 6, ply, start_t=start, slices=slices, actions=a, rewards=r, terminated=t, mask=m if mask else None, obs=o if obs else None)
            ply += steps
            if ply % (8 * steps) == 0 or ply < 3 * steps or ply >= 150:
                seen += [x.clone() for x in (m, o, r, t, a)]
        seen += list(e.export_state().values())
        got.append(seen)
    for i, (x, y) in enumerate(zip(*got)):
        assert torch.equal(x, y), i


@pytest.mark.parametrize("B,steps,obs,team", [
    (16384, 0, True, (0, 1)), (16384, 1, True, (0, 1)), (10240, 2, True, (5, 3)), (10241, 3, True, (0, 1)), (16384, 4, True, (5, 3)), (16385, 99, True, (0, 1)),
    (5120, 2, False, (5, 2)), (5121, 3, False, (0, 1)), (12288, 4, False, (5, 2)), (12289, 15, False, (0, 1)), (16384, 16, False, (5, 2)), (16385, 16, False, (0, 1)),
    (20480, 16, True, (0, 1))])
def test_which_rollouts_go_by_teams(B, steps, obs, team):
    env = pg.HexEnv(B)
    assert env.boards_per_team(steps, obs=obs) == team
    assert env.boards_per_team(steps, mask=False, obs=False) == (0, 1)
    if steps:
        assert bench.hex_rollout_kernel(env, steps, obs) == ("hex_rollout_team_kernel" if team[0] else "hex_rollout_lane_kernel" if B == 20480 else "hex_rollout_kernel")
    for mapping in (1, 2):
        env.set_mapping(mapping)
        assert env.boards_per_team(steps, obs=obs) == (0, 1)
    env.set_mapping(0)
    assert env.boards_per_team(steps, obs=obs) == team

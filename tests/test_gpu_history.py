"""The history as the state keeps it: games whose rings of positions begin at different places in one wavefront (games that sat
out different plies), their first and ninth position, restarted games, and what a rollout or an import hands on to the step calls."""
import numpy as np
import pytest
import torch

import paper_2303_17503_amd as pg
from gpu_common import Pair, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("N,B", [(9, 1), (9, 25), (19, 2), (19, 37)])
def test_rings_that_begin_anywhere(N, B):
    p = Pair(B, N, seed=11, auto_reset=True, max_steps=23)   # every game is re-initialised within the test
    rng = np.random.default_rng(N * B)
    t = 0
    for plies in (9, 14):
        for _ in range(plies):
            a = p.orc.random_actions(5, t)
            a[rng.random(B) < 0.35] = -1                      # a game that sits out keeps its history where it is
            a[rng.random(B) < 0.05] = N * N                   # a pass repeats the position in the history
            p.step(torch.as_tensor(a, device="cuda"), a)
            t += 1
            p.compare(f"t={t}", state=True)
        p.env.rollout(3, 5, t)                                # registers of another form, written back with every ring at its beginning
        for _ in range(3):
            p.orc.step(p.orc.random_actions(5, t))
            t += 1
        a = p.orc.random_actions(5, t)
        assert (to_np(p.env.random_actions(5, t)) == a).all()
        p.step(torch.as_tensor(a, device="cuda"), a)
        t += 1
        p.compare(f"after the rollout, t={t}", state=True)
        p.env.import_state(p.env.export_state())              # (its rewards are zero until the next ply)
        a = p.orc.random_actions(5, t)
        p.step(torch.as_tensor(a, device="cuda"), a)
        t += 1
        p.compare("after an import of what was exported", state=True)


@pytest.mark.parametrize("B,superko,more", [(1, 0, {}), (37, 0, {}), (37, 1, {}), (38, 2, {}), (37, 0, {"mask_pitch": 364}), (38, 2, {"mask_pitch": 364}), (37, 1, {"mask_pitch": 364})])
def test_rollouts_without_observation_keep_the_same_history(B, superko, more):
    """Where nothing is emitted a 19x19 rollout by single wavefronts leaves the rings as they are; what follows sees the same eight positions."""
    envs = [pg.GoEnv(B, 19, seed=8, auto_reset=True, max_steps=40, **more) for _ in range(2)]
    obs = [torch.zeros((1, B, envs[0].obs_pitch), dtype=torch.uint8, device="cuda"), None]
    start = torch.arange(B, dtype=torch.int32, device="cuda") % 7 * 5   # some wait
    for e in envs:
        e.set_boards_per_wavefront(3)
        if superko:
            e.enable_superko(superko)
    rng = np.random.default_rng(B)
    t = 0
    for plies in (1, 2, 9, 1, 30):
        a = envs[0].random_actions(8, t)
        a[torch.as_tensor(rng.random(B) < 0.4, device="cuda")] = -1   # a game that sits out keeps its ring where it is
        for e, o in zip(envs, obs):
            e.step(a)
            e.rollout(plies, 8, t + 1, start_t=start, obs=o)
        t += 1 + plies
        x, y = (e.export_state() for e in envs)
        for k in x:
            assert torch.equal(x[k], y[k]), (t, k)
        assert torch.equal(envs[0].observe(), envs[1].observe()) and torch.equal(*(e.mask_view(e.legal_mask()) for e in envs)), t

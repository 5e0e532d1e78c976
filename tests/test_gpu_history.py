"""The history as the state keeps it: games whose rings of positions begin at different places in one wavefront (games that sat
out different plies), their first and ninth position, restarted games, and what a rollout or an import hands on to the step calls."""
import numpy as np
import pytest
import torch

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

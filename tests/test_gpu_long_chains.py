"""Plies on boards filled by two interleaved spirals: chains of up to 180 stones whose few liberties lie far apart, so that a
flood takes many looks at them, and captures of a whole spiral."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def spiral(N):
    """+1 on a one-point-wide path that winds from the corner to the middle, -1 on what it leaves between its turns."""
    board = -np.ones((N, N), np.int8)
    r = c = 0
    dr, dc = 0, 1
    board[0, 0] = 1

    def free(r, c):
        return 0 <= r < N and 0 <= c < N and board[r, c] < 0

    for _ in range(N * N):
        ahead_r, ahead_c = r + 2 * dr, c + 2 * dc
        beyond = 0 <= ahead_r < N and 0 <= ahead_c < N and board[ahead_r, ahead_c] > 0
        if not free(r + dr, c + dc) or beyond:
            dr, dc = dc, -dr
            ahead_r, ahead_c = r + 2 * dr, c + 2 * dc
            if not free(r + dr, c + dc) or (0 <= ahead_r < N and 0 <= ahead_c < N and board[ahead_r, ahead_c] > 0):
                break
        r, c = r + dr, c + dc
        board[r, c] = 1
    return board


def positions(N, count, seed):
    rng = np.random.default_rng(seed)
    base = spiral(N).reshape(-1)
    boards = np.empty((count, N * N), np.int8)
    for i in range(count):
        b = base.copy()
        for colour in (1, -1):   # the pieces a spiral falls into end at the points taken out of it: every chain has a liberty
            own = np.flatnonzero(base == colour)
            b[rng.choice(own, size=int(rng.integers(1, 4)), replace=False)] = 0
        boards[i] = b if i % 2 == 0 else -b
    return boards


@pytest.mark.parametrize("N,per_wavefront", [(9, 1), (9, 5), (9, 6), (19, 1), (19, 2), (19, 3)])
def test_spirals(N, per_wavefront):
    from gpu_common import Pair
    B = 97
    p = Pair(B, N, seed=3, auto_reset=False)
    assert p.env.set_boards_per_wavefront(per_wavefront) == per_wavefront
    st = p.orc.export_state()
    st.board[...] = positions(N, B, seed=N).reshape(st.board.shape)
    st.to_play[...] = np.where(np.arange(B) % 3 == 0, 1, -1)
    p.orc.import_state(st)
    dev = {k: torch.as_tensor(getattr(st, k), device="cuda") for k in st.__slots__}
    dev["episode"] = dev["episode"].to(torch.int32)
    p.env.import_state(dev)
    p.compare("imported", state=False)
    before = np.abs(p.orc.export_state().board.astype(np.int64)).sum(1)
    largest = 0
    for t in range(12):
        a = p.orc.random_actions(9, t)
        assert (p.env.random_actions(9, t).cpu().numpy() == a).all()
        p.step(torch.as_tensor(a, device="cuda"), a)
        p.compare(f"t={t}")
        after = np.abs(p.orc.export_state().board.astype(np.int64)).sum(1)
        largest = max(largest, int((before - after).max()))
        before = after
    assert largest > N   # whole stretches of a spiral were taken


def test_spiral_shape():
    for N, least in ((9, 40), (19, 180)):
        b = spiral(N)
        assert (b > 0).sum() >= least and (b < 0).sum() >= least - 20

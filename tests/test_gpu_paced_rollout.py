"""Recorded rollouts large enough to be written in time slots (recordings that outgrow the memory-side cache): every slice equals
what the same plies give one launch each, for dense, line-padded and other pitches, with the repetition rule, and for more games
than the machine holds at once."""
import pytest
import torch

import paper_2303_17503_amd as pg

pytestmark = pytest.mark.gpu


def check(make, slices, seed, mask_of, obs_of, generations):
    rec, one = make(), make()
    B = rec.B
    slots, games = rec.rollout_in_time_slots(slices, slices)
    assert slots and not one.rollout_in_time_slots(1, 1)[0]
    assert (B > games) == generations, games
    new = lambda *shape, dtype=torch.uint8: torch.zeros(*shape, dtype=dtype, device="cuda")  # noqa: E731
    mask, obs = new(slices, B, mask_of(rec)), new(slices, B, obs_of(rec))
    rew, term, act = new(slices, B, 2, dtype=torch.float32), new(slices, B), new(slices, B, dtype=torch.int32)
    m1, o1, r1, t1, a1 = new(1, B, mask_of(rec)), new(1, B, obs_of(rec)), new(1, B, 2, dtype=torch.float32), new(1, B), new(1, B, dtype=torch.int32)
    for env in (rec, one):
        env.rollout(70, seed, 0)
    for _ in range(2):   # the second launch writes over the first one's slices
        t = 70 + _ * slices
        rec.rollout(slices, seed, t, slices=slices, actions=act, rewards=rew, terminated=term, mask=mask, obs=obs)
        for i in range(slices):
            one.rollout(1, seed, t + i, actions=a1, rewards=r1, terminated=t1, mask=m1, obs=o1)
            for name, x, y in (("mask", mask, m1), ("obs", obs, o1), ("rewards", rew, r1), ("terminated", term, t1), ("actions", act, a1)):
                assert torch.equal(x[i], y[0]), (name, t, i)
    a, b = rec.export_state(), one.export_state()
    for k in a:
        assert torch.equal(a[k], b[k]), k


@pytest.mark.parametrize("N,B,slices,superko,more", [   # the last four: more games than the machine holds at once
    (9, 17001, 13, 0, {}),
    (9, 17001, 13, 0, {"obs_pitch": 1400, "mask_pitch": 90}),
    (9, 17001, 13, 2, {}),
    (9, 17001, 13, 1, {"obs_pitch": 1379}),
    (19, 5003, 10, 0, {"line_padded": True}),
    (19, 5003, 10, 1, {}),
    (19, 5003, 10, 2, {"mask_pitch": 363}),
    (19, 19001, 3, 0, {}),
    (9, 52001, 4, 0, {}),
    (9, 75001, 3, 0, {}),
    (19, 26001, 2, 2, {}),
])
def test_go(N, B, slices, superko, more):
    def make():
        env = pg.GoEnv(B, N, seed=4, auto_reset=True, **more)
        if superko:
            env.enable_superko(superko)
        return env
    check(make, slices, 11, lambda e: e.mask_pitch, lambda e: e.obs_pitch, B > 19000 or (N == 9 and B > 37000))


@pytest.mark.parametrize("B,slices", [(45001, 12), (470003, 2)])
def test_hex(B, slices):
    check(lambda: pg.HexEnv(B, seed=4, auto_reset=True), slices, 11, lambda e: e.A, lambda e: e.OBS, B > 400000)


@pytest.mark.parametrize("game,steps,slices,slots", [
    ("go", 1, 16, False), ("go", 2, 16, False), ("go", 2, 2, False), ("go", 16, 2, False), ("go", 3, 16, True), ("go", 3, 3, True), ("go", 50, 16, True),
    ("go", 50, 1, False), ("go", 0, 16, False), ("hex", 1, 8, False), ("hex", 2, 8, True), ("hex", 8, 8, True), ("hex", 8, 1, False)])
def test_what_counts_is_what_a_launch_writes(game, steps, slices, slots):
    """107 MB a ply in Go, 159 MB in Hex: two and one of them stay in the 256 MB cache, however many slices the buffers have"""
    env = pg.GoEnv(16384, 19) if game == "go" else pg.HexEnv(262144)
    assert env.rollout_in_time_slots(steps, slices)[0] == slots


def test_fewer_plies_than_slices():
    B, slices, seed = 16384, 6, 5
    a, b = (pg.GoEnv(B, 19, seed=2, auto_reset=True) for _ in range(2))
    new = lambda n, pitch: torch.full((n, B, pitch), 7, dtype=torch.uint8, device="cuda")  # noqa: E731
    mask, obs, m1, o1 = new(slices, a.mask_pitch), new(slices, a.obs_pitch), new(1, a.mask_pitch), new(1, a.obs_pitch)
    t = 0
    for steps in (1, 4, 2):   # without slots, with them, without
        mask.fill_(7)
        obs.fill_(7)
        a.rollout(steps, seed, t, slices=slices, mask=mask, obs=obs)
        for i in range(steps):
            b.rollout(1, seed, t + i, mask=m1, obs=o1)
            assert torch.equal(mask[i], m1[0]) and torch.equal(obs[i], o1[0]), (steps, i)
        assert (mask[steps:] == 7).all() and (obs[steps:] == 7).all(), steps
        t += steps


@pytest.mark.parametrize("game,B,superko,steps,slices,slots", [
    ("go", 16384, 0, 4, 4, True), ("go", 16384, 0, 6, 4, False), ("go", 16384, 0, 50, 4, False), ("go", 16384, 0, 50, 8, True),
    ("go", 65536, 0, 2, 2, True), ("go", 65536, 0, 3, 2, False), ("go", 65536, 0, 50, 4, False), ("go", 65536, 0, 50, 8, True),
    ("go", 8000, 0, 24, 8, True), ("go", 8000, 0, 60, 6, False), ("go", 16384, 2, 50, 3, True), ("go", 16384, 1, 50, 3, True),
    ("hex", 262144, 0, 3, 3, True), ("hex", 262144, 0, 30, 3, False), ("hex", 262144, 0, 80, 8, True), ("hex", 1000000, 0, 6, 3, False)])
def test_rewritten_slices_stay_in_the_cache(game, B, superko, steps, slices, slots):
    """Plies that rewrite what the launch itself has written find much of it in the memory-side cache, which is faster than slots made for
    DRAM: only footprints far beyond the cache are written in slots then."""
    env = pg.GoEnv(B, 19) if game == "go" else pg.HexEnv(B)
    if superko:
        env.enable_superko(superko)
    assert env.rollout_in_time_slots(steps, slices)[0] == slots

"""The native argument checks of the per-ply calls refuse what the Python checks refuse, and pass on what they pass on."""
import ctypes as C

import pytest
import torch

import paper_2303_17503_amd as pg
from paper_2303_17503_amd import binding

fast = pytest.importorskip("paper_2303_17503_amd._fastcall")


def test_nothing_but_cuda_tensors_reaches_the_entry_point():
    calls = []
    stub = C.CFUNCTYPE(C.c_int, C.c_void_p, C.c_void_p)(lambda h, p: calls.append(1) or 0)
    address = C.cast(stub, C.c_void_p).value
    for bad in (torch.zeros(3, dtype=torch.int32), None, 5, "x", [0, 0, 0]):
        assert fast.step(address, 1, 3, bad) is None
    assert fast.step(address, 1, 3) is None and fast.step("x", 1, 3, None) is None
    assert not calls


def variants(t):
    """(what, tensor, accepted)"""
    class Sub(torch.Tensor):
        pass
    yield "as it is", t, True
    yield "subclass", t.clone().as_subclass(Sub), True
    yield "offset view", torch.cat([t, t])[t.shape[0]:], True
    yield "type", t.to(torch.int64 if t.dtype == torch.int32 else torch.int8), False
    yield "on the host", t.cpu(), False
    yield "too short", t[:-1].clone(), False
    yield "one dimension more", t[None].contiguous(), False
    if t.shape[0] > 1:
        yield "strided", torch.stack([t, t], -1)[..., 0], False


def outcome(f):
    try:
        f()
    except Exception as e:  # noqa: BLE001
        return type(e).__name__
    return "ok"


@pytest.mark.gpu
@pytest.mark.parametrize("game", ["go", "hex"])
def test_same_verdicts_as_in_python(game, monkeypatch):
    from paper_2303_17503_amd import hex_binding
    B, n = 12, 4
    make = (lambda: pg.GoEnv(B, 9, seed=1)) if game == "go" else (lambda: pg.HexEnv(B, seed=1))
    full = torch.zeros(B, dtype=torch.int32, device="cuda")
    slots = [torch.arange(n, dtype=torch.int32, device="cuda"), torch.zeros(n, dtype=torch.int32, device="cuda"),
             torch.arange(n, 2 * n, dtype=torch.int32, device="cuda"), torch.zeros(n, 82, dtype=torch.uint8, device="cuda"),
             torch.zeros(n, 1377, dtype=torch.uint8, device="cuda"), torch.zeros(n, 2, device="cuda"), torch.zeros(n, dtype=torch.uint8, device="cuda")]

    def calls(env):
        for what, t, good in variants(full):
            yield "step " + what, good, lambda t=t: env.step(t)
            yield "random " + what, good, lambda t=t: env.random_actions(1, 0, out=t)
            yield "random start " + what, good, lambda t=t: env.random_actions(1, 0, t, out=full)
            yield "sample " + what, good, lambda t=t: env.step_sample(t, 1, 0, out=torch.zeros_like(full))
            yield "sample out " + what, good, lambda t=t: env.step_sample(torch.zeros_like(full), 1, 0, out=t)
        yield "sample in place", False, lambda: env.step_sample(full, 1, 0, out=full)
        if game == "go":
            for k, a in enumerate(slots):
                for what, t, good in variants(a):
                    args = list(slots)
                    args[k] = t
                    yield f"slots {k} {what}", good, lambda args=args: env.step_slots(*args)
            yield "slots without outputs", True, lambda: env.step_slots(*slots[:3])
            yield "slots, 0-dim source", False, lambda: env.step_slots(slots[0][0], *slots[1:])
            yield "slots, more than the pool", False, lambda: env.step_slots(*[torch.zeros(B + 1, dtype=torch.int32, device="cuda")] * 3)

    native = [(w, g, outcome(f)) for w, g, f in calls(make())]
    with monkeypatch.context() as m:
        m.setattr(binding, "_fast", None)
        m.setattr(hex_binding, "_fast", None)
        python = [(w, g, outcome(f)) for w, g, f in calls(make())]
    torch.cuda.synchronize()
    assert native == python
    for what, good, got in native:
        assert (got == "ok") == good, (what, got)

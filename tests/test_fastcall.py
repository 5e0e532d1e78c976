"""The native argument checks of the per-ply calls refuse what the Python checks refuse, and pass on what they pass on."""
import ctypes as C
import os
import subprocess
import sys

import pytest
import torch

import paper_2303_17503_amd as pg
from paper_2303_17503_amd import _fastcall as fast
from paper_2303_17503_amd import binding, build

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def python(code):
    return subprocess.run([sys.executable, "-W", "always", "-c", code], cwd=ROOT, capture_output=True, text=True)


def test_an_extension_that_does_not_load_is_reported():
    r = python("import sys; sys.modules['paper_2303_17503_amd._fastcall'] = None\n"
               "import paper_2303_17503_amd as pg; pg.lib(); pg.hex_binding.lib()\n"
               "assert pg.binding._fast is None and pg.hex_binding._fast is None")
    assert r.returncode == 0 and r.stderr.count("check their arguments in Python") == 1, r.stderr


def test_an_extension_built_after_the_import_is_used():
    r = python("import sys; sys.modules['paper_2303_17503_amd._fastcall'] = None\n"
               "import paper_2303_17503_amd as pg; del sys.modules['paper_2303_17503_amd._fastcall']\n"
               "pg.lib(); pg.hex_binding.lib(); assert pg.binding._fast is not None and pg.hex_binding._fast is pg.binding._fast")
    assert r.returncode == 0 and "in Python" not in r.stderr, r.stderr


def test_the_library_is_built_without_a_host_compiler(monkeypatch, tmp_path):
    run = subprocess.run

    def no_compiler(cmd, **kw):
        if cmd[0] == "g++":
            raise FileNotFoundError("g++")
        return run(["true"], **kw)   # stands for hipcc

    monkeypatch.setattr(build, "FAST", str(tmp_path / "_fastcall.so"))
    (tmp_path / "_fastcall.so").write_text("an older build")
    monkeypatch.setattr(build.subprocess, "run", no_compiler)
    with pytest.warns(RuntimeWarning, match="not built"):
        assert build.build() == build.LIB
    assert not (tmp_path / "_fastcall.so").exists()


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

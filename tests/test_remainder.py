"""remainder_of (remainder.hpp), the draw's hash mod legal_count in floats: right for every count the games can have, also with reciprocals one
unit in the last place off either way, as the hardware's instruction may give them.  Once restated in numpy, then the function itself, compiled
for the CPU with a reciprocal of the test's, and as the GPU runs it."""
import os
import subprocess

import numpy as np
import pytest

import paper_2303_17503_amd.build as build


def remainder_of(n, d, ulp):
    f32 = np.float32
    f = (f32(1) / d.astype(f32)).view(np.int32) + np.int32(ulp)
    f = f.view(f32)
    q = np.minimum(n.astype(f32) * f, f32(4294967040.0)).astype(np.uint64).astype(np.uint32)
    left = (n - q * d).view(np.int32)
    # the fused multiply-add rounds once: exact in 64 bits, then rounded
    v = (left.astype(f32).astype(np.float64) * f.astype(np.float64) + (f32(0.5) * f).astype(np.float64)).astype(f32)
    return (left - np.floor(v).astype(np.int32) * d.astype(np.int32)).view(np.uint32)


@pytest.mark.parametrize("ulp", [-1, 0, 1])
def test_every_count(ulp):
    rng = np.random.default_rng(5)
    for count in list(range(1, 1025)):
        n = rng.integers(0, 1 << 32, 500, dtype=np.uint32)
        multiple = n // np.uint32(count) * np.uint32(count)
        edge = np.arange(500, dtype=np.uint32)
        n = np.concatenate([n, multiple, multiple - np.uint32(1), multiple + np.uint32(count - 1), edge, ~edge])
        assert np.array_equal(remainder_of(n, np.full_like(n, count), ulp), n % np.uint32(count)), count


# most n lie around multiples of d all over the 32 bits (s: a stride of quotients), where a quotient can be one off; the rest are hashes and both ends
PROGRAM = r"""
#include <cstdint>
#include <cstdio>
#include <cstring>
static int off_by;   // units in the last place
static float reciprocal(float d) { float f = 1.0f / d; int32_t b; memcpy(&b, &f, 4); b += off_by; memcpy(&f, &b, 4); return f; }
static int mul24(int a, int b) { return (int)((int64_t)((int32_t)((uint32_t)a << 8) >> 8) * ((int32_t)((uint32_t)b << 8) >> 8)); }
#define __device__
#define __forceinline__ inline
#define __builtin_amdgcn_rcpf reciprocal
#define __mul24 mul24
#include "remainder.hpp"
int main() {
  uint64_t wrong = 0, looked = 0;
  uint32_t x = 1;
  auto look = [&](uint32_t n, uint32_t d) { wrong += pgxwave::remainder_of(n, d) != n % d; ++looked; };
  for (off_by = -1; off_by <= 1; ++off_by)
    for (uint32_t d = 1; d <= 1024; ++d) {
      const uint64_t most = 0xFFFFFFFFu / d, s = most / 25000 + 1;
      for (uint64_t q = 0; q <= most; q += s) {
        const uint32_t m = (uint32_t)q * d;
        look(m, d); look(m - 1, d); look(m + 1, d); look(m + d - 1, d);
      }
      for (uint32_t n = 0; n < 4096; ++n) { look(n, d); look(~n, d); x = x * 1664525u + 1013904223u; look(x, d); }
    }
  printf("%llu wrong of %llu\n", (unsigned long long)wrong, (unsigned long long)looked);
  return wrong != 0;
}
"""


def test_the_function_itself_for_every_count(tmp_path):
    src, exe = tmp_path / "remainder.cpp", tmp_path / "remainder"
    src.write_text(PROGRAM)
    subprocess.run(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-I", os.path.join(os.path.dirname(build.__file__), "csrc"), "-o", str(exe), str(src)], check=True)
    r = subprocess.run([str(exe)], capture_output=True, text=True)
    assert r.returncode == 0 and r.stdout.startswith("0 wrong of "), r.stdout


@pytest.mark.gpu
def test_the_function_on_the_gpu_for_every_count():
    import torch

    import paper_2303_17503_amd as pg

    rng = np.random.default_rng(6)
    for first in range(1, 1025, 64):   # 64 counts a launch
        d = np.arange(first, first + 64, dtype=np.uint64)[:, None]
        multiple = (rng.random((64, 25000)) * (2.0**32 / d)).astype(np.uint64) * d
        n = np.concatenate([multiple, multiple + 1, multiple + d - 1, multiple - 1, multiple[:, :4096] * 0 + np.arange(4096, dtype=np.uint64)], axis=1)
        n = np.concatenate([n, ~n[:, -4096:]], axis=1).astype(np.uint32)
        d = np.broadcast_to(d, n.shape).astype(np.uint32)
        got = pg.remainder_probe(*(torch.as_tensor(np.ascontiguousarray(v).view(np.int32), device="cuda") for v in (n, d)))
        assert np.array_equal(got.cpu().numpy().view(np.uint32), n % d), first

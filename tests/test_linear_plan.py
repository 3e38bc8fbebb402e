"""The host plan of the linear layers (csrc/linear_plan.cpp, built with g++
under the address and undefined-behaviour sanitizers) on the CPU: the layers
that the GPU tests run for one path of the kernels take that path."""

from __future__ import annotations

import os
import random
import shutil
import subprocess

import pytest

import linear_cases as LC
from paper_2506_14489_amd import workloads as WL

HERE = os.path.dirname(os.path.abspath(__file__))
CSRC = os.path.join(os.path.dirname(HERE), "paper_2506_14489_amd", "csrc")

pytestmark = pytest.mark.skipif(shutil.which("g++") is None or not os.path.isdir("/opt/rocm/include"),
                                reason="needs g++ and the HIP headers")


@pytest.fixture(scope="module")
def plan_of(tmp_path_factory):
    """plans([(moduli, shape, c_out, kh, kw, stride, pad), ...]) -> a dict of
    plan fields per layer (rc alone where it is refused)."""
    exe = str(tmp_path_factory.mktemp("plan") / "linear_plan_check")
    r = subprocess.run(["g++", "-std=c++17", "-fsanitize=address,undefined", "-fno-sanitize-recover=undefined", "-g",
                        "-O1", "-D__HIP_PLATFORM_AMD__", "-I/opt/rocm/include",
                        os.path.join(HERE, "linear_plan_check.cpp"), os.path.join(CSRC, "linear_plan.cpp"),
                        os.path.join(CSRC, "plan.cpp"), "-o", exe], capture_output=True, text=True)
    assert r.returncode == 0, r.stderr[-4000:]

    def plans(layers):
        lines = []
        for moduli, shape, c_out, kh, kw, stride, pad in layers:
            lines.append(" ".join(str(int(v)) for v in (len(moduli), *moduli, *[0] * (16 - len(moduli)), *shape, c_out, kh,
                                                        kw, stride, pad)))
        env = {k: v for k, v in os.environ.items() if k != "LD_PRELOAD"}
        r = subprocess.run([exe], input="\n".join(lines) + "\n", capture_output=True, text=True, env=env, timeout=300)
        assert r.returncode == 0, (r.stdout + r.stderr)[-4000:]
        return [{k: int(v) for k, v in (f.split("=") for f in line.split())} for line in r.stdout.splitlines()]

    return plans


def test_full_size_layers_take_their_paths(plan_of):
    got = plan_of([(w.moduli, w.in_shape, w.w_shape[0], w.w_shape[2], w.w_shape[3], w.stride, w.pad)
                   for w, _want in LC.SEVERAL_CHUNKS])
    for (w, want), plan in zip(LC.SEVERAL_CHUNKS, got):
        assert plan["ncc"] > 1
        assert {k: plan.get(k) for k in want} == want, (w.name, plan)


def test_small_layers_take_the_paths_they_are_named_for(plan_of):
    seen = set()
    for (name, *_layer), plan in zip(LC.SMALL, plan_of([c[1:] for c in LC.SMALL])):
        assert plan["rc"] == 0, name
        want = {"fold": (1, None), "no-fold": (0, None), "flat": (0, 1), "no-flat": (0, 0)}
        kind = next((k for k in ("no-fold", "no-flat", "fold", "flat") if name.startswith(k + "-")), None)
        if kind is None:
            continue
        seen.add(kind)
        fold, flat = want[kind]
        assert (plan["fold_c"] > 0) == bool(fold), (name, plan)
        assert flat is None or plan["flat"] == flat, (name, plan)
        if name.startswith("flat-32-"):
            assert plan["xt"] == 32, (name, plan)
    assert len(seen) == 4


def test_folded_planes_are_no_larger_than_their_windows(plan_of):
    """A folded layer's plane holds c_in bytes per position up to the last
    window's end, and takes no more than the ck bytes of every column a window
    can begin at; every byte of a window that is read lies in the plane.  (With
    columns that no window reads in the planes, the first layer was refused and
    the second one's working buffer was 1.9 times as large.)"""
    rng = random.Random(11)
    layers = [((5,), (1, 8, 100_000_000, 1), 1, 4, 4, 4, 3), (tuple(WL.PRIMES_12), (202, 10, 12633, 4), 43, 3, 3, 4, 1)]
    while len(layers) < 400:
        kh, kw = rng.randint(1, 16), rng.randint(2, 16)
        if kh * kw > 64:
            continue
        layers.append(((2, 3, 251), (rng.randint(1, 3), rng.randint(1, 15), rng.randint(1, 40), rng.randint(1, 40)),
                       rng.randint(1, 70), kh, kw, rng.choice([1, 2, 3, rng.randint(1, 40)]), rng.randint(0, min(kh, kw) - 1)))
    folded = 0
    for (moduli, (n, c, h, w), _co, kh, kw, stride, pad), plan in zip(layers, plan_of(layers)):
        if plan["rc"] or not plan["fold_c"]:
            continue
        folded += 1
        rows, cols = n * (h + 2 * pad), (w + 2 * pad - kw) // stride + 1
        windows = rows * ((cols - 1) * stride + 1) * plan["ck"]
        assert plan["plane_bytes"] <= windows, (n, c, h, w, kh, kw, stride, pad, plan)
        assert plan["cp"] == c and plan["xlast"] == (cols - 1) * stride and plan["xlast"] + kw <= plan["wp"] <= w + 2 * pad
        last = ((rows - 1) * plan["wp"] + plan["xlast"]) * c + plan["ck"]
        assert max(last, -(-rows * plan["wp"] * c // 4) * 4) <= plan["plane_bytes"]
    assert folded > 100
    first, second = plan_of(layers[:2])
    assert first["rc"] == 0 and second["plane_bytes"] < 90_000_000

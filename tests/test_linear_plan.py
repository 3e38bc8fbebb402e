"""The host plan of the linear layers (csrc/linear_plan.cpp, built with g++
under the address and undefined-behaviour sanitizers) on the CPU: the layers
that the GPU tests run for one path of the kernels take that path."""

from __future__ import annotations

import os
import shutil
import subprocess

import pytest

import linear_cases as LC

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
        assert {k: plan.get(k) for k in want} == want, (w.name, plan)

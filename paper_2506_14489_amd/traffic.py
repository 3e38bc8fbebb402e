"""Measured HBM traffic (and vector instruction count) of an evaluation call,
from hardware counters.

The figures were taken with rocprofv3 counter passes over ``bench.py``
(``--pmc FETCH_SIZE``, then ``--pmc WRITE_SIZE``; KiB per dispatch, the
dispatches of one call added: ``k_eval`` on the whole rounds and
``k_eval_split`` on the rest) and scaled by what the same counters read for a plain
device-to-device copy of known size (``bench.py --copy-calibration 1024``:
a 1 GiB copy reads FETCH_SIZE = 524,300 KiB and WRITE_SIZE = 1,048,576 KiB,
so FETCH_SIZE is scaled by 2 and WRITE_SIZE by 1).

A figure is only valid for the kernels it was taken on: ``traffic_bytes``
returns None as soon as any source file that defines the evaluation kernels
differs from the one the counters were read on (a SHA-256 over those
sources, in a fixed order; the linear-layer source and the C header, which
the kernel does not depend on beyond the plan, are not part of it).
"""

from __future__ import annotations

import hashlib
import os

from . import build as _build

# 1 GiB device-to-device copy: counter reading -> bytes moved
FETCH_FACTOR = 1048576 / 524300
WRITE_FACTOR = 1048576 / 1048576

# workload name -> counters per call (KiB; k_eval + k_eval_split) and the source hash
MEASURED = {
    "batched": {
        "kernel": "k_eval",
        "fetch_kib": 12693988.0 + 279081.0,  # means of four calls, within 50 KiB
        "write_kib": 1376256.0 + 98529.0,
        "valu_insts": 3346025062 + 70022396,  # SQ_INSTS_VALU (wave instructions; two calls, equal)
        "sources_sha256": "fff0dca832ca7ae83231d6af31f1aa3d5b06d759a472a560729b3ef9ae36e13d",
    },
}


# the files that define the evaluation kernels: their source, the device helpers, the plan and the AES tables
EVAL_SOURCES = ("redash.hip", "device.hpp", "plan.cpp", "plan.hpp", "aes_tables.hpp")


def sources_sha256() -> str:
    """SHA-256 over the evaluation kernel's source files (name and contents)."""
    h = hashlib.sha256()
    paths = [p for p in _build.SOURCES + _build.HEADERS if os.path.basename(p) in EVAL_SOURCES]
    for path in sorted(paths, key=os.path.basename):
        h.update(os.path.basename(path).encode())
        with open(path, "rb") as f:
            h.update(f.read())
    return h.hexdigest()


def valu_instructions(workload: str):
    """Vector ALU wave instructions per evaluation call on ``workload``
    (SQ_INSTS_VALU), or None as for traffic_bytes."""
    rec = MEASURED.get(workload)
    if rec is None or rec["sources_sha256"] != sources_sha256() or "valu_insts" not in rec:
        return None
    return rec["valu_insts"]


def traffic_bytes(workload: str):
    """HBM bytes (reads + writes) per evaluation call on ``workload``, or None
    if no counters were taken on it or the kernel sources changed since."""
    rec = MEASURED.get(workload)
    if rec is None or rec["sources_sha256"] != sources_sha256():
        return None
    return (rec["fetch_kib"] * FETCH_FACTOR + rec["write_kib"] * WRITE_FACTOR) * 1024.0

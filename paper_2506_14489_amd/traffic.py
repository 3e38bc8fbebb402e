"""Measured HBM traffic (and vector instruction count) of the evaluation
kernel, from hardware counters.

The figures were taken with two rocprofv3 counter passes over
``bench.py`` (``--pmc FETCH_SIZE``, then ``--pmc WRITE_SIZE``; KiB per
dispatch) and scaled by what the same counters read for a plain
device-to-device copy of known size (``bench.py --copy-calibration 1024``:
a 1 GiB copy reads FETCH_SIZE = 524,300 KiB and WRITE_SIZE = 1,048,576 KiB,
so FETCH_SIZE is scaled by 2 and WRITE_SIZE by 1).

A figure is only valid for the kernel it was taken on: ``traffic_bytes``
returns None as soon as any source file that defines the evaluation kernel
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

# workload name -> counters per k_eval dispatch (KiB) and the source hash
MEASURED = {
    # per call: k_eval on the whole rounds and k_eval_split on the rest
    "batched": {
        "kernel": "k_eval",
        "fetch_kib": 12693669.0 + 279096.0,  # means of four calls, within 50 KiB
        "write_kib": 1376256.0 + 98311.0,
        "valu_insts": 3350366242 + 70021476,  # SQ_INSTS_VALU (wave instructions; four calls, equal)
        "sources_sha256": "9d70f3527be7f2f35c2ea1cc8a53d835e195c7dba7f679751341c7f63eaafb52",
    },
}


# the files that define k_eval: its source, the device helpers, the plan and the AES tables
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
    """Vector ALU wave instructions per k_eval launch on ``workload``
    (SQ_INSTS_VALU), or None as for traffic_bytes."""
    rec = MEASURED.get(workload)
    if rec is None or rec["sources_sha256"] != sources_sha256() or "valu_insts" not in rec:
        return None
    return rec["valu_insts"]


def traffic_bytes(workload: str):
    """HBM bytes (reads + writes) per k_eval launch on ``workload``, or None
    if no counters were taken on it or the kernel sources changed since."""
    rec = MEASURED.get(workload)
    if rec is None or rec["sources_sha256"] != sources_sha256():
        return None
    return (rec["fetch_kib"] * FETCH_FACTOR + rec["write_kib"] * WRITE_FACTOR) * 1024.0

"""Layers whose path through the layer kernels the tests name: the GPU tests
run them, and the CPU test of the host plan checks that each still takes the
path it stands for."""

from __future__ import annotations

from paper_2506_14489_amd import workloads as WL


def _conv(name, seed, in_shape, c_out, stride=1):
    return WL._conv(name, WL.PRIMES_12, (11,), seed, in_shape, c_out, 3, stride, 1)


# 3x3 layers over several channel chunks at full size: (workload, what the
# plan has to say).  word_split 0: each modulus has one workgroup per tile
# and channel group, 1: each packed word has one.
SEVERAL_CHUNKS = [
    (_conv("l2.b-batch4", 31, (4, 128, 28, 28), 128), {"ncc": 2, "flat": 1, "xt": 32, "word_split": 0, "og_xcd": 0}),
    (_conv("row-tiles-56x56", 32, (1, 128, 56, 56), 64), {"ncc": 2, "flat": 0, "xt": 16, "word_split": 0, "og_xcd": 0}),
    (_conv("stride2-batch8", 33, (8, 128, 28, 28), 256, 2), {"ncc": 2, "flat": 0, "xt": 16, "word_split": 0, "og_xcd": 0}),
]

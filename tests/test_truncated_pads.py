"""CPU check of the gadgets in pad_cases.py: the hash that the evaluator takes
at the named gate gives other digits from its leading limbs than from all of
them (so a kernel that missed the case would return other labels)."""

from __future__ import annotations

import re
import os

import pytest

from oracle import oracle as O
from pad_cases import PAD_CASES

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _pad_limbs():
    """kPadLimbs of the library's plan: limbs that a word with r words after it is taken from."""
    with open(os.path.join(ROOT, "paper_2506_14489_amd", "csrc", "plan.hpp")) as f:
        m = re.search(r"kPadLimbs\[6\] = \{([0-9, ]+)\}", f.read())
    return [int(v) for v in m.group(1).split(",")]


def _digits(V: int, m: int, limbs=None):
    """The pad's packed words as base-m numbers, from the fraction V / 2^256
    (limbs: for every word only so many of the top 32-bit limbs, products and
    fraction cut below them)."""
    lam, g = O.lam(m), 32 // (m - 1).bit_length()
    W = -(-lam // g)
    out = []
    for w in range(W):
        n = g if w + 1 < W else lam - (W - 1) * g
        if limbs:
            keep = 256 - 32 * limbs[W - 1 - w]
            V = V >> keep << keep
        V *= m ** n
        out.append(V >> 256)
        V &= (1 << 256) - 1
    return out


@pytest.mark.parametrize("name", PAD_CASES)
def test_the_leading_limbs_give_other_digits(name):
    moduli, S, seed, hits = PAD_CASES[name]
    limbs = _pad_limbs()
    op = O.make_params(list(moduli), list(S), 1, seed)
    gates = O.gate_list(op)
    for a, g, x in hits:
        src, dst = gates[g][0], gates[g][1]
        q, m = moduli[src], moduli[dst]
        A = O.trace(op, a, x)["ev_in"][g][: O.lam(q)]
        V = O.hash_parts(q, m, A, seed, a * len(gates) + g)[2]
        V = sum(int(v) << (32 * l) for l, v in enumerate(V))
        full = _digits(V, m)
        # the full digits are the hash's
        h = [int(d) for d in O.hash_label(q, m, A, seed, a * len(gates) + g)]
        got, per = [], 32 // (m - 1).bit_length()
        for w, D in enumerate(full):
            n = min(per, len(h) - w * per)
            got += [D // m ** (n - 1 - j) % m for j in range(n)]
        assert got == h
        assert _digits(V, m, limbs) != full, (name, a, g)

"""Gadgets in which a pad taken from the leading limbs of the hash alone would
be wrong (a carry out of the left-out limbs reaches a digit: about one pad in
10^6), so that the kernels have to notice it and take all limbs.

Found by search over gadget indices with the oracle's hash.  Per base: moduli,
scaling set, seed, and (gadget, gate, x): with the input x the evaluator hashes
such a label at that gate; the garbler hashes it among the gate's labels.  The
gates cover every place a digit label comes from in the one-gadget-per-lane
evaluator (input, output, working storage, the block's own register slot) and
both kinds of free operation.  test_truncated_pads.py checks each on the CPU.
"""

PRIMES_12 = (2, 3, 5, 7, 11, 13, 17, 19, 23, 29, 31, 37)

PAD_CASES = {
    "12primes-by-31-37": (PRIMES_12, (10, 11), 501, [
        (4167, 0, 70466450130),       # 31 -> 37, the input label
        (36876, 9, -1458108801533),   # 31 -> 23
        (27046, 19, -1359938076086),  # 37 -> 23, an output label
        (44872, 15, -3585498194274),  # 37 -> 11
        (6093, 43, -1765046340000),   # 5 -> 11, a working label
        (11316, 44, 2590167994107),   # 5 -> 13
        (15311, 73, 1374347342273),   # 17 -> 23
        (3870, 83, -1659922546565),   # 23 -> 37, added to an accumulator
        (23869, 65, -1193292591419),  # 11 -> 37
    ]),
    "3-23-37-97-by-3": ((3, 23, 37, 97), (0,), 503, [
        (1217, 3, -115603),           # 23 -> 37, the block's own first target
        (38256, 3, 115020),
        (53973, 3, 115565),
        (26179, 1, 83572),            # 3 -> 37
        (31848, 2, 18608),            # 3 -> 97 (no byte table)
        (211, 4, -107650),            # 23 -> 97
        (7873, 6, -63522),            # 37 -> 97
    ]),
    "short-by-32": ((32, 97, 107), (0,), 502, [
        (1672, 0, 148512),            # 32 -> 97
        (7329, 1, 7379),              # 32 -> 107
        (143907, 2, -6964),           # 97 -> 107
        (199703, 2, -125600),
    ]),
}

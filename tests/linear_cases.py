"""Layers whose path through the layer kernels the tests name: the GPU tests
run them, and the CPU test of the host plan checks that each still takes the
path it stands for."""

from __future__ import annotations

from paper_2506_14489_amd import workloads as WL


def _conv(name, seed, in_shape, c_out, stride=1):
    return WL._conv(name, WL.PRIMES_12, (11,), seed, in_shape, c_out, 3, stride, 1)


# Small layers, compared word for word.  The names of the flattened and the
# folded ones say which path they are for.
SMALL = [
    # name, moduli, (batch, c_in, h, w), c_out, kh, kw, stride, pad
    ("conv3x3-12primes", tuple(WL.PRIMES_12), (2, 5, 6, 7), 3, 3, 3, 1, 1),
    ("conv3x3-wide-row", (2, 3, 5, 7, 11), (1, 16, 3, 70), 8, 3, 3, 1, 1),
    ("conv-stride2", (3, 5, 7, 32), (1, 20, 9, 18), 6, 3, 3, 2, 1),
    ("stem-like-7x7s2", (5, 7, 11), (1, 3, 20, 21), 9, 7, 7, 2, 3),
    ("conv-chunks-and-groups", (2, 251), (1, 130, 3, 4), 70, 3, 3, 1, 1),
    ("conv-1x1-stride2", (13, 16, 17), (2, 17, 6, 6), 5, 1, 1, 2, 0),
    ("conv-2x3-nopad", (4, 5, 7), (1, 4, 5, 6), 3, 2, 3, 1, 0),
    ("dense", tuple(WL.PRIMES_12), (33, 100, 1, 1), 70, 1, 1, 1, 0),
    ("dense-batch1", (32, 167, 173), (1, 512, 1, 1), 10, 1, 1, 1, 0),
    ("short-base-conv", (32, 97, 107), (1, 64, 5, 5), 64, 3, 3, 1, 1),
    # one 64-channel chunk: the kernel with independent waves, 3x3 paths
    ("conv3x3-64ch-ragged-tiles", (3, 5, 7, 11, 13), (1, 64, 4, 70), 8, 3, 3, 1, 1),
    ("conv3x3-64ch-stride2", (2, 3, 5, 7), (2, 64, 9, 20), 6, 3, 3, 2, 1),
    ("conv3x3-64ch-m251-three-groups", (2, 251), (1, 64, 5, 9), 130, 3, 3, 1, 1),
    ("conv3x3-64ch-whole-tiles", (5, 7, 64), (1, 64, 3, 64), 64, 3, 3, 1, 1),
    # kernels one column wide and taller than one row (the tap's row and column
    # from one division by kw = 1), and one row high
    ("conv-3x1", (2, 3, 5, 7), (1, 20, 9, 7), 6, 3, 1, 1, 0),
    ("conv-5x1-two-chunks", (3, 4, 5, 13), (2, 119, 9, 6), 5, 5, 1, 1, 0),
    ("conv-2x1-stride3-two-chunks", (3, 4, 5, 13), (2, 119, 9, 6), 5, 2, 1, 3, 0),
    ("conv-1x3", (2, 3, 5, 7, 11), (1, 33, 5, 12), 9, 1, 3, 1, 0),
    # several 64-channel chunks, 3x3, rows of at most 16 outputs: the next
    # chunk's weights are loaded into registers while a stage computes
    ("conv3x3-three-chunks-7x7", (2, 3, 5, 7, 37), (1, 192, 7, 7), 64, 3, 3, 1, 1),
    ("conv3x3-two-chunks-stride2", (3, 5, 7, 31), (1, 128, 14, 14), 70, 3, 3, 2, 1),
    # flattened tiles (3x3 stride 1 over several chunks)
    ("flat-narrow-batch2-ragged", (2, 3, 5, 7, 37), (2, 128, 5, 6), 70, 3, 3, 1, 1),
    ("flat-narrow-nopad-m251", (3, 5, 251), (2, 130, 9, 8), 9, 3, 3, 1, 0),
    # flattened 32-position tiles, ragged last tiles, up to 38 plane columns; 1 to
    # 16 output channel groups
    ("flat-32-one-group", (223, 227, 229, 233, 239, 241, 251), (2, 65, 20, 34), 3, 3, 3, 1, 1),
    ("flat-32-36-columns", (223, 227, 229, 233, 239, 241, 251), (4, 65, 9, 36), 2, 3, 3, 1, 1),
    ("flat-two-groups", (2, 3, 5, 7, 11, 13), (1, 65, 4, 5), 128, 3, 3, 1, 1),
    ("flat-three-groups", (2, 3, 37), (1, 70, 4, 5), 190, 3, 3, 1, 1),
    ("flat-four-groups", (3, 8, 13), (1, 65, 3, 5), 250, 3, 3, 1, 1),
    ("flat-eight-groups", (2, 251), (1, 65, 3, 4), 510, 3, 3, 1, 1),
    ("flat-sixteen-groups", (5,), (1, 66, 3, 4), 1000, 3, 3, 1, 1),
    ("flat-wide-rows", (3, 5), (2, 65, 8, 20), 130, 3, 3, 1, 1),
    ("no-flat-39-plane-columns", (5, 7), (1, 65, 3, 37), 4, 3, 3, 1, 1),
    # column fold (fewer than 16 channels, kw c_in <= 64: kh x 1 over kw c_in channels)
    ("fold-48-channels-stride4-rows", (3, 16, 251), (1, 12, 9, 18), 70, 3, 4, 4, 0),
    ("fold-32-rows-16-channels", (2, 3), (1, 8, 40, 9), 3, 32, 2, 1, 0),
    ("fold-63-channels-m251", (2, 251), (1, 9, 11, 13), 5, 7, 7, 1, 3),
    ("fold-63-channels-stride2", (2, 251), (1, 9, 11, 13), 5, 7, 7, 2, 3),
    ("fold-one-channel-5x5", (3, 5, 7, 11), (2, 1, 9, 23), 4, 5, 5, 1, 2),
    ("fold-1x4-stride3", (2, 3, 5, 7), (1, 2, 4, 17), 6, 1, 4, 3, 0),
    ("no-fold-65-channels", (5, 7), (1, 13, 6, 8), 3, 5, 5, 1, 2),
    # the staged windows of a 16-position tile: 512 pieces, and 576
    ("fold-8x7-last", (2, 251), (1, 8, 12, 11), 5, 8, 7, 1, 3),
    ("no-fold-9x7", (2, 251), (1, 8, 12, 11), 5, 9, 7, 1, 3),
    # windows apart from each other (columns between them and past the last are
    # not in the planes), one output column
    ("fold-8x8-stride8", (2, 3, 5, 251), (2, 3, 24, 33), 9, 8, 8, 8, 0),
    ("fold-2x6-stride21", (3, 7, 16), (2, 5, 9, 28), 3, 2, 6, 21, 1),
    ("fold-4x4-stride4-one-column", (5, 11), (3, 8, 17, 1), 6, 4, 4, 4, 3),
]

# 3x3 layers over several channel chunks at full size: (workload, what the
# plan has to say), one for each form of the kernel.  word_split 0: each modulus
# has one workgroup per tile and channel group, 1: each packed word has one;
# og_xcd 1: the channel groups are dealt to the XCDs.
def _form(flat, xt, word_split, og_xcd=0):
    return {"flat": flat, "xt": xt, "word_split": word_split, "og_xcd": og_xcd}


SEVERAL_CHUNKS = [
    (_conv("rows-modulus-39-columns", 32, (1, 128, 56, 56), 64), _form(0, 16, 0)),
    (_conv("rows-modulus-stride2", 33, (8, 128, 28, 28), 256, 2), _form(0, 16, 0)),
    (_conv("rows-modulus", 34, (2, 96, 32, 32), 96), _form(0, 16, 0)),
    (_conv("rows-word", 35, (1, 128, 16, 16), 128), _form(0, 16, 1)),
    (_conv("flat16-modulus", 36, (16, 96, 5, 5), 320), _form(1, 16, 0)),
    (_conv("flat16-word", 37, (4, 128, 7, 7), 128), _form(1, 16, 1)),
    (_conv("flat16-word-dealt-8", 38, (1, 256, 5, 5), 512), _form(1, 16, 1, 1)),
    (_conv("flat32-modulus", 39, (4, 96, 30, 30), 96), _form(1, 32, 0)),
    (_conv("flat32-word", 31, (2, 128, 28, 28), 128), _form(1, 32, 1)),
    (_conv("flat32-word-dealt-2", 40, (1, 512, 20, 20), 96), _form(1, 32, 1, 1)),
    (_conv("flat32-word-dealt-4", 41, (1, 256, 14, 14), 256), _form(1, 32, 1, 1)),
    (_conv("flat32-word-dealt-8", 42, (2, 96, 7, 7), 512), _form(1, 32, 1, 1)),
]

"""The deal of a batch as the dealt launch makes it, on the host, and the
batches whose coverage rests on it."""

import math

import numpy as np


def deal(lengths, H_Q, H_KV, cus=256):
    """The dealt launch's cuts: tiles a workgroup takes, the pieces of each
    sequence, the most sequences a workgroup passes and the most 32-key tiles
    between a wave's first and last one of a sequence (in pages of 32 keys)."""
    g = H_Q // H_KV
    hpt = next(h for h in range(min(g, 32), 0, -1) if g % h == 0)
    groups = max(1, cus // (H_Q // hpt))
    T = [max(1, -(-n // 32)) for n in lengths]
    total, top = sum(T), max(T)
    floor = max(4, int(np.float32(0.7 if hpt <= 16 else 1.1) * np.float32(math.sqrt(top))))
    per = max(-(-total // groups), -(-top // 63), floor)
    starts = np.concatenate([[0], np.cumsum(T)])
    pieces = [int((starts[b] + T[b] - 1) // per - starts[b] // per + 1) for b in range(len(T))]
    passed = pages = 0
    waves = 2 if hpt <= 16 else 4
    for lo in range(0, total, per):
        hi = min(lo + per, total)
        parts = [min(hi, starts[b] + T[b]) - max(lo, starts[b]) for b in range(len(T))]
        parts = [int(n) for n in parts if n > 0]
        passed = max(passed, len(parts))
        # contiguous parts, or alternate tiles of the whole part (two waves, key rows of at most 1 KiB)
        pages = max(pages, max(parts) if waves == 2 and H_KV <= 4 else max(parts) // waves)
    return {"per": per, "pieces": pieces, "passed": passed, "pages": pages, "hpt": hpt}


# (H_Q, H_KV, lengths)
CASES = [
    (8, 1, [1]),                                          # one tile
    (8, 1, [0, 0, 0]),                                    # nothing to read
    (8, 1, [31, 32, 33, 0, 1, 64, 0]),                    # tile edges, empty sequences between
    (64, 8, [512]),                                       # one sequence over many workgroups
    (8, 1, [9000]),                                       # 26 pieces of 11 tiles
    (8, 1, [9000, 5, 0, 4100, 31]),                       # long and short in turn
    (32, 4, [3000, 17, 0, 900, 2100, 64]),                # head, whole and tail pieces in one workgroup
    (16, 2, [int(x) for x in np.random.default_rng(7).integers(0, 300, 200)]),   # several windows of 64 sequences
    (16, 16, [700, 33, 1200]),                            # one head per KV head
    (32, 1, [300, 40, 511, 2000]),                        # 32-head tiles (two column tiles, four waves)
    (128, 2, [700, 33, 1500]),                            # 32-head tiles, two readers per KV head
    (66, 2, [130, 700, 31]),                              # 33-head groups: three readers per KV head
    (12, 4, [300, 95]),                                   # group of 3
]

# One sequence cut into as many pieces as the merge holds.
MOST_PIECES = (8, 1, [300, 70560])

# On a stream of 64 CUs, in 32-key pages: a wave's part of one sequence passes
# the 64 page ids it holds at a time, and the next sequence's does again.
# Alternate tiles (key rows of 256 bytes) and contiguous parts (2 KiB).
PAGE_WINDOWS_CUS = 64
PAGE_WINDOWS = [(8, 1, [200000, 1000, 85000]), (64, 8, [30000, 9000])]

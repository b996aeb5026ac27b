"""Which entries the finishing kernel of block minima asks for, by a model of the blocks on the host: every slot of a block is
an entry of the padded cache, each entry is in one block, and a block that holds an entry may hold slots past the last one.  The
stored rows end with the last entry, so a kernel that re-scores whole blocks has to bound every slot's row, as rescore_rows8
does."""
import os
import re

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))), "paper_2002_02645_amd", "csrc")


def _first_entry():
    """block_first_entry as the source has it."""
    text = open(os.path.join(CSRC, "aux_kernels.hip")).read()
    body = re.search(r"block_first_entry\(int blk\)\s*\{\s*return ([^;]*);", text).group(1).replace("kTileN", "256")
    assert re.fullmatch(r"[\sblk0-9()&>*+]*", body)
    return lambda blk: eval(body, {"__builtins__": {}}, {"blk": blk})   # noqa: S307 (digits, brackets and blk alone)


def _entry(first, slot_block, e):
    return first(slot_block) + (e & 3) + (e >> 2 & 1) * 16


@pytest.mark.parametrize("n", [1, 3, 4, 5, 15, 16, 17, 19, 20, 21, 31, 32, 33, 255, 256, 257, 300, 2000, 2016, 20011, 50000])
def test_slots_of_blocks_with_an_entry(n):
    first = _first_entry()
    n_pad = -(-n // 256) * 256
    of = np.array([[_entry(first, blk, e) for e in range(8)] for blk in range(n_pad // 8)])
    assert np.array_equal(np.sort(of.ravel()), np.arange(n_pad))     # each entry once
    held = (of < n).any(1)
    assert np.array_equal(held, of[:, 0] < n)                        # a block's first slot is an entry where any is
    past = of[held] >= n
    assert past.any() == (n % 32 != 0)       # ... and others are not, unless the cache ends with a group of four blocks
    clamped = np.where(of[held] < n, of[held], n - 1)
    assert clamped.min() >= 0 and clamped.max() < n

"""Sizes of the depth sort's bins (csrc/sort.hip): the sampled splitters
emulated on the distances of uniform scenes, with the sort's own constants.
Every bin has to fit a workgroup: one that does not is sorted in memory, at
many times the cost of all the others."""
import os
import re

import numpy as np
import pytest

SRC = open(os.path.join(os.path.dirname(os.path.abspath(__file__)), "..", "paper_2511_22793_amd", "csrc", "sort.hip")).read()


def _const(name):
    """The constant's value: a product of numbers, shifts and other constants."""
    text = re.search(r"constexpr int %s = ([^;]+);" % name, SRC).group(1)
    return int(eval(re.sub(r"[A-Z]\w+", lambda m: str(_const(m.group(0))), text), {"__builtins__": {}}))


ONE, MAX, MAX_BINS, BIN, OVER, CAP = (_const("DS_" + k) for k in ("ONE", "MAX", "MAX_BINS", "BIN", "OVER", "CAP"))


def _largest_bin(key):
    n = len(key)
    bins = 16
    while bins < MAX_BINS and n // bins > BIN:
        bins *= 2
    m = OVER * bins
    i = np.arange(m, dtype=np.uint64)
    h = (i * np.uint64(0x9E3779B1)) & np.uint64(0xFFFFFFFF)
    at = i * np.uint64(n) // np.uint64(m) + ((h * np.uint64(n // m)) >> np.uint64(32))
    full = (key.view(np.uint32).astype(np.uint64) << np.uint64(32)) | np.arange(n, dtype=np.uint64)
    split = np.sort(full[at.astype(np.int64)])[::OVER]
    return int(np.bincount(np.searchsorted(split[1:], full, side="right"), minlength=bins).max())


def _distances(rng, n):
    """FP32 distances of n means uniform in a 10 x 10 x 3 room to a receiver in it."""
    p = rng.random((3, n), dtype=np.float32) - rng.random((3, 1), dtype=np.float32)
    p *= np.array([[10.0], [10.0], [3.0]], np.float32)
    return np.sqrt((p * p).sum(0, dtype=np.float32))


@pytest.mark.parametrize("n", [ONE + 1, 20_000, 163_840, 327_680, 400_000, 500_000, MAX])
def test_every_bin_fits_a_workgroup(n):
    rng = np.random.default_rng(n)
    assert max(_largest_bin(_distances(rng, n)) for _ in range(48 if n > 300_000 else 24)) <= CAP


def test_largest_sizes_leave_room():
    # a bin between OVER samples of uniform rank is close to a gamma variable
    # of shape OVER: the chance that one of the bins passes the limit
    mean = max(MAX / MAX_BINS, float(BIN))
    x = OVER * CAP / mean
    tail = np.exp(-x) * sum(x ** k / float(np.prod(range(1, k + 1)) or 1) for k in range(OVER))
    assert MAX_BINS * tail < 1e-5

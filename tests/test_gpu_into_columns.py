"""dmi_observe_into with request tables that are too long for the launch's arguments as they are: columns whose values are evenly
spaced travel as a start and a step, the others as lists (832 words in all), and what does not fit that either is staged.  On
both sides of each line, in every kernel that reads such a table: the records are dmi_observe's byte for byte."""
import numpy as np
import pytest
import torch

from workloads import prng

from test_gpu_into_tables import B, DEV, _both  # noqa: F401  (the fixture and the comparison)

pytestmark = pytest.mark.gpu


def _ids(n, how, rng):
    return {"even": 5000 + 3 * np.arange(n), "falling": 0xFFFFFFF0 - 7 * np.arange(n, dtype=np.int64) % (1 << 32),
            "listed": rng.permutation(1 << 20)[:n]}[how]


@pytest.mark.parametrize("n", [167, 277, 278, 416, 417, 832, 833, 1024])
@pytest.mark.parametrize("ids", ["even", "falling", "listed"])
@pytest.mark.parametrize("rows", ["in_order", "strided", "slots"])
def test_one_row_per_request(B, n, ids, rows):  # noqa: F811
    rng = np.random.default_rng(n)
    x = prng.randn_bf16(n, 2100 * 512, DEV).view(2100, 512)
    at = {"in_order": 5 + np.arange(n), "strided": 2 * np.arange(n), "slots": rng.permutation(2100)[:n]}[rows]
    reqs = np.stack([_ids(n, ids, rng), at // 2, at - at // 2, np.ones(n, int), 1 + np.arange(n) % 3], axis=1) & 0xFFFFFFFF
    _both(B, x, reqs, summary_mask=5)                                       # the decode-shaped kernel
    reqs[:, 4] = 1
    _both(B, x.float(), reqs, out_dtype=3)                                  # capture_rows_kernel
    _both(B, x[:, :40], reqs, out_dtype=4, summary_mask=2)                  # the general kernel, short rows
    keep = rng.integers(0, 2, n)
    _both(B, x, reqs, keep=keep)
    _both(B, x[:, 3:], reqs, out_dtype=2, keep=keep)
    _both(B, x, reqs, index=rng.permutation(2100)[:n])


@pytest.mark.parametrize("n", [167, 277, 278, 500, 833])
@pytest.mark.parametrize("counts", ["equal", "listed"])
def test_several_rows_per_request(B, n, counts):  # noqa: F811
    rng = np.random.default_rng(n)
    x = prng.randn_bf16(n, 6000 * 128, DEV).view(6000, 128)
    count = np.full(n, 3) if counts == "equal" else rng.integers(0, 7, n)
    first = np.concatenate([[0], np.cumsum(count)[:-1]])
    reqs = np.stack([rng.permutation(1 << 20)[:n], first, np.zeros(n, int), count, np.ones(n, int)], axis=1)
    index = rng.permutation(6000)[:int(count.sum())]
    for keep in (None, rng.integers(0, 2, n)):
        _both(B, x, reqs, keep=keep)
        _both(B, x.float(), reqs, out_dtype=0, summary_mask=7, keep=keep)
        _both(B, x, reqs, out_dtype=4, index=index, keep=keep)

"""Top-k's short ways on the GPU: one wave that finishes a digit's few keys, and long rows cut into parts, against the oracle or
numpy's stable sort, at the sizes and values where they hand over to the general form."""
import numpy as np
import pytest
import torch

from paper_2605_28213_amd import gemm, topk
from tests.test_topk_gpu import check, run_state

pytestmark = pytest.mark.gpu


def rows(kind, batch, n, ld, rng):
    x = rng.standard_normal((batch, ld)).astype(np.float32)
    if kind == "steps":                       # many elements equal the threshold
        x = np.round(x * 2) / 2
    elif kind == "zeros":                     # one value, of both signs
        x = np.where(x > 0, np.float32(0.0), np.float32(-0.0))
    elif kind == "ascending":                 # the large values are neighbours
        x[:, :n] = np.sort(x[:, :n], axis=1)
    elif kind == "close":                     # keys that differ in their last bits only
        x = (np.float32(1.0) + rng.integers(0, 600, x.shape) * np.float32(2.0 ** -23)).astype(np.float32)
    elif kind == "infinite":
        x[:, ::3] = -np.inf
        x[:, 5::1009] = np.inf
    elif kind == "lowest":
        x[:] = np.finfo(np.float32).min
        x[:, 3::97] = rng.standard_normal(x[:, 3::97].shape)
    x[:, n:] = 1e30
    return x


KINDS = ["normal", "steps", "zeros", "ascending", "close", "infinite", "lowest"]


@pytest.mark.parametrize("kind", KINDS)
@pytest.mark.parametrize("n,k", [(5, 2), (600, 511), (3001, 1), (4096, 2048), (4099, 700), (9001, 4000)])
def test_resident_rows(kind, n, k):
    """At most and more than 512 keys in the first digit, rows that leave lanes without elements, four and sixteen keys a lane."""
    check(2, rows(kind, 2, n, (n + 3) // 4 * 4, np.random.default_rng(n + k)), n, k)


def by_sort(x, n, k):
    order = np.argsort(-(x[:, :n].astype(np.float64) + 0.0), axis=1, kind="stable")[:, :k]
    return np.sort(order, axis=1)

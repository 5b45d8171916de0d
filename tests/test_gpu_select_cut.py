"""Branch-point selection through the bound from the threads' maxima and through
the radix select, against the oracle: exact in positions, scores and order."""
import numpy as np
import pytest
import torch

from oracle import hdl_oracle as O
from tests.gpu_helpers import require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hdl():
    return require_gpu()


def _check(hdl, lo, hi, mask, k):
    oi, osc, oc = O.select_branch_points(lo, hi, mask, k)
    idx, score, count, _ = hdl.select_branch_points(torch.from_numpy(lo).cuda(), torch.from_numpy(hi).cuda(),
                                                    None if mask is None else torch.from_numpy(mask).cuda(), k)
    assert np.array_equal(count.cpu().numpy(), oc)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(score.cpu().numpy(), np.asarray(osc, np.float32))


# fewer positions than threads, one each, more; the longest root that is held
# in LDS and one more; k at the edges of the orderings (64, 256 collected
# positions) and of the bound (128; 512 on long roots)
@pytest.mark.parametrize("T", [1, 63, 1024, 1025, 5000, 16384, 32768, 32769])
@pytest.mark.parametrize("k", [1, 64, 128, 129, 256, 257, 512, 513, 1024])
def test_edges(hdl, T, k):
    rng = np.random.default_rng(T * 1031 + k)
    lo = rng.standard_normal((2, T)).astype(np.float32)
    hi = rng.standard_normal((2, T)).astype(np.float32)
    mask = (rng.random((2, T)) < 0.7).astype(np.uint8)
    _check(hdl, lo, hi, mask, min(k, T))


# scores in order (the largest all in one thread's or one wave's range), a few
# distinct scores with more ties than slots, all equal, few candidates,
# subnormal and zero scores
@pytest.mark.parametrize("kind", ["up", "down", "stride", "ties", "equal", "few", "tiny"])
@pytest.mark.parametrize("T,k", [(3000, 8), (32768, 32), (32768, 512), (40000, 100)])
def test_orders_and_ties(hdl, kind, T, k):
    rng = np.random.default_rng(T + k)
    t = np.arange(T, dtype=np.float32)
    d = {"up": t, "down": T - t, "stride": np.where(t % 1024 == 5, 100 + t, rng.random(T)),
         "ties": np.floor(rng.random(T) * 4), "equal": np.ones(T), "few": t,
         "tiny": np.where(t % 3 == 0, 0, (t % 1000) * 1e-42)}[kind].astype(np.float32)
    mask = np.ones((1, T), np.uint8)
    if kind == "few":
        mask[:] = 0
        mask[0, rng.choice(T, k // 2 + 1, replace=False)] = 1
    _check(hdl, np.zeros((1, T), np.float32), d[None], mask, k)


# scores within a per cent of each other (next-token entropies near ln V), and
# many positions at exactly the k-th score: with fewer than k above it, with k
# and more above it in a few threads' positions only, and at both ends of a wave's
# range
@pytest.mark.parametrize("kind", ["narrow", "one narrow", "plateau", "hidden above", "two plateaus"])
@pytest.mark.parametrize("T,k", [(300, 8), (300, 128), (1024, 100), (1025, 64), (8192, 8), (8192, 128), (20000, 512),
                                 (32768, 32), (40000, 100)])
def test_narrow_and_plateaus(hdl, kind, T, k):
    rng = np.random.default_rng(T + k)
    v = 11.90 + 0.03 * rng.random((2, T))
    if kind == "one narrow":
        v[:, rng.integers(0, T, 3)] = (-4.0, 1e-30, 90.0)
    elif kind == "plateau":
        v = np.where(rng.random((2, T)) < 0.5, 2.5, rng.random((2, T)))
        v[:, rng.choice(T, k // 2, replace=False)] = 3.0 + rng.random((2, k // 2))
    elif kind == "hidden above":   # (positions 1024 apart belong to one thread)
        v = np.full((2, T), 2.5)
        v[:, np.arange(T) % 1024 < 4] = 7.0
    elif kind == "two plateaus":
        v = np.where(np.arange(T) % 7 < 3, 2.5, -2.5) * np.ones((2, 1))
        v[1] = -v[0]
    v = v.astype(np.float32)
    mask = (rng.random((2, T)) < 0.9).astype(np.uint8)
    oi, osc, oc = O.select_by_value(v, mask, k)
    idx, score, count = hdl.select_top_k(torch.from_numpy(v).cuda(), torch.from_numpy(mask).cuda(), k)
    assert np.array_equal(count.cpu().numpy(), oc)
    assert np.array_equal(idx.cpu().numpy(), oi)
    assert np.array_equal(score.cpu().numpy(), np.asarray(osc, np.float32))

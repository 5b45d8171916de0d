"""fp32 operands, multiplied as three bf16 pieces each: against the float64
oracle at fp32's own rounding, and with values that the split cannot take
(infinities, values that round to infinity in bf16), which leave the other rows'
bits alone, or whose pieces are zero or denormal."""
import numpy as np
import pytest
import torch

from oracle import hdl_oracle as O
from tests.gpu_helpers import as_f64, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hdl():
    return require_gpu()


def _inputs(n, d, V, seed=11):
    g = torch.Generator().manual_seed(seed)
    return (torch.randn(n, d, generator=g), torch.randn(V, d, generator=g) * 0.05,
            torch.randint(0, V, (n,), generator=g, dtype=torch.int32))


# row tiles of 64, 128 and 256 rows; whole K-slices, a K tail, rows shorter
# than a slice; one ragged vocabulary tile, several
@pytest.mark.parametrize("n", [1, 64, 100, 300])
@pytest.mark.parametrize("d,V", [(256, 1500), (72, 300), (8, 5000), (1024, 700)])
def test_fp32_rounding(hdl, n, d, V):
    H, W, y = _inputs(n, d, V)
    logp, lse = hdl.token_logprobs(H.cuda(), W.cuda(), y.cuda())
    ref_p, ref_l = O.token_logprobs(as_f64(H), as_f64(W), y.numpy())
    # what d fp32 additions in any order can lose of a logit (u = 2^-24 each,
    # what the split leaves out of the products counted as one more), plus the normaliser's
    # exp, sum and log: 64 u of the result's size
    mag = (as_f64(H)[:, None, :].__abs__() * np.abs(as_f64(W))[None]).sum(2).max(1)
    tol = 2.0 ** -24 * ((d + 1) * mag + 64 * (1 + np.abs(ref_l)))
    assert (np.abs(lse.cpu().double().numpy() - ref_l) <= tol).all()
    assert (np.abs(logp.cpu().double().numpy() - ref_p) <= 2 * tol).all()


# a weight of -inf meets hidden values whose lower pieces are zero (1.0): its
# word's probability is 0 and nothing else changes.  Weights at both sides of the
# split's limit (2^60) times small hidden values, the smallest of them denormal.
@pytest.mark.parametrize("weight,h", [(-float("inf"), 1.0), (3.4e38, 1e-38), (2.0 ** 60, 3e-18), (1.1e18, 3e-18),
                                      (-3.4e38, 2.0)])
@pytest.mark.parametrize("col", [0, 37, 71])
@pytest.mark.parametrize("n", [50, 257])
def test_weights_beyond_the_split(hdl, n, col, weight, h):
    H, W, y = _inputs(n, 72, 600)
    H[:, col] = h
    W[:, col] = 0.0
    rows = [3, 130, 599]
    W[rows, col] = weight
    y[y == 3] = 4
    y[(y == 130) | (y == 599)] = 5
    logp, lse = hdl.token_logprobs(H.cuda(), W.cuda(), y.cuda())
    keep = np.ones(600, bool)
    z = as_f64(H) @ np.where(np.isinf(as_f64(W)), 0.0, as_f64(W)).T
    if h >= 1.0:
        keep[rows] = False   # z = -inf or about -7e38
    z = z[:, keep]
    m = z.max(1)
    ref_l = m + np.log(np.exp(z - m[:, None]).sum(1))
    ref_p = (as_f64(H) * as_f64(W)[y.numpy()]).sum(1) - ref_l
    tol = 2.0 ** -24 * (80 * 30 + 64 * (1 + np.abs(ref_l)))
    assert (np.abs(lse.cpu().double().numpy() - ref_l) <= tol).all()
    assert (np.abs(logp.cpu().double().numpy() - ref_p) <= 2 * tol).all()


def test_infinite_hidden_and_positive_infinite_weight(hdl):
    H, W, y = _inputs(130, 64, 300)
    H[7, 3] = float("inf")
    logp, lse = hdl.token_logprobs(H.cuda(), W.cuda(), y.cuda())
    clean, _ = hdl.token_logprobs(H[8:].cuda(), W.cuda(), y[8:].cuda())
    assert torch.isnan(logp[7]) and torch.isnan(lse[7])
    assert torch.equal(logp[8:], clean)
    H[7, 3] = 1.0
    W[9, 5] = float("inf")
    H[:, 5] = 1.0
    logp, lse = hdl.token_logprobs(H.cuda(), W.cuda(), y.cuda())
    assert torch.isnan(logp).all() and torch.isnan(lse).all()


# a row's results have the same bits whatever the other rows hold: rows that
# the split cannot take, in the first, a middle and the last fragment of a tile
# (of 64, 128 and 256 rows), with and without weights that it cannot take
@pytest.mark.parametrize("n", [50, 100, 300])
@pytest.mark.parametrize("value", [float("inf"), float("nan"), 2.0 ** 60, -3.4e38])
@pytest.mark.parametrize("weight", [0.01, 2.0 ** 61])
def test_rows_do_not_depend_on_each_other(hdl, n, value, weight):
    H, W, y = _inputs(n, 72, 600)
    W[[3, 130, 599], 30] = weight
    H[:, 30] = 1e-19
    ref = hdl.token_logprobs(H.cuda(), W.cuda(), y.cuda(), None, want_entropy=True)
    bad = [0, 21, n - 1]
    for r, c in zip(bad, (0, 40, 71)):
        H[r, c] = value
    got = hdl.token_logprobs(H.cuda(), W.cuda(), y.cuda(), None, want_entropy=True)
    keep = torch.ones(n, dtype=torch.bool)
    keep[bad] = False
    for a, b in zip(ref, got):
        assert torch.isfinite(a).all()
        assert torch.equal(a.cpu()[keep], b.cpu()[keep])


# such a row itself: the fp32 MFMA's results for it, one word far above the rest
@pytest.mark.parametrize("n", [50, 300])
def test_large_rows(hdl, n):
    H, W, y = _inputs(n, 72, 600)
    W[:, 40] = -1e-30 * (1 + torch.arange(600) % 7)
    H[5, 40] = 1e30   # logits between about -7 and -1 from this column
    ref_p, ref_l = O.token_logprobs(as_f64(H), as_f64(W), y.numpy())
    logp, lse = hdl.token_logprobs(H.cuda(), W.cuda(), y.cuda())
    tol = 2.0 ** -24 * (80 * 30 + 64 * (1 + np.abs(ref_l)))
    assert (np.abs(lse.cpu().double().numpy() - ref_l) <= tol).all()
    assert (np.abs(logp.cpu().double().numpy() - ref_p) <= 2 * tol).all()

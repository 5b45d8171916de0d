"""Row tiles of 64, 128 and 256 token rows (narrow ones for the last rows of a
call and for calls with few rows) against the float64 oracle, and against each
other: with the same chunking a row has the same bits whatever tile holds it."""
import numpy as np
import pytest
import torch

from oracle import hdl_oracle as O
from tests.gpu_helpers import as_f64, grad_tol, require_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def hdl():
    return require_gpu()


def _inputs(n, d, V, dtype, seed=5):
    g = torch.Generator().manual_seed(seed)
    H = torch.randn(n, d, generator=g).to(dtype)
    W = (torch.randn(V, d, generator=g) * 0.05).to(dtype)
    y = torch.randint(0, V, (n,), generator=g, dtype=torch.int32)
    return H, W, y


# d: whole K-slices, a K tail, rows shorter than one slice (and than a ring
# of them); V: one ragged tile, many tiles
@pytest.mark.parametrize("d,V", [(256, 70000), (200, 3000), (24, 300), (8, 1000)])
@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
def test_row_tile_edges(hdl, d, V, dtype):
    N = 700
    H, W, y = _inputs(N, d, V, dtype)
    ref_p, ref_l = O.token_logprobs(as_f64(H), as_f64(W), y.numpy())
    Hd, Wd, yd = H.cuda(), W.cuda(), y.cuda()
    full = None
    tol = 2e-3 if dtype == torch.bfloat16 else 1e-4
    for n in (700, 1, 16, 63, 64, 65, 127, 128, 129, 192, 255, 256, 257, 320, 321, 383, 384, 385, 448, 511, 512, 513):
        logp, lse, ent = hdl.token_logprobs(Hd[:n], Wd, yd[:n], None, want_entropy=True)
        plain, _ = hdl.token_logprobs(Hd[:n], Wd, yd[:n], None)
        lp = logp.cpu().numpy()
        assert np.abs(lp - ref_p[:n]).max() <= tol, n
        assert np.abs(lse.cpu().numpy() - ref_l[:n]).max() <= tol, n
        assert torch.equal(plain, logp), n
        if full is None:
            full = (logp, lse, ent)
        elif V > 256:   # the same chunking at every n here: one vocabulary tile per chunk
            for a, b in zip(full, (logp, lse, ent)):
                assert torch.equal(a[:n], b), n


@pytest.mark.parametrize("n", [1, 64, 65, 128, 129, 257, 321, 385, 449])
def test_row_tile_edges_backward(hdl, n):
    H, W, y = _inputs(n, 136, 1500, torch.bfloat16, seed=6)
    g = torch.randn(n, generator=torch.Generator().manual_seed(7))
    _, ref_l = O.token_logprobs(as_f64(H), as_f64(W), y.numpy())
    ref_h, ref_w, mag_h, mag_w = O.token_logprobs_backward(as_f64(H), as_f64(W), y.numpy(), g.double().numpy())
    dh, dw = hdl.token_logprobs_backward(H.cuda(), W.cuda(), y.cuda(), None, torch.from_numpy(ref_l).float().cuda(),
                                         g.cuda())
    assert (np.abs(dh.cpu().numpy() - ref_h) <= grad_tol(mag_h)).all()
    assert (np.abs(dw.cpu().numpy() - ref_w) <= grad_tol(mag_w)).all()


# the merge's two numbers of chunk segments at their line (96 chunks of one
# vocabulary tile each): against the oracle, log p and lse with the same bits
# whether the entropy is computed or not
@pytest.mark.parametrize("chunks", [9, 95, 96, 97])
@pytest.mark.parametrize("n", [40, 300])
def test_merge_segments(hdl, chunks, n):
    H, W, y = _inputs(n, 64, 256 * chunks - 3, torch.bfloat16, seed=chunks)
    ref_p, ref_l = O.token_logprobs(as_f64(H), as_f64(W), y.numpy())
    plain = hdl.token_logprobs(H.cuda(), W.cuda(), y.cuda())
    logp, lse, _ = hdl.token_logprobs(H.cuda(), W.cuda(), y.cuda(), None, want_entropy=True)
    assert torch.equal(plain[0], logp) and torch.equal(plain[1], lse)
    assert np.abs(logp.cpu().numpy() - ref_p).max() <= 2e-3 and np.abs(lse.cpu().numpy() - ref_l).max() <= 2e-3


# and its form for many rows (131,072 of the call and more), few of them scored
# or all: every row's segments are one thread's
@pytest.mark.parametrize("masked", [False, True])
@pytest.mark.parametrize("n", [131071, 131077])
def test_merge_many_rows(hdl, n, masked):
    H, W, y = _inputs(n, 16, 256 * 10 - 3, torch.bfloat16, seed=n)
    mask = (torch.rand(n, generator=torch.Generator().manual_seed(n)) < 0.03).to(torch.uint8) if masked else None
    args = (H.cuda(), W.cuda(), y.cuda(), None if mask is None else mask.cuda())
    plain = hdl.token_logprobs(*args)
    logp, lse, _ = hdl.token_logprobs(*args, want_entropy=True)
    assert torch.equal(plain[0], logp) and torch.equal(plain[1], lse)
    on = torch.ones(n, dtype=torch.bool) if mask is None else mask != 0
    assert not logp.cpu()[~on].any() and not lse.cpu()[~on].any()
    at = torch.nonzero(on).view(-1)
    at = torch.cat([at[:300], at[-300:]])
    ref_p, ref_l = O.token_logprobs(as_f64(H[at]), as_f64(W), y[at].numpy())
    assert np.abs(logp.cpu()[at].numpy() - ref_p).max() <= 2e-3 and np.abs(lse.cpu()[at].numpy() - ref_l).max() <= 2e-3

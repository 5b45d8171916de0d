"""fp32 operands are multiplied as products of bf16 pieces.  One-hot hidden rows
make a logit a single product, and a word of logit 0 above all others makes
log p that logit itself, so every product of pieces that the kernel owes is seen
(shown on the CPU by leaving each one out in turn)."""
import pytest
import torch

from tests.gpu_helpers import require_gpu

SIX = [(0, 0), (0, 1), (1, 0), (0, 2), (1, 1), (2, 0)]   # (piece of w, piece of h)


def _values(n, g):
    """n values of 24 significant bits whose second and third bf16 pieces are
    close to the largest there are (2^-8 and 2^-17 of the leading power)."""
    lead = 1 + torch.randint(0, 8, (n,), generator=g).double() * 2.0 ** -7
    x = lead + 2.0 ** -8 - 2.0 ** -17 - torch.randint(1, 40, (n,), generator=g).double() * 2.0 ** -23
    return (x * 2.0 ** torch.randint(0, 4, (n,), generator=g)).float()


def _inputs(n, d, V):
    g = torch.Generator().manual_seed(n * d + V)
    H = torch.zeros(n, d)
    H[torch.arange(n), torch.arange(n) % d] = _values(n, g)
    W = -32 * _values(V * d, g).view(V, d)   # logits of -32 and less beside word 0's 0
    W[0] = 0
    y = torch.randint(1, V, (n,), generator=g, dtype=torch.int32)
    return H, W, y


def _exact(H, W, y):
    return (H.double() * W[y.long()].double()).sum(1)


def _tol(z):
    # u = 2^-24 of z.  Left out: second times third piece twice, 2 x 2^-25 (third
    # times third 2^-34).  The last accumulation keeps the result's 24 bits, cut
    # or rounded: one unit in the last place, 2 u at most.  The sum of the small
    # products before it lies at 2^-6 of z and its roundings at that times as much.
    return 2.0 ** -24 * (3 + 2.0 ** -4) * z.abs()


def _split(x):
    p = []
    for _ in range(3):
        p.append(x.bfloat16().float())
        x = x - p[-1]
    assert not x.any()
    return [q.double() for q in p]


def test_each_product_is_needed():
    H, W, y = _inputs(300, 72, 600)
    h, w = _split(H), _split(W[y.long()])
    z = _exact(H, W, y)

    def off(products):
        s = sum((w[a] * h[b]).sum(1) for a, b in products)
        return (s.float().double() - z).abs() > _tol(z)

    assert not off(SIX).any()
    for p in SIX:
        assert off([q for q in SIX if q != p]).all(), p
    for p in [(0, 1), (0, 2)]:   # a piece paired with the wrong one
        assert off([q for q in SIX if q != p] + [p[::-1]]).any(), p


# row tiles of 64, 128 and 256 rows; whole K-slices, a K tail, rows shorter
# than a slice
@pytest.mark.gpu
@pytest.mark.parametrize("n", [50, 100, 300])
@pytest.mark.parametrize("d,V", [(64, 600), (72, 600), (8, 300)])
def test_single_products(n, d, V):
    hdl = require_gpu()
    H, W, y = _inputs(n, d, V)
    logp, lse = hdl.token_logprobs(H.cuda(), W.cuda(), y.cuda())
    z = _exact(H, W, y)
    assert not lse.cpu().any()
    assert ((logp.cpu().double() - z).abs() <= _tol(z)).all()

"""fp32 products on the 256 x 256 tiles, whose operands are split into three
bf16 planes: K around the K-step and its halves, ragged edges, values whose
parts leave the range of normal numbers, against 64-bit products."""
import pytest
import torch

from gpu_util import gamma
from test_gpu_split import operand, output

pytestmark = pytest.mark.gpu

B, N = 33000, 520                 # fills the chip with large tiles; ragged both ways


def _gs():
    from paper_2608_01528_amd import gramspace
    return gramspace


def bound(a, b, K):
    """Any order of the sum (gamma), 2^-23 per product for the parts left out."""
    return (gamma(K + 8) + 2.0 ** -23) * (a.abs() @ b.abs()) + 1e-36


@pytest.mark.parametrize("K", [4, 15, 16, 17, 33, 100, 259])
def test_planes_products(K):
    gs = _gs()
    X, _ = operand(B, K, torch.float32, 1, "aligned")
    Y, _ = operand(B, K, torch.float32, 2, "aligned")
    Q, _ = operand(N, K, torch.float32, 3, "aligned")
    C, _ = operand(K, N, torch.float32, 4, "aligned")
    x, y, q, c = (t.double() for t in (X, Y, Q, C))
    buf, out = output(B, N, torch.float32, "aligned")
    _, n2 = gs.gs_project(X, Q, out=out, xnorm2=True)
    assert torch.all((out.double() - x @ q.T).abs() <= bound(x, q.T, K))
    assert torch.all((n2.double() - (x * x).sum(1)).abs() <= gamma(K + 8) * (x * x).sum(1))
    assert torch.all(buf[:, N:] == 7.0)
    Tb = gs.gs_project(X, Q, out_dtype=torch.bfloat16)
    assert torch.all((Tb.double() - x @ q.T).abs() <= bound(x, q.T, K) * 1.01 + 2.0 ** -8 * (x @ q.T).abs())
    buf, out = output(B, N, torch.float32, "aligned")
    gs.gs_reconstruct(X, C, out=out)
    assert torch.all((out.double() - x @ c).abs() <= bound(x, c, K))
    assert torch.all(buf[:, N:] == 7.0)
    Z = gs.gs_reconstruct(X, C, T2=Y, bind="mul")
    e1, e2 = bound(x, c, K), bound(y, c, K)
    lim = e1 * (y @ c).abs() + e2 * (x @ c).abs() + e1 * e2
    assert torch.all((Z.double() - (x @ c) * (y @ c)).abs() <= lim + 2.0 ** -23 * ((x @ c) * (y @ c)).abs())
    # scores of a codebook that fits one tile column, norms given and summed here
    R = C[:, :200].T.contiguous() if K % 4 == 0 else operand(200, K, torch.float32, 5, "aligned")[0]
    r = R.double()
    f = 1.0 / (x.norm(dim=1)[:, None] * r.norm(dim=1)[None, :])
    lim = f * bound(x, r.T, K) + (gamma(K + 8) + 1e-6) * (f * (x @ r.T)).abs()
    for given in (False, True):
        S, idx = gs.gs_similarity(X, R, qnorm2=(x * x).sum(1).float() if given else None,
                                  cnorm=r.norm(dim=1).float() if given else None)
        assert torch.all((S.double() - f * (x @ r.T)).abs() <= lim)
        assert torch.all(S.gather(1, idx.long()[:, None])[:, 0] == S.amax(1))


@pytest.mark.parametrize("scale", [1e-37, 1e-30, 1e18, 1e35])
def test_planes_keep_the_range_of_fp32(scale):
    """Rows of tiny and of huge values, beside ordinary ones of the same tile:
    the error bound of an fp32 sum holds for each (2^-149: one unit of the
    smallest numbers)."""
    gs = _gs()
    K = 60
    X, _ = operand(B, K, torch.float32, 6, "aligned")
    Q, _ = operand(N, K, torch.float32, 7, "aligned")
    X[11] *= scale
    X[32990] *= scale
    T = gs.gs_project(X, Q).double()
    x, q = X.double(), Q.double()
    assert torch.all((T - x @ q.T).abs() <= (gamma(K + 8) + 2.0 ** -23) * (x.abs() @ q.T.abs()) + K * 2.0 ** -149)


def test_planes_infinities_and_nan():
    """An infinite input gives the signed infinities of an fp32 product, a NaN
    stays in its row, other rows of the tile are as without them."""
    gs = _gs()
    K = 70
    X, _ = operand(B, K, torch.float32, 8, "aligned")
    Q, _ = operand(N, K, torch.float32, 9, "aligned")
    x, q = X.double(), Q.double()
    X[7, 69] = float("inf")
    X[300, 3] = float("nan")
    T = gs.gs_project(X, Q)
    assert torch.equal(T[7], torch.where(Q[:, 69] > 0, float("inf"), float("-inf")))
    assert torch.all(T[300].isnan())
    keep = torch.ones(B, dtype=torch.bool, device="cuda")
    keep[7] = keep[300] = False
    assert torch.all(((T.double() - x @ q.T).abs() <= bound(x, q.T, K))[keep])


def test_planes_row_norms_rounding():
    """||x||^2 beside the product: a thread sums K / 2 squares, eight of a
    K-step first, so the long sum is rounded n = K / 16 times.  A rounding is
    2^-24 / sqrt(3) of the sum so far at most, in the root mean square, and
    the sum grows evenly: 2^-24 sqrt(n) / 3 for a half, less for both."""
    gs = _gs()
    K = 8192
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    X = torch.randn(16384, K, generator=g, device="cuda")
    Q = torch.randn(2048, K, generator=g, device="cuda")
    _, n2 = gs.gs_project(X, Q, xnorm2=True)
    exact = torch.cat([x.double().square().sum(1) for x in X.split(4096)])
    rel = (n2.double() - exact) / exact
    assert rel.square().mean().sqrt() <= 2.0 ** -24 * (K / 16) ** 0.5 / 3

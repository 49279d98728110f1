"""fp32 products on the 256 x 256 tiles, whose operands are split into three
bf16 planes: K around the K-step and its halves, ragged edges, values whose
parts leave the range of normal numbers, against 64-bit products."""
import pytest
import torch

from gpu_util import gamma
from test_gpu_split import operand, output
from test_product_routes import BF16, BIND, PROJECT, RESTORE, SCORES, SPLIT, TILES256, route

pytestmark = pytest.mark.gpu

# four rounds of large tiles, ragged both ways (every choice below asserts that
# they are taken)
B, N = 32700, 1990


def _gs():
    from paper_2608_01528_amd import gramspace
    return gramspace


def bound(a, b, K):
    """Any order of the sum (gamma), 2^-23 per product for the parts left out."""
    return (gamma(K + 8) + 2.0 ** -23) * (a.abs() @ b.abs()) + 1e-36


def twice(X):
    """The rows of X and again, in a batch that fills the chip with whole-row tiles."""
    X2 = _gs().alloc_rows(2 * B, X.shape[1], torch.float32, "cuda")
    X2[:B] = X
    X2[B:] = X
    return X2


@pytest.mark.parametrize("K", [4, 15, 16, 17, 33, 100, 259])
def test_planes_products(K):
    gs = _gs()
    assert route(PROJECT, B, N, K) == route(RESTORE, B, N, K) == route(PROJECT, B, N, K, out=BF16) == TILES256
    assert route(BIND, B, N, K) == (TILES256 if K >= 33 else SPLIT)
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
    X, x = twice(X), torch.cat([x, x])
    assert route(SCORES, 2 * B, 200, K) == TILES256
    R = C[:, :200].T.contiguous() if K % 4 == 0 else operand(200, K, torch.float32, 5, "aligned")[0]
    r = R.double()
    f = 1.0 / (x.norm(dim=1)[:, None] * r.norm(dim=1)[None, :])
    lim = f * bound(x, r.T, K) + (gamma(K + 8) + 1e-6) * (f * (x @ r.T)).abs()
    for given in (False, True):
        S, idx = gs.gs_similarity(X, R, qnorm2=(x * x).sum(1).float() if given else None,
                                  cnorm=r.norm(dim=1).float() if given else None)
        assert torch.all((S.double() - f * (x @ r.T)).abs() <= lim)
        assert torch.all(S.gather(1, idx.long()[:, None])[:, 0] == S.amax(1))


@pytest.mark.parametrize("scale", [1e-37, 1e-30, 1e18, 1e30, 1e35])
def test_planes_keep_the_range_of_fp32(scale):
    """Rows of tiny and of huge values, beside ordinary ones of the same tile:
    the error bound of an fp32 sum holds for each (2^-149: one unit of the
    smallest numbers)."""
    gs = _gs()
    K = 60
    assert route(PROJECT, B, N, K) == TILES256
    X, _ = operand(B, K, torch.float32, 6, "aligned")
    Q, _ = operand(N, K, torch.float32, 7, "aligned")
    X[11] *= scale
    X[32690] *= scale
    T = gs.gs_project(X, Q).double()
    x, q = X.double(), Q.double()
    assert torch.all((T - x @ q.T).abs() <= (gamma(K + 8) + 2.0 ** -23) * (x.abs() @ q.T.abs()) + K * 2.0 ** -149)


def test_planes_smallest_normal_numbers():
    """Values just above 2^-126 whose last plane is a subnormal bf16 of one
    sign: K = 8 keeps the bound of the sum (1.1e-6) below what losing that plane
    would show (2^-18.5 = 2.7e-6)."""
    gs = _gs()
    K = 8
    assert route(PROJECT, B, N, K) == TILES256
    g = torch.Generator(device="cuda")
    g.manual_seed(12)
    v = torch.rand(1 << 18, generator=g, device="cuda") + 1.0
    h = v.bfloat16().float()
    m = (v - h).bfloat16().float()
    v = v[(v - h - m) / v > 2.0 ** -18.5][:B // 256 * K]
    X, _ = operand(B, K, torch.float32, 13, "aligned")
    X[:v.numel() // K * 256:256] = v.view(-1, K) * 2.0 ** -126
    assert X[0].min() >= 2.0 ** -126 and v.numel() >= 100 * K
    Q = (torch.rand(N, K, generator=g, device="cuda") + 1.0) * 2.0 ** 60
    T = gs.gs_project(X, Q).double()
    x, q = X.double(), Q.double()
    assert torch.all((T - x @ q.T).abs() <= (gamma(K + 8) + 2.0 ** -23) * (x.abs() @ q.T.abs()))


@pytest.mark.parametrize("K", [70, 300, 1100])
def test_planes_tiles_done_again(K):
    """Rows with an infinity, of NaN, with a value or sums beyond the scaled
    range: their tiles are multiplied again in fp32 (among others of the same
    work-group that are not), an infinity gives the signed infinities of an
    fp32 product, a NaN stays in its row, and every other row, norm and column
    is as without them."""
    gs = _gs()
    assert route(PROJECT, B, N, K) == route(RESTORE, B, N, K) == route(BIND, B, N, K) == TILES256
    X, _ = operand(B, K, torch.float32, 8, "aligned")
    Q, _ = operand(N, K, torch.float32, 9, "aligned")
    C, _ = operand(K, N, torch.float32, 10, "aligned")
    X[5000, 3] = 1.5 * 2.0 ** 112
    X[9000] *= 1e30
    x, q, c = X.double(), Q.double(), C.double()
    X[7, K - 1] = float("inf")
    X[31000, 2] = float("-inf")
    X[300] = float("nan")
    rows = torch.ones(B, dtype=torch.bool, device="cuda")
    rows[[7, 31000, 300]] = False

    def signed(v):
        return torch.where(v > 0, float("inf"), float("-inf"))

    def check(T, b, dtype):
        T = T.float()
        assert torch.equal(T[7], signed(b[K - 1])) and torch.equal(T[31000], signed(-b[2]))
        assert torch.all(T[300].isnan())
        e = bound(x, b, K)
        if dtype == torch.bfloat16:
            e = e * 1.01 + 2.0 ** -8 * (x @ b).abs()
        assert torch.all(((T.double() - x @ b).abs() <= e)[rows])

    for dtype in (torch.float32, torch.bfloat16):
        T, n2 = gs.gs_project(X, Q, out_dtype=dtype, xnorm2=True)
        check(T, q.T, dtype)
        rows[[5000, 9000]] = False                   # (their squares are beyond fp32)
        n64 = (x * x).sum(1)
        assert torch.all((n2[rows].double() - n64[rows]).abs() <= gamma(K + 8) * n64[rows])
        assert torch.all(n2[[5000, 9000, 7, 31000]].isinf()) and n2[300].isnan()
        rows[[5000, 9000]] = True
        check(gs.gs_reconstruct(X, C, out_dtype=dtype), c, dtype)
    # a column that is not finite: one tile column is done again
    C2 = C.clone()
    C2[K // 2, 700] = float("inf")
    T = gs.gs_reconstruct(X, C2)
    assert torch.equal(T[rows, 700], signed(x[rows, K // 2]))
    T[:, 700] = gs.gs_reconstruct(X, C)[:, 700]
    check(T, c, torch.float32)
    # the bound product, whose second factor is done again
    Y, _ = operand(B, K, torch.float32, 11, "aligned")
    y = Y.double()
    Z = gs.gs_reconstruct(Y, C, T2=X, bind="mul")
    assert torch.all(Z[300].isnan()) and torch.all(Z[7].isinf())
    e1, e2 = bound(y, c, K), bound(x, c, K)
    lim = e1 * (x @ c).abs() + e2 * (y @ c).abs() + e1 * e2 + 2.0 ** -23 * ((x @ c) * (y @ c)).abs()
    assert torch.all(((Z.double() - (x @ c) * (y @ c)).abs() <= lim)[rows])


@pytest.mark.parametrize("K", [70, 1100])
def test_planes_score_tiles_done_again(K):
    """The same for cosine scores whose norms the product sums itself."""
    gs = _gs()
    M = 200
    assert route(SCORES, 2 * B, M, K) == TILES256
    X, _ = operand(B, K, torch.float32, 14, "aligned")
    R, _ = operand(M, K, torch.float32, 15, "aligned")
    x, r = X.double(), R.double()
    X[7, K - 1] = float("inf")
    X[300] = float("nan")
    X, x = twice(X), torch.cat([x, x])
    rows = torch.ones(2 * B, dtype=torch.bool, device="cuda")
    rows[[7, 300, B + 7, B + 300]] = False
    S, idx = gs.gs_similarity(X, R)
    f = 1.0 / (x.norm(dim=1)[:, None] * r.norm(dim=1)[None, :])
    lim = f * bound(x, r.T, K) + (gamma(K + 8) + 1e-6) * (f * (x @ r.T)).abs()
    assert torch.all(((S.double() - f * (x @ r.T)).abs() <= lim)[rows])
    assert torch.all((S.gather(1, idx.long()[:, None])[:, 0] == S.amax(1))[rows])
    assert torch.all(S[300].isnan())


def test_planes_row_norms_rounding():
    """||x||^2 beside the product: a thread sums K / 2 squares, eight of a
    K-step first, so the long sum is rounded n = K / 16 times.  A rounding is
    2^-24 / sqrt(3) of the sum so far at most, in the root mean square, and
    the sum grows evenly: 2^-24 sqrt(n) / 3 for a half, less for both."""
    gs = _gs()
    K = 8192
    assert route(PROJECT, 16384, 2048, K) == TILES256
    g = torch.Generator(device="cuda")
    g.manual_seed(11)
    X = torch.randn(16384, K, generator=g, device="cuda")
    Q = torch.randn(2048, K, generator=g, device="cuda")
    _, n2 = gs.gs_project(X, Q, xnorm2=True)
    exact = torch.cat([x.double().square().sum(1) for x in X.split(4096)])
    rel = (n2.double() - exact) / exact
    assert rel.square().mean().sqrt() <= 2.0 ** -24 * (K / 16) ** 0.5 / 3

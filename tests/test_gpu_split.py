"""Products on small tiles with the K range shared out over the waves of a
work-group: sizes around the edges of the tiles, of a K-step and of a 16-byte
piece, rows at any alignment, against 64-bit products of the values the
kernel reads."""
import numpy as np
import pytest
import torch

from gpu_util import gamma
from test_product_routes import BF16, F32, PROJECT, TILES128, route

pytestmark = pytest.mark.gpu

U_OUT = {torch.float32: 2.0 ** -24, torch.bfloat16: 2.0 ** -8}
# rows, K, columns: one of everything; around 32 x 32 tiles and K-steps of 32
# (fp32) and 64 (bf16); several waves per tile; 64 x 64 tiles
SIZES = [(1, 8, 8), (3, 13, 9), (31, 33, 65), (33, 64, 31), (64, 65, 96), (40, 127, 130), (257, 300, 67),
         (20, 1025, 40), (1100, 260, 1030)]


def _gs():
    from paper_2608_01528_amd import gramspace
    return gramspace


def operand(rows, cols, dtype, seed, layout):
    """rows x cols values inside a NaN-filled buffer: 'aligned' rows start on
    16-byte boundaries, 'odd' rows at odd elements with an odd stride."""
    g = np.random.default_rng(seed)
    v = torch.from_numpy(g.standard_normal((rows, cols)).astype(np.float32)).to(dtype)
    ld = (cols + 15) // 8 * 8 if layout == "aligned" else cols + 1 + (cols % 2)
    off = 0 if layout == "aligned" else 1
    buf = torch.full((rows * ld + off + 8,), float("nan"), dtype=dtype, device="cuda")
    t = buf[off:off + rows * ld].view(rows, ld)[:, :cols]
    t.copy_(v)
    return t, v.double().numpy()


def output(rows, cols, dtype, layout):
    ld = (cols + 15) // 8 * 8 if layout == "aligned" else cols + 3
    buf = torch.full((rows, ld), 7.0, dtype=dtype, device="cuda")
    return buf, buf[:, :cols]


def check(buf, got, exact, bound, cols):
    g = got.detach().cpu().double().numpy()
    assert np.all(np.abs(g - exact) <= bound), float((np.abs(g - exact) / bound).max())
    assert torch.all(buf[:, cols:] == 7.0)          # nothing written past the columns


def product_bound(a, b, K, dtype):
    """fp32 sum of K products in any order, then one rounding of the result."""
    e = gamma(K + 8) * (np.abs(a) @ np.abs(b))
    return e + (np.abs(a @ b) + e) * U_OUT[dtype] + 1e-30


@pytest.mark.parametrize("layout", ["aligned", "odd"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("rows,K,cols", SIZES)
def test_split_products(rows, K, cols, dtype, layout):
    gs = _gs()
    X, x = operand(rows, K, dtype, 1, layout)
    Y, y = operand(rows, K, dtype, 2, layout)
    Q, q = operand(cols, K, dtype, 3, layout)
    B, b = operand(K, cols, dtype, 4, layout)
    for ot in (torch.float32, torch.bfloat16):
        buf, out = output(rows, cols, ot, layout)
        _, n2 = gs.gs_project(X, Q, out=out, xnorm2=True)
        check(buf, out, x @ q.T, product_bound(x, q.T, K, ot), cols)
        n64 = (x * x).sum(1)
        assert np.all(np.abs(n2.cpu().double().numpy() - n64) <= gamma(K + 8) * n64)
        buf, out = output(rows, cols, ot, layout)
        gs.gs_reconstruct(X, B, out=out)
        check(buf, out, x @ b, product_bound(x, b, K, ot), cols)
        buf, out = output(rows, cols, ot, layout)
        gs.gs_reconstruct(X, B, T2=Y, bind="mul", out=out)
        e1, e2 = (product_bound(v, b, K, torch.float32) for v in (x, y))
        bound = e1 * np.abs(y @ b) + e2 * np.abs(x @ b) + e1 * e2
        bound += (np.abs((x @ b) * (y @ b)) + bound) * (U_OUT[ot] + 2.0 ** -24)
        check(buf, out, (x @ b) * (y @ b), bound, cols)


@pytest.mark.parametrize("layout", ["aligned", "odd"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("rows,K,cols", [(33, 40, 70), (70, 65, 65), (300, 129, 100), (40, 1030, 90)])
def test_split_scores(rows, K, cols, dtype, layout):
    gs = _gs()
    X, x = operand(rows, K, dtype, 5, layout)
    R, r = operand(cols, K, dtype, 6, layout)
    nx, nr = np.linalg.norm(x, axis=1), np.linalg.norm(r, axis=1)
    qn = torch.from_numpy((nx * nx).astype(np.float32)).cuda()
    cn = torch.from_numpy(nr.astype(np.float32)).cuda()
    for given in (False, True):
        buf, out = output(rows, cols, torch.float32, layout)
        S, idx = gs.gs_similarity(X, R, qnorm2=qn if given else None, cnorm=cn if given else None, scale=0.5, out=out)
        f = 0.5 / (nx[:, None] * nr[None, :])
        exact = f * (x @ r.T)
        bound = f * gamma(K + 8) * (np.abs(x) @ np.abs(r.T)) + (gamma(K + 8) + 1e-6) * np.abs(exact)
        check(buf, S, exact, bound, cols)
        assert torch.equal(idx.long(), S.argmax(1))
        A, O = gs.gs_attention(X, R, qnorm2=qn if given else None, cnorm=cn if given else None, beta=4.0,
                               weighted_sum=True, out_dtype=torch.float32)
        s = 4.0 * f / 0.5 * (x @ r.T)
        a = np.exp(s - s.max(1, keepdims=True))
        a /= a.sum(1, keepdims=True)
        assert np.abs(A.cpu().double().numpy() - a).max() <= 2e-5 * 4.0
        o = A.cpu().double().numpy() @ r
        assert np.abs(O.cpu().double().numpy() - o).max() <= gamma(cols + 8) * (a @ np.abs(r)).max() + 1e-6


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("M,r", [(70, 70), (300, 270), (130, 150)])
def test_split_echelon(M, r, dtype):
    """A flagged call on a lower-echelon R gives what the unflagged one gives,
    bit for bit (the skipped terms are zeros)."""
    gs = _gs()
    P, p = operand(90, M, dtype, 8, "aligned")
    R, _ = operand(M, r, dtype, 9, "aligned")
    R.copy_(torch.tril(R))
    r64 = R.cpu().double().numpy()
    T = [gs.gs_prob2vec(P, R, out_dtype=torch.float32, echelon=e) for e in (False, True)]
    assert torch.equal(T[0], T[1])
    for T in T:
        assert np.all(np.abs(T.cpu().double().numpy() - p @ r64) <= product_bound(p, r64, M, torch.float32))
    X, x = operand(90, r, dtype, 10, "aligned")
    qn = torch.ones(90, device="cuda")
    cn = torch.ones(M, device="cuda")
    S = [gs.gs_similarity(X, R, qnorm2=qn, cnorm=cn, echelon=e)[0] for e in (False, True)]
    assert torch.equal(S[0], S[1])
    d = np.abs(S[1].cpu().double().numpy() - x @ r64.T)
    assert np.all(d <= product_bound(x, r64.T, r, torch.float32) + 1e-6 * np.abs(x @ r64.T))


def test_split_infinities_stay_in_their_row():
    gs = _gs()
    X, _ = operand(40, 100, torch.float32, 11, "odd")
    Q, _ = operand(50, 100, torch.float32, 12, "odd")
    X[7, 99] = float("inf")
    Q[3, 98] = float("nan")
    T = gs.gs_project(X, Q)
    bad = ~torch.isfinite(T)
    want = torch.zeros_like(bad)
    want[7, :] = True
    want[:, 3] = True
    assert torch.equal(bad, want)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("r", [500, 505])
def test_scores_with_norms_summed_in_their_own_pass(dtype, r):
    """Cosine scores of a full batch over several column tiles without given
    norms: ||t|| from a pass over T, scores and winners as with the 64-bit
    norms, flagged and unflagged alike (also for gs_similarity_attention)."""
    gs = _gs()
    B, M = 33000, 520
    T, t = operand(B, r, dtype, 21, "aligned")
    R, _ = operand(M, r, dtype, 22, "aligned")
    R.copy_(torch.tril(R))
    T[5, :] = 0
    t[5, :] = 0
    r64 = R.cpu().double().numpy()
    S0, i0 = gs.gs_similarity(T, R)
    S1, i1 = gs.gs_similarity(T, R, echelon=True)
    S2, i2, _ = gs.gs_similarity_attention(T, R, echelon=True)
    assert torch.equal(S0, S1) and torch.equal(i0, i1) and torch.equal(S0, S2) and torch.equal(i0, i2)
    rows = np.concatenate([np.arange(300), np.arange(B - 300, B)])
    nx, nr = np.linalg.norm(t[rows], axis=1), np.linalg.norm(r64, axis=1)
    f = 1.0 / np.maximum(nx[:, None] * nr[None, :], 1e-30)
    exact = f * (t[rows] @ r64.T)
    bound = f * gamma(r + 8) * (np.abs(t[rows]) @ np.abs(r64.T)) + (gamma(r + 8) + 1e-6) * np.abs(exact) + 1e-30
    g = S1[torch.from_numpy(rows).cuda()].cpu().double().numpy()
    assert np.all(np.abs(g - exact) <= bound)
    assert torch.equal(i1.long(), S1.argmax(1)) or torch.all(S1.gather(1, i1.long()[:, None])[:, 0] == S1.amax(1))
    assert int(i1[5]) == 0 and torch.all(S1[5] == 0)


@pytest.mark.parametrize("layout", ["aligned", "odd"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("rows,K,cols", [(64, 3, 100), (1000, 7, 200), (70, 1, 33), (300, 2, 2)])
def test_short_k(rows, K, cols, dtype, layout):
    """Fewer than 16 bytes of K or of a row of B (128 x 128 tiles; K = 7 in
    fp32: small ones)."""
    gs = _gs()
    X, x = operand(rows, K, dtype, 21, layout)
    Y, y = operand(rows, K, dtype, 22, layout)
    Q, q = operand(cols, K, dtype, 23, layout)
    B, b = operand(K, cols, dtype, 24, layout)
    for ot in (torch.float32, torch.bfloat16):
        buf, out = output(rows, cols, ot, layout)
        _, n2 = gs.gs_project(X, Q, out=out, xnorm2=True)
        check(buf, out, x @ q.T, product_bound(x, q.T, K, ot), cols)
        n64 = (x * x).sum(1)
        assert np.all(np.abs(n2.cpu().double().numpy() - n64) <= gamma(K + 8) * n64)
        buf, out = output(rows, cols, ot, layout)
        gs.gs_reconstruct(X, B, out=out)
        check(buf, out, x @ b, product_bound(x, b, K, ot), cols)
        buf, out = output(rows, cols, ot, layout)
        gs.gs_reconstruct(X, B, T2=Y, bind="mul", out=out)
        e1, e2 = (product_bound(a, b, K, torch.float32) for a in (x, y))
        lim = e1 * np.abs(y @ b) + e2 * np.abs(x @ b) + e1 * e2
        check(buf, out, (x @ b) * (y @ b), lim + U_OUT[ot] * 1.01 * np.abs((x @ b) * (y @ b)) + 1e-30, cols)
    buf, S = output(rows, cols, torch.float32, layout)
    gs.gs_similarity(X, Q, mode="dot", out=S, argmax=False)
    check(buf, S, x @ q.T, product_bound(x, q.T, K, torch.float32), cols)


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
def test_strides_beyond_32_bit_offsets(dtype):
    """Rows 2^22 elements apart (128 x 128 tiles: 64-bit addresses, here with
    the long K ranges that the small tiles take otherwise)."""
    gs = _gs()
    rows, K, cols, ld = 37, 1001, 200, 1 << 22
    ty = BF16 if dtype == torch.bfloat16 else F32
    assert route(PROJECT, rows, cols, K, ty, ld=ld) == TILES128
    g = torch.Generator(device="cuda")
    g.manual_seed(25)
    buf = torch.zeros(rows, ld, dtype=dtype, device="cuda")
    X = buf[:, :K]
    X.normal_(generator=g)
    x = X.cpu().double().numpy()
    Q, q = operand(cols, K, dtype, 26, "aligned")
    B, b = operand(K, cols, dtype, 27, "aligned")
    Y, y = operand(rows, K, dtype, 28, "aligned")
    out, T = output(rows, cols, torch.float32, "aligned")
    _, n2 = gs.gs_project(X, Q, out=T, xnorm2=True)
    check(out, T, x @ q.T, product_bound(x, q.T, K, torch.float32), cols)
    n64 = (x * x).sum(1)
    assert np.all(np.abs(n2.cpu().double().numpy() - n64) <= gamma(K + 8) * n64)
    out, Z = output(rows, cols, torch.float32, "aligned")
    gs.gs_reconstruct(X, B, T2=Y, bind="mul", out=Z)
    e1, e2 = product_bound(x, b, K, torch.float32), product_bound(y, b, K, torch.float32)
    check(out, Z, (x @ b) * (y @ b), e1 * np.abs(y @ b) + e2 * np.abs(x @ b) + e1 * e2 + 1e-30, cols)
    out, S = output(rows, cols, torch.float32, "aligned")
    gs.gs_similarity(X, Q, mode="dot", out=S, argmax=False)
    check(out, S, x @ q.T, product_bound(x, q.T, K, torch.float32), cols)

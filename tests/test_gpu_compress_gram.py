"""Rank decisions of compress from a panel's Gram matrix, and where they must
be left to the factor of the rows: copies inside and outside a panel, rows
close to either side of the line between the two, chains of small pivots,
squares out of range, short panels; rank, kept rows and factors against the
oracle."""
import numpy as np
import pytest
import torch

import oracle

pytestmark = pytest.mark.gpu


def codebook(kind, M, D):
    g = np.random.default_rng(5)
    C = g.choice([-1.0, 1.0], size=(M, D))
    if kind == "copies":                    # of an earlier panel, of the own panel, a negation, a zero row
        C[40 % M] = C[3]
        C[M - 1] = C[M - 3]
        C[20] = -C[10]
        C[25] = 0.0
    elif kind == "line":                    # residuals of 0.005, 0.0099, 0.0101, 0.02 and 1e-7 of the norm
        for i, f in ((9, 5e-3), (17, 9.9e-3), (30, 1.01e-2), (34 % M, 2e-2), (M - 2, 1e-7)):
            u = g.standard_normal(D)
            base = C[1] + C[2]
            u -= np.linalg.lstsq(C[:9].T, u, rcond=None)[0] @ C[:9]
            C[i] = base + f * np.linalg.norm(base) * u / np.linalg.norm(u)
    elif kind == "tiny":
        C *= 1e-130
    elif kind == "huge":
        C *= 1e130
    elif kind == "mixed":                   # one row's squares out of range
        C[7] *= 1e-120
    return C


@pytest.mark.parametrize("M,D", [(33, 200), (70, 333), (96, 1030)])
@pytest.mark.parametrize("kind", ["plain", "copies", "line", "tiny", "huge", "mixed"])
def test_compress_decisions(kind, M, D):
    from paper_2608_01528_amd import gramspace as gs
    C = codebook(kind, M, D)
    Q, R, r, kept, cn = gs.gs_compress(torch.from_numpy(C).cuda())
    Qo, Ro, kept_o, ro = oracle.compress(C)
    assert r == ro
    assert np.array_equal(kept.cpu().numpy(), np.asarray(kept_o)[:ro])
    q, rr = Q.cpu().numpy(), R.cpu().numpy()
    scale = np.abs(C).max(1, keepdims=True).clip(1e-300)
    # fp64 throughout: n eps with n the rows summed, times a margin for the
    # second projections
    assert np.abs(q @ q.T - np.eye(r)).max() <= 4 * M * 2.0 ** -52
    assert (np.abs(rr @ q - C) / scale).max() <= 64 * M * 2.0 ** -52
    # a kept row's residual of relative size f fixes its vector to eps / f
    f = 1e-7 if kind == "line" else 0.1
    assert np.abs(np.abs(np.sum(q * Qo[:r], 1)) - 1.0).max() <= (64 * M * 2.0 ** -52 / f) + 1e-12


def chain(n, a, kind, dependent, seed, D=512):
    """Rows whose pivots are each a fair part of their norm while the errors
    of the earlier ones grow by about 1 / a from row to row: an orthonormal
    (or nearly orthogonal bipolar) v_i, c_0 = v_0 and c_i the previous vector
    plus a little of v_i.  dependent: one more row, inside their span."""
    g = np.random.default_rng(seed)
    if kind == "orthonormal":
        v, b = np.linalg.qr(g.standard_normal((D, n)))[0].T, np.sqrt(1 - a * a)
    else:
        v, b = g.choice([-1.0, 1.0], size=(n, D)), 1.0
    C = np.vstack([v[:1], b * v[:-1] + a * v[1:]])
    if dependent:
        C = np.vstack([C, g.standard_normal(n) @ v if kind == "orthonormal" else v[-1]])
    return np.ascontiguousarray(C)


@pytest.mark.parametrize("n,a,kind,dependent,tol", [
    (11, 0.168, "orthonormal", True, 1e-4), (14, 0.25, "orthonormal", True, 1e-4),
    (18, 0.3, "orthonormal", True, 1e-6), (5, 0.0123, "bipolar", True, 1e-6), (6, 0.05, "bipolar", True, 1e-6),
    (4, 0.0123, "bipolar", True, 1e-8), (4, 0.3, "bipolar", True, 1e-10),
    (8, 0.0123, "bipolar", False, 1e-10), (20, 0.05, "orthonormal", False, 1e-10),
    (24, 0.2, "orthonormal", False, 1e-10)])
def test_compress_chained_pivots(n, a, kind, dependent, tol):
    from paper_2608_01528_amd import gramspace as gs
    for seed in range(12):
        C = chain(n, a, kind, dependent, seed)
        Q, R, r, kept, _ = gs.gs_compress(torch.from_numpy(C).cuda(), tol=tol)
        _, Ro, kept_o, ro = oracle.compress(C, tol)
        assert r == ro == n, seed
        assert np.array_equal(kept.cpu().numpy(), np.asarray(kept_o)[:ro])
        q, rr = Q.cpu().numpy(), R.cpu().numpy()
        M, D = C.shape
        norm = np.linalg.norm(C, axis=1)
        # inner products of D terms, and the M rows' combinations
        assert np.abs(q @ q.T - np.eye(r)).max() <= (D + 4 * M) * 2.0 ** -53, seed
        # a basis vector is a combination of rows: it carries the rounding of
        # the largest term, 2^-53 times its weights; a dependent row may also
        # leave out tol of its norm
        weight = (np.abs(np.linalg.inv(Ro[:n])) * norm[:n]).sum(1).max()
        off = np.linalg.norm(rr @ q - C, axis=1) / norm
        assert off[:n].max() <= M * 2.0 ** -53 * max(weight, 64), seed
        assert off.max() <= tol + M * 2.0 ** -53 * max(weight, 64), seed

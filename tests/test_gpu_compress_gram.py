"""Rank decisions of compress from a panel's Gram matrix, and where they must
be left to the factor of the rows: copies inside and outside a panel, rows
close to either side of the line between the two, squares out of range, short
panels; rank, kept rows and factors against the oracle."""
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

"""Small codebooks on both sides of the rule that gives a call to the
streaming kernels or to the product on small tiles (entries 15/16/25/33/64,
coordinates 7/8, rows 33/16384/16385/65536/65537), against 64-bit results."""
import pytest
import torch

from gpu_util import gamma
from test_gpu_split import operand

pytestmark = pytest.mark.gpu

U_OUT = {torch.float32: 2.0 ** -24, torch.bfloat16: 2.0 ** -8}
CASES = [(33, 15, 15), (33, 16, 7), (33, 16, 8), (100, 25, 7), (100, 25, 25), (1000, 33, 33), (1000, 64, 63),
         (16384, 40, 40), (16385, 40, 33), (65536, 24, 24), (65537, 24, 24), (65537, 32, 8), (65537, 33, 33)]


@pytest.mark.parametrize("layout", ["aligned", "odd"])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16], ids=["f32", "bf16"])
@pytest.mark.parametrize("B,M,r", CASES)
def test_small_codebook_either_path(B, M, r, dtype, layout):
    from paper_2608_01528_amd import gramspace as gs
    P, _ = operand(B, M, dtype, 1, layout)
    P.abs_()
    R, _ = operand(M, r, dtype, 2, layout)
    T, _ = operand(B, r, dtype, 3, layout)
    T[5] = 0
    R.copy_(torch.tril(R))
    p, rr, t = P.double(), R.double(), T.double()
    for ech in (False, True):
        g = gs.gs_prob2vec(P, R, out_dtype=dtype, echelon=ech).double()
        e = gamma(M + 8) * (p @ rr.abs())
        assert torch.all((g - p @ rr).abs() <= e + ((p @ rr).abs() + e) * U_OUT[dtype] + 1e-30)
    dot = t @ rr.T
    f = 1.0 / (t.norm(dim=1).clamp_min(1e-30)[:, None] * rr.norm(dim=1).clamp_min(1e-30)[None, :])
    exact = f * dot
    lim = f * gamma(r + 8) * (t.abs() @ rr.abs().T) + (gamma(r + 8) + 1e-6) * exact.abs() + 1e-30
    cn = rr.norm(dim=1).float()
    for given in (None, cn):
        S, idx = gs.gs_similarity(T, R, cnorm=given)
        S2, idx2, A2 = gs.gs_similarity_attention(T, R, cnorm=given, beta=4.0)
        A, O = gs.gs_attention(T, R, cnorm=given, beta=4.0)
        w = torch.softmax(4.0 * exact, 1)
        for s, i in ((S, idx), (S2, idx2)):
            assert torch.all((s.double() - exact).abs() <= lim)
            assert torch.all(s.gather(1, i.long()[:, None])[:, 0] == s.amax(1)) and int(i[5]) == 0
        for a in (A, A2):
            assert (a.double() - w).abs().max() <= 1e-4
    _, only = gs.gs_similarity(T, R, cnorm=cn, scores=False)
    assert torch.all(exact.gather(1, only.long()[:, None])[:, 0] >= exact.amax(1) - 2 * lim.amax(1))

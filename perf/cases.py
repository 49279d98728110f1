"""Timed cases of the Gram-Space operators, through the torch binding.

Each case is one thing a program that serves or builds a VSA codebook does,
at sizes of the named workloads (tiny, vsa, large, binary, stress), of the
paper's setting (codebooks of 5 to 40 entries, dimensions 256 to 8192), or
between them: a request stream rarely fills the batch the largest workloads
are quoted at.  `listed` names fixed cases, `draw` gives others of the same
ranges.

Kinds (key "kind"):
  lookup    superposed vectors of a small codebook, from probabilities to
            scores, winner and weights, restored: prob2vec, similarity_attention,
            reconstruct
  soft      the fused soft selection over the attribute codebooks of a task
  query     dense queries against a codebook: project (with ||x||^2), cosine
            scores, winner and attention weights
  project   the projection alone (what a store of coordinates is filled by)
  scores    prob2vec and scores of a large codebook, lower-echelon R
  restore   coordinates back to the original domain
  bind      two coordinate batches restored, multiplied, projected again
  conv      circular convolution / correlation of restored vectors
  compress  basis and coordinates of a codebook (once per codebook)

Inputs, codebooks and reference results are made with torch on the GPU from
the seed alone.  Normal distributions are read as N(mu, sigma^2).
"""
import math

import torch

from paper_2608_01528_amd import gramspace as gs

DEV = "cuda"
DT = {"f32": torch.float32, "bf16": torch.bfloat16}
BETA = 16.0          # attention sharpness, as the benchmark uses


# ------------------------------------------------------------------ cases

def listed():
    return [
        # one reasoning step of a single problem (16 panels): latency and launches
        {"name": "lookup_tiny", "kind": "lookup", "dtype": "f32", "B": 16, "M": 10, "D": 1024},
        # the global codebook (4 attributes x 10 values) over a ragged batch
        {"name": "lookup_global", "kind": "lookup", "dtype": "f32", "B": 3001, "M": 40, "D": 2048},
        # 4096 problems x 16 panels, four attribute codebooks, one launch
        {"name": "soft_vsa", "kind": "soft", "dtype": "f32", "B": 65536, "Ms": "5,6,10,22", "coords": False},
        # hard selection, a request batch of ordinary size with ragged sizes
        {"name": "query_request", "kind": "query", "dtype": "f32", "B": 777, "M": 203, "D": 4096},
        # hard selection at the full batch
        {"name": "query_large", "kind": "query", "dtype": "f32", "B": 65536, "M": 256, "D": 8192},
        # binding a request's worth of pairs against a mid-sized binary codebook
        {"name": "bind_request", "kind": "bind", "dtype": "f32", "B": 512, "M": 360, "D": 4096},
        # the binary workload: restore and bind 16384 pairs, project back
        {"name": "bind_binary", "kind": "bind", "dtype": "f32", "B": 16384, "M": 1000, "D": 4096},
        # the stress pipeline's three stages at its full batch
        {"name": "project_stress", "kind": "project", "dtype": "bf16", "B": 262144, "M": 2048, "D": 16384,
         "dup": 205, "norms": True},
        {"name": "scores_stress", "kind": "scores", "dtype": "bf16", "B": 262144, "M": 2048, "D": 16384, "dup": 205},
        {"name": "restore_stress", "kind": "restore", "dtype": "bf16", "B": 262144, "M": 2048, "D": 16384, "dup": 205},
        # binding by circular convolution of restored vectors, whole rows
        {"name": "conv_rows", "kind": "conv", "dtype": "f32", "B": 16384, "D": 4096, "L": 4096, "op": "conv"},
        # building the binary workload's codebook
        {"name": "compress_binary", "kind": "compress", "dtype": "f32", "M": 1000, "D": 4096, "dup": 0,
         "binary": True},
    ]


def _log(rng, lo, hi):
    """An integer whose logarithm is uniform over [lo, hi]."""
    return int(min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _dim(rng, lo, hi):
    """A vector dimension: mostly a multiple of 64, sometimes any number."""
    d = _log(rng, lo, hi)
    return d if rng.random() < 0.2 else max(lo, d // 64 * 64)


def draw(rng):
    kind = rng.choice(["lookup", "soft", "query", "query", "project", "scores", "restore", "bind", "conv",
                       "compress"])
    dtype = rng.choice(["f32", "f32", "bf16"])
    cap = 1.2e12 if dtype == "f32" else 1.2e13      # products of the longest passes
    if kind == "lookup":
        return {"kind": kind, "dtype": dtype, "B": _log(rng, 1, 16384), "M": rng.randint(5, 64),
                "D": _dim(rng, 256, 8192)}
    if kind == "soft":
        ms = [rng.randint(3, 32) for _ in range(rng.randint(1, 6))]
        return {"kind": kind, "dtype": dtype, "B": _log(rng, 64, 65536), "Ms": ",".join(map(str, ms)),
                "coords": rng.random() < 0.3}
    if kind == "conv":
        lg = rng.randint(6, 13)
        return {"kind": kind, "dtype": dtype, "B": _log(rng, 16, 16384), "L": 1 << lg,
                "D": (1 << lg) * rng.randint(1, max(1, 8192 >> lg)), "op": rng.choice(["conv", "corr"])}
    if kind == "compress":
        M = _log(rng, 5, 1200)
        return {"kind": kind, "dtype": "f32", "M": M, "D": _dim(rng, max(256, 2 * M), 16384 if M < 400 else 8192),
                "dup": rng.choice([0, 0, M // 10]), "binary": rng.random() < 0.5}
    M = _log(rng, 16, 1000 if dtype == "f32" else 2048)
    D = _dim(rng, max(256, 2 * M), 8192 if dtype == "f32" else 16384)
    if kind == "bind":
        return {"kind": kind, "dtype": "f32", "M": min(M, 1000), "D": min(D, 8192),
                "B": _log(rng, 1, min(16384, 4e11 / (min(D, 8192) * min(M, 1000) * 2)))}
    per = 2 * M * (M if kind == "scores" else D)
    c = {"kind": kind, "dtype": dtype, "B": _log(rng, 1, min(262144 if dtype == "bf16" else 65536, cap / per)),
         "M": M, "D": D}
    if kind == "project":
        c["norms"] = rng.random() < 0.5
    if kind in ("project", "scores", "restore"):
        c["dup"] = rng.choice([0, M // 10])
    return c


# ----------------------------------------------------------------- inputs

def _gen(seed, stream):
    g = torch.Generator(device=DEV)
    g.manual_seed((int(seed) * 1000003 + stream) & 0x7FFFFFFF)
    return g


def _codebook(case, seed, M=None, D=None, stream=1):
    """Bipolar (or binary) codebook, M x D fp32; the last `dup` rows of a
    random order are copies of others."""
    M, D = M or case["M"], D or case["D"]
    g = _gen(seed, stream)
    C = torch.randint(0, 2, (M, D), generator=g, device=DEV).float()
    if not case.get("binary") and case["kind"] != "bind":
        C = 2 * C - 1
    n = case.get("dup", 0)
    if n:
        order = torch.randperm(M, generator=g, device=DEV)
        src = order[torch.randint(0, M - n, (n,), generator=g, device=DEV)]
        C[order[M - n:]] = C[src]
    return C


def _first(C):
    """For each row of C the index of the first row equal to it (the row
    itself unless it is a copy)."""
    v = torch.randn(C.shape[1], 2, generator=_gen(7, 7), device=DEV, dtype=torch.float64)
    h = C.double() @ v
    same = (h[:, None, :] - h[None, :, :]).abs().amax(2) < 1e-6
    return same.int().argmax(1)


def _basis64(C):
    """(Q, R, kept) of C in 64 bits: rows in index order, copies dependent,
    positive pivots (the Cholesky factor of the kept rows' Gram matrix)."""
    first = _first(C)
    kept = torch.nonzero(first == torch.arange(C.shape[0], device=DEV)).flatten()
    K = C[kept].double()
    Lo = torch.linalg.cholesky(K @ K.T)
    Q = torch.cat([torch.linalg.solve_triangular(Lo, k, upper=False) for k in K.split(2048, 1)], 1)
    at = torch.searchsorted(kept, first)
    return Q, Lo[at], kept


def _probs(B, M, seed, stream, kind, dtype):
    """Probability rows: softmax of N(0, 2) logits (attribute distributions),
    Dirichlet(0.5) (mixtures over a large codebook) or Dirichlet(0.05)
    (nearly one entry per row), in rows aligned to 16 bytes."""
    g = _gen(seed, stream)
    P = gs.alloc_rows(B, M, dtype, DEV)
    for a in range(0, B, 65536):
        b = min(B, a + 65536)
        if kind == "softmax":
            p = torch.softmax(math.sqrt(2.0) * torch.randn(b - a, M, generator=g, device=DEV), 1)
        elif kind == "dir0.5":
            p = torch.randn(b - a, M, generator=g, device=DEV).square_()
            p = p / p.sum(1, keepdim=True)
        else:
            p = torch._standard_gamma(torch.full((b - a, M), 0.05, device=DEV), generator=g) + 1e-30
            p = p / p.sum(1, keepdim=True)
        P[a:b] = p.to(dtype)
    return P


def _queries(case, C, seed):
    """Dense query rows x = p C + N(0, 0.1), contiguous as a front end hands
    them over, in the case's type."""
    B, D, dtype = case["B"], case["D"], DT[case["dtype"]]
    P = _probs(B, case["M"], seed, 3, "dir0.5", torch.float32)
    g = _gen(seed, 4)
    X = torch.empty(B, D, dtype=dtype, device=DEV)
    for a in range(0, B, 16384):
        b = min(B, a + 16384)
        x = P[a:b] @ C
        x += math.sqrt(0.1) * torch.randn(b - a, D, generator=g, device=DEV)
        X[a:b] = x.to(dtype)
    return X


def _inputs(case, seed):
    """What run reads besides the compressed codebooks: a dict of tensors."""
    kind, dtype = case["kind"], DT[case["dtype"]]
    if kind == "soft":
        ms = [int(m) for m in case["Ms"].split(",")]
        return {"C": [_codebook(case, seed, m, 1024, 20 + i) for i, m in enumerate(ms)],
                "P": [_probs(case["B"], m, seed, 40 + i, "softmax", dtype) for i, m in enumerate(ms)]}
    if kind == "conv":
        g = _gen(seed, 5)
        # restored mixtures of bipolar vectors look Gaussian per component
        X, Y = (torch.randn(case["B"], case["D"], generator=g, device=DEV).to(dtype) for _ in range(2))
        return {"X": X, "Y": Y}
    C = _codebook(case, seed)
    if kind == "compress":
        return {"C": C}
    if kind in ("query", "project"):
        return {"C": C, "X": _queries(case, C, seed)}
    law = {"lookup": "softmax", "scores": "dir0.5", "restore": "dir0.5", "bind": "dir0.05"}[kind]
    x = {"C": C, "P": _probs(case["B"], case["M"], seed, 3, law, dtype)}
    if kind == "bind":
        x["P2"] = _probs(case["B"], case["M"], seed, 6, law, dtype)
    return x


def prepare(case, seed):
    """Inputs, the compressed codebook in the case's type, and the output
    buffers a serving loop keeps."""
    kind, dtype = case["kind"], DT[case["dtype"]]
    x = _inputs(case, seed)
    s = {"case": case}
    if kind == "conv":
        s.update(x, out=gs.alloc_rows(case["B"], case["D"], dtype, DEV))
        return s
    if kind == "compress":
        need = gs.compress_workspace_bytes(case["M"], case["D"])
        s.update(x, ws=torch.empty(need + 256, dtype=torch.uint8, device=DEV))
        return s
    B = case["B"]
    if kind == "soft":
        groups = []
        for C, P in zip(x["C"], x["P"]):
            _, R, r, _, cn = gs.gs_compress(C, q_dtype=dtype, r_dtype=dtype)
            M = C.shape[0]
            groups.append({"P": P, "R": R, "cnorm": cn, "S": torch.empty(B, M, device=DEV),
                           "argmax": torch.empty(B, dtype=torch.int32, device=DEV),
                           "A": torch.empty(B, M, device=DEV)})
            if case["coords"]:
                groups[-1]["T"] = gs.alloc_rows(B, r, dtype, DEV)
        s.update(groups=groups, prepared=gs.soft_groups(groups))
        return s
    Q, R, r, _, cn = gs.gs_compress(x["C"], q_dtype=dtype, r_dtype=dtype)
    M, D = case["M"], case["D"]
    s.update(Q=Q, R=R, cn=cn)
    for k in ("X", "P", "P2"):
        if k in x:
            s[k] = x[k]
    if kind in ("restore", "bind"):
        # the coordinates come from an earlier stage of the program
        s["T"] = gs.gs_prob2vec(s.pop("P"), R)
        if kind == "bind":
            s["T2"] = gs.gs_prob2vec(s.pop("P2"), R)
    else:
        s["T"] = gs.alloc_rows(B, r, dtype, DEV)
        s["xn"] = torch.empty(B, device=DEV)
    if kind in ("lookup", "query", "scores"):
        s["S"], s["A"] = torch.empty(B, M, device=DEV), torch.empty(B, M, device=DEV)
        s["idx"] = torch.empty(B, dtype=torch.int32, device=DEV)
    if kind in ("lookup", "restore", "bind"):
        s["out"] = gs.alloc_rows(B, D, dtype, DEV)
    if kind == "bind":
        s["Z"] = gs.alloc_rows(B, r, dtype, DEV)
    return s


# -------------------------------------------------------------------- run

def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "soft":
        gs.gs_soft_select(None, mode="cosine", beta=BETA, prepared=s["prepared"])
        return [[g["S"], g["argmax"], g["A"]] + ([g["T"]] if case["coords"] else []) for g in s["groups"]]
    if kind == "conv":
        return gs.gs_bind_restored(s["X"], s["Y"], case["op"], case["L"], out=s["out"])
    if kind == "compress":
        Q, R, r, kept, cn = gs.gs_compress(s["C"], q_dtype=torch.float32, r_dtype=torch.float32, workspace=s["ws"])
        return [Q, R, r, kept, cn]
    if kind == "project":
        T = gs.gs_project(s["X"], s["Q"], xnorm2=case["norms"], out=s["T"], xnorm2_out=s["xn"])
        return list(T) if case["norms"] else [T]
    if kind == "restore":
        return [gs.gs_reconstruct(s["T"], s["Q"], out=s["out"])]
    if kind == "bind":
        X = gs.gs_reconstruct(s["T"], s["Q"], T2=s["T2"], bind="mul", out=s["out"])
        return [X, gs.gs_project(X, s["Q"], out=s["Z"])]
    if kind == "query":
        T, xn = gs.gs_project(s["X"], s["Q"], xnorm2=True, out=s["T"], xnorm2_out=s["xn"])
        S, idx, A = gs.gs_similarity_attention(T, s["R"], qnorm2=xn, cnorm=s["cn"], beta=BETA, out=s["S"],
                                               argmax_out=s["idx"], a_out=s["A"], echelon=True)
        return [T, xn, S, idx, A]
    T = gs.gs_prob2vec(s["P"], s["R"], out=s["T"], echelon=True)
    S, idx, A = gs.gs_similarity_attention(T, s["R"], cnorm=s["cn"], beta=BETA, out=s["S"], argmax_out=s["idx"],
                                           a_out=s["A"], echelon=True)
    if kind == "scores":
        return [T, S, idx, A]
    return [T, S, idx, A, gs.gs_reconstruct(T, s["Q"], out=s["out"])]


# ------------------------------------------------------------- yardsticks

def _rank(case):
    return case["M"] - case.get("dup", 0)


def work(case):
    """Bytes read and written once, and the products that are due (the zero
    half of a lower-echelon R not counted)."""
    kind = case["kind"]
    e = 2 if case["dtype"] == "bf16" else 4
    if kind == "soft":
        by = fl = 0
        for m in map(int, case["Ms"].split(",")):
            by += case["B"] * (e * m + 8 * m + 4 + (e * m if case["coords"] else 0)) + e * m * m
            fl += case["B"] * 2 * m * m * (2 if case["coords"] else 1)
        return {"bytes": by, "flops": fl}
    if kind == "conv":
        B, D, lg = case["B"], case["D"], math.log2(case["L"])
        return {"bytes": 3 * e * B * D, "flops": B * D * (10 * lg + 6)}
    M, D, r = case["M"], case["D"], _rank(case)
    if kind == "compress":
        return {"bytes": 4 * M * D + 4 * r * D + 4 * M * r, "flops": 2 * r * r * D}
    B = case["B"]
    tri = r * (M - 0.5 * r)                 # entries of R that may be nonzero
    score_b = e * tri + B * (8 * M + 4)
    if kind == "project":
        return {"bytes": e * (B * D + r * D + B * r) + (4 * B if case["norms"] else 0), "flops": 2 * B * D * r}
    if kind == "restore":
        return {"bytes": e * (B * D + r * D + B * r), "flops": 2 * B * D * r}
    if kind == "bind":
        return {"bytes": e * (B * D + r * D + 3 * B * r), "flops": 6 * B * D * r}
    if kind == "query":
        return {"bytes": e * (B * D + r * D + B * r) + 4 * B + score_b, "flops": 2 * B * r * D + 2 * B * tri}
    by, fl = e * (B * M + B * r) + score_b, 4 * B * tri
    if kind == "lookup":
        by, fl = by + e * (r * D + B * D), fl + 2 * B * r * D
    return {"bytes": by, "flops": fl}


def tolerance(case):
    if case["kind"] == "compress":
        return {"rel": 1e-6, "max": 1e-5}           # 64-bit work, results rounded to fp32
    if case["dtype"] == "bf16":
        # results stored in bf16 (half a unit in the last place is 2e-3);
        # scores in fp32 from coordinates rounded to bf16
        return {"rel": 8e-3, "max": 0.3, "differ": 5e-3}
    return {"rel": 1e-5, "max": 4e-4, "differ": 1e-3}


# -------------------------------------------------------------- reference

def _softmax_scores(T, xn2, R, cn, out):
    S = (T @ R.T) / (xn2.sqrt()[:, None] * cn[None, :])
    out.append(S)
    out.append(None)                        # the winner is a whole number
    out.append(torch.softmax(BETA * S, 1))


def exact(case, seed):
    """run()'s results in 64 bits from the same inputs, without the library.
    The basis and R are those of the 64-bit factorisation, rounded to the
    type the program keeps them in."""
    kind, dtype = case["kind"], DT[case["dtype"]]
    x = _inputs(case, seed)
    if kind == "conv":
        B, D, L = case["B"], case["D"], case["L"]
        out = torch.empty(B, D, dtype=torch.float64, device=DEV)
        for a in range(0, B, 4096):
            b = min(B, a + 4096)
            X, Y = (torch.fft.rfft(x[k][a:b].double().reshape(b - a, D // L, L)) for k in ("X", "Y"))
            Z = X * Y if case["op"] == "conv" else X * Y.conj()
            out[a:b] = torch.fft.irfft(Z, n=L).reshape(b - a, D)
        return out
    if kind == "soft":
        res = []
        for C, P in zip(x["C"], x["P"]):
            _, R, _ = _basis64(C)
            R = R.to(dtype).double()
            T = P.double() @ R
            row = []
            _softmax_scores(T, T.square().sum(1), R, C.double().norm(dim=1), row)
            res.append(row + ([T] if case["coords"] else []))
        return res
    C = x["C"]
    Q, R, kept = _basis64(C)
    if kind == "compress":
        return [Q, R, None, None, C.double().norm(dim=1)]
    Q, R, cn = Q.to(dtype).double(), R.to(dtype).double(), C.double().norm(dim=1)
    if kind in ("query", "project"):
        X = x["X"]
        T = torch.empty(case["B"], Q.shape[0], dtype=torch.float64, device=DEV)
        xn = torch.empty(case["B"], dtype=torch.float64, device=DEV)
        for a in range(0, case["B"], 32768):
            xd = X[a:a + 32768].double()
            T[a:a + 32768] = xd @ Q.T
            xn[a:a + 32768] = xd.square().sum(1)
        if kind == "project":
            return [T, xn] if case["norms"] else [T]
        out = [T, xn]
        _softmax_scores(T, xn, R, cn, out)
        return out
    if kind in ("restore", "bind"):
        # the coordinates run is given, in the type it is given them
        T = (x["P"].double() @ R).to(dtype).double()
        if kind == "restore":
            return [T @ Q]
        X = (T @ Q) * ((x["P2"].double() @ R).to(dtype).double() @ Q)
        return [X, X @ Q.T]
    T = x["P"].double() @ R
    out = [T]
    _softmax_scores(T, T.square().sum(1), R, cn, out)
    if kind == "lookup":
        out.append(T @ Q)
    return out

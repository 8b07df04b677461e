"""The work that users of the library have it do, as cases to time.

Greedy column subset selection is called in a few ways: on a matrix small
enough to be explored interactively, on data sets of tens of thousands of
instances, and on matrices of gigabytes; with the matrix itself or a concise
target to reconstruct; in one selection or over column blocks; and around the
selection there are the target's projection, the error of a given subset, the
conversion to a storage format and the rank-k factors.  The listed cases take
each of them at sizes of this repository's workloads or at generic (ragged)
ones; ``draw`` gives others of the same ranges.

Inputs are columns of a low-rank signal with a power-law spectrum plus noise,
with log-normal column norms.  Every number comes from the seed.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

import paper_1312_6838_amd as gcss

DEVICE = "cuda"
CHUNK = 32768  # columns made at a time
CACHE_BYTES = 256 << 20  # the last-level cache: a larger matrix is read again by every step


def listed():
    return [
        # a first look at a small matrix: target, selection and error in one go
        dict(name="small whole", kind="whole", m=500, n=1000, k=20, store="f32"),
        # a small table with a concise target, nothing a round number
        dict(name="small ragged", kind="select", m=333, n=5003, r=50, k=25, store="f32", target="f32"),
        # an image data set of 32 x 32 pixels, stored as bfloat16
        dict(name="images bf16", kind="select", m=1024, n=60001, r=128, k=50, store="bf16", target="f32"),
        # more features than usual against the instances, none a multiple of a tile
        dict(name="tall ragged", kind="select", m=3001, n=20011, r=200, k=64, store="f32", target="f32"),
        # the centralized problem at full size: Gram matrix, scores, selection, error
        dict(name="large whole", kind="whole", m=4096, n=65536, k=200, store="f32"),
        # a million instances, the concise target in hand
        dict(name="million f32", kind="select", m=2048, n=1048576, r=256, k=100, store="f32", target="f32"),
        # the largest features, FP8 storage and a long selection
        dict(name="wide fp8", kind="select", m=8192, n=262144, r=512, k=500, store="fp8", target="bf16"),
        # the distributed selection: uneven blocks, then the merge
        dict(name="blocks bf16", kind="batched", m=1024, blocks=64, wlo=2048, whi=32768, wseed=0, r=128,
             k=20, merge=100, store="bf16"),
        # the concise target of a new matrix (with its initial scores)
        dict(name="project f32", kind="project", m=2048, n=262144, r=256, store="f32"),
        # how good a given subset is: the baselines that a selection is compared with
        dict(name="subset error", kind="error", m=1024, n=60001, r=128, k=100, store="f32", target="f32"),
        # a matrix brought to its storage format
        dict(name="quantize fp8", kind="quantize", m=8192, n=32768, store="fp8"),
        # the approximate truncated SVD from a selection's embedding
        dict(name="rank k", kind="rank", m=1024, n=60000, l=100, k=50, store="f32"),
    ]


def _log_int(rng, lo, hi):
    """An integer of [lo, hi], spread over the logarithm; odd ones among them."""
    v = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    return max(lo, min(hi, v + rng.choice((0, 0, 1))))


def draw(rng: random.Random) -> dict:
    kind = rng.choice(("select", "select", "select", "select", "whole", "whole", "batched",
                       "project", "error", "quantize", "rank"))
    store = rng.choice(("f32", "f32", "bf16", "fp8"))
    m = _log_int(rng, 100, 8192)
    n = _log_int(rng, max(1000, 2 * m if kind == "rank" else 0), min(1048576, 400_000_000 // m))
    if kind == "select":
        k = min(_log_int(rng, 10, 200), m // 4, n // 8)
        return dict(kind=kind, m=m, n=n, r=_log_int(rng, 16, 512), k=k, store=store,
                    target=rng.choice(("f32", "f32", "bf16")))
    if kind == "whole":
        m = min(m, 4096)
        n = min(n, 100_000)
        return dict(kind=kind, m=m, n=n, k=min(_log_int(rng, 10, 200), m // 4, n // 8), store=store)
    if kind == "batched":
        m, blocks = min(m, 2048), rng.choice((8, 16, 33, 64))
        whi = max(600, min(16384, 300_000_000 // (m * blocks)))
        k = rng.randint(5, 20)
        return dict(kind=kind, m=m, blocks=blocks, wlo=256, whi=whi, wseed=rng.randrange(1 << 20),
                    r=_log_int(rng, 16, 256), k=k, merge=min(_log_int(rng, 10, 100), blocks * k // 2, m // 4),
                    store=store)
    if kind == "project":
        return dict(kind=kind, m=m, n=n, r=_log_int(rng, 16, 512), store=store)
    if kind == "error":
        return dict(kind=kind, m=m, n=n, r=_log_int(rng, 16, 512), k=min(_log_int(rng, 10, 200), m // 4, n // 8),
                    store=store, target="f32")
    if kind == "quantize":
        return dict(kind=kind, m=m, n=n, store=rng.choice(("bf16", "fp8")))
    m, n = min(m, 2048), min(n, 100_000)
    l = max(10, min(_log_int(rng, 10, 200), m // 4))
    return dict(kind=kind, m=m, n=n, l=l, k=max(1, l // 2), store="f32")


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------
_BYTES = {"f32": 4, "bf16": 2, "fp8": 1}


def _lda(m, es):
    per = 256 // es
    return (m + per - 1) // per * per


def _gen(seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return g


def _offsets(case):
    w = random.Random(case["wseed"])
    off = [0]
    for _ in range(case["blocks"]):
        off.append(off[-1] + w.randint(case["wlo"], case["whi"]))
    return off


def _columns(case):
    return _offsets(case)[-1] if case["kind"] == "batched" else case["n"]


def _stored(case, seed):
    """The matrix as a column store (n, lda) in its storage type, and FP8 scales."""
    m, n, store = case["m"], _columns(case), case["store"]
    plain = store if case["kind"] != "quantize" else "f32"
    es = _BYTES[plain]
    dt = {"f32": torch.float32, "bf16": torch.bfloat16, "fp8": torch.float8_e4m3fn}[plain]
    g = _gen(seed)
    rank = max(8, min(256, m // 2))
    s = torch.arange(1, rank + 1, device=DEVICE, dtype=torch.float32) ** -0.5
    basis = torch.randn(rank, m, generator=g, device=DEVICE) * (s / math.sqrt(m))[:, None]
    lda = _lda(m, es)
    out = torch.zeros(n, lda, dtype=dt, device=DEVICE)
    scales = torch.empty(n, device=DEVICE) if plain == "fp8" else None
    for i in range(0, n, CHUNK):
        c = min(CHUNK, n - i)
        blk = torch.randn(c, rank, generator=g, device=DEVICE) @ basis
        blk += (0.2 / math.sqrt(m)) * torch.randn(c, m, generator=g, device=DEVICE)
        blk *= torch.exp(0.5 * torch.randn(c, 1, generator=g, device=DEVICE))
        if plain == "fp8":
            sc = blk.abs().amax(dim=1) / 448.0
            scales[i:i + c] = sc
            blk = blk / sc[:, None]
        out[i:i + c, :m] = blk.to(dt)
    return out, scales


def _values(A, scales, i, c):
    """Columns i .. i+c of a stored matrix in binary32."""
    v = A[i:i + c].float()
    return v * scales[i:i + c, None] if scales is not None else v


def _omega(case, seed):
    g = _gen(seed + 7)
    return torch.randn(_columns(case), case["r"], generator=g, device=DEVICE) / math.sqrt(case["r"])


def _target(case, seed, A, scales):
    """B = A Omega as a column store (r, ldb): the concise target of the matrix."""
    om = _omega(case, seed)
    B = torch.zeros(case["r"], A.shape[1], device=DEVICE)
    for i in range(0, A.shape[0], CHUNK):
        c = min(CHUNK, A.shape[0] - i)
        B += om[i:i + c].T.contiguous() @ _values(A, scales, i, c)
    m = case["m"]
    es = 2 if case.get("target") == "bf16" else 4
    out = torch.zeros(case["r"], _lda(m, es), device=DEVICE, dtype=torch.bfloat16 if es == 2 else torch.float32)
    out[:, :m] = B[:, :m].to(out.dtype)
    return out


def _subset(case, seed):
    g = np.random.default_rng(seed + 13)
    return np.sort(g.choice(case["n"], case["k"], replace=False)).astype(np.int64)


# ---------------------------------------------------------------------------
# the program around one pass, and the pass
# ---------------------------------------------------------------------------
def prepare(case, seed):
    kind, m = case["kind"], case["m"]
    A, scales = _stored(case, seed)
    st = dict(case=case, A=A, scales=scales)
    if kind == "quantize":
        return st
    if kind in ("whole", "rank"):
        kmax = case["l"] if kind == "rank" else case["k"]
        sel = gcss.Selector(A, m, k_max=kmax, self_target=True, scales=scales)
        if kind == "rank":
            sel.set_embedding(torch.empty(kmax, A.shape[0], device=DEVICE))
            sel.set_target(None)
            sel.select(kmax)
    elif kind == "batched":
        off = _offsets(case)
        sel = gcss.Selector(A, m, k_max=case["k"], r_max=case["r"], scales=scales,
                            batched=(case["blocks"], case["k"], case["merge"]))
        sel.set_target(_target(case, seed, A, scales))
        st["off"] = off
    elif kind == "project":
        sel = gcss.Selector(A, m, k_max=16, r_max=case["r"], scales=scales)
        st["omega"] = _omega(case, seed)
    else:
        sel = gcss.Selector(A, m, k_max=case["k"], r_max=case["r"], scales=scales)
        sel.set_target(_target(case, seed, A, scales))
        if kind == "error":
            st["idx"] = _subset(case, seed)
    st["sel"] = sel
    return st


def run(state):
    case, sel = state["case"], state.get("sel")
    kind = case["kind"]
    if kind == "select":
        idx, obj, ns, _ = sel.select(case["k"])
        return dict(idx=idx, obj=obj, ns=ns)
    if kind == "whole":
        sel.set_target(None)
        idx, obj, ns, _ = sel.select(case["k"])
        return dict(idx=idx, obj=obj, ns=ns, err=sel.reconstruction_error(idx[:ns]))
    if kind == "batched":
        ib, im, om, nm, _ = sel.select_batched(state["off"], case["k"], case["merge"])
        return dict(idx_block=ib, idx=im, obj=om, ns=nm)
    if kind == "project":
        return dict(B=sel.project_target(state["omega"])[:, :case["m"]])
    if kind == "error":
        return dict(err=sel.reconstruction_error(state["idx"]))
    if kind == "quantize":
        codes, scales = gcss.quantize_tensor(state["A"], case["m"], case["store"])
        return dict(codes=codes) if scales is None else dict(codes=codes, scales=scales)
    U, sigma, V, err = sel.rank_k(case["l"], case["k"])
    return dict(U=U, sigma=sigma, V=V, err=err)


# ---------------------------------------------------------------------------
# what a pass cannot do without
# ---------------------------------------------------------------------------
def work(case):
    kind, m, n = case["kind"], case["m"], _columns(case)
    es = _BYTES[case["store"]]
    a = float(m) * n * es
    if kind == "quantize":
        return dict(bytes=m * n * 4.0 + a + (4.0 * n if case["store"] == "fp8" else 0), flops=1.0 * m * n)
    if kind == "project":
        r = case["r"]
        # the product and the scores f_i = |B^T A_i|^2
        return dict(bytes=a + 4.0 * n * r + 4.0 * m * r, flops=4.0 * m * n * r)
    if kind == "error":
        r, k = case["r"], case["k"]
        return dict(bytes=float(m) * k * es + 4.0 * m * r, flops=2.0 * m * k * k + 4.0 * m * k * r)
    if kind == "rank":
        l, k = case["l"], case["k"]
        return dict(bytes=4.0 * l * n + 4.0 * k * n + 8.0 * m * (l + k), flops=float(l) * l * n + 2.0 * l * k * (n + m))
    # every step's scores wait for the pick before it, so a matrix that no
    # cache holds is read once per step: the dots with q and z of each column
    k = case["k"]
    steps = k if kind == "whole" else k - 1
    byts = (a if a <= CACHE_BYTES else a * steps) + 32.0 * n
    flops = 4.0 * m * n * steps
    if kind == "whole":
        flops += 2.0 * m * m * n  # the Gram matrix's triangle and the scores from it
        byts += 4.0 * m * m
    elif kind == "batched":
        p, r = float(case["blocks"] * k), case["r"]
        flops += 2.0 * p * (p / 2 + r) * m
        byts += 4.0 * m * r
    else:
        byts += (2.0 if case["target"] == "bf16" else 4.0) * m * case["r"]
    return dict(bytes=byts, flops=flops)


# ---------------------------------------------------------------------------
# the same in 64 bits, in plain torch
# ---------------------------------------------------------------------------
def _wide(A, scales, m):
    out = torch.empty(A.shape[0], m, dtype=torch.float64, device=DEVICE)
    for i in range(0, A.shape[0], CHUNK):
        v = A[i:i + CHUNK, :m].to(torch.float32).double()
        out[i:i + CHUNK] = v * scales[i:i + CHUNK, None].double() if scales is not None else v
    return out


def _greedy(A, B, k, tau=1e-4):
    """Picks, objective and basis (rows) of the greedy selection over the rows
    of A (n, m); B (r, m), or None for B = A."""
    n, m = A.shape
    g = torch.cat([A[i:i + CHUNK].square().sum(1) for i in range(0, n, CHUNK)])
    g0 = g.clone()
    if B is None:
        C = A.T @ A
        f = torch.cat([((A[i:i + CHUNK] @ C) * A[i:i + CHUNK]).sum(1) for i in range(0, n, CHUNK)])
        F = float(g.sum())
    else:
        f = torch.cat([(A[i:i + CHUNK] @ B.T).square().sum(1) for i in range(0, n, CHUNK)])
        F = float(B.square().sum())
    free = torch.ones(n, dtype=torch.bool, device=DEVICE)
    Q = torch.zeros(k, m, dtype=torch.float64, device=DEVICE)
    idx, obj = [], [F]
    for t in range(k):
        p = int(torch.where(free & (g > tau * g0), f / g, torch.full_like(f, -math.inf)).argmax())
        free[p] = False
        q = A[p].clone()
        for _ in range(2):
            q -= Q[:t].T @ (Q[:t] @ q)
        q /= q.norm()
        om = A @ q
        w = A.T @ om if B is None else B.T @ (B @ q)
        u2 = float(q @ w)
        z = w - Q[:t].T @ (Q[:t] @ w)
        f += -2.0 * om * (A @ z) + u2 * om.square()
        g -= om.square()
        Q[t] = q
        idx.append(p)
        obj.append(obj[-1] - u2)
    return idx, np.array(obj), Q


def exact(case, seed):
    kind, m = case["kind"], case["m"]
    if kind == "quantize":
        return None
    A32, scales = _stored(case, seed)
    B = None
    if kind not in ("whole", "rank", "project"):
        B = _target(case, seed, A32, scales)[:, :m].double()
    if kind == "project":
        om = _omega(case, seed)
        B = torch.zeros(case["r"], m, dtype=torch.float64, device=DEVICE)
        for i in range(0, A32.shape[0], CHUNK):
            a = _wide(A32[i:i + CHUNK], None if scales is None else scales[i:i + CHUNK], m)
            B += om[i:i + CHUNK].double().T.contiguous() @ a
        return dict(B=B)
    if kind == "error":
        i = torch.from_numpy(_subset(case, seed)).to(DEVICE)
        S = _wide(A32[i], None if scales is None else scales[i], m)
        Q = torch.linalg.qr(S.T.cpu())[0].T.contiguous().to(DEVICE)
        return dict(err=float((B - (B @ Q.T) @ Q).square().sum()))
    A = _wide(A32, scales, m)
    del A32
    if kind == "select":
        return dict(idx=None, obj=_greedy(A, B, case["k"])[1], ns=None)
    if kind == "whole":
        obj = _greedy(A, None, case["k"])[1]
        return dict(idx=None, obj=obj, ns=None, err=float(obj[-1]))
    if kind == "batched":
        off = _offsets(case)
        pool = []
        for a, b in zip(off, off[1:]):
            pool += [a + i for i in _greedy(A[a:b], B, case["k"])[0]]
        obj = _greedy(A[torch.tensor(pool, device=DEVICE)], B, case["merge"])[1]
        return dict(idx_block=None, idx=None, obj=obj, ns=None)
    _, obj, Q = _greedy(A, None, case["l"])
    W = Q @ A.T
    lam, vec = torch.linalg.eigh((W @ W.T).cpu())
    lam, vec = lam.flip(0).to(DEVICE), vec.flip(1).contiguous().to(DEVICE)
    k = case["k"]
    sigma = lam[:k].clamp(min=0).sqrt()
    U = (Q.T @ vec[:, :k]).T.contiguous()
    sign = torch.sign(U.gather(1, U.abs().argmax(1, keepdim=True)))
    V = (vec[:, :k].T.contiguous() @ W) / sigma[:, None] * sign
    return dict(U=U * sign, sigma=sigma, V=V, err=float(obj[-1]) + float(lam[k:].clamp(min=0).sum()))

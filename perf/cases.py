"""Performance cases of the GRAM step: what a training program has this library do, sized like the
workloads of `workloads.py`, the tests and `bench.py`, plus ragged sizes between them.

Every case goes through the public binding (`paper_2204_04179_amd.gram`).  The kinds:

  window    K steps of one accumulation window (dedup, forward to positions, gradient
            accumulation) and the end of the window (weight gradient and export): a training loop
            between two encoder updates
  dense     the same with the one-row-per-ID buffer, ended by the 64-bit export (windows of epoch
            length)
  unique    the dedup alone (a data loader that wants unique lists ahead of time)
  forward   the forward to positions of a batch whose dedup is in hand
  pseudo    a step that also takes the pseudo-targets and feeds them to the positions
  batch     one content-encoder batch of the regression towards stored pseudo-targets
  mlp_fwd   the forward of the two-layer encoder, activations kept
  mlp_bwd   its backward pass over one content-encoder batch

Inputs are drawn on the GPU from the seed alone: item IDs from a bounded Zipf law through a random
rank-to-ID permutation, normal features, weights and gradients.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2204_04179_amd import gram

BF16, F32 = "bf16", "f32"


def _window(name, B, L, N, s, d_in, d, K, padding="none", dtype=BF16, kind="window", h=F32, d_hidden=0, n=0):
    case = dict(kind=kind, B=B, L=L, N=N, s=s, d_in=d_in, d=d, K=K, padding=padding, dtype=dtype, h=h,
                d_hidden=d_hidden, n=n)
    if name:
        case["name"] = name
    return case


def listed():
    return [
        # the smallest call: a handful of short histories in float32 (a unit test, a tutorial, a smoke run)
        _window("tiny_step_f32", 4, 16, 100, 1.1, 64, 32, 1, "last3", F32),
        # one Single-step update of a knowledge-tracing model, padded histories
        _window("kt_step", 64, 100, 13_000, 1.0, 768, 256, 1, "uniform20"),
        # one Single-step update of a news recommender: large vocabulary, width no power of two
        _window("news_step", 128, 55, 100_000, 1.2, 768, 400, 1),
        # a Multi-step window on the knowledge-tracing shape
        _window("kt_multi_window", 256, 200, 20_000, 0.9, 768, 256, 8),
        # the large Multi-step window: a million items, wide features
        _window("large_window", 1024, 200, 1_000_000, 1.05, 1024, 1024, 4),
        # a long window in the one-row-per-ID buffer, padded histories, 64-bit export
        _window("long_window_dense", 256, 200, 20_000, 0.9, 768, 256, 12, "uniform20", kind="dense"),
        # the dedup alone, ragged number of positions, vocabulary past a power of two
        _window("dedup_ragged", 997, 131, 262_147, 1.05, 64, 32, 1, "uniform20", kind="unique"),
        # the forward of the large batch with the positions stored in bf16
        _window("forward_large_bf16", 1024, 200, 1_000_000, 1.05, 1024, 1024, 1, kind="forward", h=BF16),
        # a step that takes and feeds pseudo-targets, ragged in every size
        _window("pseudo_target_step", 333, 77, 50_021, 1.1, 776, 392, 1, "uniform20", kind="pseudo"),
        # one large content-encoder batch of the regression towards stored targets
        _window("encoder_batch", 1, 32_768, 1_000_000, 1.0, 1024, 1024, 1, kind="batch", n=32_768),
        # the two-layer encoder's forward on a mid-sized news batch
        _window("mlp_forward", 300, 150, 100_000, 1.0, 768, 400, 1, kind="mlp_fwd", d_hidden=1536),
        # and its backward pass over one large batch
        _window("mlp_backward", 1, 32_768, 1_000_000, 1.0, 1024, 1024, 1, kind="mlp_bwd", d_hidden=1024, n=32_768),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges."""
    kind = rng.choice(["window", "window", "window", "dense", "unique", "forward", "pseudo", "batch", "mlp_fwd", "mlp_bwd"])
    d_in, d = 8 * _log(rng, 8, 128), 8 * _log(rng, 4, 128)
    s, padding = rng.choice([0.9, 1.0, 1.05, 1.1, 1.2]), rng.choice(["none", "uniform20", "last3"])
    L = rng.randint(16, 200)
    if kind in ("batch", "mlp_bwd"):
        n = _log(rng, 32, 32_768)
        return _window("", 1, n, _log(rng, max(n + 1, 1000), 1_000_000), 1.0, d_in, d, 1, kind=kind, n=n,
                       d_hidden=8 * _log(rng, 8, 128) if kind == "mlp_bwd" else 0)
    if kind == "dense":
        return _window("", _log(rng, 16, 256), L, _log(rng, 2000, 50_000), s, d_in, d, rng.randint(2, 12), padding, kind=kind)
    B, N = _log(rng, 4, 1024), _log(rng, 100, 1_000_000)
    if kind == "unique":
        return _window("", B, L, N, s, 64, 32, 1, padding, kind=kind)
    h = rng.choice([F32, BF16]) if kind == "forward" else F32
    dtype, K = BF16, 1
    if kind == "window":
        K = rng.choice([1, 1, 2, 4])
        if B * L <= 2048 and d_in * d <= 65_536 and N <= 10_000 and rng.random() < 0.5:
            dtype = F32
    return _window("", B, L, N, s, d_in, d, K, padding, dtype, kind=kind, h=h,
                   d_hidden=8 * _log(rng, 8, 128) if kind == "mlp_fwd" else 0)


# ---- inputs -----------------------------------------------------------------


def _probs(case):
    ranks = np.arange(1, case["N"], dtype=np.float64)
    p = ranks ** (-case["s"])
    return p / p.sum()


def _ids(case, gen, cdf, perm):
    """int32 [B * L] item IDs of one step, 0 = padding."""
    B, L = case["B"], case["L"]
    u = torch.rand((B, L), generator=gen, device="cuda", dtype=torch.float64)
    r = torch.searchsorted(cdf, u).clamp_(max=case["N"] - 2)
    out = perm[r]
    if case["padding"] == "last3":
        out[:, L - 3:] = 0
    elif case["padding"] == "uniform20":
        lens = torch.randint(min(20, L), L + 1, (B, 1), generator=gen, device="cuda")
        out = torch.where(torch.arange(L, device="cuda")[None, :] >= lens, 0, out)
    return out.to(torch.int32).reshape(-1).contiguous()


def _inputs(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 7919 + 1)
    kind, N, d_in, d, K = case["kind"], case["N"], case["d_in"], case["d"], case["K"]
    dt = torch.bfloat16 if case["dtype"] == BF16 else torch.float32
    normal = lambda shape, scale=1.0, dtype=torch.float32: (  # noqa: E731
        torch.randn(shape, generator=gen, device="cuda", dtype=dtype).mul_(scale))
    x = {}
    perm = torch.randperm(N - 1, generator=gen, device="cuda") + 1
    if kind in ("batch", "mlp_bwd"):        # distinct items in no particular order (a shuffled epoch)
        x["ids"] = [perm[: case["n"]].to(torch.int32).contiguous()]
    else:
        p = torch.arange(1, N, device="cuda", dtype=torch.float64).pow_(-case["s"])
        cdf = torch.cumsum(p, 0)
        cdf /= cdf[-1].clone()
        x["ids"] = [_ids(case, gen, cdf, perm) for _ in range(K)]
    if kind == "unique":
        return x
    x["X"] = normal((N, d_in), dtype=dt)
    dh = case["d_hidden"]
    if dh:
        x["W1"], x["W2"] = normal((d_in, dh), d_in ** -0.5, dt), normal((dh, d), dh ** -0.5, dt)
    else:
        x["W"] = normal((d_in, d), d_in ** -0.5, dt)
    if kind in ("batch", "mlp_bwd"):
        x["Ht"] = normal((case["n"], d))
    elif kind in ("window", "dense", "pseudo"):
        x["dH"] = [normal((case["B"] * case["L"], d)) for _ in range(K)]
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    kind, N, d_in, d, K, dh = (case[k] for k in ("kind", "N", "d_in", "d", "K", "d_hidden"))
    M = case["B"] * case["L"]
    g = gram.Gram(gram.make_config(N, d_in, d, M, K, 0, 0, gram.BF16 if case["dtype"] == BF16 else gram.F32,
                                   1 if kind == "dense" else 0, dh, gram.BF16 if case["h"] == BF16 else gram.F32))
    zeros = lambda shape, dtype=torch.float32: torch.zeros(shape, dtype=dtype, device="cuda")  # noqa: E731
    st = dict(x, case=case, g=g, M=M)
    cap = min(M, N)
    st["uniq"], st["counts"] = zeros(cap, torch.int32), zeros(cap, torch.int32)
    st["inverse"], st["u"] = zeros(M, torch.int32), zeros(1, torch.int32)
    if kind == "unique":
        return st
    if kind in ("batch", "mlp_bwd"):
        st["loss"] = zeros(1, torch.float64)
        if dh:
            st["work"] = torch.empty(g.mlp_batch_bytes(case["n"]), dtype=torch.uint8, device="cuda")
            st["dW1"], st["dW2"] = zeros((d_in, dh)), zeros((dh, d))
        else:
            st["R"], st["dW"] = zeros((case["n"], d)), zeros((d_in, d))
        return st
    hdt = torch.bfloat16 if case["h"] == BF16 else torch.float32
    st["H"] = [zeros((M, d), hdt) for _ in range(K)]
    if kind in ("forward", "mlp_fwd"):
        g.unique(x["ids"][0], st["uniq"], st["inverse"], st["counts"], st["u"])
        if dh:
            st["A1"] = zeros((cap, dh), torch.bfloat16)
        return st
    if kind == "pseudo":
        st["E"], st["Ht"], st["Htpos"], st["loss"] = zeros((cap, d)), zeros((cap, d)), zeros((M, d)), zeros(1, torch.float64)
    st["dW"] = zeros((d_in, d))
    rows = N if kind == "dense" else min(K * M, N)
    st["uniq_total"] = zeros(rows, torch.int32)
    st["counts_total"] = zeros(rows, torch.int64 if kind == "dense" else torch.int32)
    st["G_total"], st["u_total"] = zeros((rows, d)), zeros(1, torch.int32)
    return st


def run(st):
    case, g, M = st["case"], st["g"], st["M"]
    kind = case["kind"]
    if kind == "unique":
        g.unique(st["ids"][0], st["uniq"], st["inverse"], st["counts"], st["u"])
        return {k: st[k] for k in ("uniq", "inverse", "counts", "u")}
    if kind == "forward":
        g.encode_gather(st["X"], st["W"], st["uniq"], st["inverse"], st["u"], M, None, st["H"][0])
        return {"H": st["H"][0]}
    if kind == "mlp_fwd":
        g.mlp_encode_gather(st["X"], st["W1"], st["W2"], st["uniq"], st["inverse"], st["u"], M, st["A1"], None, st["H"][0])
        return {"A1": st["A1"], "H": st["H"][0]}
    if kind == "batch":
        g.pseudo_loss_grad(st["X"], st["W"], st["ids"][0], st["Ht"], case["n"], st["R"], st["dW"], False, st["loss"])
        return {"R": st["R"], "dW": st["dW"], "loss": st["loss"]}
    if kind == "mlp_bwd":
        g.mlp_backward(st["X"], st["W1"], st["W2"], st["ids"][0], None, st["Ht"], case["n"], st["work"], st["dW1"],
                       st["dW2"], False, st["loss"])
        return {"dW1": st["dW1"], "dW2": st["dW2"], "loss": st["loss"]}
    for k in range(case["K"]):
        g.unique(st["ids"][k], st["uniq"], st["inverse"], st["counts"], st["u"])
        g.encode_gather(st["X"], st["W"], st["uniq"], st["inverse"], st["u"], M, st.get("E"), st["H"][k])
        g.grad_accumulate(st["dH"][k], M, k)
    out = {k: st[k] for k in ("uniq", "inverse", "counts", "u", "H", "dW", "uniq_total", "counts_total", "G_total", "u_total")}
    if kind == "pseudo":
        g.pseudo_target(st["E"], st["Ht"], st["loss"])
        g.gather(st["Ht"], st["inverse"], M, st["Htpos"])
        out.update({k: st[k] for k in ("E", "Ht", "Htpos", "loss")})
    if kind == "dense":
        g.encoder_wgrad(st["X"], st["dW"])
        g.flush64(st["uniq_total"], st["counts_total"], st["G_total"], st["u_total"])
    else:
        g.window_end(st["X"], st["dW"], st["uniq_total"], st["counts_total"], st["G_total"], st["u_total"])
    return out


# ---- what a pass cannot do without --------------------------------------------


def _expected(case):
    """Expected (unique items of a step, items of the window, unpadded positions of a step)."""
    M, L = case["B"] * case["L"], case["L"]
    lo = min(20, L)
    valid = {"none": 1.0, "last3": (L - 3) / L, "uniform20": (lo + L) / 2 / L}[case["padding"]] * M
    miss = np.log1p(-np.minimum(_probs(case), 1 - 1e-12))
    pad = 1 if case["padding"] != "none" else 0
    return (float(np.sum(-np.expm1(valid * miss))) + pad, float(np.sum(-np.expm1(case["K"] * valid * miss))) + pad, valid)


def work(case):
    d_in, d, K, dh, kind = case["d_in"], case["d"], case["K"], case["d_hidden"], case["kind"]
    s, M, n = (2 if case["dtype"] == BF16 else 4), case["B"] * case["L"], case["n"]
    if kind == "batch":
        return {"bytes": n * (4 + s * d_in + 8 * d) + d_in * d * (s + 4), "flops": 4.0 * n * d_in * d}
    if kind == "mlp_bwd":
        return {"bytes": n * (4 + s * d_in + 4 * d) + dh * (d_in + d) * (s + 4), "flops": n * dh * (4.0 * d_in + 6.0 * d)}
    u, ut, valid = _expected(case)
    dedup = 8 * M + 8 * u
    if kind == "unique":
        return {"bytes": dedup, "flops": 0}
    hs = 2 if case["h"] == BF16 else 4
    if kind == "forward":
        return {"bytes": 4 * M + u * (4 + s * d_in) + s * d_in * d + hs * M * d, "flops": 2.0 * u * d_in * d}
    if kind == "mlp_fwd":
        return {"bytes": 4 * M + u * (4 + s * d_in + 2 * dh) + s * dh * (d_in + d) + hs * M * d,
                "flops": 2.0 * u * dh * (d_in + d)}
    step = dedup + hs * M * d + 4 * valid * d
    total = K * step + ut * (s * d_in + 4 * d + 8) + d_in * d * (s + 4)
    if kind == "pseudo":
        total += 8 * u * d + 4 * M * d
    return {"bytes": total, "flops": 2.0 * (K * u + ut) * d_in * d}


def tolerance(case):
    # float32 results of bf16 or float32 inputs differ by the order of float32 sums (measured 3e-7 to
    # 1e-6 against 64 bits); a weight gradient on bf16 matrix cores rounds one operand to bf16 and a
    # kept activation or a bf16 position is rounded as it is stored (measured 1.5e-3 to 3e-3)
    if case["kind"] == "unique":
        return "exact"
    if case["dtype"] == F32:
        return {"rel": 1e-5}
    return {"rel": 1e-2}


# ---- the same in 64 bits --------------------------------------------------------


def exact(case, seed):
    kind, N, d_in, d, dh, K = (case[k] for k in ("kind", "N", "d_in", "d", "d_hidden", "K"))
    if kind == "unique":
        return None
    x = _inputs(case, seed)
    M, f64 = case["B"] * case["L"], torch.float64
    X = x["X"]

    def rows_of(ids):
        """Features in 64 bits, the padding item's row zero."""
        r = X[ids.long()].to(f64)
        r[ids == 0] = 0
        return r

    if kind in ("batch", "mlp_bwd"):
        ids, Ht = x["ids"][0], x["Ht"].to(f64)
        xr = rows_of(ids)
        if kind == "batch":
            R = xr @ x["W"].to(f64) - Ht
            return {"R": R, "dW": xr.T @ R, "loss": 0.5 * R.square().sum().reshape(1)}
        W2 = x["W2"].to(f64)
        a = (xr @ x["W1"].to(f64)).clamp_(min=0)
        R = a @ W2 - Ht
        dz = (R @ W2.T) * (a > 0)
        return {"dW1": xr.T @ dz, "dW2": a.T @ R, "loss": 0.5 * R.square().sum().reshape(1)}
    cap = min(M, N)
    G = torch.zeros((N, d), dtype=f64, device="cuda") if kind in ("window", "dense", "pseudo") else None
    seen = torch.zeros(N, dtype=torch.bool, device="cuda")
    Hs = []
    for k in range(K):
        uniq, inv = torch.unique(x["ids"][k], sorted=True, return_inverse=True)
        xr = rows_of(uniq)
        if dh:
            a = (xr @ x["W1"].to(f64)).clamp_(min=0)
            E = a @ x["W2"].to(f64)
        else:
            E = xr @ x["W"].to(f64)
        Hs.append(E[inv])
        if G is not None:
            keep = x["ids"][k] != 0
            G.index_add_(0, x["ids"][k][keep].long(), x["dH"][k][keep].to(f64))
            seen[uniq.long()] = True
    if kind == "forward":
        return {"H": Hs[0]}
    full = lambda rows, t: torch.cat([t, torch.zeros((rows - t.shape[0], t.shape[1]), dtype=f64, device="cuda")])  # noqa: E731
    if kind == "mlp_fwd":
        return {"A1": full(cap, a), "H": Hs[0]}
    items = seen.nonzero().reshape(-1)
    rows = N if kind == "dense" else min(K * M, N)
    Gi = G[items]
    dW = torch.zeros((d_in, d), dtype=f64, device="cuda")
    for i in range(0, items.numel(), 65_536):
        dW += rows_of(items[i:i + 65_536]).T @ Gi[i:i + 65_536]
    out = {k: None for k in ("uniq", "inverse", "counts", "u", "uniq_total", "counts_total", "u_total")}
    out.update(H=Hs, dW=dW, G_total=full(rows, Gi))
    if kind == "pseudo":
        Ht = E - G[uniq.long()]
        out.update(E=full(cap, E), Ht=full(cap, Ht), Htpos=Ht[inv], loss=0.5 * G[uniq.long()].square().sum().reshape(1))
    return out

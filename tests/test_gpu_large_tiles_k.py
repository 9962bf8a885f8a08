"""The 256-row contraction where K is no multiple of its slabs of 64: one slab, half a slab, odd and even numbers of slabs with and
without half a slab before them, in every form it stores.  Every row of the features that the batch does not name is NaN: a slab
that took a part of such a row for K would show.  Against float64.  Bounds: float32 sums of K products
of bf16 values, a few 1e-7 of the norm; activations and misses that are stored as bf16 are rounded once (2^-9 per element, 6e-3
of the norm of a product of two such)."""
import pytest

pytestmark = pytest.mark.gpu

ITEMS = 33_025        # 130 row tiles: with two column tiles the 256-row kernel, the last row tiles cut in two


def _features(n, k, ids, torch):
    X = torch.full((n, k), float("nan"), device="cuda", dtype=torch.bfloat16)
    X[ids.long()] = torch.randn(ids.numel(), k, device="cuda", dtype=torch.bfloat16)
    return X


def _forward(gram, torch, n, k, d, h_bf16, last_row):
    ids = (torch.randperm(n - 2, device="cuda")[:ITEMS] + 1).to(torch.int32)
    if last_row:
        ids[7] = n - 1
    X = _features(n, k, ids, torch)
    ids[ITEMS - 1] = 0
    W = (torch.randn(k, d, device="cuda") * k ** -0.5).to(torch.bfloat16)
    g = gram.Gram(gram.make_config(n, k, d, ITEMS, 1, 0, 0, gram.BF16, 0, 0, gram.BF16 if h_bf16 else gram.F32))
    uniq, counts, inverse = (torch.empty(ITEMS, dtype=torch.int32, device="cuda") for _ in range(3))
    u = torch.zeros(1, dtype=torch.int32, device="cuda")
    assert g.unique(ids, uniq, inverse, counts, u, want_host_u=True) == ITEMS
    E = torch.full((ITEMS, d), float("nan"), device="cuda")
    H = torch.full((ITEMS, d), float("nan"), device="cuda", dtype=torch.bfloat16 if h_bf16 else torch.float32)
    g.encode_gather(X, W, uniq, inverse, u, ITEMS, E, H)
    x = X[uniq.long()].double()
    x[uniq == 0] = 0
    want = x @ W.double()
    assert float((E.double() - want).norm(dim=1).max()) <= 2e-6 * float(want.norm(dim=1).max())
    assert bool((E[0] == 0).all()) and torch.equal(H, E[inverse.long()].to(H.dtype))
    g.close()


@pytest.mark.parametrize("k", [32, 64, 96, 128, 160, 192, 224])
@pytest.mark.parametrize("h_bf16", [0, 1])
def test_forward(k, h_bf16):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(k)
    _forward(gram, torch, 60_000, k, 504, h_bf16, True)


def test_forward_of_features_beyond_4_gib():
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(1)
    _forward(gram, torch, 22_400_000, 96, 264, 0, True)      # 4.3 GB, its last row among the items


@pytest.mark.parametrize("k,dh,d", [(32, 288, 512), (96, 480, 352), (128, 512, 320)])
def test_two_layer_backward(k, dh, d):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(k)
    n = 60_000
    ids = torch.randperm(n, device="cuda")[:ITEMS].to(torch.int32)
    X = _features(n, k, ids, torch)
    ids[5] = ids[ITEMS - 1] = 0
    W1 = (torch.randn(k, dh, device="cuda") * k ** -0.5).to(torch.bfloat16)
    W2 = (torch.randn(dh, d, device="cuda") * dh ** -0.5).to(torch.bfloat16)
    Ht, loss = torch.randn(ITEMS, d, device="cuda"), torch.zeros(1, dtype=torch.float64, device="cuda")
    g = gram.Gram(gram.make_config(n, k, d, ITEMS, 1, 0, 0, gram.BF16, 0, dh))
    work = torch.empty(g.mlp_batch_bytes(ITEMS), dtype=torch.uint8, device="cuda")
    dW1, dW2 = torch.empty(k, dh, device="cuda"), torch.empty(dh, d, device="cuda")
    g.mlp_backward(X, W1, W2, ids, None, Ht, ITEMS, work, dW1, dW2, loss_dev=loss)
    x = X[ids.long()].double()
    x[ids == 0] = 0
    a = (x @ W1.double()).clamp(min=0).to(torch.bfloat16).double()
    r = a @ W2.double() - Ht.double()
    r[ids == 0] = 0
    half = 0.5 * float((r ** 2).sum())
    assert abs(float(loss) - half) <= 1e-4 * half
    assert float((dW2.double() - a.T @ r).norm()) <= 6e-3 * float((a.T @ r).norm())
    want = x.T @ ((r @ W2.double().T) * (a > 0))
    assert float((dW1.double() - want).norm()) <= 6e-3 * float(want.norm())
    g.close()


# (up to K = 160, widths from 257 to 320 go to the mid-sized kernel)
@pytest.mark.parametrize("k,d", [(32, 504), (96, 504), (128, 504), (160, 264), (160, 336), (160, 344), (192, 264)])
def test_subtracting(k, d):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(k + 1)
    n = 60_000
    ids = torch.randperm(n, device="cuda")[:ITEMS].to(torch.int32)
    X = _features(n, k, ids, torch)
    ids[5] = ids[ITEMS - 1] = 0
    W = (torch.randn(k, d, device="cuda") * k ** -0.5).to(torch.bfloat16)
    Ht, R, dW = torch.randn(ITEMS, d, device="cuda"), torch.empty(ITEMS, d, device="cuda"), torch.empty(k, d, device="cuda")
    g = gram.Gram(gram.make_config(n, k, d, ITEMS, 1, 0, 0, gram.BF16))
    g.pseudo_loss_grad(X, W, ids, Ht, ITEMS, R, dW)
    x = X[ids.long()].double()
    x[ids == 0] = 0
    want = x @ W.double() - Ht.double()
    want[ids == 0] = 0
    assert float((R.double() - want).norm(dim=1).max()) <= 2e-6 * float(want.norm(dim=1).max())
    assert float((dW.double() - x.T @ want).norm()) <= 6e-3 * float((x.T @ want).norm())
    g.close()

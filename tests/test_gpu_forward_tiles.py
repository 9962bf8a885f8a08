"""The forward of small and mid-sized batches (tiles of 64 x 64 and 128 x 64, K cut between two wave groups; tiles of 128 x 128
for long K) and of large ones (tiles of 256 x 256) against a float64 product, at the item counts and widths where tiles, slabs
of 64 and the number of groups end, and where the tile shape changes.  Bound: float32 sums of K products of bf16 values, a few
1e-7 of the norm; bf16 results are rounded once (2^-9 per element)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("items,k,d", [(1, 8, 8), (63, 64, 64), (65, 72, 72), (129, 136, 136), (640, 192, 512),
                                       (1281, 200, 520), (2600, 320, 512), (5200, 264, 264), (9000, 512, 128)])
@pytest.mark.parametrize("pads", [0, 1])
def test_every_row_against_float64(items, k, d, pads):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(items + d)
    n = 10_000
    X = torch.randn(n, k, device="cuda", dtype=torch.bfloat16)
    W = (torch.randn(k, d, device="cuda") * k ** -0.5).to(torch.bfloat16)
    ids = (torch.randperm(n - 1, device="cuda")[:items] + 1).to(torch.int32)
    ids[items // 2] = 0 if pads else ids[items // 2]
    cap = min(2 * items, n)
    g = gram.Gram(gram.make_config(n, k, d, 2 * items, 1, 0, 0, gram.BF16))
    both = torch.cat([ids, ids])
    uniq, counts = (torch.full((cap,), 2**31 - 1, dtype=torch.int32, device="cuda") for _ in range(2))
    inverse = torch.empty(2 * items, dtype=torch.int32, device="cuda")
    u = torch.zeros(1, dtype=torch.int32, device="cuda")
    E = torch.full((cap, d), float("nan"), device="cuda")
    H = torch.full((2 * items, d), float("nan"), device="cuda")
    assert g.unique(both, uniq, inverse, counts, u, want_host_u=True) == items
    # (entries of uniq behind the items stay what they were: the foreign buffers below hold IDs that do not exist)
    for uq in (uniq, uniq.clone()):
        E.fill_(float("nan"))
        g.encode_gather(X, W, uq, inverse, u, 2 * items, E, H)
        want = X[uniq[:items].long()].double() @ W.double()
        want[uniq[:items] == 0] = 0
        err = float((E[:items].double() - want).norm()) / max(float(want.norm()), 1e-30)
        assert err < 2e-6, err
        assert bool(torch.isnan(E[items:]).all())
        assert torch.equal(H, E[inverse.long()])
        if pads:
            assert bool((E[0] == 0).all())
    g.close()


@pytest.mark.parametrize("items,k,dh,d", [(70, 72, 136, 72), (3000, 200, 264, 136)])
def test_rectified_and_subtracting_forms(items, k, dh, d):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(items)
    n = 6000
    X = torch.randn(n, k, device="cuda", dtype=torch.bfloat16)
    W1 = (torch.randn(k, dh, device="cuda") * k ** -0.5).to(torch.bfloat16)
    W2 = (torch.randn(dh, d, device="cuda") * dh ** -0.5).to(torch.bfloat16)
    ids = torch.randperm(n, device="cuda")[:items].to(torch.int32)
    ids[3] = 0
    g = gram.Gram(gram.make_config(n, k, d, n, 1, 0, 0, gram.BF16, 0, dh))
    uniq, counts = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    inverse, u = torch.empty(items, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    U = g.unique(ids, uniq, inverse, counts, u, want_host_u=True)
    A1 = torch.empty(n, dh, device="cuda", dtype=torch.bfloat16)
    H = torch.empty(items, d, device="cuda")
    g.mlp_encode_gather(X, W1, W2, uniq, inverse, u, items, A1, None, H)
    x = X[uniq[:U].long()].double()
    x[uniq[:U] == 0] = 0
    a = (x @ W1.double()).clamp(min=0)
    assert float((A1[:U].double() - a).norm()) <= 3e-3 * float(a.norm())
    want = A1[:U].double() @ W2.double()
    assert float((H.double() - want[inverse.long()]).norm()) <= 2e-6 * float(want[inverse.long()].norm())
    g.close()
    g = gram.Gram(gram.make_config(n, k, dh, n, 1, 0, 0, gram.BF16))
    Ht, R, dW = torch.randn(items, dh, device="cuda"), torch.empty(items, dh, device="cuda"), torch.empty(k, dh, device="cuda")
    g.pseudo_loss_grad(X, W1, ids, Ht, items, R, dW)
    x = X[ids.long()].double()
    want = x @ W1.double() - Ht.double()
    want[ids == 0] = 0
    assert float((R.double() - want).norm()) <= 2e-6 * float(want.norm())
    assert bool((R[ids == 0] == 0).all())
    g.close()


# 256-row tiles of which the last ones are cut in two: around the edges of halves, around the most that are
# cut (64 row tiles with two column tiles on 256 CUs), none left over, one row left over.
@pytest.mark.parametrize("items", [1, 127, 129, 257, 16_384, 16_385, 32_768, 32_769, 33_025, 49_153])
@pytest.mark.parametrize("h_bf16", [0, 1])
def test_large_tiles_cut_at_the_end(items, h_bf16):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(items)
    n, k, d, m = 60_000, 64, 504, 50_000
    X = torch.randn(n, k, device="cuda", dtype=torch.bfloat16)
    W = (torch.randn(k, d, device="cuda") * k ** -0.5).to(torch.bfloat16)
    pool = (torch.randperm(n - 1, device="cuda")[:items] + 1).to(torch.int32)
    pool[items - 1] = 0
    ids = pool[torch.arange(m, device="cuda") % items]
    g = gram.Gram(gram.make_config(n, k, d, m, 1, 0, 0, gram.BF16, 0, 0, gram.BF16 if h_bf16 else gram.F32))
    uniq, counts = (torch.empty(m, dtype=torch.int32, device="cuda") for _ in range(2))
    inverse, u = torch.empty(m, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    assert g.unique(ids, uniq, inverse, counts, u, want_host_u=True) == items
    E = torch.full((m, d), float("nan"), device="cuda")
    H = torch.full((m, d), float("nan"), device="cuda", dtype=torch.bfloat16 if h_bf16 else torch.float32)
    g.encode_gather(X, W, uniq, inverse, u, m, E, H)
    want = X[uniq[:items].long()].double() @ W.double()
    want[uniq[:items] == 0] = 0
    err = (E[:items].double() - want).norm(dim=1) / want.norm(dim=1).clamp(min=1e-30)
    assert float(err.max()) < 2e-6
    assert bool((E[0] == 0).all()) and bool(torch.isnan(E[items:]).all())
    assert torch.equal(H, E[inverse.long()].to(H.dtype))
    E2 = torch.full((m, d), float("nan"), device="cuda", dtype=H.dtype)
    g.encode_gather(X, W, uniq, inverse, u, m, None, E2)
    assert torch.equal(H, E2)
    g.close()


@pytest.mark.parametrize("items", [32_769, 40_000, 49_153])
def test_large_subtracting_tiles_cut_at_the_end(items):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(items)
    n, k, d = 60_000, 64, 504
    X = torch.randn(n, k, device="cuda", dtype=torch.bfloat16)
    W = (torch.randn(k, d, device="cuda") * k ** -0.5).to(torch.bfloat16)
    ids = (torch.randperm(n - 1, device="cuda")[:items] + 1).to(torch.int32)
    ids[items - 1] = 0
    Ht, R, dW = torch.randn(items, d, device="cuda"), torch.empty(items, d, device="cuda"), torch.empty(k, d, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    g = gram.Gram(gram.make_config(n, k, d, items, 1, 0, 0, gram.BF16))
    g.pseudo_loss_grad(X, W, ids, Ht, items, R, dW, loss_dev=loss)
    want = X[ids.long()].double() @ W.double() - Ht.double()
    want[ids == 0] = 0
    assert float((R.double() - want).norm(dim=1).max()) <= 2e-6 * float(want.norm(dim=1).max())
    assert bool((R[ids == 0] == 0).all())
    half_sum = 0.5 * float((R.double() ** 2).sum())
    assert abs(float(loss) - half_sum) < 1e-9 * half_sum
    g.close()


# lists trimmed to the items, and hidden activations that end (or turn into NaN) behind their rows: item counts
# inside a tile, in the tiles of 64 columns (those of 128 x 128: below)
@pytest.mark.parametrize("items,m,dh", [(70, 900, 136), (641, 8000, 520), (2500, 20_000, 520)])
def test_lists_and_activations_that_end_with_the_items(items, m, dh):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(items)
    n, k, d = 50_000, 200, 136
    X = torch.randn(n, k, device="cuda", dtype=torch.bfloat16)
    W1 = (torch.randn(k, dh, device="cuda") * k ** -0.5).to(torch.bfloat16)
    W2 = (torch.randn(dh, d, device="cuda") * dh ** -0.5).to(torch.bfloat16)
    pool = torch.randperm(n, device="cuda")[:items].to(torch.int32)
    ids = pool[torch.arange(m, device="cuda") % items]
    g = gram.Gram(gram.make_config(n, k, d, m, 1, 0, 0, gram.BF16, 0, dh))
    uniq, counts = (torch.empty(m, dtype=torch.int32, device="cuda") for _ in range(2))
    inverse, u = torch.empty(m, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    assert g.unique(ids, uniq, inverse, counts, u, want_host_u=True) == items
    x = X[uniq[:items].long()].double()
    x[uniq[:items] == 0] = 0
    a = (x @ W1.double()).clamp(min=0)
    for trimmed in (uniq, uniq[:items].clone()):
        kept = torch.full((items + 300, dh), float("nan"), device="cuda", dtype=torch.bfloat16)
        H = torch.full((m, d), float("nan"), device="cuda")
        g.mlp_encode_gather(X, W1, W2, trimmed, inverse if trimmed is uniq else inverse.clone(), u, m, kept[:items], None, H)
        assert bool(torch.isnan(kept[items:]).all())
        A1 = kept[:items]
        assert float((A1.double() - a).norm()) <= 3e-3 * float(a.norm())
        want = (A1.double() @ W2.double())[inverse.long()]
        assert float((H.double() - want).norm()) <= 2e-6 * float(want.norm())
    g.close()


# The rectified and the two subtracting forms in each tile shape: 64 rows up to one tile per CU (256 of them; five
# column tiles: 51 row tiles), 128 rows beyond, 128 x 128 for long K and more than 640 of the small tiles.
@pytest.mark.parametrize("items,k", [(3264, 200), (3265, 200), (7000, 200), (9000, 264), (9000, 392)])
def test_forms_in_every_tile_shape(items, k):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(items + k)
    n, dh, d = 20_000, 264, 264
    X = torch.randn(n, k, device="cuda", dtype=torch.bfloat16)
    W1 = (torch.randn(k, dh, device="cuda") * k ** -0.5).to(torch.bfloat16)
    W2 = (torch.randn(dh, d, device="cuda") * dh ** -0.5).to(torch.bfloat16)
    ids = torch.randperm(n, device="cuda")[:items].to(torch.int32)
    ids[items - 1] = ids[70] = 0
    x = X[ids.long()].double()
    x[ids == 0] = 0
    # subtracting, float32 result and the block sums of the pseudo-loss
    g = gram.Gram(gram.make_config(n, k, dh, n, 1, 0, 0, gram.BF16))
    Ht, R, dW = torch.randn(items, dh, device="cuda"), torch.empty(items, dh, device="cuda"), torch.empty(k, dh, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    g.pseudo_loss_grad(X, W1, ids, Ht, items, R, dW, loss_dev=loss)
    want = x @ W1.double() - Ht.double()
    want[ids == 0] = 0
    assert float((R.double() - want).norm(dim=1).max()) <= 2e-6 * float(want.norm(dim=1).max())
    half = 0.5 * float((R.double() ** 2).sum())
    assert abs(float(loss) - half) <= 1e-9 * half
    g.close()
    # rectified (bf16), and subtracting with a bf16 result: the two-layer backward.  Activations and misses are
    # rounded to bf16 once each, 2^-9 per element
    g = gram.Gram(gram.make_config(n, k, d, n, 1, 0, 0, gram.BF16, 0, dh))
    work = torch.empty(g.mlp_batch_bytes(items), dtype=torch.uint8, device="cuda")
    dW1, dW2 = torch.empty(k, dh, device="cuda"), torch.empty(dh, d, device="cuda")
    g.mlp_backward(X, W1, W2, ids, None, Ht, items, work, dW1, dW2, loss_dev=loss)
    a = (x @ W1.double()).clamp(min=0).to(torch.bfloat16).double()
    r = a @ W2.double() - Ht.double()
    r[ids == 0] = 0
    half = 0.5 * float((r ** 2).sum())
    assert abs(float(loss) - half) <= 1e-4 * half
    assert float((dW2.double() - a.T @ r).norm()) <= 6e-3 * float((a.T @ r).norm())
    want = x.T @ ((r @ W2.double().T) * (a > 0))
    assert float((dW1.double() - want).norm()) <= 6e-3 * float(want.norm())
    # rectified, item order of a dedup
    uniq, counts, inverse = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(3))
    u = torch.zeros(1, dtype=torch.int32, device="cuda")
    U = g.unique(ids, uniq, inverse, counts, u, want_host_u=True)
    A1, H = torch.full((n, dh), float("nan"), device="cuda", dtype=torch.bfloat16), torch.empty(items, d, device="cuda")
    g.mlp_encode_gather(X, W1, W2, uniq, inverse, u, items, A1, None, H)
    x = X[uniq[:U].long()].double()
    x[uniq[:U] == 0] = 0
    a = (x @ W1.double()).clamp(min=0)
    assert float((A1[:U].double() - a).norm()) <= 3e-3 * float(a.norm()) and bool(torch.isnan(A1[U:]).all())
    want = (A1[:U].double() @ W2.double())[inverse[:items].long()]
    assert float((H.double() - want).norm()) <= 2e-6 * float(want.norm())
    g.close()


# Around the number of items from which the row tile changes (nine column tiles: 28 row tiles of 64, 1,792 items on 256
# CUs), with the bound that the grid is made for at the items and far above them.
@pytest.mark.parametrize("items", [1, 1791, 1792, 1793, 1856, 2048])
@pytest.mark.parametrize("m", [0, 3584, 9000])
def test_row_tile_chosen_on_the_device(items, m):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(items + m)
    n, k, d = 30_000, 136, 520
    m = max(m, items)
    X = torch.randn(n, k, device="cuda", dtype=torch.bfloat16)
    W = (torch.randn(k, d, device="cuda") * k ** -0.5).to(torch.bfloat16)
    pool = torch.randperm(n, device="cuda")[:items].to(torch.int32)
    pool[items // 2] = 0
    ids = pool[torch.arange(m, device="cuda") % items]
    items = int(torch.unique(ids).numel())
    g = gram.Gram(gram.make_config(n, k, d, m, 1, 0, 0, gram.BF16))
    uniq, counts, inverse = (torch.empty(m, dtype=torch.int32, device="cuda") for _ in range(3))
    u = torch.zeros(1, dtype=torch.int32, device="cuda")
    assert g.unique(ids, uniq, inverse, counts, u, want_host_u=True) == items
    E, H = torch.full((m, d), float("nan"), device="cuda"), torch.full((m, d), float("nan"), device="cuda")
    g.encode_gather(X, W, uniq, inverse, u, m, E, H)
    want = X[uniq[:items].long()].double() @ W.double()
    want[uniq[:items] == 0] = 0
    err = (E[:items].double() - want).norm(dim=1) / want.norm(dim=1).clamp(min=1e-30)
    assert float(err.max()) < 2e-6
    assert bool(torch.isnan(E[items:]).all()) and torch.equal(H, E[inverse.long()])
    g.close()


# 128 x 128 tiles (K above 256 and more than 640 tiles of 64 x 64 by the host's guess of the items, here 0.6 of the rows there is
# room for) with far fewer items than that, inside and around the edges of a tile: lists and activations that end with the items,
# nothing stored behind them
@pytest.mark.parametrize("items", [1, 127, 128, 129, 2500, 19_999])
def test_square_tiles_with_few_items(items):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(items)
    n, m, k, dh, d = 20_000, 51_200, 264, 776, 392
    guess = min(m, n) * 3 // 5
    assert n <= m < 8 * n and all(kk > 256 and (guess + 63) // 64 * ((c + 63) // 64) * 2 > 5 * 256 for kk, c in ((k, dh), (dh, d)))
    X = torch.randn(n, k, device="cuda", dtype=torch.bfloat16)
    W1 = (torch.randn(k, dh, device="cuda") * k ** -0.5).to(torch.bfloat16)
    W2 = (torch.randn(dh, d, device="cuda") * dh ** -0.5).to(torch.bfloat16)
    pool = torch.randperm(n, device="cuda")[:items].to(torch.int32)
    if items > 2:
        pool[0] = 0
    ids = pool[torch.arange(m, device="cuda") % items]
    items = int(torch.unique(ids).numel())
    g = gram.Gram(gram.make_config(n, k, d, m, 1, 0, 0, gram.BF16, 0, dh))
    uniq, counts = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    inverse, u = torch.empty(m, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    assert g.unique(ids, uniq, inverse, counts, u, want_host_u=True) == items
    x = X[uniq[:items].long()].double()
    x[uniq[:items] == 0] = 0
    a = (x @ W1.double()).clamp(min=0)
    for trimmed in (uniq, uniq[:items].clone()):
        kept = torch.full((items + 300, dh), float("nan"), device="cuda", dtype=torch.bfloat16)
        E, H = torch.full((n, d), float("nan"), device="cuda"), torch.full((m, d), float("nan"), device="cuda")
        g.mlp_encode_gather(X, W1, W2, trimmed, inverse if trimmed is uniq else inverse.clone(), u, m, kept[:items], E, H)
        assert bool(torch.isnan(kept[items:]).all()) and bool(torch.isnan(E[items:]).all())
        A1 = kept[:items]
        assert float((A1.double() - a).norm(dim=1).max()) <= 3e-3 * float(a.norm(dim=1).max())
        want = A1.double() @ W2.double()
        assert float((E[:items].double() - want).norm(dim=1).max()) <= 2e-6 * float(want.norm(dim=1).max())
        assert torch.equal(H, E[inverse.long()])
    g.close()

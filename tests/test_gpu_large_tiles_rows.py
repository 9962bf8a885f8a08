"""The 256-row contraction where the rows end inside a tile: 1, 127, 129 and 255 rows past one, in tiles of 256 rows and in the
halves that the last ones are cut into (two column tiles on 256 CUs: up to 64 row tiles behind a full round are cut), in the forms
that store straight from the accumulators.  Nothing behind the rows may change: activations and representations that end in
NaN, a workspace of known bytes.  Against float64, row by row.  Bounds: what is stored as bf16 is rounded once (2^-9 per element,
2^-8 with the float32 sums of values that were rounded before); float32 sums of K products a few 1e-7 of the norm."""
import pytest

pytestmark = pytest.mark.gpu

N, K, DH, D = 60_000, 64, 480, 504
# 101 and 193 row tiles: whole ones; 129: cut in two
ROWS = [r + e for r in (25_600, 32_768, 49_152) for e in (1, 127, 129, 255)]


def _close(got, want, tol):
    assert float((got.double() - want).norm(dim=1).max()) <= tol * float(want.norm(dim=1).max())


def _weights(torch, k, dh, d):
    X = torch.randn(N, k, device="cuda", dtype=torch.bfloat16)
    W1 = (torch.randn(k, dh, device="cuda") * k ** -0.5).to(torch.bfloat16)
    W2 = (torch.randn(dh, d, device="cuda") * dh ** -0.5).to(torch.bfloat16)
    return X, W1, W2


@pytest.mark.parametrize("items", [1, 127, 129, 255] + ROWS)
def test_rectified_and_plain(items):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(items)
    X, W1, W2 = _weights(torch, K, DH, D)
    m = 50_000
    pool = torch.randperm(N, device="cuda")[:items].to(torch.int32)
    pool[0] = 0 if items > 1 else pool[0]
    ids = pool[torch.arange(m, device="cuda") % items]
    items = int(torch.unique(ids).numel())
    g = gram.Gram(gram.make_config(N, K, D, m, 1, 0, 0, gram.BF16, 0, DH))
    uniq, counts, inverse = (torch.empty(m, dtype=torch.int32, device="cuda") for _ in range(3))
    u = torch.zeros(1, dtype=torch.int32, device="cuda")
    assert g.unique(ids, uniq, inverse, counts, u, want_host_u=True) == items
    x = X[uniq[:items].long()].double()
    x[uniq[:items] == 0] = 0
    a = (x @ W1.double()).clamp(min=0)
    # the call's own lists (positions stored by the contraction) and the caller's (rows stored, then gathered)
    for uq, inv in ((uniq, inverse), (uniq[:items].clone(), inverse.clone())):
        kept = torch.full((items + 300, DH), float("nan"), device="cuda", dtype=torch.bfloat16)
        E, H = torch.full((m + 300, D), float("nan"), device="cuda"), torch.full((m, D), float("nan"), device="cuda")
        g.mlp_encode_gather(X, W1, W2, uq, inv, u, m, kept[:items], E, H)
        _close(kept[:items], a, 2.0 ** -8)
        _close(E[:items], kept[:items].double() @ W2.double(), 2e-6)
        assert torch.equal(H, E[inverse.long()])
        assert bool(kept[items:].isnan().all()) and bool(E[items:].isnan().all())
    g.close()


@pytest.mark.parametrize("n", ROWS[4:])
def test_rectified_and_gated(n):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(n)
    d = 512
    X, W1, W2 = _weights(torch, K, DH, d)
    ids = torch.randperm(N, device="cuda")[:n].to(torch.int32)
    ids[n // 2] = ids[n - 1] = 0
    Ht = torch.randn(n, d, device="cuda")
    g = gram.Gram(gram.make_config(N, K, d, n, 1, 0, 0, gram.BF16, 0, DH))
    work = torch.full((g.mlp_batch_bytes(n),), 0x5A, dtype=torch.uint8, device="cuda")
    dW1, dW2 = torch.empty(K, DH, device="cuda"), torch.empty(DH, d, device="cuda")
    g.mlp_backward(X, W1, W2, ids, None, Ht, n, work, dW1, dW2)
    # the parts of the workspace: dL/dz (bf16, half of its part), activations, a part that is not used, misses (bf16)
    up = lambda b: (b + 255) // 256 * 256  # noqa: E731
    at = [0, up(n * DH * 4), up(n * DH * 4) + up(n * DH * 2)]
    at.append(at[2] + up(n * d * 4))
    z, a = (work[o:o + n * DH * 2].view(torch.bfloat16).view(n, DH) for o in at[:2])
    r = work[at[3]:at[3] + n * d * 2].view(torch.bfloat16).view(n, d)
    x = X[ids.long()].double()
    x[ids == 0] = 0
    _close(a, (x @ W1.double()).clamp(min=0), 2.0 ** -8)
    want = a.double() @ W2.double() - Ht.double()
    want[ids == 0] = 0
    _close(r, want, 2.0 ** -8)
    _close(z, (r.double() @ W2.double().T) * (a > 0), 2.0 ** -8)
    assert bool((z[ids == 0] == 0).all()) and bool((r[ids == 0] == 0).all())
    for lo, hi in ((n * DH * 2, at[1]), (at[1] + n * DH * 2, at[3]), (at[3] + n * d * 2, work.numel())):
        assert bool((work[lo:hi] == 0x5A).all())
    g.close()


# widths that are no multiple of 8: the weights are read from a transposed copy
@pytest.mark.parametrize("n", [32_769, 32_895, 49_153, 49_407])
@pytest.mark.parametrize("k,d", [(32, 508), (64, 508), (96, 508), (256, 300)])
def test_subtracting_from_a_transposed_copy(n, k, d):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(n + k)
    X = torch.randn(N, k, device="cuda", dtype=torch.bfloat16)
    W = (torch.randn(k, d, device="cuda") * k ** -0.5).to(torch.bfloat16)
    ids = torch.randperm(N, device="cuda")[:n].to(torch.int32)
    ids[n // 2] = ids[n - 1] = 0
    Ht, R, dW = torch.randn(n, d, device="cuda"), torch.full((n + 300, d), float("nan"), device="cuda"), torch.empty(k, d, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    g = gram.Gram(gram.make_config(N, k, d, n, 1, 0, 0, gram.BF16))
    g.pseudo_loss_grad(X, W, ids, Ht, n, R[:n], dW, loss_dev=loss)
    x = X[ids.long()].double()
    x[ids == 0] = 0
    want = x @ W.double() - Ht.double()
    want[ids == 0] = 0
    _close(R[:n], want, 2e-6)
    assert bool((R[:n][ids == 0] == 0).all()) and bool(R[n:].isnan().all())
    half = 0.5 * float((R[:n].double() ** 2).sum())
    assert abs(float(loss) - half) <= 1e-9 * half
    g.close()

"""Content-encoder batches in which the padding ID stands any number of times (a last batch filled up to a fixed
size, IDs out of range): no such row may enter the miss, the loss or a weight gradient, whatever kernel the size of the
batch selects.  Against float64.  Bounds: the miss of the linear encoder is a float32 sum (a few 1e-7 of the norm,
float32 sums of K products); activations, misses and dL/dz of the two-layer encoder are rounded to bf16 (2^-9 per
element, 2e-3 of the norm of a product of two such), likewise one operand of the linear weight gradient."""
import pytest

pytestmark = pytest.mark.gpu

PAD, N = 5, 60_000


def _ids(n, share, torch):
    ids = torch.randperm(N, device="cuda")[:n].to(torch.int32)
    ids[torch.rand(n, device="cuda") < share] = PAD
    ids[n // 2:n // 2 + 3] = PAD               # neighbours, whatever was drawn
    return ids


def _rows(X, ids):
    x = X[ids.long()].double()
    x[ids == PAD] = 0
    return x


def _close(got, want, tol):
    assert float((got.double() - want).norm()) <= tol * float(want.norm())


# 300 items: 64-row tiles; 3,000: the mid-sized forward; 33,025: 256-row tiles, the last ones cut in two
@pytest.mark.parametrize("n", [300, 3000, 33_025])
@pytest.mark.parametrize("share", [0.01, 0.5])
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_linear_encoder(n, share, dtype):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(n)
    if dtype == "f32" and n > 3000:
        n = 4097
    k, d = 64, 504
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    X = torch.randn(N, k, device="cuda", dtype=dt)
    W = (torch.randn(k, d, device="cuda") * k ** -0.5).to(dt)
    ids, Ht = _ids(n, share, torch), torch.randn(n, d, device="cuda")
    R, dW = torch.full((n, d), float("nan"), device="cuda"), torch.empty(k, d, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    g = gram.Gram(gram.make_config(N, k, d, n, 1, PAD, 0, gram.BF16 if dtype == "bf16" else gram.F32))
    g.pseudo_loss_grad(X, W, ids, Ht, n, R, dW, loss_dev=loss)
    x = _rows(X, ids)
    want = x @ W.double() - Ht.double()
    want[ids == PAD] = 0
    assert bool((R[ids == PAD] == 0).all())
    _close(R, want, 2e-6)
    half = 0.5 * float((R.double() ** 2).sum())
    assert abs(float(loss) - half) <= 1e-9 * half
    _close(dW, x.T @ want, 6e-3 if dtype == "bf16" else 2e-6)
    g.close()


@pytest.mark.parametrize("n", [300, 3000, 33_025])
@pytest.mark.parametrize("share", [0.01, 0.5])
@pytest.mark.parametrize("targets", [True, False])
def test_two_layer_encoder(n, share, targets):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(n + 1)
    k, dh, d = 64, 512, 512
    X = torch.randn(N, k, device="cuda", dtype=torch.bfloat16)
    W1 = (torch.randn(k, dh, device="cuda") * k ** -0.5).to(torch.bfloat16)
    W2 = (torch.randn(dh, d, device="cuda") * dh ** -0.5).to(torch.bfloat16)
    ids, rows = _ids(n, share, torch), torch.randn(n, d, device="cuda")
    g = gram.Gram(gram.make_config(N, k, d, n, 1, PAD, 0, gram.BF16, 0, dh))
    work = torch.empty(g.mlp_batch_bytes(n), dtype=torch.uint8, device="cuda")
    dW1, dW2 = torch.empty(k, dh, device="cuda"), torch.empty(dh, d, device="cuda")
    loss = torch.zeros(1, dtype=torch.float64, device="cuda")
    bad = ids.clone()
    bad[n // 2 + 1] = N                        # counts as the padding item (and is reported, below)
    g.mlp_backward(X, W1, W2, bad, None if targets else rows, rows if targets else None, n, work, dW1, dW2,
                   loss_dev=loss if targets else None)
    x = _rows(X, ids)
    a = (x @ W1.double()).clamp(min=0).to(torch.bfloat16).double()
    r = a @ W2.double() - rows.double() if targets else rows.double().clone()
    r[ids == PAD] = 0
    if targets:
        # the squares' sum follows a, whose roundings differ from the kernel's in a few last places of 2^-9
        half = 0.5 * float((r ** 2).sum())
        assert abs(float(loss) - half) <= 1e-4 * half
    _close(dW2, a.T @ r, 6e-3)
    _close(dW1, x.T @ ((r @ W2.double().T) * (a > 0)), 6e-3)
    with pytest.raises(gram.GramError) as e:
        g.check()
    assert e.value.status == gram.ERR_RANGE
    g.close()

"""The weight gradient of bf16 rows by a row list (first layer of the two-layer encoder) in batches too long for the short kernel:
numbers of rows that end inside a group of four entries of the list and inside a slab of 32, ranges of slabs that differ between
blocks, features and columns that end inside a tile of 256, shuffled IDs, padding any number of times and IDs out of range.  The last rows
weigh as much as all others together, so that a lost or a wrong one shows.  Against float64.  Bound: dL/dz is rounded to bf16
once as it is stored, from rows and activations that were (2^-9 per element each): 6e-3 of the norm."""
import pytest

pytestmark = pytest.mark.gpu

N = 60_000


@pytest.mark.parametrize("n", [32_769, 32_770, 32_771, 33_025, 40_000])
@pytest.mark.parametrize("k,dh", [(776, 520), (520, 776), (512, 512)])
def test_last_entries_of_the_list(n, k, dh):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(n + k)
    d = 64
    # the size rule of the short kernel (128 x 64 tiles times rows) does not take it
    tiles = (k + 127) // 128 * ((dh + 63) // 64)
    assert n * tiles > (650_000 if tiles <= 32 else 450_000)
    X = torch.randn(N, k, device="cuda", dtype=torch.bfloat16)
    W1 = (torch.randn(k, dh, device="cuda") * k ** -0.5).to(torch.bfloat16)
    W2 = (torch.randn(dh, d, device="cuda") * dh ** -0.5).to(torch.bfloat16)
    ids = torch.randperm(N - 1, device="cuda")[:n].to(torch.int32) + 1
    pad = torch.rand(n, device="cuda") < 0.5
    pad[:3], pad[n - 4:] = False, False
    ids[pad] = 0
    rows = torch.randn(n, d, device="cuda")
    rows[n - 3:] *= 100.0
    g = gram.Gram(gram.make_config(N, k, d, n, 1, 0, 0, gram.BF16, 0, dh))
    work = torch.empty(g.mlp_batch_bytes(n), dtype=torch.uint8, device="cuda")
    dW1, dW2 = torch.empty(k, dh, device="cuda"), torch.empty(dh, d, device="cuda")
    given = ids.clone()
    given[n // 3], given[n // 3 + 1] = N, -1          # count as padding (and are reported)
    ids[n // 3:n // 3 + 2] = 0
    x = X[ids.long()].double()
    x[ids == 0] = 0
    a = (x @ W1.double()).clamp(min=0).to(torch.bfloat16).double()
    r = rows.to(torch.bfloat16).double()
    want = x.T @ ((r @ W2.double().T) * (a > 0))
    for acc in (False, True):
        g.mlp_backward(X, W1, W2, given, rows, None, n, work, dW1, dW2, accumulate=acc)
        assert float((dW1.double() - (2 if acc else 1) * want).norm()) <= 6e-3 * (2 if acc else 1) * float(want.norm())
        assert float((dW2.double() - (2 if acc else 1) * (a.T @ r)).norm()) <= 6e-3 * (2 if acc else 1) * float((a.T @ r).norm())
    # any one of the last rows missing would show
    z = (r @ W2.double().T) * (a > 0)
    assert all(float(torch.outer(x[n - j], z[n - j]).norm()) > 0.1 * float(want.norm()) for j in (1, 2, 3))
    g.close()

"""The weight gradient of short windows (tiles of 128 x 64, ranges of rows over blocks and wave groups)
against a plain float64 product, at the row counts and widths where its tiles, slabs of 32 rows, ranges
and the hand-over to the long kernel end.  Bound: one operand is rounded to bf16 (2^-9 per element,
2e-3 of the norm seen), the rest are float32 sums."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d_in,d", [(8, 4), (128, 64), (136, 68), (264, 132), (776, 392)])
@pytest.mark.parametrize("rows", [1, 31, 32, 33, 640, 641, 700, 4100, 9200, 13000])
def test_rows_and_widths(rows, d_in, d):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(rows * 7 + d)
    n = 20_000
    X = torch.randn(n, d_in, device="cuda", dtype=torch.bfloat16)
    ids = (torch.randperm(n - 1, device="cuda")[:rows] + 1).to(torch.int32)
    ids[rows // 2] = 0                                     # the padding item: its row does not count
    G = torch.randn(rows, d, device="cuda")
    # the buffer is larger than what it holds (what lies behind the rows held is never summed)
    g = gram.Gram(gram.make_config(n, d_in, d, rows + 100, 1, 0, 0, gram.BF16))
    g.window_import(ids, torch.ones(rows, dtype=torch.int64, device="cuda"), G, rows)
    Xi = X[ids.long()].double()
    Xi[ids == 0] = 0

    def close(got, want):
        scale = max(float(want.norm()), 1e-30)
        assert float((got.double() - want).norm()) <= 6e-3 * scale

    dW = torch.full((d_in, d), float("nan"), device="cuda")
    g.encoder_wgrad(X, dW)
    close(dW, Xi.T @ G.double())
    # a range of rows that starts and ends inside slabs, added to what is there
    a, b = rows // 3, max(1, rows // 2)
    part = torch.ones((d_in, d), device="cuda")
    g.encoder_wgrad_chunk(X, part, a, b, True)
    close(part - 1, Xi[a:a + b].T @ G[a:a + b].double())
    # the same with the export: the rows come out in ascending-ID order, unchanged
    dW2 = torch.full((d_in, d), float("nan"), device="cuda")
    ut = torch.empty(rows + 100, dtype=torch.int32, device="cuda")
    Gt = torch.full((rows + 100, d), float("nan"), device="cuda")
    assert g.window_end(X, dW2, ut, None, Gt, want_host_u=True) == rows
    assert torch.equal(dW, dW2)
    order = torch.argsort(ids)
    assert torch.equal(ut[:rows], ids[order]) and torch.equal(Gt[:rows], G[order]) and bool(torch.isnan(Gt[rows:]).all())
    g.close()


@pytest.mark.parametrize("n_items,d_in,d", [(5, 64, 32), (300, 768, 256), (2000, 264, 132)])
def test_listed_rows_and_identity_rows(n_items, d_in, d):
    """Content-encoder batches: rows listed by the caller, and the dense buffer's (row = ID)."""
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(d)
    n = 4000
    X = torch.randn(n, d_in, device="cuda", dtype=torch.bfloat16)
    W = torch.randn(d_in, d, device="cuda", dtype=torch.bfloat16) * d_in ** -0.5
    ids = torch.randperm(n, device="cuda")[:n_items].to(torch.int32)
    ids[0] = 0
    Ht = torch.randn(n_items, d, device="cuda")
    g = gram.Gram(gram.make_config(n, d_in, d, n, 1, 0, 0, gram.BF16, 1))
    R, dW = torch.empty(n_items, d, device="cuda"), torch.empty(d_in, d, device="cuda")
    g.pseudo_loss_grad(X, W, ids, Ht, n_items, R, dW)
    Xi = X[ids.long()].double()
    Xi[ids == 0] = 0
    want = Xi.T @ R.double()
    assert float((dW.double() - want).norm()) <= 6e-3 * float(want.norm())
    g.window_import(ids, torch.ones(n_items, dtype=torch.int64, device="cuda"), Ht, n_items)
    g.encoder_wgrad(X, dW)
    want = Xi.T @ Ht.double()
    assert float((dW.double() - want).norm()) <= 6e-3 * float(want.norm())
    g.close()

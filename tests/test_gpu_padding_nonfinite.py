"""Padding rows are exactly zero whatever the weights hold: a product of the zero row with an Inf or NaN weight is
NaN, so no kernel may leave it to the product.  One case per kernel the forward may take: the three tile shapes of
mid-sized batches, the 256-row tiles, the 64-row kernel (a width that is not a multiple of 8) and float32."""
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(20_000, 5000, 72, 520), (20_000, 10_000, 72, 520), (20_000, 16_000, 72, 520), (40_000, 40_000, 64, 520),
          (20_000, 300, 72, 12)]


@pytest.mark.parametrize("n,m,k,d", SHAPES)
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
def test_linear_encoder(n, m, k, d, dtype):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(m)
    dt = torch.bfloat16 if dtype == "bf16" else torch.float32
    X, W = torch.randn(n, k, device="cuda", dtype=dt), torch.randn(k, d, device="cuda", dtype=dt)
    W[k // 2, 1], W[0, d - 1], W[k - 1, d // 2] = float("inf"), float("nan"), -float("inf")
    ids = torch.randint(1, n, (m,), device="cuda", dtype=torch.int32)
    ids[torch.rand(m, device="cuda") < 0.2] = 0
    g = gram.Gram(gram.make_config(n, k, d, m, 1, 0, 0, gram.BF16 if dtype == "bf16" else gram.F32))
    uniq, counts = (torch.empty(m, dtype=torch.int32, device="cuda") for _ in range(2))
    inverse, u = torch.empty(m, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    E, H = torch.full((m, d), float("nan"), device="cuda"), torch.full((m, d), float("nan"), device="cuda")
    U = g.unique(ids, uniq, inverse, counts, u, want_host_u=True)
    assert int(uniq[0]) == 0
    for want_e in (E, None):
        H.fill_(float("nan"))
        g.encode_gather(X, W, uniq, inverse, u, m, want_e, H)
        assert bool((H[ids == 0] == 0).all()) and bool((E[0] == 0).all())
        finite = torch.isfinite(W.float()).all(dim=0)
        assert bool(torch.isfinite(H[ids != 0][:, finite]).all())
        assert not bool(torch.isfinite(E[1:U][:, ~finite]).any())
    g.close()


# (the hidden width decides the second contraction's kernel: a multiple of 32 takes the 256-row tiles where there
# are enough of them)
@pytest.mark.parametrize("n,m,dh,d", [(20_000, 5000, 72, 520), (20_000, 10_000, 72, 520), (20_000, 16_000, 72, 520),
                                      (40_000, 40_000, 64, 520), (20_000, 300, 72, 72)])
@pytest.mark.parametrize("h_bf16", [0, 1])
def test_two_layer_encoder(n, m, dh, d, h_bf16):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(m)
    k, bf = 64, torch.bfloat16
    X, W1 = torch.randn(n, k, device="cuda", dtype=bf), torch.randn(k, dh, device="cuda", dtype=bf)
    W2 = torch.randn(dh, d, device="cuda", dtype=bf)
    W1[3, dh - 1], W2[dh // 2, 1], W2[0, d - 1] = float("nan"), float("inf"), float("nan")
    ids = torch.randint(0, n, (m,), device="cuda", dtype=torch.int32)
    pad = int(ids.max())                       # the last row of the list
    ids[torch.rand(m, device="cuda") < 0.2] = pad
    g = gram.Gram(gram.make_config(n, k, d, m, 1, pad, 0, gram.BF16, 0, dh, gram.BF16 if h_bf16 else gram.F32))
    uniq, counts = (torch.empty(m, dtype=torch.int32, device="cuda") for _ in range(2))
    inverse, u = torch.empty(m, dtype=torch.int32, device="cuda"), torch.zeros(1, dtype=torch.int32, device="cuda")
    E, A1 = torch.full((m, d), float("nan"), device="cuda"), torch.full((m, dh), float("nan"), device="cuda", dtype=bf)
    H = torch.empty((m, d), device="cuda", dtype=bf if h_bf16 else torch.float32)
    U = g.unique(ids, uniq, inverse, counts, u, want_host_u=True)
    assert int(uniq[U - 1]) == pad
    for uq in (uniq, uniq[:U].clone()):
        H.fill_(float("nan"))
        g.mlp_encode_gather(X, W1, W2, uq, inverse, u, m, A1, E, H)
        assert bool((A1[U - 1] == 0).all()) and bool((E[U - 1] == 0).all()) and bool((H[ids == pad] == 0).all())
        assert bool(torch.isnan(E[:U - 1, d - 1]).all())
        assert bool(torch.isfinite(H[ids != pad][:, 2:d - 1]).all())
    g.close()

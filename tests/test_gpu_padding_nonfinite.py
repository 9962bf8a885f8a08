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

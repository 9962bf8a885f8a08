"""Items with many positions, whose rows the fused forward leaves to a copy kernel: widths at which a row takes part of a
block, a whole one or several passes of it, one to thousands of positions per item (32 and 33 lie on either side of the line), runs
that begin and end anywhere in a block's 64 sorted rows, both types of H.  A copy: bit for bit, in bf16 the nearest even of the float32 row."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d", [8, 12, 64, 200, 268, 1032, 2056])
@pytest.mark.parametrize("h", ["f32", "bf16", "bf16_off_8"])
def test_copies(d, h):
    import torch
    from paper_2204_04179_amd import gram
    torch.manual_seed(d)
    n, m, k = 70_000, 65_600, 32         # 257 row tiles
    sizes = [1, 32, 33, 63, 64, 65, 127, 200, 1024, 5000]
    ids = torch.randint(100, n, (m,), dtype=torch.int32, device="cuda")
    at = 0
    for j, c in enumerate(sizes * 3):
        ids[at:at + c] = j + 1
        at += c
    ids[at:at + 700] = 0
    ids = ids[torch.randperm(m, device="cuda")]
    X = torch.randn(n, k, device="cuda", dtype=torch.bfloat16)
    W = (torch.randn(k, d, device="cuda") * k ** -0.5).to(torch.bfloat16)
    dt = torch.float32 if h == "f32" else torch.bfloat16
    g = gram.Gram(gram.make_config(n, k, d, m, 1, 0, 0, gram.BF16, 0, 0, gram.F32 if h == "f32" else gram.BF16))
    uniq, counts, inverse = (torch.empty(m, dtype=torch.int32, device="cuda") for _ in range(3))
    u = torch.zeros(1, dtype=torch.int32, device="cuda")
    g.unique(ids, uniq, inverse, counts, u)
    E = torch.full((m, d), float("nan"), device="cuda")
    room = torch.full((m * d + 8,), float("nan"), device="cuda", dtype=dt)
    skip = 4 if h == "bf16_off_8" else 0
    H = room[skip:skip + m * d].view(m, d)
    g.profile_enable(["gather_heavy"], max_launches=4)
    g.encode_gather(X, W, uniq, inverse, u, m, E, H)
    torch.cuda.synchronize()
    assert {a: v[0] for a, v in g.profile_read().items()} == {"gather_heavy": 1}
    x = X[ids.long()].double()
    x[ids == 0] = 0
    want = x @ W.double()
    assert torch.equal(H, E[inverse.long()].to(dt)) and bool((H[ids == 0] == 0).all())
    assert float((H.double() - want).norm()) <= (2.0 ** -8 if dt == torch.bfloat16 else 2e-6) * float(want.norm())
    assert bool(room[:skip].isnan().all()) and bool(room[skip + m * d:].isnan().all())
    g.close()

"""The dedup's ways of doing its work (ranks by comparison in one or two launches, larger batches
otherwise) against numpy, at the batch sizes where they change over, over a window of three steps so
that items already in the buffer and new ones meet in a batch.  Whole numbers: bit-exact."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def _batch(rng, m, n, kind):
    if kind == "few":                       # a handful of items: long runs, every slice sees equal IDs
        ids = rng.choice(np.array([0, 1, n // 2, n - 1]), size=m)
    elif kind == "one":                     # one item that is not padding in every position but the last few
        ids = np.full(m, n // 2 + 1)
        ids[m - min(m, 5):] = rng.integers(0, n, size=min(m, 5))
    elif kind == "runs":                    # sorted: runs that begin anywhere in a thread's four positions
        ids = np.sort(np.minimum((rng.pareto(0.7, size=m) * 3).astype(np.int64), n - 1))
    elif kind == "distinct_first":          # ascending, then all equal
        ids = np.minimum(np.arange(m), n - 1)
    else:                                   # popular items, padding, the largest ID
        ids = np.minimum((rng.pareto(0.7, size=m) * 3).astype(np.int64), n - 1)
        ids[rng.random(m) < 0.2] = 0
        ids[::97] = n - 1
    return ids.astype(np.int32)


def check_dedup_window(m, n, kind, steps=3, m_last=None):
    import torch
    from paper_2204_04179_amd import gram
    rng = np.random.default_rng(m * 31 + n)
    d = 4
    g = gram.Gram(gram.make_config(n, 8, d, m, steps, 0, 0, gram.F32))
    cap = min(m, n)
    seen, total = [], np.zeros(n, np.int64)
    for k in range(steps):
        mk = m_last if (m_last and k == steps - 1) else m
        ids = _batch(rng, mk, n, kind)
        dev = torch.from_numpy(ids).cuda()
        uniq = torch.full((cap,), -7, dtype=torch.int32, device="cuda")
        counts = torch.full((cap,), -7, dtype=torch.int32, device="cuda")
        inverse = torch.full((mk,), -7, dtype=torch.int32, device="cuda")
        U = g.unique(dev, uniq, inverse, counts, want_host_u=True)
        ru, ri, rc = np.unique(ids, return_inverse=True, return_counts=True)
        assert U == ru.size
        np.testing.assert_array_equal(uniq.cpu().numpy()[:U], ru)
        np.testing.assert_array_equal(counts.cpu().numpy()[:U], rc)
        np.testing.assert_array_equal(inverse.cpu().numpy(), ri.reshape(-1))
        assert bool((uniq[U:] == -7).all()) and bool((counts[U:] == -7).all())
        # every gradient row is the same whole number: sums are exact and tell lost or doubled rows apart
        dH = torch.full((mk, d), float(k + 1), device="cuda")
        g.grad_accumulate(dH, mk, k)
        total += np.bincount(ids, minlength=n) * (k + 1)
        seen.append(ids)
    rows = min(steps * m, n)
    ut = torch.empty(rows, dtype=torch.int32, device="cuda")
    ct = torch.empty(rows, dtype=torch.int32, device="cuda")
    Gt = torch.empty((rows, d), device="cuda")
    T = g.flush(ut, ct, Gt, want_host_u=True)
    ru, rc = np.unique(np.concatenate(seen), return_counts=True)
    assert T == ru.size
    np.testing.assert_array_equal(ut.cpu().numpy()[:T], ru)
    np.testing.assert_array_equal(ct.cpu().numpy()[:T], rc)
    want = total[ru].astype(np.float64)
    want[ru == 0] = 0
    np.testing.assert_array_equal(Gt.cpu().numpy()[:T].astype(np.float64), np.repeat(want[:, None], d, 1))
    g.close()


@pytest.mark.parametrize("kind", ["popular", "few", "distinct_first"])
@pytest.mark.parametrize("m", [1, 3, 511, 512, 513, 1024, 1025, 8191, 8192, 8193, 12287, 12288, 12289])
def test_small_batches(m, kind):
    check_dedup_window(m, 200_001 if m > 8192 else 5001, kind)      # (large vocabulary: not counted by ID)


@pytest.mark.parametrize("m", [700, 9000])
def test_largest_ids_of_the_type(m):
    """IDs up to 2^31 - 2 through the call that needs no context (nothing is sized by the vocabulary)."""
    import torch
    from paper_2204_04179_amd import gram
    n = 2**31 - 1
    rng = np.random.default_rng(m)
    ids = rng.choice(np.array([0, 1, 2**30, n - 2, n - 1], np.int64), size=m).astype(np.int32)
    dev = torch.from_numpy(ids).cuda()
    uniq, counts, inverse = (torch.empty(m, dtype=torch.int32, device="cuda") for _ in range(3))
    u, err = (torch.zeros(1, dtype=torch.int32, device="cuda") for _ in range(2))
    gram.unique_static(dev, n, 0, uniq, inverse, counts, u, err)
    ru, ri, rc = np.unique(ids, return_inverse=True, return_counts=True)
    assert int(u) == ru.size and int(err) == 0
    np.testing.assert_array_equal(uniq.cpu().numpy()[:ru.size], ru)
    np.testing.assert_array_equal(counts.cpu().numpy()[:ru.size], rc)
    np.testing.assert_array_equal(inverse.cpu().numpy(), ri.reshape(-1))


@pytest.mark.parametrize("kind", ["popular", "few"])
@pytest.mark.parametrize("m,n", [(8450, 9001), (12289, 100), (20001, 5001), (13000, 127), (13000, 128), (13000, 129), (65535, 20000),
                                 (65535, 65536), (30000, 65537), (49152, 131072), (16384, 131071),
                                 # beyond the counting dedup: positions, vocabulary, size of its table
                                 (65536, 20000), (30000, 131073), (49153, 131072)])
def test_mid_sized_batches(m, n, kind):
    check_dedup_window(m, n, kind, m_last=m - 257)


def test_mid_sized_batch_of_one_item_and_out_of_range_ids():
    import torch
    from paper_2204_04179_amd import gram
    m, n = 65535, 3000
    g = gram.Gram(gram.make_config(n, 8, 4, m, 1, 0, 0, gram.F32))
    uniq, counts = (torch.empty(n, dtype=torch.int32, device="cuda") for _ in range(2))
    inverse = torch.empty(m, dtype=torch.int32, device="cuda")
    ids = torch.full((m,), 2999, dtype=torch.int32, device="cuda")      # a count of 65,535: the counters' largest
    assert g.unique(ids, uniq, inverse, counts, want_host_u=True) == 1
    assert int(uniq[0]) == 2999 and int(counts[0]) == m and int(inverse.abs().max()) == 0
    for bad in (n, -1, 2**31 - 1, -2**31):
        ids[m // 2] = bad
        with pytest.raises(gram.GramError) as e:
            g.unique(ids, uniq, inverse, counts, want_host_u=True)
        assert e.value.status == gram.ERR_RANGE
    g.close()


@pytest.mark.parametrize("over", ["inverse", "uniq", "counts"])
@pytest.mark.parametrize("m,n", [(300, 1000), (6000, 1000), (11_000, 200_001), (9000, 5001), (65_535, 20_000), (30_000, 131_072),
                                 (70_000, 20_000)])
def test_an_output_in_the_buffer_of_the_ids(m, n, over):
    """The IDs' own buffer as one of the outputs: one launch, ranks, the counting dedup with one and two parts of the
    vocabulary, and the sort."""
    import torch
    from paper_2204_04179_amd import gram
    rng = np.random.default_rng(m)
    ids = _batch(rng, m, n, "popular")
    ru, ri, rc = np.unique(ids, return_inverse=True, return_counts=True)
    g = gram.Gram(gram.make_config(n, 8, 4, m, 1, 0, 0, gram.F32))
    dev = torch.from_numpy(ids).cuda()
    out = {k: torch.empty(m, dtype=torch.int32, device="cuda") for k in ("uniq", "inverse", "counts")}
    out[over] = dev
    assert g.unique(dev, out["uniq"], out["inverse"], out["counts"], want_host_u=True) == ru.size
    np.testing.assert_array_equal(out["uniq"].cpu().numpy()[:ru.size], ru)
    np.testing.assert_array_equal(out["counts"].cpu().numpy()[:ru.size], rc)
    np.testing.assert_array_equal(out["inverse"].cpu().numpy()[:m], ri.reshape(-1))
    if over != "inverse":               # entries behind the items are untouched
        np.testing.assert_array_equal(dev.cpu().numpy()[ru.size:], ids[ru.size:])
    # and the batch's sums: whole numbers
    g.grad_accumulate(torch.ones(m, 4, device="cuda"), m, 0)
    Gt = torch.empty(min(m, n), 4, device="cuda")
    assert g.flush(None, None, Gt, want_host_u=True) == ru.size
    np.testing.assert_array_equal(Gt.cpu().numpy()[:ru.size, 0], np.where(ru == 0, 0, rc))
    g.close()


@pytest.mark.parametrize("m", [1, 300, 512, 513, 5000, 12_288, 12_289, 40_000])
def test_error_word_of_the_call_without_a_context(m):
    """The scratch array keeps the last call's contents: a bad ID is reported by its own call and not by the next."""
    import torch
    from paper_2204_04179_amd import gram
    n = 1000
    ids = torch.randint(0, n, (m,), dtype=torch.int32, device="cuda")
    bad = ids.clone()
    bad[m - 1] = n
    uniq, counts, inverse = (torch.empty(m, dtype=torch.int32, device="cuda") for _ in range(3))
    u, err = torch.zeros(1, dtype=torch.int32, device="cuda"), torch.full((1,), 77, dtype=torch.int32, device="cuda")
    for batch, want in ((bad, 1), (ids, 0), (bad, 1), (bad, 1), (ids, 0)):
        gram.unique_static(batch, n, 0, uniq, inverse, counts, u, err)
        assert int(err) == want
        assert torch.equal(uniq[inverse.long()], torch.where(batch >= n, 0, batch))


# The one-launch dedup: where its keys change from IDs to numbers in a bitmap (the line depends on whether the buffer may hold
# items already), the largest vocabulary of either, positions per block and per thread, the last sizes it takes and the next.
@pytest.mark.parametrize("m,n", [(513, 8), (640, 55_472), (640, 55_473), (700, 63_792), (700, 63_793), (8192, 524_288), (8193, 524_288),
                                 (8193, 524_289), (12_288, 70_000), (12_289, 55_472), (12_289, 70_000), (16_383, 20_000), (16_384, 20_000),
                                 (16_385, 20_000)])
@pytest.mark.parametrize("kind", ["popular", "few", "distinct_first"])
def test_one_launch(m, n, kind):
    check_dedup_window(m, n, kind, m_last=m - 3)


@pytest.mark.parametrize("m,n", [(700, 1000), (9001, 50_000), (2050, 300_000)])
@pytest.mark.parametrize("pad", [-1, 0, 17, "last", "absent"])
def test_one_launch_padding_and_bad_ids(m, n, pad):
    """The padding ID anywhere in the vocabulary, absent or none at all, over two steps; IDs out of range count as padding (as
    item 0 where there is none) and are reported."""
    import torch
    from paper_2204_04179_amd import gram
    rng = np.random.default_rng(m)
    pad_id = n - 1 if pad == "last" else 5 if pad == "absent" else pad
    g = gram.Gram(gram.make_config(n, 8, 4, m, 2, pad_id, 0, gram.F32))
    total = np.zeros(n, np.int64)
    for k in range(2):
        ids = _batch(rng, m, n, "popular")
        if pad == "absent":
            ids[ids == 5] = 6
        elif pad_id >= 0:
            ids[rng.random(m) < 0.4] = pad_id
        if k and pad != "absent":
            given = ids.copy()
            given[[0, m // 2, m - 1]] = [n, -1, 2**31 - 1]
            ids[[0, m // 2, m - 1]] = max(pad_id, 0)
        else:
            given = ids
        uniq, counts = (torch.full((min(m, n),), -7, dtype=torch.int32, device="cuda") for _ in range(2))
        inverse = torch.empty(m, dtype=torch.int32, device="cuda")
        g.unique(torch.from_numpy(given).cuda(), uniq, inverse, counts)
        g.grad_accumulate(torch.ones(m, 4, device="cuda"), m, k)
        ru, ri, rc = np.unique(ids, return_inverse=True, return_counts=True)
        np.testing.assert_array_equal(uniq.cpu().numpy()[:ru.size], ru)
        np.testing.assert_array_equal(counts.cpu().numpy()[:ru.size], rc)
        np.testing.assert_array_equal(inverse.cpu().numpy(), ri.reshape(-1))
        assert bool((uniq[ru.size:] == -7).all()) and bool((counts[ru.size:] == -7).all())
        total += np.bincount(ids, minlength=n)
    if pad != "absent":
        with pytest.raises(gram.GramError) as e:
            g.check()
        assert e.value.status == gram.ERR_RANGE
    rows = min(2 * m, n)
    ut, Gt = torch.empty(rows, dtype=torch.int32, device="cuda"), torch.empty(rows, 4, device="cuda")
    T = g.flush(ut, None, Gt, want_host_u=True)
    items = np.flatnonzero(total)
    np.testing.assert_array_equal(ut.cpu().numpy()[:T], items)
    want = np.where(items == pad_id, 0, total[items])
    np.testing.assert_array_equal(Gt.cpu().numpy()[:T, 0], want)
    g.close()


# A thread's four neighbouring positions are counted together where they are equal: all of them, any of them
@pytest.mark.parametrize("m,n", [(513, 8), (1001, 300_000), (8190, 20_000), (12_288, 300_000), (16_384, 20_000)])
@pytest.mark.parametrize("kind", ["one", "runs", "few"])
def test_one_launch_of_equal_neighbours(m, n, kind):
    check_dedup_window(m, n, kind, m_last=m - 2)


# Where the one-launch dedup goes from IDs to numbers in a bitmap in small batches, first step and later ones, and where later
# steps are left to the counting dedup: either side of every line, the last step on another side than those before it
@pytest.mark.parametrize("m,n,m_last", [(2048, 16_384, 1000), (2048, 16_385, 2047), (2049, 16_385, 2048), (2048, 32_769, 513), (4096, 32_768, 4095),
                                        (4097, 32_769, 4096), (8193, 40_960, 8192), (8193, 40_961, 8192), (16_384, 40_960, 16_383),
                                        (16_384, 40_961, 16_383), (16_384, 131_072, 12_288), (12_288, 131_073, 9000)])
@pytest.mark.parametrize("kind", ["popular", "one"])
def test_one_launch_lines(m, n, m_last, kind):
    check_dedup_window(m, n, kind, m_last=m_last)

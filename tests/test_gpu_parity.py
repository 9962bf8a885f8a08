"""Parity of the HIP path (through the C ABI) with the CPU oracle.

Bars: unique / inverse / counts bit-exact; float results norm-wise relative
(max-norm and Frobenius) within 1e-5 for float32 inputs and 2e-2 for bf16
inputs with float32 accumulation.  The float32 bar follows from the
arithmetic: sums of at most a few hundred float32 terms in a fixed order carry
a relative error of a few 1e-7 against the float64 oracle; bf16 results differ
from the oracle by float32 accumulation (1e-6) for E/H/G and, for dW, by the
rounding of G to bf16 (2^-9 per element, averaging down over the contraction).
"""
import numpy as np
import pytest

from oracle import gram_oracle as orc
from paper_2204_04179_amd import workloads as wl
from harness import assert_close, run_window

pytestmark = pytest.mark.gpu

TOL = {wl.F32: 1e-5, wl.BF16: 2e-2}
# E, H, G only see float32 accumulation, whatever the input dtype
TOL_SUM = {wl.F32: 1e-5, wl.BF16: 1e-4}


def say(*a):
    print(*a, flush=True)


def check_step_exact(st, ref):
    np.testing.assert_array_equal(st["uniq"], ref["uniq"])
    np.testing.assert_array_equal(st["inverse"], ref["inverse"])
    np.testing.assert_array_equal(st["counts"], ref["counts"])
    assert st["uniq_tail_untouched"]


def full_window_check(w, batches, X, W, out, tol, tol_sum):
    mm = orc.GramMulti(X, W, pad_id=0)
    for k, (ids, dH) in enumerate(batches):
        ref = mm.step(ids, dH)
        st = out["steps"][k]
        check_step_exact(st, ref)
        if ref["E"].size:
            assert_close(st["E"], ref["E"], tol_sum, f"E step {k}")
            assert_close(st["H"], ref["H"], tol_sum, f"H step {k}")
            np.testing.assert_array_equal(st["H"], st["E"][st["inverse"]])   # gather is a pure copy
        pad_rows = ids.reshape(-1) == 0
        assert np.all(st["H"][pad_rows] == 0.0)
    ref = mm.finish()
    np.testing.assert_array_equal(out["uniq_total"], ref["uniq"])
    np.testing.assert_array_equal(out["counts_total"], ref["counts"])
    e = assert_close(out["G_total"], ref["G"], tol_sum, "G_total")
    assert np.all(out["G_total"][ref["uniq"] == 0] == 0.0)
    e2 = assert_close(out["dW"], ref["dW"], tol, "dW")
    say(f"   {w.name}: U_total={ref['uniq'].size} G err={e[0]:.2e} dW err={e2[0]:.2e}")
    return ref


@pytest.mark.parametrize("name", ["tiny", "kt", "news", "kt_multi"])
def test_paper_shaped_workloads_match_oracle(name):
    w = wl.get(name)
    say(f"workload {name}: B={w.B} L={w.L} N={w.N} d_in={w.d_in} d={w.d} K={w.K} {w.xw_dtype}")
    X, W = wl.features(w), wl.weights(w)
    batches = [(wl.ids(w, k).reshape(-1), wl.upstream_grad(w, k)) for k in range(w.K)]
    out = run_window(X, W, batches, vocab_n=w.N, k_steps=w.K)
    ref = full_window_check(w, batches, X, W, out, TOL[w.xw_dtype], TOL_SUM[w.xw_dtype])
    if w.K == 1:
        # Section 4.1: the same gradient as per-interaction end-to-end training
        _, dW_e2e = orc.e2e(batches[0][0], X, W, batches[0][1])
        assert_close(out["dW"], dW_e2e, TOL[w.xw_dtype], "dW vs E2E")
        assert_close(ref["dW"], dW_e2e, 1e-12, "oracle GRAM vs oracle E2E")


_STRESS = {}


def stress_inputs():
    """(workload, X, W) of the stress configuration, drawn once per test process (2 GB, half a minute)."""
    if not _STRESS:
        w = wl.get("stress")
        _STRESS["v"] = (w, wl.features(w), wl.weights(w))
    return _STRESS["v"]


def test_stress_workload_against_oracle():
    """Full-size large configuration in the launch shape the benchmark times.  Integer outputs,
    G_total and the gather (H == E[inverse]) are compared in full; with at least 8 host cores so
    are every row of E of the first step and every entry of dW (the oracle then needs about as
    long as the benchmark's CPU baseline); with fewer cores, and for E of the later steps,
    sampled rows and entries that the oracle computes one by one."""
    import torch
    w, X, W = stress_inputs()
    full = orc.num_threads() >= 8
    say(f"workload stress: M={w.M} N={w.N} d_in={w.d_in} d={w.d} K={w.K}; oracle on {orc.num_threads()} threads: "
        f"{'FULL compare of E (step 0) and dW' if full else 'SAMPLED compare of E and dW (fewer than 8 cores)'}")
    rng = np.random.default_rng(7)
    batches = [(wl.ids(w, k).reshape(-1), wl.upstream_grad(w, k)) for k in range(w.K)]
    # the window ends as in the benchmark: weight gradient and export in one call
    out = run_window(X, W, batches, vocab_n=w.N, k_steps=w.K, keep_H=False, keep_E=False, window_end=True)
    assert out["G_tail_untouched"]
    say("   GPU window done")
    acc = orc.GramMulti(X, W, pad_id=0)
    for k, (ids, dH) in enumerate(batches):
        st = out["steps"][k]
        uniq, inverse, counts = orc.unique(ids, w.N)
        check_step_exact(st, dict(uniq=uniq, inverse=inverse, counts=counts))
        E_dev, H_dev, inv_dev = st["E_dev"], st["H_dev"], st["inverse_dev"]
        U = st["U"]
        # the gather is a pure copy, everywhere
        assert bool((H_dev[:w.M] == E_dev[inv_dev[:w.M].long()]).all().item())
        if full and k == 0:
            E_ref = orc.encode(uniq, X, W, 0)
            e = assert_close(E_dev[:U].cpu().numpy(), E_ref, TOL_SUM[wl.BF16], f"E all rows step {k}")
            what = f"E all {U} rows err={e[0]:.2e}"
            del E_ref
        else:
            rows = rng.choice(U, size=192, replace=False)
            E_ref = orc.encode(uniq[rows], X, W, 0)
            assert_close(E_dev[torch.from_numpy(rows).cuda()].cpu().numpy(), E_ref, TOL_SUM[wl.BF16], f"E sample step {k}")
            what = "E sample ok"
        G = orc.grad_accumulate(dH, inverse, uniq, 0)
        orc._check(orc.lib().oracle_buffer_add(acc._buf, orc._p(uniq, orc.C.c_int32), orc._p(counts, orc.C.c_int32),
                                               orc._p(G, orc.C.c_double), uniq.size), "buffer_add")
        say(f"   step {k}: U={U} exact, {what}")
    ids_t, counts_t, G_t = acc.export()
    np.testing.assert_array_equal(out["uniq_total"], ids_t)
    np.testing.assert_array_equal(out["counts_total"], counts_t)
    assert counts_t.sum() == w.K * w.M
    e = assert_close(out["G_total"], G_t, TOL_SUM[wl.BF16], "G_total")
    dW = out["dW"]
    if full:
        e2 = assert_close(dW, orc.wgrad(ids_t, X, G_t, 0), TOL[wl.BF16], "dW, every entry")
        say(f"   U_total={ids_t.size} G err={e[0]:.2e} dW (all {dW.size} entries) err={e2[0]:.2e}")
    else:
        rows = rng.integers(0, w.d_in, size=1500).astype(np.int32)
        cols = rng.integers(0, w.d, size=1500).astype(np.int32)
        ref = orc.wgrad_entries(ids_t, X, G_t, 0, rows, cols)
        err = np.abs(dW[rows, cols] - ref).max() / np.abs(ref).max()
        say(f"   U_total={ids_t.size} G err={e[0]:.2e} dW sampled err={err:.2e}")
        assert np.all(np.isfinite(dW)) and err <= TOL[wl.BF16]


def test_encoder_update_rows_at_the_stress_shape_sampled_against_oracle():
    """The content-encoder batch calls in the launch configuration the benchmark times (stress
    vocabulary and widths, batches of 32,768 items): outputs are compared on sampled rows and
    entries that the oracle computes one by one."""
    import torch
    from paper_2204_04179_amd import gram
    from harness import to_dev
    w, X, W = stress_inputs()
    say("stress-shaped encoder batches: inputs drawn")
    rng = np.random.default_rng(11)
    n = 32768
    items = np.sort(rng.choice(np.arange(0, w.N), size=n, replace=False)).astype(np.int32)
    items[0] = 0                                                   # the padding item is in the batch
    Xd, Wd = to_dev(X, torch), to_dev(W, torch)
    items_d = torch.from_numpy(items).cuda()
    rows_s = np.sort(rng.choice(n, size=96, replace=False))
    cols_s = np.sort(rng.choice(w.d, size=24, replace=False))
    W_sub = np.ascontiguousarray(W[:, cols_s])

    # --- linear encoder: regression towards stored targets
    Ht = rng.standard_normal((n, w.d)).astype(np.float32)
    g = gram.Gram(gram.make_config(w.N, w.d_in, w.d, w.M, w.K, 0, 0, gram.BF16))
    R = torch.full((n, w.d), float("nan"), device="cuda")
    dW = torch.full((w.d_in, w.d), float("nan"), device="cuda")
    g.pseudo_loss_grad(Xd, Wd, items_d, torch.from_numpy(Ht).cuda(), n, R, dW)
    g.check()
    miss_rows = orc.pseudo_loss_grad(items[rows_s], X, W, Ht[rows_s].astype(np.float64))[0]
    assert_close(R[torch.from_numpy(rows_s).cuda()].cpu().numpy(), miss_rows, TOL_SUM[wl.BF16], "R sample")
    miss_cols = orc.encode(items, X, W_sub, 0) - Ht[:, cols_s].astype(np.float64)   # all items, sampled columns
    miss_cols[items == 0] = 0.0
    ii = rng.integers(0, w.d_in, size=600).astype(np.int32)
    cc = rng.integers(0, cols_s.size, size=600).astype(np.int32)
    ref = orc.wgrad_entries(items, X, miss_cols, 0, ii, cc)
    got = dW.cpu().numpy()[ii, cols_s[cc]]
    err = np.abs(got - ref).max() / np.abs(ref).max()
    say(f"   linear: dW sampled err={err:.2e}")
    assert err <= TOL[wl.BF16]
    g.close()
    del R, dW

    # --- two-layer encoder: backward from gradient rows
    d_hid = 1024
    W1 = wl.f32_to_bf16_bits((rng.standard_normal((w.d_in, d_hid)) / np.sqrt(w.d_in)).astype(np.float32))
    W2 = wl.f32_to_bf16_bits((rng.standard_normal((d_hid, w.d)) / np.sqrt(d_hid)).astype(np.float32))
    G_rows = rng.standard_normal((n, w.d)).astype(np.float32)
    G_rows[0] = 0.0
    g = gram.Gram(gram.make_config(w.N, w.d_in, w.d, w.M, w.K, 0, 0, gram.BF16, 0, d_hid))
    work = torch.empty(g.mlp_batch_bytes(n), dtype=torch.uint8, device="cuda")
    dW1 = torch.full((w.d_in, d_hid), float("nan"), device="cuda")
    dW2 = torch.full((d_hid, w.d), float("nan"), device="cuda")
    g.mlp_backward(Xd, to_dev(W1, torch), to_dev(W2, torch), items_d, torch.from_numpy(G_rows).cuda(), None, n,
                   work, dW1, dW2)
    g.check()
    k = 160
    i1, q1 = rng.integers(0, w.d_in, size=k), rng.integers(0, d_hid, size=k)
    q2, c2 = rng.integers(0, d_hid, size=k), rng.integers(0, w.d, size=k)
    r1, r2 = orc.mlp_grad_entries(items, X, W1, W2, G_rows.astype(np.float64), i1, q1, q2, c2)
    e1 = np.abs(dW1.cpu().numpy()[i1, q1] - r1).max() / np.abs(r1).max()
    e2 = np.abs(dW2.cpu().numpy()[q2, c2] - r2).max() / np.abs(r2).max()
    say(f"   two-layer: dW1 sampled err={e1:.2e} dW2 sampled err={e2:.2e}")
    assert e1 <= TOL[wl.BF16] and e2 <= TOL[wl.BF16]
    assert bool(torch.isfinite(dW1).all()) and bool(torch.isfinite(dW2).all())
    g.close()


# ---------------------------------------------------------------- edge cases --

def small_problem(seed, m, n, d_in=16, d=8, bf16=False, pad_frac=0.2, ids=None):
    rng = np.random.default_rng(seed)
    if ids is None:
        ids = rng.integers(1, n, size=m).astype(np.int32)
        ids[rng.random(m) < pad_frac] = 0
    X = rng.standard_normal((n, d_in)).astype(np.float32)
    W = (rng.standard_normal((d_in, d)) / np.sqrt(d_in)).astype(np.float32)
    if bf16:
        X, W = wl.f32_to_bf16_bits(X), wl.f32_to_bf16_bits(W)
    dH = rng.standard_normal((ids.size, d)).astype(np.float32)
    return ids, X, W, dH


def check_single(ids, X, W, dH, n, tol, tol_sum, **kw):
    out = run_window(X, W, [(ids, dH)], vocab_n=n, **kw)
    ref = orc.gram_single(ids, X, W, dH, pad_id=kw.get("pad_id", 0))
    st = out["steps"][0]
    check_step_exact(st, ref)
    if ids.size:
        if "E" in st:
            assert_close(st["E"], ref["E"], tol_sum, "E")
        assert_close(st["H"], ref["H"], tol_sum, "H")
        assert_close(out["G_total"], ref["G"], tol_sum, "G")
    np.testing.assert_array_equal(out["uniq_total"], ref["uniq"])
    np.testing.assert_array_equal(out["counts_total"], ref["counts"])
    if np.abs(ref["dW"]).max() > 0:
        assert_close(out["dW"], ref["dW"], tol, "dW")
    else:
        assert np.all(out["dW"] == 0.0)
    return out, ref


# batches of up to 8192 positions take the one-launch dedup kernel, larger ones the multi-kernel sort
@pytest.mark.parametrize("m", [1, 2, 63, 64, 65, 255, 1023, 1025, 4097, 8191, 8192, 8193, 20001])
@pytest.mark.parametrize("bf16", [False, True])
def test_ragged_sizes(m, bf16):
    say(f"ragged m={m} bf16={bf16}")
    ids, X, W, dH = small_problem(m, m, 50, d_in=24, d=12, bf16=bf16)
    check_single(ids, X, W, dH, 50, TOL[wl.BF16 if bf16 else wl.F32], TOL_SUM[wl.BF16 if bf16 else wl.F32])


def test_degenerate_batches():
    n = 300
    for label, ids in (("all distinct", np.random.default_rng(0).permutation(n - 1).astype(np.int32)[:200] + 1),
                       ("all equal", np.full(777, 5, np.int32)),
                       ("all equal, multi-kernel path", np.full(9000, 5, np.int32)),
                       ("all padding", np.zeros(300, np.int32)),
                       ("all padding, multi-kernel path", np.zeros(10000, np.int32)),
                       ("empty", np.zeros(0, np.int32))):
        say("degenerate:", label)
        ids, X, W, dH = small_problem(1, ids.size, n, ids=ids)
        out, ref = check_single(ids, X, W, dH, n, 1e-5, 1e-5, max_positions=max(1024, ids.size))
        if label == "all distinct":
            # G is a row permutation of dH: bit-exact
            np.testing.assert_array_equal(out["G_total"][ref["inverse"]], dH)
        if label.startswith("all padding"):
            assert out["U_total"] == 1 and np.all(out["G_total"] == 0) and np.all(out["dW"] == 0)
        if label == "empty":
            assert out["U_total"] == 0


@pytest.mark.parametrize("m", [5000, 20000])
@pytest.mark.parametrize("vocab_bits", [1, 8, 9, 10, 11, 16, 17, 20, 21, 24])
def test_vocabulary_sizes_change_the_radix_plan(vocab_bits, m):
    n = (1 << vocab_bits) + (1 if vocab_bits in (10, 20) else 0)   # 2^b + 1 needs b+1 bits
    say(f"vocab n={n} m={m}")
    rng = np.random.default_rng(vocab_bits)
    ids = rng.integers(0, n, size=m).astype(np.int32)
    ids[::7] = n - 1
    ids[::11] = 0
    X = np.zeros((n, 8), np.float32)
    X[ids] = rng.standard_normal((m, 8)).astype(np.float32)
    W = rng.standard_normal((8, 4)).astype(np.float32)
    dH = rng.standard_normal((m, 4)).astype(np.float32)
    check_single(ids, X, W, dH, n, 1e-5, 1e-5)


def test_segment_lengths_around_tile_and_long_thresholds():
    """Runs of 1..400 equal IDs laid out so that segments start and end at every
    offset relative to the 32-row tiles and cross the 'long segment' threshold (32 rows at this
    batch size; the 64-row threshold of large batches is crossed in the fused-forward test)."""
    lengths = [1, 2, 31, 32, 33, 1, 127, 128, 129, 1, 1, 160, 63, 64, 65, 400, 3, 96, 255, 256, 257, 5, 1000, 1,
               4000, 7, 2500]      # 10,618 rows: beyond the one-launch dedup as well
    ids = np.concatenate([np.full(L, i + 1, np.int32) for i, L in enumerate(lengths)])
    rng = np.random.default_rng(3)
    ids = ids[rng.permutation(ids.size)]
    n = len(lengths) + 2
    for bf16 in (False, True):
        say(f"segments bf16={bf16} m={ids.size}")
        ids_, X, W, dH = small_problem(5, ids.size, n, d_in=16, d=260, bf16=bf16, ids=ids)
        check_single(ids_, X, W, dH, n, TOL[wl.BF16 if bf16 else wl.F32], TOL_SUM[wl.BF16 if bf16 else wl.F32], pad_id=-1)


def test_one_item_owning_hundreds_of_scan_tiles_over_a_two_step_window():
    """An item with 300,000 of 640,000 positions: its segment covers about 293 of the 1024-row tiles
    of the head scan, more than the 256 tiles the count of a segment looks ahead at a time; an
    item of 70,000 and the padding item with 90,000 positions sit beside it, the rest are items
    seen once or a few times.  Two steps with different mixes, so that rows worked out by the
    dedup are committed on top of existing ones; everything against the oracle."""
    n, d_in, d, m = 200000, 8, 4, 640000
    batches = []
    for k, (big, second, pads) in enumerate([(300000, 70000, 90000), (5, 260000, 1000)]):
        rng = np.random.default_rng(60 + k)
        rest = m - big - second - pads
        ids = np.concatenate([np.full(big, 777, np.int32), np.full(second, 150001, np.int32),
                              np.zeros(pads, np.int32), rng.integers(1, n, size=rest).astype(np.int32)])
        ids = ids[rng.permutation(m)]
        batches.append((ids, rng.standard_normal((m, d)).astype(np.float32)))
    rng = np.random.default_rng(59)
    X = rng.standard_normal((n, d_in)).astype(np.float32)
    W = (rng.standard_normal((d_in, d)) / np.sqrt(d_in)).astype(np.float32)
    say(f"one item over hundreds of scan tiles: m={m}")
    out = run_window(X, W, batches, vocab_n=n, k_steps=2, keep_H=True, keep_E=False, window_end=True)
    acc = orc.GramMulti(X, W, pad_id=0)
    for k, (ids, dH) in enumerate(batches):
        ref = acc.step(ids, dH)
        check_step_exact(out["steps"][k], ref)
        assert_close(out["steps"][k]["H"], ref["H"], 1e-5, f"H step {k}")
    ref = acc.finish()
    np.testing.assert_array_equal(out["uniq_total"], ref["uniq"])
    np.testing.assert_array_equal(out["counts_total"], ref["counts"])
    # sums of up to 300,000 float32 terms in tile order against float64
    assert_close(out["G_total"], ref["G"], 1e-4, "G_total")
    assert_close(out["dW"], ref["dW"], 1e-4, "dW")


@pytest.mark.parametrize("m", [1_500_000, 5_000_000])
def test_batch_of_more_than_a_million_positions(m):
    """1,500,000 positions: a wave of the radix passes owns more keys than it fetches ahead at once
    (several batches of 16 rounds per wave), the head scan has 1,465 tiles; 5,000,000: the keys per
    wave reach their cap and the passes run more blocks than there are compute units.  Two steps
    with Zipf-like repeats and padding; everything against the oracle."""
    n, d_in, d = 300000, 8, 4
    rng = np.random.default_rng(93)
    X = rng.standard_normal((n, d_in)).astype(np.float32)
    W = (rng.standard_normal((d_in, d)) / np.sqrt(d_in)).astype(np.float32)
    p = np.arange(1, n, dtype=np.float64) ** -1.05
    p /= p.sum()
    batches = []
    for k in range(2):
        ids = (rng.permutation(n - 1)[rng.choice(n - 1, size=m, p=p)] + 1).astype(np.int32)
        ids[rng.random(m) < 0.1] = 0
        batches.append((ids, rng.standard_normal((m, d)).astype(np.float32)))
    say(f"more than a million positions: m={m}")
    out = run_window(X, W, batches, vocab_n=n, k_steps=2, keep_E=False, window_end=True)
    acc = orc.GramMulti(X, W, pad_id=0)
    for k, (ids, dH) in enumerate(batches):
        ref = acc.step(ids, dH)
        check_step_exact(out["steps"][k], ref)
        assert_close(out["steps"][k]["H"], ref["H"], 1e-5, f"H step {k}")
    ref = acc.finish()
    np.testing.assert_array_equal(out["uniq_total"], ref["uniq"])
    np.testing.assert_array_equal(out["counts_total"], ref["counts"])
    # the most popular item sums 160,000 to 500,000 float32 terms per step in tile order against float64
    assert_close(out["G_total"], ref["G"], 1e-4, "G_total")
    assert_close(out["dW"], ref["dW"], 1e-4, "dW")


@pytest.mark.parametrize("d,variant", [(256, "E requested"), (256, "E = NULL"), (320, "E = NULL"),
                                       (260, "E = NULL"), (256, "foreign uniq/inverse"),
                                       (64, "E = NULL, two padding positions")])
def test_fused_forward_stores_representations_to_positions(d, variant):
    """Batches with tiles for every CU take the forward whose contraction epilogue stores each
    representation to the positions of its item, and a copy kernel for items with more than
    gram_light_max() positions.  Item multiplicities sit on both sides of that limit; the padding
    ID is the heaviest item (zero rows); d = 320 leaves a ragged last column tile; d = 260 is not a
    multiple of 8, so the contraction takes the transposed copy of the weights instead of reading
    them as they are."""
    from paper_2204_04179_amd import gram
    T = gram.load().gram_light_max()
    n, m = 70000, 70000
    rng = np.random.default_rng(11)
    runs = [(1, 1), (2, T - 1), (3, T), (4, T + 1), (5, 2 * T), (6, 2 * T + 1), (7, 5000), (n - 1, T + 7), (n - 2, 3)]
    fixed = np.concatenate([np.full(c, i, np.int32) for i, c in runs])
    rest = rng.integers(8, n - 2, size=m - fixed.size).astype(np.int32)
    if "two padding" in variant:
        rest[:2] = 0                          # the padding item is a light one here
    else:
        rest[rng.random(rest.size) < 0.1] = 0
    ids = np.concatenate([fixed, rest])
    ids = ids[rng.permutation(m)]
    say(f"fused forward d={d} {variant}: m={m}")
    ids, X, W, dH = small_problem(12, m, n, d_in=64, d=d, bf16=True, ids=ids)
    out, ref = check_single(ids, X, W, dH, n, TOL[wl.BF16], TOL_SUM[wl.BF16], pass_E="E = NULL" not in variant,
                            foreign_buffers=variant.startswith("foreign"),
                            profile=["gather_heavy", "gather_rows"])
    cnt = ref["counts"]
    assert (cnt > T).sum() >= 5 and (cnt == T).any() and (cnt == T + 1).any()
    # equal IDs get bit-identical rows whichever kernel wrote them
    H = out["steps"][0]["H"]
    first = np.full(ref["uniq"].size, -1)
    first[ref["inverse"][::-1]] = np.arange(m)[::-1]
    assert H.tobytes() == H[first[ref["inverse"]]].tobytes()
    launches = {k: v[0] for k, v in out["profile"].items()}
    say("   launches:", launches)
    assert launches == ({"gather_rows": 1} if variant.startswith("foreign") else {"gather_heavy": 1})


def test_fused_forward_reads_the_dedup_kept_in_the_context():
    """The fused forward is chosen when the caller hands back the buffers gram_unique wrote.  It
    takes both the unique list and the sort order from the context, so a caller that has
    overwritten those buffers in between still gets the rows of the batch it deduplicated:
    representations and positions can never come from two different sources."""
    import torch
    from paper_2204_04179_amd import gram
    n, m, d_in, d = 70000, 70000, 64, 256
    rng = np.random.default_rng(31)
    ids = rng.integers(1, n, size=m).astype(np.int32)
    ids[rng.random(m) < 0.05] = 0
    ids, X, W, dH = small_problem(13, m, n, d_in=d_in, d=d, bf16=True, ids=ids)
    ref = orc.gram_single(ids, X, W, dH, pad_id=0)
    from harness import to_dev
    g = gram.Gram(gram.make_config(n, d_in, d, m, 1, 0, 0, gram.BF16))
    i32 = dict(dtype=torch.int32, device="cuda")
    uniq, counts, inverse = torch.zeros(n, **i32), torch.zeros(n, **i32), torch.zeros(m, **i32)
    u_dev = torch.zeros(1, **i32)
    H = torch.full((m, d), float("nan"), device="cuda")
    g.unique(torch.from_numpy(ids).cuda(), uniq, inverse, counts, u_dev)
    torch.cuda.synchronize()
    uniq.fill_(1)                 # the caller scribbles over its copies of the dedup outputs
    inverse.zero_()
    u_dev.fill_(3)
    g.profile_enable(["gather_heavy", "gather_rows"], max_launches=16)
    g.encode_gather(to_dev(X, torch), to_dev(W, torch), uniq, inverse, u_dev, m, None, H)
    torch.cuda.synchronize()
    assert {k: v[0] for k, v in g.profile_read().items()} == {"gather_heavy": 1}
    assert_close(H.cpu().numpy(), ref["H"], TOL_SUM[wl.BF16], "H after the caller's buffers changed")
    g.close()


def test_feature_matrix_beyond_4_gib_takes_the_wide_address_kernels():
    """X of 4.3 GB cannot be addressed through a 32-bit buffer descriptor.  X is drawn on the
    device; the oracle sees only the rows a batch names, under IDs renumbered in ascending order
    (which leaves uniq order, inverse, H, G and dW unchanged).
    Batch 1 (6,000 positions): few tiles, so the forward is the 64x64 kernel (plain 64-bit
    addresses) followed by the gather; the weight gradient takes its wide-address variant.
    Batch 2 (76,000 positions, about 66,000 unique items): a tile for every compute unit, so the
    forward is the wide-address variant of the 256x256 contraction with the gather fused into its
    epilogue, once with E requested and once without."""
    import torch
    n, d_in, d = 2_100_000, 1024, 256
    say(f"wide addresses: X = {n * d_in * 2 / 2**30:.2f} GiB")
    g = torch.Generator(device="cuda").manual_seed(5)
    X_dev = torch.empty(n, d_in, dtype=torch.bfloat16, device="cuda")
    X_dev.normal_(generator=g)
    rng = np.random.default_rng(21)
    W = wl.f32_to_bf16_bits((rng.standard_normal((d_in, d)) / np.sqrt(d_in)).astype(np.float32))

    def run(ids, dH, pass_E, names):
        out = run_window(np.zeros((1, 1), np.uint16), W, [(ids, dH)], vocab_n=n, X_dev=X_dev, W_dev=None,
                         pass_E=pass_E, profile=names)
        uniq = np.unique(ids)
        rows = X_dev[torch.from_numpy(uniq.astype(np.int64)).cuda()].view(torch.int16).cpu().numpy().view(np.uint16)
        small_ids = np.searchsorted(uniq, ids).astype(np.int32)       # 0 stays 0: the padding ID is the smallest
        assert uniq[0] == 0
        ref = orc.gram_single(small_ids, rows, W, dH, pad_id=0)
        st = out["steps"][0]
        np.testing.assert_array_equal(st["uniq"], uniq)
        np.testing.assert_array_equal(st["inverse"], ref["inverse"])
        np.testing.assert_array_equal(st["counts"], ref["counts"])
        if pass_E:
            assert_close(st["E"], ref["E"], TOL_SUM[wl.BF16], "E")
        assert_close(st["H"], ref["H"], TOL_SUM[wl.BF16], "H")
        assert np.all(st["H"][ids == 0] == 0.0)
        assert_close(out["G_total"], ref["G"], TOL_SUM[wl.BF16], "G")
        assert_close(out["dW"], ref["dW"], TOL[wl.BF16], "dW")
        launches = {k: v[0] for k, v in out["profile"].items()}
        say("   launches:", launches)
        out["gram"].close()
        return launches

    names = ["encode_bf16", "encode_bf16_wide", "gather_rows", "gather_heavy", "wgrad_bf16", "wgrad_bf16_wide"]
    m = 6000
    ids = rng.integers(1, n, size=m).astype(np.int32)
    ids[: m // 3] = rng.choice(ids[m // 3:], size=m // 3)         # repeats
    ids[rng.random(m) < 0.1] = 0
    ids[-1] = n - 1                                                # the last row of X
    say(f"   batch 1: m={m}")
    launches = run(ids, rng.standard_normal((m, d)).astype(np.float32), True, names)
    assert launches == {"encode_bf16": 1, "gather_rows": 1, "wgrad_bf16_wide": 1}

    from paper_2204_04179_amd import gram
    T = gram.load().gram_light_max()
    m = 76_000
    distinct = rng.choice(np.arange(1, n - 1), size=66_000, replace=False).astype(np.int32)
    repeats = np.concatenate([np.full(c, i, np.int32) for i, c in
                              ((distinct[0], 3000), (distinct[1], T), (distinct[2], T + 1), (distinct[3], 2 * T + 5),
                               (n - 1, 7))])
    rest = rng.choice(distinct, size=m - distinct.size - repeats.size - 800)
    ids = np.concatenate([distinct, repeats, rest, np.zeros(800, np.int32)]).astype(np.int32)
    ids = ids[rng.permutation(ids.size)]
    assert ids.size == m and np.unique(ids).size >= 65_537        # 256 row tiles of 256 at d = 256: one per compute unit
    dH = rng.standard_normal((m, d)).astype(np.float32)
    for pass_E in (True, False):
        say(f"   batch 2: m={m} unique={np.unique(ids).size} E requested={pass_E}")
        launches = run(ids, dH, pass_E, names)
        assert launches == {"encode_bf16_wide": 1, "gather_heavy": 1, "wgrad_bf16_wide": 1}
    del X_dev
    torch.cuda.empty_cache()


def test_no_padding_id_and_other_padding_id():
    ids, X, W, dH = small_problem(9, 500, 40, pad_frac=0.3)
    for pad in (-1, 0, 7):
        say(f"pad_id={pad}")
        check_single(ids, X, W, dH, 40, 1e-5, 1e-5, pad_id=pad)


def test_multi_step_window_and_bitwise_reproducibility():
    K, n = 4, 3000
    probs = [small_problem(100 + k, 6000, n, d_in=64, d=48, bf16=True) for k in range(K)]
    X, W = probs[0][1], probs[0][2]
    batches = [(p[0], p[3]) for p in probs]
    say("multi-step K=4")
    out1 = run_window(X, W, batches, vocab_n=n, k_steps=K)
    w = wl.Workload("adhoc", 1, 6000, n, 1.0, 64, 48, wl.BF16, K, None)
    full_window_check(w, batches, X, W, out1, TOL[wl.BF16], TOL_SUM[wl.BF16])
    # same context, next window, same data: bit-identical (no float atomics, fixed orders)
    out2 = run_window(X, W, batches, vocab_n=n, k_steps=K, gram_obj=out1["gram"])
    assert out1["G_total"].tobytes() == out2["G_total"].tobytes()
    assert out1["dW"].tobytes() == out2["dW"].tobytes()
    for a, b in zip(out1["steps"], out2["steps"]):
        assert a["H"].tobytes() == b["H"].tobytes()
    # a window of one step is Single-step GRAM (Section 4.3)
    out3 = run_window(X, W, batches[:1], vocab_n=n, k_steps=1)
    ref = orc.gram_single(batches[0][0], X, W, batches[0][1])
    assert_close(out3["G_total"], ref["G"], TOL_SUM[wl.BF16], "G K=1")
    assert_close(out3["dW"], ref["dW"], TOL[wl.BF16], "dW K=1")


def test_pseudo_targets_and_pseudo_loss_over_a_window():
    """Algorithm 1 step 3 (Eq. 6) with the gradient accumulated over the window (Section 4.2), the
    pseudo-loss of Eq. 7, and the gather of pseudo-targets to positions."""
    K, n = 3, 2500
    for bf16, d in ((False, 12), (True, 64)):
        probs = [small_problem(200 + k, 7000 + 500 * k, n, d_in=32, d=d, bf16=bf16) for k in range(K)]
        X, W = probs[0][1], probs[0][2]
        batches = [(p[0], p[3]) for p in probs]
        say(f"pseudo-targets K={K} bf16={bf16}")
        out = run_window(X, W, batches, vocab_n=n, k_steps=K, max_positions=8000, pseudo=True)
        mm = orc.GramMulti(X, W)
        tol = TOL_SUM[wl.BF16 if bf16 else wl.F32]
        for k, (ids, dH) in enumerate(batches):
            ref = mm.step(ids, dH)
            Ht_ref, loss_ref = orc.pseudo_target(ref["E"], mm.rows(ref["uniq"]))
            st = out["steps"][k]
            assert_close(st["Ht"], Ht_ref, tol, f"Ht step {k}")
            assert abs(st["loss"] - loss_ref) <= tol * loss_ref
            assert st["Ht_tail_untouched"]
            np.testing.assert_array_equal(st["H_tilde"], st["Ht"][ref["inverse"]])     # a pure row copy
            pad = ref["uniq"] == 0
            assert pad.any() and np.all(st["Ht"][pad] == 0.0)
        # one-step window: the pseudo-target of an item met once is h - dL/dh of that position
        one = run_window(X, W, batches[:1], vocab_n=n, k_steps=1, pseudo=True)["steps"][0]
        ref = orc.gram_single(batches[0][0], X, W, batches[0][1])
        once = np.flatnonzero((ref["counts"] == 1) & (ref["uniq"] != 0))
        first = np.full(ref["uniq"].size, -1)
        first[ref["inverse"][::-1]] = np.arange(batches[0][0].size)[::-1]
        np.testing.assert_array_equal(one["Ht"][once], (one["E"][once] - batches[0][1][first[once]]).astype(np.float32))


def test_pseudo_targets_after_the_fused_forward():
    """Large batch: E comes from the contraction that also stored H to the positions."""
    n, m = 70000, 70000
    rng = np.random.default_rng(31)
    ids = rng.integers(1, 3000, size=m).astype(np.int32)         # every item many times ...
    ids[: m // 2] = rng.integers(1, n, size=m // 2)              # ... or about once
    ids[rng.random(m) < 0.05] = 0
    ids, X, W, dH = small_problem(32, m, n, d_in=64, d=256, bf16=True, ids=ids)
    say("pseudo-targets after the fused forward")
    out = run_window(X, W, [(ids, dH)], vocab_n=n, pseudo=True, profile=["gather_heavy", "pseudo_target", "pseudo_loss"])
    assert {k: v[0] for k, v in out["profile"].items()} == {"gather_heavy": 1, "pseudo_target": 1, "pseudo_loss": 1}
    ref = orc.gram_single(ids, X, W, dH)
    Ht_ref, loss_ref = orc.pseudo_target(ref["E"], ref["G"])
    st = out["steps"][0]
    assert_close(st["Ht"], Ht_ref, TOL_SUM[wl.BF16], "Ht")
    assert abs(st["loss"] - loss_ref) <= TOL_SUM[wl.BF16] * loss_ref
    np.testing.assert_array_equal(st["H_tilde"], st["Ht"][ref["inverse"]])


@pytest.mark.parametrize("bf16", [False, True])
def test_weight_gradient_in_chunks_of_items(bf16):
    """The encoder update walked in batches of items (content-encoder batch size): each chunk of
    buffer rows gives the weight gradient of exactly those items, and the chunks add up to the
    whole.  Buffer order = order of first appearance: ascending ID within a step, step by step."""
    K, n, d_in, d = 3, 1200, 64, 40
    probs = [small_problem(400 + k, 2500, n, d_in=d_in, d=d, bf16=bf16) for k in range(K)]
    X, W = probs[0][1], probs[0][2]
    batches = [(p[0], p[3]) for p in probs]
    chunks = [(0, 100), (100, 37), (137, 500), (637, 1), (638, 100000), (5000, 10)]   # ragged, unaligned, past the end, empty
    say(f"chunked wgrad bf16={bf16}")
    out = run_window(X, W, batches, vocab_n=n, k_steps=K, wgrad_chunks=chunks)
    mm = orc.GramMulti(X, W)
    order, seen = [], set()
    for ids, dH in batches:
        st = mm.step(ids, dH)
        for i in st["uniq"]:
            if int(i) not in seen:
                seen.add(int(i))
                order.append(int(i))
    order = np.array(order, np.int32)
    assert order.size == out["U_total"]
    tol = TOL[wl.BF16 if bf16 else wl.F32]
    full = mm.finish()["dW"]
    scale = np.abs(full).max()
    for (a, nrows), got in zip(chunks, out["dW_chunks"]):
        items = order[a:a + nrows]
        ref = orc.wgrad(items, X, mm_rows(batches, X, W, items), 0) if items.size else np.zeros_like(full)
        assert np.abs(got - ref).max() <= tol * scale, (a, nrows)
    assert_close(out["dW_chunked"], full, tol, "sum of chunks")
    assert_close(out["dW"], full, tol, "dW")


def mm_rows(batches, X, W, items):
    """Gradient rows of `items` at the end of the window, from a fresh oracle run."""
    mm = orc.GramMulti(X, W)
    for ids, dH in batches:
        mm.step(ids, dH)
    return mm.rows(items)


def encoder_batches(X, W_now, items, Ht, splits, vocab_n, max_positions):
    """gram_pseudo_loss_grad over consecutive batches of `items` (sizes in `splits`), the gradient
    accumulated across them.  Returns (R rows, per-batch losses, dW)."""
    import torch
    from paper_2204_04179_amd import gram
    from harness import to_dev
    d_in, d = W_now.shape
    xw = gram.F32 if X.dtype == np.float32 else gram.BF16
    g = gram.Gram(gram.make_config(vocab_n, d_in, d, max_positions, 1, 0, 0, xw))
    Xd, Wd = to_dev(X, torch), to_dev(W_now, torch)
    items_d = torch.from_numpy(items).cuda()
    Ht_d = torch.from_numpy(Ht.astype(np.float32)).cuda()
    R = torch.full((max(1, items.size) + 1, d), float("nan"), device="cuda")
    dW = torch.full((d_in, d), float("nan"), device="cuda")
    losses, a = [], 0
    for i, n in enumerate(splits):
        loss = torch.full((1,), float("nan"), dtype=torch.float64, device="cuda")
        g.pseudo_loss_grad(Xd, Wd, items_d[a:a + n], Ht_d[a:a + n], n, R[a:a + n], dW, accumulate=i > 0,
                           loss_dev=loss)
        losses.append(float(loss.item()))
        a += n
    g.check()
    assert bool(torch.isnan(R[a:]).all())                       # rows past the batches are untouched
    out = R[:a].cpu().numpy(), losses, dW.cpu().numpy()
    g.close()
    return out


@pytest.mark.parametrize("bf16", [False, True])
def test_encoder_update_in_batches_against_stored_pseudo_targets(bf16):
    """Algorithm 1 step 4 one content-encoder batch at a time (Eq. 7): regression miss, pseudo-loss
    and gradient at weights that differ from those the targets came from; ragged batch sizes, a
    batch of one, an empty batch, the padding item inside a batch."""
    n, d_in, d = 3000, 64, 40
    rng = np.random.default_rng(77)
    _, X, W_now, _ = small_problem(500, 10, n, d_in=d_in, d=d, bf16=bf16)
    items = np.sort(rng.choice(np.arange(1, n), size=1500, replace=False)).astype(np.int32)
    items[700] = 0                                              # the padding item, mid-batch
    Ht = rng.standard_normal((items.size, d)).astype(np.float32)
    splits = [100, 37, 1, 0, 1000, 362]
    say(f"encoder batches bf16={bf16}")
    R, losses, dW = encoder_batches(X, W_now, items, Ht, splits, n, 4000)
    miss_ref, loss_ref, dW_ref = orc.pseudo_loss_grad(items, X, W_now, Ht.astype(np.float64))
    dt = wl.BF16 if bf16 else wl.F32
    assert_close(R, miss_ref, TOL_SUM[dt], "R")
    assert np.all(R[700] == 0.0)
    a = 0
    for n_b, got in zip(splits, losses):
        ref = orc.pseudo_loss_grad(items[a:a + n_b], X, W_now, Ht[a:a + n_b].astype(np.float64))[1]
        assert abs(got - ref) <= TOL_SUM[dt] * max(ref, 1e-300), (a, n_b)
        a += n_b
    assert abs(sum(losses) - loss_ref) <= TOL_SUM[dt] * loss_ref
    assert_close(dW, dW_ref, TOL[dt], "dW")


def test_encoder_update_batch_with_tiles_for_every_compute_unit():
    """A batch large enough for the 256x256 contraction kernels on both sides."""
    n, d_in, d = 80000, 64, 256
    rng = np.random.default_rng(78)
    _, X, W_now, _ = small_problem(501, 10, n, d_in=d_in, d=d, bf16=True)
    items = np.sort(rng.choice(np.arange(0, n), size=70001, replace=False)).astype(np.int32)
    Ht = rng.standard_normal((items.size, d)).astype(np.float32)
    say("encoder batch, large")
    R, losses, dW = encoder_batches(X, W_now, items, Ht, [items.size], n, 80000)
    miss_ref, loss_ref, dW_ref = orc.pseudo_loss_grad(items, X, W_now, Ht.astype(np.float64))
    assert_close(R, miss_ref, TOL_SUM[wl.BF16], "R")
    assert abs(losses[0] - loss_ref) <= TOL_SUM[wl.BF16] * loss_ref
    assert_close(dW, dW_ref, TOL[wl.BF16], "dW")


@pytest.mark.parametrize("bf16", [False, True])
def test_encoder_update_with_fresh_targets_gives_the_window_gradient(bf16):
    """Proposition (Eq. 1-3) through the library: the pseudo-targets gram_pseudo_target wrote,
    regressed at the same weights, give the weight gradient gram_encoder_wgrad took from the
    buffer, and the end-to-end gradient of the oracle."""
    import torch
    from paper_2204_04179_amd import gram
    from harness import to_dev
    n, d_in, d = 2500, 32, 64
    ids, X, W, dH = small_problem(502, 7000, n, d_in=d_in, d=d, bf16=bf16)
    say(f"proposition through the library bf16={bf16}")
    out = run_window(X, W, [(ids, dH)], vocab_n=n, pseudo=True)
    st = out["steps"][0]
    R, losses, dW = encoder_batches(X, W, st["uniq"], st["Ht"], [500, st["uniq"].size - 500], n, 8000)
    dt = wl.BF16 if bf16 else wl.F32
    _, dW_e2e = orc.e2e(ids, X, W, dH)
    assert_close(dW, dW_e2e, TOL[dt], "dW vs end-to-end")
    assert_close(dW, out["dW"], TOL[dt], "dW vs gram_encoder_wgrad")
    assert abs(sum(losses) - st["loss"]) <= 1e-4 * st["loss"]
    assert_close(R, out["G_total"], 1e-4, "miss vs accumulated gradient")


def test_encoder_update_argument_errors():
    import torch
    from paper_2204_04179_amd import gram
    n, d_in, d = 100, 16, 8
    g = gram.Gram(gram.make_config(n, d_in, d, 50, 1, 0, 100, gram.F32))     # 100 buffer rows
    X = torch.zeros(n, d_in, device="cuda")
    W = torch.zeros(d_in, d, device="cuda")
    ids = torch.arange(0, 100, dtype=torch.int32, device="cuda")
    Ht = torch.zeros(100, d, device="cuda")
    R = torch.zeros(100, d, device="cuda")
    dW = torch.ones(d_in, d, device="cuda")

    def status(fn):
        with pytest.raises(gram.GramError) as e:
            fn()
        return e.value.status

    assert status(lambda: g.pseudo_loss_grad(X, W, ids, Ht, 101, R, dW)) == gram.ERR_ARG      # beyond max(50, 100) rows
    assert status(lambda: g.pseudo_loss_grad(X, W, ids, Ht, -1, R, dW)) == gram.ERR_ARG
    assert status(lambda: g.pseudo_loss_grad(X, W, None, Ht, 5, R, dW)) == gram.ERR_ARG
    g.pseudo_loss_grad(X, W, None, None, 0, None, dW)            # an empty batch overwrites dW with zeros
    g.check()
    assert not bool(dW.any())
    ids[3] = 100                                                 # outside [0, N): latched, no bad access
    g.pseudo_loss_grad(X, W, ids, Ht, 100, R, dW)
    assert status(lambda: g.check()) == gram.ERR_RANGE
    g.close()


def test_long_window_reaches_the_whole_vocabulary():
    """Epoch-scale accumulation (Section 4.2 with a long period): 40 steps over a vocabulary of 1,500,
    so the buffer ends up holding every item; counts and rows are sums over all steps."""
    K, n, m = 40, 1500, 2500
    rng = np.random.default_rng(77)
    X = rng.standard_normal((n, 16)).astype(np.float32)
    W = (rng.standard_normal((16, 12)) / 4).astype(np.float32)
    batches = []
    for k in range(K):
        ids = rng.integers(0, n, size=m).astype(np.int32)
        batches.append((ids, rng.standard_normal((m, 12)).astype(np.float32)))
    say(f"long window K={K}")
    out = run_window(X, W, batches, vocab_n=n, k_steps=K, keep_H=False, keep_E=False)
    mm = orc.GramMulti(X, W)
    for ids, dH in batches:
        mm.step(ids, dH)
    ref = mm.finish()
    assert out["U_total"] == n                      # every item (and the padding ID) was met
    np.testing.assert_array_equal(out["uniq_total"], ref["uniq"])
    np.testing.assert_array_equal(out["counts_total"], ref["counts"])
    assert out["counts_total"].sum() == K * m
    assert_close(out["G_total"], ref["G"], 1e-5, "G_total")
    assert_close(out["dW"], ref["dW"], 1e-5, "dW")


# ------------------------------------------------------- two-layer stand-in encoder --

def mlp_weights(seed, n, d_in, d_hid, d):
    rng = np.random.default_rng(seed)
    X = wl.f32_to_bf16_bits(rng.standard_normal((n, d_in)).astype(np.float32))
    W1 = wl.f32_to_bf16_bits((rng.standard_normal((d_in, d_hid)) / np.sqrt(d_in)).astype(np.float32))
    W2 = wl.f32_to_bf16_bits((rng.standard_normal((d_hid, d)) / np.sqrt(d_hid)).astype(np.float32))
    return X, W1, W2


def run_mlp_step(X, W1, W2, ids, dH, vocab_n, batches_of, targets=None, W_now=None):
    """One single-step window with the two-layer encoder through the library: forward, accumulate,
    flush, then the backward pass over the window's items in batches of the given sizes (from the
    accumulated gradient rows, or from `targets` [U, d] at the weights W_now)."""
    import torch
    from paper_2204_04179_amd import gram
    from harness import to_dev
    (d_in, d_hid), d = W1.shape, W2.shape[1]
    m = ids.size
    g = gram.Gram(gram.make_config(vocab_n, d_in, d, m, 1, 0, 0, gram.BF16, 0, d_hid))
    Xd, W1d, W2d = to_dev(X, torch), to_dev(W1, torch), to_dev(W2, torch)
    cap_u = min(m, vocab_n)
    i32 = dict(dtype=torch.int32, device="cuda")
    uniq, counts, inverse = torch.full((cap_u,), -7, **i32), torch.empty(cap_u, **i32), torch.empty(m, **i32)
    u_dev = torch.zeros(1, **i32)
    A1 = torch.full((cap_u, d_hid), float("nan"), dtype=torch.bfloat16, device="cuda")
    E = torch.full((cap_u, d), float("nan"), device="cuda")
    H = torch.full((m, d), float("nan"), device="cuda")
    U = g.unique(torch.from_numpy(ids).cuda(), uniq, inverse, counts, u_dev, want_host_u=True)
    g.mlp_encode_gather(Xd, W1d, W2d, uniq, inverse, u_dev, m, A1, E, H)
    g.grad_accumulate(torch.from_numpy(dH).cuda(), m, 0)
    ut, ct = torch.empty(cap_u, **i32), torch.empty(cap_u, **i32)
    Gt = torch.empty(cap_u, d, device="cuda")
    assert g.flush(ut, ct, Gt, None, want_host_u=True) == U
    if W_now is not None:
        W1d, W2d = to_dev(W_now[0], torch), to_dev(W_now[1], torch)
    Ht = torch.from_numpy(targets.astype(np.float32)).cuda() if targets is not None else None
    dW1 = torch.full((d_in, d_hid), float("nan"), device="cuda")
    dW2 = torch.full((d_hid, d), float("nan"), device="cuda")
    work = torch.empty(max(1, g.mlp_batch_bytes(max(batches_of))), dtype=torch.uint8, device="cuda")
    losses, a = [], 0
    for i, n in enumerate(batches_of):
        loss = torch.full((1,), float("nan"), dtype=torch.float64, device="cuda")
        g.mlp_backward(Xd, W1d, W2d, ut[a:a + n], None if Ht is not None else Gt[a:a + n],
                       Ht[a:a + n] if Ht is not None else None, n, work, dW1, dW2, accumulate=i > 0,
                       loss_dev=loss)
        losses.append(float(loss.item()))
        a += n
    g.check()
    assert a == U
    out = dict(U=U, uniq=uniq[:U].cpu().numpy(), inverse=inverse.cpu().numpy(),
               A1=A1[:U].float().cpu().numpy(), A1_tail_untouched=bool(torch.isnan(A1[U:].float()).all()),
               E=E[:U].cpu().numpy(), H=H.cpu().numpy(), G=Gt[:U].cpu().numpy(), dW1=dW1.cpu().numpy(),
               dW2=dW2.cpu().numpy(), losses=losses)
    g.close()
    return out


def test_mlp_encoder_step_matches_oracle_and_end_to_end():
    """Forward with kept activations, accumulate, and the backward pass in ragged batches of items:
    against the oracle's per-unique-item run and its per-interaction (end-to-end) gradients."""
    n, d_in, d_hid, d = 2500, 32, 48, 24
    X, W1, W2 = mlp_weights(800, n, d_in, d_hid, d)
    ids, _, _, dH = small_problem(801, 7000, n, d_in=8, d=d)
    say("two-layer encoder, small")
    ref = orc.mlp_gram_single(ids, X, W1, W2, dH)
    U = ref["uniq"].size
    out = run_mlp_step(X, W1, W2, ids, dH, n, [500, 1, 0, U - 501])
    np.testing.assert_array_equal(out["uniq"], ref["uniq"])
    np.testing.assert_array_equal(out["inverse"], ref["inverse"])
    assert out["A1_tail_untouched"]
    assert_close(out["A1"], ref["A1"], 2.0 ** -8, "A1 (kept in bf16)")
    assert_close(out["E"], ref["E"], TOL[wl.BF16], "E")
    np.testing.assert_array_equal(out["H"], out["E"][out["inverse"]])
    pad = ref["uniq"] == 0
    assert pad.any() and not out["A1"][pad].any() and not out["E"][pad].any()
    assert_close(out["G"], ref["G"], TOL_SUM[wl.BF16], "G")
    _, dW1_e2e, dW2_e2e = orc.mlp_e2e(ids, X, W1, W2, dH)
    assert_close(out["dW1"], dW1_e2e, TOL[wl.BF16], "dW1 vs end-to-end")
    assert_close(out["dW2"], dW2_e2e, TOL[wl.BF16], "dW2 vs end-to-end")


def test_mlp_encoder_step_with_tiles_for_every_compute_unit():
    """Sizes at which both contractions of the forward (the second with the fused gather) and all
    three of the backward run in the 256x256 kernels."""
    n, d_in, d_hid, d = 90000, 32, 256, 128
    X, W1, W2 = mlp_weights(802, n, d_in, d_hid, d)
    rng = np.random.default_rng(803)
    m = 72000
    ids = rng.permutation(np.arange(1, n))[:m].astype(np.int32)      # nearly all distinct ...
    ids[:3000] = rng.integers(1, 50, size=3000)                      # ... a few heavy items ...
    ids[rng.random(m) < 0.02] = 0                                    # ... and padding
    dH = rng.standard_normal((m, d)).astype(np.float32)
    say("two-layer encoder, large")
    ref = orc.mlp_gram_single(ids, X, W1, W2, dH)
    U = ref["uniq"].size
    assert U > 65536
    out = run_mlp_step(X, W1, W2, ids, dH, n, [U])
    assert out["A1_tail_untouched"]
    assert_close(out["E"], ref["E"], TOL[wl.BF16], "E")
    np.testing.assert_array_equal(out["H"], out["E"][out["inverse"]])
    assert_close(out["dW1"], ref["dW1"], TOL[wl.BF16], "dW1")
    assert_close(out["dW2"], ref["dW2"], TOL[wl.BF16], "dW2")


def test_mlp_encoder_regression_towards_stored_targets():
    """Algorithm 1 step 4 (Eq. 7) with the two-layer encoder at weights that have moved."""
    n, d_in, d_hid, d = 1200, 64, 40, 16
    X, W1, W2 = mlp_weights(804, n, d_in, d_hid, d)
    _, V1, V2 = mlp_weights(805, n, d_in, d_hid, d)
    ids, _, _, dH = small_problem(806, 3000, n, d_in=8, d=d)
    uniq = np.unique(ids)
    Ht = np.random.default_rng(807).standard_normal((uniq.size, d)).astype(np.float32)
    say("two-layer encoder, regression")
    out = run_mlp_step(X, W1, W2, ids, dH, n, [300, uniq.size - 300], targets=Ht, W_now=(V1, V2))
    miss, loss, dW1, dW2 = orc.mlp_pseudo_loss_grad(uniq, X, V1, V2, Ht.astype(np.float64))
    assert abs(sum(out["losses"]) - loss) <= TOL[wl.BF16] * loss
    assert_close(out["dW1"], dW1, TOL[wl.BF16], "dW1")
    assert_close(out["dW2"], dW2, TOL[wl.BF16], "dW2")


def test_mlp_encoder_argument_errors():
    import torch
    from paper_2204_04179_amd import gram
    with pytest.raises(gram.GramError):
        gram.Gram(gram.make_config(100, 16, 8, 50, 1, 0, 0, gram.F32, 0, 16))     # bf16 only
    with pytest.raises(gram.GramError):
        gram.Gram(gram.make_config(100, 16, 8, 50, 1, 0, 0, gram.BF16, 0, 12))    # d_hidden % 8
    lin = gram.Gram(gram.make_config(100, 16, 8, 50, 1, 0, 0, gram.BF16))
    mlp = gram.Gram(gram.make_config(100, 16, 8, 50, 1, 0, 0, gram.BF16, 0, 16))
    z = torch.zeros(4096, device="cuda")
    ids = torch.zeros(8, dtype=torch.int32, device="cuda")
    assert lin.mlp_batch_bytes(8) == 0 and mlp.mlp_batch_bytes(8) == 5 * 256

    def status(fn):
        with pytest.raises(gram.GramError) as e:
            fn()
        return e.value.status

    assert status(lambda: lin.mlp_backward(z, z, z, ids, z, None, 8, z, z, z)) == gram.ERR_ARG
    assert status(lambda: mlp.mlp_backward(z, z, z, ids, z, z, 8, z, z, z)) == gram.ERR_ARG      # both sources
    assert status(lambda: mlp.mlp_backward(z, z, z, ids, None, None, 8, z, z, z)) == gram.ERR_ARG
    assert status(lambda: mlp.mlp_backward(z, z, z, ids, z, None, 101, z, z, z)) == gram.ERR_ARG
    assert status(lambda: mlp.mlp_encode_gather(z, z, z, ids, ids, None, 8, None, None, z)) == gram.ERR_SEQUENCE
    dW1, dW2 = torch.ones(16, 16, device="cuda"), torch.ones(16, 8, device="cuda")
    mlp.mlp_backward(z, z, z, None, None, None, 0, None, dW1, dW2)                                # empty batch
    mlp.check()
    assert not bool(dW1.any()) and not bool(dW2.any())
    lin.close()
    mlp.close()


# ---------------------------------------------- dense-by-vocabulary buffer (long windows) --

@pytest.mark.parametrize("bf16", [False, True])
def test_dense_buffer_window_matches_oracle(bf16):
    """One row per ID instead of the slot table (Section 4.2 at epoch scale): every output of a
    multi-step window, pseudo-targets, weight gradient whole and in ID ranges, and a second window
    on the same context (the rows of the first must be zero again)."""
    class W_:                      # name only, for the report line of full_window_check
        name = f"dense bf16={bf16}"
    K, n, d_in, d = 3, 1500, 64, 40
    probs = [small_problem(600 + k, 4000 + 300 * k, n, d_in=d_in, d=d, bf16=bf16) for k in range(K)]
    X, W = probs[0][1], probs[0][2]
    batches = [(p[0], p[3]) for p in probs]
    dt = wl.BF16 if bf16 else wl.F32
    chunks = [(0, 100), (100, 37), (137, 1000), (1137, 100000), (5000, 3)]
    say(W_.name)
    out = run_window(X, W, batches, vocab_n=n, k_steps=K, max_positions=5000, dense=True, pseudo=True,
                     wgrad_chunks=chunks)
    assert out["counts_total"].dtype == np.int64
    ref = full_window_check(W_, batches, X, W, out, TOL[dt], TOL_SUM[dt])
    mm = orc.GramMulti(X, W)
    for k, (ids, dH) in enumerate(batches):
        st_ref = mm.step(ids, dH)
        Ht_ref, loss_ref = orc.pseudo_target(st_ref["E"], mm.rows(st_ref["uniq"]))
        assert_close(out["steps"][k]["Ht"], Ht_ref, TOL_SUM[dt], f"Ht step {k}")
        assert abs(out["steps"][k]["loss"] - loss_ref) <= TOL_SUM[dt] * loss_ref
    scale = np.abs(ref["dW"]).max()
    for (a, nrows), got in zip(chunks, out["dW_chunks"]):
        sel = (ref["uniq"] >= a) & (ref["uniq"] < a + nrows)
        want = orc.wgrad(ref["uniq"][sel], X, ref["G"][sel], 0) if sel.any() else np.zeros_like(ref["dW"])
        assert np.abs(got - want).max() <= TOL[dt] * scale, (a, nrows)
    assert_close(out["dW_chunked"], ref["dW"], TOL[dt], "sum of ID ranges")
    # second window, other batches first: nothing of the first window may be left in the rows
    again = run_window(X, W, batches[::-1], vocab_n=n, k_steps=K, max_positions=5000, dense=True,
                       gram_obj=out["gram"])
    full_window_check(W_, batches[::-1], X, W, again, TOL[dt], TOL_SUM[dt])


def test_dense_buffer_on_a_paper_shaped_multi_step_workload():
    w = wl.get("kt_multi")
    X, W = wl.features(w), wl.weights(w)
    batches = [(wl.ids(w, k).reshape(-1), wl.upstream_grad(w, k)) for k in range(w.K)]
    say("dense kt_multi")
    out = run_window(X, W, batches, vocab_n=w.N, k_steps=w.K, dense=True)
    full_window_check(w, batches, X, W, out, TOL[w.xw_dtype], TOL_SUM[w.xw_dtype])


def test_dense_buffer_window_saved_and_resumed_and_wide_counts():
    """A window exported after two steps (gram_flush64), merged back (gram_window_import) and
    continued ends like the uninterrupted window; counts beyond 2^31 stay exact in 64 bits and
    saturate in gram_flush."""
    import torch
    from paper_2204_04179_amd import gram
    K, n, d_in, d = 4, 700, 16, 8
    probs = [small_problem(700 + k, 2000, n, d_in=d_in, d=d) for k in range(K)]
    X, W = probs[0][1], probs[0][2]
    batches = [(p[0], p[3]) for p in probs]
    say("dense save / resume")
    first = run_window(X, W, batches[:2], vocab_n=n, k_steps=K, max_positions=2000, dense=True)
    saved = (first["uniq_total"], first["counts_total"], first["G_total"])
    second = run_window(X, W, batches[2:], vocab_n=n, k_steps=K, max_positions=2000, dense=True,
                        gram_obj=first["gram"], resume=saved)
    mm = orc.GramMulti(X, W)
    for ids, dH in batches:
        mm.step(ids, dH)
    ref = mm.finish()
    np.testing.assert_array_equal(second["uniq_total"], ref["uniq"])
    np.testing.assert_array_equal(second["counts_total"], ref["counts"])
    assert_close(second["G_total"], ref["G"], 1e-5, "G after resume")
    assert_close(second["dW"], ref["dW"], 1e-5, "dW after resume")
    # a resumed window alone (no further step) can take its weight gradient and be exported
    g = first["gram"]
    big_ids = torch.tensor([0, 7, 699], dtype=torch.int32, device="cuda")
    big_cnt = torch.tensor([2 ** 31 + 5, 2 ** 40, 3], dtype=torch.int64, device="cuda")
    rows = torch.arange(3 * d, dtype=torch.float32, device="cuda").reshape(3, d)
    rows[0] = 0.0                                                  # the padding item's row is zero
    g.window_import(big_ids, big_cnt, rows, 3)
    dW = torch.full((d_in, d), float("nan"), device="cuda")
    g.encoder_wgrad(first["X_dev"], dW)
    want = orc.wgrad(np.array([0, 7, 699], np.int32), X, rows.cpu().numpy().astype(np.float64), 0)
    assert_close(dW.cpu().numpy(), want, 1e-5, "dW of an imported window")
    # one more step on top, then the 64-bit export
    ids = np.array([7, 0, 0, 9, 0], np.int32)
    after = run_window(X, W, [(ids, np.ones((5, d), np.float32))], vocab_n=n, k_steps=K, max_positions=2000,
                       dense=True, gram_obj=g)
    assert after["uniq_total"].tolist() == [0, 7, 9, 699]
    assert after["counts_total"].tolist() == [2 ** 31 + 8, 2 ** 40 + 1, 1, 3]
    np.testing.assert_array_equal(after["G_total"][1], rows[1].cpu().numpy() + 1.0)
    assert not after["G_total"][0].any()                           # the padding item keeps a zero row ...
    # ... and the 32-bit export saturates
    g.window_import(big_ids, big_cnt, None, 3)
    u = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    c32 = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    assert g.flush(u, c32, None, None, want_host_u=True) == 3
    assert c32[:3].tolist() == [2 ** 31 - 1, 2 ** 31 - 1, 3] and u[:3].tolist() == [0, 7, 699]
    assert g.flush64(u, None, None, None, want_host_u=True) == 0   # empty again


def test_slot_table_window_saved_and_resumed():
    """The same save / resume through the default slot-table buffer: export with widened counts
    (gram_flush64), import into the emptied buffer, continue; items of the saved state keep their
    sums, new items take rows behind them, and the export is in ascending ID order again."""
    import torch
    K, n, d_in, d = 4, 700, 16, 8
    probs = [small_problem(720 + k, 2000, n, d_in=d_in, d=d) for k in range(K)]
    X, W = probs[0][1], probs[0][2]
    batches = [(p[0], p[3]) for p in probs]
    say("slot table save / resume")
    first = run_window(X, W, batches[:2], vocab_n=n, k_steps=K, max_positions=2000)
    perm = np.random.default_rng(5).permutation(first["uniq_total"].size)        # any order of distinct IDs
    saved = (first["uniq_total"][perm], first["counts_total"][perm].astype(np.int64), first["G_total"][perm])
    second = run_window(X, W, batches[2:], vocab_n=n, k_steps=K, max_positions=2000, gram_obj=first["gram"],
                        resume=saved)
    mm = orc.GramMulti(X, W)
    for ids, dH in batches:
        mm.step(ids, dH)
    ref = mm.finish()
    np.testing.assert_array_equal(second["uniq_total"], ref["uniq"])
    np.testing.assert_array_equal(second["counts_total"], ref["counts"])
    assert_close(second["G_total"], ref["G"], 1e-5, "G after resume")
    assert_close(second["dW"], ref["dW"], 1e-5, "dW after resume")
    # an imported state alone: weight gradient and a 64-bit export; the slot table counts in 64 bits
    g = first["gram"]
    ids3 = torch.tensor([699, 7, 0], dtype=torch.int32, device="cuda")
    cnt3 = torch.tensor([3, 2 ** 40, 2 ** 31 + 5], dtype=torch.int64, device="cuda")
    rows = torch.arange(3 * d, dtype=torch.float32, device="cuda").reshape(3, d)
    rows[2] = 0.0
    g.window_import(ids3, cnt3, rows, 3)
    g.window_import(ids3[:1], cnt3[:1], rows[:1], 1)                 # a second import meets item 699 again
    dW = torch.full((d_in, d), float("nan"), device="cuda")
    g.encoder_wgrad(first["X_dev"], dW)
    r = rows.cpu().numpy().astype(np.float64)
    r[0] *= 2
    want = orc.wgrad(np.array([699, 7, 0], np.int32), X, r, 0)
    assert_close(dW.cpu().numpy(), want, 1e-5, "dW of an imported window")
    u = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    c64 = torch.full((n,), -7, dtype=torch.int64, device="cuda")
    Gt = torch.full((n, d), float("nan"), device="cuda")
    assert g.flush64(u, c64, Gt, None, want_host_u=True) == 3
    assert u[:3].tolist() == [0, 7, 699] and c64[:3].tolist() == [2 ** 31 + 5, 2 ** 40, 6]
    np.testing.assert_array_equal(Gt[:3].cpu().numpy(), np.stack([r[2], r[1], r[0]]).astype(np.float32))
    assert g.flush(u, None, None, None, want_host_u=True) == 0
    # counts beyond 2^31 keep growing step after step (no wrap), and only the 32-bit export saturates
    g.window_import(ids3, cnt3, None, 3)
    ids_d = torch.from_numpy(batches[0][0]).cuda()
    uq, cn = (torch.zeros(n, dtype=torch.int32, device="cuda") for _ in range(2))
    inv = torch.zeros(ids_d.numel(), dtype=torch.int32, device="cuda")
    g.unique(ids_d, uq, inv, cn)
    g.grad_accumulate(torch.from_numpy(batches[0][1]).cuda(), ids_d.numel(), 0)
    c32 = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    n_items = g.flush(u, c32, None, None, want_host_u=True)
    ref_u, ref_c = np.unique(batches[0][0], return_counts=True)
    want = dict(zip(ref_u.tolist(), ref_c.tolist()))
    for i, c in ((699, 3), (7, 2 ** 40), (0, 2 ** 31 + 5)):
        want[i] = want.get(i, 0) + c
    assert n_items == len(want)
    assert u[:n_items].tolist() == sorted(want)
    assert c32[:n_items].tolist() == [min(want[i], 2 ** 31 - 1) for i in sorted(want)]


def test_dense_buffer_window_of_two_thousand_steps():
    """An accumulation period in the thousands (the half-epoch / one-epoch periods of the
    experiments): 2,000 mini-batches into the one-row-per-ID buffer, then one weight gradient and
    one export, against the oracle's window."""
    import torch
    from paper_2204_04179_amd import gram
    K, n, d_in, d, m = 2000, 3000, 16, 8, 512
    rng = np.random.default_rng(950)
    X = rng.standard_normal((n, d_in)).astype(np.float32)
    W = (rng.standard_normal((d_in, d)) / 4).astype(np.float32)
    ids_all = rng.zipf(1.3, size=(K, m)).astype(np.int64) % n          # popular items recur in every batch
    ids_all[rng.random((K, m)) < 0.1] = 0
    ids_all = ids_all.astype(np.int32)
    dH_all = rng.standard_normal((K, m, d)).astype(np.float32)
    say("dense window of 2000 steps")
    g = gram.Gram(gram.make_config(n, d_in, d, m, K, 0, 0, gram.F32, 1))
    Xd, Wd = torch.from_numpy(X).cuda(), torch.from_numpy(W).cuda()
    ids_d, dH_d = torch.from_numpy(ids_all).cuda(), torch.from_numpy(dH_all).cuda()
    i32 = dict(dtype=torch.int32, device="cuda")
    uniq, counts, inverse, u_dev = torch.empty(m, **i32), torch.empty(m, **i32), torch.empty(m, **i32), torch.zeros(1, **i32)
    H = torch.empty(m, d, device="cuda")
    for k in range(K):
        g.unique(ids_d[k], uniq, inverse, counts, u_dev)
        g.encode_gather(Xd, Wd, uniq, inverse, u_dev, m, None, H)
        g.grad_accumulate(dH_d[k], m, k)
    dW = torch.empty(d_in, d, device="cuda")
    g.encoder_wgrad(Xd, dW)
    ut, ct = torch.empty(n, **i32), torch.empty(n, dtype=torch.int64, device="cuda")
    Gt = torch.empty(n, d, device="cuda")
    u_total = g.flush64(ut, ct, Gt, None, want_host_u=True)
    mm = orc.GramMulti(X, W)
    for k in range(K):
        uq, inv, cnt = orc.unique(ids_all[k], n)
        Gk = orc.grad_accumulate(dH_all[k], inv, uq, 0)
        orc._check(orc.lib().oracle_buffer_add(mm._buf, orc._p(uq, orc.C.c_int32), orc._p(cnt, orc.C.c_int32),
                                               orc._p(Gk, orc.C.c_double), uq.size), "buffer_add")
    ref = mm.finish()
    assert u_total == ref["uniq"].size
    np.testing.assert_array_equal(ut[:u_total].cpu().numpy(), ref["uniq"])
    np.testing.assert_array_equal(ct[:u_total].cpu().numpy(), ref["counts"])
    assert int(ref["counts"].sum()) == K * m
    # 2,000 float32 additions per row in a fixed order against float64: a few 1e-6 relative at most
    assert_close(Gt[:u_total].cpu().numpy(), ref["G"], 2e-5, "G after 2000 steps")
    assert_close(dW.cpu().numpy(), ref["dW"], 2e-5, "dW after 2000 steps")
    g.close()


def test_dense_buffer_argument_errors():
    import torch
    from paper_2204_04179_amd import gram
    with pytest.raises(gram.GramError):
        gram.Gram(gram.make_config(100, 16, 8, 50, 1, 0, 5, gram.F32, 1))        # one row per ID: no other capacity
    with pytest.raises(gram.GramError):
        gram.Gram(gram.make_config(100, 16, 8, 50, 1, 0, 0, gram.F32, 2))        # unknown layout
    slots = gram.Gram(gram.make_config(100, 16, 8, 50, 1, 0, 0, gram.F32))
    u = torch.zeros(100, dtype=torch.int32, device="cuda")
    c64 = torch.zeros(100, dtype=torch.int64, device="cuda")
    with pytest.raises(gram.GramError) as e:
        slots.window_import(u, c64, None, 51)                                    # more items than buffer rows
    assert e.value.status == gram.ERR_ARG
    dense = gram.Gram(gram.make_config(100, 16, 8, 50, 1, 0, 0, gram.F32, 1))
    with pytest.raises(gram.GramError) as e:
        dense.window_import(u, c64, None, 101)
    assert e.value.status == gram.ERR_ARG
    u[3] = 100                                                                   # outside [0, N): skipped, latched
    c64[:] = 1
    dense.window_import(u[3:4], c64[3:4], None, 1)
    with pytest.raises(gram.GramError) as e:
        dense.check()
    assert e.value.status == gram.ERR_RANGE
    assert dense.flush64(u, c64, None, None, want_host_u=True) == 0
    slots.close()
    dense.close()


def bf16_round(a):
    """float32 array rounded to bf16 (nearest even) and widened again."""
    return wl.bf16_bits_to_f32(wl.f32_to_bf16_bits(np.ascontiguousarray(a, dtype=np.float32)))


@pytest.mark.parametrize("case", ["small", "fused", "fused_with_E", "foreign"])
def test_positions_output_in_bf16(case):
    """h_dtype = bf16: every way the forward reaches the positions (gather kernel, fused epilogue for
    light items + copy kernel for heavy ones, gram_gather of pseudo-targets) stores exactly the
    nearest-even bf16 of the float32 representation; E, G and dW are untouched by the option."""
    if case == "small":
        n, m, d_in, d = 2500, 7000, 32, 24
        ids = None
    else:
        n, m, d_in, d = 70000, 70000, 64, 256
        rng = np.random.default_rng(41)
        ids = rng.integers(1, 3000, size=m).astype(np.int32)
        ids[: m // 2] = rng.integers(1, n, size=m // 2)
        ids[rng.random(m) < 0.05] = 0
    ids, X, W, dH = small_problem(42, m, n, d_in=d_in, d=d, bf16=True, ids=ids)
    say(f"bf16 H, {case}")
    kw = dict(pass_E=case != "fused", foreign_buffers=case == "foreign", pseudo=case in ("small", "fused_with_E"))
    out = run_window(X, W, [(ids, dH)], vocab_n=n, h_bf16=True, **kw)
    base = run_window(X, W, [(ids, dH)], vocab_n=n, **kw)
    st, st0 = out["steps"][0], base["steps"][0]
    ref = orc.gram_single(ids, X, W, dH)
    np.testing.assert_array_equal(st["H"], bf16_round(st0["H"]))            # pure rounding of the same values
    assert_close(st["H"], ref["H"], 2.0 ** -8, "H (bf16)")
    assert np.all(st["H"][ids == 0] == 0.0)
    if "E" in st:
        np.testing.assert_array_equal(st["E"], st0["E"])
    if kw["pseudo"]:
        np.testing.assert_array_equal(st["H_tilde"], bf16_round(st["Ht"])[ref["inverse"]])
    assert out["G_total"].tobytes() == base["G_total"].tobytes() and out["dW"].tobytes() == base["dW"].tobytes()


@pytest.mark.parametrize("end", ["two_calls", "one_call"])
def test_window_captured_in_a_hip_graph_replays_like_eager(end):
    """The calls only enqueue kernels (no memset nodes, no host read-backs unless asked for), so a
    whole window can be captured once and replayed; every replay, with eager work and
    synchronisations in between, must reproduce the eager window bit for bit.  The window ends with
    gram_encoder_wgrad + gram_flush, or with gram_window_end."""
    import torch
    from paper_2204_04179_amd import gram
    from harness import to_dev
    K, n, d_in, d, m = 2, 3000, 64, 32, 9000
    probs = [small_problem(900 + k, m, n, d_in=d_in, d=d, bf16=True) for k in range(K)]
    X, W = to_dev(probs[0][1], torch), to_dev(probs[0][2], torch)
    ids = [torch.from_numpy(p[0]).cuda() for p in probs]
    dH = [torch.from_numpy(p[3]).cuda() for p in probs]
    g = gram.Gram(gram.make_config(n, d_in, d, m, K, 0, 0, gram.BF16))
    i32 = dict(dtype=torch.int32, device="cuda")
    uniq, counts, inverse, u_dev = torch.empty(n, **i32), torch.empty(n, **i32), torch.empty(m, **i32), torch.zeros(1, **i32)
    H = torch.empty(m, d, device="cuda")
    dW = torch.empty(d_in, d, device="cuda")
    ut, ct, Gt, n_t = torch.empty(n, **i32), torch.empty(n, **i32), torch.empty(n, d, device="cuda"), torch.zeros(1, **i32)
    outs = (H, dW, ut, ct, Gt, n_t)

    def window():
        for k in range(K):
            g.unique(ids[k], uniq, inverse, counts, u_dev)
            g.encode_gather(X, W, uniq, inverse, u_dev, m, None, H)
            g.grad_accumulate(dH[k], m, k)
        if end == "one_call":
            g.window_end(X, dW, ut, ct, Gt, n_t)
        else:
            g.encoder_wgrad(X, dW)
            g.flush(ut, ct, Gt, n_t)

    def snapshot():
        torch.cuda.synchronize()
        u = int(n_t.item())
        return [t.clone() if t is not ut and t is not ct and t is not Gt else t[:u].clone() for t in outs]

    say(f"graph capture of a window ({end})")
    window()
    eager = snapshot()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        window()                                   # warm-up on a capture-capable stream
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        window()
    for rep in range(3):
        for t in outs:
            t.zero_()                              # eager work between the replays
        torch.cuda.synchronize()
        graph.replay()
        got = snapshot()
        for a, b in zip(eager, got):
            assert torch.equal(a, b), f"replay {rep}"
    window()                                       # and eager again after the replays
    for a, b in zip(eager, snapshot()):
        assert torch.equal(a, b)
    g.check()
    g.close()


def test_flush_variants_and_back_to_back_windows():
    """gram_flush with and without the G export gives the same IDs and counts; a second flush of an
    empty window returns nothing; a context runs window after window with one- and multi-step
    windows mixed (the count of buffer rows restarts with each window)."""
    import torch
    n, K = 900, 3
    probs = [small_problem(300 + k, 3000, n, d_in=16, d=8) for k in range(K)]
    X, W = probs[0][1], probs[0][2]
    batches = [(p[0], p[3]) for p in probs]
    a = run_window(X, W, batches, vocab_n=n, k_steps=K, want_G=True)
    b = run_window(X, W, batches, vocab_n=n, k_steps=K, want_G=False, gram_obj=a["gram"])
    np.testing.assert_array_equal(a["uniq_total"], b["uniq_total"])
    np.testing.assert_array_equal(a["counts_total"], b["counts_total"])
    assert a["dW"].tobytes() == b["dW"].tobytes()
    g = a["gram"]
    u = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    cnt = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    ud = torch.full((1,), -7, dtype=torch.int32, device="cuda")
    assert g.flush(u, cnt, None, ud, want_host_u=True) == 0          # empty window
    assert int(ud.item()) == 0 and bool((u == -7).all().item())
    # a one-step window on the same context, then the full window again
    c = run_window(X, W, batches[:1], vocab_n=n, k_steps=K, gram_obj=g, max_positions=3000)
    ref = orc.gram_single(batches[0][0], X, W, batches[0][1])
    np.testing.assert_array_equal(c["uniq_total"], ref["uniq"])
    assert_close(c["G_total"], ref["G"], 1e-5, "G one-step window")
    d = run_window(X, W, batches, vocab_n=n, k_steps=K, gram_obj=g)
    assert d["G_total"].tobytes() == a["G_total"].tobytes() and d["dW"].tobytes() == a["dW"].tobytes()


@pytest.mark.parametrize("case", ["multi_step", "one_step", "three_feature_tiles", "resumed", "no_rows_wanted",
                                  "float32", "dense_falls_back"])
def test_window_end_in_one_call_equals_weight_gradient_then_flush(case):
    """gram_window_end against gram_encoder_wgrad followed by gram_flush on the same window: IDs,
    counts, every row of G_total and every entry of dW bit for bit, rows beyond the export
    untouched, and the context ready for the next window.  The shapes take the weight-gradient
    kernel through split ranges of the rows, one to three feature tiles (each buffer row is
    written by one of them), a window whose rows are already in ID order (one step) and one that
    needs the sort; float32 features and the dense buffer take the two steps one after the other."""
    K, n, d_in, d, m, bf16 = 3, 30000, 512, 256, 9000, True
    kw = {}
    if case == "one_step":
        K = 1
    elif case == "three_feature_tiles":
        d_in, d, n, m = 640, 264, 9000, 5000
    elif case == "float32":
        bf16, d_in, d, n, m = False, 48, 24, 2000, 3000
    elif case == "no_rows_wanted":
        kw["want_G"] = False
    probs = [small_problem(500 + k, m, n, d_in=d_in, d=d, bf16=bf16) for k in range(K)]
    X, W = probs[0][1], probs[0][2]
    batches = [(p[0], p[3]) for p in probs]
    if case == "resumed":
        rng = np.random.default_rng(3)
        r_ids = np.sort(rng.choice(n, size=700, replace=False)).astype(np.int32)
        kw["resume"] = (r_ids, rng.integers(1, 9, size=700).astype(np.int64),
                        rng.standard_normal((700, d)).astype(np.float32))
    if case == "dense_falls_back":
        import torch
        a = run_window(X, W, batches, vocab_n=n, k_steps=K, dense=True)
        g = a["gram"]
        for k, (ids, dH) in enumerate(batches):
            ids_d, dH_d = torch.from_numpy(ids).cuda(), torch.from_numpy(dH).cuda()
            uq = torch.empty(min(m, n), dtype=torch.int32, device="cuda")
            inv = torch.empty(m, dtype=torch.int32, device="cuda")
            cn, ud = torch.empty_like(uq), torch.zeros(1, dtype=torch.int32, device="cuda")
            H = torch.empty(m, d, device="cuda")
            g.unique(ids_d, uq, inv, cn, ud)
            g.encode_gather(a["X_dev"], a["W_dev"], uq, inv, ud, m, None, H)
            g.grad_accumulate(dH_d, m, k)
        dW = torch.full((d_in, d), float("nan"), device="cuda")
        ut = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        ct = torch.full((n,), -7, dtype=torch.int32, device="cuda")
        Gt = torch.full((n, d), float("nan"), device="cuda")
        nn = g.window_end(a["X_dev"], dW, ut, ct, Gt, None, want_host_u=True)
        assert nn == a["U_total"]
        np.testing.assert_array_equal(ut[:nn].cpu().numpy(), a["uniq_total"])
        np.testing.assert_array_equal(ct[:nn].cpu().numpy().astype(np.int64), a["counts_total"])
        assert Gt[:nn].cpu().numpy().tobytes() == a["G_total"].tobytes()
        assert dW.cpu().numpy().tobytes() == a["dW"].tobytes()
        return
    prof = ["wgrad_bf16", "wgrad_f32", "flush_rows", "flush_meta"]
    a = run_window(X, W, batches, vocab_n=n, k_steps=K, **kw)
    b = run_window(X, W, batches, vocab_n=n, k_steps=K, gram_obj=a["gram"], window_end=True, profile=prof, **kw)
    launches = {k: v[0] for k, v in b["profile"].items() if v[0]}
    say(f"{case}: U_total={a['U_total']} launches of the one call: {launches}")
    if case == "resumed":
        assert launches.pop("flush_rows") == 1       # gram_window_import's row kernel is counted under this name
    # bf16: no launch of the export's row copy (with no rows wanted there is none either way); after a
    # single step the weight-gradient launch exports the IDs and counts as well
    assert launches == ({"wgrad_bf16": 1} if case == "one_step" else
                        {"wgrad_bf16": 1, "flush_meta": 1} if bf16 else {"wgrad_f32": 1, "flush_rows": 1})
    assert a["U_total"] == b["U_total"] and a["U_total"] > 0
    np.testing.assert_array_equal(a["uniq_total"], b["uniq_total"])
    np.testing.assert_array_equal(a["counts_total"], b["counts_total"])
    assert a["dW"].tobytes() == b["dW"].tobytes()
    if case != "no_rows_wanted":
        assert a["G_total"].tobytes() == b["G_total"].tobytes()
        assert b["G_tail_untouched"]
    # against the oracle as well, and the next window on the same context starts clean
    acc = orc.GramMulti(X, W, pad_id=0)
    if case == "resumed":
        acc.resume(*kw["resume"])
    for ids, dH in batches:
        acc.step(ids, dH)
    ids_t, counts_t, G_t = acc.export()
    np.testing.assert_array_equal(b["uniq_total"], ids_t)
    np.testing.assert_array_equal(b["counts_total"], counts_t)
    tol = TOL[wl.BF16 if bf16 else wl.F32]
    if case != "no_rows_wanted":
        assert_close(b["G_total"], G_t, TOL_SUM[wl.BF16 if bf16 else wl.F32], "G_total of the one call")
    assert_close(b["dW"], orc.wgrad(ids_t, X, G_t, 0), tol, "dW of the one call")
    c = run_window(X, W, batches, vocab_n=n, k_steps=K, gram_obj=a["gram"], **kw)
    assert c["dW"].tobytes() == a["dW"].tobytes()
    np.testing.assert_array_equal(c["counts_total"], a["counts_total"])


@pytest.mark.parametrize("m", [3000, 30000])
def test_buffer_rows_are_assigned_afresh_when_the_window_changed_after_the_dedup(m):
    """gram_unique works out the buffer rows of the batch's items from the slot table as it is;
    if the table changes before gram_grad_accumulate (here: a saved state is merged in between),
    the accumulate step must not use them.  Both dedup variants (one block, sorted tiles);
    checked against the oracle's resumed window."""
    import torch
    from paper_2204_04179_amd import gram
    from harness import to_dev
    n, d_in, d = 5000, 32, 16
    ids, X, W, dH = small_problem(77, m, n, d_in=d_in, d=d)
    ids2, _, _, dH2 = small_problem(78, m, n, d_in=d_in, d=d)
    rng = np.random.default_rng(5)
    r_ids = np.sort(rng.choice(n, size=900, replace=False)).astype(np.int32)
    r_cnt = rng.integers(1, 5, size=900).astype(np.int64)
    r_G = rng.standard_normal((900, d)).astype(np.float32)
    g = gram.Gram(gram.make_config(n, d_in, d, m, 2, 0, 0, gram.F32))
    Xd, Wd = to_dev(X, torch), to_dev(W, torch)
    cap_u = min(m, n)
    uq = torch.empty(cap_u, dtype=torch.int32, device="cuda")
    cn, inv = torch.empty_like(uq), torch.empty(m, dtype=torch.int32, device="cuda")
    ud = torch.zeros(1, dtype=torch.int32, device="cuda")
    H = torch.empty(m, d, device="cuda")
    # step 0: dedup first, THEN the import, then accumulate
    g.unique(torch.from_numpy(ids).cuda(), uq, inv, cn, ud)
    g.encode_gather(Xd, Wd, uq, inv, ud, m, None, H)
    g.window_import(torch.from_numpy(r_ids).cuda(), torch.from_numpy(r_cnt).cuda(), torch.from_numpy(r_G).cuda(), 900)
    g.grad_accumulate(torch.from_numpy(dH).cuda(), m, 0)
    # step 1: the ordinary order (rows committed as worked out)
    g.unique(torch.from_numpy(ids2).cuda(), uq, inv, cn, ud)
    g.encode_gather(Xd, Wd, uq, inv, ud, m, None, H)
    g.grad_accumulate(torch.from_numpy(dH2).cuda(), m, 1)
    dW = torch.empty(d_in, d, device="cuda")
    ut = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    ct = torch.full((n,), -7, dtype=torch.int32, device="cuda")
    Gt = torch.full((n, d), float("nan"), device="cuda")
    nn = g.window_end(Xd, dW, ut, ct, Gt, None, want_host_u=True)
    acc = orc.GramMulti(X, W, pad_id=0)
    acc.resume(r_ids, r_cnt, r_G)
    acc.step(ids, dH)
    acc.step(ids2, dH2)
    ref = acc.finish()
    assert nn == ref["uniq"].size
    np.testing.assert_array_equal(ut[:nn].cpu().numpy(), ref["uniq"])
    np.testing.assert_array_equal(ct[:nn].cpu().numpy(), ref["counts"])
    assert_close(Gt[:nn].cpu().numpy(), ref["G"], 1e-5, "G_total")
    assert_close(dW.cpu().numpy(), ref["dW"], 1e-5, "dW")


@pytest.mark.parametrize("K", [1, 2])
def test_window_end_with_a_full_buffer_drops_the_same_rows_as_the_two_calls(K):
    """A buffer smaller than the window's items: the rows beyond its capacity are dropped (never
    written out of bounds) and the error is latched; gram_window_end exports exactly what
    gram_encoder_wgrad + gram_flush export, and an empty window is refused by both."""
    import torch
    from paper_2204_04179_amd import gram
    from harness import to_dev
    n, d_in, d, m, cap = 4000, 64, 32, 3000, 700
    probs = [small_problem(40 + k, m, n, d_in=d_in, d=d, bf16=True) for k in range(K)]
    X, W = to_dev(probs[0][1], torch), to_dev(probs[0][2], torch)
    res = []
    for one_call in (False, True):
        g = gram.Gram(gram.make_config(n, d_in, d, m, K, 0, cap, gram.BF16))
        dW = torch.full((d_in, d), float("nan"), device="cuda")
        with pytest.raises(gram.GramError) as e:
            (g.window_end if one_call else g.encoder_wgrad)(X, dW)
        assert e.value.status == gram.ERR_SEQUENCE
        uq = torch.empty(min(m, n), dtype=torch.int32, device="cuda")
        cn, inv = torch.empty_like(uq), torch.empty(m, dtype=torch.int32, device="cuda")
        ud = torch.zeros(1, dtype=torch.int32, device="cuda")
        H = torch.empty(m, d, device="cuda")
        for k, p in enumerate(probs):
            g.unique(torch.from_numpy(p[0]).cuda(), uq, inv, cn, ud)
            g.encode_gather(X, W, uq, inv, ud, m, None, H)
            g.grad_accumulate(torch.from_numpy(p[3]).cuda(), m, k)
        ut = torch.full((cap + 8,), -7, dtype=torch.int32, device="cuda")
        ct = torch.full((cap + 8,), -7, dtype=torch.int32, device="cuda")
        Gt = torch.full((cap + 8, d), float("nan"), device="cuda")
        nt = torch.zeros(1, dtype=torch.int32, device="cuda")
        if one_call:
            g.window_end(X, dW, ut, ct, Gt, nt)
        else:
            g.encoder_wgrad(X, dW)
            g.flush(ut, ct, Gt, nt)
        torch.cuda.synchronize()
        with pytest.raises(gram.GramError) as e:
            g.check()
        assert e.value.status == gram.ERR_CAPACITY
        assert int(nt.item()) == cap
        assert bool((ut[cap:] == -7).all().item()) and bool(torch.isnan(Gt[cap:]).all().item())
        res.append([t.cpu().numpy().tobytes() for t in (ut[:cap], ct[:cap], Gt[:cap], dW)])
        g.close()
    assert res[0] == res[1]


def test_error_paths():
    import torch
    from paper_2204_04179_amd import gram
    n, d_in, d, m = 50, 8, 4, 64
    cfg = gram.make_config(n, d_in, d, m, 2, 0, 0, gram.F32)
    g = gram.Gram(cfg)
    ids = torch.randint(1, n, (m,), dtype=torch.int32, device="cuda")
    uniq = torch.empty(n, dtype=torch.int32, device="cuda")
    cnt = torch.empty(n, dtype=torch.int32, device="cuda")
    inv = torch.empty(m, dtype=torch.int32, device="cuda")
    dH = torch.randn(m, d, device="cuda")
    X = torch.randn(n, d_in, device="cuda")
    dW = torch.empty(d_in, d, device="cuda")

    def status(fn):
        with pytest.raises(gram.GramError) as e:
            fn()
        return e.value.status

    say("errors: sequence")
    assert status(lambda: g.grad_accumulate(dH, m, 0)) == gram.ERR_SEQUENCE        # no unique yet
    assert status(lambda: g.pseudo_target(dH, dH)) == gram.ERR_SEQUENCE            # nothing accumulated yet
    assert status(lambda: g.encoder_wgrad(X, dW)) == gram.ERR_SEQUENCE             # empty window
    g.unique(ids, uniq, inv, cnt)
    assert status(lambda: g.grad_accumulate(dH, m, 1)) == gram.ERR_SEQUENCE        # wrong step index
    assert status(lambda: g.grad_accumulate(dH, m - 1, 0)) == gram.ERR_ARG         # m mismatch
    g.grad_accumulate(dH, m, 0)
    assert status(lambda: g.grad_accumulate(dH, m, 1)) == gram.ERR_SEQUENCE        # batch already used
    g.unique(ids, uniq, inv, cnt)
    g.grad_accumulate(dH, m, 1)
    g.unique(ids, uniq, inv, cnt)
    assert status(lambda: g.grad_accumulate(dH, m, 2)) == gram.ERR_SEQUENCE        # window is full
    assert g.flush(want_host_u=True) == int(torch.unique(ids).numel())
    say("errors: capacity / range")
    big = torch.zeros(m + 1, dtype=torch.int32, device="cuda")
    assert status(lambda: g.unique(big, uniq, inv, cnt)) == gram.ERR_CAPACITY
    bad = ids.clone()
    bad[5] = n
    bad[9] = -3
    assert status(lambda: g.unique(bad, uniq, inv, cnt, want_host_u=True)) == gram.ERR_RANGE
    assert g.unique(ids, uniq, inv, cnt, want_host_u=True) == int(torch.unique(ids).numel())   # flag cleared
    with pytest.raises(gram.GramError):
        gram.Gram(gram.make_config(n, d_in, 6, m, 1, 0, 0, gram.F32))               # d not a multiple of 4
    # a deliberately small persistent buffer overflows on the device and is reported at the next sync
    g2 = gram.Gram(gram.make_config(n, d_in, d, m, 1, 0, 3, gram.F32))
    g2.unique(ids, uniq, inv, cnt)
    g2.grad_accumulate(dH, m, 0)
    assert status(lambda: g2.check()) == gram.ERR_CAPACITY
    assert g2.flush(want_host_u=True) == 3
    g.close()
    g2.close()


# ------------------------------------------------- randomly drawn shapes --

def random_case(seed):
    """A window of valid inputs with every shape parameter drawn at random: vocabulary, widths,
    steps, batch sizes (some empty), popularity law, padding ID (0, none, any other ID) and share,
    buffer layout, how the window is ended, E requested or not, caller buffers own or foreign,
    output type of H.  The oracle's contraction is kept affordable."""
    rng = np.random.default_rng(seed)
    bf16 = rng.random() < 0.8
    n = int(2 ** rng.uniform(1, 16.5))
    d_in = int(rng.choice([8, 16, 24, 32, 40, 64, 96, 128, 200, 256, 264, 512])) if bf16 else int(rng.integers(1, 70))
    d = int(rng.choice([4, 8, 12, 32, 64, 100, 128, 256, 260, 320, 512, 1024]))
    K = int(rng.choice([1, 1, 2, 3, 5]))
    big = rng.random() < 0.3
    m_hi = 150000 if big else 20000
    pad_mode = rng.choice(["zero", "none", "other"], p=[0.6, 0.2, 0.2])
    pad_id = 0 if pad_mode == "zero" else (-1 if pad_mode == "none" else int(rng.integers(0, n)))
    pad_frac = float(rng.choice([0.0, 0.1, 0.5]))
    s = float(rng.choice([0.0, 0.8, 1.1, 1.5]))
    dense = rng.random() < 0.15
    kw = dict(pad_id=pad_id, dense=dense, window_end=(not dense) and rng.random() < 0.6, pass_E=rng.random() < 0.5,
              foreign_buffers=rng.random() < 0.2, h_bf16=rng.random() < 0.2)
    ms = [0 if rng.random() < 0.05 else int(2 ** rng.uniform(np.log2(m_hi) - 5 if big else 0, np.log2(m_hi)))
          for _ in range(K)]
    if sum(ms) == 0:
        ms[0] = 5
    while K * max(ms) * d_in * d > 2e9:
        ms = [m // 2 for m in ms]
    p = np.arange(1, n + 1, dtype=np.float64) ** (-s)
    p /= p.sum()
    perm = rng.permutation(n)
    batches = []
    for m in ms:
        ids = perm[rng.choice(n, size=m, p=p)].astype(np.int32) if m else np.zeros(0, np.int32)
        if pad_id >= 0 and m:
            ids[rng.random(m) < pad_frac] = pad_id
        batches.append((ids, rng.standard_normal((m, d)).astype(np.float32)))
    X = rng.standard_normal((n, d_in)).astype(np.float32)
    W = (rng.standard_normal((d_in, d)) / np.sqrt(d_in)).astype(np.float32)
    if bf16:
        X, W = wl.f32_to_bf16_bits(X), wl.f32_to_bf16_bits(W)
    shape = dict(seed=seed, bf16=bf16, n=n, d_in=d_in, d=d, ms=ms, s=s, pad_frac=pad_frac, **kw)
    return shape, X, W, batches, n, K, kw


@pytest.mark.parametrize("first_seed", [0, 30, 60, 90])
def test_randomly_drawn_shapes_against_the_oracle(first_seed):
    """30 windows per case, every parameter of the problem drawn at random (see random_case);
    integers bit-exact, E / H / G_total / dW within the bars of the fixed-shape tests (H in bf16:
    its rounding, 2^-9 per element)."""
    for seed in range(first_seed, first_seed + 30):
        shape, X, W, batches, n, K, kw = random_case(seed)
        say("random shape:", shape)
        dt = wl.BF16 if shape["bf16"] else wl.F32
        out = run_window(X, W, batches, vocab_n=n, k_steps=K, max_positions=max(1, max(shape["ms"])), **kw)
        acc = orc.GramMulti(X, W, pad_id=kw["pad_id"])
        for k, (ids, dH) in enumerate(batches):
            ref = acc.step(ids, dH)
            st = out["steps"][k]
            check_step_exact(st, ref)
            if ids.size:
                if "E" in st:
                    assert_close(st["E"], ref["E"], TOL_SUM[dt], f"E step {k}")
                assert_close(st["H"], ref["H"], 8e-3 if kw["h_bf16"] else TOL_SUM[dt], f"H step {k}")
        ref = acc.finish()
        np.testing.assert_array_equal(out["uniq_total"], ref["uniq"])
        np.testing.assert_array_equal(out["counts_total"], ref["counts"])
        if ref["uniq"].size:
            assert_close(out["G_total"], ref["G"], TOL_SUM[dt], "G_total")
        assert out["G_tail_untouched"]
        if np.abs(ref["dW"]).max() > 0:
            assert_close(out["dW"], ref["dW"], TOL[dt], "dW")
        else:
            assert not out["dW"].any()
        out["gram"].close()


@pytest.mark.parametrize("first_seed", [0, 30])
def test_randomly_drawn_windows_with_pseudo_targets_chunks_and_a_resumed_state(first_seed):
    """30 windows per case with random shapes: pseudo-targets and pseudo-loss after every step, the
    weight gradient taken in a random partition of the buffer rows (the last chunk runs past the
    end), some windows resumed from a random saved state, slot table or dense buffer."""
    for seed in range(first_seed, first_seed + 30):
        rng = np.random.default_rng(10_000 + seed)
        bf16 = rng.random() < 0.7
        n = int(2 ** rng.uniform(3, 16))
        d_in = int(rng.choice([8, 16, 32, 64, 96, 128, 256, 264])) if bf16 else int(rng.integers(1, 70))
        d = int(rng.choice([4, 8, 12, 32, 64, 100, 128, 256, 260, 512]))
        K = int(rng.choice([1, 2, 3, 4]))
        big = rng.random() < 0.3
        m_hi = 100000 if big else 10000
        pad_id = int(rng.choice([0, 0, -1]))
        pad_frac = float(rng.choice([0.0, 0.2]))
        s = float(rng.choice([0.0, 0.8, 1.2]))
        dense = rng.random() < 0.3
        do_resume = rng.random() < 0.4
        ms = [max(1, int(2 ** rng.uniform(np.log2(m_hi) - 4 if big else 2, np.log2(m_hi)))) for _ in range(K)]
        while K * max(ms) * d_in * d > 2e9:
            ms = [max(1, m // 2) for m in ms]
        say("random window:", dict(seed=seed, bf16=bf16, n=n, d_in=d_in, d=d, ms=ms, pad_id=pad_id, dense=dense,
                                   resume=do_resume))
        p = np.arange(1, n + 1, dtype=np.float64) ** (-s)
        p /= p.sum()
        perm = rng.permutation(n)
        batches = []
        for m in ms:
            ids = perm[rng.choice(n, size=m, p=p)].astype(np.int32)
            if pad_id >= 0:
                ids[rng.random(m) < pad_frac] = pad_id
            batches.append((ids, rng.standard_normal((m, d)).astype(np.float32)))
        X = rng.standard_normal((n, d_in)).astype(np.float32)
        W = (rng.standard_normal((d_in, d)) / np.sqrt(d_in)).astype(np.float32)
        if bf16:
            X, W = wl.f32_to_bf16_bits(X), wl.f32_to_bf16_bits(W)
        dt = wl.BF16 if bf16 else wl.F32
        resume, u_cap = None, 0
        if do_resume:
            nr = int(rng.integers(1, max(2, min(n, 3000))))
            r_ids = np.sort(rng.choice(n, size=nr, replace=False)).astype(np.int32)
            r_G = rng.standard_normal((nr, d)).astype(np.float32)
            if pad_id >= 0:
                r_G[r_ids == pad_id] = 0.0
            resume = (r_ids, rng.integers(1, 9, size=nr).astype(np.int64), r_G)
            if not dense:
                u_cap = min(n, K * max(ms) + nr)
        cap = n if dense else min(n, K * max(ms) + (resume[0].size if resume else 0))
        cuts = np.unique(np.concatenate([[0], rng.integers(0, cap + 1, size=int(rng.integers(0, 5)))]))
        chunks = [(int(a), int(b - a)) for a, b in zip(cuts[:-1], cuts[1:])] + [(int(cuts[-1]), 10 ** 9)]
        out = run_window(X, W, batches, vocab_n=n, pad_id=pad_id, k_steps=K, max_positions=max(ms), pseudo=True,
                         wgrad_chunks=chunks, dense=dense, resume=resume, u_total_cap=u_cap)
        acc = orc.GramMulti(X, W, pad_id=pad_id)
        if resume is not None:
            acc.resume(*resume)
        for k, (ids, dH) in enumerate(batches):
            ref = acc.step(ids, dH)
            st = out["steps"][k]
            check_step_exact(st, ref)
            assert_close(st["E"], ref["E"], TOL_SUM[dt], f"E step {k}")
            assert_close(st["H"], ref["H"], TOL_SUM[dt], f"H step {k}")
            Ht_ref, loss_ref = orc.pseudo_target(ref["E"], acc.rows(ref["uniq"]))
            assert_close(st["Ht"], Ht_ref, TOL_SUM[dt], f"Ht step {k}")
            assert abs(st["loss"] - loss_ref) <= TOL_SUM[dt] * max(loss_ref, 1e-30)
            assert st["Ht_tail_untouched"]
            np.testing.assert_array_equal(st["H_tilde"], st["Ht"][ref["inverse"]])
        ref = acc.finish()
        np.testing.assert_array_equal(out["uniq_total"], ref["uniq"])
        np.testing.assert_array_equal(out["counts_total"], ref["counts"])
        assert_close(out["G_total"], ref["G"], TOL_SUM[dt], "G_total")
        if np.abs(ref["dW"]).max() > 0:
            assert_close(out["dW"], ref["dW"], TOL[dt], "dW")
            assert_close(out["dW_chunked"], ref["dW"], TOL[dt], "dW in chunks")
        out["gram"].close()


def test_randomly_drawn_steps_of_the_two_layer_encoder():
    """40 single-step windows of the two-layer encoder with random widths and batch sizes, the
    backward pass in a random partition of the items; from accumulated gradient rows (against the
    oracle's per-item run) or towards stored targets at moved weights (against the oracle's
    regression)."""
    for seed in range(40):
        rng = np.random.default_rng(20_000 + seed)
        n = int(2 ** rng.uniform(4, 16.5))
        d_in = int(rng.choice([8, 16, 32, 64, 96, 128, 264]))
        d_hid = int(rng.choice([8, 16, 40, 64, 128, 256, 264, 512]))
        d = int(rng.choice([8, 16, 24, 64, 128, 256, 264]))
        big = rng.random() < 0.3
        m_hi = 100000 if big else 8000
        m = max(2, int(2 ** rng.uniform(np.log2(m_hi) - 3 if big else 2, np.log2(m_hi))))
        while m * (d_in * d_hid + d_hid * d) > 1.5e9:
            m //= 2
        regress = rng.random() < 0.4
        s = float(rng.choice([0.0, 1.0]))
        say("random two-layer step:", dict(seed=seed, n=n, d_in=d_in, d_hid=d_hid, d=d, m=m, regress=regress))
        X, W1, W2 = mlp_weights(20_000 + seed, n, d_in, d_hid, d)
        p = np.arange(1, n + 1, dtype=np.float64) ** (-s)
        p /= p.sum()
        ids = rng.permutation(n)[rng.choice(n, size=m, p=p)].astype(np.int32)
        ids[rng.random(m) < 0.1] = 0
        dH = rng.standard_normal((m, d)).astype(np.float32)
        uniq = np.unique(ids)
        U = uniq.size
        cuts = np.unique(np.concatenate([[0, U], rng.integers(0, U + 1, size=int(rng.integers(0, 4)))]))
        parts = [int(b - a) for a, b in zip(cuts[:-1], cuts[1:])]
        if regress:
            _, V1, V2 = mlp_weights(30_000 + seed, n, d_in, d_hid, d)
            Ht = rng.standard_normal((U, d)).astype(np.float32)
            out = run_mlp_step(X, W1, W2, ids, dH, n, parts, targets=Ht, W_now=(V1, V2))
            miss, loss, dW1, dW2 = orc.mlp_pseudo_loss_grad(uniq, X, V1, V2, Ht.astype(np.float64))
            assert abs(sum(out["losses"]) - loss) <= TOL[wl.BF16] * loss
            assert_close(out["dW1"], dW1, TOL[wl.BF16], "dW1")
            assert_close(out["dW2"], dW2, TOL[wl.BF16], "dW2")
        else:
            out = run_mlp_step(X, W1, W2, ids, dH, n, parts)
            ref = orc.mlp_gram_single(ids, X, W1, W2, dH)
            np.testing.assert_array_equal(out["uniq"], ref["uniq"])
            np.testing.assert_array_equal(out["inverse"], ref["inverse"])
            assert out["A1_tail_untouched"]
            assert_close(out["A1"], ref["A1"], 2.0 ** -8, "A1 (kept in bf16)")
            assert_close(out["E"], ref["E"], TOL[wl.BF16], "E")
            np.testing.assert_array_equal(out["H"], out["E"][out["inverse"]])
            assert_close(out["G"], ref["G"], TOL_SUM[wl.BF16], "G")
            assert_close(out["dW1"], ref["dW1"], TOL[wl.BF16], "dW1")
            assert_close(out["dW2"], ref["dW2"], TOL[wl.BF16], "dW2")

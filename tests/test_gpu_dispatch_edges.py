"""Sizes at which a kernel of the path changes its form or its tiles end: one small parametrised test per such place,
against the fp64 oracle with the bars of test_gpu_parity."""
import numpy as np
import pytest

from paper_2605_24584_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import dev  # noqa: E402


@pytest.mark.parametrize("k,n,gap", [
    (1, 2046, 0.01), (1, 2047, 0.01), (1, 2048, 0.01), (7, 4089, 0.01), (2049, 2047, 0.01),      # around one and two tiles of 2048
    (6000, 9, 40.0), (4097, 2, 40.0),                                     # tiles of Gram anchors alone, entries far from every middle anchor
    (40, (1 << 22) - 40, 1e-4), (40, (1 << 22) - 39, 1e-4),                 # 2048 tiles: the last size without the spine kernel, and the next
    (3000, (1 << 22) + 5, 1e-4),
])
def test_weighted_gram_tile_edges(oracle, k, n, gap):
    """fp64 weights of one sign, |err| <= 1e-12 T: T_ij is the entry itself, so an entry that is exp(-2 * distance) of the
    nearest middle anchor, down to 1e-300, has to come from a difference of prefix sums that is exactly zero where nothing
    lies between the two anchors.  (Terms carry a few fp64 roundings each: decays are exp of exact anchor differences, sums
    of a tile are trees of depth 8 + 6 + 2, at most 2048 tiles in runs of 8: below 1e-13 relative.)"""
    r = np.random.default_rng(k + n)
    b = np.sort(r.integers(0, n, n)).astype(np.float64) * gap
    a = np.where(r.random(k) < 0.5, b[r.integers(0, n, k)], b[r.integers(0, n, k)] + gap * r.integers(0, 4, k))
    a, b = a.astype(np.float32), r.permutation(b).astype(np.float32)
    d = np.abs(r.normal(size=n)) + 0.5
    ref, tol = oracle.wgram_scan(a, b, d)
    ws = torch.empty(B.laplex_wgram_f64_workspace_bytes(k, n), dtype=torch.uint8, device="cuda")
    m = torch.full((k, k), float("nan"), dtype=torch.float64, device="cuda")
    B.laplex_wgram_f64(dev(a), dev(b), dev(d), m, ws, 0)
    torch.cuda.synchronize()
    got = m.cpu().numpy()
    assert np.all(np.isfinite(got)) and np.array_equal(got, got.T)
    assert float((np.abs(got - ref) / (1e-12 * tol + 1e-300)).max()) <= 1.0


SAMPLE_SORT_SIZES = [8193, 9217, (1 << 17) - 1, 1 << 17, (1 << 17) + 1, 1 << 18, (1 << 18) + 1, 1 << 19, (1 << 19) + 1]


def sorted_ids(keys_a, keys_b):
    """np's stable order of a ++ b, and the plan that the library builds for it (ids, and y of the product with ones)."""
    k, n = keys_a.size, keys_b.size
    ws = torch.empty(B.laplex_workspace_bytes(k, n, 1), dtype=torch.uint8, device="cuda")
    y = torch.empty(k, 1, device="cuda")
    B.laplex_apply(dev(keys_a), dev(keys_b), torch.ones(n, 1, device="cuda"), y, ws, 0)
    perm = torch.empty(k + n, dtype=torch.int32, device="cuda")
    B.laplex_get_perm(ws, k + n, perm)
    torch.cuda.synchronize()
    return perm.cpu().numpy(), y.cpu().numpy()


@pytest.mark.parametrize("kind", ["uniform", "few_values", "equal", "ascending", "repeating", "narrow_windows"])
@pytest.mark.parametrize("N", SAMPLE_SORT_SIZES)
def test_sample_sort_order_and_decays(oracle, N, kind):
    """The sort by samples at the ends of its first configurations.  `narrow_windows` takes, from every 1024 to 4096 consecutive positions, a
    few dozen neighbouring ones into one narrow window of the keys: dense bins in a stretch (stretches beyond the capacity:
    test_sample_sort_a_little_beyond_the_capacity and the one after it)."""
    r = np.random.default_rng(N)
    tile = 1024 if N <= 1 << 17 else 2048 if N <= 1 << 18 else 4096
    step = tile // 64
    if kind == "uniform":
        v = r.uniform(0, N / 64, N)
    elif kind == "few_values":
        v = r.integers(0, 37, N) * 0.25
    elif kind == "equal":
        v = np.zeros(N)
    elif kind == "ascending":
        v = np.arange(N) / 64.0
    elif kind == "repeating":
        v = (np.arange(N) % tile) * 0.5
    else:
        v = np.empty(N)
        for run in range((N + tile - 1) // tile):
            q = np.arange(tile)
            w = q / 8.0
            first = (run * 11) % step + 5 * step
            inside = (q > first) & (q < first + step)
            w[q <= first] = q[q <= first] * 0.01
            w[inside] = 50.0 + r.uniform(0, 1, step - 1)
            w[q >= first + step] += 60.0
            part = r.permutation(w)[: min(tile, N - run * tile)]
            v[run * tile: run * tile + part.size] = part
    v = v.astype(np.float32)
    k = N // 3
    ids, y = sorted_ids(v[:k], v[k:])
    assert np.array_equal(ids, np.argsort(v, kind="stable"))
    pick = r.integers(0, k, 200)                                  # decays: a few outputs against the definition
    a, b = v[:k][pick].astype(np.float64), v[k:].astype(np.float64)
    ref = np.exp(-np.abs(a[:, None] - b[None, :])).sum(axis=1)
    assert float((np.abs(y[pick, 0] - ref) / (1e-5 * ref + 1e-7)).max()) <= 1.0


@pytest.mark.parametrize("kind", ["uniform", "grid", "clusters", "wide", "ordered_blocks"])
@pytest.mark.parametrize("N", [(1 << 20) - 1, (1 << 20) + 1, 256 * 6144, 256 * 6144 + 1, 1 << 21, (1 << 21) + 1, 512 * 6144, 512 * 6144 + 1,
                               1 << 22, (1 << 22) + 1])
def test_sample_sort_order(N, kind):
    """The sort by samples where its tiles and the number of its stretches change; `wide` spreads keys over all exponents of both signs,
    `clusters` puts far more keys than bins allow into narrow windows, `ordered_blocks` makes a tile's share of a stretch very uneven."""
    r = np.random.default_rng(N)
    if kind == "uniform":
        v = r.uniform(0, N / 64, N)
    elif kind == "grid":
        v = np.round(r.uniform(0, N / 512, N) * 4) * 0.25
    elif kind == "clusters":
        v = r.integers(0, 1 + N // 3000, N) * 1000.0 + r.normal(size=N) * 1e-3
    elif kind == "wide":
        v = np.exp(r.uniform(-80, 80, N)) * r.choice([-1.0, 1.0], N)
    else:
        v = np.sort(r.uniform(0, N / 64, N))
        v = np.concatenate([v[i::3] for i in (1, 2, 0)])
    v = v.astype(np.float32)
    ids, _ = sorted_ids(v[:777], v[777:])
    assert np.array_equal(ids, np.argsort(v, kind="stable"))


@pytest.mark.parametrize("kind", ["few", "half", "equal", "nan"])
@pytest.mark.parametrize("N", [100003, 1 << 20, (1 << 21) + 5, 1 << 22])
def test_sample_sort_bounds_of_one_key(N, kind):
    """More anchors of a value than a stretch holds: many bounds share their key, at the first bound, in the middle and at the last one
    (`nan`: the largest key of all)."""
    r = np.random.default_rng(N)
    if kind == "few":
        v = r.integers(0, 31, N) * 0.25
    elif kind == "half":
        v = np.where(r.random(N) < 0.5, 3.0, r.uniform(0, N / 64, N))
    elif kind == "equal":
        v = np.full(N, -1.5)
    else:
        v = r.uniform(0, N / 64, N)
        v[r.random(N) < 0.25] = np.nan
    v = v.astype(np.float32)
    if kind == "nan":
        v.view(np.uint32)[np.isnan(v)] = 0x7FFFFFFF      # one payload: the key orders payloads, numpy does not
    ids, _ = sorted_ids(v[:777], v[777:])
    assert np.array_equal(ids, np.argsort(v, kind="stable"))


def sample_positions(N, samples):
    """Where the sort takes its samples from (sample_position in split_sort_kernels.hip)."""
    i = np.arange(samples, dtype=np.uint64)
    h = (i * 2654435761 + 40503) & 0xFFFFFFFF
    h ^= h >> 15; h = (h * 0x2C1B3C6D) & 0xFFFFFFFF; h ^= h >> 13
    width = N // samples
    at = (i * width + (h * width >> 32)).astype(np.int64)
    assert np.unique(at).size == samples and at.max() < N
    return at


@pytest.mark.parametrize("kind", ["uniform", "ties", "window"])
@pytest.mark.parametrize("over", [1, 500, 3000])
def test_sample_sort_a_little_beyond_the_capacity(kind, over):
    """An unlucky place of the samples leaves one stretch `over` pairs more than LDS holds (16384): sorted in memory, by one count or, where
    too many pairs share a bin (`window`), by digits."""
    N, buckets, per, cap = 600000, 256, 16, 16384
    r = np.random.default_rng(over)
    at = sample_positions(N, buckets * per)
    lo, hi = 100.0, 200.0                   # the stretch: keys in [lo, hi), its bounds among the samples
    inside = cap + over - per
    v = np.empty(N)
    s = np.empty(buckets * per)
    s[: 100 * per] = r.uniform(0, lo, 100 * per)
    s[100 * per: 101 * per] = np.linspace(lo, hi, per, endpoint=False)
    s[101 * per:] = np.r_[hi, r.uniform(hi, 900, buckets * per - 101 * per - 1)]
    rest = np.setdiff1d(np.arange(N), at)
    keys = np.empty(rest.size)
    keys[:inside] = r.uniform(lo, hi - 1e-3, inside) if kind != "window" else np.where(r.random(inside) < 0.6, 150.0, r.uniform(lo, hi - 1e-3, inside))
    keys[inside:] = np.where(r.random(rest.size - inside) < 0.1, r.uniform(0, lo - 1e-3, rest.size - inside), r.uniform(hi, 900, rest.size - inside))
    if kind == "ties":
        keys = np.floor(keys * 4) / 4
    v[rest], v[at] = r.permutation(keys), r.permutation(s)
    v = v.astype(np.float32)
    assert np.sum((v >= np.float32(lo)) & (v < np.float32(hi))) == cap + over
    ids, _ = sorted_ids(v[:777], v[777:])
    assert np.array_equal(ids, np.argsort(v, kind="stable"))


@pytest.mark.parametrize("ties", [False, True])
@pytest.mark.parametrize("N,samples", [(9000, 9 * 16), (200000, 98 * 16), (600000, 256 * 16)])
def test_sample_sort_beyond_the_capacity(oracle, N, samples, ties):
    """The positions that the sort takes its samples from hold the smallest keys: all others fall into the last stretch, which no
    workgroup's LDS holds."""
    r = np.random.default_rng(N + ties)
    at = sample_positions(N, samples)
    v = r.integers(50, 90, N) * 0.25 if ties else r.uniform(50, 50 + N / 64, N)
    v[at] = r.uniform(0, 40, samples)
    v = v.astype(np.float32)
    k = N // 3
    ids, y = sorted_ids(v[:k], v[k:])
    assert np.array_equal(ids, np.argsort(v, kind="stable"))
    ref, tol = oracle.apply_scan(v[:k], v[k:], np.ones((N - k, 1), np.float32))
    assert float((np.abs(y - ref) / (1e-5 * tol + 1e-7)).max()) <= 1.0


@pytest.mark.parametrize("k,n,batch,pad,shift", [
    (5000, 4000, 9, 0, 0), (5000, 4000, 10, 3, 0), (4100, 4100, 15, 0, 1), (9000, 33, 17, 0, 0), (33, 9000, 31, 1, 2), (6001, 3002, 33, 0, 0),
    (4000, 6000, 63, 0, 3), (4000, 6000, 65, 0, 0), (5000, 5000, 64, 1, 0), (5000, 5000, 12, 0, 1), (4500, 4500, 127, 0, 0), (4500, 4500, 128, 0, 2),
    (4500, 4500, 129, 0, 0), (70000, 62000, 65, 0, 0),                          # single columns again; a wavefront per tile, three spine launches
    (30000, 34000, 33, 0, 0),                                                   # 500 tiles that each read all others
    (2999, 100003, 33, 0, 0), (45000, 50000, 33, 2, 1), (100000, 110000, 13, 0, 0),    # more of them, in groups: two spine launches
    (40000, 31000, 64, 0, 0),                                                   # ... and rows that do allow it
])
def test_rows_that_allow_no_16_byte_access(oracle, k, n, batch, pad, shift):
    """Rows that start anywhere, of lengths that are no multiple of four: lanes of four columns whose last group ends with the row.  Forward,
    backward (scans saved and recomputed) and the square form; nothing beyond a row may be written or take part."""
    from test_gpu_parity import anchors, assert_close
    r = np.random.default_rng(k + 3 * n + batch + pad)
    a, b = anchors("ties", r, k, n)

    def matrix(values):           # columns beyond the batch hold NaN, rows start `shift` floats behind an allocation's start
        rows, ld = values.shape[0], batch + pad
        flat = torch.full((shift + rows * ld,), float("nan"), device="cuda")
        m = flat[shift:].view(rows, ld)
        m[:, :batch] = dev(values)
        return flat, m[:, :batch]

    x, g = r.normal(size=(n, batch)).astype(np.float32), r.normal(size=(k, batch)).astype(np.float32)
    ref, tol = oracle.apply_scan(a, b, x)
    want, tols = oracle.apply_backward_scan(a, b, x, g)
    (_, dx), (_, dg), (yf, y), (gxf, gx) = matrix(x), matrix(g), matrix(np.zeros_like(g)), matrix(np.zeros_like(x))
    da, db = dev(a), dev(b)
    ga, gb = torch.empty(k, device="cuda"), torch.empty(n, device="cuda")
    ws = torch.full((B.laplex_workspace_bytes(k, n, batch),), 255, dtype=torch.uint8, device="cuda")      # NaN wherever nothing is written
    for flags in (B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN, 0):
        B.laplex_apply(da, db, dx, y, ws, flags & ~B.LAPLEX_REUSE_PLAN)
        B.laplex_apply_backward(da, db, dx, dg, gx, ga, gb, ws, flags)
        torch.cuda.synchronize()
        assert_close("y", y.cpu().numpy(), ref, tol)
        for name, got, rv, tv in zip(("gx", "ga", "gb"), (gx, ga, gb), want, tols):
            assert_close(name, got.cpu().numpy(), rv, tv)
    if pad:
        assert torch.isnan(yf[shift:].view(k, batch + pad)[:, batch:]).all() and torch.isnan(gxf[shift:].view(n, batch + pad)[:, batch:]).all()
    wsg = torch.full((B.laplex_workspace_bytes(0, n, batch),), 255, dtype=torch.uint8, device="cuda")
    _, yg = matrix(np.zeros_like(x))
    B.laplex_gram(db, dx, yg, wsg, 0)
    torch.cuda.synchronize()
    ref, tol = oracle.apply_scan(b, b, x)
    assert_close("gram", yg.cpu().numpy(), ref, tol)


@pytest.mark.parametrize("kind", ["uniform", "ties"])
@pytest.mark.parametrize("N,batch", [(65 * 1024, 1), (255 * 1024, 1), (255 * 1024 + 1, 1), (255 * 2048 + 1, 1), (255 * 4096 + 1, 1), (255 * 512, 2), (255 * 512 + 1, 2), (255 * 256 + 1, 3),
                                     (255 * 128, 7), (255 * 128 + 1, 5),
                                     (127 * 256, 3), (127 * 256 + 1, 3), (127 * 512 + 1, 3), (79 * 128, 7), (79 * 128 + 1, 5), (79 * 256 + 1, 6), (79 * 512, 5),
                                     (79 * 512 + 1, 7)])
def test_narrow_batches_where_their_blocks_grow(oracle, N, batch, kind):
    """Single columns, up to 8 of them: blocks of one, two, four and eight wavefronts, at the sizes where they change."""
    from test_gpu_parity import anchors, assert_close, gpu_apply, gpu_backward
    r = np.random.default_rng(N + batch)
    k = N // 3
    a, b = anchors(kind, r, k, N - k)
    x, g = r.normal(size=(N - k, batch)).astype(np.float32), r.normal(size=(k, batch)).astype(np.float32)
    ref, tol = oracle.apply_scan(a, b, x)
    want, tols = oracle.apply_backward_scan(a, b, x, g)
    y, ws = gpu_apply(a, b, x, flags=B.LAPLEX_SAVE_SCANS)
    assert_close("y", y, ref, tol)
    for name, got, rv, tv in zip(("gx", "ga", "gb"), gpu_backward(a, b, x, g, flags=B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN, ws=ws), want, tols):
        assert_close(name, got, rv, tv)


def families(call):
    """The kernel families that the call launches, and how often."""
    B.laplex_profile_begin("*")
    call()
    B.laplex_profile_end()
    return {name: launches for name, (_, launches) in B.laplex_profile_families().items()}


@pytest.mark.parametrize("k,n,batch", [(64, 255 * 4096 - 64, 1), (1, 9000, 1), (50, 120000, 2), (64, 250000, 3), (10000, 4, 3), (100000, 40, 7), (16, 30000, 5), (20, 500000, 7),
                                       ((1 << 21) - 1, 1, 2)])
def test_few_rows_on_one_side_visit_every_short_block(oracle, k, n, batch):
    """Narrow batches of single columns, a handful of inputs or outputs, up to 512 blocks: none is listed by a launch of its own."""
    from test_gpu_parity import anchors, assert_close
    r = np.random.default_rng(k + n + batch)
    a, b = anchors("uniform", r, k, n)
    x, g = r.normal(size=(n, batch)).astype(np.float32), r.normal(size=(k, batch)).astype(np.float32)
    ref, tol = oracle.apply_scan(a, b, x)
    want, tols = oracle.apply_backward_scan(a, b, x, g)
    da, db, dx, dg = dev(a), dev(b), dev(x), dev(g)
    y, gx, ga, gb = torch.empty_like(dg), torch.empty_like(dx), torch.empty_like(da), torch.empty_like(db)
    ws = torch.empty(B.laplex_workspace_bytes(k, n, batch), dtype=torch.uint8, device="cuda")

    def step():
        B.laplex_apply(da, db, dx, y, ws, B.LAPLEX_SAVE_SCANS)
        B.laplex_apply_backward(da, db, dx, dg, gx, ga, gb, ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
    seen = families(step)
    assert seen["scan_reduce.fwd"] == seen["scan_reduce.bwd"] == 1
    assert not any(name.startswith(("scan_meta", "scan_down_sparse")) for name in seen), seen
    assert_close("y", y.cpu().numpy(), ref, tol)
    for name, got, rv, tv in zip(("gx", "ga", "gb"), (gx, ga, gb), want, tols):
        assert_close(name, got.cpu().numpy(), rv, tv)


@pytest.mark.parametrize("kind", ["uniform", "ties", "all_equal", "clustered"])
@pytest.mark.parametrize("k,n,batch,one", [(4096, 4097, 8, True), (98304, 98304, 8, True), (98304, 98305, 8, False), (4096, 4097, 64, True), (12285, 12291, 64, True), (9001, 3000, 33, True),
                                           (5000, 3200, 13, True), (393216, 393216, 1, True), (393216, 393217, 1, False), (4096, 4097, 1, True), (150000, 5000, 3, True), (20000, 21000, 5, True),
                                           (4097, 4096, 65, True), (4500, 4501, 97, True), (6144, 6144, 128, True), (6144, 6145, 128, False),
                                           (0, 98303, 8, True), (0, 20001, 1, True), (0, 9001, 64, True), (0, 12001, 33, True), (0, 9002, 128, True)])
def test_scans_in_one_launch(oracle, k, n, batch, one, kind):
    """Few blocks: they publish their summaries and add up each other's in the launch that scans, at both ends of that range (768 wavefronts); and
    again with no wait for the others, whose summaries every block then forms itself: the same bits (k = 0: the Gram form, whose backward is not one launch beyond 8 columns)."""
    from test_gpu_parity import anchors, assert_close
    r = np.random.default_rng(k + n + batch)
    a, b = anchors(kind, r, k or n, n)
    x, g = r.normal(size=(n, batch)).astype(np.float32), r.normal(size=(k or n, batch)).astype(np.float32)
    if k:
        ref, tol = oracle.apply_scan(a, b, x)
        want, tols = oracle.apply_backward_scan(a, b, x, g)
    else:
        ref, tol = oracle.gram_scan(a, x)
        want, tols = oracle.gram_backward_scan(a, x, g)
    da, db, dx, dg = dev(a), dev(b), dev(x), dev(g)
    y, gx, ga, gb = torch.empty_like(dg), torch.empty_like(dx), torch.empty_like(da), torch.empty_like(db)
    ws = torch.empty(B.laplex_workspace_bytes(k, n, batch), dtype=torch.uint8, device="cuda")

    def step(flags):
        if k:
            B.laplex_apply(da, db, dx, y, ws, flags | B.LAPLEX_SAVE_SCANS)
            B.laplex_apply_backward(da, db, dx, dg, gx, ga, gb, ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
        else:
            B.laplex_gram(da, dx, y, ws, flags | B.LAPLEX_SAVE_SCANS)
            B.laplex_gram_backward(da, dx, dg, gx, ga, ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
        torch.cuda.synchronize()

    def check():
        assert_close("y", y.cpu().numpy(), ref, tol)
        for name, got, rv, tv in zip(("gx", "ga", "gb"), (gx, ga, gb), want, tols):
            assert_close(name, got.cpu().numpy(), rv, tv)
    step(0)
    check()
    seen = families(lambda: step(B.LAPLEX_REUSE_PLAN))
    launches = {name for name in seen if name.startswith(("scan_spine", "scan_down"))}
    assert any(name.endswith(".fwd") for name in launches) == (not one), seen
    assert any(name.endswith(".bwd") for name in launches) == (not one or (k == 0 and batch > 8)), seen
    waited = [v.clone() for v in (y, gx, ga, gb)]
    B.laplex_diag_set_wait_limit(ws, k + n, 0)
    step(B.LAPLEX_REUSE_PLAN)
    check()
    assert all(torch.equal(v, w) for v, w in zip((y, gx, ga, gb) if k else (y, gx, ga), waited))


def masked_stream(units):
    """A stream whose workgroups run on the device's first `units` compute units, and what destroys it."""
    import ctypes
    with open("/proc/self/maps") as maps:
        path = next(line.split()[-1] for line in maps if "libamdhip64" in line)
    hip = ctypes.CDLL(path)
    words = (ctypes.c_uint32 * 8)(*[0xFFFFFFFF if 32 * (i + 1) <= units else (1 << max(units - 32 * i, 0)) - 1 for i in range(8)])
    stream = ctypes.c_void_p()
    assert hip.hipExtStreamCreateWithCUMask(ctypes.byref(stream), 8, words) == 0
    return stream.value, lambda: hip.hipStreamDestroy(stream)


@pytest.mark.parametrize("units,k,n,batch,one", [(256, 98304, 98304, 8, True), (64, 24576, 24576, 8, True), (64, 24576, 24577, 8, False), (40, 49152, 12288, 1, True), (40, 393216, 393216, 1, False),
                                                 (32, 4096, 4097, 64, False)])
def test_scans_in_one_launch_fit_the_stream(oracle, units, k, n, batch, one):
    """Blocks that wait for each other are no more than the compute units of the stream hold: three wavefronts for each."""
    from test_gpu_parity import anchors, assert_close
    r = np.random.default_rng(k + n + units)
    a, b = anchors("uniform", r, k, n)
    x = r.normal(size=(n, batch)).astype(np.float32)
    ref, tol = oracle.apply_scan(a, b, x)
    da, db, dx, y = dev(a), dev(b), dev(x), torch.empty(k, batch, device="cuda")
    ws = torch.empty(B.laplex_workspace_bytes(k, n, batch), dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    stream, destroy = masked_stream(units)
    try:
        seen = families(lambda: B.laplex_apply(da, db, dx, y, ws, 0, stream=stream))
        torch.cuda.synchronize()
    finally:
        destroy()
    assert_close("y", y.cpu().numpy(), ref, tol)
    assert any(name.startswith(("scan_spine", "scan_down")) for name in seen) == (not one), seen


@pytest.mark.parametrize("kind", ["uniform", "ties", "all_equal"])
@pytest.mark.parametrize("k,n,batch", [(70000, 70001, 33), (66000, 66000, 64), (40000, 30001, 100), (33000, 33001, 127), (300000, 240001, 13), (64, 140000, 64), (140000, 33, 48), (0, 132001, 48)])
def test_reduce_with_a_wavefront_per_tile(oracle, k, n, batch, kind):
    """More than 1024 tiles of up to 128 columns: their summaries are weighted sums of the injected rows, which are packed first (k = 0: the Gram form)."""
    from test_gpu_parity import anchors, assert_close
    r = np.random.default_rng(k + n + batch)
    a, b = anchors(kind, r, k or n, n)
    x = r.normal(size=(n, batch)).astype(np.float32)
    ref, tol = oracle.apply_scan(a, b, x) if k else oracle.gram_scan(a, x)
    ws = torch.empty(B.laplex_workspace_bytes(k, n, batch), dtype=torch.uint8, device="cuda")
    y = torch.empty(k or n, batch, device="cuda")
    step = (lambda v: B.laplex_apply(dev(a), dev(b), dev(v), y, ws, B.LAPLEX_SAVE_SCANS)) if k else (lambda v: B.laplex_gram(dev(a), dev(v), y, ws, B.LAPLEX_SAVE_SCANS))
    step(x)
    torch.cuda.synchronize()
    assert_close("y", y.cpu().numpy(), ref, tol)
    bad = x.copy()                                   # one column of them: no other column changes, and that one has no finite element left
    bad[n // 3, batch - 1] = np.inf
    first = y.cpu().numpy()
    step(bad)
    torch.cuda.synchronize()
    got = y.cpu().numpy()
    assert np.array_equal(got[:, : batch - 1], first[:, : batch - 1]) and not np.isfinite(got[:, batch - 1]).any()


@pytest.mark.parametrize("kind", ["uniform", "ties", "all_equal", "huge_gaps", "clustered"])
@pytest.mark.parametrize("n,batch", [(8193, 64), (8305, 33), (9000, 36), (9100, 63), (12301, 48), (140000, 64)])
def test_gram_backward_on_the_matrix_cores(oracle, n, batch, kind):
    """33 to 64 columns: sixteen rows a wavefront, whole and partly filled blocks, rows that end on any boundary."""
    from test_gpu_parity import anchors, assert_close
    r = np.random.default_rng(n + batch)
    a, _ = anchors(kind, r, n, 1)
    x, g = r.normal(size=(n, batch)).astype(np.float32), r.normal(size=(n, batch)).astype(np.float32)
    (rgx, rga), (tgx, tga) = oracle.gram_backward_scan(a, x, g)
    ws = torch.empty(B.laplex_workspace_bytes(0, n, batch), dtype=torch.uint8, device="cuda")
    gx, ga = torch.full((n, batch), float("nan"), device="cuda"), torch.full((n,), float("nan"), device="cuda")
    seen = families(lambda: B.laplex_gram_backward(dev(a), dev(x), dev(g), gx, ga, ws, 0))
    torch.cuda.synchronize()
    assert seen["scan_down.bwd"] == 2, seen              # (the second launch is there for values that are not finite)
    assert_close("gx", gx.cpu().numpy(), rgx, tgx)
    assert_close("ga", ga.cpu().numpy(), rga, tga)


@pytest.mark.parametrize("where", ["x", "g", "both"])
@pytest.mark.parametrize("kind", ["ties", "uniform"])
def test_gram_backward_on_the_matrix_cores_leaves_what_is_not_finite_to_the_walks(kind, where):
    """64 columns against the same in two halves, which are walked: infinities and NaN reach the same elements, and rows tied with them stay finite."""
    from test_gpu_parity import anchors
    n, batch = 9001, 64
    r = np.random.default_rng(7)
    a, _ = anchors(kind, r, n, 1)
    x, g = r.normal(size=(n, batch)).astype(np.float32), r.normal(size=(n, batch)).astype(np.float32)
    for m in ([x] if where == "x" else [g] if where == "g" else [x, g]):
        m[n // 2, 3] = np.inf
        m[n // 5, 40] = -np.inf
        m[n // 7, 50] = np.nan

    def backward(cols):
        ws = torch.empty(B.laplex_workspace_bytes(0, n, cols.stop - cols.start), dtype=torch.uint8, device="cuda")
        xs, gs = dev(np.ascontiguousarray(x[:, cols])), dev(np.ascontiguousarray(g[:, cols]))
        gx, ga = torch.empty_like(xs), torch.empty(n, device="cuda")
        for _ in range(2):                               # (the word that asks for the walks is cleared in between)
            B.laplex_gram_backward(dev(a), xs, gs, gx, ga, ws, 0)
        torch.cuda.synchronize()
        return gx.cpu().numpy(), ga.cpu().numpy()
    gx, ga = backward(slice(0, 64))
    halves = [backward(slice(0, 32)), backward(slice(32, 64))]
    both = np.concatenate([h[0] for h in halves], axis=1)
    assert np.array_equal(np.isnan(gx), np.isnan(both)) and np.array_equal(np.isinf(gx), np.isinf(both))
    assert np.array_equal(np.isfinite(ga), np.isfinite(halves[0][1]) & np.isfinite(halves[1][1]))
    fine = np.isfinite(gx)
    assert np.allclose(gx[fine], both[fine], rtol=1e-4, atol=1e-4)


@pytest.mark.parametrize("k,n,batch,launches", [(30000, 34000, 33, 1), (2999, 100003, 33, 2), (45000, 50000, 33, 2), (100000, 110000, 13, 2), (70000, 62000, 65, 3),
                                                (1000, 40000, 33, 1), (40000, 31000, 64, 2), (1500, 82000, 40, 2), (900000, 600000, 8, 2)])
def test_spine_launches(k, n, batch, launches):
    """The cases of test_direct_spine and test_rows_that_allow_no_16_byte_access that are there for a form of the spine reach it."""
    a, b, x = (torch.rand(*shape, device="cuda") for shape in ((k,), (n,), (n, batch)))
    ws = torch.empty(B.laplex_workspace_bytes(k, n, batch), dtype=torch.uint8, device="cuda")
    seen = families(lambda: B.laplex_apply(a, b, x, torch.empty(k, batch, device="cuda"), ws))
    assert seen["scan_spine.fwd"] == launches, seen


@pytest.mark.parametrize("k,n,batch,in_order", [(9000, 9000, 8, True), (3000, 9000, 4, True), (2999, 9001, 4, False), (1000, 100000, 8, False),
                                                (9000, 9000, 1, True), (1 << 18, 1 << 18, 1, True), (1 << 18, (1 << 18) + 1, 1, False), (9000, 9000, 3, False), (7000, 6000, 7, False)])
def test_which_strict_scans_wait_in_the_sorted_order(k, n, batch, in_order):
    """Where they do, the backward's reduce forms ga and no launch for the row products follows."""
    r = np.random.default_rng(k + n + batch)
    normal = lambda *shape: dev(r.normal(size=shape).astype(np.float32))
    a, b, x, g = normal(k), normal(n), normal(n, batch), normal(k, batch)
    ws = torch.empty(B.laplex_workspace_bytes(k, n, batch), dtype=torch.uint8, device="cuda")
    B.laplex_apply(a, b, x, torch.empty_like(g), ws, B.LAPLEX_SAVE_SCANS)
    gx, ga, gb = torch.empty_like(x), torch.empty_like(a), torch.empty_like(b)
    seen = families(lambda: B.laplex_apply_backward(a, b, x, g, gx, ga, gb, ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN))
    assert ("rowdot" not in seen) == in_order, seen


@pytest.mark.parametrize("wanted", [("ga",), ("gx", "ga", "gb")])
@pytest.mark.parametrize("pads", [(0, 0, 1), (1, 1, 0), (0, 1, 1), (1, 0, 0), (1, 1, 1)])
@pytest.mark.parametrize("k,n,batch", [(9000, 9000, 8), (5000, 15000, 4), (9000, 20, 8), (9000, 9000, 1), (100, 9000, 1)])
def test_strict_scans_of_rows_that_allow_no_16_byte_access(oracle, k, n, batch, pads, wanted):
    """x, y and gy each with rows on 16-byte boundaries or not: the order that the forward kept its strict scans in is the one the backward reads."""
    from test_gpu_parity import anchors, assert_close
    r = np.random.default_rng(k + n + batch)
    a, b = anchors("ties", r, k, n)
    x, g = r.normal(size=(n, batch)).astype(np.float32), r.normal(size=(k, batch)).astype(np.float32)
    want, tols = oracle.apply_backward_scan(a, b, x, g)
    padded = lambda v, pad: dev(np.pad(v, ((0, 0), (0, pad))))[:, :batch]
    da, db, dx, dy, dg = dev(a), dev(b), padded(x, pads[0]), padded(np.zeros_like(g), pads[1]), padded(g, pads[2])
    out = {"gx": torch.empty(n, batch, device="cuda"), "ga": torch.empty(k, device="cuda"), "gb": torch.empty(n, device="cuda")}
    pick = lambda: (out[v] if v in wanted else None for v in ("gx", "ga", "gb"))
    ws = torch.full((B.laplex_workspace_bytes(k, n, batch),), 255, dtype=torch.uint8, device="cuda")      # NaN wherever nothing is written

    def check():
        torch.cuda.synchronize()
        for name, ref, tol in zip(("gx", "ga", "gb"), want, tols):
            if name in wanted:
                assert_close(name, out[name].cpu().numpy(), ref, tol)
                out[name].fill_(float("nan"))

    B.laplex_apply(da, db, dx, dy, ws, B.LAPLEX_SAVE_SCANS)
    B.laplex_apply_backward(da, db, dx, dg, *pick(), ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
    check()
    B.laplex_apply_backward(da, db, dev(x), dg, *pick(), ws, B.LAPLEX_REUSE_PLAN)      # the strict scans once more, of rows that allow it
    check()
    B.laplex_apply(da, db, dx, dy, ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
    B.laplex_apply_backward(da, db, dx, dg, *pick(), ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
    check()


@pytest.mark.parametrize("saved", [True, False])
@pytest.mark.parametrize("wanted", [("ga",), ("gx", "ga"), ("ga", "gb"), ("gx", "ga", "gb")])
@pytest.mark.parametrize("k,n,batch,pad", [(9000, 3, 8, 0), (5, 9000, 1, 0), (7000, 6000, 3, 2), (6001, 5002, 7, 0), (4097, 8000, 4, 1), (9000, 9000, 2, 0),
                                           (7000, 6000, 12, 0), (100, 9000, 33, 0), (6000, 5000, 33, 1), (5000, 4000, 64, 0), (140000, 130000, 16, 0),
                                           (3000, 9000, 8, 0), (2999, 9001, 8, 0), (3000, 9000, 4, 0), (2999, 9001, 4, 1), (6000, 6000, 8, 1), (6000, 6000, 4, 3)])
def test_where_the_anchor_gradient_of_the_outputs_is_formed(oracle, k, n, batch, pad, wanted, saved):
    """Outside the small path: with 4 or 8 columns and a quarter of the rows or more outputs, ga comes from strict scans that wait in the
    sorted order, formed where gy is gathered (or, when nothing else is wanted or gy allows no 16-byte accesses, on its own); otherwise from
    the caller's order, beyond 8 columns in a workgroup's or a wavefront's reduce.  Beside every subset of the other gradients, with ties and
    padded rows."""
    from test_gpu_parity import anchors, assert_close
    r = np.random.default_rng(k + 3 * n + batch)
    a, b = anchors("ties", r, k, n)
    x, g = r.normal(size=(n, batch)).astype(np.float32), r.normal(size=(k, batch)).astype(np.float32)
    want, tols = oracle.apply_backward_scan(a, b, x, g)
    padded = lambda v: dev(np.pad(v, ((0, 0), (0, pad))))[:, :batch]
    da, db, dx, dg = dev(a), dev(b), padded(x), padded(g)
    out = {"gx": torch.empty(n, batch + pad, device="cuda")[:, :batch], "ga": torch.empty(k, device="cuda"), "gb": torch.empty(n, device="cuda")}
    ws = torch.full((B.laplex_workspace_bytes(k, n, batch),), 255, dtype=torch.uint8, device="cuda")      # NaN wherever nothing is written
    flags = 0
    if saved:
        B.laplex_apply(da, db, dx, torch.empty(k, batch, device="cuda"), ws, B.LAPLEX_SAVE_SCANS)
        flags = B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN
    B.laplex_apply_backward(da, db, dx, dg, *(out[v] if v in wanted else None for v in ("gx", "ga", "gb")), ws, flags)
    torch.cuda.synchronize()
    for name, ref, tol in zip(("gx", "ga", "gb"), want, tols):
        if name in wanted:
            assert_close(name, out[name].cpu().numpy(), ref, tol)


@pytest.mark.parametrize("kind", ["uniform", "ties", "all_equal", "clustered"])
@pytest.mark.parametrize("k,n,batch", [
    (1, 510, 1), (1, 511, 1), (256, 257, 2), (700, 323, 1), (701, 324, 3), (3000, 5192, 1), (1, 8191, 2),      # chunks of 512 rows
    (4096, 4096, 17), (4000, 4191, 30),                                          # chunks of 1024
    (513, 1024, 64), (4096, 4096, 50), (2047, 2, 100),                           # chunks of 512, four columns a workgroup
    (300, 212, 1000), (4096, 4096, 100), (128, 129, 2100),                       # chunks of 256, sixteen columns
])
def test_small_problem_chunks(oracle, kind, k, n, batch):
    """One-launch scans of small problems at the edges of their chunks, in each of the launch's four forms, forward and both
    backward forms (the strict scans saved, and recomputed beside the other problem); bars of test_gpu_parity."""
    from test_gpu_parity import anchors, assert_close, gpu_apply, gpu_backward
    r = np.random.default_rng(k + 5 * n + batch)
    a, b = anchors(kind, r, k, n)
    x, g = r.normal(size=(n, batch)).astype(np.float32), r.normal(size=(k, batch)).astype(np.float32)
    ref, tol = oracle.apply_scan(a, b, x)
    want, tols = oracle.apply_backward_scan(a, b, x, g)
    y, ws = gpu_apply(a, b, x, flags=B.LAPLEX_SAVE_SCANS)
    assert_close("y", y, ref, tol)
    saved = gpu_backward(a, b, x, g, flags=B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN, ws=ws)
    alone = gpu_backward(a, b, x, g)
    for name, u, v, rv, tv in zip(("gx", "ga", "gb"), saved, alone, want, tols):
        assert_close(name, u, rv, tv)
        assert_close(name, v, rv, tv)


@pytest.mark.parametrize("k,n,batch", [
    (4096, 4096, 133), (4096, 4096, 134), (8191, 1, 136), (1, 8191, 139), (7, 7000, 300),         # 3.5e7 values read by the chunks of 256 rows
    (2000, 2096, 520), (2000, 2096, 560), (300, 213, 22800), (300, 213, 40000), (3, 253, 140000),  # (the last: one chunk, always small)
])
def test_small_problems_with_wide_batches(oracle, k, n, batch):
    """Either side of the line from which problems of at most 8192 positions take the tiled scans: the permutation, both directions
    with and without a kept plan, a false promise of sorted anchors (small problems make no use of it); bars of test_gpu_parity."""
    from test_gpu_parity import anchors, assert_close, gpu_apply, gpu_backward, gpu_perm, gpu_plan_status
    r = np.random.default_rng(k + 3 * n + batch)
    a, b = anchors("ties", r, k, n)
    x, g = r.normal(size=(n, batch)).astype(np.float32), r.normal(size=(k, batch)).astype(np.float32)
    ref, tol = oracle.apply_scan(a, b, x)
    want, tols = oracle.apply_backward_scan(a, b, x, g)
    y, ws = gpu_apply(a, b, x, flags=B.LAPLEX_SAVE_SCANS)
    assert_close("y", y, ref, tol)
    assert np.array_equal(gpu_perm(ws, k + n), oracle.merged_permutation(a, b)) and gpu_plan_status(ws, k + n) == 0
    saved = gpu_backward(a, b, x, g, flags=B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN, ws=ws)
    alone = gpu_backward(a, b, x, g, flags=B.LAPLEX_A_SORTED | B.LAPLEX_B_SORTED)
    for name, u, v, rv, tv in zip(("gx", "ga", "gb"), saved, alone, want, tols):
        assert_close(name, u, rv, tv)
        assert_close(name, v, rv, tv)


@pytest.mark.parametrize("n,batch", [(8192, 133), (8192, 134), (4001, 700)])
def test_small_gram_with_wide_batches(oracle, n, batch):
    from test_gpu_parity import anchors, assert_close, gpu_gram, gpu_gram_backward
    r = np.random.default_rng(n + batch)
    a, _ = anchors("ties", r, n, 1)
    x, g = (r.normal(size=(n, batch)).astype(np.float32) for _ in range(2))
    ref, tol = oracle.gram_scan(a, x)
    y, ws = gpu_gram(a, x, flags=B.LAPLEX_SAVE_SCANS)
    assert_close("y", y, ref, tol)
    want, tols = oracle.gram_backward_scan(a, x, g)
    for got in (gpu_gram_backward(a, x, g, flags=B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN, ws=ws), gpu_gram_backward(a, x, g, flags=B.LAPLEX_A_SORTED)):
        for name, u, rv, tv in zip(("gx", "ga"), got, want, tols):
            assert_close(name, u, rv, tv)


def test_mix_common_launches_non_finite_anchors(oracle):
    """Values are unspecified, but the calls end, and the workspace serves a clean problem afterwards."""
    from test_gpu_parity import anchors, assert_close
    q = np.random.default_rng(77)
    r, batch = 2, 8
    for k, n in ((7000, 3000), (3000, 7000)):
        x, g = dev(q.normal(size=(n, batch)).astype(np.float32)), dev(q.normal(size=(k, batch)).astype(np.float32))
        ws = torch.empty(B.laplex_mix_workspace_bytes(r, k, n, batch), dtype=torch.uint8, device="cuda")
        w = np.array([0.5, -2.0], dtype=np.float32)
        for bad in (True, False):
            ab = [anchors("ties", q, k, n) for _ in range(r)]
            a, b = np.stack([u for u, _ in ab]), np.stack([v for _, v in ab])
            if bad:
                a[0, ::50] = np.nan; a[1, ::7] = -np.nan; a[:, 3] = np.inf; a[:, 4] = -np.inf
                b[0, ::33] = -np.nan; b[1, ::11] = np.nan; b[:, 5] = np.inf; b[:, 6] = -np.inf
            out = [torch.zeros(*v, device="cuda") for v in ((k, batch), (n, batch), (r, k), (r, n), (r,))]
            B.laplex_mix_apply(dev(a), dev(b), dev(w), x, out[0], ws, B.LAPLEX_SAVE_SCANS)
            B.laplex_mix_apply_backward(dev(a), dev(b), dev(w), x, g, *out[1:], ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
            torch.cuda.synchronize()
        ref, tol = oracle.mix_apply(a, b, w, x.cpu().numpy(), brute=False)
        assert_close("y", out[0].cpu().numpy(), ref, tol)


@pytest.mark.parametrize("kind", ["uniform", "ties", "all_equal", "clustered"])
@pytest.mark.parametrize("r,k,n,batch,pad", [
    (2, 8192, 1, 4, 0), (2, 1, 8192, 5, 0), (3, 8000, 255, 32, 0), (2, 257, 8100, 36, 4), (2, 8191, 2049, 1, 0),
    (3, 4097, 4096, 3, 2), (2, 4096, 4097, 33, 1), (2, 6000, 3000, 100, 0), (1, 30000, 600, 8, 0), (2, 700, 20000, 64, 0),
    (2, 9000, 31, 16, 0), (1, 33, 9001, 2, 0),                    # hundreds of long rows between two short ones: several tasks each
    (2, 7000, 906, 64, 0), (2, 7000, 905, 64, 0), (16, 500, 898, 256, 0),       # from 8e9 / (r batch) = N^2 on: common launches
    (3, 6831, 1, 1, 0), (3, 1, 6832, 1, 0), (16, 1500, 1500, 1, 0),             # operators sorted in a workgroup each
    (5, 3000, 400, 1, 0), (5, 400, 3001, 1, 0), (17, 999, 1, 3, 0), (17, 1, 1000, 3, 0),      # r N = 17000, the last ones ranked by counting; the first sorted
])
def test_mix_common_launches(oracle, kind, r, k, n, batch, pad):
    """Sums of operators in common launches: either side the shorter one, one and several tiles of the short side (256
    rows with 4-column lanes, 64 to 2048 with single columns), odd batches, rows that allow no 16-byte access (pad), sorted
    anchors; bars of test_gpu_parity."""
    from test_gpu_parity import anchors, assert_close
    q = np.random.default_rng(k + 3 * n + batch)
    ab = [anchors(kind, q, k, n) for _ in range(r)]
    a, b = np.stack([u for u, _ in ab]), np.stack([v for _, v in ab])
    w = q.normal(size=r).astype(np.float32)
    x, g = q.normal(size=(n, batch)).astype(np.float32), q.normal(size=(k, batch)).astype(np.float32)
    padded = lambda rows: torch.full((rows, batch + pad), float("nan"), device="cuda")[:, :batch]
    dx, dg, y, gx = padded(n), padded(k), padded(k), padded(n)
    dx.copy_(dev(x)); dg.copy_(dev(g))
    new = lambda *s: torch.full(s, float("nan"), device="cuda")
    ws = torch.empty(B.laplex_mix_workspace_bytes(r, k, n, batch), dtype=torch.uint8, device="cuda")
    for step in range(2):
        da, db, dw = dev(a), dev(b), dev(w)
        ga, gb, gw = new(r, k), new(r, n), new(r)
        flags = 0 if step == 0 else B.LAPLEX_A_SORTED | B.LAPLEX_B_SORTED
        B.laplex_mix_apply(da, db, dw, dx, y, ws, flags | B.LAPLEX_SAVE_SCANS)
        B.laplex_mix_apply_backward(da, db, dw, dx, dg, gx, ga, gb, gw, ws, flags | B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
        torch.cuda.synchronize()
        ref, tol = oracle.mix_apply(a, b, w, x, brute=False)
        want, tols = oracle.mix_backward(a, b, w, x, g, brute=False)
        assert_close("y", y.cpu().numpy(), ref, tol)
        for name, got, rv, tv in zip(("gx", "ga", "gb", "gw"), (gx, ga, gb, gw), want, tols):
            assert_close(name, got.cpu().numpy(), rv, tv)
        for pick in ((0,), (1,), (2,), (3,), (1, 3)):             # the gradients one by one, the backward standing alone
            outs = [padded(n) if i == 0 else new(*s) for i, s in enumerate(((n,), (r, k), (r, n), (r,)))]
            outs = [v if i in pick else None for i, v in enumerate(outs)]
            B.laplex_mix_apply_backward(da, db, dw, None if pick == (0,) else dx, dg, *outs, ws, flags)
            torch.cuda.synchronize()
            for i in pick:
                assert_close(str(i), outs[i].cpu().numpy(), want[i], tols[i])
        a, b = np.sort(a, axis=1), np.sort(b, axis=1)             # second round: both sides ascending


@pytest.mark.parametrize("kind", ["uniform", "ties", "all_equal", "clustered"])
@pytest.mark.parametrize("k,n,batch", [
    (4000, 4200, 1), (9000, 7385, 1),                             # one and two tiles of 8192 rows, and a row more
    (65000, 66072, 8), (65000, 66073, 8),                         # 128 tiles of 1024 rows, and one more
    (32768, 32769, 32), (20, 60000, 8),                           # few outputs: the list of heavy blocks beside the sums
    (1000, 40000, 33), (700, 30000, 256),                         # a workgroup per tile: four row-lanes, one
    (900000, 600000, 8), (30, 140000, 256),                       # two levels: groups of 32 tiles, the last one shorter
    (40000, 31000, 64), (1500, 82000, 40),                        # ... four row-lanes, 555 and 653 tiles
])
def test_direct_spine(oracle, kind, k, n, batch):
    """The spine that adds the other tiles' summaries directly, at one tile, at the ends of its groups, with runs of equal keys that
    reach over tiles (all_equal: over all of them); bars of test_gpu_parity."""
    from test_gpu_parity import anchors, assert_close, gpu_apply, gpu_backward
    r = np.random.default_rng(k + 7 * n + batch)
    a, b = anchors(kind, r, k, n)
    x, g = r.normal(size=(n, batch)).astype(np.float32), r.normal(size=(k, batch)).astype(np.float32)
    ref, tol = oracle.apply_scan(a, b, x)
    want, tols = oracle.apply_backward_scan(a, b, x, g)
    y, ws = gpu_apply(a, b, x, flags=B.LAPLEX_SAVE_SCANS)
    assert_close("y", y, ref, tol)
    grads = gpu_backward(a, b, x, g, flags=B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN, ws=ws)
    for name, u, rv, tv in zip(("gx", "ga", "gb"), grads, want, tols):
        assert_close(name, u, rv, tv)


@pytest.mark.parametrize("r,k,n,batch", [(5, 40, 530000, 2), (2, 33000, 32769, 4), (2, 32768, 33000, 4)])
def test_mix_operator_by_operator(oracle, r, k, n, batch):
    """Sums of operators beyond the common launches (more than 2^19 merged positions, or 2^15 of either kind; the last case is the first
    within): operators on the library's streams, five of them in two rounds; bars of test_gpu_parity.  A captured call keeps to its
    stream and gives the same bits on every replay."""
    from test_gpu_parity import anchors, assert_close
    q = np.random.default_rng(r + k + n)
    ab = [anchors("ties", q, k, n) for _ in range(r)]
    a, b = np.stack([u for u, _ in ab]), np.stack([v for _, v in ab])
    w = q.normal(size=r).astype(np.float32)
    x, g = q.normal(size=(n, batch)).astype(np.float32), q.normal(size=(k, batch)).astype(np.float32)
    da, db, dw, dx, dg = dev(a), dev(b), dev(w), dev(x), dev(g)
    out = [torch.full(s, float("nan"), device="cuda") for s in ((k, batch), (n, batch), (r, k), (r, n), (r,))]
    ws = torch.empty(B.laplex_mix_workspace_bytes(r, k, n, batch), dtype=torch.uint8, device="cuda")

    def run():
        B.laplex_mix_apply(da, db, dw, dx, out[0], ws, B.LAPLEX_SAVE_SCANS)
        B.laplex_mix_apply_backward(da, db, dw, dx, dg, *out[1:], ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)

    run()
    torch.cuda.synchronize()
    eager = [v.clone() for v in out]
    ref, tol = oracle.mix_apply(a, b, w, x, brute=False)
    want, tols = oracle.mix_backward(a, b, w, x, g, brute=False)
    for name, got, rv, tv in zip(("y", "gx", "ga", "gb", "gw"), eager, (ref,) + tuple(want), (tol,) + tuple(tols)):
        assert_close(name, got.cpu().numpy(), rv, tv)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        run()
    for _ in range(3):
        for v in out:
            v.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(u, v) for u, v in zip(out, eager))


@pytest.mark.parametrize("k,n,batch", [(40, 120000, 8), (120000, 40, 5), (300, 70000, 64), (70000, 300, 33), (5, 100000, 1), (3, 9000, 256)])
@pytest.mark.parametrize("kind", ["apart", "uniform", "ties", "two_values"])
def test_mix_many_long_rows_between_two_short_ones(oracle, kind, k, n, batch):
    """Sums of operators whose long side has hundreds or thousands of rows between two short anchors, or all of them beyond the last
    one (apart), or equal to two of them: intervals of up to 3750 tasks; bars of test_gpu_parity."""
    from test_gpu_parity import anchors, assert_close
    q = np.random.default_rng(k + 3 * n + batch)
    r = 2
    if kind == "apart":
        ab = [(q.uniform(0, 1, k).astype(np.float32), q.uniform(2, 9, n).astype(np.float32)) for _ in range(r)]
    elif kind == "two_values":
        ab = [(q.integers(0, 4, k).astype(np.float32), q.integers(1, 3, n).astype(np.float32)) for _ in range(r)]
    else:
        ab = [anchors(kind, q, k, n) for _ in range(r)]
    a, b = np.stack([u for u, _ in ab]), np.stack([v for _, v in ab])
    w = q.normal(size=r).astype(np.float32)
    x, g = q.normal(size=(n, batch)).astype(np.float32), q.normal(size=(k, batch)).astype(np.float32)
    out = [torch.full(s, float("nan"), device="cuda") for s in ((k, batch), (n, batch), (r, k), (r, n), (r,))]
    ws = torch.empty(B.laplex_mix_workspace_bytes(r, k, n, batch), dtype=torch.uint8, device="cuda")
    da, db, dw, dx, dg = dev(a), dev(b), dev(w), dev(x), dev(g)
    B.laplex_mix_apply(da, db, dw, dx, out[0], ws, B.LAPLEX_SAVE_SCANS)
    B.laplex_mix_apply_backward(da, db, dw, dx, dg, *out[1:], ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
    torch.cuda.synchronize()
    ref, tol = oracle.mix_apply(a, b, w, x, brute=False)
    want, tols = oracle.mix_backward(a, b, w, x, g, brute=False)
    for name, got, rv, tv in zip(("y", "gx", "ga", "gb", "gw"), out, (ref,) + tuple(want), (tol,) + tuple(tols)):
        assert_close(name, got.cpu().numpy(), rv, tv)


@pytest.mark.parametrize("r,k,n,batch", [(2, 9000, 700, 8), (2, 700, 9000, 8), (2, 300, 400, 8), (2, 33000, 33000, 2)])
def test_mix_saved_scans_survive_a_call_that_does_not_save(oracle, r, k, n, batch):
    """forward(x, saving), forward(another x, not saving), backward(x, saved): gx, ga and gb are those of x.  (gw is formed from the
    operators' products, which every forward call writes.)"""
    from test_gpu_parity import anchors, assert_close
    q = np.random.default_rng(k + n)
    ab = [anchors("uniform", q, k, n) for _ in range(r)]
    a, b = np.stack([u for u, _ in ab]), np.stack([v for _, v in ab])
    w = q.normal(size=r).astype(np.float32)
    x, other = (q.normal(size=(n, batch)).astype(np.float32) for _ in range(2))
    g = q.normal(size=(k, batch)).astype(np.float32)
    out = [torch.full(s, float("nan"), device="cuda") for s in ((k, batch), (n, batch), (r, k), (r, n))]
    ws = torch.empty(B.laplex_mix_workspace_bytes(r, k, n, batch), dtype=torch.uint8, device="cuda")
    da, db, dw, dx, dg = dev(a), dev(b), dev(w), dev(x), dev(g)
    B.laplex_mix_apply(da, db, dw, dx, out[0], ws, B.LAPLEX_SAVE_SCANS)
    B.laplex_mix_apply(da, db, dw, dev(other), out[0], ws, B.LAPLEX_REUSE_PLAN)
    B.laplex_mix_apply_backward(da, db, dw, dx, dg, *out[1:], None, ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
    torch.cuda.synchronize()
    ref, tol = oracle.mix_apply(a, b, w, other, brute=False)
    want, tols = oracle.mix_backward(a, b, w, x, g, brute=False)
    for name, got, rv, tv in zip(("y", "gx", "ga", "gb"), out, (ref,) + tuple(want[:3]), (tol,) + tuple(tols[:3])):
        assert_close(name, got.cpu().numpy(), rv, tv)


@pytest.mark.parametrize("r,k,n,batch", [(3, 9000, 700, 8), (3, 700, 9000, 5), (4, 4000, 4000, 64), (3, 60000, 9000, 4), (2, 300, 400, 8)])
def test_mix_on_plans_that_other_calls_built(oracle, r, k, n, batch):
    """LAPLEX_REUSE_PLAN for a sum of operators whose plans, at their places in the workspace, come from calls on the single operators;
    then with one of them built anew on other anchors, and for a sum of fewer operators on the same workspace."""
    from test_gpu_parity import anchors, assert_close
    q = np.random.default_rng(k + n)
    ab = [anchors("ties", q, k, n) for _ in range(r + 1)]
    a, b = np.stack([u for u, _ in ab]), np.stack([v for _, v in ab])
    w = q.normal(size=r).astype(np.float32)
    x, g = q.normal(size=(n, batch)).astype(np.float32), q.normal(size=(k, batch)).astype(np.float32)
    da, db, dw, dx, dg = dev(a), dev(b), dev(w), dev(x), dev(g)
    ws = torch.empty(B.laplex_mix_workspace_bytes(r, k, n, batch), dtype=torch.uint8, device="cuda")
    one = (B.laplex_workspace_bytes(k, n, batch) + 255) // 256 * 256
    y = torch.empty(k, batch, device="cuda")

    def check(count):
        out = [torch.full(s, float("nan"), device="cuda") for s in ((k, batch), (n, batch), (count, k), (count, n), (count,))]
        B.laplex_mix_apply(da[:count], db[:count], dw[:count], dx, out[0], ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
        B.laplex_mix_apply_backward(da[:count], db[:count], dw[:count], dx, dg, *out[1:], ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
        torch.cuda.synchronize()
        ha, hb = da[:count].cpu().numpy(), db[:count].cpu().numpy()
        ref, tol = oracle.mix_apply(ha, hb, w[:count], x, brute=False)
        want, tols = oracle.mix_backward(ha, hb, w[:count], x, g, brute=False)
        for name, got, rv, tv in zip(("y", "gx", "ga", "gb", "gw"), out, (ref,) + tuple(want), (tol,) + tuple(tols)):
            assert_close(name, got.cpu().numpy(), rv, tv)

    for p in range(r):
        B.laplex_apply(da[p], db[p], dx, y, ws[p * one:], 0)
    check(r)
    da[1].copy_(da[r]); db[1].copy_(db[r])
    B.laplex_apply(da[1], db[1], dx, y, ws[one:], 0)
    check(r)
    check(r - 1)


@pytest.mark.parametrize("r,k,n,batch", [(2, 4000, 4000, 300), (2, 4000, 4000, 64), (2, 9000, 700, 8), (3, 700, 9000, 64), (2, 300, 400, 8), (1, 2000, 1500, 900)])
def test_plain_calls_on_the_plans_of_a_sum(oracle, r, k, n, batch):
    """The plans of a sum of operators, at their places in its workspace, serve calls on the single operators (whatever route those take), and
    the sum afterwards."""
    from test_gpu_parity import anchors, assert_close
    q = np.random.default_rng(k + n + batch)
    ab = [anchors("uniform", q, k, n) for _ in range(r)]
    a, b = np.stack([u for u, _ in ab]), np.stack([v for _, v in ab])
    w = q.normal(size=r).astype(np.float32)
    x, g = q.normal(size=(n, batch)).astype(np.float32), q.normal(size=(k, batch)).astype(np.float32)
    da, db, dw, dx, dg = dev(a), dev(b), dev(w), dev(x), dev(g)
    ws = torch.zeros(B.laplex_mix_workspace_bytes(r, k, n, batch), dtype=torch.uint8, device="cuda")
    one = (B.laplex_workspace_bytes(k, n, batch) + 255) // 256 * 256
    y, y1, gx = torch.empty(k, batch, device="cuda"), torch.empty(k, batch, device="cuda"), torch.empty(n, batch, device="cuda")
    B.laplex_mix_apply(da, db, dw, dx, y, ws, 0)
    for p in range(r):
        B.laplex_apply(da[p], db[p], dx, y1, ws[p * one:], B.LAPLEX_REUSE_PLAN)
        B.laplex_apply_backward(da[p], db[p], dx, dg, gx, None, None, ws[p * one:], B.LAPLEX_REUSE_PLAN)
        torch.cuda.synchronize()
        ref, tol = oracle.apply_scan(a[p], b[p], x)
        (rgx, _, _), (tgx, _, _) = oracle.apply_backward_scan(a[p], b[p], x, g)
        assert_close("y", y1.cpu().numpy(), ref, tol)
        assert_close("gx", gx.cpu().numpy(), rgx, tgx)
    B.laplex_mix_apply(da, db, dw, dx, y, ws, B.LAPLEX_REUSE_PLAN)
    torch.cuda.synchronize()
    ref, tol = oracle.mix_apply(a, b, w, x, brute=False)
    assert_close("y", y.cpu().numpy(), ref, tol)


def _deep_sample_positions(N):
    """Where the sort of many anchors at batch 1 takes its samples (deep_geom, deep_sample_position)."""
    stretches = min((N + 767) // 768, 1 << 20)
    buckets = 1
    while buckets * buckets < N // 3600: buckets += 1
    while buckets * 1024 < stretches: buckets += 1
    per = min((stretches + buckets - 1) // buckets, 1024)
    samples = buckets * per * min(6, (1 << 22) // (buckets * per))
    step = (N << 20) // samples
    at = []
    for i in range(samples):
        lo, hi = (i * step) >> 20, ((i + 1) * step) >> 20
        h = (i * 2654435761 + 40503) & 0xFFFFFFFF
        h ^= h >> 15; h = (h * 0x2C1B3C6D) & 0xFFFFFFFF; h ^= h >> 13
        at.append(lo + (h * (hi - lo) >> 32))
    return np.array(at)


@pytest.mark.parametrize("k,n,kind", [
    (1, 8192, "uniform"), (8192, 1, "ties"), (16384, 16384, "uniform"), (16383, 1, "all_equal"), (16385, 16384, "ascending"), (40000, 9152, "uniform"),
    (3, 65533, "clustered"), (131072, 8191, "ties"), (20000, 300001, "descending"), (150000, 150000, "two_values"),
    (30000, 41000, "unsampled"), (9000, 200000, "unsampled"),
])
@pytest.mark.parametrize("flags", [0, B.LAPLEX_A_SORTED | B.LAPLEX_B_SORTED])
def test_sort_in_two_distributions(oracle, k, n, kind, flags):
    """Batch 1 on the routes through sorted order at the edges of the sort's tiles and pieces, with the outputs ending inside a tile or with it; anchors of one and
    two values and in order; and anchors whose samples all miss the middle of the range, so that one stretch holds nearly everything (beyond a
    workgroup's LDS and, with more than 65536 pairs, beyond 16-bit places).  The permutation bit for bit, the values by the bars of test_gpu_parity."""
    from test_gpu_parity import anchors, assert_close, gpu_apply, gpu_backward, gpu_perm, gpu_plan_status
    N = k + n
    r = np.random.default_rng(N + len(kind))
    span = N / 64.0
    if kind in ("uniform", "ties", "all_equal", "clustered"):
        a, b = anchors(kind, r, k, n)
    else:
        v = r.uniform(0, span, N)
        if kind == "ascending": v = np.concatenate([np.sort(v[:k]), np.sort(v[k:])])
        if kind == "descending": v = -np.sort(-v)
        if kind == "two_values": v = np.where(v < span / 3, 1.0, 2.0)
        if kind == "unsampled":
            at = _deep_sample_positions(N)
            v = span * (0.25 + 0.5 * r.permutation(N) / N)
            v[at[::2]] = r.uniform(0, 0.2 * span, at[::2].size); v[at[1::2]] = r.uniform(0.8 * span, span, at[1::2].size)
        v = v.astype(np.float32)
        a, b = v[:k], v[k:]
    if flags and kind != "ascending":
        a, b = np.sort(a), np.sort(b)
    x, g = r.normal(size=(n, 1)).astype(np.float32), r.normal(size=(k, 1)).astype(np.float32)
    ref, tol = oracle.apply_scan(a, b, x)
    want, tols = oracle.apply_backward_scan(a, b, x, g)
    B.laplex_diag_set_route_min(0)
    try:
        y, ws = gpu_apply(a, b, x, flags=flags | B.LAPLEX_SAVE_SCANS)
        assert np.array_equal(gpu_perm(ws, N), oracle.merged_permutation(a, b)) and gpu_plan_status(ws, N) == 0
        assert_close("y", y, ref, tol)
        for got in (gpu_backward(a, b, x, g, flags=flags | B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN, ws=ws), gpu_backward(a, b, x, g, flags=flags)):
            for name, u, rv, tv in zip(("gx", "ga", "gb"), got, want, tols):
                assert_close(name, u, rv, tv)
    finally:
        B.laplex_diag_set_route_min(1 << 22)


def test_sort_in_two_distributions_non_finite_anchors(oracle):
    """Values are unspecified, but the calls end, and the workspace serves a clean problem afterwards."""
    from test_gpu_parity import anchors, assert_close, gpu_perm
    q = np.random.default_rng(5)
    k, n = 30000, 50000
    x = q.normal(size=(n, 1)).astype(np.float32)
    B.laplex_diag_set_route_min(0)
    try:
        ws = torch.empty(B.laplex_workspace_bytes(k, n, 1), dtype=torch.uint8, device="cuda")
        y = torch.zeros(k, 1, device="cuda")
        for bad in (3, 2, 1, 0):
            a, b = anchors("ties", q, k, n)
            if bad: a[::50 if bad > 1 else 1] = np.nan; b[::33] = -np.nan; a[3] = np.inf; b[5] = -np.inf
            if bad > 2: b[:] = np.inf
            B.laplex_apply(dev(a), dev(b), dev(x), y, ws, 0)
            torch.cuda.synchronize()
        assert np.array_equal(gpu_perm(ws, k + n), oracle.merged_permutation(a, b))
        ref, tol = oracle.apply_scan(a, b, x)
        assert_close("y", y.cpu().numpy(), ref, tol)
    finally:
        B.laplex_diag_set_route_min(1 << 22)


@pytest.mark.parametrize("k,n,batch", [
    (1, 1, 1), (16, 255, 1), (17, 257, 1), (4096, 4096, 1), (4100, 4092, 1), (5, 8187, 1), (8187, 5, 1),      # one column: the last two sizes of the line
    (16, 1023, 2), (15, 1024, 2), (2366, 2366, 2), (7, 1025, 4), (9, 3072, 3), (3073, 9, 3), (8, 2049, 8), (1793, 1792, 8), (1793, 1793, 8),
    (33, 70, 9), (600, 601, 16), (1024, 1024, 16), (100, 130, 70),                                            # several slabs
])
@pytest.mark.parametrize("tau", [1.0, 0.37])
def test_products_pair_by_pair(oracle, k, n, batch, tau):
    """Small problems either side of the lines up to which the products come straight from the anchors: tiles of result rows, stages of injected rows and
    slabs of columns that end anywhere, ties (also after the multiplication by tau), padded rows, gradients wanted one by one, saved or not; the
    same bits whether the plan is kept or not.  Bars of test_gpu_parity."""
    from test_gpu_parity import anchors, assert_close, gpu_perm
    r = np.random.default_rng(k + 3 * n + batch)
    a, b = anchors("ties", r, k, n)
    x, g = r.normal(size=(n, batch)).astype(np.float32), r.normal(size=(k, batch)).astype(np.float32)
    ref, tol = oracle.tau_apply(a, b, tau, x, brute=True)
    (rgx, rga, rgb, _), (tgx, tga, tgb, _) = oracle.tau_backward(a, b, tau, x, g, brute=True)
    da, db, dg = dev(a), dev(b), dev(g)
    dx = torch.zeros(n, batch + 3, device="cuda")[:, :batch]; dx.copy_(dev(x))
    ws = torch.empty(B.laplex_workspace_bytes(k, n, batch), dtype=torch.uint8, device="cuda")
    y = torch.full((k, batch + 1), float("nan"), device="cuda")
    B.laplex_apply_tau(da, db, tau, dx, y[:, :batch], ws, B.LAPLEX_SAVE_SCANS)
    torch.cuda.synchronize()
    assert_close("y", y[:, :batch].cpu().numpy(), ref, tol)
    assert bool(torch.isnan(y[:, batch]).all())
    scaled = np.float32(tau) * a, np.float32(tau) * b
    assert np.array_equal(gpu_perm(ws, k + n), oracle.merged_permutation(*scaled))
    y2 = torch.zeros(k, batch, device="cuda")
    B.laplex_apply_tau(da, db, tau, dx, y2, ws, B.LAPLEX_REUSE_PLAN)
    assert_close("y on a kept plan", y2.cpu().numpy(), ref, tol)
    first = None
    for flags in (B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN, 0):
        for want in ((1, 1, 1), (0, 1, 0), (1, 0, 0), (0, 0, 1), (1, 1, 0)):
            fresh = ws if flags else torch.empty_like(ws)
            gx = torch.full((n, batch + 2), float("nan"), device="cuda")[:, :batch] if want[0] else None
            ga = torch.full((k,), float("nan"), device="cuda") if want[1] else None
            gb = torch.full((n,), float("nan"), device="cuda") if want[2] else None
            B.laplex_apply_backward_tau(da, db, tau, dx, dg, gx, ga, gb, None, fresh, flags)
            torch.cuda.synchronize()
            got = [None if v is None else v.cpu().numpy() for v in (gx, ga, gb)]
            if first is None: first = got
            for name, v, rv, tv, f in zip(("gx", "ga", "gb"), got, (rgx, rga, rgb), (tgx, tga, tgb), first):
                if v is not None:
                    assert_close(name, v, rv, tv)
                    assert not all(want) or np.array_equal(v, f), name


@pytest.mark.parametrize("n,batch", [(1, 1), (4100, 1), (4096, 1), (2121, 4), (1792, 8), (300, 20)])
def test_gram_pair_by_pair(oracle, n, batch):
    from test_gpu_parity import anchors, assert_close, gpu_gram, gpu_gram_backward
    r = np.random.default_rng(n + batch)
    a, _ = anchors("ties", r, n, 1)
    x, g = (r.normal(size=(n, batch)).astype(np.float32) for _ in range(2))
    ref, tol = oracle.gram_brute(a, x)
    y, ws = gpu_gram(a, x, flags=B.LAPLEX_SAVE_SCANS)
    assert_close("y", y, ref, tol)
    want, tols = oracle.gram_backward_brute(a, x, g)
    saved, alone = gpu_gram_backward(a, x, g, flags=B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN, ws=ws), gpu_gram_backward(a, x, g)
    for name, u, v, rv, tv in zip(("gx", "ga"), saved, alone, want, tols):
        assert_close(name, u, rv, tv)
        assert np.array_equal(u, v), name


@pytest.mark.parametrize("kind", ["uniform", "few_values", "equal", "ascending", "repeating", "narrow_windows"])
@pytest.mark.parametrize("N", [(1 << 16) - 1, 1 << 16, (1 << 16) + 1])
def test_sample_sort_short_stretches(oracle, N, kind):
    """The same where the sort's stretches go from 512 to 1024 pairs on average."""
    test_sample_sort_order_and_decays(oracle, N, kind)


@pytest.mark.parametrize("kind", ["uniform", "ties"])
@pytest.mark.parametrize("n,batch,pad", [(8193, 9, 0), (8704, 12, 4), (8705, 16, 1), (8703, 33, 0), (8449, 64, 0), (8256, 65, 3), (8255, 128, 0), (12289, 127, 0)])
def test_gram_both_matrices_in_one_walk(oracle, n, batch, pad, kind):
    """Square form, 9 to 128 columns: the backward scans x beside gy from the carries that the forward kept; whole and partial blocks (512 to 64
    rows), whole and ragged rows, equal anchors."""
    from test_gpu_parity import anchors, assert_close
    r = np.random.default_rng(n + batch)
    a, _ = anchors(kind, r, n, 1)
    x, g = (r.normal(size=(n, batch)).astype(np.float32) for _ in range(2))
    ref, tol = oracle.gram_scan(a, x)
    want, tols = oracle.gram_backward_scan(a, x, g)
    da = torch.from_numpy(a).cuda()
    wide = torch.zeros(3, n, batch + pad, device="cuda")
    dx, dg, gx = (w[:, :batch] for w in wide)
    dx.copy_(torch.from_numpy(x)); dg.copy_(torch.from_numpy(g))
    y = torch.empty(n, batch, device="cuda"); ga = torch.empty(n, device="cuda")
    ws = torch.full((B.laplex_workspace_bytes(0, n, batch),), 0xFF, dtype=torch.uint8, device="cuda")
    B.laplex_gram(da, dx, y, ws, B.LAPLEX_SAVE_SCANS)
    assert_close("y", y.cpu().numpy(), ref, tol)
    first = None
    for flags, want_gx in ((B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN, True), (B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN, False), (0, True), (0, False)):
        ga.fill_(np.nan); wide[2].fill_(np.nan)
        B.laplex_gram_backward(da, dx, dg, gx if want_gx else None, ga, ws, flags)
        torch.cuda.synchronize()
        got = gx.cpu().numpy(), ga.cpu().numpy()
        if first is None: first = got
        assert_close("ga", got[1], want[1], tols[1])
        assert np.array_equal(got[1], first[1])
        if want_gx:
            assert_close("gx", got[0], want[0], tols[0])
            assert np.array_equal(got[0], first[0])
        assert pad == 0 or bool(torch.isnan(wide[2, :, batch:]).all())


@pytest.mark.parametrize("batch", [1, 2, 4, 8])
def test_products_pair_by_pair_weights(batch):
    """One input of value one: the products are the weights exp(-d) themselves, d from 0 to beyond where they end.  Three units in the last place where they are
    normal numbers; below, where a unit is 2^-149, one and a half: half of one for the rounding, one for what the exponential is off before it."""
    d = np.concatenate([np.linspace(0, 110, 600), np.linspace(86, 104.5, 400)]).astype(np.float32)
    a, b = (d * np.where(np.arange(d.size) % 2, 1, -1)).astype(np.float32), np.zeros(1, dtype=np.float32)
    ws = torch.empty(B.laplex_workspace_bytes(a.size, 1, batch), dtype=torch.uint8, device="cuda")
    y = torch.empty(a.size, batch, device="cuda")
    B.laplex_apply(dev(a), dev(b), torch.ones(1, batch, device="cuda"), y, ws, 0)
    torch.cuda.synchronize()
    ref = np.exp(-d.astype(np.float64))[:, None]
    unit = np.spacing(ref.astype(np.float32)).astype(np.float64)
    units = np.abs(y.cpu().numpy().astype(np.float64) - ref) / unit
    low = np.broadcast_to(ref < 2.0 ** -126, units.shape)
    assert units[~low].max() <= 3.0 and units[low].max() <= 1.5, (units[~low].max(), units[low].max())


@pytest.mark.parametrize("k,n,batch", [(700, 900, 1), (4000, 4000, 1), (8000, 100, 1), (500, 400, 2), (300, 1100, 4), (900, 300, 8), (4200, 3900, 1), (2500, 2400, 8),
                                       (40, 60, 20)])
def test_small_problems_of_two_clusters_far_apart(oracle, k, n, batch):
    """Outputs 88 to 103 away from every input, rows of size 1e30: weights that are no normal numbers, sums that are.  |err| against fp64 is at most
    2^-149 (a unit of such a weight) and 1e-6 of the weight (anchors of size 100 differ by exact numbers; products of two normal decays in the scans) for
    every term; either side of the lines up to which the products are formed pair by pair."""
    r = np.random.default_rng(k + batch)
    a, b = r.uniform(0, 7, k).astype(np.float32), r.uniform(95, 103, n).astype(np.float32)
    x, g = (r.choice([-1e30, 1e30], (s, batch)) * r.uniform(1, 2, (s, batch)) for s in (n, k))
    x, g = x.astype(np.float32), g.astype(np.float32)
    ws = torch.empty(B.laplex_workspace_bytes(k, n, batch), dtype=torch.uint8, device="cuda")
    y, gx, ga, gb = (torch.full(s, float("nan"), device="cuda") for s in ((k, batch), (n, batch), (k,), (n,)))
    B.laplex_apply(dev(a), dev(b), dev(x), y, ws, B.LAPLEX_SAVE_SCANS)
    B.laplex_apply_backward(dev(a), dev(b), dev(x), dev(g), gx, ga, gb, ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
    torch.cuda.synchronize()
    w = np.exp(-np.abs(a.astype(np.float64)[:, None] - b.astype(np.float64)[None, :]))
    off = 2.0 ** -149 + 1e-6 * w
    x, g = x.astype(np.float64), g.astype(np.float64)
    ref = w @ x, w.T @ g, np.sum(g * (w @ x), 1), -np.sum(x * (w.T @ g), 1)
    bar = off @ np.abs(x), off.T @ np.abs(g), np.sum(np.abs(g) * (off @ np.abs(x)), 1), np.sum(np.abs(x) * (off.T @ np.abs(g)), 1)
    for name, got, rv, tv in zip(("y", "gx", "ga", "gb"), (y, gx, ga, gb), ref, bar):
        worst = float((np.abs(got.cpu().numpy().astype(np.float64) - rv) / tv).max())
        assert worst <= 1.0, f"{name}: {worst:.3g} times the bar"


@pytest.mark.parametrize("k,n,batch,forward,backward", [
    (4096, 4096, 1, True, True), (3000, 10, 1, True, True), (10, 3000, 1, True, True),
    (3072, 900, 4, True, True), (900, 3073, 4, False, False), (16, 3000, 2, True, True), (1700, 1500, 8, True, True),
    (2048, 100, 8, True, True), (100, 2048, 8, True, True), (2049, 100, 8, True, False), (100, 2049, 8, False, False),     # 256 workgroups; two stages
    (3000, 10, 8, False, False), (500, 13, 32, True, True), (700, 13, 32, True, False), (900, 13, 32, False, False),       # several slabs: 252, 352, 452 workgroups
    (10, 2000, 32, True, False), (3000, 10, 256, False, False), (10, 3000, 256, False, False), (575, 648, 9, True, True), (640, 1979, 9, False, False),
])
def test_which_small_problems_go_pair_by_pair(oracle, k, n, batch, forward, backward):
    """Problems of many result rows and hardly any injected ones, whose workgroups queue up however few the pairs are, stay with the scans (3000 x 10, batch 256, forward and
    backward: 49.7 us, 336 pair by pair); what either product is formed by shows in the launches.  The sums where the two go different ways."""
    from test_gpu_parity import anchors, assert_close
    r = np.random.default_rng(k + 5 * n + batch)
    a, b = anchors("ties", r, k, n)
    x, g = r.normal(size=(n, batch)).astype(np.float32), r.normal(size=(k, batch)).astype(np.float32)
    ref, tol = oracle.apply_scan(a, b, x)
    want, tols = oracle.apply_backward_scan(a, b, x, g)
    da, db, dx, dg = dev(a), dev(b), dev(x), dev(g)
    ws = torch.empty(B.laplex_workspace_bytes(k, n, batch), dtype=torch.uint8, device="cuda")
    y, gx, ga, gb = torch.empty_like(dg), torch.empty_like(dx), torch.empty_like(da), torch.empty_like(db)
    seen = families(lambda: B.laplex_apply(da, db, dx, y, ws, B.LAPLEX_SAVE_SCANS))
    assert seen == ({"small_pairs": 1} if forward else {"small_sort": 1, "small": 1})
    assert_close("y", y.cpu().numpy(), ref, tol)
    seen = families(lambda: B.laplex_apply_backward(da, db, dx, dg, gx, None, gb, ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN))
    assert ("small_pairs" in seen, "small" in seen) == (backward, not backward)
    first = None
    for flags in (B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN, B.LAPLEX_REUSE_PLAN, 0):
        for v in (gx, ga, gb): v.fill_(float("nan"))
        B.laplex_apply_backward(da, db, dx, dg, gx, ga, gb, ws, flags)
        torch.cuda.synchronize()
        got = [v.cpu().numpy() for v in (gx, ga, gb)]
        if first is None: first = got
        for name, v, rv, tv, f in zip(("gx", "ga", "gb"), got, want, tols, first):
            assert_close(name, v, rv, tv)
            assert np.array_equal(v, f), name


@pytest.mark.parametrize("r,k,n,batch,forward,backward", [
    (16, 100, 39, 1, True, True), (2, 2300, 582, 1, True, True), (8, 632, 944, 1, False, False), (12, 15, 1640, 9, False, False), (6, 143, 87, 9, True, True),
    (16, 100, 900, 8, False, False), (16, 10, 600, 32, True, False), (4, 7, 300, 9, True, False), (16, 10, 1100, 8, False, False), (16, 10, 1100, 1, True, False),
    (12, 328, 878, 1, False, False), (10, 6, 1554, 1, True, False),      # one column, beside 14000 and 15000 ranks: many and few pairs
])
def test_which_small_sums_go_pair_by_pair(oracle, r, k, n, batch, forward, backward):
    """The same for sums of operators; those sorted by samples in a launch of their own (more than 17000 anchors) only with one column."""
    from test_gpu_parity import assert_close
    q = np.random.default_rng(r + k + n)
    a, b = (np.round(q.uniform(0, (k + n) / 64, (r, s)) * 8).astype(np.float32) / 8 for s in (k, n))
    x, g, w = q.normal(size=(n, batch)).astype(np.float32), q.normal(size=(k, batch)).astype(np.float32), q.normal(size=r).astype(np.float32)
    da, db, dw, dx, dg = dev(a), dev(b), dev(w), dev(x), dev(g)
    ws = torch.empty(B.laplex_mix_workspace_bytes(r, k, n, batch), dtype=torch.uint8, device="cuda")
    y, gx, ga, gb, gw = torch.empty_like(dg), torch.empty_like(dx), torch.empty_like(da), torch.empty_like(db), torch.empty_like(dw)
    seen = families(lambda: B.laplex_mix_apply(da, db, dw, dx, y, ws, B.LAPLEX_SAVE_SCANS))
    assert ("small_pairs" in seen, "small" in seen) == (forward, not forward), seen
    seen = families(lambda: B.laplex_mix_apply_backward(da, db, dw, dx, dg, gx, ga, gb, gw, ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN))
    assert ("small_pairs" in seen, "small" in seen) == (backward, not backward), seen
    ref, tol = oracle.mix_apply(a, b, w, x, brute=False)
    assert_close("y", y.cpu().numpy(), ref, tol)
    want, tols = oracle.mix_backward(a, b, w, x, g, brute=False)
    for name, v, rv, tv in zip(("gx", "ga", "gb", "gw"), (gx, ga, gb, gw), want, tols):
        assert_close(name, v.cpu().numpy(), rv, tv)


@pytest.mark.parametrize("r,k,n,batch", [(2, 40000, 25536, 2), (2, 40000, 25537, 2), (3, 31072, 100000, 1)])
def test_mix_sorted_by_samples_up_to_2_to_17(oracle, r, k, n, batch):
    """Sums whose operators have 2^16 to 2^17 anchors: each is sorted with twice as many samples as such a problem by itself, in scratch that has to be sized for them."""
    from test_gpu_parity import assert_close, gpu_perm
    q = np.random.default_rng(k + n)
    a, b = (np.round(q.uniform(0, (k + n) / 64, (r, s)) * 8).astype(np.float32) / 8 for s in (k, n))
    x, w = q.normal(size=(n, batch)).astype(np.float32), q.normal(size=r).astype(np.float32)
    ws = torch.empty(B.laplex_mix_workspace_bytes(r, k, n, batch), dtype=torch.uint8, device="cuda")
    y = torch.empty(k, batch, device="cuda")
    B.laplex_mix_apply(dev(a), dev(b), dev(w), dev(x), y, ws, 0)
    torch.cuda.synchronize()
    ref, tol = oracle.mix_apply(a, b, w, x, brute=False)
    assert_close("y", y.cpu().numpy(), ref, tol)
    one = (B.laplex_workspace_bytes(k, n, batch) + 255) // 256 * 256
    for p in range(r):
        assert np.array_equal(gpu_perm(ws[p * one:], k + n), oracle.merged_permutation(a[p], b[p])), p


@pytest.mark.parametrize("kind", ["uniform", "ties", "all_equal"])
@pytest.mark.parametrize("k,n,ld", [(9000, 200000, 1), (65536, 65537, 2), (1, 8192, 1), (40003, 9, 3), (0, 70001, 1), (0, 98304, 2)])
def test_one_column_in_order(oracle, k, n, ld, kind):
    """Batch 1 on the routes through sorted order, anchors that arrive in order and are promised to (k = 0: Gram form): merged, not sorted, and rows fetched by the ids. The plan
    serves calls without the promise, which find no tables of moves in it, and a plan that was sorted serves calls with it; the same bits either way."""
    from test_gpu_parity import anchors, assert_close, gpu_perm, gpu_plan_status
    r = np.random.default_rng(k + n + ld)
    gram = k == 0
    a, b = anchors(kind, r, k or 1, n)
    a, b = np.sort(a), np.sort(b)
    rows = n if gram else k
    x, g = r.normal(size=(n, 1)).astype(np.float32), r.normal(size=(rows, 1)).astype(np.float32)
    if gram:
        (ref, tol), (want, tols) = oracle.gram_scan(b, x), oracle.gram_backward_scan(b, x, g)
        promise = B.LAPLEX_A_SORTED
    else:
        (ref, tol), (want, tols) = oracle.apply_scan(a, b, x), oracle.apply_backward_scan(a, b, x, g)
        promise = B.LAPLEX_A_SORTED | B.LAPLEX_B_SORTED
    wide = [torch.zeros(s, ld, device="cuda") for s in (n, rows)]
    dx, dg = (w[:, :1] for w in wide)
    dx.copy_(dev(x)); dg.copy_(dev(g))
    da, db = dev(a), dev(b)
    y, gx, ga, gb = torch.empty(rows, 1, device="cuda"), torch.empty(n, 1, device="cuda"), torch.empty(rows, device="cuda"), torch.empty(n, device="cuda")
    ws = torch.full((B.laplex_workspace_bytes(k, n, 1),), 0xFF, dtype=torch.uint8, device="cuda")

    def forward(flags):
        B.laplex_gram(db, dx, y, ws, flags) if gram else B.laplex_apply(da, db, dx, y, ws, flags)

    def backward(flags):
        B.laplex_gram_backward(db, dx, dg, gx, ga, ws, flags) if gram else B.laplex_apply_backward(da, db, dx, dg, gx, ga, gb, ws, flags)

    perm = np.argsort(b, kind="stable") if gram else oracle.merged_permutation(a, b)
    B.laplex_diag_set_route_min(0)
    try:
        first = None
        for built, later in ((promise, promise), (promise, 0), (0, promise), (0, 0)):
            seen = families(lambda: forward(built | B.LAPLEX_SAVE_SCANS))
            assert ("merge" in seen) == ("move_in_order.fwd" in seen) == (built != 0) and ("deep_sort" in seen) == (built == 0), seen
            assert np.array_equal(gpu_perm(ws, k + n), perm) and gpu_plan_status(ws, k + n) == 0
            for again in (False, True):
                if again: y.fill_(np.nan); forward(later | B.LAPLEX_REUSE_PLAN)
                torch.cuda.synchronize()
                assert_close("y", y.cpu().numpy(), ref, tol)
            for flags in (B.LAPLEX_REUSE_PLAN, 0):
                for v in (gx, ga, gb): v.fill_(np.nan)
                backward(later | flags)
                torch.cuda.synchronize()
                got = [y.cpu().numpy(), gx.cpu().numpy(), ga.cpu().numpy()] + ([] if gram else [gb.cpu().numpy()])
                if first is None: first = got
                for name, v, rv, tv, f in zip(("gx", "ga", "gb"), got[1:], want, tols, first[1:]):
                    assert_close(name, v, rv, tv)
                    assert np.array_equal(v, f), name
                assert np.array_equal(got[0], first[0])
    finally:
        B.laplex_diag_set_route_min(1 << 22)


def test_one_column_in_order_with_a_wrong_promise():
    """Anchors that are not in order, and not finite: any values, but the calls end and the workspace serves a clean problem afterwards."""
    from test_gpu_parity import gpu_perm
    q = np.random.default_rng(7)
    k, n = 30000, 50001
    x = torch.ones(n, 1, device="cuda")
    y = torch.empty(k, 1, device="cuda")
    ws = torch.empty(B.laplex_workspace_bytes(k, n, 1), dtype=torch.uint8, device="cuda")
    promise = B.LAPLEX_A_SORTED | B.LAPLEX_B_SORTED
    B.laplex_diag_set_route_min(0)
    try:
        for bad in (True, False):
            a, b = q.uniform(0, 1000, k).astype(np.float32), q.uniform(0, 1000, n).astype(np.float32)
            if bad: a[::50] = np.nan; b[3] = np.inf
            for flags in (promise, B.LAPLEX_REUSE_PLAN, promise | B.LAPLEX_REUSE_PLAN):
                B.laplex_apply(dev(a), dev(b), x, y, ws, flags)
                torch.cuda.synchronize()
        a, b = np.sort(a), np.sort(b)
        B.laplex_apply(dev(a), dev(b), x, y, ws, promise)
        pos = np.empty(k + n, np.int64); pos[gpu_perm(ws, k + n)] = np.arange(k + n)
        v = np.concatenate([a, b])
        assert np.all(np.diff(v[np.argsort(pos)]) >= 0)
    finally:
        B.laplex_diag_set_route_min(1 << 22)


@pytest.mark.parametrize("k,n", [((1 << 23) + 5, (1 << 23) + 9), ((1 << 25) + 3, (1 << 25) + 12345), ((1 << 28) + 11, (1 << 28) + 7777), (3 << 21, 1 << 20), ((1 << 22) + 1, 5)])
def test_one_column_every_output_at_large_sizes(k, n):
    """Batch 1 beyond what an oracle on the host can check output by output: tiles of 16384 (beyond 2^24 positions), more than 64 chunks of them (2^26), units of 8192 pairs (2^29), windows of
    8192 and 16384.  Anchors are distinct floats from 2^30 on, 128 and more apart, so that a weight is one or nothing, and an output is its tied input, or zero."""
    import gc
    gc.collect(); torch.cuda.empty_cache()
    gen = torch.Generator(device="cuda"); gen.manual_seed(k)
    m = max(k, n)
    first = 0x4E800000                                       # 2^30
    at_a, at_b = (torch.randperm(m, generator=gen, device="cuda", dtype=torch.int32)[:s] for s in (k, n))
    a, b = ((v + first).view(torch.float32) for v in (at_a, at_b))
    x, g = (torch.randn(s, 1, generator=gen, device="cuda") for s in (n, k))
    ws = torch.empty(B.laplex_workspace_bytes(k, n, 1), dtype=torch.uint8, device="cuda")
    y, gx, ga, gb = torch.empty_like(g), torch.empty_like(x), torch.empty_like(a), torch.empty_like(b)
    for flags in (B.LAPLEX_SAVE_SCANS, 0):
        B.laplex_apply(a, b, x, y, ws, flags)
        B.laplex_apply_backward(a, b, x, g, gx, ga, gb, ws, flags | B.LAPLEX_REUSE_PLAN)
        torch.cuda.synchronize()
        of = torch.zeros(m, device="cuda")
        of[at_b] = x[:, 0]
        assert torch.equal(y[:, 0], of[at_a])
        of.zero_(); of[at_a] = g[:, 0]
        assert torch.equal(gx[:, 0], of[at_b])
        assert not bool(ga.any()) and not bool(gb.any())
        y.fill_(float("nan")); gx.fill_(float("nan")); ga.fill_(float("nan")); gb.fill_(float("nan"))
        del of


def test_one_column_bucket_of_many_pieces(oracle):
    """A bucket of more pieces than a workgroup has threads (512 in the sort, 256 where values move): its stretches that would fit LDS are handled in memory, too."""
    test_sort_in_two_distributions(oracle, 2500000, 2300000, "unsampled", 0)


@pytest.mark.parametrize("kind", ["from_zero", "both_sides", "subnormal", "wide", "not_finite"])
@pytest.mark.parametrize("N", [9000, 65536, 100000, 600000, 5000000])
def test_sample_sort_grid_near_zero(N, kind):
    """Some 32 equal anchors to a multiple of 1/4 (of 2^-140; beside 2^60; beside anchors that are not finite), zero among them: the stretches where a step of the grid is many
    times as many keys as elsewhere are counted by the multiple and the id.  The order is numpy's stable one."""
    r = np.random.default_rng(N + len(kind))
    v = np.round(r.uniform(0 if kind in ("from_zero", "subnormal") else -N / 256, N / 128, N) * 4)
    v = (v * (2.0 ** -140 if kind == "subnormal" else 0.25)).astype(np.float32)
    if kind == "wide": v[::7] = 2.0 ** 60; v[1::11] = -2.0 ** -60
    if kind == "not_finite": v[::500] = np.inf; v[1::700] = -np.inf
    v += 0.0          # (-0.0 sorts as 0.0)
    k = N // 3
    ids, _ = sorted_ids(v[:k], v[k:])
    assert np.array_equal(ids.view(np.uint32), np.argsort(v, kind="stable").astype(np.uint32))

"""Values at equal anchors and of non-finite rows.  Tied pairs contribute exactly nothing to anchor gradients, however large their
rows are; so the bars here scale with the strict sums alone (the usual denominators include the tied terms, which hide what is
lost beside them)."""
import numpy as np
import pytest

from paper_2605_24584_amd import binding as B

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import dev  # noqa: E402


def runs_of_ties(count, spacing, lengths):
    """`count` ascending anchors `spacing` apart, in runs of equal ones of the given lengths, over and over."""
    v, q = [], 0
    while len(v) < count:
        v += [q * spacing] * lengths[q % len(lengths)]
        q += 1
    return np.array(v[:count], dtype=np.float32)


def mix_step(a, b, w, x, g, flags, ws=None):
    """y, gx, ga, gb, gw of one forward + backward pair (flags: LAPLEX_SAVE_SCANS or 0)."""
    r, k, n, batch = a.shape[0], a.shape[1], b.shape[1], x.shape[1]
    ws = torch.empty(B.laplex_mix_workspace_bytes(r, k, n, batch), dtype=torch.uint8, device="cuda") if ws is None else ws
    out = [torch.full(s, float("nan"), device="cuda") for s in ((k, batch), (n, batch), (r, k), (r, n), (r,))]
    da, db, dw, dx, dg = dev(a), dev(b), dev(w), dev(x), dev(g)
    B.laplex_mix_apply(da, db, dw, dx, out[0], ws, flags)
    B.laplex_mix_apply_backward(da, db, dw, dx, dg, *out[1:], ws, flags | B.LAPLEX_REUSE_PLAN)
    torch.cuda.synchronize()
    return [v.cpu().numpy().astype(np.float64) for v in out]


def strict_gradients(oracle, a, b, w, x, g):
    """ga, gb and their denominators over the strictly separated pairs, one operator after the other (fp64)."""
    res = [[], [], [], []]
    for q in range(a.shape[0]):
        for at, (src, val, query, mult) in enumerate(((b[q], x, a[q], g), (a[q], g, b[q], x))):
            _, ls, rs = oracle._dual(src, val, query, want=(False, True, True))
            _, la, ra = oracle._dual(src, val, query, use_abs=True, want=(False, True, True))
            m = float(w[q]) * mult.astype(np.float64)
            res[at].append(np.sum(m * (rs - ls), axis=1))
            res[2 + at].append(np.sum(np.abs(m) * (la + ra), axis=1))
    return [np.stack(v) for v in res]


@pytest.mark.parametrize("spacing", [2.0, 12.0, 16.0])
@pytest.mark.parametrize("k,n,batch", [(2600, 7000, 1), (7000, 2600, 4), (2600, 7000, 33), (7000, 2600, 33), (2600, 7000, 64),
                                       (7000, 2600, 64), (5000, 5000, 8)])
def test_mix_strict_sums_beside_large_ties(oracle, k, n, batch, spacing):
    """Sums of operators in common launches: runs of up to 300 equal short anchors (tiles of 64 to 2048 rows), each tied with a
    couple of hundred long rows of size 1e6.  A strict sum is exp(-spacing) of its tied neighbours at most; formed as a difference
    it would keep 24 bits of those, an error of 2^-24 exp(spacing): 1e-2 at 12, where the bar is 1e-5 (fp32 decays and sums over a
    few hundred rows: below 2e-6)."""
    q = np.random.default_rng(k + batch)
    r = 2
    short, long_ = min(k, n), max(k, n)
    s = runs_of_ties(short, spacing, (1, 3, 300, 2))
    sides = []
    for _ in range(r):
        l = s[q.integers(0, short, long_)]
        sides.append((q.permutation(s), l) if k <= n else (l, q.permutation(s)))
    if k == n:
        sides = [(v, u) for u, v in sides]
    a, b = np.stack([u for u, _ in sides]), np.stack([v for _, v in sides])
    w = np.array([0.75, -1.5], dtype=np.float32)
    x = (1e6 * q.normal(size=(n, batch))).astype(np.float32)
    g = (1e6 * q.normal(size=(k, batch))).astype(np.float32)
    ga, gb, ta, tb = strict_gradients(oracle, a, b, w, x, g)
    for flags in (B.LAPLEX_SAVE_SCANS, 0):
        _, _, got_a, got_b, _ = mix_step(a, b, w, x, g, flags)
        for name, got, ref, tol in (("ga", got_a, ga, ta), ("gb", got_b, gb, tb)):
            worst = float((np.abs(got - ref) / (1e-5 * tol + 1e-30)).max())
            assert worst <= 1.0, f"{name}: {worst:.3g} times the bar"


@pytest.mark.parametrize("k,n,batch", [(3000, 7000, 4), (7000, 3000, 4), (3000, 7000, 33), (7000, 3000, 1), (2500, 6000, 64)])
def test_mix_infinite_row_at_a_tie(oracle, k, n, batch):
    """One infinite value in a long row that equals short anchors, everything within reach of it: the product at the tied anchors,
    and on either side, is infinite, and the tied anchors' gradients, which it does not enter, are finite and right."""
    q = np.random.default_rng(k + n + batch)
    a, b = (np.round(q.uniform(0, 40, s) * 4).astype(np.float32) / 4 for s in (k, n))
    w = np.array([2.0], dtype=np.float32)
    x, g = (q.normal(size=(s, batch)).astype(np.float32) for s in (n, k))
    col = batch // 2
    ga, gb, ta, tb = strict_gradients(oracle, a[None], b[None], w, x, g)
    if k <= n:
        x[n // 3, col] = np.inf
        tied, at, name = a == b[n // 3], 3, "ga"
    else:
        g[k // 3, col] = np.inf
        tied, at, name = b == a[k // 3], 3, "gb"
    assert 0 < tied.sum() < tied.size
    y, gx, got_a, got_b, _ = mix_step(a[None], b[None], w, x, g, B.LAPLEX_SAVE_SCANS)
    product = y if k <= n else gx
    assert np.all(np.isposinf(product[:, col])) and np.all(np.isfinite(np.delete(product, col, axis=1)))
    got, ref, tol = (got_a[0], ga[0], ta[0]) if k <= n else (got_b[0], gb[0], tb[0])
    assert float((np.abs(got - ref) / (1e-5 * tol + 1e-30))[tied].max()) <= 1.0, name
    assert not np.any(np.isfinite(got[~tied]))


def assert_all_non_finite(name, v, cols=slice(None)):
    v = v.cpu().numpy() if hasattr(v, "cpu") else v
    bad = np.isfinite(v if v.ndim == 1 else v[:, cols])
    assert not bad.any(), f"{name}: {int(bad.sum())} of {bad.size} values finite"


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("k,n,batch", [
    (700, 300, 1), (4000, 4100, 2), (513, 1024, 64), (4000, 4000, 100), (300, 212, 1000),        # small problems, each form
    (30, 8000, 1100), (2000, 2000, 2100),
    (10000, 9000, 1), (9000, 8000, 8), (65000, 66072, 8), (1000, 40000, 33), (700, 30000, 256),  # larger ones, each form of the spine
    (900000, 600000, 8), (30, 140000, 256), (2500000, 2200000, 1),
])
def test_non_finite_rows_reach_every_row(k, n, batch, bad):
    """As in the dense product (0 * NaN and 0 * inf are NaN), one non-finite value of x or gy shows in every row of its column and in
    every anchor gradient, also where all decays between underflow: anchors spread over 3000 decay lengths."""
    q = np.random.default_rng(k + batch)
    a, b = (q.uniform(0, 3000, s).astype(np.float32) for s in (k, n))
    x, g = (q.normal(size=(s, batch)).astype(np.float32) for s in (n, k))
    col = batch // 2
    new = lambda *s: torch.zeros(*s, device="cuda")
    ws = torch.empty(B.laplex_workspace_bytes(k, n, batch), dtype=torch.uint8, device="cuda")
    da, db = dev(a), dev(b)
    for side in ("x", "gy"):
        dx, dg = dev(x), dev(g)
        (dx if side == "x" else dg)[q.integers(0, n if side == "x" else k), col] = bad
        y, gx, ga, gb = new(k, batch), new(n, batch), new(k), new(n)
        B.laplex_apply(da, db, dx, y, ws, B.LAPLEX_SAVE_SCANS)
        B.laplex_apply_backward(da, db, dx, dg, gx, ga, gb, ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
        torch.cuda.synchronize()
        if side == "x":
            assert_all_non_finite("y", y, col); assert_all_non_finite("ga", ga)
        else:
            assert_all_non_finite("gx", gx, col); assert_all_non_finite("gb", gb)
        finite = (y if side == "gy" else gx)
        assert bool(torch.isfinite(finite).all())


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("n,batch", [(9000, 1), (9000, 8), (8193, 9), (9001, 33), (20000, 64), (30011, 128), (9000, 130), (300, 16)])
def test_gram_non_finite_rows_reach_every_row(n, batch, bad):
    """The same for the Gram form: one row of x or gy shows in its column of y or gx, and through either scan in every anchor's gradient (9 to 128 columns of more than 8192 rows: x
    is scanned again beside gy, from the states that the forward kept)."""
    q = np.random.default_rng(n + batch)
    b = dev(q.uniform(0, 3000, n).astype(np.float32))
    x, g = (q.normal(size=(n, batch)).astype(np.float32) for _ in "xg")
    col = batch // 2
    ws = torch.empty(B.laplex_workspace_bytes(0, n, batch), dtype=torch.uint8, device="cuda")
    for side in ("x", "gy"):
        for save in (B.LAPLEX_SAVE_SCANS, 0):
            dx, dg = dev(x), dev(g)
            (dx if side == "x" else dg)[q.integers(0, n), col] = bad
            y, gx, ga = torch.zeros(n, batch, device="cuda"), torch.zeros(n, batch, device="cuda"), torch.zeros(n, device="cuda")
            B.laplex_gram(b, dx, y, ws, save)
            B.laplex_gram_backward(b, dx, dg, gx, ga, ws, save | B.LAPLEX_REUSE_PLAN)
            torch.cuda.synchronize()
            assert_all_non_finite("ga", ga)
            assert_all_non_finite("y" if side == "x" else "gx", y if side == "x" else gx, col)
            assert bool(torch.isfinite(gx if side == "x" else y).all())


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("k,n,batch", [(10000, 9000, 1), (9000, 8000, 8), (65000, 66072, 8), (7000, 2000, 3), (5000, 4000, 5), (6000, 3001, 33), (4097, 4097, 64), (5000, 4000, 128),
                                       (0, 9000, 1), (0, 9000, 8), (0, 8193, 9), (0, 9001, 33), (0, 20000, 64), (0, 9003, 127)])
def test_non_finite_rows_reach_blocks_that_do_not_wait(k, n, batch, bad):
    """The two tests above where a scan is one launch, with no block waiting for the others (k = 0: the Gram form)."""
    q = np.random.default_rng(k + n + batch)
    a, b = (dev(q.uniform(0, 3000, s).astype(np.float32)) for s in (k or n, n))
    x, g = (q.normal(size=(s, batch)).astype(np.float32) for s in (n, k or n))
    col = batch // 2
    ws = torch.empty(B.laplex_workspace_bytes(k, n, batch), dtype=torch.uint8, device="cuda")
    built = 0
    for side in ("x", "gy"):
        dx, dg = dev(x), dev(g)
        (dx if side == "x" else dg)[q.integers(0, n if side == "x" else k or n), col] = bad
        y, gx, ga, gb = torch.zeros_like(dg), torch.zeros_like(dx), torch.zeros_like(a), torch.zeros_like(b)
        for again in range(2):                       # the first pass builds the plan, the second scans on it without waiting
            flags = B.LAPLEX_SAVE_SCANS | built
            if k:
                B.laplex_apply(a, b, dx, y, ws, flags)
                B.laplex_apply_backward(a, b, dx, dg, gx, ga, gb, ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
            else:
                B.laplex_gram(b, dx, y, ws, flags)
                B.laplex_gram_backward(b, dx, dg, gx, ga, ws, B.LAPLEX_SAVE_SCANS | B.LAPLEX_REUSE_PLAN)
            if not built:
                B.laplex_diag_set_wait_limit(ws, k + n, 0)
                built = B.LAPLEX_REUSE_PLAN
                for v in (y, gx, ga, gb):
                    v.zero_()
        torch.cuda.synchronize()
        if side == "x" or not k:
            assert_all_non_finite("ga", ga)
        if side == "gy" and k:
            assert_all_non_finite("gb", gb)
        assert_all_non_finite("y" if side == "x" else "gx", y if side == "x" else gx, col)
        assert bool(torch.isfinite(gx if side == "x" else y).all())


@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
@pytest.mark.parametrize("r,k,n,batch", [(2, 3000, 7000, 1), (2, 7000, 3000, 33), (3, 5000, 5000, 64), (2, 300, 400, 8), (4, 33000, 33000, 2)])
def test_mix_non_finite_rows_reach_every_row(r, k, n, batch, bad):
    """The same for sums of operators, on each of their routes."""
    q = np.random.default_rng(k + batch)
    a, b = (q.uniform(0, 3000, (r, s)).astype(np.float32) for s in (k, n))
    w = np.ones(r, dtype=np.float32)
    x, g = (q.normal(size=(s, batch)).astype(np.float32) for s in (n, k))
    col = batch // 2
    for side in ("x", "gy"):
        bx, bg = x.copy(), g.copy()
        (bx if side == "x" else bg)[q.integers(0, n if side == "x" else k), col] = bad
        y, gx, ga, gb, gw = mix_step(a, b, w, bx, bg, B.LAPLEX_SAVE_SCANS)
        assert_all_non_finite("gw", gw)
        if side == "x":
            assert_all_non_finite("y", y, col)
            for v in ga:
                assert_all_non_finite("ga", v)
        else:
            assert_all_non_finite("gx", gx, col)
            for v in gb:
                assert_all_non_finite("gb", v)


@pytest.mark.parametrize("n,batch", [(9001, 64), (60000, 33), (150001, 64)])
def test_gram_steps_with_and_without_non_finite_rows_on_one_plan(n, batch):
    """What a step with a value that is not finite leaves in the plan changes no later step; forward and backward, and the backward alone."""
    q = np.random.default_rng(n + batch)
    a, x, g = (dev(v.astype(np.float32)) for v in (q.uniform(0, 3000, n), q.normal(size=(n, batch)), q.normal(size=(n, batch))))
    ws = torch.empty(B.laplex_workspace_bytes(0, n, batch), dtype=torch.uint8, device="cuda")

    def step(flags, x, g, forward):
        y, gx, ga = torch.zeros_like(g), torch.zeros_like(x), torch.zeros_like(a)
        if forward:
            B.laplex_gram(a, x, y, ws, flags | B.LAPLEX_SAVE_SCANS)
        B.laplex_gram_backward(a, x, g, gx, ga, ws, B.LAPLEX_REUSE_PLAN | (B.LAPLEX_SAVE_SCANS if forward else 0))
        torch.cuda.synchronize()
        return y, gx, ga
    xn, gn = x.clone(), g.clone()
    xn[n // 3, batch // 2] = float("nan")
    gn[n // 5, batch // 3] = float("inf")
    want = step(0, x, g, True)
    alone = step(B.LAPLEX_REUSE_PLAN, x, g, False)
    for xs, gs in ((xn, g), (x, gn), (xn, gn)):
        for forward in (True, False):
            y, gx, ga = step(B.LAPLEX_REUSE_PLAN, xs, gs, forward)
            assert_all_non_finite("ga", ga)
            if gs is gn:
                assert_all_non_finite("gx", gx, batch // 3)
            assert bool(torch.isfinite(gx[:, 0]).all())
            for again, first in ((True, want), (False, alone), (True, want)):
                assert all(torch.equal(v, w) for v, w in zip(step(B.LAPLEX_REUSE_PLAN, x, g, again)[0 if again else 1:], first[0 if again else 1:]))

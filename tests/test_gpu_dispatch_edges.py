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

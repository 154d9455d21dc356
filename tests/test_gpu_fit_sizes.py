"""The fit on both sides of the size from which hits are loaded a layer ahead:
the tracks of a large call are the same as in small ones, bit for bit, with
holes, in both states and both arithmetics."""
import numpy as np
import pytest

from paper_1711_06571_amd import datagen, presets

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_common import host, to_dev  # noqa: E402


@pytest.mark.parametrize("hybrid", [False, True])
@pytest.mark.parametrize("f64", [False, True])
def test_large_call_equals_small_calls(hybrid, f64):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1711_06571_amd import kftrack as kf
    w = presets.build()
    g, n, part = w.geometry, 8192 + 65, 4096
    H = datagen.track_hits(datagen.generate(g, w.gen, 0, n)).astype(np.float32)
    ld = H.shape[2]
    assert ld >= n
    Hd = to_dev(H)
    s = kf.kf_seed(g, n, Hd[:3].contiguous())
    rng = np.random.default_rng(3)
    holes = rng.integers(0, 1 << g.n_layers, ld).astype(np.int32)
    holes[::3] = 0
    bad = H.copy()
    bad[5, 2, ::97] = np.nan
    Bd, hd = to_dev(bad), to_dev(holes)
    fit = kf.kf_fit_hybrid if hybrid else kf.kf_fit
    arith = kf.ARITH_F64 if f64 else kf.ARITH_F32
    keys = ("par", "cov", "chi2", "ndof", "status")
    big = fit(g, n, 3, Bd, s["par"], s["cov"], s["q"], hole_mask=hd, arith=arith)
    big = {k: host(big[k])[..., :n] for k in keys}
    assert len(np.unique(big["status"])) > 1
    for a in range(0, n, part):
        m = min(part, n - a)
        cut = lambda t: t[..., a:a + m].contiguous()
        o = fit(g, m, 3, cut(Bd), cut(s["par"]), cut(s["cov"]), cut(s["q"]), hole_mask=cut(hd), arith=arith)
        for k in keys:
            assert np.array_equal(host(o[k])[..., :m], big[k][..., a:a + m], equal_nan=True), (k, a)

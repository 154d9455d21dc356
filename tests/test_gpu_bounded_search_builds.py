"""The bounded hit search against the search of every hit (a build that asks
for the work counters) where test_gpu_bounded_search.py does not look: the
learned window, FP32 in the hybrid state, batches of uneven events, rows of
few hits (many z bins), few bins, wide and whole-layer windows.  Bit-identical
outputs."""
import dataclasses

import numpy as np
import pytest

from paper_1711_06571_amd import presets, workloads

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_common import host, to_dev  # noqa: E402

BATCHES = {  # tracks per event, n_phi, n_z
    "uneven": ([20000, 30, 1, 3000, 300], 63, 16),
    "many_rows": ([100] * 40, 8, 64),
    "few_bins": ([6000], 5, 1),
}


@pytest.fixture(scope="module")
def batches():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1711_06571_amd import kftrack as kf
    w, out = presets.build(), {}
    for name, (tracks, n_phi, n_z) in BATCHES.items():
        parts = [workloads.event_batch(w, [e], n_tracks=n, seed_layers=3) for e, n in enumerate(tracks)]
        cat = lambda f: np.ascontiguousarray(np.concatenate([f(p) for p in parts], axis=-1))
        n_hits = [p.layer.shape[0] for p in parts]
        off = np.concatenate([[0], np.cumsum(n_hits)]).astype(np.int32)
        sev = np.repeat(np.arange(len(tracks)), [p.n_seeds for p in parts]).astype(np.int32)
        n = sev.shape[0]
        H = cat(lambda p: p.seed_hits[..., :p.n_seeds])
        ld = (n + 63) // 64 * 64
        Hp = np.zeros(H.shape[:2] + (ld,), np.float32)
        Hp[..., :n] = H
        b = kf.hit_bin(w.geometry, n_phi, n_z, to_dev(cat(lambda p: p.layer)), to_dev(cat(lambda p: p.xyz)),
                       to_dev(cat(lambda p: p.cov)), event_offsets=to_dev(off))
        out[name] = (w, b, kf.kf_seed(w.geometry, n, to_dev(Hp)), to_dev(sev), n)
    rng = np.random.default_rng(1)
    blk = kf.mlp_block((rng.standard_normal(kf.MLP_NPARAM) * 0.1).astype(np.float32), np.zeros(27), np.ones(27),
                       np.array([0.01, 0.1]))
    return out, blk


@pytest.mark.parametrize("name", sorted(BATCHES))
@pytest.mark.parametrize("learned", [0, 1])
@pytest.mark.parametrize("arith,state", [(0, 0), (0, 1), (1, 0), (1, 1)])
@pytest.mark.parametrize("nsigma,chi2", [(3.0, 30.0), (40.0, 1e4)])
def test_equals_search_of_every_hit(batches, name, learned, arith, state, nsigma, chi2):
    from paper_1711_06571_amd import kftrack as kf
    w, b, s, sev, n = batches[0][name]
    cuts = dataclasses.replace(w.cuts, nsigma=nsigma, chi2_cut=chi2)
    bp = kf.build_params(cuts, arith=arith, state=state, window_mode=learned, mlp_block=batches[1] if learned else None)
    cnt = torch.zeros(4, dtype=torch.int64, device="cuda:0")
    ex = kf.BuildExtra()
    ex.seed_event = sev.data_ptr()
    got = kf.kf_build(w.geometry, bp, b, n, s["par"], s["cov"], s["q"], extra=ex)
    ex.counters = cnt.data_ptr()
    every = kf.kf_build(w.geometry, bp, b, n, s["par"], s["cov"], s["q"], extra=ex)
    for k in got:
        a, c = host(got[k])[..., :n], host(every[k])[..., :n]
        assert np.array_equal(a.view(np.int32), c.view(np.int32)), k
    assert int(cnt[2]) > n  # the search of every hit gave many a chi2

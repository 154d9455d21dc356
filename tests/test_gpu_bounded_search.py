"""The bounded hit search (wide windows searched only where a hit that can
survive may lie) against the search of every hit: a build that asks for the
work counters looks at every hit of every window, and its outputs are
bit-identical to those of a build that does not.  A full event holds windows
from none to whole layers; caps at both ends and with seeds that straddle the
pool's size; every slot at its limit of holes, or none allowed."""
import dataclasses

import numpy as np
import pytest

from paper_1711_06571_amd import datagen, presets

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_common import host, to_dev  # noqa: E402


@pytest.fixture(scope="module")
def event():
    from paper_1711_06571_amd import kftrack as kf
    w = presets.build()
    ev = datagen.generate(w.geometry, w.gen, 7, w.n_tracks)
    b = kf.hit_bin(w.geometry, w.cuts.n_phi_bins, w.cuts.n_z_bins, to_dev(ev.layer), to_dev(ev.xyz.astype(np.float32)),
                   to_dev(ev.cov.astype(np.float32)))
    return w, b, kf.kf_seed(w.geometry, w.n_tracks, to_dev(datagen.track_hits(ev)))


@pytest.mark.parametrize("cap", [1, 2, 5, 6, 8])
@pytest.mark.parametrize("holes", [0, 1, 3])
@pytest.mark.parametrize("arith,state", [(0, 0), (1, 0), (1, 1)])
def test_equals_search_of_every_hit(event, cap, holes, arith, state):
    from paper_1711_06571_amd import kftrack as kf
    w, b, s = event
    n = w.n_tracks
    cuts = dataclasses.replace(w.cuts, max_holes=holes)
    bp = kf.build_params(cuts, cap=cap, arith=arith, state=state)
    cnt = torch.zeros(4, dtype=torch.int64, device="cuda:0")
    ex = kf.BuildExtra()
    ex.counters = cnt.data_ptr()
    every = kf.kf_build(w.geometry, bp, b, n, s["par"], s["cov"], s["q"], extra=ex)
    got = kf.kf_build(w.geometry, bp, b, n, s["par"], s["cov"], s["q"])
    for k in got:
        a, c = host(got[k])[..., :n], host(every[k])[..., :n]
        assert np.array_equal(a.view(np.int32), c.view(np.int32)), (k, cap, holes, arith, state)
    assert int(cnt[2]) > 10 * n  # the search of every hit gave many a chi2

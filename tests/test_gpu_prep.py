"""The per-call preparation of a build (fine phi index in passes of 4 096
entries): builds over bin counts whose index rows end just below, at and
above one pass and over two are bit-identical to builds whose rows fit one
small pass (one sub-bin per phi bin)."""
import dataclasses

import numpy as np
import pytest

from paper_1711_06571_amd import datagen, presets

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_common import host, to_dev  # noqa: E402


@pytest.mark.parametrize("n_phi", [63, 64, 65, 129])
@pytest.mark.parametrize("n_tracks", [3, 700])
def test_index_passes(n_phi, n_tracks):
    from paper_1711_06571_amd import kftrack as kf
    w = presets.build()
    g = w.geometry
    cuts = dataclasses.replace(w.cuts, n_phi_bins=n_phi)
    ev = datagen.generate(g, w.gen, 5, n_tracks)
    b = kf.hit_bin(g, n_phi, cuts.n_z_bins, to_dev(ev.layer), to_dev(ev.xyz.astype(np.float32)),
                   to_dev(ev.cov.astype(np.float32)))
    s = kf.kf_seed(g, n_tracks, to_dev(datagen.track_hits(ev)))
    got = [kf.kf_build(g, kf.build_params(cuts, phi_refine=r), b, n_tracks, s["par"], s["cov"], s["q"]) for r in (64, 1)]
    for k in got[0]:
        a, c = (host(o[k])[..., :n_tracks] for o in got)
        assert np.array_equal(a.view(np.int32), c.view(np.int32)), (n_phi, n_tracks, k)

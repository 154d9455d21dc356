"""The fine phi index written by a wave per row (many short rows) and by a
block per row (few): a batch of many small events, built at once and in small
groups of events, gives the same builds bit for bit, over index rows of one
entry a bin, of one pass of a wave and of several."""
import numpy as np
import pytest

from paper_1711_06571_amd import presets, workloads

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_common import host, to_dev  # noqa: E402


@pytest.mark.parametrize("n_phi,n_z,refine", [(63, 16, 1), (63, 16, 8), (64, 16, 8), (63, 16, 64), (9, 64, 57), (1, 16, 1)])
def test_wave_rows_equal_block_rows(n_phi, n_z, refine):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1711_06571_amd import kftrack as kf
    w = presets.build()
    E, group, L = 24, 6, w.geometry.n_layers
    assert E * L * n_z >= 4096 > group * L * n_z or n_z != 16
    eb = workloads.event_batch(w, range(E), n_tracks=40, seed_layers=3)
    seeds = kf.kf_seed(w.geometry, eb.n_seeds, to_dev(eb.seed_hits))
    sev = np.asarray(eb.seed_event)[:eb.n_seeds]
    layer, xyz, cov = np.asarray(eb.layer), np.asarray(eb.xyz), np.asarray(eb.cov)

    def build(e0, e1):
        h = slice(int(eb.hit_offsets[e0]), int(eb.hit_offsets[e1]))
        s = np.flatnonzero((sev >= e0) & (sev < e1))
        idx = torch.from_numpy(s).to("cuda:0")
        off = to_dev((eb.hit_offsets[e0:e1 + 1] - eb.hit_offsets[e0]).astype(np.int32))
        b = kf.hit_bin(w.geometry, n_phi, n_z, to_dev(np.ascontiguousarray(layer[h])),
                       to_dev(np.ascontiguousarray(xyz[:, h])), to_dev(np.ascontiguousarray(cov[:, h])),
                       event_offsets=off)
        ev = to_dev((sev[s] - e0).astype(np.int32))
        ex = kf.BuildExtra()
        ex.seed_event = ev.data_ptr()
        o = kf.kf_build(w.geometry, kf.build_params(w.cuts, phi_refine=refine), b, len(s),
                        seeds["par"][:, idx].contiguous(), seeds["cov"][:, idx].contiguous(),
                        seeds["q"][idx].contiguous(), extra=ex)
        torch.cuda.synchronize()
        return {k: host(v)[..., :len(s)].view(np.int32) for k, v in o.items()}

    whole = build(0, E)
    parts = [build(e, e + group) for e in range(0, E, group)]
    for k in whole:
        assert np.array_equal(whole[k], np.concatenate([p[k] for p in parts], axis=-1)), k

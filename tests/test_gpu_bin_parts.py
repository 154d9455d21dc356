"""Grouped hit_bin, where a range takes several blocks: offsets and order
bit-exact against the oracle, around the sizes of a part, of a chunk of the
staged range and of the pieces of a bin."""
import numpy as np
import pytest

import oracle
from paper_1711_06571_amd import presets

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_common import host, to_dev  # noqa: E402

CASES = {
    # one event, the ends of waves, blocks and parts of 1 024 hits
    "edges": ([[0, 1, 2, 63, 64, 65, 1023, 1024, 1025, 2047, 2048, 2049, 0, 3073, 4096, 4097, 5121]], 63, 16),
    # many parts to a range, whose hits are read one by one
    "gathered": ([[20000, 0, 8191, 8192, 8193, 1] + [300] * 11], 63, 16),
    # four parts and two chunks to a range
    "staged": ([[8190 + l for l in range(17)]] * 8, 63, 16),
    # whole ranges in one part; no pieces (4 096 bins), many pieces (6 bins)
    "no_pieces": ([[700 + 13 * l for l in range(17)]] * 3, 64, 64),
    "many_pieces": ([[900 + 31 * l for l in range(17)]] * 3, 3, 2),
    "empty": ([[0] * 17, [5] + [0] * 16, [0] * 17, [0] * 16 + [7], [0] * 17], 63, 16),
}


@pytest.mark.parametrize("name", sorted(CASES))
@pytest.mark.parametrize("seed", [1, 2])
def test_parts_of_a_range(name, seed):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1711_06571_amd import kftrack as kf
    counts, n_phi, n_z = CASES[name]
    g, rng = presets.build().geometry, np.random.default_rng(seed)
    assert g.n_layers == 17
    events = []
    for c in counts:
        n = sum(c)
        layer = np.repeat(np.arange(17), c).astype(np.int32)
        phi, r = rng.uniform(0, 2 * np.pi, n), 30.0 + 40.0 * layer
        phi[rng.random(n) < 0.02] = 1.25  # equal angles: the index decides
        xyz = np.stack([r * np.cos(phi), r * np.sin(phi), rng.uniform(-1.1, 1.1, n) * g.z_half]).astype(np.float32)
        events.append((layer, xyz, rng.random((6, n)).astype(np.float32)))
    off = np.cumsum([0] + [e[0].shape[0] for e in events]).astype(np.int32)
    layer, xyz, cov = (np.concatenate([e[k] for e in events], axis=-1) for k in range(3))
    b = kf.hit_bin(g, n_phi, n_z, to_dev(layer), to_dev(xyz), to_dev(cov),
                   event_offsets=to_dev(off) if len(events) > 1 else None)
    torch.cuda.synchronize()
    assert int(host(b.bad)[0]) == 0
    offsets, orig, xyzphi, scov = host(b.offsets), host(b.orig), host(b.xyzphi), host(b.cov)
    for e, (lay, x, c) in enumerate(events):
        o = oracle.hit_bin(g, n_phi, n_z, lay, x)
        sl = slice(off[e], off[e + 1])
        assert np.array_equal(offsets[e] - off[e], o["offsets"])
        assert np.array_equal(orig[sl], o["order"])
        assert np.array_equal(xyzphi[3, sl], o["phi"])
        assert np.array_equal(xyzphi[:3, sl], x[:, o["order"]])
        assert np.array_equal(scov[:, sl], c[:, o["order"]])


def test_more_ranges_than_32_bits_of_pieces():
    """45 000 events of one bin a layer: 765 000 ranges, which 3 072 pieces
    each would number past 32 bits.  Hits in the first, some middle and the
    last events."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1711_06571_amd import kftrack as kf
    g, rng, E = presets.build().geometry, np.random.default_rng(5), 45000
    used = [0, 1, 20000, 41000, 41120, 41121, E - 1]
    n_of = np.zeros(E, np.int64)
    n_of[used] = 17 * 40
    off = np.concatenate([[0], np.cumsum(n_of)]).astype(np.int32)
    n = int(off[-1])
    layer = np.tile(np.repeat(np.arange(17), 40), len(used)).astype(np.int32)
    phi, r = rng.uniform(0, 2 * np.pi, n), 30.0 + 40.0 * layer
    xyz = np.stack([r * np.cos(phi), r * np.sin(phi), rng.uniform(-1, 1, n) * g.z_half]).astype(np.float32)
    b = kf.hit_bin(g, 1, 1, to_dev(layer), to_dev(xyz), to_dev(rng.random((6, n)).astype(np.float32)),
                   event_offsets=to_dev(off))
    torch.cuda.synchronize()
    offsets, orig = host(b.offsets).reshape(E, 17, 2), host(b.orig)
    empty = np.setdiff1d(np.arange(E), used)
    assert np.array_equal(offsets[empty], np.broadcast_to(off[empty][:, None, None], (empty.size, 17, 2)))
    for e in used:
        sl = slice(off[e], off[e + 1])
        o = oracle.hit_bin(g, 1, 1, np.ascontiguousarray(layer[sl]), np.ascontiguousarray(xyz[:, sl]))
        assert np.array_equal(offsets[e].ravel() - off[e], np.asarray(o["offsets"]).ravel())
        assert np.array_equal(orig[sl], o["order"])

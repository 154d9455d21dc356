"""General hit_bin over bins of very uneven sizes (any order of the hits):
offsets and order bit-exact against the oracle where bins that are ranked
together hold from no hits to many times 64, for each number of lanes a bin
(mean bins below 8, below 16, and more), in shuffled input and in ordered
input that holds a bin too large for the grouped path."""
import numpy as np
import pytest

import oracle
from paper_1711_06571_amd import presets

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_common import host, to_dev  # noqa: E402

SIZES = [0, 1, 15, 16, 17, 0, 0, 700, 63, 64, 65, 2, 0, 2100, 33, 31, 1, 1, 1, 1, 130, 128, 129, 127]


@pytest.mark.parametrize("base", [0, 7, 20])
@pytest.mark.parametrize("shuffled", [True, False])
def test_uneven_bins(base, shuffled):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1711_06571_amd import kftrack as kf
    g, n_phi, n_z = presets.barrel(17), 63, 16
    rng = np.random.default_rng(base + shuffled)
    L, P, Z = [], [], []
    for l in (2, 16):
        for row in (0, 7, 15):
            for k, c in enumerate(SIZES):
                L.append(np.full(c, l))
                P.append((k + rng.uniform(0.05, 0.95, c)) * 2 * np.pi / n_phi)
                Z.append(np.full(c, -100 + (row + 0.5) * 200 / n_z))
    m = base * 17 * n_phi * n_z  # uniform hits below the uneven ones set the mean
    L.append(rng.integers(0, 17, m)); P.append(rng.uniform(0, 2 * np.pi, m)); Z.append(rng.uniform(-110, 110, m))
    layer, phi, z = (np.concatenate(a) for a in (L, P, Z))
    phi[rng.random(phi.shape[0]) < 0.01] = 2.5  # equal angles: the index decides
    n = layer.shape[0]
    perm = rng.permutation(n)
    if not shuffled:
        perm = perm[np.argsort(layer[perm], kind="stable")]
    layer = layer[perm].astype(np.int32)
    r = 4.0 * (layer + 1)
    xyz = np.stack([r * np.cos(phi[perm]), r * np.sin(phi[perm]), z[perm]]).astype(np.float32)
    cov = rng.random((6, n)).astype(np.float32)
    need = kf.hit_bin_workspace_bytes(1, 17, n_phi, n_z, n)
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    b = kf.hit_bin(g, n_phi, n_z, to_dev(layer), to_dev(xyz), to_dev(cov), ws=ws)
    torch.cuda.synchronize()
    assert int(ws[need - 256:need - 252].view(torch.int32).cpu()[0]) == 1
    o = oracle.hit_bin(g, n_phi, n_z, layer, xyz)
    assert np.array_equal(host(b.offsets)[0], o["offsets"])
    assert np.array_equal(host(b.orig), o["order"])
    assert np.array_equal(host(b.xyzphi)[3], o["phi"])
    assert np.array_equal(host(b.xyzphi)[:3], xyz[:, o["order"]])
    assert np.array_equal(host(b.cov), cov[:, o["order"]])

"""hit_bin with event offsets that do not tile the hits: the call goes to the
general path, which places every hit (in the event that the search of the
offsets gives) and keeps its arrays."""
import numpy as np
import pytest

from paper_1711_06571_amd import presets

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_common import host, to_dev  # noqa: E402


@pytest.mark.parametrize("eoff", [[0, 60, 20, 100], [0, 60, 60, 100], [7, 60, 80, 100], [0, 60, 80, 90],
                                  [0, 60, 80, 120], [-5, 60, 80, 100], [100, 0, 100, 0]])
def test_offsets_that_do_not_tile(eoff, monkeypatch):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1711_06571_amd import kftrack as kf
    monkeypatch.setenv("KFTRACK_HIT_BIN_PATH", "grouped")
    g, n, n_phi, n_z = presets.barrel(2), 100, 63, 16
    rng = np.random.default_rng(1)
    phi = rng.uniform(0, 2 * np.pi, n)
    xyz = np.stack([4 * np.cos(phi), 4 * np.sin(phi), rng.uniform(-90, 90, n)]).astype(np.float32)
    cov = rng.random((6, n)).astype(np.float32)
    need = kf.hit_bin_workspace_bytes(3, 2, n_phi, n_z, n)
    ws = torch.full((need,), 0x77, dtype=torch.uint8, device="cuda:0")  # (what an unwritten word would hold)
    b = kf.hit_bin(g, n_phi, n_z, to_dev(np.zeros(n, np.int32)), to_dev(xyz), to_dev(cov),
                   event_offsets=to_dev(np.asarray(eoff, np.int32)), ws=ws)
    torch.cuda.synchronize()
    tiling = eoff == [0, 60, 60, 100]
    assert int(ws[need - 256:need - 252].view(torch.int32).cpu()[0]) == (0 if tiling else 1)
    off = host(b.offsets)
    assert int(host(b.bad)[0]) == 0
    assert off.min() == 0 and off.max() == n and np.all(np.diff(off.ravel()) >= 0)
    got, ref = host(b.xyzphi)[:3], xyz
    assert np.array_equal(got[:, np.lexsort(got)], ref[:, np.lexsort(ref)])


def test_more_ranges_than_a_grid_of_parts_holds():
    """250 000 events of 17 layers, one bin each: 4.25 M ranges, which a block
    of 1 024 threads each would take past 2^32 threads."""
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1711_06571_amd import kftrack as kf
    g, E = presets.barrel(17), 250000
    off = (np.arange(E + 1) // 1000 * 40).astype(np.int32)  # 40 hits in every thousandth event
    n = int(off[-1])
    rng = np.random.default_rng(2)
    layer = np.sort(rng.integers(0, 17, (n // 40, 40)), axis=1).astype(np.int32).ravel()
    phi = rng.uniform(0, 2 * np.pi, n)
    r = 4.0 * (layer + 1)
    xyz = np.stack([r * np.cos(phi), r * np.sin(phi), rng.uniform(-90, 90, n)]).astype(np.float32)
    b = kf.hit_bin(g, 1, 1, to_dev(layer), to_dev(xyz), to_dev(rng.random((6, n)).astype(np.float32)),
                   event_offsets=to_dev(off))
    torch.cuda.synchronize()
    phi64 = np.arctan2(xyz[1].astype(np.float64), xyz[0].astype(np.float64))
    phi32 = np.where(phi64 < 0, phi64 + 2 * np.pi, phi64).astype(np.float32)
    ev = np.repeat(np.arange(n // 40) * 1000 + 999, 40)
    order = np.lexsort((phi32, layer, ev))
    assert np.array_equal(host(b.xyzphi)[:3], xyz[:, order])
    assert np.array_equal(host(b.orig), order - off[ev[order]])
    counts = np.bincount(ev.astype(np.int64) * 17 + layer, minlength=E * 17)
    start = np.concatenate([[0], np.cumsum(counts)])
    assert np.array_equal(host(b.offsets).reshape(-1, 2), np.stack([start[:-1], start[1:]], 1))

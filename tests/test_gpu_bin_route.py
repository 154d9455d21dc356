"""Which path sorts a binning, and that each gives the same arrays: the
grouped path's shapes (parts, staged and gathered, pieces of a bin, parts that
do not fit) each reported and bit-identical to the general path, and the
default choice by ranges and bins."""
import numpy as np
import pytest

from paper_1711_06571_amd import presets
from test_gpu_bin_parts import CASES

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_common import host, to_dev  # noqa: E402


@pytest.fixture
def kf():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1711_06571_amd import kftrack
    return kftrack


def _hits(counts, rng):
    n = int(np.sum(counts))
    layer = np.concatenate([np.repeat(np.arange(17), c) for c in counts]).astype(np.int32)
    phi, r = rng.uniform(0, 2 * np.pi, n), 4.0 * (layer + 1)
    phi[rng.random(n) < 0.02] = 1.25  # equal angles: the index decides
    xyz = np.stack([r * np.cos(phi), r * np.sin(phi), rng.uniform(-110, 110, n)]).astype(np.float32)
    off = np.concatenate([[0], np.cumsum([np.sum(c) for c in counts])]).astype(np.int32)
    return layer, xyz, rng.random((6, n)).astype(np.float32), off


def _bin(kf, monkeypatch, path, n_phi, n_z, layer, xyz, cov, off):
    if path:
        monkeypatch.setenv("KFTRACK_HIT_BIN_PATH", path)
    else:
        monkeypatch.delenv("KFTRACK_HIT_BIN_PATH", raising=False)
    g, E = presets.barrel(17), len(off) - 1
    need = kf.hit_bin_workspace_bytes(E, 17, n_phi, n_z, layer.shape[0])
    ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
    b = kf.hit_bin(g, n_phi, n_z, to_dev(layer), to_dev(xyz), to_dev(cov), event_offsets=to_dev(off), ws=ws)
    torch.cuda.synchronize()
    return b, int(ws[need - 256:need - 252].view(torch.int32).cpu()[0])


def _same(a, b):
    for k in ("offsets", "orig", "xyzphi", "cov", "bad"):
        assert np.array_equal(host(getattr(a, k)).view(np.int32), host(getattr(b, k)).view(np.int32)), k


# per event 17 counts, n_phi, n_z
GROUPED = dict(CASES)
GROUPED["large_edges"] = ([[0, 8191, 8192, 8193, 6783, 6784, 6785, 13568, 13569] + [9000] * 8], 63, 16)


@pytest.mark.parametrize("name", sorted(GROUPED))
def test_grouped_path_sorts_and_equals_the_general_path(kf, monkeypatch, name):
    counts, n_phi, n_z = GROUPED[name]
    h = _hits(counts, np.random.default_rng(3))
    a, grouped = _bin(kf, monkeypatch, "grouped", n_phi, n_z, *h)
    b, general = _bin(kf, monkeypatch, "general", n_phi, n_z, *h)
    assert (grouped, general) == (0, 1)
    _same(a, b)


@pytest.mark.parametrize("per,before,hot,threads", [(205000, 6600, 2000, 1024), (205000, 6600, 1500, 1024),
                                                    (4000, 1320, 800, 256), (4000, 1320, 700, 256)])
def test_part_above_its_memory_gives_way(kf, monkeypatch, per, before, hot, threads):
    """A part that ends in a bin of equal angles (one piece) holds the hits
    before the bin and all of the bin: above eight a thread the call goes to
    the general path."""
    rng = np.random.default_rng(4)
    layers = 17 if threads == 1024 else 1  # (3.5 M hits: parts of 6 613; 4 000 hits: parts of 1 333)
    counts = [[per] * layers + [0] * (17 - layers)]
    layer, _, cov, off = _hits(counts, rng)
    k = np.arange(layer.shape[0]) % per
    row = np.where(k < before + hot, 0, 1 + k % 15)
    cell = np.where(k < before, k % 10, np.where(k < before + hot, 10, k % 63))
    frac = np.where((k >= before) & (k < before + hot), 0.5, rng.uniform(0.05, 0.95, k.shape[0]))
    phi, r = (cell + frac) * 2 * np.pi / 63, 4.0 * (layer + 1)
    xyz = np.stack([r * np.cos(phi), r * np.sin(phi), -100 + (row + 0.5) * 12.5]).astype(np.float32)
    a, path = _bin(kf, monkeypatch, "grouped", 63, 16, layer, xyz, cov, off)
    assert path == (1 if before + hot > 8 * threads else 0)
    b, _ = _bin(kf, monkeypatch, "general", 63, 16, layer, xyz, cov, off)
    _same(a, b)


@pytest.mark.parametrize("events,per,n_phi,n_z,path", [
    (1, 20000, 63, 16, 1),   # few ranges, small bins
    (1, 20000, 8, 2, 0),     # bins of 1 250
    (1, 500, 63, 16, 1),
    (4, 3000, 63, 16, 1),
    (1, 60000, 63, 16, 1),   # bins of 60, but many
    (1, 15000, 63, 4, 0),    # bins of 60
    (16, 3000, 63, 16, 0),   # ranges for every CU
    (64, 100, 63, 16, 0),
    (64, 100, 4, 4, 1),      # few bins, few hits
    (64, 700, 4, 4, 0),
    (16, 1000, 128, 64, 1),  # more bins than the grouped path takes
])
def test_default_choice(kf, monkeypatch, events, per, n_phi, n_z, path):
    h = _hits([[per] * 17] * events, np.random.default_rng(5))
    a, got = _bin(kf, monkeypatch, None, n_phi, n_z, *h)
    assert got == path
    b, _ = _bin(kf, monkeypatch, "general", n_phi, n_z, *h)
    _same(a, b)
    perm = np.random.default_rng(6).permutation(h[0].shape[0] // events)  # any order: general, whatever the sizes
    if events == 1:
        _, got = _bin(kf, monkeypatch, None, n_phi, n_z, h[0][perm], np.ascontiguousarray(h[1][:, perm]),
                      np.ascontiguousarray(h[2][:, perm]), h[3])
        assert got == 1

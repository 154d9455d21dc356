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
    return b, int(ws[need - 252:need - 248].view(torch.int32).cpu()[0])


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
    (1, 500, 63, 16, 1),     # the smallest calls
    (1, 3500, 63, 16, 1),
    (1, 4000, 63, 16, 0),    # 68 000 hits
    (1, 20000, 63, 16, 0),
    (1, 20000, 8, 2, 0),
    (64, 30, 63, 16, 0),     # few hits, many bins
    (64, 30, 4, 4, 1),
    (64, 100, 4, 4, 1),      # few hits, few bins
    (64, 160, 4, 4, 0),
    (16, 1000, 128, 64, 1),  # more bins than the grouped path takes
])
def test_default_choice(kf, monkeypatch, events, per, n_phi, n_z, path):
    h = _hits([[per] * 17] * events, np.random.default_rng(5))
    a, got = _bin(kf, monkeypatch, None, n_phi, n_z, *h)
    assert got == path
    b, general = _bin(kf, monkeypatch, "general", n_phi, n_z, *h)
    assert general == 1
    _same(a, b)


@pytest.mark.parametrize("disorder", ["all", "one_block", "half", "bad"])
def test_large_calls_in_any_order(kf, monkeypatch, disorder):
    """Calls of 2^19 hits and more, whose blocks may count during the attempt:
    all, one or half of the blocks out of order, and bad hits among them."""
    layer, xyz, cov, off = _hits([[2100] * 17] * 16, np.random.default_rng(7))
    n = layer.shape[0]
    assert n >= 1 << 19
    rng = np.random.default_rng(8)
    perm = np.arange(n)
    if disorder == "one_block":  # within one event's hits
        perm[300:900] = 300 + rng.permutation(600)
        perm[[200, 20000]] = perm[[20000, 200]]
    else:
        for e in range(16 if disorder != "half" else 8):
            perm[off[e]:off[e + 1]] = off[e] + rng.permutation(off[e + 1] - off[e])
    layer, xyz, cov = layer[perm], np.ascontiguousarray(xyz[:, perm]), np.ascontiguousarray(cov[:, perm])
    n_bad = 0
    if disorder == "bad":
        i = rng.permutation(n)[:5000]
        layer[i[:2500]] = 17
        xyz[0, i[2500:]] = np.nan
        n_bad = 5000
    a, path = _bin(kf, monkeypatch, None, 63, 16, layer, xyz, cov, off)
    b, _ = _bin(kf, monkeypatch, "general", 63, 16, layer, xyz, cov, off)
    assert path == 1 and int(host(a.bad)[0]) == int(host(b.bad)[0]) == n_bad
    m = n - n_bad
    for k in ("offsets", "orig", "xyzphi", "cov"):
        x, y = host(getattr(a, k)), host(getattr(b, k))
        if k != "offsets":
            x, y = x[..., :m], y[..., :m]
        assert np.array_equal(x.view(np.int32), y.view(np.int32)), k
    for e in (0, 15):
        sl = slice(off[e], off[e + 1])
        import oracle
        ok = (layer[sl] < 17) & np.isfinite(xyz[0, sl])
        o = oracle.hit_bin(presets.barrel(17), 63, 16, np.ascontiguousarray(layer[sl]), np.ascontiguousarray(xyz[:, sl]))
        s0 = host(a.offsets)[e, 0, 0]
        assert np.array_equal(host(a.orig)[s0:s0 + int(ok.sum())], np.asarray(o["order"])[:int(ok.sum())])


def test_path_word_beside_the_reported_word(kf, monkeypatch):
    """The first of the two words reports the grouped path only for calls of
    six ranges a compute unit and forced ones; the second is the path."""
    layer, xyz, cov, off = _hits([[4000] * 17], np.random.default_rng(9))
    perm = np.random.default_rng(10).permutation(layer.shape[0])
    shuffled = (layer[perm], np.ascontiguousarray(xyz[:, perm]), np.ascontiguousarray(cov[:, perm]))
    need = kf.hit_bin_workspace_bytes(1, 17, 63, 16, layer.shape[0])
    for env, hits, words in ((None, (layer, xyz, cov), [1, 0]), ("grouped", (layer, xyz, cov), [0, 0]),
                             ("general", (layer, xyz, cov), [1, 1]), (None, shuffled, [1, 1]),
                             ("grouped", shuffled, [1, 1])):
        if env:
            monkeypatch.setenv("KFTRACK_HIT_BIN_PATH", env)
        else:
            monkeypatch.delenv("KFTRACK_HIT_BIN_PATH", raising=False)
        ws = torch.empty(need, dtype=torch.uint8, device="cuda:0")
        kf.hit_bin(presets.barrel(17), 63, 16, *(to_dev(h) for h in hits), ws=ws)
        torch.cuda.synchronize()
        assert ws[need - 256:need - 248].view(torch.int32).cpu().tolist() == words, env

"""Network gradient at the row counts where its split can go wrong: one row,
the ends of a 64-row block, and 15 to 33 blocks, whose partial gradients are
summed 16 at a time.  The exact sum over rows of one-row gradients (64-bit)
bounds the reordering; BF16 activations are the same in both."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

from gpu_common import host, to_dev  # noqa: E402
from test_gpu_mlp import _setup  # noqa: E402


@pytest.mark.parametrize("n", [1, 63, 64, 65, 960, 1024, 1025, 2049])
def test_gradient_is_the_mean_of_its_blocks(n, rng):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1711_06571_amd import kftrack as kf
    p, rows = _setup(rng, n)
    master = np.concatenate([p[k].ravel() for k in ("W1", "b1", "W2", "b2", "W3", "b3")]).astype(np.float32)
    blk = kf.mlp_block(master, p["mu"], p["sd"], p["scale"])
    g = host(kf.kf_mlp_grad(blk, to_dev(rows))).astype(np.float64)
    ref, size = np.zeros_like(g), np.zeros_like(g)
    for r in range(0, n, 64):
        part = rows[r:r + 64]
        d = host(kf.kf_mlp_grad(blk, to_dev(np.ascontiguousarray(part)))).astype(np.float64) * part.shape[0]
        ref += d
        size += np.abs(d)
    # one rounding per addition and two of the scale: (blocks + 4) ulp of the sum of magnitudes
    tol = ((n + 63) // 64 + 4) * 2.0 ** -24 * size / n
    assert np.all(np.abs(g - ref / n) <= tol)
    assert np.linalg.norm(g) > 0

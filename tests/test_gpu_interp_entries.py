"""The interpolation's entry kernels at the edges of a workgroup (32 points) and of a batch of
loads (8 entries), for channel counts with and without 16-byte groups: points that share sites,
points that share none, and one site crowded by every point, against the oracle."""
import numpy as np
import pytest

from test_gpu_interp import _check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("channels", [1, 3, 4, 104])
@pytest.mark.parametrize("m", [1, 2, 31, 32, 33, 257])
@pytest.mark.parametrize("spread", ["near", "far", "one"])
def test_entries(m, channels, spread):
    rng = np.random.default_rng(m + channels)
    grid = 24
    cells = np.stack(np.meshgrid(*[np.arange(grid)] * 3, indexing="ij"), -1).reshape(-1, 3)
    cells = cells[rng.permutation(len(cells))[:len(cells) // 2]]
    coords = np.concatenate([np.zeros((len(cells), 1), int), cells], 1)
    feats = rng.standard_normal((len(coords), channels))
    if spread == "near":
        pts = 6.0 + np.sort(rng.uniform(0, 4, m))[:, None] + rng.uniform(-1, 1, (m, 3))
    elif spread == "far":
        pts = rng.uniform(-2, grid + 2, (m, 3))
    else:
        pts = cells[0] + 0.5 + rng.uniform(-0.4, 0.4, (m, 3))
    _check(coords, grid, feats.astype(np.float32), pts.astype(np.float32), None,
           rng.standard_normal((m, channels)).astype(np.float32))

"""The fp32 feature gradient by every kernel that its cost model may pick (the fp32 matrix cores, the pair lists,
three bf16 parts) and by its own choice, against fp64: few and many rows, sparse and dense sites, channels in
multiples of 8, of 4 and of neither, generated output sites, one offset, cut tiles past 64 MiB of scratch."""
import numpy as np
import pytest
import torch

import paper_2111_07383_amd as ss
from test_gpu_gather_split import _dense, _inverse

pytestmark = pytest.mark.gpu

AUTO, PLAIN, PAIRS, NO_PAIRS, PARTS = 0, 3, 9, 10, 13
LAYERS = [(1, 8, 3, 1, 4, 8), (300, 32, 3, 1, 104, 104), (300, 32, 5, 1, 24, 24), (700, 20, 3, 2, 60, 120),
          (700, 20, 3, 2, 71, 45), (2000, 16, 3, 1, 8, 4), (2000, 16, 5, 1, 16, 36), (5000, 24, 1, 1, 40, 33),
          (7000, 20, 3, 1, 32, 64), (7000, 20, 3, 1, 13, 130), (25000, 36, 3, 1, 208, 208)]


@pytest.mark.parametrize("n,grid,ksize,stride,ci,co", LAYERS)
def test_routes(n, grid, ksize, stride, ci, co):
    """|error| <= (terms + 8) 2^-24 of the sum of magnitudes: at most a rounding per product on any path."""
    cells = np.sort(np.random.default_rng(n).permutation(grid ** 3)[:n])
    xyz = np.stack(np.unravel_index(cells, (grid,) * 3), 1)
    coords = torch.from_numpy(np.concatenate([np.zeros((n, 1)), xyz], 1).astype(np.int32)).cuda()
    rb = ss.build_rulebook(coords, grid, ksize, stride, stride == 1)
    g = torch.Generator("cuda").manual_seed(n)
    x = torch.randn((rb.n_in, ci), device="cuda", generator=g)
    dy = torch.randn((rb.n_out, co), device="cuda", generator=g)
    W = torch.randn((ksize ** 3, co, ci), device="cuda", generator=g)
    want, mag = _dense(dy, W.transpose(1, 2).contiguous(), _inverse(rb.neighbours(), rb.n_in))
    for variant in (AUTO, PLAIN, PAIRS, NO_PAIRS, PARTS):
        ss.debug_set(3, variant)
        try:
            dx = ss.backward(x, dy, rb, W, need_coeffs=False)[0]
        finally:
            ss.debug_set(3, 0)
        assert ((dx.double() - want).abs() <= (ksize ** 3 * co + 8) * 2.0 ** -24 * mag).all(), variant

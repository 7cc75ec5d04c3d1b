"""Infinities and NaN reach the sites that gather them and no others, in the forward and in the feature
gradient: rows lie next to each other in memory, also rows of different batch entries, and a kernel that
reads in pieces of 8 channels or chunks of 32 must not take a piece of the next one.

Channel counts leave every rest that the chunks know: 8 and 16 (shared by several offsets), 24 (padded),
none, and counts that are no multiple of 8."""
import numpy as np
import pytest
import torch

import paper_2111_07383_amd as ss

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,variant", [(torch.bfloat16, 0), (torch.float32, 0), (torch.float32, 13)])
@pytest.mark.parametrize("channels", [8, 16, 24, 45, 56, 88, 96, 120])
def test_only_the_neighbours(channels, dtype, variant):
    rng = np.random.default_rng(channels)
    cells = np.sort(rng.permutation(2 * 16 ** 3)[:1200])
    coords = np.stack(np.unravel_index(cells, (2, 16, 16, 16)), 1).astype(np.int32)
    rb = ss.build_rulebook(torch.from_numpy(coords).cuda(), 16, 3)
    nbr, n = rb.neighbours(), len(coords)
    g = torch.Generator("cuda").manual_seed(1)
    x = torch.randn((n, channels), device="cuda", generator=g).to(dtype)
    bad = torch.zeros(n, dtype=torch.bool, device="cuda")
    # first channels of a row (what follows the row before it), the first row of the second batch entry included
    rows = [1, 2, 300, 700, int(np.flatnonzero(coords[:, 0] == 1)[0])]
    for k, r in enumerate(rows):
        x[r, k % 8] = (float("nan"), float("inf"), -float("inf"))[k % 3]
        bad[r] = True
    touched = (bad[nbr.clamp(min=0).long()] & (nbr >= 0)).any(0)
    assert touched.any() and not touched.all()
    W = torch.randn((27, 33, channels), device="cuda", generator=g).to(dtype)
    Wt = torch.randn((27, channels, 33), device="cuda", generator=g).to(dtype)
    other = torch.randn((n, 33), device="cuda", generator=g).to(dtype)
    ss.debug_set(3, variant)
    try:
        y = ss.forward(x, rb, W)
        dx = ss.backward(other, x, rb, Wt, need_coeffs=False)[0]
    finally:
        ss.debug_set(3, 0)
    # (a submanifold layer gathers the same rows in both directions)
    for out in (y, dx):
        assert torch.equal(~torch.isfinite(out.float()).all(1), touched)

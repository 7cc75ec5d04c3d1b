"""ssconv_backward works in the workspace that the caller gives it: on the tile kernels (rows read in place,
padded or split; tiles cut between workgroups or not) it allocates nothing of its own."""
import numpy as np
import pytest
import torch

import paper_2111_07383_amd as ss

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,ci,co", [(torch.bfloat16, 64, 40), (torch.bfloat16, 71, 45), (torch.float32, 104, 96)])
@pytest.mark.parametrize("grads", [(True, True), (True, False), (False, True)])
@pytest.mark.parametrize("n,stride", [(700, 1), (7000, 1), (7000, 2)])
def test_allocates_nothing(dtype, ci, co, grads, n, stride):
    cells = np.sort(np.random.default_rng(n).permutation(20 ** 3)[:n])
    xyz = np.stack(np.unravel_index(cells, (20,) * 3), 1)
    coords = torch.from_numpy(np.concatenate([np.zeros((n, 1)), xyz], 1).astype(np.int32)).cuda()
    rb = ss.build_rulebook(coords, 20, 3, stride, stride == 1)
    desc = ss.basis_desc(((0, ci),), ((0, co),), 3, (0.0, 1.0))
    basis = torch.from_numpy(ss.basis_build(desc)).cuda()
    g = torch.Generator("cuda").manual_seed(n)
    x = torch.randn((rb.n_in, ci), device="cuda", generator=g).to(dtype)
    dy = torch.randn((rb.n_out, co), device="cuda", generator=g).to(dtype)
    W = torch.randn((27, co, ci), device="cuda", generator=g).to(dtype)
    # the tile kernel at every size in fp32
    ss.debug_set(3, 13 if dtype == torch.float32 else 0)
    try:
        run = lambda: ss.backward(x, dy, rb, W, desc, basis, need_feats=grads[0], need_coeffs=grads[1])  # noqa: E731
        want = run()
        ss.debug_set(2, 1)   # the next device allocation of the library fails
        got = run()
    finally:
        ss.debug_set(2, 0)
        ss.debug_set(3, 0)
    for a, b in zip(got, want):
        assert (a is None and b is None) or torch.equal(a, b)

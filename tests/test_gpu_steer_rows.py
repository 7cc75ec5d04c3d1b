"""Steering through rows staged in LDS against the kernels that address memory by field (features
off a 16-byte boundary): the same bits, at the edges of a workgroup's rows and for rows too wide
for LDS; also against the oracle."""
import numpy as np
import pytest

from test_gpu_steer import P, _check, torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fields", [((0, 3),), ((0, 2), (1, 2), (2, 1), (3, 1), (4, 1)), ((4, 2), (1, 1)),
                                    ((0, 16), (1, 16), (2, 8)), ((4, 250),)])
@pytest.mark.parametrize("n", [1, 3, 4, 5, 2050])
def test_staged_rows(n, fields):
    rng = np.random.default_rng(n)
    cells = np.stack(np.meshgrid(*[np.arange(16)] * 3, indexing="ij"), -1).reshape(-1, 3)
    coords = np.concatenate([np.zeros((n, 1)), cells[np.sort(rng.permutation(4096)[:n])]], 1).astype(np.int32)
    C = sum(m * (2 * l + 1) for l, m in fields)
    feats = rng.standard_normal((n, C)).astype(np.float32)
    q, _ = np.linalg.qr(rng.standard_normal((3, 3)))
    R = q * np.linalg.det(q)
    t = rng.uniform(-1, 1, 3)
    origin = (-8.0, -8.0, -8.0)
    c, f, r = _check(coords, feats, fields, R, t, 1, origin, 1.0, 16)
    off = torch.empty(feats.size + 1, device="cuda")[1:].view(feats.shape)
    off.copy_(torch.from_numpy(feats))
    c2, f2, r2 = P.steer(torch.from_numpy(coords).cuda(), off, fields, R, t, 1, origin, 1.0, 16)
    assert torch.equal(c, c2) and torch.equal(r, r2) and torch.equal(f, f2)

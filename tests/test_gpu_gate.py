"""The gate's kernels that stage rows through LDS against the ones that address memory by field
(taken for few rows and for arrays that start off a 16-byte boundary): the same bits, at the edges of a workgroup's
rows and at widths that just fit or exceed LDS; both against the oracle."""
import numpy as np
import pytest
import torch

import paper_2111_07383_amd as P
from oracle import conv as oc

pytestmark = pytest.mark.gpu

FIELDS = [((0, 5),), ((0, 3), (1, 2), (4, 1)), ((2, 1), (0, 1), (3, 2)), ((0, 32), (1, 32), (2, 16)), ((4, 50),),
          ((1, 300), (0, 7))]


def shifted(t):
    """The same values in memory that starts one element past a 16-byte boundary."""
    buf = torch.empty(t.numel() + 1, dtype=t.dtype, device=t.device)
    v = buf[1:].view(t.shape)
    v.copy_(t)
    assert v.data_ptr() % 16 != 0
    return v


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("fields", FIELDS)
@pytest.mark.parametrize("n", [1, 7, 8, 9, 4099])
def test_staged_rows(fields, n, dtype):
    C = sum(m * (2 * l + 1) for l, m in fields)
    G = sum(m for l, m in fields if l > 0)
    rng = np.random.default_rng(n)
    x = torch.from_numpy(rng.standard_normal((n, C + G)).astype(np.float32)).to("cuda", dtype)
    dy = torch.from_numpy(rng.standard_normal((n, C)).astype(np.float32)).to("cuda", dtype)
    x[0, 0] = float("nan")
    x[-1, -1] = float("inf")
    P.debug_set(3, 13)   # staged at any number of rows
    try:
        y, dx = P.gate_forward(fields, x), P.gate_backward(fields, x, dy)
    finally:
        P.debug_set(3, 0)
    assert torch.equal(y.view(torch.uint8), P.gate_forward(fields, shifted(x)).view(torch.uint8))
    assert torch.equal(dx.view(torch.uint8), P.gate_backward(fields, shifted(x), shifted(dy)).view(torch.uint8))
    # a few roundings of fp32 (the sigmoid's exponential), one rounding of the result's type
    eps = 2.0 ** -8 if dtype == torch.bfloat16 else 2.0 ** -20
    with np.errstate(invalid="ignore", over="ignore"):
        want = oc.gate_forward(x.double().cpu().numpy(), fields)
    rows = slice(1, n - 1)
    assert np.all(np.abs(y.double().cpu().numpy() - want)[rows] <= eps * np.abs(want[rows]) + 1e-30)

"""The fp32 output-stationary kernel on three bf16 parts per value, against the same sums in fp64.

Shapes sit at the edges of its tiles (64 / 128 / 256 rows, 16-column blocks, up to 128 columns a tile),
of its chunks (32 channels; rests of 8 and 16 shared by four and two offsets, a rest of 24 padded) and
of its cuts (whole tiles, tiles cut between workgroups)."""
import numpy as np
import pytest
import torch

import paper_2111_07383_amd as ss

pytestmark = pytest.mark.gpu


def _rulebook(n, ksize, stride=1, grid=24, seed=0):
    cells = np.random.default_rng(seed).permutation(grid ** 3)[:n]
    xyz = np.stack(np.unravel_index(np.sort(cells), (grid,) * 3), 1)
    coords = torch.from_numpy(np.concatenate([np.zeros((n, 1)), xyz], 1).astype(np.int32)).cuda()
    return ss.build_rulebook(coords, grid, ksize, stride, stride == 1)


def _dense(x, W, nbr):
    """(sum, sum of magnitudes) per output in fp64."""
    out = torch.zeros((nbr.shape[1], W.shape[1]), dtype=torch.float64, device=x.device)
    mag = torch.zeros_like(out)
    for s in range(W.shape[0]):
        o = (nbr[s] >= 0).nonzero()[:, 0]
        a, b = x.double()[nbr[s][o].long()], W[s].double().T
        out[o] += a @ b
        mag[o] += a.abs() @ b.abs()
    return out, mag


def _inverse(nbr, n_in):
    inv = torch.full((nbr.shape[0], n_in), -1, dtype=torch.int32, device=nbr.device)
    for s in range(nbr.shape[0]):
        o = (nbr[s] >= 0).nonzero()[:, 0]
        inv[s, nbr[s][o].long()] = o.int()
    return inv


SHAPES = [(1, 1, 1, 1, 1), (63, 3, 1, 8, 16), (65, 3, 1, 7, 3), (300, 3, 1, 24, 40), (257, 5, 1, 40, 113), (300, 5, 1, 16, 24), (129, 1, 1, 33, 17),
          (3000, 3, 1, 56, 128), (3000, 3, 2, 104, 129), (5000, 5, 1, 16, 96), (9000, 3, 1, 120, 60), (13000, 5, 1, 48, 256)]


@pytest.mark.parametrize("n,ksize,stride,ca,cb", SHAPES)
def test_against_fp64(n, ksize, stride, ca, cb):
    """Per output, |error| <= (2 chunks + 8) 2^-24 sum |a b|: each 32-channel chunk adds its low and its
    high products with one rounding each, the parts of a value leave less than 2^-24 of a product."""
    rb = _rulebook(n, ksize, stride)
    nbr = rb.neighbours()
    g = torch.Generator("cuda").manual_seed(1)
    x = torch.randn((rb.n_in, ca), device="cuda", generator=g)
    W = torch.randn((ksize ** 3, cb, ca), device="cuda", generator=g)
    dy = torch.randn((rb.n_out, cb), device="cuda", generator=g)
    ss.debug_set(3, 13)   # this kernel at every size, never the pair-list path
    try:
        y = ss.forward(x, rb, W)
        dx, _ = ss.backward(x, dy, rb, W, need_coeffs=False)
        y2 = ss.forward(x, rb, W)
    finally:
        ss.debug_set(3, 0)
    assert torch.equal(y, y2)
    for got, (want, mag), c in ((y, _dense(x, W, nbr), ca), (dx, _dense(dy, W.transpose(1, 2).contiguous(), _inverse(nbr, rb.n_in)), cb)):
        bound = (2 * ksize ** 3 * (c / 32 + 1) + 8) * 2.0 ** -24 * mag
        assert ((got.double() - want).abs() <= bound).all()


@pytest.mark.parametrize("n", [300, 4000])
def test_values_the_parts_cannot_carry(n):
    """Infinities, NaN, values above bf16's largest and below 2^-110 give what plain fp32 gives."""
    rb = _rulebook(n, 3)
    nbr = rb.neighbours()
    g = torch.Generator("cuda").manual_seed(2)
    x = torch.randn((n, 40), device="cuda", generator=g)
    W = torch.randn((27, 24, 40), device="cuda", generator=g)
    x[5, 3], x[17, 20], x[40, 39], x[90, 1] = float("inf"), -float("inf"), float("nan"), 3.4e38
    x[200:240] = 0
    W[:, 3] *= 1e-3
    x[210] = 1e-36 * torch.randn(40, device="cuda", generator=g)
    ss.debug_set(3, 13)
    try:
        y = ss.forward(x, rb, W)
    finally:
        ss.debug_set(3, 0)
    want, mag = _dense(x, W, nbr)
    f32 = want.float()
    assert torch.equal(torch.isnan(y), torch.isnan(f32))
    fine = ~torch.isnan(f32)
    assert torch.equal(torch.isinf(y[fine]), torch.isinf(f32[fine]))
    fine &= torch.isfinite(f32)
    bound = 27 * 40 * 2.0 ** -24 * mag + 1e-43
    assert ((y.double() - want).abs()[fine] <= bound[fine]).all()


@pytest.mark.parametrize("small", [-112, -120, -124, -140])
@pytest.mark.parametrize("where", ["rows", "kernel"])
def test_small_operands_keep_their_bits(where, small):
    """An operand so small that bf16 has no room for its third part, times one that brings the result back to
    ordinary size: the bound of the plain fp32 sums (a rounding per product), in both directions."""
    rb = _rulebook(700, 3)
    nbr = rb.neighbours()
    g = torch.Generator("cuda").manual_seed(3)
    x, W = torch.randn((700, 40), device="cuda", generator=g), torch.randn((27, 24, 40), device="cuda", generator=g)
    dy = torch.randn((700, 24), device="cuda", generator=g)
    big = min(-small - 8, 110)
    if where == "rows":
        x, dy, W = x * 2.0 ** small, dy * 2.0 ** small, W * 2.0 ** big
    else:
        x, dy, W = x * 2.0 ** big, dy * 2.0 ** big, W * 2.0 ** small
    ss.debug_set(3, 13)
    try:
        y = ss.forward(x, rb, W)
        dx = ss.backward(x, dy, rb, W, need_coeffs=False)[0]
    finally:
        ss.debug_set(3, 0)
    Wt = W.transpose(1, 2).contiguous()
    for got, (want, mag), c in ((y, _dense(x, W, nbr), 40), (dx, _dense(dy, Wt, _inverse(nbr, rb.n_in)), 24)):
        assert ((got.double() - want).abs() <= 27 * c * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("n", [300, 4000])
def test_whole_maps_of_them(n):
    """Every value infinite, NaN or past fp32's range in the sums: what the fp32 matrix cores' kernel gives."""
    rb = _rulebook(n, 3)
    g = torch.Generator("cuda").manual_seed(4)
    W, dy = torch.rand((27, 24, 40), device="cuda", generator=g) + 0.5, torch.rand((n, 24), device="cuda", generator=g) + 0.5
    for x in (torch.full((n, 40), float("nan"), device="cuda"), torch.full((n, 40), -float("inf"), device="cuda"),
              3e38 * torch.rand((n, 40), device="cuda", generator=g), 1e-37 * torch.rand((n, 40), device="cuda", generator=g)):
        out = []
        for variant in (13, 3):   # 3: the fp32 matrix cores
            ss.debug_set(3, variant)
            try:
                out.append((ss.forward(x, rb, W), ss.backward(x, dy * x[:, :24], rb, W, need_coeffs=False)[0]))
            finally:
                ss.debug_set(3, 0)
        for a, b in zip(*out):
            a, b = a.double().cpu().numpy(), b.double().cpu().numpy()
            np.testing.assert_allclose(a, b, rtol=27 * 40 * 2.0 ** -24, atol=0)   # (one sign of values)


def test_parts_down_to_their_limit():
    """Three parts carry every bit of a value from 2^-110 on (parts that are subnormal in bf16 count), and below
    it the plain kernel does: single products with a power of two are exact."""
    n = 4096
    rb = _rulebook(n, 1)
    g = torch.Generator("cuda").manual_seed(5)
    for lo, hi in ((-110, -96), (-126, -110), (100, 127)):
        e = torch.randint(lo, hi, (n, 8), device="cuda", generator=g)
        x = torch.ldexp(1 + torch.rand((n, 8), device="cuda", generator=g), e)
        W = 2.0 ** (-60 if lo > 0 else 60) * torch.eye(8, device="cuda")[None].contiguous()
        ss.debug_set(3, 13)
        try:
            y = ss.forward(x, rb, W)
        finally:
            ss.debug_set(3, 0)
        assert torch.equal(y, x * W[0, 0, 0])

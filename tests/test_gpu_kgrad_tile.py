"""The kernel gradient on the bf16 matrix cores (bf16 rows, or fp32 rows as three bf16 parts) and the bf16
gather at channel counts that are not multiples of 8, through the coefficient and feature gradients of
layers of scalar fields, against fp64.

Channel counts sit at the edges of its tiles (32, 64, 128 and 224 channels, more than one tile) and of the
padding of rows; pair counts at the edges of its 32-pair chunks and 512-pair blocks."""
import numpy as np
import pytest
import torch

import paper_2111_07383_amd as ss

pytestmark = pytest.mark.gpu


def _layer(n, ksize, ci, co, dtype, seed=0):
    rng = np.random.default_rng(seed)
    cells = np.sort(rng.permutation(20 ** 3)[:n])
    xyz = np.stack(np.unravel_index(cells, (20,) * 3), 1)
    coords = torch.from_numpy(np.concatenate([np.zeros((n, 1)), xyz], 1).astype(np.int32)).cuda()
    rb = ss.build_rulebook(coords, 20, ksize)
    desc = ss.basis_desc(((0, ci),), ((0, co),), ksize, tuple(float(m) for m in range(ksize // 2 + 1)))
    g = torch.Generator("cuda").manual_seed(seed)
    x = torch.randn((n, ci), device="cuda", generator=g).to(dtype)
    dy = torch.randn((n, co), device="cuda", generator=g).to(dtype)
    W = torch.randn((ksize ** 3, co, ci), device="cuda", generator=g).to(dtype)
    return rb, desc, torch.from_numpy(ss.basis_build(desc)).cuda(), x, dy, W


def _coeff_grad(rb, basis, nq, x, dy):
    """(sum, sum of magnitudes) of the coefficient gradient of a scalar layer in fp64."""
    nbr, K = rb.neighbours(), rb.K
    B = basis.double().reshape(nq, K)
    out = torch.zeros((dy.shape[1], x.shape[1], nq), dtype=torch.float64, device=x.device)
    mag = torch.zeros_like(out)
    for s in range(K):
        o = (nbr[s] >= 0).nonzero()[:, 0]
        a, b = dy[o].double(), x[nbr[s][o].long()].double()
        out += (a.T @ b)[:, :, None] * B[:, s]
        mag += (a.abs().T @ b.abs())[:, :, None] * B[:, s].abs()
    return out.reshape(-1), mag.reshape(-1)


# (fp32 layers of few pairs take the fp32 ring kernel)
CASES = [(1, 3, 1, 1), (33, 3, 5, 8), (200, 3, 40, 33), (7900, 3, 64, 65), (8000, 3, 71, 45), (2000, 5, 60, 128),
         (300, 5, 16, 24), (3000, 3, 129, 100), (7950, 3, 208, 225), (8000, 3, 2, 4)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,ksize,ci,co", CASES)
def test_coefficient_gradient(n, ksize, ci, co, dtype):
    """|error| <= (pairs / 32 + K + 64) 2^-24 of the sum of magnitudes: one rounding per 32 pairs and per
    offset and partial; products are exact (bf16) or kept to 2^-24 (three parts)."""
    rb, desc, basis, x, dy, W = _layer(n, ksize, ci, co, dtype)
    nq = ksize // 2 + 1
    gc = ss.backward(x, dy, rb, W, desc, basis, need_feats=False)[1]
    assert torch.equal(gc, ss.backward(x, dy, rb, W, desc, basis, need_feats=False)[1])
    want, mag = _coeff_grad(rb, basis, nq, x, dy)
    bound = (rb.pair_counts.max() / 32 + rb.K + 64) * 2.0 ** -24 * mag + 1e-30
    assert ((gc.double() - want).abs() <= bound).all()


@pytest.mark.parametrize("n,ksize,ci,co", CASES)
def test_bf16_ragged_forward_and_feature_gradient(n, ksize, ci, co):
    """bf16 outputs within one rounding (2^-8) of the value and the fp32 sum's error of the magnitudes."""
    rb, _, _, x, dy, W = _layer(n, ksize, ci, co, torch.bfloat16)
    nbr = rb.neighbours()
    y = ss.forward(x, rb, W)
    dx = ss.backward(x, dy, rb, W, need_coeffs=False)[0]
    for got, a, b in ((y, x, W), (dx, dy, W.flip(0).transpose(1, 2).contiguous())):
        want = torch.zeros((n, b.shape[1]), dtype=torch.float64, device="cuda")
        mag = torch.zeros_like(want)
        for s in range(rb.K):
            o = (nbr[s] >= 0).nonzero()[:, 0]
            r, k = a.double()[nbr[s][o].long()], b[s].double().T
            want[o] += r @ k
            mag[o] += r.abs() @ k.abs()
        assert ((got.double() - want).abs() <= 2.0 ** -8 * want.abs() + 2.0 ** -20 * mag).all()


def test_values_the_parts_cannot_carry():
    rb, desc, basis, x, dy, W = _layer(7900, 3, 24, 40, torch.float32)
    dy *= 1e-3   # sums with the value past bf16's largest stay below fp32's
    x[7, 3], x[90, 5], dy[11, 2] = float("inf"), 3.4e38, float("nan")
    gc = ss.backward(x, dy, rb, W, desc, basis, need_feats=False)[1]
    want = _coeff_grad(rb, basis, 2, x, dy)[0]
    fine = torch.isfinite(want.float())
    assert torch.equal(torch.isfinite(gc), fine)
    assert torch.equal(torch.isnan(gc), torch.isnan(want))
    assert fine.any() and not fine.all()


def _forced(f):
    """f() on the kernels on three bf16 parts at every size."""
    ss.debug_set(3, 13)
    try:
        return f()
    finally:
        ss.debug_set(3, 0)


# pairs per offset at the edges of the 32-pair chunks and 512-pair blocks; 3x3x3: empty and one-pair lists too
SPLIT = [(n, 1) for n in (1, 31, 32, 33, 511, 512, 513, 2000)] + [(2, 3), (40, 3), (1100, 3), (7900, 3)]


@pytest.mark.parametrize("scale", [(0, 0), (-120, 112), (100, -126)])
@pytest.mark.parametrize("ci,co", [(8, 5), (40, 33), (104, 120)])
@pytest.mark.parametrize("n,ksize", SPLIT)
def test_split_rows_keep_24_bits(n, ksize, ci, co, scale):
    """fp32 rows as three parts: a third part that is lost or taken from another place leaves 2^-18 of a product.
    Per entry |error| <= (roundings + K + 8) 2^-24 of the sum of magnitudes, with a rounding per 32 pairs (scaled
    values, which the fp32 matrix cores take over: per pair), which catches that up to some 30 pairs.  Over all
    entries the errors are random, and their root mean square stays under 2^-24 (0.3 + 1 / sqrt(pairs)) (0.6 with a
    rounding per pair): a running sum of n random terms is about 1 / sqrt(n) of their magnitudes, each rounding a
    third of a unit of it, and sqrt(roundings) of them add up."""
    rb, desc, basis, x, dy, W = _layer(n, ksize, ci, co, torch.float32, seed=n)
    x, dy = x * 2.0 ** scale[0], dy * 2.0 ** scale[1]
    gc = _forced(lambda: ss.backward(x, dy, rb, W, desc, basis, need_feats=False)[1])
    want, mag = _coeff_grad(rb, basis, ksize // 2 + 1, x, dy)
    err = (gc.double() - want).abs() / mag
    per, part = (32, 0.3) if scale == (0, 0) else (1, 0.6)
    assert (err <= (rb.pair_counts.max() / per + rb.K + 8) * 2.0 ** -24).all()
    assert err.square().mean().sqrt() <= 2.0 ** -24 * (part + max(rb.n_pairs, 1) ** -0.5)


def test_whole_maps_the_parts_cannot_carry():
    rb, desc, basis, x, dy, W = _layer(3000, 3, 24, 40, torch.float32)
    dy = dy.abs() + 0.5
    for v in (float("nan"), float("inf"), 3e36, 1e-37):
        y = (x.abs() + 0.5) * v
        run = lambda: ss.backward(y, dy, rb, W, desc, basis, need_feats=False)[1]  # noqa: E731
        got = _forced(run).double()
        ss.debug_set(3, 7)   # rows in registers, the fp32 matrix cores
        try:
            want = run().double()
        finally:
            ss.debug_set(3, 0)
        assert torch.equal(torch.isnan(got), torch.isnan(want)) and torch.equal(torch.isinf(got), torch.isinf(want))
        fine = torch.isfinite(want)
        assert ((got - want).abs()[fine] <= 2 * (3000 + 64) * 2.0 ** -24 * want.abs()[fine]).all()


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("ci,co", [(16, 24), (71, 45), (208, 225)])
def test_one_long_list(ci, co, dtype):
    """Isolated sites: the centre holds every pair, the other offsets none, so that one list is cut into most of
    the units.  The bound of the sums over 32 pairs."""
    cells = np.stack(np.meshgrid(*[np.arange(0, 40, 2)] * 3, indexing="ij"), -1).reshape(-1, 3)
    n = len(cells)
    coords = torch.from_numpy(np.concatenate([np.zeros((n, 1)), cells], 1).astype(np.int32)).cuda()
    rb = ss.build_rulebook(coords, 40, 3)
    assert rb.n_pairs == n
    desc = ss.basis_desc(((0, ci),), ((0, co),), 3, (0.0, 1.0))
    basis = torch.from_numpy(ss.basis_build(desc)).cuda()
    g = torch.Generator("cuda").manual_seed(0)
    x = torch.randn((n, ci), device="cuda", generator=g).to(dtype)
    dy = torch.randn((n, co), device="cuda", generator=g).to(dtype)
    W = torch.zeros((27, co, ci), device="cuda", dtype=dtype)
    gc = _forced(lambda: ss.backward(x, dy, rb, W, desc, basis, need_feats=False)[1])
    want, mag = _coeff_grad(rb, basis, 2, x, dy)
    assert ((gc.double() - want).abs() <= (n / 32 + rb.K + 64) * 2.0 ** -24 * mag).all()


@pytest.mark.parametrize("n,ksize,ci,co", CASES)
def test_bf16_tiles_at_every_count(n, ksize, ci, co):
    """Ragged bf16 layers of short lists, which the generic kernel takes otherwise."""
    rb, desc, basis, x, dy, W = _layer(n, ksize, ci, co, torch.bfloat16)
    gc = _forced(lambda: ss.backward(x, dy, rb, W, desc, basis, need_feats=False)[1])
    want, mag = _coeff_grad(rb, basis, ksize // 2 + 1, x, dy)
    assert ((gc.double() - want).abs() <= (rb.pair_counts.max() / 32 + rb.K + 64) * 2.0 ** -24 * mag + 1e-30).all()


@pytest.mark.parametrize("c", [8, 104])
def test_long_fp32_units_keep_their_precision(c):
    """13M pairs.  A rounding is of random sign and of about 0.4 2^-24 of a sum that grows along its run: 8 channels
    (ring kernel, 256 roundings between two folds) and 104 (tile kernel, one per 32 of 26k pairs) stay under 16 of
    2^-24 of the result, runs over a whole unit of 6500 pairs would be at 24 and more."""
    n, ksize = 48, 5
    ax = torch.arange(n, device="cuda", dtype=torch.int32)
    xyz = torch.cartesian_prod(ax, ax, ax)
    rb = ss.build_rulebook(torch.cat([torch.zeros_like(xyz[:, :1]), xyz], 1).contiguous(), n, ksize)
    assert rb.n_pairs > 12_000_000
    desc = ss.basis_desc(((0, c),), ((0, c),), ksize, (0.0, 1.0, 2.0))
    basis = torch.from_numpy(ss.basis_build(desc)).cuda()
    g = torch.Generator("cuda").manual_seed(7)
    x, dy = (torch.randn((n ** 3, c), device="cuda", generator=g) for _ in range(2))
    gc = ss.backward(x, dy, rb, torch.zeros((ksize ** 3, c, c), device="cuda"), desc, basis, need_feats=False)[1]
    want = _coeff_grad(rb, basis, 3, x, dy)[0]
    assert (gc.double() - want).norm() <= 16 * 2.0 ** -24 * want.norm()

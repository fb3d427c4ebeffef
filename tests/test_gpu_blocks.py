"""Column passes on both sides of the rule that picks their block size, and the
row and column passes at the lengths where the points per thread change
(L = 256 | 512 | 1024), against the oracle.

The rule: a view whose large column blocks (512 threads) would number fewer
than 256 takes small ones.  On 3-D plans the z pass sees n1 n2 columns and the
y pass n3 slices of n1, so both sides are reached by small plans.  Bars as in
the 3-D parity tests: product 1e-13 ||M||_inf ||z||_inf, FP64 preconditioner
1e-12 and FP32 2e-5 of the result's largest value.
"""

import numpy as np
import pytest
import torch

import oracle as O
from bars import assert_precond
from workloads.configs import domain_mask, SHAPES
from workloads.three_d import ellipsoid_mask

pytestmark = pytest.mark.gpu

rsfde = pytest.importorskip("paper_2102_11576_amd")
from paper_2102_11576_amd import RsfdePlan, make_opts  # noqa: E402

DEV = "cuda:0"


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), device=DEV).reshape(-1)


# z views of 8001 and 8255 columns (L = 128: large from 8161 on, 16 pairs a
# block); y views of 127 and 129 slices; L = 512 along y and z (8 pairs a
# block: large from 4081 columns on); the chirp form on both sides
@pytest.mark.parametrize("shape", [(127, 63, 63), (129, 64, 40), (65, 127, 63), (127, 15, 255),
                                   (31, 255, 15), (63, 65, 200), (17, 255, 255), (63, 255, 7)],
                         ids=lambda s: "x".join(map(str, s)))
def test_operators3_across_block_rule(shape):
    n1, n2, n3 = shape
    box = (0.0, 1.0, -0.1, 1.2, 0.2, 1.1)
    p = O.Problem3(n1, n2, n3, box, 1.55, 1.75, 1.85, 1.0, 0.8, 1.2, 1e-6, 1.0 / 16,
                   ellipsoid_mask(n1, n2, n3))
    rng = np.random.default_rng(n1 + 3 * n2 + 7 * n3)
    V = rng.standard_normal(p.shape)
    nm = 1.0 + p.d + 2 * sum(np.abs(c).sum() for c in (
        p.cx * O.toeplitz_first_column(p.alpha1, n1), p.cy * O.toeplitz_first_column(p.alpha2, n2),
        p.cz * O.toeplitz_first_column(p.alpha3, n3)))
    ref = O.precond3_apply(p, V)
    with RsfdePlan.setup3(shape, box, (p.alpha1, p.alpha2, p.alpha3), (p.kx, p.ky, p.kz),
                          torch.as_tensor(p.mask), p.eta, p.dt, 2) as pl:
        w = pl.matvec(_t(V)).cpu().numpy().reshape(p.shape)
        z64 = pl.precond(_t(V)).cpu().numpy().reshape(p.shape)
        z32 = pl.precond(_t(V), precision="fp32").cpu().numpy().reshape(p.shape)
    assert np.abs(w - O.matvec3(p, V)).max() <= 1e-13 * nm * np.abs(V).max()
    assert np.abs(z64 - ref).max() <= 1e-12 * np.abs(ref).max()
    assert np.abs(z32 - ref).max() <= 2e-5 * np.abs(ref).max()


# products: L = 2 next_pow2(n) per direction; chirp: L >= 2n - 1
@pytest.mark.parametrize("n1,n2", [(1, 1), (2, 4), (5, 3), (64, 65), (128, 129), (129, 256),
                                   (256, 257), (257, 513), (512, 128), (514, 300), (1024, 100),
                                   (3, 1025), (1, 300), (300, 1)])
def test_operators2_across_transform_lengths(n1, n2):
    box = (0.0, 1.0, 0.0, 1.0)
    mask = domain_mask(n1, n2, box, SHAPES["ellipse"](0.5, 0.5, 0.45, 0.3, 20.0))
    p = O.Problem(n1, n2, box, 1.4, 1.7, 1.0, 0.6, 1e-6, 1.0 / 16, mask)
    V = np.random.default_rng(n1 + 5 * n2).standard_normal((n2, n1))
    nm = 1.0 + p.d + 2 * np.abs(p.cx * O.toeplitz_first_column(p.alpha1, n1)).sum() \
        + 2 * np.abs(p.cy * O.toeplitz_first_column(p.alpha2, n2)).sum()
    with RsfdePlan(n1, n2, box, 1.4, 1.7, 1.0, 0.6, torch.as_tensor(mask), 1e-6, 1.0 / 16, 2) as pl:
        w = pl.matvec(_t(V)).cpu().numpy().reshape(n2, n1)
        z64 = pl.precond(_t(V)).cpu().numpy().reshape(n2, n1)
        z32 = pl.precond(_t(V), precision="fp32").cpu().numpy().reshape(n2, n1)
    assert np.abs(w - O.matvec(p, V)).max() <= 1e-13 * nm * np.abs(V).max()
    ref = O.precond_apply(p, V)
    assert_precond(z64, ref, p, "fp64")
    assert_precond(z32, ref, p, "fp32")


# Lines around the changes of the chirp transforms' lengths and form (n <= 2^k <
# n + 1; the symmetric form from 2049 points on, 4n = L at 4096), alone and mixed
# with the other forms, odd and even counts
@pytest.mark.parametrize("n1,n2", [(512, 513), (513, 512), (514, 33), (33, 515), (1023, 1000),
                                   (1024, 601), (1025, 701), (2048, 6), (2049, 5), (7, 2050),
                                   (2051, 514), (4096, 3), (2, 4096), (1, 600), (600, 1)])
def test_chirp_forms(n1, n2):
    box = (0.0, 1.0, 0.0, 1.0)
    mask = domain_mask(n1, n2, box, SHAPES["ellipse"](0.5, 0.5, 0.45, 0.3, 20.0))
    p = O.Problem(n1, n2, box, 1.4, 1.7, 1.0, 0.6, 1e-6, 1.0 / 16, mask)
    V = np.random.default_rng(n1 + 5 * n2).standard_normal((n2, n1))
    with RsfdePlan(n1, n2, box, 1.4, 1.7, 1.0, 0.6, torch.as_tensor(mask), 1e-6, 1.0 / 16, 2) as pl:
        z64 = pl.precond(_t(V)).cpu().numpy().reshape(n2, n1)
        z32 = pl.precond(_t(V), precision="fp32").cpu().numpy().reshape(n2, n1)
    ref = O.precond_apply_fft(p, V)
    assert_precond(z64, ref, p, "fp64")
    assert_precond(z32, ref, p, "fp32")


# Column pairs of the product with one load and store each: one column in all,
# an odd last column, rows that start at odd addresses; a z view of one column
# and of an odd number of columns
@pytest.mark.parametrize("shape", [(1, 5, 0), (2, 5, 0), (3, 1, 0), (511, 9, 0), (5, 2047, 0),
                                   (9, 4095, 0), (1, 1, 7), (1, 3, 5), (3, 3, 31), (7, 5, 1)],
                         ids=lambda s: "x".join(map(str, s)))
def test_matvec_column_pairs(shape):
    n1, n2, n3 = shape
    rng = np.random.default_rng(sum(shape))
    if n3:
        box = (0.0, 1.0, -0.1, 1.2, 0.2, 1.1)
        p = O.Problem3(n1, n2, n3, box, 1.55, 1.75, 1.85, 1.0, 0.8, 1.2, 1e-6, 1.0 / 16,
                       ellipsoid_mask(n1, n2, n3))
        pl = RsfdePlan.setup3(shape, box, (p.alpha1, p.alpha2, p.alpha3), (p.kx, p.ky, p.kz),
                              torch.as_tensor(p.mask), p.eta, p.dt, 2)
        V = rng.standard_normal(p.shape)
        ref, cols = O.matvec3(p, V), ((p.cx, p.alpha1, n1), (p.cy, p.alpha2, n2), (p.cz, p.alpha3, n3))
    else:
        box = (0.0, 1.0, 0.0, 1.0)
        mask = domain_mask(n1, n2, box, SHAPES["disk"](0.5, 0.5, 0.4))
        p = O.Problem(n1, n2, box, 1.4, 1.7, 1.0, 0.6, 1e-6, 1.0 / 16, mask)
        pl = RsfdePlan(n1, n2, box, 1.4, 1.7, 1.0, 0.6, torch.as_tensor(mask), 1e-6, 1.0 / 16, 2)
        V = rng.standard_normal((n2, n1))
        ref, cols = O.matvec(p, V), ((p.cx, p.alpha1, n1), (p.cy, p.alpha2, n2))
    nm = 1.0 + p.d + 2 * sum(np.abs(c * O.toeplitz_first_column(a, n)).sum() for c, a, n in cols)
    with pl:
        # an output 8 bytes off a 16-byte boundary, with guard values on both sides
        x, out = torch.zeros(V.size + 3, dtype=torch.float64, device=DEV), None
        x[1:1 + V.size] = _t(V)
        out = torch.full((V.size + 3,), 7.0, dtype=torch.float64, device=DEV)
        w = pl.matvec(x[1:1 + V.size], out[1:1 + V.size]).cpu().numpy().reshape(V.shape)
        g = out.cpu().numpy()
    assert np.abs(w - ref).max() <= 1e-13 * nm * np.abs(V).max()
    assert g[0] == 7.0 and g[-2] == 7.0 and g[-1] == 7.0


# The symmetric transform of 2048 points: 8 points per thread up to 1023 lines
# (511 in FP32), 16 beyond, in either direction, with an odd last row pair and
# column pair in both forms; and a product fused behind the last pass (a step)
@pytest.mark.parametrize("n1,n2", [(1023, 511), (511, 1023), (1023, 1023), (1023, 2047),
                                   (2047, 1023), (1023, 1), (1, 1023)])
def test_sine_transform_of_many_lines(n1, n2):
    box = (0.0, 1.0, 0.0, 1.0)
    mask = domain_mask(n1, n2, box, SHAPES["ellipse"](0.5, 0.5, 0.45, 0.3, 20.0))
    p = O.Problem(n1, n2, box, 1.4, 1.7, 1.0, 0.6, 1e-6, 1.0 / 16, mask)
    V = np.random.default_rng(n1 + 5 * n2).standard_normal((n2, n1))
    ref = O.precond_apply_fft(p, V)
    b = O.rhs(p, np.abs(V) * mask, O.F_LOGISTIC)
    with RsfdePlan(n1, n2, box, 1.4, 1.7, 1.0, 0.6, torch.as_tensor(mask), 1e-6, 1.0 / 16) as pl:
        z64 = pl.precond(_t(V)).cpu().numpy().reshape(n2, n1)
        z32 = pl.precond(_t(V), precision="fp32").cpu().numpy().reshape(n2, n1)
        outs = [pl.step(_t(np.abs(V) * mask), None, O.F_LOGISTIC,
                        make_opts(30, 10000, 1e-8, precision))[0].cpu().numpy().reshape(n2, n1)
                for precision in ("fp64", "fp32")]
    assert_precond(z64, ref, p, "fp64")
    assert_precond(z32, ref, p, "fp32")
    for u in outs:
        assert np.linalg.norm(b - O.matvec_fast(p, u)) <= (1e-8 + 1e-12) * np.linalg.norm(b)


# Row pass of the product with 2048 points: one transform per block up to 260 row
# pairs and beyond 512, two between
@pytest.mark.parametrize("n1,n2", [(520, 512), (1023, 513), (520, 520), (520, 521), (1023, 531),
                                   (520, 1024), (520, 1025)])
def test_matvec_row_blocks(n1, n2):
    box = (0.0, 1.0, 0.0, 1.0)
    mask = domain_mask(n1, n2, box, SHAPES["disk"](0.5, 0.5, 0.4))
    p = O.Problem(n1, n2, box, 1.4, 1.7, 1.0, 0.6, 1e-6, 1.0 / 16, mask)
    V = np.random.default_rng(n1 + n2).standard_normal((n2, n1))
    nm = 1.0 + p.d + 2 * np.abs(p.cx * O.toeplitz_first_column(p.alpha1, n1)).sum() \
        + 2 * np.abs(p.cy * O.toeplitz_first_column(p.alpha2, n2)).sum()
    with RsfdePlan(n1, n2, box, 1.4, 1.7, 1.0, 0.6, torch.as_tensor(mask), 1e-6, 1.0 / 16, 2) as pl:
        w = pl.matvec(_t(V)).cpu().numpy().reshape(n2, n1)
    assert np.abs(w - O.matvec(p, V)).max() <= 1e-13 * nm * np.abs(V).max()


# Axes of more than 2048 points on both sides of the number of lines from which the
# symmetric form is used: rows 129 (FP64) and 385 (FP32), columns 257 (FP64; any in
# FP32), with 4n = L in both directions and one direction in each form
@pytest.mark.parametrize("n1,n2", [(2050, 128), (2049, 129), (2051, 384), (4096, 385), (256, 2049),
                                   (257, 4096), (1, 2050), (2049, 1), (2049, 2050)])
def test_chirp_forms_across_line_rule(n1, n2):
    box = (0.0, 1.0, 0.0, 1.0)
    mask = domain_mask(n1, n2, box, SHAPES["ellipse"](0.5, 0.5, 0.45, 0.3, 20.0))
    p = O.Problem(n1, n2, box, 1.4, 1.7, 1.0, 0.6, 1e-6, 1.0 / 16, mask)
    V = np.random.default_rng(n1 + 5 * n2).standard_normal((n2, n1))
    with RsfdePlan(n1, n2, box, 1.4, 1.7, 1.0, 0.6, torch.as_tensor(mask), 1e-6, 1.0 / 16, 2) as pl:
        z64 = pl.precond(_t(V)).cpu().numpy().reshape(n2, n1)
        z32 = pl.precond(_t(V), precision="fp32").cpu().numpy().reshape(n2, n1)
    ref = O.precond_apply_fft(p, V)
    assert_precond(z64, ref, p, "fp64")
    assert_precond(z32, ref, p, "fp32")

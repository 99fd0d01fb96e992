"""The n - 1 coefficients of the cell records, bit for bit: sums of unrounded products K rho, one fused
multiply-add after the other in a fixed order.  Saved surrogates carry a checksum of these bits."""
from fractions import Fraction

import numpy as np
import pytest

from paper_1812_05902_amd import pbr

K = 2.26e-4


def _fma(a, b, c):
    return float(Fraction(a) * Fraction(b) + Fraction(c))  # exact, rounded once


def _record(d):
    """d[x + 2 y + 4 z]: densities at a cell's corners, as doubles."""
    d000, d100, d010, d110, d001, d101, d011, d111 = (float(v) for v in d)
    f000, f100, f010, f110 = (K * v for v in (d000, d100, d010, d110))

    def total(first, *terms):
        for sign, v in terms:
            first = _fma(sign * K, v, first)
        return first

    return [f000, total(-f000, (1, d100)), total(-f000, (1, d010)), total(-f000, (1, d001)),
            total(-f100, (1, d110), (-1, d010), (1, d000)), total(-f100, (1, d101), (-1, d001), (1, d000)),
            total(-f010, (1, d011), (-1, d001), (1, d000)),
            total(-f110, (1, d111), (-1, d101), (-1, d011), (1, d100), (1, d010), (1, d001), (-1, d000))]


def _records(rho):
    nz, ny, nx = rho.shape
    corners = np.stack([rho[z:nz - 1 + z, y:ny - 1 + y, x:nx - 1 + x] for z in (0, 1) for y in (0, 1) for x in (0, 1)], -1)
    return np.array([_record(d) for d in corners.reshape(-1, 8)]).reshape(nz - 1, ny - 1, nx - 1, 8).astype(np.float32)


def _rho(shape, levels):
    """Noise, or a few levels: corners of the same density leave the roundings of the products alone."""
    rng = np.random.default_rng(shape[2])
    return (rng.integers(0, levels, shape) * 0.1 + 1.2 if levels else rng.uniform(1.2, 1.21, shape)).astype(np.float32)


def test_the_order_of_the_sums_shows_in_the_bits():
    """Sums of rounded products give other records: the test below tells them apart."""
    rho = _rho((10, 9, 8), 2)
    want = _records(rho)
    f = K * rho.astype(np.float64)
    plain = (f[1:, 1:, 1:] - f[:-1, 1:, 1:] - f[1:, :-1, 1:] - f[1:, 1:, :-1] + f[:-1, :-1, 1:] + f[:-1, 1:, :-1] +
             f[1:, :-1, :-1] - f[:-1, :-1, :-1]).astype(np.float32)
    assert (plain != want[..., 7]).mean() > 0.1


@pytest.mark.gpu
@pytest.mark.parametrize("shape", [(2, 2, 2), (3, 2, 9), (10, 9, 8), (9, 10, 18)])
@pytest.mark.parametrize("levels", [0, 1, 2, 3])
def test_index_coefficients_bit_for_bit(shape, levels):
    rho = _rho(shape, levels)
    nz, ny, nx = shape
    r = pbr.Renderer(rays_per_chunk=256)
    r.set_density_field(rho, (0.0, 0.0, 0.0), (1e-4,) * 3, K, 1.2)
    r.torch.cuda.synchronize()
    got = r.ws[:(nx - 1) * (ny - 1) * (nz - 1) * 32].cpu().numpy().reshape(nz - 1, ny - 1, nx - 1, 8, 4)
    assert np.array_equal(got[..., 0], _records(rho))

"""The prepared field itself, both layouts, against its definition in double rounded once to float32:
grids smaller than a brick of 8^3 cells, exactly one, one cell beyond, ragged and with two-node axes."""
import numpy as np
import pytest

from paper_1812_05902_amd import pbr

pytestmark = pytest.mark.gpu

K, SPACING = 2.26e-4, (1.37e-4, 2.11e-4, 3.3e-4)


def _gradient(rho, ax):
    v = np.moveaxis(rho, ax, 0)
    d = np.empty_like(v)
    if len(v) == 2:
        d[:] = v[1] - v[0]
    else:
        d[1:-1] = 0.5 * (v[2:] - v[:-2])
        d[0] = -1.5 * v[0] + 2.0 * v[1] - 0.5 * v[2]
        d[-1] = 1.5 * v[-1] - 2.0 * v[-2] + 0.5 * v[-3]
    return np.moveaxis(d, 0, ax)


@pytest.mark.parametrize("shape", [(2, 2, 2), (3, 2, 9), (9, 9, 9), (10, 9, 8), (10, 17, 33), (34, 26, 2), (65, 64, 63)])
@pytest.mark.parametrize("levels", [0, 3], ids=["noise", "levels"])
def test_field_records(shape, levels):
    nz, ny, nx = shape
    rng = np.random.default_rng(nx + 10 * ny)
    rho = (rng.integers(0, levels, shape) * 0.1 + 1.2 if levels else rng.uniform(1.2, 1.21, shape)).astype(np.float32)
    d = rho.astype(np.float64)
    q = [K * d] + [(K / SPACING[a]) * _gradient(d, 2 - a) for a in range(3)]
    for nodes in (True, False):
        r = pbr.Renderer(rays_per_chunk=4096)
        r.set_density_field(rho, (0.0, 0.1, 0.2), SPACING, K, 1.2, nodes=nodes)
        r.torch.cuda.synchronize()
        if nodes:
            got = r.ws[:nx * ny * nz * 4].cpu().numpy().reshape(nz, ny, nx, 4)
            for m in range(4):
                assert np.array_equal(got[..., m], q[m].astype(np.float32))
            continue
        got = r.ws[:(nx - 1) * (ny - 1) * (nz - 1) * 32].cpu().numpy().reshape(nz - 1, ny - 1, nx - 1, 8, 4)
        for m in range(4):
            def f(x, y, z):
                return q[m][z:nz - 1 + z, y:ny - 1 + y, x:nx - 1 + x]
            c = [f(0, 0, 0), f(1, 0, 0) - f(0, 0, 0), f(0, 1, 0) - f(0, 0, 0), f(0, 0, 1) - f(0, 0, 0),
                 f(1, 1, 0) - f(1, 0, 0) - f(0, 1, 0) + f(0, 0, 0), f(1, 0, 1) - f(1, 0, 0) - f(0, 0, 1) + f(0, 0, 0),
                 f(0, 1, 1) - f(0, 1, 0) - f(0, 0, 1) + f(0, 0, 0),
                 f(1, 1, 1) - f(1, 1, 0) - f(1, 0, 1) - f(0, 1, 1) + f(1, 0, 0) + f(0, 1, 0) + f(0, 0, 1) - f(0, 0, 0)]
            for e in range(8):
                want = c[e].astype(np.float32)
                if m:  # the gradients' sums take the rounded products
                    assert np.array_equal(got[..., e, m], want), (m, e)
                else:  # n - 1: unrounded products, up to eight half-ulps of K rho apart before the rounding
                    assert np.abs(got[..., e, 0].astype(np.float64) - want).max() <= 8 * 2.0 ** -54 * 2.9e-4 + \
                        2.0 ** -24 * np.abs(want).max() * (e > 0)


def test_brick_steepness_is_the_largest_gradient_at_its_nodes():
    """pbr_calibrate_precision's threshold comes from the bricks' largest |grad n|."""
    shape = (20, 17, 26)
    rng = np.random.default_rng(1)
    rho = np.full(shape, 1.2, np.float32)
    rho[9:12, 3:6, 17:20] = rng.uniform(1.2, 1.4, (3, 3, 3)).astype(np.float32)
    d = rho.astype(np.float64)
    g = np.sqrt(sum(((K / SPACING[a]) * _gradient(d, 2 - a)) ** 2 for a in range(3)))
    r = pbr.Renderer(rays_per_chunk=4096)
    org = (-12.5 * SPACING[0], -8 * SPACING[1], 0.0)
    r.set_density_field(rho, org, SPACING, K, 1.2)
    r.set_optics(0.5, 0.05, 8.0)
    r.set_sensor(64, 64, 2e-5)
    rep = r.calibrate_precision(1e-4, steep_frac=0.0)
    nb = [-(-(n - 1) // 8) for n in shape]
    steep = sum(bool((g[8 * z:8 * z + 9, 8 * y:8 * y + 9, 8 * x:8 * x + 9] > 0).any())
                for z in range(nb[0]) for y in range(nb[1]) for x in range(nb[2]))
    assert rep["n_bricks"] == int(np.prod(nb)) and rep["n_steep"] == steep
    assert rep["grad_max"] == float(np.float32(g.max()))

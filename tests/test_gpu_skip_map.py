"""The map of uniform gas (distance to the nearest brick with a gradient, run of uniform columns towards +z)
against its definition, below and above the size at which one block builds it."""
import numpy as np
import pytest

from paper_1812_05902_amd import pbr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bricks", [(1, 1, 1), (3, 2, 5), (1, 1, 300), (64, 64, 1), (16, 16, 16), (16, 17, 16), (1, 2, 2100),
                                    (70, 61, 1)])  # along x, y, z; 4096 is the largest of one block
@pytest.mark.parametrize("marks", [0, 1, 9])
def test_words_of_the_map(bricks, marks):
    bx, by, bz = bricks
    rng = np.random.default_rng(bx + 7 * marks)
    rho = np.full((8 * bz + 1, 8 * by, 8 * bx + 1), 1.2, np.float32)  # the last bricks along y are cut
    for _ in range(marks):
        z, y, x = (8 * rng.integers(0, b) + 3 for b in (bz, by, bx))
        rho[z:z + 2, y:y + 2, x:x + 2] = 1.3
    d = rho.astype(np.float64)
    grad = sum(np.abs(np.gradient(d, axis=a)) for a in range(3)) > 0
    has = np.array([[[grad[8 * k:8 * k + 9, 8 * j:8 * j + 9, 8 * i:8 * i + 9].any() for i in range(bx)] for j in range(by)]
                    for k in range(bz)])
    at = np.argwhere(has)
    q = np.indices(has.shape).reshape(3, -1).T
    dist = np.full(len(q), 127)
    for m in at:
        dist = np.minimum(dist, np.abs(q - m).max(1))
    dist = dist.reshape(has.shape)
    pad = np.pad(has, ((0, 0), (1, 1), (1, 1)))
    shut = sum(pad[:, 1 + j:1 + j + by, 1 + i:1 + i + bx] for j in (-1, 0, 1) for i in (-1, 0, 1)) > 0
    run = np.zeros(has.shape, np.int64)
    for k in range(bz - 1, -1, -1):
        run[k] = np.where(shut[k], 0, 1 + (run[k + 1] if k + 1 < bz else 0))
    r = pbr.Renderer(rays_per_chunk=256)
    r.set_density_field(rho, (0.0, 0.0, 0.0), (1e-4,) * 3, 2.26e-4, 1.2, nodes=True)
    r.torch.cuda.synchronize()
    off = (rho.size * 16 + 255) // 256 * 64
    word = r.ws[off:off + has.size].cpu().numpy().view(np.uint32).reshape(has.shape)
    want = 0x80000000 + (run << 8) + dist
    assert np.array_equal(word[~has], want[~has].astype(np.uint32))
    assert (word[has].view(np.float32) > 0).all()
    assert not r.brick_flags().any()  # their bytes serve as scratch

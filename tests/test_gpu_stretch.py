"""Runs of steps through gas without a gradient where there is no map of it to look at (FP64 flags of the
caller's own on such gas): as long as anywhere else."""
import numpy as np
import pytest

from paper_1812_05902_amd import inputs, pbr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nodes", [False, True], ids=["cells", "nodes"])
def test_runs_without_a_map_are_not_cut(nodes):
    sc = inputs.tomo_piv_shock(n=129, n_src=2000, rays_per_src=100)
    src = inputs.sources(sc)
    uniform = np.full((sc.nz, sc.ny, sc.nx), 1.2, np.float32)
    ms = []
    for rho in (None, uniform):  # None: the shock, uniform gas on either side
        r = pbr.Renderer.from_scene(sc, rho=rho, nodes=nodes)
        f = r.brick_flags()
        f[0] = 1  # one brick in a corner
        r.brick_flags(f)
        ms.append(min(r.emit_and_trace(src, sc.rays_per_src, sc.ray_seed, sc.ds, pbr.PBR_CLEAR_FIRST |
                                       pbr.PBR_PREC_SHOCK_FP64, stats=True)["box_ms"] for _ in range(5)))
        r.close()
    print(f"{ms[0]:.3f} ms with the shock, {ms[1]:.3f} ms without")
    # the same steps; where those in uniform gas are cut to four at a time, each run waits for the rays of
    # its wave that are not: 2.4 to 3 times as long
    assert ms[0] < 1.5 * ms[1]

"""Uniform gas beside a gradient, few rays: a render is not held up by the rays that have nothing to integrate.
The same image with a slight slope everywhere, where every step is taken, takes at least as long."""
import numpy as np
import pytest

from paper_1812_05902_amd import inputs, pbr

pytestmark = pytest.mark.gpu


def _scene(kind):
    if kind == "shock":
        sc = inputs.tomo_piv_shock(n=195, n_src=2000, rays_per_src=100)
    else:  # a bump far narrower than the box: uniform to the rounding of its density towards the corners
        sc = inputs.tiny_bos().replace(nx=100, ny=100, nz=100, origin=(-0.025, -0.025, 0.1), spacing=(0.05 / 99,) * 3,
                                       n_src=300, rays_per_src=50,
                                       field_params=dict(rho0=1.2, amp=0.1, sigma=0.006, centre=(0.0, 0.0, 0.125)))
    return sc, inputs.density(sc)


@pytest.mark.parametrize("kind", ["shock", "bump"])
def test_calm_rays_do_not_hold_up_their_wave(kind):
    sc, rho = _scene(kind)
    src = inputs.sources(sc)
    slope = rho + np.float32(2e-4) * np.arange(sc.nz, dtype=np.float32)[:, None, None]
    ms = []
    for field in (rho, slope):
        r = pbr.Renderer.from_scene(sc, rho=field, nodes=True)
        r.set_source_order(r.morton_order(src))
        ms.append(min(r.emit_and_trace(src, sc.rays_per_src, sc.ray_seed, sc.ds, pbr.PBR_CLEAR_FIRST | pbr.PBR_SOURCE_ORDER,
                                       stats=True)["box_ms"] for _ in range(8)))
        r.close()
    print(f"{kind}: {ms[0]:.3f} ms, {ms[1]:.3f} ms with a slope everywhere")
    # looking for uniform gas every four steps, or jumping a few steps at a time, made it 1.3 to 1.5 times as long
    assert ms[0] < 1.2 * ms[1]

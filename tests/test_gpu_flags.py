"""FP64 flags that a caller saves and writes back are the calibration's flags: a render with them takes the
uniform gas at once as before."""
import pytest

from paper_1812_05902_amd import inputs, pbr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nodes", [False, True], ids=["cells", "nodes"])
def test_restored_flags_keep_the_skip_through_uniform_gas(nodes):
    sc = inputs.tomo_piv_shock(n=129, n_src=2000, rays_per_src=100)
    src = inputs.sources(sc)
    r = pbr.Renderer.from_scene(sc, nodes=nodes)
    r.calibrate_precision(sc.ds, tol_px=1e-7, steep_frac=0.1)
    flags = r.brick_flags()
    assert 0 < flags.sum() < flags.size

    def render():
        runs = []
        for _ in range(4):
            st = r.emit_and_trace(src, sc.rays_per_src, sc.ray_seed, sc.ds,
                                  pbr.PBR_CLEAR_FIRST | pbr.PBR_PREC_SHOCK_FP64, stats=True)
            runs.append(st["box_ms"])
        return pbr.u64_image_to_numpy(r.read_image()), st, min(runs)

    image, st, ms = render()
    r.brick_flags(flags)
    image2, st2, ms2 = render()
    print(f"{ms:.3f} ms with the calibration's flags, {ms2:.3f} ms with the same flags restored")
    assert (image2 == image).all()
    assert st2["rkn_steps_fp64"] == st["rkn_steps_fp64"] > 0 and st2["rkn_steps"] == st["rkn_steps"]
    assert ms2 < 2.0 * ms  # stepping through the gas on either side of the shock takes 3.5 times as long

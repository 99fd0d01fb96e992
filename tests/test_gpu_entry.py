"""GPU parity of rays at the edges of the integration's cell search: rays that enter through the side
faces of the box (on the upper faces the state starts at fraction 1 of the last cell) and run along
them, in both field layouts, FP32, FP64 and calibrated mixed precision, against the FP64 oracle."""
import numpy as np
import pytest

import oracle
from paper_1812_05902_amd import inputs, pbr

pytestmark = pytest.mark.gpu

# FP32: stage points are rounded to 2^-24 cells (7.5e-12 m here) and the direction's accumulated change
# to 2^-24 of itself; over 100 steps of 1e-4 m that is below 1e-10 m and 1e-10 rad, i.e. 1e-6 px at
# M / pitch = 1.2e4 px/m over the 0.25 m to the dots.  A lost fraction of the entry cell is 1e-5 px or more.
BARS = {0: 5e-6, pbr.PBR_PREC_FP64_ALL: 1e-7, pbr.PBR_PREC_SHOCK_FP64: 5e-6}


@pytest.mark.parametrize("nodes", [False, True], ids=["cells", "nodes"])
@pytest.mark.parametrize("flags", list(BARS), ids=["fp32", "fp64", "mixed"])
def test_rays_entering_through_the_side_faces(nodes, flags):
    sc = inputs.bos_slice(n=129, n_src=400, rays_per_src=16)
    rng = np.random.default_rng(21)
    src = np.zeros((sc.n_src, 4), np.float32)
    edge = rng.uniform(0.0210, 0.0218, sc.n_src)  # their rays reach |x| = 16 mm inside the box's depth
    other = rng.uniform(-0.02, 0.02, sc.n_src)
    side = np.arange(sc.n_src) % 4
    src[:, 0] = np.where(side == 0, edge, np.where(side == 1, -edge, other))
    src[:, 1] = np.where(side == 2, edge, np.where(side == 3, -edge, other))
    src[:, 3] = 1.0
    r = pbr.Renderer.from_scene(sc, nodes=nodes)
    if flags == pbr.PBR_PREC_SHOCK_FP64:
        f = r.brick_flags()
        f[::2] = 1  # every other brick along x
        r.brick_flags(f)
    r.set_exit_recording(0, 1, sc.n_rays)
    st = r.emit_and_trace(src, sc.rays_per_src, 5, sc.ds, flags | pbr.PBR_CLEAR_FIRST | pbr.PBR_RECORD_EXITS,
                          stats=True)
    got = r.read_ray_exits()
    ref = oracle.scene_oracle(sc.replace(ray_seed=5)).trace_ids(src, sc.rays_per_src, np.arange(sc.n_rays))
    assert np.array_equal(got["entered"], ref["entered"])
    lo = np.asarray(sc.origin)
    hi = np.asarray(sc.box_max())
    both = (got["status"] == 0) & (ref["status"] == 0) & (got["entered"] == 1)
    assert (got["status"] != ref["status"]).sum() <= 1
    assert both.sum() > 500
    on_side = (np.abs(ref["n_steps"][both] * sc.ds - (hi[2] - lo[2])) > 2 * sc.ds).sum()
    assert on_side > 200  # entered or left through a side face
    assert np.abs(got["n_steps"][both] - ref["n_steps"][both]).max() <= 1
    err = np.abs(got["sensor_px"][both] - ref["sensor_px"][both]).max()
    print(f"{both.sum()} rays, {on_side} with a side face: max |dpx| {err:.2e}, {st['rkn_steps_fp64']} FP64 steps")
    assert err <= BARS[flags]

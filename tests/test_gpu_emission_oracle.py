"""Rays that the integration kernels emit themselves, each kernel of them (FP32, FP64, mixed precision with some
bricks in FP64; both layouts) and the emission kernel (lane refill), against the FP64 oracle's rays: dots behind
the box, particles inside it, sources whose rays miss it."""
import numpy as np
import pytest

import oracle
from paper_1812_05902_amd import inputs, pbr

pytestmark = pytest.mark.gpu

MIXED = pbr.PBR_PREC_SHOCK_FP64
CASES = [(n, f) for n in ("cells", "nodes") for f in (0, pbr.PBR_PREC_FP64_ALL, MIXED)] + [("cells", pbr.PBR_LANE_REFILL)]


@pytest.mark.parametrize("layout,flags", CASES)
def test_emitted_rays_against_the_oracle(layout, flags):
    sc = inputs.tiny_bos().replace(n_src=60, rays_per_src=13)
    lo, hi = np.asarray(sc.origin), np.asarray(sc.box_max())
    rng = np.random.default_rng(4)
    src = inputs.sources(sc)
    src[20:40, :3] = rng.uniform(lo + 0.1 * (hi - lo), hi - 0.1 * (hi - lo), (20, 3))  # inside the box
    src[40:, 0] = hi[0] + 10 * (hi[0] - lo[0])  # beside it: their rays pass the box
    r = pbr.Renderer.from_scene(sc, rays_per_chunk=300, nodes=layout == "nodes")
    if flags == MIXED:
        f = r.brick_flags()
        f[::2] = 1
        r.brick_flags(f)
    r.set_exit_recording(0, 1, sc.n_rays)
    st = r.emit_and_trace(src, sc.rays_per_src, sc.ray_seed, sc.ds, pbr.PBR_CLEAR_FIRST | pbr.PBR_RECORD_EXITS | flags,
                          stats=True)
    got = r.read_ray_exits()
    ref = oracle.scene_oracle(sc).trace_ids(src, sc.rays_per_src, np.arange(sc.n_rays))
    assert st["rkn_steps"] > 0
    if flags == MIXED:
        assert 0 < st["rkn_steps_fp64"] < st["rkn_steps"]
    else:
        assert st["rkn_steps_fp64"] == (st["rkn_steps"] if flags == pbr.PBR_PREC_FP64_ALL else 0)
    assert np.array_equal(got["entered"], ref["entered"]) and np.array_equal(got["status"], ref["status"])
    ent = ref["entered"] == 1
    assert ent.sum() == 40 * 13
    # beside the box: straight from the source, both in FP64, the direction held as a pair of floats (2^-48)
    assert np.abs(got["vol_exit_pos"] - ref["vol_exit_pos"])[~ent].max() <= 1e-15
    assert np.abs(got["vol_exit_dir"] - ref["vol_exit_dir"])[~ent].max() <= 1e-14
    # inside: the field's values are floats, 2^-24 of the bend (below 1e-3 rad) over 0.05 m; FP32 steps also
    # round each increment three times, 1.8e-7 of a way across the axis below 0.1 x 0.05 m
    pos, ang = (3e-12, 6e-11) if flags == pbr.PBR_PREC_FP64_ALL else (9e-10, 2e-10)
    dx = np.abs(got["vol_exit_pos"] - ref["vol_exit_pos"])[ent].max()
    du = np.abs(got["vol_exit_dir"] - ref["vol_exit_dir"])[ent].max()
    both = ent & (ref["status"] == oracle.DEPOSITED)
    px = np.abs(got["sensor_px"] - ref["sensor_px"])[both].max()
    print(f"{layout}, flags {flags}: |dx| {dx:.1e} m, |du| {du:.1e}, |dpx| {px:.1e} of {both.sum()} rays")
    assert dx <= pos and du <= ang
    # M / pitch below 1e4 px/m at the focused plane, 0.15 m at most from where a ray leaves the box
    assert both.sum() > 300 and px <= 1e4 * (pos + 0.15 * ang)

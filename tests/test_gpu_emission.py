"""Rays emitted by the integration kernels themselves and by the emission kernel (lane refill) are the same
rays, wherever they start: dots behind the box, particles inside it, sources whose rays miss it."""
import numpy as np
import pytest

import oracle
from paper_1812_05902_amd import inputs, pbr

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nodes", [False, True], ids=["cells", "nodes"])
@pytest.mark.parametrize("flags", [0, pbr.PBR_PREC_FP64_ALL, pbr.PBR_PREC_SHOCK_FP64], ids=["fp32", "fp64", "mixed"])
def test_states_do_not_depend_on_where_rays_are_emitted(flags, nodes):
    sc = inputs.tiny_bos().replace(n_src=60, rays_per_src=13)
    lo, hi = np.asarray(sc.origin), np.asarray(sc.box_max())
    rng = np.random.default_rng(4)
    src = inputs.sources(sc)
    src[20:40, :3] = rng.uniform(lo + 0.1 * (hi - lo), hi - 0.1 * (hi - lo), (20, 3))  # inside the box
    src[40:, 0] = hi[0] + 10 * (hi[0] - lo[0])  # beside it: their rays pass the box
    runs = [(1 << 16, 0), (64, 0), (77, 0)]
    if flags == 0 and not nodes:
        runs.append((100, pbr.PBR_LANE_REFILL))
    out = []
    for chunk, extra in runs:
        r = pbr.Renderer.from_scene(sc, rays_per_chunk=chunk, nodes=nodes)
        r.set_exit_recording(0, 1, sc.n_rays)
        st = r.emit_and_trace(src, sc.rays_per_src, sc.ray_seed, sc.ds,
                              pbr.PBR_CLEAR_FIRST | pbr.PBR_RECORD_EXITS | flags | extra, stats=True)
        out.append((pbr.u64_image_to_numpy(r.read_image()), r.read_ray_exits(), st))
        r.close()
    image, rec, st = out[0]
    for other, rec2, st2 in out[1:]:
        assert np.array_equal(other, image)
        for f in pbr.RAY_EXIT_DTYPE.names:
            assert np.array_equal(rec2[f], rec[f]), f
        assert st2["status"] == st["status"] and st2["rkn_steps"] == st["rkn_steps"]
    ref = oracle.scene_oracle(sc).trace_ids(src, sc.rays_per_src, np.arange(sc.n_rays))
    assert np.array_equal(rec["entered"], ref["entered"])
    entered = rec["entered"].reshape(sc.n_src, -1)
    assert entered[20:40].all() and not entered[40:].any()

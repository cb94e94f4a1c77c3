"""A point that no view sees has an all-zero row, scores of 0 and the mean of y, whatever the lower bound of the norm: it has no norm to
divide by.  With a bound of 0 that must hold in every fusion kernel, and a point's result must not depend on the points of its tile."""
import numpy as np
import pytest
import torch

from workloads.scenes import make_scene

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def H():
    import gpu_harness
    assert torch.cuda.is_available()
    return gpu_harness


STEPS = {"single": "step_single_pass", "two": "step_single_pass_two_kernels", "step": "step_combined", "staged": "step",
         "staged_two": "step_two_kernels"}


# the kernels of one call after the other: a tile per wave with and without long rows of materials; four producers with a scoring wave,
# with the scoring kernel, with rows; the two kernels; one producer with several objects; the gather of fp32 maps; the gather of few points
@pytest.mark.parametrize("step,N,B,V,D,K,dtype", [
    ("single", 60_000, 1, 5, 512, 24, "f16"), ("single", 60_000, 2, 5, 1024, 40, "bf16"), ("single", 280_000, 1, 10, 256, 24, "f16"),
    ("single", 100_000, 1, 12, 512, 24, "bf16"), ("single", 100_000, 1, 12, 512, 40, "f16"), ("step", 100_000, 1, 12, 512, 24, "f16"),
    ("two", 60_000, 1, 6, 256, 24, "f16"), ("step", 40_000, 5, 4, 512, 24, "f16"), ("staged", 60_000, 1, 6, 768, 24, "bf16"),
    ("staged_two", 60_000, 1, 6, 768, 24, "bf16"), ("staged", 5_000, 1, 4, 384, 10, "f32"), ("staged", 5_000, 1, 4, 512, 10, "f16"),
])
def test_unseen_points_are_zero_for_any_bound_of_the_norm(H, step, N, B, V, D, K, dtype):
    s = make_scene("c1" if B == 1 else "c5", n_points=N // B, n_objects=B, overrides=dict(V=V, D=D, K=K, G=0, grid=16, dtype=dtype))
    # in every second tile a point that nobody sees: far behind the one object, or behind all cameras of the arc
    s.xyz[7::64] = s.cam[0, 6:9] * (1e4 if B == 1 else -1e4)
    s.xyz[320:960] = s.xyz[7]            # and tiles of nothing else
    d = H.DeviceScene(s)
    out = []
    for eps in (1e-12, 1e-40, 0.0):
        d.params.norm_eps = d.params_two.norm_eps = eps
        d.clear_outputs()
        getattr(d, STEPS[step])()
        out.append(d.results())
    unseen = out[0]["count"] == 0
    assert unseen[7::64].all() and unseen[320:960].all() and not unseen.all()
    mean = s.y.astype(np.float64).mean(0)
    for o in out:
        assert (o["scores"][unseen] == 0).all() and (step in ("single", "two") or (o["fused"][unseen] == 0).all())
        assert (o["label"][unseen] == 0).all() and np.allclose(o["prop"][unseen], mean, rtol=2e-6)   # (K additions of 2^-24 each)
        for k in out[0]:
            assert np.array_equal(o[k].view(np.uint8), out[0][k].view(np.uint8)), k

"""k_tile_fused of calls without rows, a tile per wave (tile_waves.hip), where it can go wrong: lists longer than a wave's LDS, as long as
the quota and longer, views on both sides of a group of eight and of sixteen, material tiles, ragged last tiles, objects without
points or views, and the launch with four producers behind it.  References: the two kernels (the same bits up to 16 views, beyond
which they add up k-steps of other cells) and the oracle."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from workloads.scenes import make_scene

pytestmark = pytest.mark.gpu
KEYS = ("vis", "count", "scores", "prop", "label", "mass", "n_used")


@pytest.fixture(scope="module")
def H():
    import gpu_harness
    assert torch.cuda.is_available()
    return gpu_harness


@pytest.fixture(scope="module")
def orc():
    from oracle import aura_oracle
    return aura_oracle


def _objects(sizes, views, **kw):
    """Objects of the given numbers of points and views: parts of one cloud, each begun somewhere else."""
    base = make_scene("c1", n_points=max(sizes), overrides=dict(V=max(views), G=0, **kw))
    return replace(base, xyz=np.concatenate([np.roll(base.xyz, -977 * b, 0)[:n] for b, n in enumerate(sizes)]),
                   pt_offsets=np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64),
                   view_offsets=np.concatenate([[0], np.cumsum(views)]).astype(np.int32), material_of_point=None,
                   **{k: np.concatenate([getattr(base, k)[:v] for v in views]) for k in ("cam", "depth", "feat")})


def _run(H, s, flags=0):
    """Outputs of the single pass as two kernels and as it is, and the k-steps per tile that the two kernels had."""
    d = H.DeviceScene(s, flags=flags, want_fused=False)
    out = []
    for step in (d.step_single_pass_two_kernels, d.step_single_pass):
        H.mark_workspaces(d)
        d.clear_outputs()
        step()
        out.append(d.results())
        if len(out) == 1:
            tiles = int(np.sum((np.diff(s.pt_offsets) + 31) // 32))
            steps = d.ws_single[:tiles * 144].cpu().numpy().view(np.int32).reshape(tiles, 36)[:, 0].copy()
    return out, steps, d


# sizes, views: objects; steps: what the longest lists of the scene must reach (5 and 7 k-steps fit a wave's LDS, up to eight views and
# beyond).  (test_waves_dispatch.py checks that all these take the kernel.)
SAME_BITS = [
    ((30_001, 30_033), (8, 8), 512, 24, 1, 32, "f16", 6),
    ((30_001, 28_000), (8, 5), 1024, 33, 3, 32, "bf16", 6),
    ((27_001, 26_500), (12, 9), 256, 40, 2, 32, "f16", 8),
    ((45_001, 39_000), (16, 7), 768, 65, 1, 32, "bf16", 8),
    ((25_003, 0, 33, 31_000), (9, 2, 0, 10), 512, 128, 8, 24, "f16", 5),
    ((40_001, 40_001), (4, 1), 1024, 1, 1, 16, "bf16", 1),
    ((12_001, 11_950, 12_033), (8, 3, 8), 256, 9, 1, 32, "f16", 6),
]
MORE_VIEWS = [((40_001, 38_000), (17, 24), 256, 24, 24), ((65_000, 60_001), (32, 25), 512, 40, 16)]
QUOTA = [24, 70]
MASK_VIEWS = [(8, 3), (2, 6)]


@pytest.mark.parametrize("sizes,views,D,K,P,grid,dtype,steps", SAME_BITS)
def test_same_bits_as_two_kernels(H, orc, sizes, views, D, K, P, grid, dtype, steps):
    s = _objects(sizes, views, D=D, K=K, P=P, grid=grid, dtype=dtype)
    (two, one), n, d = _run(H, s)
    assert n.max() >= steps
    for k in KEYS:
        assert np.array_equal(one[k].view(np.uint8), two[k].view(np.uint8)), k
    H.compare_points(one, H.oracle_points(orc, s), s, no_fused=True)
    assert not d.status_words()["fuse_score_integrate"]


@pytest.mark.parametrize("sizes,views,D,K,grid", MORE_VIEWS)
def test_more_views_than_a_list_is_filled_up_for(H, orc, sizes, views, D, K, grid):
    s = _objects(sizes, views, D=D, K=K, grid=grid, dtype="f16")
    (two, one), n, _ = _run(H, s)
    assert n.max() > 7
    assert all(np.array_equal(one[k], two[k]) for k in ("vis", "count"))
    H.compare_points(one, H.oracle_points(orc, s), s, no_fused=True)


@pytest.mark.parametrize("K", QUOTA)
def test_lists_longer_than_the_quota(H, orc, K):
    """Every 20th tile's points in no order and no depth test: such tiles are fused point by point, the others as they are."""
    s = _objects((20_001, 20_033), (8, 8), D=512, K=K, grid=24, dtype="f16")
    at = (np.arange(3, 1250, 20)[:, None] * 32 + np.arange(32)).ravel()
    s.xyz[at] = s.xyz[np.random.default_rng(1).permutation(at)]
    (two, one), n, d = _run(H, s, flags=1)
    assert (n < 0).sum() > 10 and (n > 5).any()
    for k in KEYS:
        assert np.array_equal(one[k].view(np.uint8), two[k].view(np.uint8)), k
    assert d.status_words(word=1)["fuse_score_integrate"] == (n < 0).sum()
    H.compare_points(one, H.oracle_points(orc, s, flags=1), s, no_fused=True)


@pytest.mark.parametrize("blind,kw", [(False, dict(V=32, D=768, grid=56)), (True, dict(V=32, D=768, grid=56)),
                                      (False, dict(V=16, D=512, grid=112, HW=336, f=375.0))])   # cells of eight and of three pixels
def test_long_lists_of_one_object(H, blind, kw):
    """Many views and 262 145 points: where the sieve makes no list, the launch with four producers does the work that the
    waves leave; with tiles that nobody sees in the sample, the waves do it."""
    s = make_scene("c2", n_points=262_145, overrides=dict(K=24, G=0, **kw))
    if blind:
        s.xyz[32 * 512:32 * 1100] = s.cam[0, 6:9] * 1e4   # (far behind every object that the cameras look at)
    (two, one), n, _ = _run(H, s)
    assert (n > 7).any() and ((n == 0).sum() > 500) == blind
    tol = 2 * H.check_tol(s)
    assert all(np.array_equal(one[k], two[k]) for k in ("vis", "count"))
    assert np.abs(one["scores"] - two["scores"]).max() <= tol
    assert (np.abs(one["prop"] - two["prop"]) / np.abs(s.y).max(0)).max() <= tol
    assert np.abs(one["mass"] - two["mass"]).max() <= tol * np.abs(two["mass"]).max()


@pytest.mark.parametrize("views", MASK_VIEWS)
def test_mask_columns_beyond_the_views_of_an_object_whose_tiles_outgrow_their_lists(H, orc, views):
    """Rows of the mask are as wide as the object with the most views; a tile that is fused point by point clears the rest of them too."""
    s = _objects((20_001, 20_033), views, D=512, K=24, grid=24, dtype="f16")
    at = (np.arange(3, 1250, 20)[:, None] * 32 + np.arange(32)).ravel()
    s.xyz[at] = s.xyz[np.random.default_rng(1).permutation(at)]
    (two, one), n, d = _run(H, s, flags=1)
    widths = np.repeat(views, np.diff(s.pt_offsets))
    assert n.min() < 0 and not two["vis"][np.arange(max(views)) >= widths[:, None]].any()
    assert d.status_words(word=1)["fuse_score_integrate"] == (n < 0).sum()
    for k in KEYS:
        assert np.array_equal(one[k].view(np.uint8), two[k].view(np.uint8)), k
    H.compare_points(one, H.oracle_points(orc, s, flags=1), s, no_fused=True)

"""Which calls without rows take k_tile_fused with a tile per wave, without a GPU (launch_recorder.cpp stands in for the HIP runtime)."""
import pytest

from test_launches import F16, MEAN_ONLY, TWO_KERNELS, _call, recorder  # noqa: F401


def _kernels(recorder, **kw):
    (status, log), = recorder([_call(**kw)])
    assert status == 0
    return [x[0] for x in log if x not in ("S", "E")]


def _by_waves(name):
    return name.startswith("k_tile_fused<") and name.count(",") == 3


@pytest.mark.parametrize("kw,waves", [
    (dict(N=60_000, V=5, Hf=16), True), (dict(N=20_000, V=4, D=1024, Hf=16), True), (dict(N=40_000, V=8, Hf=37), False),
    (dict(N=262_113, V=8, Hf=224), True), (dict(N=262_112, V=12, Hf=16), False), (dict(N=262_113, V=12, Hf=16), True),
    (dict(N=60_000, V=16, B=2, Hf=16), True), (dict(N=120_000, V=24 * 3, B=3, Hf=37), False),
    # several objects: 512 channels and more up to 12 k-steps (8 of up to eight views and 3000 tiles), 256 up to 40 or any number where
    # there are 5000 tiles; not where a few tiles outgrow theirs
    (dict(N=30 * 4800, B=30, V=30 * 8, Hf=16, K=40), True), (dict(N=30 * 3500, B=30, V=30 * 8, Hf=16, K=40), False),
    (dict(N=2 * 16_000, B=2, V=16, Hf=32, H=224), False), (dict(N=2 * 26_000, B=2, V=16, Hf=32, H=224), True),
    (dict(N=2 * 32_000, B=2, V=20, Hf=32, H=224), True),
    (dict(N=16 * 3000, B=16, V=16 * 8, Hf=16, D=256), True), (dict(N=30 * 6000, B=30, V=30 * 8, Hf=24, D=256), True),
    (dict(N=64 * 3000, B=64, V=64 * 6, Hf=16, D=256), True), (dict(N=64 * 3000, B=64, V=64 * 8, Hf=24, D=256), True),
    (dict(N=16 * 3000, B=16, V=16 * 24, Hf=16, D=256), False), (dict(N=16 * 3700, B=16, V=16 * 24, Hf=16, D=256, K=40), True),
    (dict(N=6 * 6200, B=6, V=12, Hf=37, D=1024), False), (dict(N=21 * 12_000, B=21, V=42, Hf=56, D=1024), True),
    (dict(N=1_000_000, V=33, Hf=16), False), (dict(D=1536), False), (dict(flags=TWO_KERNELS), False), (dict(call="scores"), False),
])
def test_who_takes_a_tile_per_wave(recorder, kw, waves):
    names = _kernels(recorder, **kw)
    assert any(_by_waves(n) for n in names) == waves
    if waves:
        assert names[-1] in ("k_mass_final", "k_mass_points_small") and not any(n.startswith("k_tile_scores") for n in names)


def test_the_scenes_of_the_gpu_tests_take_it(recorder):
    import test_gpu_waves as g
    cases = [(sizes, views, D, K, grid) for sizes, views, D, K, _, grid, _, _ in g.SAME_BITS] + g.MORE_VIEWS
    cases += [((20_001, 20_033), (8, 8), 512, K, 24) for K in g.QUOTA] + [((20_001, 20_033), v, 512, 24, 24) for v in g.MASK_VIEWS]
    for sizes, views, D, K, grid in cases:   # (as many objects, each with the most views)
        names = _kernels(recorder, N=sum(sizes), B=len(sizes), V=len(sizes) * max(views), H=224, Hf=grid, D=D, K=K)
        assert any(_by_waves(n) for n in names), (sizes, views)


def test_views_and_materials_choose_the_instance(recorder):
    for V, K, dtype in ((8, 32, F16), (9, 32, 1), (8, 33, 1), (9, 128, F16)):
        name, = [n for n in _kernels(recorder, N=1_000_000, V=V, Hf=16, K=K, dtype=dtype) if _by_waves(n)]
        assert name == f"k_tile_fused<{dtype},{int(V > 8)},{4 if K > 32 else 1},1>"


@pytest.mark.parametrize("kw,both", [(dict(K=24), True), (dict(K=24, D=512), True), (dict(K=40, D=512), False), (dict(K=40), True),
                                     (dict(D=256), False), (dict(N=5_000_000), False),
                                     # cells of one, two and three pixels
                                     (dict(N=330_000, V=16, H=224, Hf=224), True), (dict(N=330_000, V=16, H=224, Hf=224, D=512, K=40), False),
                                     (dict(N=330_000, V=11, H=224, Hf=224), False), (dict(N=600_000, V=24, H=224, Hf=224), False),
                                     (dict(N=288_000, V=25, H=224, Hf=112), False), (dict(N=288_000, V=25, H=336, Hf=112, D=512), True)])
def test_long_lists_are_left_to_the_producers_where_all_tiles_are_seen(recorder, kw, both):
    names = _kernels(recorder, **dict(dict(N=262_145, V=32, Hf=56, D=768), **kw))
    fused = [n for n in names if n.startswith("k_tile_fused<")]
    assert _by_waves(fused[0]) and len(fused) == 1 + both
    assert any(n.startswith("k_tile_scores") for n in names) == (both and kw.get("K", 24) > 32)


def _form(name):
    """(product waves, producers, scoring wave) of an instance with producers."""
    a = name[len("k_tile_fused<"):-1].split(",")
    return int(a[1]), int(a[5]), int(a[6])


@pytest.mark.parametrize("kw,scoring", [
    # 256 and 512 channels, one producer, no rows; not where the stage beside it is short
    (dict(N=16 * 3000, B=16, V=16 * 8, Hf=16), 1), (dict(N=64 * 3000, B=64, V=64 * 4, Hf=24), 1), (dict(N=8 * 6000, B=8, V=8 * 3, Hf=48, D=256), 1),
    (dict(N=16 * 3000, B=16, V=16 * 8, Hf=16, K=33), 0), (dict(N=16 * 3000, B=16, V=16 * 8, Hf=16, call="scores"), 0),
    (dict(N=6 * 10_000, B=6, V=6 * 6, D=768, Hf=40), 0),
    (dict(N=30 * 2000, B=30, V=30 * 8, Hf=24), 0), (dict(N=30 * 2000, B=30, V=30 * 7, Hf=24), 1),
])
def test_one_producer_scores_its_tiles_where_it_pays(recorder, kw, scoring):
    names = _kernels(recorder, **kw)
    fused, = [n for n in names if n.startswith("k_tile_fused<")]
    assert not _by_waves(fused) and _form(fused)[1:] == (1, scoring)
    assert any(n.startswith("k_tile_scores") for n in names) == (not scoring)

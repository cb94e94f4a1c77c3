"""The sieve in front of the one-kernel fusion (tile_sift.hip) where its branches can go wrong: objects without views or points, lists of
a few tiles, two launch tables, objects whose sample is all seen while other tiles are not, rows of any pitch and alignment, tiles
that outgrow their k-steps.  The reference is the two kernels, which project every tile."""
from dataclasses import replace

import numpy as np
import pytest
import torch

from workloads.scenes import make_scene

pytestmark = pytest.mark.gpu
TILE = 32
KEYS = ("vis", "count", "scores", "prop", "label", "mass", "n_used")


@pytest.fixture(scope="module")
def H():
    import gpu_harness
    assert torch.cuda.is_available()
    return gpu_harness


def _away(cam):
    """A place that no camera has in its picture, by a wide margin."""
    rng = np.random.default_rng(3)
    for _ in range(1000):
        p = rng.standard_normal(3)
        p *= 50 / np.linalg.norm(p)
        c = np.einsum("vij,j->vi", cam[:, :9].reshape(-1, 3, 3).astype(np.float64), p) + cam[:, 9:12]
        u = np.abs(cam[:, 12] * c[:, 0]) - 1.5 * cam[:, 14] * np.abs(c[:, 2])
        v = np.abs(cam[:, 13] * c[:, 1]) - 1.5 * cam[:, 15] * np.abs(c[:, 2])
        if ((c[:, 2] < -1) | (u > 0) | (v > 0)).all():
            return p.astype(np.float32)
    raise AssertionError("the cameras see everywhere")


def _hide(s, tiles, b=0):
    """Moves the points of these tiles of object b out of every picture."""
    p = _away(s.cam)
    for t in tiles:
        at = s.pt_offsets[b] + TILE * t
        s.xyz[at:min(at + TILE, s.pt_offsets[b + 1])] = p


def _sample(n):
    """The tiles that the sieve's sample of an object of n tiles consists of: four pairs."""
    return [t for w in range(4) for t in range(2 * ((2 * w + 1) * ((n + 1) // 2) // 8), n)[:2]]


def _show(s, tiles):
    """Moves the points of these tiles of the first object to the point that is nearest to the first camera."""
    p = s.xyz[np.argmin(s.xyz.astype(np.float64) @ s.cam[0, 6:9])].copy()
    for t in tiles:
        s.xyz[TILE * t:TILE * t + TILE] = p


def _objects(sizes, views, **kw):
    """Objects of the given numbers of points and views: parts of one cloud, each begun somewhere else."""
    base = make_scene("c5", n_points=max(sizes), n_objects=1, overrides=dict(V=max(views), G=0, **kw))
    return replace(base, xyz=np.concatenate([np.roll(base.xyz, -977 * b, 0)[:n] for b, n in enumerate(sizes)]),
                   pt_offsets=np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64),
                   view_offsets=np.concatenate([[0], np.cumsum(views)]).astype(np.int32), material_of_point=None,
                   **{k: np.concatenate([getattr(base, k)[:v] for v in views]) for k in ("cam", "depth", "feat")})


def _lists(d):
    """What the sieve left for each object: the length of its list of seen tiles, or -1 where it made none."""
    from paper_2511_03126_amd import binding
    s, first = d.scene, -((32 * d.scene.B + 255) // 256 * 64)
    return [binding.fuse_status_word(binding.CALL_FUSE_SCORE_INTEGRATE, d.views, s.N, d.ws_single, B=s.B, K=s.K, P=s.P, G=s.G,
                                     word=first + 8 * b + 7) for b in range(s.B)]


def _expected_lists(s, count):
    """The same from the points' view counts, and whether the object has tiles that nobody sees.  (Objects of up to eight views: the
    sample looks at all of them.)"""
    lists, unseen = [], []
    for b in range(s.B):
        c = count[s.pt_offsets[b]:s.pt_offsets[b + 1]]
        n = -(-len(c) // TILE)
        seen = (np.pad(c, (0, n * TILE - len(c))).reshape(n, TILE) > 0).any(1)
        lists.append(-1 if n and seen[_sample(n)].all() else int(seen.sum()))
        unseen.append(int((~seen).sum()))
    return lists, unseen


def _check(H, s, flags=0, sieved=True):
    """Single pass with the sieve and as two kernels: the same bits; zeros for unseen points.  Returns the lists and numbers of unseen tiles."""
    from paper_2511_03126_amd import binding
    d = H.DeviceScene(s, flags=flags, want_fused=False)
    out = []
    for step in (d.step_single_pass_two_kernels, d.step_single_pass):
        H.mark_workspaces(d)
        d.clear_outputs()
        step()
        out.append(d.results())
    for k in KEYS:
        assert np.array_equal(out[0][k].view(np.uint8), out[1][k].view(np.uint8)), k
    blind = out[1]["count"] == 0
    assert blind.any() and not any(out[1][k][blind].any() for k in ("vis", "scores", "label"))
    assert out[1]["prop"][blind].any() == (flags & binding.UNSEEN_ZERO == 0)
    lists, unseen = _expected_lists(s, out[1]["count"])
    assert not sieved or _lists(d) == lists
    return lists, unseen


@pytest.mark.parametrize("zero", [0, 16])   # 16: AURA_UNSEEN_ZERO
@pytest.mark.parametrize("D,V,K", [(512, 7, 45), (512, 7, 24), (1024, 8, 24), (256, 5, 100)])
def test_unseen_tiles_of_an_object_whose_sample_is_all_seen(H, D, V, K, zero):
    """No list is made there: the fusion and the scoring kernel (or the scoring wave) come across the unseen tiles themselves."""
    s = make_scene("c1", n_points=262_145, overrides=dict(V=V, D=D, K=K, G=0, dtype="f16"))
    _show(s, _sample(8_193))
    _hide(s, [3, *range(40, 80), *range(4_000, 4_100), 5_122, 8_192])
    lists, unseen = _check(H, s, flags=zero)
    assert lists == [-1] and unseen[0] >= 143


# Table of 64 objects and one of six.  1: fewer points than a workgroup of the sieve has tiles for; 3: a list of three tiles; 4: of none
@pytest.mark.parametrize("D,flags", [(256, 0), (256, 1), (512, 0), (512, 1)])   # 1: without the depth test
def test_objects_of_two_launch_tables_without_views_points_or_seen_tiles(H, D, flags):
    sizes = [0, 167, 44_000, 43_001, 43_001, 43_001] + [86_017] * 58 + [90_001] * 6
    views = [2, 2, 0, 3, 2, 3] + [2 + b % 2 for b in range(64)]
    s = _objects(sizes, views, D=D, K=9, P=2)
    _hide(s, range(5), 1)
    _hide(s, [t for t in range(1344) if t not in (700, 701, 1343)], 3)
    _hide(s, range(1344), 4)
    _hide(s, range(0, 1344, 2), 5)
    for b in range(6, 70):
        _hide(s, range(5 * b, 11 * b if b < 64 else 5 * b + 10), b)
    _hide(s, range(_sample(2813)[0] - 10, _sample(2813)[0] + 10), 67)
    lists, unseen = _check(H, s, flags)
    assert lists[0] == lists[2] == lists[4] == 0 and lists[1] <= 1 and lists[3] <= 3
    assert min(unseen[2:]) > 0 and lists[67] > 0
    if flags:
        assert [-1 in part for part in (lists[:64], lists[64:])] == [True, True] and lists[33] > 0


def test_a_list_of_four_hundred_thousand_tiles(H):
    """No limit to a list's length: a cloud of 6250 tiles, 65 times over."""
    s = _objects([200_000], [3], D=256, K=5, P=1)
    s = replace(s, xyz=np.tile(s.xyz, (65, 1)), pt_offsets=np.array([0, 13_000_000], np.int64))
    _hide(s, [*range(7), *range(300_000, 300_100), 406_249])
    lists, unseen = _check(H, s)
    assert lists[0] > 100_000 and lists[0] + unseen[0] == 406_250


@pytest.mark.parametrize("K,P,shift,pitch", [(45, 3, 1, 3), (24, 1, 1, 4), (24, 2, 2, 8), (128, 8, 3, 5)])
def test_rows_of_any_pitch_and_alignment_stay_in_place(H, K, P, shift, pitch):
    """Every output begins `shift` elements beyond a place that is aligned, the mask is wider than the object has views."""
    import paper_2511_03126_amd as aura
    s = _objects([300_001], [3], D=512, K=K, P=P)
    d = H.DeviceScene(s, want_fused=False)
    d.step_single_pass()   # (its workspace)
    out = []
    for params in (d.params_two, d.params):
        bufs = {k: torch.full((shift + s.N * n + 8,), 77, dtype=t, device="cuda:0") for k, n, t in
                (("vis", pitch, torch.uint8), ("count", 1, torch.int32), ("scores", K, torch.float32), ("prop", P, torch.float32),
                 ("label", 1, torch.int32))}
        rows = {k: b[shift:len(b) - 8].view(s.N, -1) for k, b in bufs.items()}
        aura.fuse_score_integrate(d.views, params, d.xyz, d.temb, d.y, rows["scores"], d.mass, count=rows["count"].view(-1),
                                  vis=rows["vis"], prop=rows["prop"], label=rows["label"].view(-1), n_used=d.n_used, workspace=d.ws_single)
        out.append({k: b.cpu().numpy() for k, b in bufs.items()} | dict(mass=d.mass.cpu().numpy()))
    assert _lists(d) == _expected_lists(s, out[1]["count"][shift:-8])[0] and _lists(d)[0] > 0
    for k in out[0]:
        assert np.array_equal(out[0][k].view(np.uint8), out[1][k].view(np.uint8)), k
        assert k == "mass" or ((out[1][k][:shift] == 77).all() and (out[1][k][-8:] == 77).all()), k
    assert not out[1]["vis"][shift:-8].reshape(s.N, pitch)[:, 3:].any()


@pytest.mark.parametrize("D,K", [(512, 24), (512, 45), (768, 24), (1024, 45)])
def test_listed_tiles_that_outgrow_their_k_steps(H, D, K):
    """Points of every 40th tile in no order: such tiles are fused point by point at the end, also where the fusion follows a list.  The
    two kernels hold more k-steps per tile, so results are compared by the bounds of the oracle's tests."""
    s = make_scene("c2", n_points=262_200, overrides=dict(V=12, D=D, K=K, G=0))
    rng = np.random.default_rng(1)
    at = (np.arange(7, 8_000, 40)[:, None] * TILE + np.arange(TILE)).ravel()
    s.xyz[at] = s.xyz[rng.permutation(at)]
    _hide(s, [*range(600), _sample(-(-s.N // TILE))[2]])
    d = H.DeviceScene(s, want_fused=False)
    out = []
    for step in (d.step_single_pass_two_kernels, d.step_single_pass):
        d.clear_outputs()
        step()
        out.append(d.results())
    assert _lists(d) == _expected_lists(s, out[1]["count"])[0] and _lists(d)[0] > 0
    assert d.status_words(word=1)["fuse_score_integrate"] > 0
    two, one = out
    for k in ("vis", "count"):
        assert np.array_equal(one[k], two[k]), k
    assert np.abs(one["scores"] - two["scores"]).max() <= 2 * H.check_tol(s)
    assert (np.abs(one["prop"] - two["prop"]) / np.abs(s.y).max(0)).max() <= 2 * H.check_tol(s)
    other = one["label"] != two["label"]
    rows = two["scores"][other]
    assert (rows[np.arange(len(rows)), two["label"][other]] - rows[np.arange(len(rows)), one["label"][other]] <= 4 * H.check_tol(s)).all()
    assert np.abs(one["mass"] - two["mass"]).max() <= 2 * H.check_tol(s) * np.abs(two["mass"]).max()


@pytest.mark.parametrize("N,V,sieved", [(384_000, 6, True), (384_001, 6, True), (262_112, 7, False), (262_113, 7, True)])
def test_one_object_of_one_producer_and_of_four(H, N, V, sieved):
    """256 channels and more than 32 materials: one producer from 12 001 tiles on; the sieve from 8 192."""
    s = make_scene("c1", n_points=N, overrides=dict(V=V, D=256, K=40, P=2, G=0, dtype="bf16"))
    _hide(s, [*range(100, 5_000), -(-N // TILE) - 1])
    assert _check(H, s, sieved=sieved)[0][0] > 0

"""GPU parity of aura_select_views (Sec. 3.2.2) and aura_fuse_selected (Sec. 3.2.3) against the CPU oracle on the
same seeded inputs.

Selection: which views are visible is bit-exact (Eq. 1); scores within 1e-5 (fp32 against fp64); the kept views
identical, in order, wherever the oracle's scores around the cut and between consecutive kept views are further apart
than the accuracy of an fp32 score (pairs inside that margin may swap: they must be rare and the library's choice must
still be k visible views whose oracle scores are the k largest up to the margin).  Fusion over a selection: both
sides get the ORACLE's selection; fused rows to the bar of the hot path, counts exact."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

SCORE_TOL = 1e-5


def _scene(name, **kw):
    from workloads.scenes import make_scene, synthetic_normals
    s = make_scene(name, **kw)
    return s, synthetic_normals(s.xyz, s.pt_offsets, s.meta["seed"])


def _gpu_select(d, s, nrm, k, want_all=True):
    import paper_2511_03126_amd as aura
    N = s.N
    sel_view = torch.full((N, k), -7, dtype=torch.int32, device=d.dev)
    sel_score = torch.full((N, k), float("nan"), device=d.dev) if want_all else None
    sel_mask = torch.full((N, s.vis_pitch), 9, dtype=torch.uint8, device=d.dev) if want_all else None
    n_sel = torch.full((N,), -7, dtype=torch.int32, device=d.dev) if want_all else None
    aura.select_views(d.views, d.params, d.xyz, torch.from_numpy(nrm).to(d.dev), k, sel_view, sel_score, sel_mask, n_sel,
                      d.pt_offsets, d.view_offsets)
    torch.cuda.synchronize()
    f = lambda t: None if t is None else t.cpu().numpy()
    return dict(sel_view=f(sel_view), sel_score=f(sel_score), sel_mask=f(sel_mask), n_sel=f(n_sel))


def _check_selection(g, ref, k):
    assert np.array_equal(g["n_sel"], ref["n_sel"])                      # the visible views are the same: Eq. 1
    assert np.abs(g["sel_score"] - ref["sel_score"]).max(initial=0.0) <= SCORE_TOL
    # mask = exactly the kept views
    assert np.array_equal(g["sel_mask"].sum(1), g["n_sel"]) and g["sel_mask"].max(initial=0) <= 1
    rows, cols = np.nonzero(g["sel_view"] >= 0)
    assert g["sel_mask"][rows, g["sel_view"][rows, cols]].all()
    assert ((g["sel_view"] >= 0).sum(1) == g["n_sel"]).all()
    # identical ranking away from near-ties
    d = -np.diff(ref["sel_score"], axis=1)
    both = (ref["sel_view"][:, 1:] >= 0) if k > 1 else np.zeros((len(d), 0), bool)
    last = np.take_along_axis(ref["sel_score"], np.maximum(ref["n_sel"] - 1, 0)[:, None], 1)[:, 0]
    # scores of exactly 0 (views that see the back of the surface) are 0 on both sides and go by view index
    cut_clear = (ref["gap"] > SCORE_TOL) | ((ref["gap"] == 0) & (last == 0))
    clear = cut_clear & ((d > SCORE_TOL) | ((d == 0) & (ref["sel_score"][:, 1:] == 0)) | ~both).all(1)
    assert clear.mean() > 0.97, f"too many near-ties: {1 - clear.mean():.4f}"
    assert np.array_equal(g["sel_view"][clear], ref["sel_view"][clear])
    assert np.array_equal(g["sel_mask"][clear], ref["sel_mask"][clear])
    # inside the margin: every kept view is visible and scores, by the oracle, within the margin of the oracle's choice
    for i in np.nonzero(~clear)[0]:
        kept = g["sel_view"][i][g["sel_view"][i] >= 0]
        assert len(set(kept.tolist())) == len(kept)
        s_or = ref["score_all"][i, kept]
        assert (s_or >= 0).all()
        assert np.abs(np.sort(s_or)[::-1] - ref["sel_score"][i, :len(kept)]).max(initial=0.0) <= 2 * SCORE_TOL


@pytest.mark.parametrize("name,kw,k", [("c1", {}, 3), ("c1", {}, 1), ("c1", {}, 8), ("c2", dict(n_points=30_011), 3),
                                       ("c5", dict(n_points=3_001, n_objects=5), 2), ("c5", dict(n_points=3_001, n_objects=70), 3),
                                       ("c1", dict(n_points=7_001, overrides=dict(dtype="f16", V=12)), 5)])
def test_selection_matches_oracle(orc, name, kw, k):
    import gpu_harness as H
    s, nrm = _scene(name, **kw)
    d = H.DeviceScene(s)
    g = _gpu_select(d, s, nrm, k)
    ref = orc.select_views(s.cam, s.depth, s.xyz, nrm, k, tau=s.tau, z_near=s.z_near, pt_offsets=d.pt_offsets,
                           view_offsets=d.view_offsets, mask_pitch=s.vis_pitch)
    _check_selection(g, ref, k)
    only = _gpu_select(d, s, nrm, k, want_all=False)
    assert np.array_equal(only["sel_view"], g["sel_view"])


# Small calls give a wave to every point, large ones a thread: the same points in calls of every size must get the same
# choice.  Scores are at most 1 and come from two sums of three products of unit vectors, a root and two divisions: where the
# compiler contracts the sums differently in the two kernels they differ by at most 16 roundings.
@pytest.mark.parametrize("name,kw,k", [("c1", dict(n_points=70_000), 3), ("c3", dict(n_points=70_000, overrides=dict(V=32, HW=112, grid=112)), 8)])
def test_a_wave_per_point_chooses_as_a_thread_per_point(name, kw, k):
    import paper_2511_03126_amd as aura
    import gpu_harness as H
    s, nrm = _scene(name, **kw)
    d = H.DeviceScene(s)
    whole = _gpu_select(d, s, nrm, k)
    first = differ = 0
    for n in (1, 3, 4, 5, 64, 1_001):
        part = slice(first, first + n)
        out = [torch.full((n, k), -7, dtype=torch.int32, device=d.dev), torch.full((n, k), float("nan"), device=d.dev),
               torch.full((n, s.vis_pitch), 9, dtype=torch.uint8, device=d.dev), torch.full((n,), -7, dtype=torch.int32, device=d.dev)]
        aura.select_views(d.views, d.params, d.xyz[part].contiguous(), torch.from_numpy(nrm[part]).to(d.dev), k, *out)
        view, score, mask, n_sel = (t.cpu().numpy() for t in out)
        assert np.array_equal(n_sel, whole["n_sel"][part])
        assert np.abs(score - whole["sel_score"][part]).max() <= 16 * 2.0 ** -24
        same = (view == whole["sel_view"][part]).all(axis=1)   # (views whose scores differ by less than that may change places)
        differ += int((~same).sum())
        assert np.array_equal(mask[same], whole["sel_mask"][part][same])
        first += n
    assert differ <= 2


# The wave has a lane per view, up to 64; a thread per point takes more views, and calls of more than 16 384 points.  Rows of
# the mask longer than the wave.
@pytest.mark.parametrize("V,N,k", [(33, 1_001, 3), (64, 1_001, 8), (65, 1_001, 8), (40, 16_384, 4), (40, 16_385, 4)])
def test_views_in_both_halves_of_the_wave(orc, V, N, k):
    import paper_2511_03126_amd as aura
    import gpu_harness as H
    s, nrm = _scene("c1", n_points=N, overrides=dict(V=V, D=32))
    d = H.DeviceScene(s)
    out = [torch.full((N, k), -7, dtype=torch.int32, device=d.dev), torch.full((N, k), float("nan"), device=d.dev),
           torch.full((N, 80), 9, dtype=torch.uint8, device=d.dev), torch.full((N,), -7, dtype=torch.int32, device=d.dev)]
    aura.select_views(d.views, d.params, d.xyz, torch.from_numpy(nrm).to(d.dev), k, *out)
    ref = orc.select_views(s.cam, s.depth, s.xyz, nrm, k, tau=s.tau, z_near=s.z_near, mask_pitch=80)
    _check_selection(dict(zip(("sel_view", "sel_score", "sel_mask", "n_sel"), (t.cpu().numpy() for t in out))), ref, k)
    assert ref["sel_view"].max() >= 32


def test_equal_scores_in_both_halves_of_the_wave():
    """Views 32 to 63 are the cameras and depth maps of 0 to 31 again: every choice is a view and its copy, the lower first."""
    import paper_2511_03126_amd as aura
    import gpu_harness as H
    s, nrm = _scene("c1", n_points=3_001, overrides=dict(V=32, D=32))
    d = H.DeviceScene(s)
    one = _gpu_select(d, s, nrm, 4)
    views = aura.Views(cam=torch.cat([d.views.cam] * 2), depth=torch.cat([d.views.depth] * 2), feat=None)
    sel = torch.full((s.N, 8), -7, dtype=torch.int32, device=d.dev)
    score = torch.full((s.N, 8), float("nan"), device=d.dev)
    aura.select_views(views, d.params, d.xyz, torch.from_numpy(nrm).to(d.dev), 8, sel, score)
    v, sc = one["sel_view"], one["sel_score"]
    want = np.stack([v, np.where(v >= 0, v + 32, -1)], 2).reshape(s.N, 8)
    n = 2 * (v >= 0).sum(1)
    own = np.where(np.arange(8) < n[:, None], want, -1)
    distinct = ~((sc[:, 1:] == sc[:, :-1]) & (v[:, 1:] >= 0)).any(1)     # (two cameras of one score: both before their copies)
    assert distinct.mean() > 0.5 and np.array_equal(sel.cpu().numpy()[distinct], own[distinct])
    assert np.array_equal(score.cpu().numpy(), np.repeat(sc, 2, axis=1))


def test_a_point_is_given_the_same_scores_in_any_call():
    import paper_2511_03126_amd as aura
    import gpu_harness as H
    s, nrm = _scene("c1", n_points=20_000, overrides=dict(V=32, D=32))
    d = H.DeviceScene(s)
    whole = _gpu_select(d, s, nrm, 8)
    sel = torch.full((10_000, 8), -7, dtype=torch.int32, device=d.dev)
    score = torch.full((10_000, 8), float("nan"), device=d.dev)
    aura.select_views(d.views, d.params, d.xyz[:10_000], torch.from_numpy(nrm[:10_000]).to(d.dev), 8, sel, score)
    assert np.array_equal(score.cpu().numpy(), whole["sel_score"][:10_000])
    assert np.array_equal(sel.cpu().numpy(), whole["sel_view"][:10_000])


def test_hand_worked_rig_on_the_gpu():
    """Cameras on a line at known distances: S_total = 1 / (1 + distance), nearest first; equal distances by index; a
    camera behind the surface scores 0 and comes last."""
    import paper_2511_03126_amd as aura
    dev = "cuda:0"
    cam = lambda zc, flip=False: np.array(([-1, 0, 0, 0, 1, 0, 0, 0, -1] if flip else [1, 0, 0, 0, 1, 0, 0, 0, 1])
                                          + [0, 0, (zc if flip else -zc)] + [100, 100, 500, 500], np.float32)
    # camera centres at z = -2, -2, -1 looking along +z; one at z = +1 looking back along -z (R = diag(-1, 1, -1))
    cams = np.stack([cam(1.0, flip=True), cam(-2.0), cam(-2.0), cam(-1.0)])
    views = aura.Views(cam=torch.from_numpy(cams).to(dev), depth=None, feat=None, H=1000, W=1000)
    params = aura.Params(flags=1)   # frustum only
    xyz = torch.tensor([[0.0, 0.0, 0.0]], device=dev)
    nrm = torch.tensor([[0.0, 0.0, -1.0]], device=dev)
    sel_view = torch.empty((1, 4), dtype=torch.int32, device=dev)
    sel_score = torch.empty((1, 4), device=dev)
    aura.select_views(views, params, xyz, nrm, 4, sel_view, sel_score)
    torch.cuda.synchronize()
    assert sel_view.cpu().tolist() == [[3, 1, 2, 0]]
    assert np.allclose(sel_score.cpu().numpy(), [[0.5, 1 / 3, 1 / 3, 0.0]], rtol=1e-6)


@pytest.mark.parametrize("name,kw,k", [("c1", {}, 3), ("c2", dict(n_points=30_011), 3), ("c2", dict(n_points=30_011), 1),
                                       ("c5", dict(n_points=7_001, n_objects=5), 2), ("c1", dict(n_points=11_001, overrides=dict(dtype="f16", V=12, D=512)), 3)])
def test_fusion_over_the_oracle_selection(orc, name, kw, k):
    import gpu_harness as H
    import paper_2511_03126_amd as aura
    s, nrm = _scene(name, **kw)
    d = H.DeviceScene(s)
    sel = orc.select_views(s.cam, s.depth, s.xyz, nrm, k, tau=s.tau, z_near=s.z_near, pt_offsets=d.pt_offsets,
                           view_offsets=d.view_offsets, mask_pitch=s.vis_pitch)
    ref = orc.fuse_features(s.cam, s.depth, s.feat, s.feat_dtype, s.xyz, tau=s.tau, z_near=s.z_near,
                            pt_offsets=d.pt_offsets, view_offsets=d.view_offsets, sel_mask=sel["sel_mask"])
    mask = torch.from_numpy(sel["sel_mask"]).to(d.dev)
    H.mark_workspaces(d)
    for ws in ([d.ws_fuse, None] if d.ws_fuse is not None else [None]):     # matrix-core path and gather path
        d.fused.fill_(float("nan"))
        d.count_fuse.fill_(-7)
        aura.fuse_selected(d.views, d.params, d.xyz, mask, d.fused, d.count_fuse, d.pt_offsets, d.view_offsets, ws)
        torch.cuda.synchronize()
        fg = d.fused.cpu().numpy().astype(np.float64)
        assert np.array_equal(d.count_fuse.cpu().numpy(), ref["count"])
        assert np.array_equal(ref["count"], sel["n_sel"])
        nr = np.linalg.norm(ref["fused"], axis=1)
        err = np.linalg.norm(fg - ref["fused"], axis=1) / np.maximum(nr, 1e-12)
        err[(nr == 0) & (np.linalg.norm(fg, axis=1) == 0)] = 0.0
        assert err.max() <= H.check_tol(s), f"fused rel err {err.max()}"
    d._ran.add("fuse_features")     # fuse_selected shares its workspace
    assert all(H.took_tiles(d).values()) and (H.took_tiles(d) or s.feat_dtype == "f32")


def test_full_size_pipeline_c2(orc):
    """C2 at full size: select on the device, fuse over the device's own selection; the oracle selects and fuses on its
    own.  Points whose selection is unambiguous (all but a few near-ties) must agree to the bar of the hot path."""
    import gpu_harness as H
    import paper_2511_03126_amd as aura
    s, nrm = _scene("c2")
    d = H.DeviceScene(s)
    g = _gpu_select(d, s, nrm, 3)
    mask = torch.from_numpy(g["sel_mask"]).to(d.dev)
    aura.fuse_selected(d.views, d.params, d.xyz, mask, d.fused, d.count_fuse, None, None, d.ws_fuse)
    torch.cuda.synchronize()
    ref_sel = orc.select_views(s.cam, s.depth, s.xyz, nrm, 3, tau=s.tau, z_near=s.z_near, mask_pitch=s.vis_pitch)
    _check_selection(g, ref_sel, 3)
    same = (g["sel_mask"] == ref_sel["sel_mask"]).all(1)
    assert same.mean() > 0.99
    rng = np.random.default_rng(3)
    idx = np.sort(rng.choice(np.nonzero(same)[0], 4000, replace=False))
    ref = orc.fuse_features(s.cam, s.depth, s.feat, s.feat_dtype, s.xyz[idx], tau=s.tau, z_near=s.z_near,
                            sel_mask=ref_sel["sel_mask"][idx])
    fg = d.fused.cpu().numpy()[idx].astype(np.float64)
    err = np.linalg.norm(fg - ref["fused"], axis=1) / np.maximum(np.linalg.norm(ref["fused"], axis=1), 1e-12)
    err[np.linalg.norm(ref["fused"], axis=1) == 0] = 0.0
    assert err.max() <= H.check_tol(s)
    assert np.array_equal(d.count_fuse.cpu().numpy()[idx], ref["count"])

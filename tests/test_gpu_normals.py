"""GPU parity of aura_estimate_normals (Sec. 3.2.2) against the CPU oracle on the same seeded inputs.  Both sides
select the neighbours with the same fp32 distance chain (ties by index), so the neighbour sets are the same and the
rest is fp64 on both sides.  Bar: eigenvalues within 1e-5 of the largest one (they are stored as fp32); normals within
3e-7 per component (fp32 output) wherever the plane is well defined (gap between the two smallest eigenvalues above 1e-3 of the largest) and
the outward test is not at right angles; elsewhere the library's vector must still minimise the oracle's covariance
to the same accuracy (Rayleigh quotient), whatever its sign."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def _gpu(xyz, queries, centre, k, po=None, qo=None, want_evals=True):
    import paper_2511_03126_amd as aura
    dev = "cuda:0"
    M = len(queries)
    normals = torch.full((max(M, 1), 3), float("nan"), device=dev)
    evals = torch.full((max(M, 1), 3), float("nan"), device=dev) if want_evals else None
    t = lambda a: torch.from_numpy(np.ascontiguousarray(a, np.float32)).to(dev).reshape(-1, 3)
    aura.estimate_normals(t(xyz), t(queries), centre, k, normals, evals, po, qo)
    torch.cuda.synchronize()
    return normals.cpu().numpy()[:M].astype(np.float64), None if evals is None else evals.cpu().numpy()[:M].astype(np.float64)


def _compare(g_n, g_w, ref, queries, centre_of_query, xyz, po, qo):
    lam = ref["evals"]
    top = np.maximum(lam[:, 2], 1e-30)
    assert np.abs(g_w - lam).max() <= 1e-5 * top.max()
    assert np.allclose(np.linalg.norm(g_n, axis=1), 1.0, atol=1e-6)
    out = queries.astype(np.float64) - centre_of_query
    out /= np.maximum(np.linalg.norm(out, axis=1, keepdims=True), 1e-30)
    well = ((lam[:, 1] - lam[:, 0]) > 1e-3 * top) & (np.abs(np.einsum("ij,ij->i", ref["normals"], out)) > 1e-3)
    assert well.mean() > 0.9
    assert np.abs(g_n[well] - ref["normals"][well]).max() < 3e-7            # the output is fp32: 6e-8 per component
    # everywhere: the vector minimises the quadratic form of the oracle's neighbours
    B = len(po) - 1
    for b in range(B):
        P = xyz[po[b]:po[b + 1]].astype(np.float64)
        for m in range(int(qo[b]), int(qo[b + 1])):
            idx = ref["nn_idx"][m]
            idx = idx[idx >= 0]
            nb = P[idx]
            cov = np.cov(nb.T, bias=True) if len(nb) > 1 else np.zeros((3, 3))
            assert g_n[m] @ cov @ g_n[m] <= lam[m, 0] + 1e-6 * top[m] + 1e-30


@pytest.mark.parametrize("name,kw,Mq,k", [("c1", {}, 150, 30), ("c1", {}, 40, 8), ("c1", dict(n_points=25), 10, 30),
                                          ("c2", dict(n_points=50_000), 100, 30), ("c5", dict(n_points=2_000, n_objects=5), 20, 16),
                                          ("c5", dict(n_points=500, n_objects=70), 3, 12)])
def test_scenes(orc, name, kw, Mq, k):
    from workloads.scenes import make_scene
    s = make_scene(name, **kw)
    po = s.pt_offsets
    # queries: voxel centroids (not members of the cloud) and members, mixed
    q, qo = [], [0]
    for b in range(s.B):
        P = s.xyz[po[b]:po[b + 1]]
        vox = orc.voxel_downsample(P, Mq)["xyz"].astype(np.float32)[: Mq // 2]
        mem = P[np.linspace(0, len(P) - 1, Mq - len(vox)).astype(np.int64)]
        q.append(np.concatenate([vox, mem]))
        qo.append(qo[-1] + len(q[-1]))
    q, qo = np.concatenate(q), np.array(qo, np.int64)
    centre = np.stack([s.xyz[po[b]:po[b + 1]].mean(0) for b in range(s.B)]).astype(np.float32)
    single = s.B == 1
    g_n, g_w = _gpu(s.xyz, q, centre, k, None if single else po, None if single else qo)
    ref = orc.estimate_normals(s.xyz, q, centre, k, po, qo)
    cq = np.concatenate([np.repeat(centre[b:b + 1], qo[b + 1] - qo[b], 0) for b in range(s.B)]).astype(np.float64)
    _compare(g_n, g_w, ref, q, cq, s.xyz, po, qo)
    only, none = _gpu(s.xyz, q, centre, k, None if single else po, None if single else qo, want_evals=False)
    assert none is None and np.array_equal(only, g_n)


def test_plane_ties_and_empty_objects(orc):
    rng = np.random.default_rng(7)
    flat = np.concatenate([rng.uniform(-1, 1, (4000, 2)), np.full((4000, 1), 0.25)], 1).astype(np.float32)
    g_n, g_w = _gpu(flat, flat[:64], [[0, 0, -3]], 20)
    assert np.abs(g_n - [0, 0, 1]).max() < 1e-6 and np.abs(g_w[:, 0]).max() < 1e-9
    # every point twice: equal distances everywhere, the lower index wins on both sides
    dup = np.concatenate([flat[:1500], flat[:1500]])
    dup[:, 2] += (rng.uniform(-0.05, 0.05, 1500).astype(np.float32))[np.r_[0:1500, 0:1500]]
    ref = orc.estimate_normals(dup, dup[:50], [[0, 0, -3]], 7)
    assert (ref["gap"] == 0).mean() > 0.3                       # the k-th and the next one tie for many queries
    g_n, g_w = _gpu(dup, dup[:50], [[0, 0, -3]], 7)
    assert np.abs(g_w - ref["evals"]).max() <= 1e-5 * ref["evals"].max()
    well = (ref["evals"][:, 1] - ref["evals"][:, 0]) > 1e-3 * ref["evals"][:, 2]
    assert np.abs(g_n[well] - ref["normals"][well]).max() < 3e-7
    # an object without points, an object with one point, no queries for the last one
    xyz = np.concatenate([flat[:300], flat[300:301]])
    po, qo = np.array([0, 300, 300, 301, 301], np.int64), np.array([0, 2, 4, 6, 6], np.int64)
    q = flat[[0, 1, 2, 3, 4, 5]]
    centre = np.array([[0, 0, -3]] * 4, np.float32)
    g_n, g_w = _gpu(xyz, q, centre, 10, po, qo)
    assert np.abs(g_n[:2] - [0, 0, 1]).max() < 1e-6
    assert (g_n[2:4] == 0).all() and (g_w[2:4] == 0).all()       # no points
    assert np.allclose(np.linalg.norm(g_n[4:6], axis=1), 1.0, atol=1e-6) and (g_w[4:6] == 0).all()   # one point: any unit vector


def test_full_size_c2(orc):
    from workloads.scenes import make_scene
    s = make_scene("c2")
    q = orc.voxel_downsample(s.xyz, 150)["xyz"].astype(np.float32)
    centre = s.xyz.mean(0, keepdims=True).astype(np.float32)
    g_n, g_w = _gpu(s.xyz, q, centre, 30)
    ref = orc.estimate_normals(s.xyz, q, centre, 30)
    _compare(g_n, g_w, ref, q, np.repeat(centre.astype(np.float64), len(q), 0), s.xyz, s.pt_offsets, np.array([0, len(q)]))


def test_full_size_c4_cloud(orc):
    """The 1.68 M voxel centres of c4 as the cloud (one sweep per query over 20 MB), ~150 sampled points as queries."""
    from workloads.scenes import make_scene
    s = make_scene("c4")
    q = orc.voxel_downsample(s.xyz, 150)["xyz"].astype(np.float32)
    centre = s.xyz.mean(0, keepdims=True).astype(np.float32)
    g_n, g_w = _gpu(s.xyz, q, centre, 30)
    ref = orc.estimate_normals(s.xyz, q, centre, 30)
    # a regular voxel grid: many equal distances (ties at the k-th place go by index on both sides) and neighbourhoods
    # inside the solid that are not planes at all: the eigenvalues and the quadratic form decide, not the direction
    lam = ref["evals"]
    assert np.abs(g_w - lam).max() <= 1e-5 * lam[:, 2].max()
    P = s.xyz.astype(np.float64)
    for m in range(len(q)):
        nb = P[ref["nn_idx"][m]]
        cov = np.cov(nb.T, bias=True)
        assert g_n[m] @ cov @ g_n[m] <= lam[m, 0] + 1e-6 * lam[m, 2] + 1e-30


@pytest.mark.parametrize("k", [1, 255, 256, 257, 600])
def test_neighbourhood_sizes_around_the_limit_of_the_one_sweep_path(orc, k):
    """k up to 256 takes one sweep and an on-chip list, larger k the three-sweep radix select over the cloud; a cloud where
    thousands of points share the k-th distance overflows the list and takes the general path too."""
    from workloads.scenes import make_scene
    s = make_scene("c1", n_points=30_000)
    q = s.xyz[np.linspace(0, s.N - 1, 24).astype(np.int64)]
    centre = s.xyz.mean(0, keepdims=True).astype(np.float32)
    g_n, g_w = _gpu(s.xyz, q, centre, k)
    ref = orc.estimate_normals(s.xyz, q, centre, k)
    assert np.abs(g_w - ref["evals"]).max() <= 1e-5 * ref["evals"][:, 2].max()
    if k >= 255:      # many neighbours: a well-defined plane everywhere
        assert np.abs(np.abs(np.einsum("ij,ij->i", g_n, ref["normals"])) - 1.0).max() < 1e-6
    if k == 1:        # a shell of 6000 points at one distance from the query: more candidates than the list holds
        rng = np.random.default_rng(3)
        d = rng.standard_normal((6000, 3)); d /= np.linalg.norm(d, axis=1, keepdims=True)
        shell = np.concatenate([np.zeros((1, 3)), 0.5 * d]).astype(np.float32)
        shell[1:] = (0.5 * np.sign(d) * (np.abs(d) == np.abs(d).max(1, keepdims=True))).astype(np.float32)   # exactly 0.5 away
        g_n, g_w = _gpu(shell, np.zeros((1, 3), np.float32), [[0, 0, -1]], 200)
        ref = orc.estimate_normals(shell, np.zeros((1, 3), np.float32), [[0, 0, -1]], 200)
        assert np.abs(g_w - ref["evals"]).max() <= 1e-5 * ref["evals"][:, 2].max()


# The candidate list holds 8192 points: shells of points at one distance just inside and beyond it; and clouds on both sides
# of the sizes at which the strided subset halves (8192 points, and k times the stride above 1500).
@pytest.mark.parametrize("n,k", [(8_191, 200), (8_192, 200), (9_001, 200)])
def test_candidate_list_full_and_overflowing(orc, n, k):
    rng = np.random.default_rng(n)
    d = rng.standard_normal((n - 1, 3))
    far = (0.5 * np.sign(d) * (np.abs(d) == np.abs(d).max(1, keepdims=True))).astype(np.float32)   # exactly 0.5 away
    shell = np.concatenate([np.zeros((1, 3), np.float32), far])
    q = np.zeros((1, 3), np.float32)
    _, g_w = _gpu(shell, q, [[0, 0, -1]], k)
    ref = orc.estimate_normals(shell, q, [[0, 0, -1]], k)
    assert np.abs(g_w - ref["evals"]).max() <= 1e-5 * ref["evals"][:, 2].max()


@pytest.mark.parametrize("n,k", [(8_192, 30), (8_193, 30), (16_385, 256), (409_600, 30), (409_601, 30), (40_000, 256),
                                 (245_760, 256), (245_761, 256), (245_763, 256)])      # the subset's runs: quads, then points
def test_subset_sizes(orc, n, k):
    rng = np.random.default_rng(n + k)
    cloud = rng.standard_normal((n, 3)).astype(np.float32) * np.array([1.0, 0.6, 0.3], np.float32)
    q = cloud[:: n // 5][:5]
    centre = cloud.mean(0, keepdims=True).astype(np.float32)
    _, g_w = _gpu(cloud, q, centre, k)
    ref = orc.estimate_normals(cloud, q, centre, k)
    assert np.abs(g_w - ref["evals"]).max() <= 1e-5 * ref["evals"][:, 2].max()


@pytest.mark.parametrize("n,k", [(300_000, 30), (1_000_003, 128)])      # quads, then single points
def test_cloud_in_scanner_order(orc, n, k):
    """A surface stored row after row, where the points of a quad are next to each other in space."""
    rng = np.random.default_rng(k)
    rows = int(np.sqrt(n / 2))
    cols = -(-n // rows)
    z = np.repeat(1 - 2 * (np.arange(rows) + 0.5) / rows, cols)[:n]
    a = np.tile(np.arange(cols) * (2 * np.pi / cols), rows)[:n]
    r = np.sqrt(1 - z * z)
    cloud = (np.stack([r * np.cos(a), r * np.sin(a), z], 1) * [1.0, 0.7, 0.45] + 0.1 / rows * rng.standard_normal((n, 3))).astype(np.float32)
    q = cloud[rng.integers(0, n, 40)]
    q[0], q[1] = cloud[0], cloud[-1]
    centre = np.zeros((1, 3), np.float32)
    g_n, g_w = _gpu(cloud, q, centre, k)
    ref = orc.estimate_normals(cloud, q, centre, k)
    _compare(g_n, g_w, ref, q, np.zeros((len(q), 3)), cloud, np.array([0, n]), np.array([0, len(q)]))


# The selects end with the first of three passes (11, 11 and 10 bits of the distance) that separates the k-th from the next: pairs
# that each of them separates, neighbouring floats, and a tie.  The two points lie along different axes, so taking the
# wrong one changes the eigenvalues by far more than the bar.
@pytest.mark.parametrize("n,k", [(3_000, 5), (10_000, 200), (10_000, 300)])      # whole cloud in the list, one sweep, general path
@pytest.mark.parametrize("next_r", [1.25, 0.8015, 0.80001, "float", "tie"])
def test_distances_that_each_pass_of_the_select_separates(orc, n, k, next_r):
    rng = np.random.default_rng(k)
    r = np.float32(0.8)
    r_next = {"float": np.nextafter(r, np.float32(1)), "tie": r}.get(next_r, next_r)
    d = rng.standard_normal((n, 3))
    d *= np.concatenate([rng.uniform(0.2, 0.5, k - 1), [1, 1], rng.uniform(2, 3, n - k - 1)])[:, None] / np.linalg.norm(d, axis=1, keepdims=True)
    cloud = d.astype(np.float32)
    cloud[k - 1], cloud[k] = [r, 0, 0], [0, r_next, 0]
    cloud = cloud[rng.permutation(n)]
    q = np.zeros((1, 3), np.float32)
    _, g_w = _gpu(cloud, q, [[0, 0, -1]], k)
    ref = orc.estimate_normals(cloud, q, [[0, 0, -1]], k)
    assert np.abs(g_w - ref["evals"]).max() <= 1e-5 * ref["evals"][:, 2].max()


# Covariances that the rotations meet as special cases: no entry off the diagonal, one, equal entries on the diagonal with a
# positive and a negative one beside them, equal entries everywhere, one and no dimension.
_AXES = np.concatenate([np.diag(s * np.array([1.0, 2.0, 4.0])) for s in (1, -1)])


@pytest.mark.parametrize("cloud", [
    pytest.param(_AXES, id="diagonal"),
    pytest.param(_AXES[:, ::-1], id="diagonal descending"),
    pytest.param(np.concatenate([np.eye(3), -np.eye(3)]), id="sphere"),
    pytest.param([[1, 1, 0], [-1, -1, 0], [0, 0, 2], [0, 0, -2]], id="positive in xy"),
    pytest.param([[1, -1, 0], [-1, 1, 0], [0, 0, 2], [0, 0, -2]], id="negative in xy"),
    pytest.param([[1, 0, -1], [-1, 0, 1], [0, 2, 0], [0, -2, 0]], id="negative in xz"),
    pytest.param([[0, 1, -1], [0, -1, 1], [2, 0, 0], [-2, 0, 0]], id="negative in yz"),
    pytest.param([[1, 1, 1], [-1, -1, -1], [2, 2, 2]], id="line, positive"),
    pytest.param([[1, -1, 1], [-1, 1, -1], [2, -2, 2]], id="line, mixed signs"),
    pytest.param([[0, 0, 3], [0, 0, -3]], id="line along an axis"),
    pytest.param([[0, 0, 0], [0, 0, 0]], id="one place"),
])
@pytest.mark.parametrize("scale", [1.0, 1e-17, 1e17])      # fp32 squares of the distances are subnormal, or nearly the largest
def test_special_covariances(cloud, scale):
    cloud = (np.asarray(cloud, np.float64) * scale).astype(np.float32)
    g_n, g_w = _gpu(cloud, np.zeros((1, 3), np.float32), [[0.5, 0.25, -3]], len(cloud))
    cov = np.cov(cloud.astype(np.float64).T, bias=True)
    lam = np.linalg.eigvalsh(cov)
    # sums, rotations and the reference are fp64 with a few dozen operations; eigenvalues are stored as fp32 (half a unit: 6e-8,
    # below 1.2e-38 half of 1.4e-45)
    assert np.abs(g_w[0] - lam).max() <= 1e-7 * lam[2] + 1e-45
    assert abs(np.linalg.norm(g_n[0]) - 1) < 2e-7 and g_n[0] @ cov @ g_n[0] <= lam[0] + 1e-12 * lam[2]

"""The subset of a cloud that bounds the k-th distance in aura_estimate_normals, on the CPU: how many points lie within the bound,
against what the kernel's list holds.  A query that finds more is answered by several sweeps of one workgroup, ten times as
long as the others, and sets the time of its call."""
import ctypes
import subprocess
from pathlib import Path

import numpy as np
import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2511_03126_amd" / "csrc"


@pytest.fixture(scope="module")
def subset(tmp_path_factory):
    d = tmp_path_factory.mktemp("subset")
    (d / "s.cpp").write_text('#include "normals_subset.hpp"\n'
                             'extern "C" void subset(int n, int k, int* o) {\n'
                             '  const aura::NrmSubset s = aura::nrm_subset(n, k);\n'
                             '  o[0] = s.run; o[1] = s.stride; o[2] = s.count; o[3] = aura::kNrmCand; o[4] = aura::kNrmSub;\n}\n'
                             'extern "C" void quad(int g, int n, int* o) {\n'
                             '  const aura::NrmQuad q = aura::nrm_quad(g, n);\n'
                             '  o[0] = q.first; o[1] = q.skip; o[2] = aura::nrm_quads(n);\n}\n')
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", "-o", str(d / "s.so"), str(d / "s.cpp")], check=True)
    lib = ctypes.CDLL(str(d / "s.so"))

    def call(n, k):
        o = (ctypes.c_int * 5)()
        lib.subset(n, k, o)
        return list(o)

    def quad(g, n):
        o = (ctypes.c_int * 3)()
        lib.quad(g, n, o)
        return list(o)
    call.quad = quad
    return call


def _scan(n, seed):
    """An ellipsoid's surface in the order of a scanner: row after row, neighbours next to each other."""
    rng = np.random.default_rng(seed)
    rows = int(np.sqrt(n / 2))
    cols = -(-n // rows)
    z = np.repeat(1 - 2 * (np.arange(rows) + 0.5) / rows, cols)[:n]
    a = np.tile(np.arange(cols) * (2 * np.pi / cols), rows)[:n]
    r = np.sqrt(1 - z * z)
    p = np.stack([r * np.cos(a), r * np.sin(a), z], 1) * np.array([1.0, 0.7, 0.45])
    return (p + 0.1 / rows * rng.standard_normal((n, 3))).astype(np.float32)


def _morton(p):
    q = ((p - p.min(0)) / (p.max(0) - p.min(0)) * 1023).astype(np.int64)
    key = sum(((q[:, a] >> b) & 1) << (3 * b + a) for b in range(10) for a in range(3))
    return p[np.argsort(key, kind="stable")]


@pytest.mark.parametrize("n,k,order", [(200_000, 30, "scan"), (1_000_000, 30, "scan"), (1_500_000, 64, "scan"),
                                       (3_000_000, 30, "scan"), (2_000_000, 30, "morton"), (300_000, 200, "scan")])
def test_candidates_fit_the_list(subset, n, k, order):
    p = _scan(n, n + k) if order == "scan" else _morton(_scan(n, n + k))
    run, stride, count, cap, _ = subset(n, k)
    idx = (np.arange(count)[:, None] * (run * stride) + np.arange(run)).reshape(-1)
    over = 0
    for m in np.random.default_rng(7).integers(0, n, 60):
        d = ((p - p[m]) ** 2).sum(1)
        over += int((d <= np.partition(d[idx], k - 1)[k - 1]).sum()) > cap
    assert over == 0


def test_subset_stays_in_the_cloud_and_in_its_array(subset):
    for n in [8_193, 8_194, 8_195, 8_196, 16_384, 16_385, 40_000, 409_600, 409_601, 1_000_003, 2_999_999, 2 ** 31 - 1]:
        for k in (1, 2, 30, 64, 200, 256):
            run, stride, count, _, most = subset(n, k)
            assert (count - 1) * run * stride + run <= n and k <= count * run <= most


@pytest.mark.parametrize("n", [8_193, 8_194, 8_195, 8_196, 2 ** 31 - 16_384, 2 ** 31 - 4, 2 ** 31 - 3, 2 ** 31 - 2, 2 ** 31 - 1])
def test_sweep_reads_every_point_once(subset, n):
    """The first quads and the last, and those that threads beyond the end read: inside the cloud, every point added once."""
    quads = subset.quad(0, n)[2]
    assert 4 * (quads - 1) < n <= 4 * quads
    for g in [0, 1, quads // 2]:
        assert subset.quad(g, n)[:2] == [4 * g, 0]
    added = []
    for g in range(quads - 3, quads + 4 * 1024):
        first, skip, _ = subset.quad(g, n)
        assert 0 <= first and first + 4 <= n and skip >= 0
        added += range(first + min(skip, 4), first + 4)
    assert added == list(range(4 * (quads - 3), n))

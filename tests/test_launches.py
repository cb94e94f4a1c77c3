"""What the fusion calls launch, without a GPU: launch_recorder.cpp stands in for the HIP runtime."""
import re
import subprocess
from pathlib import Path

import pytest

ROOT = Path(__file__).resolve().parent.parent
PKG = ROOT / "paper_2511_03126_amd"
F16, MEAN_ONLY, GATHER, TWO_KERNELS = 2, 2, 4, 8


@pytest.fixture(scope="module")
def recorder(tmp_path_factory):
    from paper_2511_03126_amd import build
    if not build.LIB.exists():
        build.build()
    exe = tmp_path_factory.mktemp("recorder") / "recorder"
    subprocess.run(["g++", "-O1", "-std=c++17", "-rdynamic", str(ROOT / "tests" / "launch_recorder.cpp"), "-o", str(exe), f"-L{PKG}",
                    "-l:libaura_fuse.so", f"-Wl,-rpath,{PKG}", "-Wl,--allow-shlib-undefined"], check=True)

    def run(lines):
        """Per line its status and its launches: (kernel with template arguments, grid x, grid y, block), "S" and "E"."""
        out = subprocess.run([str(exe)], input="\n".join(lines), capture_output=True, text=True, check=True).stdout.splitlines()
        assert len(out) == len(lines)
        return [(int(o.split()[0]), [_launch(x) for x in o.split()[1:]]) for o in out]
    run.names = lambda: subprocess.run([str(exe), "names"], capture_output=True, text=True, check=True).stdout.split()
    return run


def _launch(text):
    m = re.fullmatch(r"(\S+)\((\d+),(\d+),(\d+)\)", text)
    return (_short(m[1]), int(m[2]), int(m[3]), int(m[4])) if m else text


def _short(mangled):
    """k_tile_fused<2,4,1,2,0,4,1,1> of its mangled name."""
    m = re.match(r"_ZN4aura(\d+)", mangled)
    end = m.end() + int(m[1])
    args = re.findall(r"L[ib](\d+)E", re.split(r"EEv", mangled[end:])[0] + "E")
    return mangled[m.end():end] + (f"<{','.join(args)}>" if args else "")


def _call(call="single", N=1_000_000, B=1, V=8, H=448, Hf=56, D=512, dtype=F16, K=24, P=1, flags=0, eps=1e-12, T=0.1, fail="-"):
    return f"{call} {N} {B} {V} {H} {Hf} {D} {dtype} {K} {P} {flags} {eps} {T} {fail}"


@pytest.mark.parametrize("kw,kernels", [
    (dict(), ["k_tile_sift", "k_tile_fused"]),
    (dict(call="scores"), ["k_tile_fused"]),
    (dict(call="fuse", flags=TWO_KERNELS), ["k_tile_prepare", "k_tile_product"]),
    (dict(call="fuse", N=10_000, V=2, Hf=16), ["k_fuse_gather"]),
])
def test_both_events_are_recorded_whichever_launch_fails(recorder, kw, kernels):
    """A caller that timed a call waits for the second event: it is recorded on every way out once the first one is."""
    for fail in ["-"] + kernels:
        (status, log), = recorder([_call(**kw, fail=fail)])
        assert (status == 0) == (fail == "-") and log.count("S") == log.count("E") == 1, (fail, log)
        inside = [x[0].split("<")[0] for x in log[log.index("S") + 1:log.index("E")]]
        assert inside == (kernels if fail == "-" else kernels[:kernels.index(fail) + 1])


def test_every_instance_of_the_one_kernel_fusion_is_launched_by_some_call(recorder):
    """Over channels, types, objects, points, views, cells and materials on both sides of every line of the dispatch."""
    calls = [_call(call, N=N, B=B, V=V * B, Hf=Hf, D=D, dtype=dtype, K=K)
             for call in ("single", "scores", "fuse", "selected") for dtype in (1, F16) for D in (256, 512, 768, 1024)
             for B in (1, 2, 3, 12, 64) for N in (20_000, 100_000, 300_000, 1_000_000, 3_000_000) for V in (2, 4, 7, 12)
             for Hf in (28, 224) for K in (24, 45)]
    launched = {x[0] for status, log in recorder(calls) if status == 0 for x in log if x[0].startswith("k_tile_fused<")}
    assert launched == {_short(n) for n in recorder.names() if "k_tile_fused" in n}


@pytest.mark.parametrize("kw,sieve", [
    (dict(), True), (dict(K=100), True), (dict(T="inf"), True),        # (weights of exp(0 * 0))
    (dict(eps=0.0), True), (dict(eps=1e-31), True), (dict(eps=0.0, flags=MEAN_ONLY), True),   # (the factor of an unseen point is 0)
    (dict(T=1e-39), False),                                            # exp(0 * inf)
    (dict(call="scores"), False), (dict(N=262_112), False), (dict(N=262_113), True),
    (dict(N=384_033, V=6, D=256, K=40), True), (dict(N=262_112, V=6, D=256, K=40), False),   # one producer, four
    (dict(N=8 * 49_152 * 32), True), (dict(N=8 * 49_152 * 32 + 1), True), (dict(N=50_000_000), True),   # lists of any length
    (dict(N=5 * 78_625, B=5, V=20, Hf=16), False), (dict(N=5 * 79_969, B=5, V=20, Hf=16), True),    # several objects: 12 288 tiles in all,
    (dict(N=3 * 131_000, B=3, V=12, Hf=16), False), (dict(N=3 * 131_073, B=3, V=12, Hf=16), True),  # 2500 for each
])
def test_the_sieve_is_left_out_where_unseen_tiles_are_not_zero_or_not_worth_it(recorder, kw, sieve):
    (status, log), = recorder([_call(**kw)])
    kernels = [x[0] for x in log if x not in ("S", "E")]
    fused, = [k for k in kernels if k.startswith("k_tile_fused<")]
    assert status == 0 and ("k_tile_sift" in kernels) == sieve and fused.endswith(",1>" if sieve else ",0>")


@pytest.mark.parametrize("D,staged", [(512, True), (500, False), (1 << 25, True), ((1 << 25) + 32, False), (1 << 26, False)])
def test_the_densification_stages_rows_whose_places_fit_32_bits(recorder, D, staged):
    """A wave's 32 rows are reached by 32-bit offsets in bytes there: longer ones go through registers."""
    (status, log), = recorder([_call("densify", N=64, B=64, D=D)])
    kernel, = [x[0] for x in log if x[0].startswith("k_knn_densify<")]
    assert status == 0 and kernel == f"k_knn_densify<2,1,{int(staged)}>"

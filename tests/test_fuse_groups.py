"""How many workgroups an object gets in one launch of the one-kernel fusion over several objects, on the CPU: the launch must
not end in a last round that is a small part of what the machine holds."""
import ctypes
import subprocess
from pathlib import Path

import pytest

CSRC = Path(__file__).resolve().parent.parent / "paper_2511_03126_amd" / "csrc"


@pytest.fixture(scope="module")
def groups(tmp_path_factory):
    d = tmp_path_factory.mktemp("groups")
    (d / "g.cpp").write_text('#include "fuse_tile_groups.hpp"\n'
                             'extern "C" int groups(int s, int np, int n, int resident, int tiles) {\n'
                             '  return aura::fused_groups_per_object(s, np, n, resident, tiles);\n}\n')
    subprocess.run(["g++", "-O2", "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", "-o", str(d / "g.so"), str(d / "g.cpp")], check=True)
    return ctypes.CDLL(str(d / "g.so")).groups


# (channels / 256, producers, resident workgroups) of the forms that store rows
@pytest.mark.parametrize("s,np,resident", [(1, 1, 1024), (2, 1, 512), (2, 4, 256), (3, 4, 256), (4, 4, 256)])
def test_few_objects_keep_the_larger_number(groups, s, np, resident):
    for n in range(2, 65):
        got = groups(s, np, n, resident, 6250)
        assert got in (128, 256)
        if s > 1 and n * 128 < (4 if np == 1 else 6) * resident:      # (256 channels: 128 measured faster from five objects on)
            assert got == 256
        for tiles in (1, 63, 64, 153, 1000, 1500):     # at least eight tiles per workgroup, whole rounds of the XCDs
            got = groups(s, np, n, resident, tiles)
            assert got * 8 <= tiles and got % 8 == 0 and got <= 256

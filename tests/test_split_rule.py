"""The rule that splits a workgroup's waves into groups on small grids, on the
host: the function and its constants are taken from the sources and compiled
with g++, and its choices compared with measured times."""
import re
import shutil
import subprocess
from pathlib import Path

import ctypes
import pytest

CSRC = Path(__file__).resolve().parents[1] / "paper_2609_34420_amd" / "csrc"
KINDS = ("fwd", "dq", "dkdv")

# (kernel, heads, rows = columns, head dim): us with 1, 2 and 4 groups
MEASURED = [
    ("fwd", 32768, 64, 64, 1063, 1501, 1422), ("fwd", 16384, 128, 64, 694, 787, 826),
    ("fwd", 8192, 256, 64, 520, 572, 928), ("fwd", 1600, 576, 64, 432, 441, 543),
    ("fwd", 192, 1536, 64, 197, 212, 232), ("fwd", 8, 8256, 64, 277, 313, 275),
    ("fwd", 16, 4096, 64, 142, 89, 104), ("fwd", 8, 4160, 64, 145, 82, 102),
    ("fwd", 16, 6000, 64, 216, 239, 227), ("fwd", 16, 5500, 64, 198, 223, 199),
    ("dq", 4, 8256, 64, 190, 215, 198), ("dq", 4, 9000, 64, 209, 239, 216),
    ("fwd", 8, 16384, 64, 655, 662, 737), ("fwd", 16384, 128, 8, 485, 516, 676),
    ("fwd", 8, 8256, 8, 234, 243, 197), ("fwd", 16, 4096, 8, 115, 65, 73),
    ("dq", 32768, 64, 64, 991, 1218, 1243), ("dq", 16384, 128, 64, 654, 710, 1218),
    ("dq", 8, 8256, 64, 403, 333, 329), ("dq", 8, 4160, 64, 101, 117, 109),
    ("dq", 8, 16384, 64, 869, 914, 1063), ("dq", 8, 8256, 8, 267, 212, 200),
    ("dkdv", 8, 8256, 64, 680, 577, 569), ("dkdv", 16, 6144, 64, 521, 450, 524),
    ("dkdv", 8, 16384, 64, 1510, 1537, 1744), ("dkdv", 3200, 320, 64, 594, 637, 845),
    ("dkdv", 16, 6144, 8, 411, 321, 382), ("dkdv", 3200, 320, 8, 356, 405, 515),
]


@pytest.fixture(scope="module")
def pick(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no g++")
    head, src = (CSRC / "kernels.hpp").read_text(), (CSRC / "fwd.hip").read_text()
    parts = [re.search(r"struct SplitCost \{.*?\n\};", head, re.S).group(0)]
    parts += [re.search(rf"inline SplitCost {k}_split_cost\(int D\) \{{.*?\n\}}", head, re.S).group(0) for k in KINDS]
    parts.append(re.search(r"^int pick_split\(.*?\n\}", src, re.S | re.M).group(0))
    parts += [f'extern "C" int pick_{k}(int64_t n, int64_t heads, int D) '
              f"{{ return pick_split(n, n, heads, {k}_split_cost(D)); }}" for k in KINDS]
    d = tmp_path_factory.mktemp("split")
    (d / "s.cpp").write_text("#include <cstdint>\n" + "\n".join(parts) + "\n")
    subprocess.run([cxx, "-O1", "-shared", "-fPIC", str(d / "s.cpp"), "-o", str(d / "s.so")], check=True)
    lib = ctypes.CDLL(str(d / "s.so"))
    out = {}
    for k in KINDS:
        out[k] = getattr(lib, f"pick_{k}")
        out[k].argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int]
    return out


@pytest.mark.parametrize("kind,heads,n,d,t1,t2,t4", MEASURED)
def test_choice_is_close_to_the_best(pick, kind, heads, n, d, t1, t2, t4):
    """Within 3 % of the best of the three."""
    t = {1: t1, 2: t2, 4: t4}
    ks = pick[kind](n, heads, 64 if d == 64 else 32)
    assert t[ks] <= 1.03 * min(t.values()), (ks, t)


def test_cost_constants_match_the_kernels(pick):
    """Rows and tiles of the costs are the kernels'."""
    text = (CSRC / "stage.hpp").read_text() + (CSRC / "bwd_dkdv.hip").read_text()
    assert "64 * KS < (D == 64 ? 128 : 256) ? 64 * KS : (D == 64 ? 128 : 256)" in text
    assert "D == 64 && QS == 2 ? 64 : (QS == 1 ? 64 : 128)" in text
    head = (CSRC / "kernels.hpp").read_text()
    for rows in (512, 256):
        assert f"{{{rows}, {{64, 128, 128}}" in head and f"{{{rows}, {{64, 128, 256}}" in head

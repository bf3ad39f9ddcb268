"""Which plane segments of a batch share a launch (plane_lists.hpp, host code):
every segment exactly once, no more of them in a launch than its argument
block holds, the same launches whichever shape the batch names first, and a
launch of their own only for much smaller planes (LDS under 60 %) with enough
workgroups on both sides."""
import ctypes
import os
import random
import shutil
import subprocess

import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2204_08834_amd", "csrc")
SRC = r"""
#include "plane_lists.hpp"
extern "C" int launches(const long *lds, const long *planes, int n, int max_seg, int *out)
{
    std::vector<pk::PlaneSeg> s(n);
    for (int i = 0; i < n; ++i) s[i] = pk::PlaneSeg{(size_t)lds[i], planes[i]};
    const auto r = pk::plane_launches(s, max_seg);
    int k = 0;
    for (size_t j = 0; j < r.size(); ++j)
        for (int i : r[j]) { out[2 * k] = (int)j; out[2 * k + 1] = i; ++k; }
    return k;
}
"""


@pytest.fixture(scope="module")
def launches(tmp_path_factory):
    cxx = shutil.which("g++")
    if not cxx:
        pytest.skip("no host compiler")
    d = tmp_path_factory.mktemp("plane_lists")
    src, so = d / "t.cpp", d / "t.so"
    src.write_text(SRC)
    subprocess.run([cxx, "-std=c++17", "-O1", "-shared", "-fPIC", f"-I{CSRC}", str(src), "-o", str(so)],
                   check=True)
    fn = ctypes.CDLL(str(so)).launches

    def run(segs, max_seg=8):
        n = len(segs)
        arr = ctypes.c_long * n
        out = (ctypes.c_int * (2 * n + 2))()
        k = fn(arr(*[s[0] for s in segs]), arr(*[s[1] for s in segs]), n, max_seg, out)
        assert k == n
        got = [[] for _ in range(out[2 * (k - 1)] + 1 if k else 0)]
        for i in range(k):
            got[out[2 * i]].append(out[2 * i + 1])
        return got
    return run


def _lds(nx, ny):
    """Bytes of an FP32 plane, about (the tile; the tables are small)."""
    return 8 * (nx // 2 + 1) * ny


def test_small_deep_planes_before_large_shallow_ones(launches):
    # 16 problems of 64x64x96 (first by points) and 8 of 128x128x16
    a, b = (_lds(64, 64), 16 * 96), (_lds(128, 128), 8 * 16)
    assert launches([a, b]) == [[1], [0]]
    assert launches([b, a]) == [[0], [1]]


def test_few_planes_share_one_launch(launches):
    segs = [(_lds(64, 64), 64), (_lds(128, 128), 64), (_lds(96, 96), 48), (_lds(64, 128), 80),
            (_lds(128, 64), 50), (_lds(48, 96), 64), (_lds(32, 64), 96)]
    got = launches(segs)
    assert len(got) == 1 and sorted(got[0]) == list(range(7))


def test_rule_over_random_batches(launches):
    rng = random.Random(4)
    for _ in range(300):
        n = rng.randint(0, 20)
        segs = [(rng.randint(1, 160) * 1024, int(2 ** rng.uniform(0, 12))) for _ in range(n)]
        max_seg = rng.choice([1, 2, 8])
        got = launches(segs, max_seg)
        assert sorted(i for one in got for i in one) == list(range(n))
        assert all(1 <= len(one) <= max_seg for one in got)
        flat = [i for one in got for i in one]
        assert all(segs[i][0] >= segs[j][0] for i, j in zip(flat, flat[1:]))
        for one, nxt in zip(got, got[1:]):
            held = sum(segs[i][1] for i in one)
            rest = sum(segs[i][1] for later in got[got.index(nxt):] for i in later)
            small = 5 * segs[nxt[0]][0] < 3 * segs[one[0]][0]
            assert len(one) == max_seg or (small and held >= 128 and rest >= 512)
        order = list(range(n))
        rng.shuffle(order)
        again = launches([segs[i] for i in order], max_seg)
        assert [[segs[order[i]][0] for i in one] for one in again] == \
            [[segs[i][0] for i in one] for one in got] or len({s[0] for s in segs}) < n

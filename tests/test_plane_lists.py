"""Which plane segments of a batch share a launch (plane_lists.hpp, host code):
every segment exactly once and in order, no more of them in a launch than its
argument block holds, and a launch of their own only for planes of much smaller
or much larger LDS (60 %) with enough workgroups to gain from it."""
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
extern "C" int launches(const long *lds, const long *planes, const int *threads, int n, int max_seg, int *out)
{
    std::vector<pk::PlaneSeg> s(n);
    for (int i = 0; i < n; ++i) s[i] = pk::PlaneSeg{(size_t)lds[i], threads[i], planes[i]};
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
        k = fn(arr(*[s[0] for s in segs]), arr(*[s[1] for s in segs]),
               (ctypes.c_int * n)(*[s[2] for s in segs]), n, max_seg, out)
        assert k == n
        got = [[] for _ in range(out[2 * (k - 1)] + 1 if k else 0)]
        for i in range(k):
            got[out[2 * i]].append(out[2 * i + 1])
        return got
    return run


def _seg(nx, ny, planes):
    """An FP32 plane: bytes of its tile (the tables are small), planes, threads."""
    return 8 * (nx // 2 + 1) * ny, planes, -(-(nx // 2 * ny) // 512) * 64


def test_small_deep_planes_before_large_shallow_ones(launches):
    # 16 problems of 64x64x96 (more points) and 8 of 128x128x16, and few large
    # planes with more points than the many small ones after them
    assert launches([_seg(64, 64, 16 * 96), _seg(128, 128, 8 * 16)]) == [[0], [1]]
    assert launches([_seg(128, 128, 200), _seg(32, 32, 2000)]) == [[0], [1]]
    assert launches([_seg(64, 64, 300), _seg(128, 128, 20)]) == [[0, 1]]


def test_few_planes_share_one_launch(launches):
    segs = [_seg(128, 128, 64), _seg(64, 128, 80), _seg(96, 96, 48), _seg(128, 64, 50),
            _seg(48, 96, 64), _seg(64, 64, 64), _seg(32, 64, 96)]
    assert launches(segs) == [list(range(7))]


def test_a_large_batch_is_split_by_plane_size(launches):
    segs = [_seg(128, 128, 16 * 64), _seg(96, 96, 24 * 48), _seg(64, 64, 24 * 64)]
    assert launches(segs) == [[0], [1], [2]]
    # two shapes: one round of the smaller planes is enough
    assert launches([_seg(96, 128, 924), _seg(48, 128, 340)]) == [[0], [1]]
    assert launches([_seg(128, 128, 256), _seg(32, 32, 256)]) == [[0, 1]]


def test_rule_over_random_batches(launches):
    rng = random.Random(4)
    for _ in range(300):
        n = rng.randint(0, 20)
        segs = [(rng.randint(1, 160) * 1024, int(2 ** rng.uniform(0, 12)), 64 * rng.randint(1, 16))
                for _ in range(n)]
        max_seg = rng.choice([1, 2, 8])
        got = launches(segs, max_seg)
        assert [i for one in got for i in one] == list(range(n))
        assert all(1 <= len(one) <= max_seg for one in got)
        for one, nxt in zip(got, got[1:]):
            lds = [segs[i][0] for i in one]
            new = segs[nxt[0]][0]
            small, large = 5 * new < 3 * max(lds), 5 * min(lds) < 3 * new
            assert len(one) == max_seg or small or large
            if len(one) < max_seg:  # a split of fewer than 300 planes never pays
                assert sum(segs[i][1] for i in (range(nxt[0], n) if small else one)) >= 300

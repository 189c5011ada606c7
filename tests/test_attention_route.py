"""The rule that picks the attention kernel of a batch (attention_route.h, host code
without device types), compiled and called on the CPU: its lines from both sides,
and what every answer has to keep: a grid the launch takes, parts that fit the
workspace's slots, and whole items only where one CU's time for the longest
context is short."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

CSRC = os.path.join(os.path.dirname(os.path.dirname(os.path.abspath(__file__))),
                    "paper_2609_29364_amd", "csrc")
CUS, SLOTS = 256, 4096


@pytest.fixture(scope="module")
def route(tmp_path_factory):
    cxx = shutil.which(os.environ.get("CXX", "g++")) or shutil.which("c++")
    if not cxx:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("route")
    (d / "route.cpp").write_text(
        '#include "attention_route.h"\n'
        'extern "C" int route(int64_t items, int64_t b, int d, int mt, int fuse, int cus,\n'
        '                     int64_t slots) {\n'
        '  return item_split(items, b, d, mt, fuse != 0, cus, slots);\n}\n')
    subprocess.run([cxx, "-std=c++17", "-shared", "-fPIC", f"-I{CSRC}", str(d / "route.cpp"), "-o",
                    str(d / "route.so")], check=True)
    f = ctypes.CDLL(str(d / "route.so")).route
    f.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int, ctypes.c_int,
                  ctypes.c_int, ctypes.c_int64]

    def call(items, tokens, d, mt, fuse, cus=CUS, slots=SLOTS):
        return f(items, tokens * d * 4, d, mt, fuse, cus, slots)
    return call


def test_every_answer_can_be_launched(route):
    rng = np.random.default_rng(0)
    shapes = [(int(2 ** rng.uniform(0, 33)), int(2 ** rng.uniform(0, 31)), int(rng.choice([64, 128])),
               int(rng.integers(1, 5)), int(rng.integers(0, 2)), int(rng.choice([64, 256, 304])))
              for _ in range(20000)]
    shapes += [(n, t, d, mt, f, CUS) for n in (1, 128, 129, 2048, 2049, 16384, 16385, 1 << 24, 1 << 31)
               for t in (1, 256, 1024) for d in (64, 128) for mt in (1, 4) for f in (0, 1)]
    for items, tokens, d, mt, fuse, cus in shapes:
        slots = 16 * cus
        n = route(items, tokens, d, mt, fuse, cus, slots)
        assert 0 <= n
        assert items * n * 256 < 1 << 32                      # threads of one launch
        assert n <= 1 or items * n <= slots


def test_whole_items_are_short(route):
    """A whole item streams at about 49 bytes per ns from one CU: neither one, nor two that meet
    on a CU where items are more than CUs, may outlast the wave split of a batch whose other
    contexts are short (about 24 us at head_dim 64, 34 at 128, 41 with several row tiles)."""
    for d in (64, 128):
        for mt in range(1, 5):
            for fuse in (0, 1):
                for items in (1, 100, 129, 192, 256, 257, 512, 513, 2048, 4096, 16384):
                    most = (1024 if items <= CUS else 384 if d == 64 else 768) << 10
                    if fuse or d * mt > 384:       # (their wave split takes 45 us and more)
                        most = 768 << 10
                    for tokens in range(64, 70000, 64):
                        if route(items, tokens, d, mt, fuse) == 1:
                            assert tokens * d * 4 <= most


# (items, tokens, head_dim, row tiles, fused) just inside a line -> what is just outside it
@pytest.mark.parametrize("inside,outside", [
    ((256, 2048, 128, 2, 0), (256, 2049, 128, 2, 0)),
    ((256, 4096, 64, 2, 0), (256, 4097, 64, 2, 0)),
    ((256, 2048, 128, 1, 0), (257, 2048, 128, 1, 0)),
    ((512, 1536, 128, 2, 0), (513, 1536, 128, 2, 0)),
    ((512, 1536, 128, 3, 0), (512, 1537, 128, 3, 0)),
    ((512, 1024, 128, 1, 0), (512, 1025, 128, 1, 0)),
    ((512, 1536, 64, 2, 0), (512, 1537, 64, 2, 0)),
    ((2048, 1024, 128, 2, 0), (2049, 1024, 128, 2, 0)),
    ((16384, 1024, 128, 1, 0), (16385, 1024, 128, 1, 0)),
    ((16384, 1536, 64, 2, 0), (16384, 1537, 64, 2, 0)),
    ((2048, 1536, 64, 3, 0), (2049, 1536, 64, 3, 0)),
    ((256, 1536, 128, 2, 1), (256, 1537, 128, 2, 1)),
    ((512, 1024, 128, 2, 1), (513, 1024, 128, 2, 1)),
    ((2048, 512, 128, 2, 1), (2049, 512, 128, 2, 1)),
    ((16384, 512, 64, 2, 1), (16384, 513, 64, 2, 1)),
    ((512, 1024, 128, 4, 0), (513, 1024, 128, 4, 0)),
    ((512, 1024, 128, 4, 1), (512, 1025, 128, 4, 1)),
])
def test_lines(route, inside, outside):
    assert route(*inside) == 1 and route(*outside) == 0


@pytest.mark.parametrize("shape,cut", [
    ((128, 1025, 128, 2, 0), True), ((129, 4096, 128, 2, 0), False),
    ((128, 513, 128, 2, 1), True), ((16, 1025, 128, 4, 0), True), ((17, 1025, 128, 4, 0), False),
    ((128, 4096, 128, 2, 1), True), ((128, 4097, 128, 2, 1), False),
])
def test_cut_items(route, shape, cut):
    n = route(*shape)
    assert n > 1 if cut else n == 0

"""The integer arithmetic of the work partition (csrc/partition.h, the functions
that the kernels and the launches use), compiled for the host and compared with
the definition: range w of W starts at page floor(pages * w / W)."""
import ctypes
import os
import random
import subprocess

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = """
#include "partition.h"
using namespace tsattn;
extern "C" int64_t start(int64_t ptot, int w, int ranges) {
    return range_start(ptot, w, ranges, range_reciprocal(ranges));
}
extern "C" int split(int64_t ptot, int64_t us, int np, int W, int *wlo_whi, int *slots, int cap) {
    const UnitSplit u = unit_split(ptot, us, np, W);
    wlo_whi[0] = u.wlo;
    wlo_whi[1] = u.whi;
    for (int k = 0; k < u.nparts && k < cap; k++)
        slots[k] = u.slot(k);
    return u.nparts;
}
"""


@pytest.fixture(scope="module")
def part(tmp_path_factory):
    d = tmp_path_factory.mktemp("partition")
    (d / "shim.cpp").write_text(SHIM)
    subprocess.run(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2608_22788_amd", "csrc"), str(d / "shim.cpp"), "-o", str(d / "shim.so")],
                   check=True)
    lib = ctypes.CDLL(str(d / "shim.so"))
    lib.start.argtypes, lib.start.restype = [ctypes.c_int64, ctypes.c_int, ctypes.c_int], ctypes.c_int64
    lib.split.argtypes = [ctypes.c_int64, ctypes.c_int64, ctypes.c_int, ctypes.c_int] + [ctypes.c_void_p] * 2 + [
        ctypes.c_int]
    return lib


def test_range_begin_is_the_exact_quotient(part):
    rng = random.Random(1)
    for ranges in list(range(1, 70)) + [255, 256, 768, 1000, 1023, 1024, 4096, 65537, 1 << 20, (1 << 22) - 1]:
        ptots = [0, 1, 2, ranges - 1, ranges, ranges + 1] + [rng.randrange(1, 1 << 22) for _ in range(40)]
        ptots += [0xFFFFFFFF // ranges, rng.randrange(1, 1 << 40), 1 << 32, (1 << 32) - 1]
        for ptot in ptots:
            for w in {0, 1, ranges // 2, ranges - 1, ranges, rng.randrange(ranges + 1)}:
                assert part.start(ptot, w, ranges) == ptot * w // ranges, (ptot, w, ranges)


def test_range_begin_at_the_top_of_its_range(part):
    """Products on both sides of 2^32, where the 64-bit division takes over."""
    rng = random.Random(2)
    for _ in range(20000):
        ranges = rng.randrange(1, 1 << rng.randrange(1, 23))
        w = rng.randrange(1, ranges + 1)
        top = 0xFFFFFFFF // w
        ptot = max(0, top - rng.randrange(-3, 4))
        assert part.start(ptot, w, ranges) == ptot * w // ranges, (ptot, w, ranges)


@pytest.mark.parametrize("sparse", [False, True])
def test_pieces_of_a_unit(part, sparse):
    """Every unit's workers and slots against the ranges themselves, with more
    pages than workers and with fewer (a loose bound on the context lengths):
    a piece that starts its worker's range takes slot 2 w, any other 2 w + 1."""
    rng = random.Random(3 + sparse)
    lo_hi, slots = (ctypes.c_int * 2)(), (ctypes.c_int * 4096)()
    for _ in range(300):
        sizes = [rng.choice([1, 1, 2, 3, 7, 40, 300]) for _ in range(rng.randrange(1, 40))]
        ptot = sum(sizes)
        W = rng.randrange(ptot + 1, 4 * ptot + 2) if sparse else rng.randrange(1, ptot + 1)
        begin = [part.start(ptot, w, W) for w in range(W + 1)]
        us = 0
        for np_ in sizes:
            want = []
            for w in range(W):
                first, last = max(begin[w], us), min(begin[w + 1], us + np_)
                if first < last:
                    want.append((w, 2 * w if first == begin[w] else 2 * w + 1))
            n = part.split(ptot, us, np_, W, lo_hi, slots, len(slots))
            assert (lo_hi[0], lo_hi[1]) == (want[0][0], want[-1][0])
            assert n == len(want) and list(slots[:n]) == [s for _, s in want], (ptot, W, us, np_)
            us += np_


def test_groups_need_no_larger_workspace_than_single_wavefronts():
    """The automatic kernel choice fits every workspace that was sized for
    single-wavefront workers (TS_VARIANT_WAVE), and the other way round."""
    from paper_2608_22788_amd import binding
    for B in (1, 2, 3, 8, 40, 300):
        for hkv in (1, 2, 8):
            for ctx in (1, 16, 17, 100, 181, 700, 1878, 4000, 60000):
                for G, Q, D in ((1, 1, 64), (4, 1, 128), (4, 4, 128), (8, 4, 128), (4, 12, 64), (4, 16, 64)):
                    maxp = (ctx + 15) // 16
                    size = [binding.workspace_size(binding.make_shape(B, G * hkv, hkv, D, Q, maxp, ctx, B * maxp, 0, 16, v))
                            for v in (0, 1)]
                    assert 0 < size[0] <= size[1], (B, hkv, ctx, G, Q, D, size)
                    assert size[0] == size[1], (B, hkv, ctx, G, Q, D, size)

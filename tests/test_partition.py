"""The 32-bit start of a worker's page range (range_begin in attn_common.h),
written out in Python integers, against the exact quotient."""
import random


def range_begin(ptot, w, ranges):
    inv = 0xFFFFFFFF // ranges
    x = ptot * w
    assert x < 1 << 32
    q = (x * inv) >> 32
    return q + (((x - q * ranges) & 0xFFFFFFFF) >= ranges)


def test_range_begin_is_the_exact_quotient():
    rng = random.Random(1)
    for ranges in list(range(1, 70)) + [255, 256, 768, 1000, 1023, 1024, 4096, 65537, 1 << 20, (1 << 22) - 1]:
        ptots = [0, 1, 2, ranges - 1, ranges, ranges + 1] + [rng.randrange(1, 1 << 22) for _ in range(40)]
        for ptot in ptots + [0xFFFFFFFF // ranges]:
            for w in {0, 1, ranges // 2, ranges - 1, ranges, rng.randrange(ranges + 1)}:
                if w <= ranges and ptot * w < 1 << 32:
                    assert range_begin(ptot, w, ranges) == ptot * w // ranges, (ptot, w, ranges)


def test_range_begin_at_the_top_of_its_range():
    rng = random.Random(2)
    for _ in range(20000):
        ranges = rng.randrange(1, 1 << rng.randrange(1, 23))
        w = rng.randrange(1, ranges + 1)
        top = 0xFFFFFFFF // w
        ptot = top - rng.randrange(min(top, 3) + 1)
        assert range_begin(ptot, w, ranges) == ptot * w // ranges


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

"""Calls that overlap on the GPU: what a call's merge workgroups may hold while
they wait for its workers."""
import pytest

pytestmark = pytest.mark.gpu

CUS = 256
LDS_PER_CU = 160 * 1024
WAVES_PER_CU = 32


def test_waiting_workgroups_hold_at_most_half_of_the_slots():
    """Merge workgroups in the launch wait for workers that may not have
    started, so two calls on two streams could block each other if those of
    one call filled an XCD.  Plans only (nothing is launched): for every kernel
    with and without a fixed worker count, against an upper bound on the
    workgroups that fit at once (LDS and wavefronts)."""
    from paper_2608_22788_amd import binding
    seen, full = set(), set()
    for D in (64, 128):
        for G, Q in ((1, 1), (4, 1), (8, 1), (4, 4), (8, 4), (4, 8), (4, 12), (16, 4), (4, 16)):
            for B in (1, 2, 3, 4, 8, 15, 16, 32):
                for Hkv in (1, 2, 4, 8):
                    for var in (0, 1, 2) if D == 128 else (0, 1):
                        for w in (0, 2048):
                            shape = binding.make_shape(B, G * Hkv, Hkv, D, Q, 2000, 32000, 2000 * B, w, 16, var)
                            plan = binding.decode_attn_plan(shape)
                            merge = plan["grid"] - plan["num_workers"]
                            if plan["combine"] != binding.COMBINE_IN_LAUNCH:
                                assert merge == 0
                                continue
                            slots = CUS * min(LDS_PER_CU // max(1, plan["lds_bytes"]),
                                              WAVES_PER_CU * 64 // plan["threads"])
                            assert 0 < merge <= slots // 2, (D, G, Q, B, Hkv, var, w, plan)
                            seen.add((plan["variant"], plan["threads"]))
                            full.add(merge == slots // 2)
    # single wavefronts, groups and teams all combine in the launch somewhere,
    # and the bound is reached
    assert {(1, 64), (1, 256), (2, 256)} <= seen and True in full

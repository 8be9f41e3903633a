"""Calls that overlap on the GPU: what a call's merge workgroups may hold while
they wait for its workers, and what happens to their rows when they give up."""
import ctypes

import pytest

from paper_2608_22788_amd import synth
from gpu_util import assert_parity, canary_ok, oracle_out, say

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


# (name, Hq, Hkv, D, Qmax, q_lens, ctx_lens, variant, num_workers); all combine
# in the launch
HAND_OVER = [
    ("group", 32, 8, 128, 4, [4, 2, 0, 3], [9000, 700, 300, 40], 0, 0),
    ("group_32_pieces", 8, 2, 128, 1, [1], [30000], 0, 0),
    ("group_two_blocks", 32, 4, 128, 4, [4, 1], [6000, 3000], 0, 0),
    ("group_d64", 16, 1, 64, 4, [4, 3], [7000, 2000], 0, 0),
    ("team", 32, 8, 128, 16, [16, 5], [20000, 900], 0, 0),
    ("wave", 32, 8, 128, 4, [4, 1], [9000, 5000], 1, 0),
    ("wave_many_pieces", 8, 1, 128, 2, [2], [40000], 1, 4096),
    ("valu", 32, 8, 128, 1, [1, 1], [9000, 30], 3, 0),
]


@pytest.mark.parametrize("case", HAND_OVER, ids=[c[0] for c in HAND_OVER])
def test_rows_of_merge_wavefronts_that_give_up(orc, case):
    """Merge wavefronts limited to 0, 1, 10 and 100 polls leave their rows to the
    worker that arrives last, all of them or some: the result is bit for bit
    that of a full wait, within the parity bar, and every counter is zero
    after each call, so that the next one on the workspace starts clean."""
    import torch
    from paper_2608_22788_amd import binding, device
    name, Hq, Hkv, D, Qmax, ql, cl, variant, workers = case
    cfg = dict(B=len(ql), Hq=Hq, Hkv=Hkv, D=D, q_len=1, lengths=("uniform", 1, 1), scale=D ** -0.5)
    wl = synth.make_workload(f"handover_{name}", seed=91, cfg=cfg, ctx_lens=cl, q_lens=ql, Qmax=Qmax,
                             poison=True, spare_pages=1)
    ref = oracle_out(orc, wl)
    t = device.upload(wl)
    shape = binding.shape_of(t["q"], t["k_pages"], t["page_table"], wl.max_ctx_len, workers, variant)
    plan = binding.decode_attn_plan(shape)
    assert plan["combine"] == binding.COMBINE_IN_LAUNCH, plan
    ws = binding.new_workspace(binding.workspace_size(shape))
    t["out_full"].fill_(device.CANARY)
    device.run(wl, t, workspace=ws, num_workers=workers, variant=variant)
    assert_parity(device.out_as_f64(t), ref, f"{name} full wait")
    want = t["out_full"].clone()
    for polls in (0, 1, 10, 100, 0):
        say(f"hand-over {name} polls={polls}")
        t["out_full"].fill_(device.CANARY)
        binding.check(binding.lib.ts_decode_attn_polls(
            ctypes.byref(shape), t["q"].data_ptr(), t["k_pages"].data_ptr(), t["v_pages"].data_ptr(),
            t["page_table"].data_ptr(), t["ctx_lens"].data_ptr(), t["q_lens"].data_ptr(), t["out"].data_ptr(),
            ctypes.c_float(wl.scale), ws.data_ptr(), ws.numel(), None, polls), "ts_decode_attn_polls")
        torch.cuda.synchronize()
        assert torch.equal(t["out_full"].view(torch.int16), want.view(torch.int16)), f"{name} polls={polls}"
        canary_ok(t, wl)
        assert int(ws[:1 << 20].count_nonzero()) == 0, f"counters left set: {name} polls={polls}"


def test_calls_on_four_streams():
    """Four streams at once, each with its own workspace: groups of one and of
    two row blocks and teams whose pieces are merged in the launch, and one
    call with the merge kernel.  Bit for bit what each gives alone."""
    import torch
    from paper_2608_22788_amd import binding, device
    #       Hq  Hkv  Qmax  contexts                   combine
    runs = [(32, 8, 4, [20000, 9000, 300, 15000], binding.COMBINE_IN_LAUNCH),
            (32, 4, 4, [20000, 9000, 300, 15000], binding.COMBINE_IN_LAUNCH),
            (32, 8, 16, [20000, 9000], binding.COMBINE_IN_LAUNCH),
            (64, 8, 4, [9000, 300, 7000, 15000, 20000], binding.COMBINE_MERGE_KERNEL)]
    calls = []
    for n, (Hq, Hkv, Qmax, ctx, combine) in enumerate(runs):
        cfg = dict(B=len(ctx), Hq=Hq, Hkv=Hkv, D=128, q_len=1, lengths=("uniform", 1, 1), scale=128 ** -0.5)
        wl = synth.make_workload(f"four_{n}", seed=50 + n, cfg=cfg, ctx_lens=ctx, q_lens=[Qmax] * len(ctx))
        t = device.upload(wl, values="device")
        shape = binding.shape_of(t["q"], t["k_pages"], t["page_table"], wl.max_ctx_len)
        plan = binding.decode_attn_plan(shape)
        assert plan["combine"] == combine, (n, plan)
        ws = binding.new_workspace(binding.workspace_size(shape))
        device.run(wl, t, workspace=ws)
        torch.cuda.synchronize()
        calls.append((wl, t, ws, t["out"].clone(), torch.cuda.Stream()))
    for rep in range(5):
        for wl, t, ws, ref, st in calls:
            t["out"].zero_()
        torch.cuda.synchronize()
        say(f"four streams, repetition {rep}")
        for _ in range(4):
            for wl, t, ws, ref, st in calls:
                binding.decode_attn(t["q"], t["k_pages"], t["v_pages"], t["page_table"], t["ctx_lens"], t["q_lens"],
                                    t["out"], wl.scale, workspace=ws, max_ctx_len=wl.max_ctx_len, stream=st)
        torch.cuda.synchronize()
        for n, (wl, t, ws, ref, st) in enumerate(calls):
            assert torch.equal(t["out"].view(torch.int16), ref.view(torch.int16)), (rep, n)
            assert int(ws[:1 << 20].count_nonzero()) == 0, (rep, n)

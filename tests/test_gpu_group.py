"""The group kernel (four wavefronts per worker whose split pieces meet in
LDS), the automatic choice up to 32 rows per unit at head_dim 128 and for
every row count at head_dim 64: every output element against the oracle at
the edges of its partition, in each way of combining the groups' partials."""
import numpy as np
import pytest

from paper_2608_22788_amd import synth
from gpu_util import assert_parity, canary_ok, oracle_out, say

pytestmark = pytest.mark.gpu

MERGE, LAST, IN_LAUNCH = 0, 1, 2
# (name, Hq, Hkv, D, Qmax, q_lens, ctx_lens, combine)
CASES = [
    # one page in all, then fewer pages than wavefronts, then a page per wavefront
    ("one_page", 4, 1, 128, 1, [1], [5], IN_LAUNCH),
    ("three_pages", 8, 1, 128, 2, [2], [47], IN_LAUNCH),
    ("page_each", 32, 8, 128, 4, [4], [512], IN_LAUNCH),
    # units that start and end inside a group, one long unit over many groups
    ("short_long", 32, 8, 128, 1, [1, 1, 1, 0, 1], [16, 9000, 33, 500, 1], IN_LAUNCH),
    ("two_blocks", 32, 4, 128, 4, [4, 1, 3], [3000, 17, 1290], IN_LAUNCH),
    # more merge workgroups than the launch takes: the merge kernel
    ("merge_kernel", 32, 8, 128, 6, [6, 1, 5, 2] * 8, [1200 + 61 * i for i in range(32)], MERGE),
    ("merge_kernel_d64", 64, 8, 64, 8, [8, 3] * 6, [2500 + 100 * i for i in range(12)], MERGE),
    # at least two units per group: the last arriver, with a long unit among short ones
    ("last", 32, 8, 128, 1, [1] * 100, [20000] + [16 + (7 * b) % 400 for b in range(99)], LAST),
    ("last_two_blocks", 32, 4, 128, 4, [4, 2, 1] * 50, [9000] + [4 + (37 * b) % 300 for b in range(149)], LAST),
    # head_dim 64 with one to four row blocks
    ("d64_1", 8, 2, 64, 1, [1, 1, 1], [3000, 16, 77], IN_LAUNCH),
    ("d64_2", 8, 2, 64, 6, [6, 2], [2000, 6], IN_LAUNCH),
    ("d64_3", 8, 2, 64, 10, [10, 7], [2010, 31], IN_LAUNCH),
    ("d64_4", 16, 1, 64, 4, [4, 4, 1], [700, 4, 5000], IN_LAUNCH),
]


@pytest.mark.parametrize("case", CASES, ids=[c[0] for c in CASES])
def test_group_kernel(orc, case):
    import torch
    from paper_2608_22788_amd import binding, device
    name, Hq, Hkv, D, Qmax, ql, cl, combine = case
    cfg = dict(B=len(ql), Hq=Hq, Hkv=Hkv, D=D, q_len=1, lengths=("uniform", 1, 1), scale=D ** -0.5)
    wl = synth.make_workload(f"group_{name}", seed=77, cfg=cfg, ctx_lens=cl, q_lens=ql, Qmax=Qmax,
                             poison=True, spare_pages=1)
    ref = oracle_out(orc, wl)
    t = device.upload(wl)
    shape = binding.shape_of(t["q"], t["k_pages"], t["page_table"], max(1, wl.max_ctx_len))
    plan = binding.decode_attn_plan(shape)
    assert plan["threads"] == 256 and plan["variant"] == 1 and plan["combine"] == combine, plan
    ws = binding.new_workspace(binding.workspace_size(shape))
    for rep in range(2):   # the second call finds the first one's partials and cleared counters
        say(f"group {name} call {rep}")
        t["out_full"].fill_(device.CANARY)
        device.run(wl, t, workspace=ws)
        assert_parity(device.out_as_f64(t), ref, f"group {name}")
        canary_ok(t, wl)
        torch.cuda.synchronize()
        assert int(ws[:1 << 20].count_nonzero()) == 0, f"counters left set: {name}"


# fewer pages than groups, as with a loose bound on the context lengths:
# (name, Hq, Hkv, D, Qmax, q_lens, ctx_lens, max_ctx_len, combine)
SPARSE = [
    ("one_block", 32, 8, 128, 4, [4, 1, 0, 1], [130, 16, 300, 1], 40000, IN_LAUNCH),
    ("two_blocks", 32, 4, 128, 4, [4, 0, 3], [400, 100, 250], 40000, IN_LAUNCH),
    ("merge_kernel", 32, 8, 128, 6, [6, 2, 1] + [0] * 29, [90, 33, 200] + [50] * 29, 8000, MERGE),
    ("last", 32, 8, 128, 1, [1, 1] + [0] * 70, [200, 17] + [40] * 70, 8000, LAST),
    ("d64_1", 8, 2, 64, 1, [1, 0, 1], [900, 20, 100], 60000, IN_LAUNCH),
    ("d64_4", 16, 1, 64, 4, [4, 0, 2], [1500, 9, 333], 60000, IN_LAUNCH),
    ("d64_last", 8, 2, 64, 2, [2, 1] + [0] * 300, [700, 90] + [0] * 300, 8000, LAST),
]


@pytest.mark.parametrize("case", SPARSE, ids=[c[0] for c in SPARSE])
def test_fewer_pages_than_groups(orc, case):
    import torch
    from paper_2608_22788_amd import binding, device
    name, Hq, Hkv, D, Qmax, ql, cl, bound, combine = case
    cfg = dict(B=len(ql), Hq=Hq, Hkv=Hkv, D=D, q_len=1, lengths=("uniform", 1, 1), scale=D ** -0.5)
    wl = synth.make_workload(f"sparse_{name}", seed=79, cfg=cfg, ctx_lens=cl, q_lens=ql, Qmax=Qmax,
                             poison=True, spare_pages=1)
    ref = oracle_out(orc, wl)
    t = device.upload(wl)
    wide = torch.zeros(wl.B, (bound + 15) // 16, dtype=torch.int32, device="cuda")
    wide[:, :t["page_table"].shape[1]] = t["page_table"]
    shape = binding.shape_of(t["q"], t["k_pages"], wide, bound)
    plan = binding.decode_attn_plan(shape)
    pages = Hkv * sum((n + 15) // 16 for n, q in zip(cl, ql) if q > 0)
    assert plan["threads"] == 256 and plan["combine"] == combine and pages < plan["num_workers"], (plan, pages)
    ws = binding.new_workspace(binding.workspace_size(shape))
    for rep in range(2):
        say(f"sparse {name} call {rep}")
        t["out_full"].fill_(device.CANARY)
        binding.decode_attn(t["q"], t["k_pages"], t["v_pages"], wide, t["ctx_lens"], t["q_lens"], t["out"], wl.scale,
                            workspace=ws, max_ctx_len=bound)
        assert_parity(device.out_as_f64(t), ref, f"sparse {name}")
        canary_ok(t, wl)
        torch.cuda.synchronize()
        assert int(ws[:1 << 20].count_nonzero()) == 0, f"counters left set: {name}"


@pytest.mark.parametrize("name,variant", [(n, v) for n in ("short_long", "two_blocks", "merge_kernel", "last",
                                                           "last_two_blocks") for v in (0, 1, 2)] +
                         [("d64_4", 0), ("d64_4", 1)])
def test_infinite_value_stays_in_its_column(name, variant):
    """An infinite value of a sequence's first token makes its dim of every
    output row infinite and leaves the others as they are bit for bit, wherever
    the unit is split and however its pieces meet (a piece that is read in place
    of a missing one, with weight 0, would turn it into NaN)."""
    import torch
    from paper_2608_22788_amd import binding, device
    _, Hq, Hkv, D, Qmax, ql, cl, _ = next(c for c in CASES if c[0] == name)
    cfg = dict(B=len(ql), Hq=Hq, Hkv=Hkv, D=D, q_len=1, lengths=("uniform", 1, 1), scale=D ** -0.5)
    wl = synth.make_workload(f"inf_{name}", seed=78, cfg=cfg, ctx_lens=cl, q_lens=ql, Qmax=Qmax)
    t = device.upload(wl)
    say(f"infinite value {name} variant={variant}")
    device.run(wl, t, variant=variant)
    want = t["out"].clone()
    first = t["page_table"][:, 0].long()
    on = torch.tensor([b for b in range(wl.B) if ql[b] > 0], device="cuda")
    t["v_pages"][first[on], :, 0, 5] = float("inf")
    for b in range(wl.B):
        want[b, :ql[b], :, 5] = float("inf")
    device.run(wl, t, variant=variant)
    torch.cuda.synchronize()
    got, exp = t["out"].view(torch.int16), want.view(torch.int16)
    bad = [b for b in range(wl.B) if not torch.equal(got[b, :ql[b]], exp[b, :ql[b]])]
    assert not bad, f"sequences {bad[:10]} of {len(bad)}"

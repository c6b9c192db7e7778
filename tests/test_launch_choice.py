"""Which kernels the launches of a problem take (fcp_launch_probe): host integer work, no GPU."""
import os
import subprocess
import sys

import numpy as np
import pytest

import paper_2605_08524_amd as fcp

F32 = 1   # FCP_FLAG_O_F32


def _problem(lens, bs, causal, c, hq, hkv, d, owned=None, flags=F32):
    plan = fcp.fcp_plan_blocks(lens, bs, causal, c, None if owned is None else np.asarray(owned, dtype=np.int32))
    return fcp.Problem(plan, hq, hkv, d, bs, 0.0, flags)


def test_few_long_chains_are_split_and_full_launches_are_not():
    info = fcp.fcp_launch_probe(_problem([8192], 1024, 1, 0, 1, 1, 64))
    assert info["split"] == (True, True, True) and info["items"] == (32, 32, 64) and sum(info["dq_queue_tiles"]) > 0
    info = fcp.fcp_launch_probe(_problem([8192] * 8, 1024, 1, 0, 32, 8, 128))
    assert info["split"] == (False, False, False)
    info = fcp.fcp_launch_probe(_problem([8192], 1024, 1, 0, 1, 1, 64), forward_only=True)
    assert info["split"][0] and sum(info["dq_queue_tiles"]) == 0


def test_probe_validates():
    with pytest.raises(fcp.FcpError):
        fcp.fcp_launch_probe(_problem([100], 64, 1, 0, 4, 4, 96))


def _forward_choices(lens, bs, causal, c, hq, hkv, d, owned=None):
    """The forward's kernel of the one pass and of every stage of a plan."""
    plan = fcp.fcp_plan_blocks(lens, bs, causal, c, None if owned is None else np.asarray(owned, dtype=np.int32))
    tables = [plan] + [fcp.fcp_stage_tables(plan, k)[0] for k in range(fcp.fcp_stage_tables(plan, 0)[1])]
    return [fcp.fcp_launch_probe(fcp.Problem(t, hq, hkv, d, bs, 0.0, F32))["split"][0] for t in tables]


@pytest.mark.parametrize("case", [([65536], 1024, 1, 16, 4, 4, 64, [(0, 62), (0, 63)]), ([65536], 1024, 1, 16, 4, 4, 128, [(0, 62), (0, 63)]),
                                  ([20000], 1024, 1, 5, 1, 1, 64, None), ([9000, 5000], 512, 0, 9, 2, 1, 128, None)])
def test_stages_of_long_slots_take_the_kernel_of_the_one_pass(case):
    """The two kernels round P against different references: only where all launches take the same one does a running result agree
    with the one-pass forward to fp32 rounding."""
    assert len(set(_forward_choices(*case))) == 1


def test_forward_without_a_workspace_takes_the_kernel_of_the_one_with():
    """fcp_block_attn_fwd_static gives the bits of fcp_queue_build + fcp_block_attn_fwd: many forward items beside few dQ or dK/dV items, and
    the other way round."""
    cases = [([800], 32, 0, 1, 1, 1, 64, None), ([1280], 32, 1, 1, 16, 16, 64, [(0, 39)]), ([640], 32, 1, 1, 32, 32, 64, [(0, 19)]),
             ([1280], 32, 1, 1, 15, 5, 64, [(0, 39)])]
    rng = np.random.default_rng(5)
    for _ in range(150):
        g = int(rng.choice([1, 2, 3, 4]))
        hkv = int(rng.choice([1, 2, 5, 16]))
        lens = [int(n) for n in rng.integers(1, 3000, size=rng.integers(1, 8))]
        bs = int(rng.choice([32, 100, 128, 512]))
        owned = None
        if rng.random() < 0.5:
            blocks = [(s, i) for s, n in enumerate(lens) for i in range(-(-n // bs))]
            owned = [b for b in blocks if rng.random() < 0.2] or [blocks[-1]]
        cases.append((lens, bs, int(rng.integers(0, 2)), int(rng.choice([0, 1, 2, 7])), g * hkv, hkv, int(rng.choice([64, 128])), owned))
    chosen = []
    for case in cases:
        p = _problem(*case)
        with_ws, without = (fcp.fcp_launch_probe(p, forward_only)["split"][0] for forward_only in (False, True))
        assert with_ws == without, case
        chosen.append(with_ws)
    assert 10 < sum(chosen) < len(chosen) - 10      # both kernels were chosen


@pytest.mark.parametrize("case", [([32] * 560 + [64], 32, 1, 1, 1, 1, 64), ([32] * 540 + [512], 256, 1, 1, 1, 1, 64), ([200] * 80 + [512], 256, 1, 1, 1, 1, 64)])
def test_stages_of_many_items_take_the_kernel_of_the_one_pass(case):
    """More than 512 items in the one pass and the first stage, one in the second."""
    assert len(set(_forward_choices(*case))) == 1


def test_a_block_of_all_rows_that_32_bits_hold():
    """2^31 - 1 query rows beside one KV block: the walk over their items must end (it is the host's, before the NULL pointers are looked at)."""
    code = """
import os
import subprocess
import sys

import numpy as np
import paper_2605_08524_amd as fcp
n = 2**31 - 1
t = lambda *row: np.array([row], dtype=np.int32)
plan = dict(kv_blocks=t(0, 0, 0, 64), q_blocks=t(0, 0, 0, n), pairs=t(0, 0, 0, 0), slots=t(0, 0, 1, 0), n_slot_rows=n)
try:
    fcp.fcp_bwd_preprocess(fcp.Problem(plan, 1, 1, 64, n, 0.0, 1), None, None, None, None)
except fcp.FcpError as e:
    assert "NULL pointer" in str(e)
    print("refused")
"""
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    assert subprocess.run([sys.executable, "-c", code], cwd=root, timeout=60, capture_output=True, text=True).stdout == "refused\n"


def test_slots_beyond_the_kv_blocks_do_not_grow_a_split_launch():
    """Two slots of one KV block each and any number without pairs: the split forward's grid is items times units."""
    def info(n_empty):
        slots = np.array([[0, 0, 1, 0], [0, 1, 1, 64]] + [[0, 2, 0, 128]] * n_empty, dtype=np.int32)
        plan = dict(kv_blocks=np.array([[0, 0, 0, 64], [0, 1, 64, 64]], dtype=np.int32), q_blocks=np.array([[0, 1, 0, 64]], dtype=np.int32),
                    pairs=np.array([[0, 0, 0, 0], [0, 1, 1, 1]], dtype=np.int32), slots=slots, n_slot_rows=192)
        return fcp.fcp_launch_probe(fcp.Problem(plan, 2, 2, 64, 64, 0.0, F32))
    assert info(1)["split"][0]
    assert info(1000)["items"][0] == 2004 and not info(1000)["split"][0]


@pytest.mark.parametrize("lens,hq,hkv,d", [([900, 50, 1300, 333], 8, 2, 128), ([4096], 8, 8, 128), ([4096], 8, 8, 64)])
def test_dq_from_ds_keeps_the_queue_order(lens, hq, hkv, d):
    """With dS kept the dQ items are drawn from eight queues, which have to hold the same work; without it the split dQ, which has no
    queues, takes the longest chains first."""
    spill = fcp.fcp_launch_probe(_problem(lens, 1024, 1, 0, hq, hkv, d, flags=F32 | fcp.FCP_FLAG_BWD_SPILL_DS))
    plain = fcp.fcp_launch_probe(_problem(lens, 1024, 1, 0, hq, hkv, d))
    assert plain["split"][1] and plain["dq_queue_tiles"][0] == max(plain["dq_queue_tiles"])
    tiles = spill["dq_queue_tiles"]
    assert max(tiles) <= sum(tiles) / 4 and max(tiles) < 0.6 * plain["dq_queue_tiles"][0]


@pytest.mark.parametrize("case,four", [
    # few long chains on 64 rows: half as many items would leave half of the chip idle
    (([65600], 1024, 1, 3, 16, 4, 128, [(0, 64)]), False), (([65600], 1024, 1, 3, 8, 1, 64, [(0, 64)]), False),
    (([8256] * 8, 1024, 1, 2, 16, 4, 128, [(s, 8) for s in range(8)]), False), (([192] * 15, 256, 1, 0, 32, 8, 128), False),
    # one round of items instead of two, or a start of fewer workgroups
    (([64] * 40, 128, 1, 0, 16, 4, 128), True), (([64] * 30, 128, 1, 0, 16, 4, 64), True),
    # more than 512 items
    (([64] * 70, 128, 1, 0, 16, 4, 128), True), (([2112] * 64, 512, 1, 1, 16, 4, 128, [(s, 4) for s in range(64)]), True),
    # no row tile of at most 64 rows; groups of two
    (([128] * 40, 128, 1, 0, 16, 4, 128), False), (([64] * 80, 128, 1, 0, 16, 8, 128), False)])
def test_four_heads_only_where_they_pay(case, four):
    p = _problem(*case)
    with_ws, without = fcp.fcp_launch_probe(p), fcp.fcp_launch_probe(p, forward_only=True)
    assert with_ws["four_heads"][0] == four and without["four_heads"][0] == four and with_ws["items"][0] == without["items"][0]
    assert fcp.fcp_workspace_bytes(p) > 0


def test_dq_of_few_items_takes_two_heads_unless_it_is_split():
    """256 items of 65 tiles: two heads run them in one round as fast as the four-headed ones half of the chip; a split launch keeps four."""
    def owned(d, flags=F32):
        return fcp.fcp_launch_probe(_problem([4160] * 16, 1024, 1, 2, 32, 8, d, [(s, 4) for s in range(16)], flags))
    whole, split = owned(128), owned(64)
    assert whole["items"][1] == 256 and not whole["four_heads"][1] and not whole["split"][1]
    assert split["split"][1] == split["four_heads"][1] and split["items"][1] == (128 if split["split"][1] else 256)
    assert not owned(64, F32 | fcp.FCP_FLAG_BWD_SPILL_DS)["four_heads"][1]      # dQ from dS is never split


def test_whole_items_flag_splits_nothing_and_keeps_the_items():
    for case in (([8192], 1024, 1, 0, 1, 1, 64), ([300, 77], 128, 1, 2, 4, 2, 128), ([64] * 40, 128, 1, 0, 16, 4, 128)):
        plain, whole = (fcp.fcp_launch_probe(_problem(*case, flags=F32 | flag)) for flag in (0, fcp.FCP_FLAG_WHOLE_ITEMS))
        assert any(plain["split"]) and whole["split"] == (False, False, False)
        assert plain["items"][2] == whole["items"][2]
        assert fcp.fcp_workspace_bytes(_problem(*case, flags=F32 | fcp.FCP_FLAG_WHOLE_ITEMS)) > 0


@pytest.mark.parametrize("case,split", [
    # the last rows of many long sequences: every 32 rows read all K and V of their sequence by themselves
    (([4160] * 16, 1024, 1, 0, 12, 4, 128, [(s, 4) for s in range(16)]), (False, None)),
    (([8256] * 8, 1024, 1, 0, 48, 16, 128, [(s, 8) for s in range(8)]), (False, None)),
    (([15500 + 9 * s for s in range(15)], 128, 1, 0, 16, 16, 128, [(s, (15500 + 9 * s - 1) // 128) for s in range(15)]), (False, None)),
    (([4160] * 16, 1024, 1, 0, 32, 8, 64, [(s, 4) for s in range(16)]), (False, False)),
    # few of them, or few heads: the chip would idle
    (([8256] * 8, 1024, 1, 0, 8, 8, 64, [(s, 8) for s in range(8)]), (True, True)),
    (([2112] * 4, 1024, 1, 0, 16, 8, 128, [(s, 2) for s in range(4)]), (True, True)),
    (([8192], 1024, 1, 0, 1, 1, 64), (True, True)), (([4000], 128, 1, 0, 4, 4, 64), (True, True))])
def test_split_where_it_was_measured_to_pay(case, split):
    """Forward and dQ; None: both forms take about the same."""
    got = fcp.fcp_launch_probe(_problem(*case))["split"]
    assert all(want is None or have == want for have, want in zip(got, split)), got


@pytest.mark.parametrize("case,joint", [(([2000], 128, 1, 0, 4, 2, 64), True), (([8192], 1024, 1, 0, 1, 1, 128), True), (([46], 777, 0, 0, 64, 16, 128), False),
                                        (([448], 128, 0, 0, 64, 8, 128, [(0, 3)]), False), (([35], 128, 0, 0, 64, 16, 64), False), (([300], 128, 1, 0, 16, 16, 64), False),
                                        (([2048], 1024, 1, 0, 16, 2, 64), True)])
def test_dq_and_dkdv_share_a_launch_only_where_the_d_pass_is_short(case, joint):
    """64 heads of 46 rows: the D pass alone takes 33 us, dQ with D in it and dK/dV 15 together."""
    info = fcp.fcp_launch_probe(_problem(*case))
    assert info["split"][1:] == (True, True) and info["joint_bwd"] == joint
    plan = fcp.fcp_plan_blocks(*case[:4], None if len(case) < 8 else np.asarray(case[7], dtype=np.int32))
    assert not fcp.fcp_launch_probe(fcp.Problem(plan, *case[4:7], case[1], 0.0, F32 | fcp.FCP_FLAG_WHOLE_ITEMS))["joint_bwd"]

"""CPU-side checks of the C-ABI library: it loads, exports every symbol the header
declares, plans blocks bit-exactly like the oracle, and reports errors as codes."""
import ctypes
import os
import re

import numpy as np
import pytest

import paper_2605_08524_amd as fcp
from oracle import fcp_oracle as orc
from paper_2605_08524_amd import binding, workloads

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def test_library_exports_every_declared_symbol():
    hdr = "".join(open(os.path.join(ROOT, "include", name)).read() for name in sorted(os.listdir(os.path.join(ROOT, "include"))))
    hdr = re.sub(r"/\*.*?\*/", "", hdr, flags=re.S)
    declared = set(re.findall(r"\b(fcp_[a-z_]+)\s*\(", hdr))
    assert declared == set(binding.EXPORTS)
    lib = ctypes.CDLL(binding.LIB_PATH)
    for name in declared:
        assert getattr(lib, name) is not None


def _same(plan_a, plan_b):
    for key in ("kv_blocks", "q_blocks", "pairs", "slots"):
        a, b = np.asarray(plan_a[key]).reshape(-1, 4), np.asarray(plan_b[key]).reshape(-1, 4)
        assert a.dtype == np.int32 and b.dtype == np.int32
        assert np.array_equal(a, b), key
    assert plan_a["n_slot_rows"] == plan_b["n_slot_rows"]


@pytest.mark.parametrize("config", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_plan_matches_oracle_on_configs(config, seed):
    wl = workloads.make_workload(config, seed)
    got = fcp.fcp_plan_blocks(wl.seq_lens, wl.block_size, wl.causal, wl.coalesce, wl.q_owned)
    want = orc.plan_blocks(wl.seq_lens, wl.block_size, wl.causal, wl.coalesce, wl.q_owned)
    _same(got, want)


def test_config3_pair_count():
    wl = workloads.make_workload(3, 0)
    plan = fcp.fcp_plan_blocks(wl.seq_lens, wl.block_size, wl.causal, wl.coalesce, wl.q_owned)
    # 32 zig-zag pairs (i, 511 - i): (i + 1) + (512 - i) = 513 KV blocks per pair of query blocks
    assert len(plan["pairs"]) == 32 * 513 and (plan["pairs"][:, 2] == 1).sum() == 64


@pytest.mark.parametrize("seq_lens,bs", [([1], 4), ([4], 4), ([5], 4), ([0, 0], 4), ([], 4), ([0, 7, 0, 1], 3),
                                         ([1000], 1), ([129, 128, 127], 128)])
@pytest.mark.parametrize("causal", [0, 1])
@pytest.mark.parametrize("c", [0, 1, 3, 16])
def test_plan_edge_cases(seq_lens, bs, causal, c):
    _same(fcp.fcp_plan_blocks(seq_lens, bs, causal, c), orc.plan_blocks(seq_lens, bs, causal, c))


def test_plan_owned_subsets_random():
    rng = np.random.default_rng(0)
    for _ in range(30):
        seq_lens = rng.integers(0, 60, size=rng.integers(1, 6))
        bs = int(rng.integers(1, 9))
        blocks = [(s, i) for s, L in enumerate(seq_lens) for i in range(-(-int(L) // bs))]
        keep = [b for b in blocks if rng.random() < 0.4]
        c = int(rng.integers(0, 4))
        causal = int(rng.integers(0, 2))
        owned = np.asarray(keep, dtype=np.int32).reshape(-1, 2)
        _same(fcp.fcp_plan_blocks(seq_lens, bs, causal, c, owned), orc.plan_blocks(seq_lens, bs, causal, c, owned))


def test_plan_error_codes():
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_plan_blocks([4], 0)
    assert e.value.code == binding.FCP_ERR_INVALID_ARG
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_plan_blocks([-3], 4)
    assert e.value.code == binding.FCP_ERR_INVALID_ARG
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_plan_blocks([8], 4, 1, 0, [(0, 2)])
    assert e.value.code == binding.FCP_ERR_INVALID_ARG and "out of range" in str(e.value)
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_plan_blocks([8], 4, 1, 0, [(0, 1), (0, 0)])
    assert e.value.code == binding.FCP_ERR_INVALID_ARG


def test_plan_capacity_too_small():
    lib = binding._lib
    sl = np.asarray([10, 3], dtype=np.int32)
    i32p = ctypes.POINTER(ctypes.c_int32)
    counts = [ctypes.c_int32(1) for _ in range(5)]
    tabs = [np.zeros((1, 4), dtype=np.int32) for _ in range(4)]
    rc = lib.fcp_plan_blocks(sl.ctypes.data_as(i32p), 2, 4, 1, 2, None, 0,
                             tabs[0].ctypes.data, ctypes.byref(counts[0]), tabs[1].ctypes.data, ctypes.byref(counts[1]),
                             tabs[2].ctypes.data, ctypes.byref(counts[2]), tabs[3].ctypes.data, ctypes.byref(counts[3]),
                             ctypes.byref(counts[4]))
    assert rc == binding.FCP_ERR_BUFFER_TOO_SMALL
    assert [c.value for c in counts] == [4, 4, 7, 5, 15]


def _problem(seq_lens=(300, 77), bs=128, hq=4, hkv=2, d=64, c=2):
    plan = fcp.fcp_plan_blocks(list(seq_lens), bs, 1, c)
    return fcp.Problem(plan, hq, hkv, d, bs)


def test_workspace_bytes_and_validation():
    assert fcp.fcp_workspace_bytes(_problem()) > 0
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_workspace_bytes(_problem(d=96))
    assert e.value.code == binding.FCP_ERR_UNSUPPORTED
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_workspace_bytes(_problem(hq=6, hkv=4))
    assert e.value.code == binding.FCP_ERR_UNSUPPORTED
    p = _problem()
    p.pairs[0, 2] = 7            # not a valid kind
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_workspace_bytes(p)
    assert e.value.code == binding.FCP_ERR_INVALID_ARG
    p = _problem()
    p.pairs[1, 2] = 1            # FULL pair of different blocks relabelled DIAG
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_workspace_bytes(p)
    assert e.value.code == binding.FCP_ERR_INVALID_ARG
    p = _problem()
    p.slots[1, 3] = 10 ** 6      # rows outside the partial buffers
    with pytest.raises(fcp.FcpError):
        fcp.fcp_workspace_bytes(p)


def test_null_pointers_are_rejected_before_any_launch():
    p = _problem()
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_queue_build(p, 0, 1 << 20)
    assert e.value.code == binding.FCP_ERR_INVALID_ARG
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_queue_build(p, 256, 8)
    assert e.value.code == binding.FCP_ERR_BUFFER_TOO_SMALL
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_block_attn_fwd(p, 0, 0, 0, 0, 0, 0)
    assert e.value.code == binding.FCP_ERR_INVALID_ARG
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_merge_partials(p, 0, 0, 0, 0, 0)
    assert e.value.code == binding.FCP_ERR_INVALID_ARG
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_block_attn_bwd(p, *([0] * 10))
    assert e.value.code == binding.FCP_ERR_INVALID_ARG


def test_mfma_probe_rejects_bad_arguments_before_any_launch():
    for kind, iters, out in ((0, 10, 0), (0, 0, 256), (3, 10, 256), (-1, 10, 256)):
        with pytest.raises(fcp.FcpError) as e:
            fcp.fcp_mfma_probe(kind, iters, out)
        assert e.value.code == binding.FCP_ERR_INVALID_ARG


def test_workload_generators_are_seeded():
    a, b = workloads.make_workload(2, 0), workloads.make_workload(2, 0)
    assert np.array_equal(a.seq_lens, b.seq_lens) and a.seq_lens.sum() == 65536
    t1 = workloads.draw_tensor(0, 1, (100, 2, 8))
    t2 = workloads.draw_tensor(0, 1, (100, 2, 8))
    assert np.array_equal(t1, t2) and t1.dtype == np.uint16
    x = workloads.bf16_to_f32(t1)
    assert abs(float(x.mean())) < 0.1 and 0.9 < float(x.std()) < 1.1
    # round-to-nearest-even on a tie
    assert workloads.bf16_bits(np.asarray([1.00390625], dtype=np.float32))[0] == 0x3F80
    assert workloads.bf16_bits(np.asarray([1.01171875], dtype=np.float32))[0] == 0x3F82


@pytest.mark.parametrize("config", [1, 2, 3, 4])
def test_stage_tables_match_oracle(config):
    wl = workloads.make_workload(config, 1)
    if config == 1:
        wl.coalesce = 2
    plan = fcp.fcp_plan_blocks(wl.seq_lens, wl.block_size, wl.causal, wl.coalesce, wl.q_owned)
    ref_plan = orc.plan_blocks(wl.seq_lens, wl.block_size, wl.causal, wl.coalesce, wl.q_owned)
    _, n_stages = fcp.fcp_stage_tables(plan, 0)
    assert n_stages == orc.stage_tables(ref_plan, 0)[2]
    for st in sorted({0, 1, n_stages // 2, n_stages - 1, n_stages}):
        got, ns = fcp.fcp_stage_tables(plan, st)
        sp, ss, ref_ns = orc.stage_tables(ref_plan, st)
        assert ns == ref_ns
        assert np.array_equal(got["pairs"], sp) and np.array_equal(got["slots"], ss)
        assert got["n_slot_rows"] == int(ref_plan["q_blocks"][:, 3].sum())
        if len(ss):
            prob = fcp.Problem(got, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.block_size, 0.0,
                               binding.FCP_FLAG_RUNNING_MERGE | binding.FCP_FLAG_O_F32)
            assert fcp.fcp_workspace_bytes(prob) > 0            # a valid problem descriptor


def test_stage_tables_errors():
    plan = fcp.fcp_plan_blocks([300, 50], 128, 1, 1)
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_stage_tables(plan, -1)
    assert e.value.code == binding.FCP_ERR_INVALID_ARG
    bad = dict(plan, slots=plan["slots"][::-1].copy())
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_stage_tables(bad, 0)
    assert e.value.code == binding.FCP_ERR_INVALID_ARG


def _units(seq_lens, bs, causal):
    from oracle import fcp_sched_oracle as sch
    flat = orc.plan_blocks(seq_lens, bs, causal, 0)["kv_blocks"]
    return sch.pack_units(flat, [int(b[3]) for b in flat], [0] * len(flat), bs)[0] if len(flat) else None


def test_packed_plan_matches_oracle_random():
    """fcp_plan_blocks_packed against the oracle's packed planner, bit for bit, on random batches and shares."""
    rng = np.random.default_rng(11)
    for trial in range(150):
        bs = int(rng.choice([4, 8, 16]))
        sl = rng.integers(0, 3 * bs, size=int(rng.integers(1, 12)))
        causal, c = int(rng.integers(0, 2)), int(rng.choice([0, 1, 2, 3]))
        unit = _units(sl, bs, causal)
        qo = None
        if unit is not None and rng.random() < 0.5:
            flat = orc.plan_blocks(sl, bs, causal, 0)["kv_blocks"]
            keep = {u for u in set(unit) if rng.random() < 0.6}
            qo = np.asarray([(int(flat[b][0]), int(flat[b][1])) for b in range(len(flat)) if unit[b] in keep], dtype=np.int32).reshape(-1, 2)
        want = orc.plan_blocks_packed(sl, bs, causal, c, qo, unit)
        got = fcp.fcp_plan_blocks_packed(sl, bs, causal, c, qo, unit)
        for key in ("kv_blocks", "q_blocks", "pairs", "slots", "segments"):
            assert np.array_equal(want[key], got[key]), (trial, key)
        assert want["n_slot_rows"] == got["n_slot_rows"]


def test_packed_plan_on_the_multimodal_config():
    """Config 4 through block costs -> scheduling units -> packed plan, all in the library, against the same chain
    in the oracles; the packed plan has fewer query blocks and pairs than the plain one."""
    from paper_2605_08524_amd.harness import packed_plan
    wl = workloads.make_workload(4, 0)
    got = packed_plan(wl)
    want = orc.plan_blocks_packed(wl.seq_lens, wl.block_size, wl.causal, wl.coalesce, wl.q_owned,
                                  _units(wl.seq_lens, wl.block_size, wl.causal))
    for key in ("kv_blocks", "q_blocks", "pairs", "slots", "segments"):
        assert np.array_equal(want[key], got[key]), key
    plain = fcp.fcp_plan_blocks(wl.seq_lens, wl.block_size, wl.causal, wl.coalesce, wl.q_owned)
    assert len(got["q_blocks"]) < len(plain["q_blocks"]) and len(got["segments"]) > 0
    assert orc.pair_nnz(want) == orc.pair_nnz(orc.plan_blocks(wl.seq_lens, wl.block_size, wl.causal, wl.coalesce, wl.q_owned))
    prob = fcp.Problem(got, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.block_size)
    assert fcp.fcp_workspace_bytes(prob) > 0


def test_packed_plan_error_codes():
    def code(*a):
        with pytest.raises(fcp.FcpError) as e:
            fcp.fcp_plan_blocks_packed(*a)
        return e.value.code
    assert code([10, 2], 4, 1, 0, None, [0, 1, 2, 2]) == -1          # a block of a long sequence shares a unit
    assert code([3, 3], 4, 1, 0, None, [0, 0]) == -1                 # the unit does not fit into a block
    assert code([2, 1, 5], 4, 1, 0, [(0, 0), (2, 0)], [0, 0, 1, 2]) == -1   # a unit owned in part
    assert code([2, 1], 4, 1, 0, None, [0, 7]) == -1                 # unit index out of range
    assert code([2, 1], 4, 1, 0, None, None) == -1                   # blocks but no unit table


def test_segment_tables_are_validated():
    plan = fcp.fcp_plan_blocks_packed([3, 2, 9], 8, 1, 0, None, [0, 0, 1, 2])
    assert plan["segments"].tolist() == [[0, 0, 0, 3], [0, 1, 3, 2]] and plan["pairs"][0].tolist() == [0, 0, 3, 0]

    def rc(mutate):
        bad = {k: (v.copy() if hasattr(v, "copy") else v) for k, v in plan.items()}
        mutate(bad)
        with pytest.raises(fcp.FcpError) as e:
            fcp.fcp_workspace_bytes(fcp.Problem(bad, 2, 2, 64, 8))
        return e.value.code
    assert rc(lambda p: p["segments"].__setitem__((1, 3), 1)) == -1      # the members do not cover their block
    assert rc(lambda p: p["segments"].__setitem__((1, 2), 2)) == -1      # a gap between members
    assert rc(lambda p: p["pairs"].__setitem__((0, 2), 1)) == -1         # a DIAG pair on a block with members
    assert rc(lambda p: p["pairs"].__setitem__((1, 2), 3)) == -1         # a PACKED pair on a block without members
    assert rc(lambda p: p.__setitem__("segments", p["segments"][::-1].copy())) == -1   # not in (kv_blk, tok_off) order


def test_packed_block_size_limit():
    """A packed block above 65 535 tokens is refused when the problem is validated: a limit of the interface, which the
    planner itself does not have."""
    plan = fcp.fcp_plan_blocks_packed([40000, 29000], 70000, 1, 0, None, [0, 0])
    assert plan["kv_blocks"].tolist() == [[0, 0, 0, 69000]] and len(plan["segments"]) == 2
    with pytest.raises(fcp.FcpError) as e:
        fcp.fcp_workspace_bytes(fcp.Problem(plan, 2, 2, 64, 70000))
    assert e.value.code == -3
    ok = fcp.fcp_plan_blocks_packed([40000, 25000], 70000, 1, 0, None, [0, 0])
    assert fcp.fcp_workspace_bytes(fcp.Problem(ok, 2, 2, 64, 70000)) > 0


def test_packed_pairs_of_a_query_block_agree_on_its_members():
    """Two PACKED slots of one query block are accepted only if their KV blocks have the same members (their rows are cut
    up once): two listings of one packed block are, blocks cut differently are refused, in either order."""
    def problem(first, second):
        segments, kv = [], []
        for b, members in enumerate((first, second)):
            kv.append((0, 0, 8 * b, 8))
            segments += [(b, m, sum(members[:m]), n) for m, n in enumerate(members)]
        plan = dict(kv_blocks=kv, q_blocks=[(0, 0, 0, 8)], pairs=[(0, 0, 3, 0), (0, 1, 3, 1)], slots=[(0, 0, 1, 0), (0, 1, 1, 8)],
                    n_slot_rows=16, segments=segments)
        return fcp.Problem({k: v if k == "n_slot_rows" else np.asarray(v, dtype=np.int32) for k, v in plan.items()}, 2, 2, 64, 8)
    assert fcp.fcp_workspace_bytes(problem([3, 5], [3, 5])) > 0
    for members in (([2, 2, 2, 2], [4, 4]), ([4, 4], [2, 2, 2, 2]), ([3, 5], [5, 3])):
        with pytest.raises(fcp.FcpError) as e:
            fcp.fcp_workspace_bytes(problem(*members))
        assert e.value.code == binding.FCP_ERR_INVALID_ARG


@pytest.mark.parametrize("packed", [False, True])
def test_queue_tables_are_built_on_the_host_before_any_gpu_call(packed):
    """Without a GPU, fcp_queue_build still validates the problem, lays out the workspace and builds every table (work
    items, dependency lists, member bounds of joined runs) in host memory; only the upload fails, with FCP_ERR_HIP.
    This is how the queue builder runs under the host sanitizers."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("needs a box without a GPU: here the upload would be attempted")
    from paper_2605_08524_amd.harness import packed_plan
    cases = [workloads.custom_workload([100, 156, 30, 70, 90, 700, 17], 256, 1, 2, 6, 2, 128, seed=1),
             workloads.custom_workload([33, 1, 200, 95, 700, 5, 129], 256, 0, 2, 4, 4, 64, seed=2),
             workloads.make_workload(4, 0)]
    for wl in cases:
        plan = packed_plan(wl) if packed else fcp.fcp_plan_blocks(wl.seq_lens, wl.block_size, wl.causal, wl.coalesce, wl.q_owned)
        for flags in (0, fcp.FCP_FLAG_DIRECT_SINGLE | fcp.FCP_FLAG_O_F32 | fcp.FCP_FLAG_BWD_SPILL_DS):
            prob = fcp.Problem(plan, wl.n_q_heads, wl.n_kv_heads, wl.head_dim, wl.block_size, 0.0, flags)
            nbytes = fcp.fcp_workspace_bytes(prob)
            with pytest.raises(fcp.FcpError) as e:
                fcp.fcp_queue_build(prob, 4096, nbytes)      # an aligned address that is never written: the upload cannot start
            assert e.value.code == -4, fcp.fcp_last_error()


def test_static_forward_accepts_every_plan_within_its_limit():
    """fcp_block_attn_fwd_static is limited by the plan as given (16 bytes a pair, 72 a forward item, 2 MiB); a plan within
    that limit is never refused because its packed blocks become more items than that.  The size check comes before any
    GPU call: without a GPU an accepted plan fails later, with FCP_ERR_HIP."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("needs a box without a GPU: here an accepted plan would be launched")
    align = lambda x: (x + 255) // 256 * 256
    bs, refused, taken = 1024, 0, 0
    for hq, hkv in ((64, 64), (32, 8), (6, 2), (8, 4), (16, 1)):
        for members in ([20] * 51, [1] * 1024, [8] * 128, [129, 1] * 7, [257, 1] * 3 + [129, 1], [700, 300]):
            rows = hq // 2 * -(-sum(members) // 128) if hq // hkv % 2 == 0 else hq * -(-sum(members) // 256)
            fit = (2 * 2 ** 20 - 1024 - 256) // (72 * rows + 16)           # about as many blocks as the limit allows
            for n in (fit - 2, fit + 8):
                if n * len(members) > 200000:
                    continue
                n_pairs, n_items = n, n * rows
                over = 1024 + align(16 * n_pairs) + align(72 * n_items) > 2 * 2 ** 20
                unit = np.repeat(np.arange(n), len(members)).astype(np.int32)
                plan = fcp.fcp_plan_blocks_packed(members * n, bs + 1, 1, 0, None, unit)
                assert len(plan["pairs"]) == n_pairs
                p = fcp.Problem(plan, hq, hkv, 64, bs + 1)
                with pytest.raises(fcp.FcpError) as e:
                    fcp.fcp_block_attn_fwd_static(p, None, None, None, None, None)
                assert e.value.code == (binding.FCP_ERR_BUFFER_TOO_SMALL if over else binding.FCP_ERR_HIP), (hq, hkv, members[:3], n)
                refused += over
                taken += not over
    assert refused > 5 and taken > 5


def test_static_forward_fills_its_array_to_the_last_byte():
    """Packed blocks of many rows and few heads reach the end of the device array (8 MiB + 16 KiB) before the limit of the plan:
    header, spans (16 bytes), forward items (80 bytes) and member bounds (2 bytes a row) that end exactly there are accepted,
    256 bytes more are not."""
    import torch
    if torch.cuda.is_available():
        pytest.skip("needs a box without a GPU: here an accepted plan would be launched")
    align = lambda x: (x + 255) // 256 * 256
    limit, header = 8 * 2 ** 20 + 16 * 2 ** 10, 4352
    blocks = 3453                                                   # of four members of 256 tokens: four spans, four items
    for last, want in ((769, binding.FCP_ERR_HIP), (897, binding.FCP_ERR_BUFFER_TOO_SMALL)):      # ... and one of 256 and `last`
        spans, items, rows = 4 * blocks + 2, 4 * blocks + 1 + 4, 1024 * blocks + 256 + last
        size = header + align(16 * spans) + align(80 * items) + align(2 * rows)
        assert size - limit == (0 if want == binding.FCP_ERR_HIP else 256)
        unit = np.repeat(np.arange(blocks + 1), [4] * blocks + [2]).astype(np.int32)
        plan = fcp.fcp_plan_blocks_packed([256] * (4 * blocks + 1) + [last], 1281, 1, 0, None, unit)
        with pytest.raises(fcp.FcpError) as e:
            fcp.fcp_block_attn_fwd_static(fcp.Problem(plan, 1, 1, 64, 1281), None, None, None, None, None)
        assert e.value.code == want, last


def test_layout_counts_without_building_the_tables():
    """A launch on a workspace that the layout registry does not know computes the layout anew, as fcp_workspace_bytes does:
    from counts, not by building what fcp_queue_build uploads (0.04 of its time here; 0.36 when it built the pair and
    dependency lists)."""
    import time
    import torch
    if torch.cuda.is_available():
        pytest.skip("needs a box without a GPU: here the upload would be attempted")
    plan = fcp.fcp_plan_blocks([1024 * 128], 128, 1, 4)
    p = fcp.Problem(plan, 4, 2, 64, 128, 0.0, fcp.FCP_FLAG_BWD_SPILL_DS)
    assert len(plan["pairs"]) == 524800
    need = fcp.fcp_workspace_bytes(p)
    layout, build = [], []
    for _ in range(4):
        t = time.perf_counter()
        fcp.fcp_workspace_bytes(p)
        layout.append(time.perf_counter() - t)
        t = time.perf_counter()
        with pytest.raises(fcp.FcpError):
            fcp.fcp_queue_build(p, 256, need, None)
        build.append(time.perf_counter() - t)
    assert min(layout) < 0.15 * min(build)


def _forward_rows(prob):
    """The forward's segments and spans as the host hands them to the queue builder: fcp::expand_problem of the same library
    fills seven std::vectors (begin, end, capacity; zeroed memory is an empty one).  Segments (start, len, out_row, first span,
    spans), spans (kv_start, kv_len, kind, column where a DIAG block starts)."""
    vectors = (ctypes.c_void_p * 21)()
    binding._lib._ZN3fcp14expand_problemEPK11fcp_problembPNS_8ExpandedE(ctypes.byref(prob.c), ctypes.c_bool(True), ctypes.byref(vectors))

    def table(i, width):
        begin, end = vectors[3 * i] or 0, vectors[3 * i + 1] or 0
        return np.frombuffer(ctypes.string_at(begin, end - begin), dtype=np.int32).reshape(-1, width)
    return table(2, 8)[:, :5], table(1, 4)


M = 1 << 28            # most rows of a span


@pytest.mark.parametrize("kv_lens,q_len,pairs", [
    ([5 * M + 77], 70, [(0, 0)]),                                    # a FULL block longer than a span
    ([M - 5, 3, 2, 1, M], 9, [(0, 0), (1, 0), (2, 0), (3, 0), (4, 0)]),   # joined up to the limit, not past it
    ([M, 640], 640, [(0, 0), (1, 1)]),                               # DIAG behind a whole span
    ([M - 640, 640], 640, [(0, 0), (1, 1)]),                         # DIAG that ends one
    ([M - 639, 640], 640, [(0, 0), (1, 1)]),
    ([64, 3 * M + 77], 3 * M + 77, [(0, 0), (1, 1)]),                # DIAG blocks longer than a span
    ([2 * M], 2 * M, [(0, 1)]),
    ([M], M, [(0, 1)]),
    ([2 * M + 1, 500], 2 * M + 1, [(0, 1), (1, 0)]),                 # ... and a FULL block behind one
])
def test_spans_of_very_long_blocks(kv_lens, q_len, pairs):
    """The forward's mask word is 4 * (columns of a span that a wave's first row sees - 64) + 2 bits in a signed 32-bit register.
    Spans and segments keep it in range whatever a block's length, and every row still sees what its pairs say."""
    kv = [(0, i, sum(kv_lens[:i]), n) for i, n in enumerate(kv_lens)]
    diag = [b for b, kind in pairs if kind]
    plan = dict(kv_blocks=kv, q_blocks=[(0, diag[0] if diag else 99, 0, q_len)], pairs=[(0, b, kind, 0) for b, kind in pairs],
                slots=[(0, 0, len(pairs), 0)], n_slot_rows=q_len)
    plan = {k: v if k == "n_slot_rows" else np.asarray(v, dtype=np.int32) for k, v in plan.items()}
    prob = fcp.Problem(plan, 1, 1, 64, max(kv_lens + [q_len]))
    assert fcp.fcp_workspace_bytes(prob) > 0
    segments, spans = _forward_rows(prob)
    assert np.array_equal(np.cumsum(segments[:, 1]) - segments[:, 1], segments[:, 0]) and segments[:, 1].sum() == q_len
    assert np.array_equal(segments[:, 2], segments[:, 0])
    for start, n, _, first, count in segments.astype(np.int64):
        mine = spans[first:first + count].astype(np.int64)
        opens = np.where(mine[:, 2] & 1, mine[:, 3] + n, mine[:, 1])             # of the last row; the first row's is less
        assert (4 * opens + 3 < 2 ** 31).all() and (opens <= mine[:, 1]).all()
        for row in sorted({0, min(63, n - 1), n // 2, n - 1}):
            def joined(parts):
                out = []
                for lo, hi in parts:
                    if out and out[-1][1] == lo:
                        out[-1][1] = hi
                    elif hi > lo:
                        out.append([lo, hi])
                return out
            got = joined((s, s + (min(length, ext + row + 1) if kind & 1 else length)) for s, length, kind, ext in mine)
            want = joined((kv[b][2], kv[b][2] + (start + row + 1 if kind else kv[b][3])) for b, kind in pairs)
            assert got == want


def test_a_name_replaced_in_the_binding_is_seen_in_the_package(monkeypatch):
    before = fcp.fcp_workspace_bytes                     # looked up once: kept in the package
    with monkeypatch.context() as m:
        m.setattr(binding, "fcp_workspace_bytes", lambda problem: 7)
        assert fcp.fcp_workspace_bytes(None) == 7
        m.delattr(binding, "fcp_stage_tables")
        with pytest.raises(AttributeError):
            fcp.fcp_stage_tables
    assert fcp.fcp_workspace_bytes is before and binding.fcp_workspace_bytes is before and fcp.fcp_stage_tables is binding.fcp_stage_tables

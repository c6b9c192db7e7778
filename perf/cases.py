"""The work whose speed counts: one worker's block-level attention as a training or inference program runs it.

A program of this framework plans a batch once (block tables, work queues, workspace) and then runs the same tables for
every layer of the model, so the plan, the queues and the output buffers belong to `prepare` and a pass is the calls one
layer makes: forward, merge of the partials, and for training the backward.

A case is a batch shape (how the sequence lengths are distributed, how many tokens, block size, coalesce degree), a head
shape, and the options of the calls:
  kind      "uniform" | "lognormal": packed batches, lengths between lo and hi (lognormal: median `mid`, sigma 1);
            "mixed": 90 % of the tokens in short sequences, the rest the tail blocks of one long resident sequence;
            "long": zig-zag pairs of query blocks of one long sequence, all its KV resident;
            "share": what the block distributor gives the first of eight workers of a lognormal batch
  mode      "fwd": forward (+ merge); "train": forward (+ merge) and backward; "running": one launch per execution stage
  spill     the backward keeps dS in the workspace instead of recomputing S and dP for dQ
  packed    short sequences share blocks (masked by member inside the kernels)
  o32, g16  final O in fp32; gradients in bf16
"""
import math

import numpy as np
import torch

import paper_2605_08524_amd as fcp

_BASE = dict(kind="lognormal", batch=0, tokens=65536, lo=16, hi=32768, mid=2048, block=1024, coalesce=16, causal=True,
             hq=32, hkv=8, d=128, mode="fwd", o32=False, g16=False, spill=False, packed=False, owned=0)


def _case(name=None, **kw):
    c = dict(_BASE)
    c.update(kw)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest call: a handful of short sequences with small blocks; launches and latency count
        _case("tiny_fwd", kind="uniform", tokens=4000, lo=100, hi=1024, block=128, coalesce=0, hq=4, hkv=4, d=64),
        # the smallest training step: partials to merge, grouped heads
        _case("tiny_train", kind="uniform", tokens=2000, lo=60, hi=400, block=128, coalesce=2, hq=4, hkv=2, d=64,
              mode="train", o32=True),
        # inference / evaluation over an ordinary packed batch of one worker
        _case("packed_fwd"),
        # the training step of one worker: dS kept in memory, fp32 gradients
        _case("train_step", mode="train", o32=True, spill=True),
        # the same step at half the tokens, larger blocks and twice the query heads; no room for dS, bf16 gradients
        _case("train_step_wide", tokens=32768, block=4096, hq=64, hkv=8, mode="train", o32=True, g16=True),
        # multimodal batch: mostly short sequences, plus the end of a long one whose KV is resident
        _case("multimodal_fwd", kind="mixed", tokens=131072, lo=64, hi=1024, block=256, hq=16, hkv=16),
        # long-context prefill: zig-zag query blocks of one long sequence, many partials per block
        _case("long_share_fwd", kind="long", tokens=262144, block=2048, owned=16),
        # the same with a running result: one launch per execution stage, no partial buffers
        _case("long_share_running", kind="long", tokens=131072, block=2048, owned=12, mode="running", o32=True),
        # training on many short sequences
        _case("short_train", kind="uniform", lo=16, hi=256, mode="train", o32=True, spill=True),
        # the same kind of batch packed into shared blocks, forward only
        _case("short_packed_fwd", kind="uniform", tokens=49152, lo=16, hi=256, packed=True),
        # training on what the distributor hands one of eight workers; every KV block is a stage of its own
        _case("worker_share_train", kind="share", tokens=131072, lo=1024, hi=131072, mid=12800, block=4096, coalesce=1,
              mode="train", o32=True),
        # bidirectional attention over medium sequences with small heads
        _case("full_train_d64", kind="uniform", tokens=16384, lo=256, hi=2048, block=512, causal=False, hq=16, hkv=16,
              d=64, mode="train", o32=True, g16=True, spill=True),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    limit = max(work(c)["flops"] for c in listed())
    while True:
        d = rng.choice([64, 128, 128])
        hkv = rng.choice([1, 2, 3, 4, 8, 16])
        group = rng.choice([1, 1, 2, 3, 4, 8])
        kind = rng.choice(["uniform", "lognormal", "lognormal", "mixed", "long", "share"])
        mode = rng.choice(["fwd", "train", "train"])
        c = _case(kind=kind, batch=rng.randrange(1 << 20), hq=hkv * group, hkv=hkv, d=d, mode=mode,
                  causal=rng.random() < 0.85, block=rng.choice([128, 256, 512, 777, 1024, 2048, 4096]),
                  coalesce=rng.choice([0, 1, 4, 16, 16]), spill=mode == "train" and rng.random() < 0.5,
                  o32=mode == "train" or rng.random() < 0.3, g16=mode == "train" and rng.random() < 0.5)
        if kind == "uniform":
            hi = _log_int(rng, 64, 4096)
            c.update(tokens=_log_int(rng, 1000, 100000), lo=min(hi - 1, _log_int(rng, 16, 256)), hi=hi)
            c["packed"] = hi < c["block"] and rng.random() < 0.5
        elif kind == "lognormal":
            c.update(tokens=_log_int(rng, 1000, 100000), mid=_log_int(rng, 128, 8192))
        elif kind == "mixed":
            c.update(tokens=_log_int(rng, 8192, 131072), lo=64, hi=1024, causal=True)
        elif kind == "long":
            if mode == "fwd" and rng.random() < 0.5:
                c.update(mode="running", o32=True, coalesce=16)
            c.update(tokens=_log_int(rng, 16384, 262144), owned=2 * rng.randrange(1, 9), causal=True,
                     block=rng.choice([1024, 2048, 4096]), spill=False)
        else:
            c.update(tokens=_log_int(rng, 16384, 131072), lo=1024, hi=131072, mid=_log_int(rng, 4096, 16384),
                     block=rng.choice([1024, 2048, 4096]), causal=True, spill=False)
        nnz = _nnz(c)
        partials = _rows(c)[2] * c["hq"] * c["d"] * 4
        if nnz and work(c)["flops"] <= limit and partials <= 6e9 and not (c["spill"] and 2 * nnz * c["hq"] > 12e9):
            return c


def _lengths(c):
    """(lengths, owned (seq, idx) pairs or None): a function of the case alone."""
    rng = np.random.default_rng([c["batch"], 0])
    bs = c["block"]

    def until(total, one):
        out, acc = [], 0
        while acc < total:
            out.append(min(int(one()), total - acc))
            acc += out[-1]
        return out

    if c["kind"] == "uniform":
        return until(c["tokens"], lambda: rng.integers(c["lo"], c["hi"])), None
    if c["kind"] in ("lognormal", "share"):
        lens = until(c["tokens"], lambda: np.clip(round(math.exp(rng.normal(math.log(c["mid"]), 1.0))), c["lo"], c["hi"]))
        if c["kind"] == "lognormal":
            return lens, None
        blocks, mem, comp = fcp.fcp_block_costs(lens, bs, 1)
        owner = fcp.fcp_assign_blocks(mem, comp, 8)[0]
        return lens, fcp.fcp_worker_blocks(blocks, owner, int(owner[0]))
    if c["kind"] == "mixed":
        short = int(c["tokens"] * 0.9)
        lens = until(short, lambda: rng.integers(c["lo"], c["hi"] + 1))
        long_len = int(rng.integers(c["tokens"] // 2, 2 * c["tokens"] + 1))
        owned = [(s, i) for s, n in enumerate(lens) for i in range(-(-n // bs))]
        n_long, tail = -(-long_len // bs), -(-(c["tokens"] - short) // bs)
        owned += [(len(lens), i) for i in range(max(0, n_long - tail), n_long)]
        return lens + [long_len], np.asarray(owned, dtype=np.int32)
    nb = -(-c["tokens"] // bs)                        # "long"
    n = max(1, min(c["owned"] // 2, nb // 2))
    low = np.sort(rng.choice(max(1, nb // 2), size=n, replace=False))
    idx = np.unique(np.concatenate([low, nb - 1 - low]))
    return [c["tokens"]], np.stack([np.zeros_like(idx), idx], axis=1).astype(np.int32)


def _owned_rows(c):
    """(first row, rows, length of its sequence) of every owned query block, by arithmetic alone."""
    lens, owned = _lengths(c)
    bs = c["block"]
    if owned is None:
        owned = [(s, i) for s, n in enumerate(lens) for i in range(-(-n // bs))]
    return lens, [(int(i) * bs, min(bs, lens[s] - int(i) * bs), lens[s]) for s, i in owned]


def _nnz(c):
    """Unmasked score entries of one query head."""
    lens, rows = _owned_rows(c)
    if not c["causal"]:
        return sum(n * length for _, n, length in rows)
    return sum(n * first + n * (n + 1) // 2 for first, n, _ in rows)


def _rows(c):
    """(query rows, KV rows, rows of the partial buffers)."""
    lens, rows = _owned_rows(c)
    parts = 0
    for first, n, length in rows:
        pairs = first // c["block"] + 1 if c["causal"] else -(-length // c["block"])
        parts += n * (1 if c["coalesce"] == 0 else -(-pairs // c["coalesce"]))
    return sum(n for _, n, _ in rows), sum(lens), parts


def work(case):
    t_q, t_kv, _ = _rows(case)
    hq, hkv, d = case["hq"], case["hkv"], case["d"]
    q, kv, o = 2 * t_q * hq * d, 2 * t_kv * hkv * d, (4 if case["o32"] else 2) * t_q * hq * d
    lse = 4 * t_q * hq
    n_bytes, flops = q + 2 * kv + o + lse, 4 * d * hq * _nnz(case)
    if case["mode"] == "train":
        g = 2 if case["g16"] else 4
        n_bytes += q + g * (t_q * hq * d + 2 * t_kv * hkv * d)       # dO in; dQ, dK, dV out
        flops += 10 * d * hq * _nnz(case)
    return {"bytes": n_bytes, "flops": flops}


def tolerance(case):
    # Operands, P and dS are bf16 (unit roundoff 2^-9), sums fp32.  Against fp64 on the same inputs the worst output
    # (bf16 gradients) is off by 2.4e-3 in the 2-norm and 3.5e-2 at its worst element (an fp32 gradient, rms as the
    # unit); two orders of the same sums differ by 9e-4 and 1.6e-2.  Four times the larger.
    return {"rel": 8e-3, "max": 0.15}


class _State:
    pass


def _workspace(problem, dev):
    n = fcp.fcp_workspace_bytes(problem)
    buf = torch.empty(n + 256, dtype=torch.uint8, device=dev)
    ptr = buf.data_ptr() + (-buf.data_ptr()) % 256
    fcp.fcp_queue_build(problem, ptr, n, torch.cuda.current_stream().cuda_stream)
    return buf, ptr


def prepare(case, seed):
    c, s, dev = case, _State(), torch.device("cuda:0")
    lens, owned = _lengths(c)
    hq, hkv, d, bs, causal = c["hq"], c["hkv"], c["d"], c["block"], int(c["causal"])
    if c["packed"]:
        blocks, mem, comp = fcp.fcp_block_costs(lens, bs, causal)
        plan = fcp.fcp_plan_blocks_packed(lens, bs, causal, c["coalesce"], owned, fcp.fcp_pack_units(blocks, mem, comp, bs)[0])
    else:
        plan = fcp.fcp_plan_blocks(lens, bs, causal, c["coalesce"], owned)
    t_q, t_kv = int(plan["q_blocks"][:, 3].sum()), int(plan["kv_blocks"][:, 3].sum())
    g = torch.Generator(device=dev).manual_seed(int(seed))

    def normal(rows, heads):
        return torch.randn((rows, heads, d), generator=g, device=dev, dtype=torch.float32).to(torch.bfloat16)

    def empty(*shape, dtype=torch.float32):
        return torch.empty(shape, dtype=dtype, device=dev)

    s.mode = c["mode"]
    s.q, s.k, s.v = normal(t_q, hq), normal(t_kv, hkv), normal(t_kv, hkv)
    s.o = empty(t_q, hq, d, dtype=torch.float32 if c["o32"] else torch.bfloat16)
    s.lse = empty(t_q, hq)
    flags = fcp.FCP_FLAG_O_F32 if c["o32"] else 0
    if s.mode == "running":
        s.stages = []
        n_stages = fcp.fcp_stage_tables(plan, 0)[1]
        for k in range(n_stages):
            stage = fcp.fcp_stage_tables(plan, k)[0]
            problem = fcp.Problem(stage, hq, hkv, d, bs, 0.0, flags | fcp.FCP_FLAG_RUNNING_MERGE)
            s.stages.append((problem,) + _workspace(problem, dev))
        return s
    flags |= fcp.FCP_FLAG_DIRECT_SINGLE
    if s.mode == "train":
        flags |= (fcp.FCP_FLAG_GRAD_BF16 if c["g16"] else 0) | (fcp.FCP_FLAG_BWD_SPILL_DS if c["spill"] else 0)
        grad = torch.bfloat16 if c["g16"] else torch.float32
        s.d_o = normal(t_q, hq)
        s.dq, s.dk, s.dv = empty(t_q, hq, d, dtype=grad), empty(t_kv, hkv, d, dtype=grad), empty(t_kv, hkv, d, dtype=grad)
    s.problem = fcp.Problem(plan, hq, hkv, d, bs, 0.0, flags)
    rows = max(1, s.problem.n_slot_rows)
    s.o_part, s.lse_part = empty(rows, hq, d), empty(rows, hq)
    s.ws, s.ws_ptr = _workspace(s.problem, dev)
    return s


def run(s):
    stream = torch.cuda.current_stream().cuda_stream
    if s.mode == "running":
        s.lse.fill_(float("-inf"))                   # "nothing yet"
        for problem, _, ws_ptr in s.stages:
            fcp.fcp_block_attn_fwd_out(problem, s.q, s.k, s.v, None, None, s.o, s.lse, ws_ptr, stream)
        return s.o, s.lse
    fcp.fcp_block_attn_fwd_out(s.problem, s.q, s.k, s.v, s.o_part, s.lse_part, s.o, s.lse, s.ws_ptr, stream)
    fcp.fcp_merge_partials(s.problem, s.o_part, s.lse_part, s.o, s.lse, s.ws_ptr, stream)
    if s.mode == "fwd":
        return s.o, s.lse
    fcp.fcp_block_attn_bwd(s.problem, s.q, s.k, s.v, s.o, s.lse, s.d_o, s.dq, s.dk, s.dv, s.ws_ptr, stream)
    return s.o, s.lse, s.dq, s.dk, s.dv

"""Which kernels the launches of a problem take (fcp_launch_probe): host integer work, no GPU."""
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

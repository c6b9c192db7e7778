"""The parity tests of small problems once more, with every problem on the kernels that walk a work item as a whole
(FCP_FLAG_WHOLE_ITEMS).  Without the flag most of these problems are small enough for the split kernels, so that the kernels
of large steps would see none of their edges: ragged tiles, short runs, packed members, tables with gaps, bf16 gradients."""
import pytest

from paper_2605_08524_amd import binding as B
from test_gpu_parity import (  # noqa: F401  (collected here a second time, under the fixture below)
    test_all_logits_strongly_negative_with_ragged_blocks, test_backward_stage_entry_points_agree, test_bf16_gradients_are_the_fp32_gradients_rounded_once,
    test_bf16_gradients_edge_cases, test_bwd_runs_from_bf16_o, test_bwd_short_runs, test_config1_tiny, test_config1_tiny_running_merge,
    test_config1_tiny_with_spilled_ds, test_edge_cases_bwd_with_spilled_ds, test_edge_cases_direct_single_slot, test_edge_cases_fwd_bwd,
    test_edge_cases_running_merge, test_few_items_split_over_waves, test_members_joined_into_runs, test_packed_blocks_fwd_bwd,
    test_packed_blocks_of_many_tiny_sequences, test_packed_blocks_through_the_other_entry_points, test_packed_query_block_with_further_slots,
    test_peaked_softmax_large_logits, test_query_blocks_without_slots, test_repeated_calls_reuse_the_workspace,
    test_spans_of_neighbouring_and_distant_blocks, test_spill_flag_keeps_ds, test_spilled_ds_backward_stage_calls_and_bf16_gradients,
    test_tables_with_gaps_and_turned_slots, test_wave_share_queue_and_staging_edges, test_whole_step_replays_from_a_hip_graph)

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def whole_items(monkeypatch):
    init = B.Problem.__init__

    def with_flag(self, plan, n_q_heads, n_kv_heads, head_dim, block_size, softmax_scale=0.0, flags=0):
        init(self, plan, n_q_heads, n_kv_heads, head_dim, block_size, softmax_scale, flags | B.FCP_FLAG_WHOLE_ITEMS)
        assert B.fcp_launch_probe(self)["split"] == (False, False, False)

    monkeypatch.setattr(B.Problem, "__init__", with_flag)

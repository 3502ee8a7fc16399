"""Sizes at which a launch changes its shape (splits, tiles, variants of a kernel), each against the CPU oracle on the same inputs."""
import pytest

import focus_inputs as fi
from test_gpu_parity import compare_steps, small_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prefix,batch,block", [(96, 1, 32), (97, 1, 32), (2016, 1, 32), (2144, 1, 32), (2140, 1, 5), (9001, 1, 32), (2144, 3, 24)])
def test_attention_context_splits_and_their_merge(prefix, batch, block):
    """Few sequences: the context is cut into ranges of two K/V tiles and more (1, 2, 16, 17 and about 70 ranges: both merge kernels and
    their edges), and the launch has workgroups that only warm the next weights.  The last case mixes lengths, so sequences with one range
    and with many share a launch.  The bf16 bound of the parity tests."""
    lengths = dict(prefix_lo=prefix, prefix_hi=prefix, prefix_dist="fixed") if batch == 1 else dict(prefix_lo=5, prefix_hi=prefix)
    compare_steps(small_bf16(batch=batch, n_q_heads=4, n_kv_heads=1, n_layers=3, block_size=block, steps=1, **lengths), 1, 2e-2, exact=False)


@pytest.mark.parametrize("shape", [dict(hidden=264, ffn=40, vocab=1003, batch=3, block_size=5),            # remainders of the 16-wide tiles
                                   dict(hidden=1032, ffn=520, vocab=515, batch=1, block_size=17),          # eight wavefronts, K not a multiple of 16
                                   dict(hidden=64, ffn=64, vocab=17, batch=2, block_size=1),               # the smallest
                                   dict(hidden=128, ffn=64, vocab=4100, batch=33, block_size=32),          # lm_head: 1072 tiles of 64 x 64
                                   dict(prefix_lo=200, prefix_hi=203, page_size=8, head_dim=128, n_q_heads=4, n_kv_heads=2)])
def test_fp32_projections_and_attention(shape):
    """fp32 models at the remainders of the projection and attention tiles and on both sides of the projections' dispatch, decisions
    exact and values within the fp32 bound of the parity tests."""
    budget = dict(budget_mode=1, keep_ratio=1.0) if shape.get("batch") == 33 else {}
    compare_steps(fi.workload("c1_tiny", **dict(shape, **budget)), 2, 1e-3, exact=True)


@pytest.mark.parametrize("shape", [dict(page_size=1, prefix_lo=3, prefix_hi=5), dict(page_size=1, prefix_lo=61, prefix_hi=64), dict(prefix_lo=0, prefix_hi=1)])
def test_admission_upload(shape):
    """Page tables longer than the prompts (the upload has a region of its own then), shorter, and prompts without tokens."""
    compare_steps(fi.workload("c1_tiny", **shape), 2, 1e-3, exact=True)


@pytest.mark.parametrize("shape", [dict(batch=3, prefix_lo=1, prefix_hi=300, vocab=512, mask_token_id=511),      # several passes, ragged last blocks
                                   dict(batch=1, prefix_lo=257, prefix_hi=257, vocab=8192, mask_token_id=8191),  # one pass, one token in its last block
                                   dict(batch=70, prefix_lo=0, prefix_hi=40, block_size=4, n_layers=2)])         # more prompts than a wavefront has lanes, some empty
def test_prefill_of_several_blocks_per_pass(shape):
    """Prompts whose blocks share a pass, and passes that end inside a prompt; keys and values of every layer show in the steps."""
    compare_steps(small_bf16(**dict(dict(prefill="prompt", steps=1), **shape)), 1, 2e-2, exact=False)


@pytest.mark.parametrize("shape", [dict(batch=5, prefix_lo=1, prefix_hi=150, block_size=13), dict(batch=1, prefix_lo=640, prefix_hi=640, page_size=1),
                                   dict(n_experts=4, experts_per_token=2, expert_ffn=64, shared_ffn=64, first_moe_layer=0, prefix_hi=200)])
def test_prefill_of_several_blocks_per_pass_fp32(shape):
    compare_steps(fi.workload("c1_tiny", **shape), 2, 1e-3, exact=True)


@pytest.mark.parametrize("batch,block", [(3, 19), (5, 18), (8, 16), (15, 10), (27, 7), (31, 7), (10, 25), (11, 25), (64, 8)])
def test_projection_tile_heights(batch, block):
    """57 to 512 rows against a vocabulary of 200 column tiles: every tile height of the pipelined projection (64 to 256 rows, by the
    vocabulary's launch) with a remainder in both directions, and K cut in parts (the layers' launches)."""
    compare_steps(small_bf16(batch=batch, block_size=block, keep_ratio=1.0, vocab=51176, mask_token_id=51175, n_layers=2, steps=1), 1, 2e-2, exact=False)


@pytest.mark.parametrize("shape", [dict(n_q_heads=17, n_kv_heads=17, batch=3), dict(n_q_heads=40, n_kv_heads=4, batch=2, block_size=64, prefix_hi=70),
                                   dict(n_q_heads=1, n_kv_heads=1, batch=300, block_size=2, hidden=64, ffn=64, vocab=64, prefill="synthetic")])
def test_head_sums_and_packing(shape):
    """Importance summed over more heads than are loaded at a time, and over one; more sequences than the packing kernel has threads."""
    compare_steps(fi.workload("c1_tiny", **shape), 1, 1e-3, exact=True)


@pytest.mark.parametrize("vocab", [40968, 66000, 140001])
def test_confidence_merge_of_many_slots(vocab):
    """Fewer than one, more than one and more than two trips of the merge's threads over the projection's column slots."""
    compare_steps(small_bf16(vocab=vocab, mask_token_id=vocab - 1, batch=5, n_layers=2, steps=1), 1, 2e-2, exact=False)

"""Sizes at which a launch changes its shape (splits, tiles, variants of a kernel), each against the CPU oracle on the same inputs."""
import numpy as np
import pytest
import torch

import focus_inputs as fi
from test_gpu_parity import DEV, Outs, _pk, compare_steps, relerr, small_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prefix,batch,block", [(96, 1, 32), (97, 1, 32), (224, 1, 32), (2016, 1, 32), (2144, 1, 32), (2140, 1, 5), (9001, 1, 32),
                                                (8928, 1, 32), (2144, 3, 24)])
def test_attention_context_splits_and_their_merge(prefix, batch, block):
    """Few sequences: the context is cut into 1, 1, 2, 16 and 17 ranges of two K/V tiles (both merge kernels at their border), 12 and 48 of
    three, 70 of two.  The last case mixes lengths, so sequences with one range and with many share a launch.  The bf16 bound of the parity tests."""
    lengths = dict(prefix_lo=prefix, prefix_hi=prefix, prefix_dist="fixed") if batch == 1 else dict(prefix_lo=5, prefix_hi=prefix)
    compare_steps(small_bf16(batch=batch, n_q_heads=4, n_kv_heads=1, n_layers=3, block_size=block, steps=1, **lengths), 1, 2e-2, exact=False)


@pytest.mark.parametrize("kv_heads,group,rows,lo,hi,dist,resident", [(65, 1, 3, 200, 2500, "uniform", 2), (65, 2, 20, 200, 2500, "uniform", 2), (65, 1, 3, 900, 900, "uniform", 4),
                                                                     (65, 2, 20, 900, 900, "uniform", 4), (120, 1, 3, 300, 1300, "uniform", 4), (130, 1, 3, 500, 1500, "uniform", 3),
                                                                     (130, 2, 20, 500, 1500, "uniform", 3), (130, 1, 2, 100, 3000, "loguniform", 2)])
def test_attention_rounds_of_uneven_sequences(kv_heads, group, rows, lo, hi, dist, resident):
    """520, 960 and 1040 (sequence, kv head) pairs, uneven and even, of one wavefront (up to 32 rows x query heads of the group) and of two: two,
    three and four workgroups per compute unit."""
    wl = small_bf16(batch=8, n_q_heads=kv_heads * group, n_kv_heads=kv_heads, hidden=256, ffn=256, vocab=512, mask_token_id=511, n_layers=2, block_size=32,
                    keep_ratio=rows / 32, prefix_lo=lo, prefix_hi=hi, prefix_dist=dist, steps=1)
    totals, groups = [x + 32 for x in wl.prefix_lens()], 8 * kv_heads       # the rule of attention_resident(), so that the lengths cannot drift off it
    mean, ratio = sum(totals) // 8, max(totals) * 8 / sum(totals)
    if groups <= 1024:
        assert resident == (2 if mean >= 768 and ratio > 1.5 else 4) and (resident == 2 or ratio < 1.4)
    else:
        assert resident == (2 if ratio > 2.55 else 3) and (resident == 2 or ratio < 2.4)
    assert 512 < groups <= 1536 and max(totals) < 4096 and (rows * group <= 32) == (group == 1)
    compare_steps(wl, 1, 2e-2, exact=False)


@pytest.mark.parametrize("block,prefix", [(32, 1100), (16, 1000)])
def test_a_step_does_not_depend_on_what_the_context_held_before(block, prefix):
    """Bitwise: one request in a fresh context; after a long request was in another slot; after many attempts to finalise its block, which
    raise the bound of the lengths that the host keeps; and by a slot list in device memory."""
    pk, runner = _pk()
    wl = small_bf16(batch=2, n_q_heads=4, n_kv_heads=1, block_size=block, prefix_lo=prefix, prefix_hi=prefix, prefix_dist="fixed", steps=1, extra_blocks=7000 // block)
    sess = runner.open_session(wl, DEV)
    f, tables = sess.focus, sess.page_tables
    outs = Outs(pk, wl, 1)

    def first_step(slot=None):
        f.focus_prefill_kv([prefix], [tables[0]])
        for t in outs.t.values():
            t.zero_()
        f.focus_step(1, seq_slot=slot, out=outs.struct)
        return outs.host()
    fresh = first_step()
    long = prefix + 7000 // block * block
    f.focus_prefill_kv([long], [tables[1]], seq_slot=[1])
    after_a_long_one = first_step()
    for _ in range(40):
        f.focus_finalize_blocks(1)
    after_finalising = first_step()
    by_slot_list = first_step(torch.zeros(1, dtype=torch.int32, device=DEV))
    for other in (after_a_long_one, after_finalising, by_slot_list):
        for k in fresh:
            assert np.array_equal(fresh[k], other[k]), k
    f.focus_free()


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


@pytest.mark.parametrize("hidden,batch,block,vocab", [(256, 2, 9, 1030), (264, 1, 16, 1030), (512, 2, 16, 8000), (512, 3, 16, 8200), (520, 1, 16, 4090), (1024, 1, 16, 4096),
                                                      (1024, 1, 17, 4096), (1032, 1, 7, 300)])
def test_fp32_rmsnorm_inside_the_projections_and_apart(hidden, batch, block, vocab):
    """Both sides of gemm_fuses_rmsnorm: all of K held by four wavefronts (256 columns), eight (512) and eight with twice the pieces (1024), with
    remainders of each, and launches of one tile more than a fused one may have."""
    wl = fi.workload("c1_tiny", hidden=hidden, ffn=136, vocab=vocab, batch=batch, block_size=block, keep_ratio=1.0, prefill="synthetic")
    compare_steps(wl, 1, 1e-3, exact=True)


@pytest.mark.parametrize("shape", [dict(page_size=16, block_size=5), dict(page_size=16, block_size=32), dict(head_dim=64, block_size=32), dict(head_dim=64, page_size=16, block_size=5),
                                   dict(page_size=16, n_q_heads=16, n_kv_heads=4, batch=8, keep_ratio=1.0, prefill="synthetic"),                    # 4096 (row, head) pairs
                                   dict(head_dim=64, page_size=32, n_q_heads=32, n_kv_heads=8, batch=8, keep_ratio=1.0, prefill="synthetic")])       # 8192
def test_bf16_attention_off_the_matrix_cores(shape):
    """Heads of 64 and pages of other than 64 tokens, with prompts (whose last blocks are ragged), and enough rows for the in-order kernel."""
    compare_steps(small_bf16(**dict(dict(prefix_lo=1, prefix_hi=150, prefill="prompt", n_layers=2, steps=1), **shape)), 1, 2e-2, exact=False)


@pytest.mark.parametrize("shape", [dict(head_dim=128, page_size=16), dict(head_dim=128, page_size=64), dict(head_dim=64, page_size=8, batch=16)])
def test_fp32_attention_of_many_rows(shape):
    """4096 to 8192 (row, head) pairs: in order on pages of less than 64 tokens, one wavefront a row on longer ones for groups of heads."""
    compare_steps(fi.workload("c1_tiny", **dict(dict(n_q_heads=16, n_kv_heads=4, batch=8, block_size=32, budget_mode=1, keep_ratio=1.0, prefix_lo=1,
                                                     prefix_hi=90, prefill="synthetic"), **shape)), 1, 1e-3, exact=True)


@pytest.mark.parametrize("shape", [dict(page_size=1, prefix_lo=3, prefix_hi=5), dict(page_size=1, prefix_lo=61, prefix_hi=64), dict(prefix_lo=0, prefix_hi=1)])
def test_admission_upload(shape):
    """Page tables longer than the prompts, shorter, and prompts without tokens."""
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


EXPERTS = dict(n_experts=64, experts_per_token=8, expert_ffn=64, shared_ffn=64, first_moe_layer=0)


@pytest.mark.parametrize("shape", [dict(EXPERTS, batch=8, vocab=64, prefix_lo=60, prefix_hi=64),           # expert buffers outweigh the logits
                                   dict(EXPERTS, batch=1, vocab=64, prefix_lo=100, prefix_hi=100),
                                   dict(batch=5, vocab=64, hidden=64, ffn=64, n_q_heads=1, n_kv_heads=1, page_size=1, block_size=4, prefix_lo=20, prefix_hi=30,
                                        extra_blocks=1000)])                                              # long page tables
def test_prefill_passes_hold_a_block_of_every_sequence(shape):
    """However little room the workspace leaves, the prompts need no more passes than the longest of them has blocks."""
    from paper_2601_23278_amd.binding import KC_KV_WRITE
    wl = fi.workload("c1_tiny", **shape)
    compare_steps(wl, 1, 1e-3, exact=True)
    pk, runner = _pk()
    sess = runner.open_session(wl, DEV)
    lens = wl.prefix_lens()
    sess.focus.focus_set_timing(True)
    sess.focus.focus_prefill_kv(lens, sess.page_tables, wl.prompt_tokens(lens))
    _, launches = sess.focus.focus_get_kernel_time(KC_KV_WRITE)                    # one per layer and pass
    assert launches <= wl.n_layers * max(-(-x // wl.block_size) for x in lens), launches
    sess.focus.focus_free()


def compare_without_logits(wl):
    """Without a logits output the vocabulary projection reduces its tiles in the epilogue and the triples are merged per row: against the
    same step with the logits, which compare_steps() holds against the oracle.  Arg-max tokens and commits are the same, confidences
    differ by the order of the sums of exponentials."""
    pk, runner = _pk()
    sess = runner.open_session(wl, DEV)
    n = wl.batch
    full = Outs(pk, wl, n)
    sess.focus.focus_step(n, out=full.struct)
    with_logits = full.host()
    sess.focus.focus_prefill_kv(sess.prefix_lens, sess.page_tables, None)          # the same block again
    lean = {k: torch.zeros_like(full.t[k]) for k in ("tokens", "mask_bits", "keep_bits", "cu_seqlens", "conf", "argmax")}
    sess.focus.focus_step(n, out=pk.make_step_out(**lean))
    torch.cuda.synchronize()
    rows = int(with_logits["cu_seqlens"][n])
    assert rows > 0
    for k in ("tokens", "mask_bits", "keep_bits", "cu_seqlens"):
        assert np.array_equal(lean[k].cpu().numpy(), with_logits[k]), k
    assert np.array_equal(lean["argmax"].cpu().numpy()[:rows], with_logits["argmax"][:rows])
    assert relerr(lean["conf"].cpu().numpy()[:rows], with_logits["conf"][:rows]) < 1e-5
    sess.focus.focus_free()


# rows that take tiles of 64, 96, 128, 160, 192, 224 and 256 rows where a launch has 63 column tiles (four tile rows fill the chip and the
# next lower height would need a fifth), the last tile with rows missing
TILE_ROWS = [(10, 25), (13, 29), (17, 29), (22, 29), (26, 29), (19, 47), (35, 29)]
# K = 128 is not cut in parts; neither 16000, 2 x 8128 nor 16100 columns fill their last column tile
WIDE = dict(n_layers=2, keep_ratio=1.0, prefix_lo=3, prefix_hi=20, hidden=128, n_q_heads=75, n_kv_heads=25, ffn=8128, vocab=16100, mask_token_id=16099, steps=1)


@pytest.mark.parametrize("batch,block", TILE_ROWS)
def test_projection_tile_heights(batch, block):
    """Every tile height with a remainder in rows and columns: bf16 store (QKV), SiLU*up (gate/up), fp32 store and confidences (vocabulary)."""
    wl = small_bf16(batch=batch, block_size=block, **WIDE)
    compare_steps(wl, 1, 2e-2, exact=False)
    compare_without_logits(wl)


@pytest.mark.parametrize("batch,block", [(17, 59), (25, 61), (33, 61), (41, 61), (50, 61), (58, 61), (66, 61)])
def test_projection_tile_heights_adding_to_the_residual_stream(batch, block):
    """The same for the projections that add to the residual stream (O and down): 16 column tiles, the last with columns missing, and 16 tile
    rows of 64 to 256 rows, the last with rows missing."""
    wl = small_bf16(batch=batch, block_size=block, **dict(WIDE, hidden=4032, n_q_heads=1, n_kv_heads=1, ffn=128, vocab=300, mask_token_id=299))
    compare_steps(wl, 1, 2e-2, exact=False)


def test_confidence_of_the_lowest_tiles():
    """185 rows x 20300 tokens: confidences from tiles of 64 rows."""
    compare_without_logits(small_bf16(batch=5, block_size=37, **dict(WIDE, vocab=20300, mask_token_id=20299)))


@pytest.mark.parametrize("batch,block", [(3, 19), (5, 18), (8, 16), (15, 10), (27, 7), (31, 7), (10, 25), (11, 25), (64, 8)])
def test_projections_of_57_to_512_rows(batch, block):
    """Few column tiles, so that K is cut in parts (the layers), and 200 of them (the vocabulary)."""
    compare_steps(small_bf16(batch=batch, block_size=block, keep_ratio=1.0, vocab=51176, mask_token_id=51175, n_layers=2, steps=1), 1, 2e-2, exact=False)


@pytest.mark.parametrize("vocab,hint,most", [(300, 200, 7), (9000, 200, 7), (9000, 60, 7), (9000, 1105, 40)])
def test_k_parts_of_a_row_count_only_the_device_knows(vocab, hint, most):
    """About 200 of 4224 rows stay.  O and down, which add to the residual stream, in four parts of K, which lie 4224 rows apart: 138 MB, beyond
    the buffer of the K parts but within the room of 9000 logits a row; with 300 there is neither and K is not cut.  With 60 rows expected the
    launch that adds the parts makes further trips, and so with 1105, more than 2048 workgroups take in one."""
    wl = small_bf16(batch=66, block_size=64, hidden=2048, n_q_heads=16, n_kv_heads=1, ffn=4096, prefix_lo=3, prefix_hi=70, vocab=vocab, mask_token_id=vocab - 1,
                    n_layers=3, budget_mode=3, steps=1)
    compare_steps(wl, 1, 2e-2, exact=False, k_override=[b % most for b in range(66)], row_hint=(hint, most - 1))


@pytest.mark.parametrize("batch,block,ffn", [(1, 32, 12288), (1, 5, 12352), (11, 3, 12288)])
def test_projections_of_few_rows_with_many_weights(batch, block, ffn):
    """Gate/up of 100 MB: 32 and 5 rows in two parts of 16 slabs, the last column tile with columns missing; 33 rows are one too many."""
    compare_steps(small_bf16(batch=batch, block_size=block, hidden=2048, ffn=ffn, n_q_heads=2, n_kv_heads=1, n_layers=2, steps=1), 1, 2e-2, exact=False)


@pytest.mark.parametrize("shape", [dict(n_q_heads=17, n_kv_heads=17, batch=3), dict(n_q_heads=40, n_kv_heads=4, batch=2, block_size=64, prefix_hi=70),
                                   dict(n_q_heads=1, n_kv_heads=1, batch=300, block_size=2, hidden=64, ffn=64, vocab=64, prefill="synthetic")])
def test_head_sums_and_packing(shape):
    """Importance summed over more heads than are loaded at a time, and over one; more sequences than the packing kernel has threads."""
    compare_steps(fi.workload("c1_tiny", **shape), 1, 1e-3, exact=True)


@pytest.mark.parametrize("vocab", [40968, 66000, 140001])
def test_confidence_merge_of_many_slots(vocab):
    """644, 1032 and 2188 slots a row: one, two and three trips of 256 threads with four slots each, 40 rows."""
    wl = small_bf16(vocab=vocab, mask_token_id=vocab - 1, batch=5, n_layers=2, steps=1)
    compare_steps(wl, 1, 2e-2, exact=False)
    compare_without_logits(wl)


@pytest.mark.parametrize("wl", [fi.workload("c1_tiny", n_layers=3), fi.workload("c1_tiny", n_layers=3, head_dim=128), small_bf16(head_dim=64),
                                small_bf16(page_size=16), small_bf16(batch=33, prefix_lo=70, prefix_hi=90),
                                small_bf16(prefix_lo=1000, prefix_hi=1100), small_bf16(batch=2, prefix_lo=8000, prefix_hi=8100)],
                         ids=["fp32", "fp32 128", "bf16 64", "bf16 small pages", "one range", "few ranges", "many ranges"])
def test_a_key_that_is_not_a_number_shows(wl):
    """Attention over a prefix with a NaN key gives NaN to that sequence's rows (never a number that hides it), and to no others."""
    pk, runner = _pk()
    sess = runner.open_session(wl, DEV)
    sess.kv_pool[wl.n_layers - 1, sess.page_tables[0][0], 0, :, 0, :] = float("nan")      # first token of sequence 0 in the last layer
    outs = Outs(pk, wl, wl.batch)
    sess.focus.focus_step(wl.batch, out=outs.struct)
    g = outs.host()
    cu = g["cu_seqlens"]
    assert cu[1] > 0 and np.all(np.isnan(g["hidden_packed"][:cu[1]]))
    assert np.all(np.isfinite(g["hidden_packed"][cu[1]:cu[-1]]))
    sess.focus.focus_free()


@pytest.mark.parametrize("wl,logits", [(fi.workload("c1_tiny"), True), (small_bf16(), True), (small_bf16(batch=33, keep_ratio=1.0), True),
                                       (small_bf16(vocab=41000, mask_token_id=40999), False)], ids=["fp32", "few rows", "many rows", "without logits"])
def test_committed_tokens_lie_in_the_vocabulary_whatever_the_logits(wl, logits):
    """Logits that are all NaN have no maximum: the steps commit tokens of the vocabulary all the same, and the next step embeds them."""
    pk, runner = _pk()
    sess = runner.open_session(wl, DEV)
    sess.weights[1].fill_(float("nan"))                       # lm_head
    outs = Outs(pk, wl, wl.batch)
    lean = pk.make_step_out(**{k: v for k, v in outs.t.items() if logits or k != "logits"})
    for _ in range(2):
        sess.focus.focus_step(wl.batch, out=lean)
        g = outs.host()
        assert np.all((g["tokens"] >= 0) & (g["tokens"] < wl.vocab)) and np.all(g["n_decoded"] > 0)
        assert np.all(np.isfinite(g["hidden_packed"]))
    sess.focus.focus_free()

"""Times that a dispatch rule or a row bound must not cost: each test sets a path against the same work on another path of the same library,
in one process, so that no figure depends on the card; the bounds lie between what the two sides measured with and without the fault."""
import pytest
import torch

import focus_inputs as fi
from paper_2601_23278_amd.binding import KC_ATTENTION, KC_EXPERTS, KC_GEMM, KC_KV_WRITE
from test_gpu_parity import DEV, _pk, small_bf16

pytestmark = pytest.mark.gpu


def open_context(wl, weights=None):
    pk, runner = _pk()
    sess = runner.open_session(wl, DEV)
    if weights is not None:
        cfg, ws = sess.focus.cfg, sess.focus.workspace
        sess.focus.focus_free()
        sess.weights = weights(*sess.weights)
        sess.focus = pk.Focus(cfg, *sess.weights, sess.kv_pool, ws)
        sess.focus.focus_prefill_kv(sess.prefix_lens, sess.page_tables, None)
    return sess


def step_us(sess, repeats=12, tries=5, **step):
    """Microseconds of a first denoising step, launches back to back, the best of a few tries."""
    f, n = sess.focus, len(sess.seq_ids)
    best = 1e30
    for _ in range(tries):
        f.focus_prefill_kv(sess.prefix_lens, sess.page_tables, None)
        begin, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        f.focus_step(n, **step)
        begin.record()
        for _ in range(repeats):
            f.focus_step(n, **step)
        end.record()
        torch.cuda.synchronize()
        best = min(best, begin.elapsed_time(end) * 1e3 / repeats)
    return best


def class_us(sess, kernel_class, tries=6, **step):
    """Microseconds of the launches of a class in a first denoising step, the best of a few tries."""
    f, best = sess.focus, 1e30
    f.focus_set_timing(True)
    for _ in range(tries):
        f.focus_prefill_kv(sess.prefix_lens, sess.page_tables, None)
        f.focus_step(len(sess.seq_ids), **step)
        best = min(best, f.focus_get_kernel_time(kernel_class)[0] * 1e3)
    f.focus_set_timing(False)
    return best


def packed_layer_us(kernel_class, rows, **model):
    """The class's time in one layer of `rows` packed rows whose count only the device knows: of 8192 rows that there can be, and of 256."""
    us = {}
    for batch in (128, 4):
        per_seq = -(-rows // batch)
        k = torch.tensor([max(0, min(per_seq, rows - b * per_seq)) for b in range(batch)], dtype=torch.int32, device=DEV)
        assert int(k.sum()) == rows
        at = {}
        for layers in (2, 8):
            wl = small_bf16(batch=batch, block_size=64, n_layers=layers, budget_mode=3, prefix_lo=3, prefix_hi=70, steps=1, **model)
            sess = open_context(wl)
            sess.focus.focus_set_row_hint(rows, per_seq)
            at[layers] = class_us(sess, kernel_class, k_override=k)
            sess.focus.focus_free()
        us[batch * 64] = (at[8] - at[2]) / 6
    print(rows, us, flush=True)
    return us


def test_adding_k_parts_costs_by_the_rows_there_are():
    """200 rows, K of QKV, gate/up and down in four parts.  Read for every row there can be, the parts made that 386 us a layer
    instead of 93."""
    us = packed_layer_us(KC_GEMM, 200, hidden=4096, n_q_heads=2, n_kv_heads=1, ffn=4096, vocab=36000, mask_token_id=35999)
    assert us[8192] <= 2 * us[256], us


def test_rotation_and_kv_write_cost_by_the_rows_there_are():
    """200 rows of 40 heads.  V of many short sequences is written by more workgroups, so that with 8192 rows that there can be a layer takes 9.7
    us, with 256 13.7; reading queries and keys of every row there can be made the former 15.7."""
    us = packed_layer_us(KC_KV_WRITE, 200, hidden=512, n_q_heads=32, n_kv_heads=8, ffn=512, vocab=512, mask_token_id=511)
    assert us[8192] <= 0.92 * us[256], us


def test_attention_off_the_matrix_cores_costs_by_the_rows_there_are():
    """200 rows of 32 heads on the fallback path: 133 us a layer where there can be 8192 rows, 121 where 256; 264 when the query of every row
    there can be was read."""
    us = packed_layer_us(KC_ATTENTION, 200, hidden=512, n_q_heads=32, n_kv_heads=32, head_dim=64, ffn=512, vocab=512, mask_token_id=511)
    assert us[8192] <= 1.5 * us[256], us


def test_experts_of_several_row_tiles_do_not_read_their_weights_anew():
    """256 experts with 128 rows each, one tile, and with 256 on average: 1.69 times the time of the expert projections,
    2.12 when each of the two or three tiles read the weights past the caches."""
    us = {}
    for batch in (128, 256):
        wl = small_bf16(batch=batch, keep_ratio=1.0, n_layers=3, hidden=2048, n_q_heads=2, n_kv_heads=1, ffn=256, vocab=512, mask_token_id=511, prefix_lo=3, prefix_hi=30,
                        steps=1, n_experts=256, experts_per_token=8, expert_ffn=512, first_moe_layer=1)
        sess = open_context(wl)
        rows = batch * 32
        routes = torch.arange(rows * 8, dtype=torch.int32, device=DEV) % 256
        if batch == 256:
            routes = torch.rand(rows, 256, device=DEV, generator=torch.Generator(DEV).manual_seed(5)).topk(8, dim=1).indices.to(torch.int32)
        sess.focus.focus_set_route_override(routes.reshape(1, rows, 8).expand(3, -1, -1).contiguous())
        us[rows // 32] = class_us(sess, KC_EXPERTS)
        sess.focus.focus_free()
    print(us, flush=True)
    assert us[256] <= 1.9 * us[128], us


@pytest.mark.parametrize("hidden,batch,block", [(256, 8, 32), (512, 16, 32), (1024, 1, 16), (1024, 8, 32), (2048, 2, 32)])
def test_rmsnorm_goes_into_fp32_projections_only_where_that_is_faster(hidden, batch, block):
    """A norm whose weights are not aligned to 16 bytes has a launch of its own.  Fused wherever the projections allowed it, the aligned model
    took 1.23 times as long with 512 rows x 512 columns, 1.16 with 256 x 1024 and 1.46 with 64 x 2048."""
    wl = fi.workload("c1_tiny", hidden=hidden, n_q_heads=hidden // 64, n_kv_heads=hidden // 64, ffn=2 * hidden, vocab=4096, n_layers=4, batch=batch, block_size=block,
                     keep_ratio=1.0, prefill="synthetic")

    def off_by_four(embed, lm_head, norm, layers):
        norm = torch.cat([norm[:1], norm])[1:]
        assert norm.data_ptr() % 16 == 4
        return embed, lm_head, norm, [dict(l, attn_norm=norm, mlp_norm=norm) for l in layers]
    us = {}
    for name, weights in (("aligned", None), ("apart", off_by_four)):
        sess = open_context(wl, weights)
        us[name] = step_us(sess)
        sess.focus.focus_free()
    print(hidden, batch, block, us, flush=True)
    assert us["aligned"] <= 1.08 * us["apart"], us

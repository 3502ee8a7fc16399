"""Sizes at which a launch changes its shape (splits, tiles, variants of a kernel), each against the CPU oracle on the same inputs."""
import pytest

from test_gpu_parity import compare_steps, small_bf16

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prefix,batch,block", [(96, 1, 32), (97, 1, 32), (2016, 1, 32), (2144, 1, 32), (2140, 1, 5), (9001, 1, 32), (2144, 3, 24)])
def test_attention_context_splits_and_their_merge(prefix, batch, block):
    """Few sequences: the context is cut into ranges of two K/V tiles and more (1, 2, 16, 17 and about 70 ranges: both merge kernels and
    their edges), and the launch has workgroups that only warm the next weights.  The last case mixes lengths, so sequences with one range
    and with many share a launch.  The bf16 bound of the parity tests."""
    lengths = dict(prefix_lo=prefix, prefix_hi=prefix, prefix_dist="fixed") if batch == 1 else dict(prefix_lo=5, prefix_hi=prefix)
    compare_steps(small_bf16(batch=batch, n_q_heads=4, n_kv_heads=1, n_layers=3, block_size=block, steps=1, **lengths), 1, 2e-2, exact=False)

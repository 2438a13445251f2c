"""Attention over head counts on both sides of the rule that gives an XCD whole
heads, at sequence lengths around the 64-row blocks."""
import pytest

from paper_2608_18469_amd import synth_tf
from tests.test_gpu_transformer import _check_bf16, _gpu_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,seq,batch", [(1, 64, 8), (3, 129, 3), (2, 1, 4), (5, 63, 13)])
def test_attention_order(heads, seq, batch):
    cfg = synth_tf.tf_config("tf_tiny", vocab=128, d=64 * heads, heads=heads, layers=1, seq=seq, batch=batch)
    params, batches = synth_tf.make_workload(cfg, seed=22, n_batches=1)
    _, gpu = _gpu_run(cfg, params, batches, "serial")
    _check_bf16(cfg, gpu, params, batches)

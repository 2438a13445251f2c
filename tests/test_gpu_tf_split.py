"""The vocabulary head's input gradient in fp32 slices (contractions of 16
64-wide steps and more), in the GEMM core's tiles and in 128x128 ones, with a
last slice shorter than the others."""
import pytest

from paper_2608_18469_amd import synth_tf
from tests.test_gpu_transformer import _bits_equal, _check_bf16, _gpu_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("vocab,heads,seq,batch", [(1024, 1, 33, 2), (1088, 3, 65, 3), (4160, 2, 64, 2), (2112, 2, 700, 2)])
def test_head_slices(vocab, heads, seq, batch):
    cfg = synth_tf.tf_config("tf_tiny", vocab=vocab, d=64 * heads, heads=heads, layers=2, seq=seq, batch=batch)
    params, batches = synth_tf.make_workload(cfg, seed=21, n_batches=1)
    _, gpu = _gpu_run(cfg, params, batches, "serial")
    _check_bf16(cfg, gpu, params, batches)
    _, again = _gpu_run(cfg, params, batches, "overlap")
    _bits_equal(gpu, again)

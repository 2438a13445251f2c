"""Attention over head counts on both sides of the rule that gives an XCD whole
heads, at sequence lengths around the 64-row blocks."""
import ctypes

import pytest

from paper_2608_18469_amd import erase, erase_tf, synth_tf
from tests.test_gpu_transformer import _check_bf16, _gpu_run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("heads,seq,batch", [(1, 64, 8), (3, 129, 3), (2, 1, 4), (5, 63, 13)])
def test_attention_order(heads, seq, batch):
    cfg = synth_tf.tf_config("tf_tiny", vocab=128, d=64 * heads, heads=heads, layers=1, seq=seq, batch=batch)
    params, batches = synth_tf.make_workload(cfg, seed=22, n_batches=1)
    _, gpu = _gpu_run(cfg, params, batches, "serial")
    _check_bf16(cfg, gpu, params, batches)


def test_attention_of_more_workgroups_than_a_grid_row():
    """2^20 sequences of one token, 8 heads: the backward has 2^24 workgroups.
    Every position attends to itself alone: o is v, dQ and dK are nothing next
    to dV, and dV of every position is written (the workspace starts as zeros)."""
    import torch
    cfg = synth_tf.tf_config("tf_tiny", vocab=64, d=512, heads=8, layers=1, seq=1, batch=1 << 20)
    params, batches = synth_tf.make_workload(cfg, seed=23, n_batches=1)
    n, d = cfg["batch"], cfg["d"]
    print(f"[attention] {n} sequences of 1, {cfg['heads']} heads", flush=True)
    tr = erase_tf.TfTrainer(cfg, params, keep_grads=False)
    tr.step(tr.device_tokens(batches[0]), "serial")
    tr.sync()

    def view(name, cols):
        p, ld = ctypes.c_void_p(), ctypes.c_int64(0)
        assert erase.lib().erase_tf_tensor(tr.ctx, 0, erase_tf.TENSORS[name], ctypes.byref(p), ctypes.byref(ld)) == 0
        off = p.value - tr.ws.data_ptr()
        raw = tr.ws[off:off + n * ld.value * 2].view(torch.bfloat16).view(n, ld.value)
        return raw[:, :cols]

    v, o, dqkv = view("qkv", 3 * d)[:, 2 * d:], view("o", d), view("dqkv", 3 * d)
    # the probability is 1 up to its rounding: o is v up to the last place of a bf16
    assert bool(((o.float() - v.float()).abs() <= 2.0 ** -7 * v.float().abs()).all())
    dv = dqkv[:, 2 * d:].float().abs().amax(1)
    assert bool((dv > 0).all())
    # dS = P (dP - D), two fp32 sums of the same 64 products: about 64 ulps of their size
    assert float(dqkv[:, :2 * d].float().abs().max()) <= 1e-3 * float(dv.max())
    tr.close()

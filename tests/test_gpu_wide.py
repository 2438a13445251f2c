"""The 256x256 GEMM tiles at ragged sizes against the oracles: every epilogue
of their forward and input-gradient kernels, split weight gradients with bias
sums, and the launch that runs both backward GEMMs of a layer.

The batch is past 128 rows of 256, so the plan takes the wide tiles, and
nothing is a multiple of them: 32900 rows, widths 500, 520 and 260.
Tolerances as in the other bf16 parity tests (bf16_gate).
"""
import numpy as np
import pytest

from paper_2608_18469_amd import erase, erase_tf, synth, synth_tf
from tests.gpu_util import assert_bit_identical, check_bf16, run_gpu
from tests.test_gpu_transformer import _bits_equal, _check_bf16, _gpu_run

pytestmark = pytest.mark.gpu


def _wide(tr, *batch, schedule):
    tr.set_timing(True)
    tr.step(*batch, schedule)
    tr.sync()
    return {(r["kind"], r["block"], r["layer"]) for r in tr.read_timing()[1:] if r["tile_m"] == 256}


def _cross_cfg():
    layers = [("cross", 500, 500), ("cross", 500, 500), ("linear_relu", 500, 520), ("linear_relu", 520, 520)]
    return synth.custom("bf16", 32900, 500, [{"input": "x", "layers": layers, "lam": 1.0}], label_p=0.2)


def _chain_cfg():
    blocks = [{"input": "x", "layers": [("linear_relu", 500, 520)], "lam": 1.0},
              {"input": "prev", "layers": [("linear_relu", 520, 260), ("linear_relu", 260, 516)], "lam": 0.5}]
    return synth.custom("bf16", 32900, 500, blocks, label_p=0.2)


@pytest.mark.parametrize("name,cfg,schedule,want", [
    ("cross", _cross_cfg(), "overlap", {("fwd_gemm", 0, 0), ("fwd_gemm", 0, 2), ("bwd_gemm", 0, 1), ("bwd_gemm", 0, 2),
                                        ("bwd_gemm", 0, 3), ("wgrad_gemm", 0, 0)}),
    ("chain", _chain_cfg(), "undetached", {("fwd_gemm", 0, 0), ("dgrad_gemm", 1, 0), ("wgrad_gemm", 0, 0)}),
])
def test_wide_tiles_vs_oracle(name, cfg, schedule, want):
    print(f"[wide] {name} {schedule}", flush=True)
    params, batches = synth.make_workload(cfg, 3, 1)
    _, g = run_gpu(cfg, params, batches, schedule)
    if schedule == "overlap":
        assert_bit_identical(g, run_gpu(cfg, params, batches, "serial")[1])
    check_bf16(cfg, g, params, batches, detach=schedule != "undetached")
    tr = erase.Trainer(cfg, params)
    got = _wide(tr, *tr.device_batch(*batches[0]), schedule=schedule)
    tr.close()
    assert want <= got, sorted(want - got)


def test_wide_tiles_transformer_vs_oracle():
    """The transformer's kinds (residual, GELU and its derivative) over 33000
    ragged positions, width 192."""
    cfg = synth_tf.tf_config("tf_tiny", vocab=512, d=192, heads=3, layers=2, seq=200, batch=165)
    params, batches = synth_tf.make_workload(cfg, seed=5, n_batches=1)
    print("[wide] transformer N 33000 d 192", flush=True)
    _, a = _gpu_run(cfg, params, batches, "serial")
    _, b = _gpu_run(cfg, params, batches, "overlap")
    _bits_equal(a, b)
    _check_bf16(cfg, a, params, batches)
    tr = erase_tf.TfTrainer(cfg, params)
    got = _wide(tr, tr.device_tokens(batches[0]), schedule="serial")
    tr.close()
    names = [{(k, w) for (k, blk, w) in got if blk == i} for i in range(2)]
    fwd = {("fwd_gemm", w) for w in (0, 1, 2, 3)} | {("dgrad_gemm", 3)}
    assert all(fwd <= n for n in names), names
    assert np.isfinite(a[0]["losses"]).all()

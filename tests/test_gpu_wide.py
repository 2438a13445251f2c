"""The 256x256 and 128x128 GEMM tiles at ragged sizes against the oracles: every
epilogue of their forward and input-gradient kernels, split weight gradients
with bias sums, and the launch that runs both backward GEMMs of a layer.  No
batch or width is a multiple of a tile.  Tolerances as in the other bf16
parity tests (bf16_gate).
"""
import numpy as np
import pytest

from paper_2608_18469_amd import erase, erase_tf, synth, synth_tf
from tests.gpu_util import assert_bit_identical, check_bf16, run_gpu
from tests.test_gpu_transformer import _bits_equal, _check_bf16, _gpu_run

pytestmark = pytest.mark.gpu


def _tiles(tr, *batch, schedule):
    tr.set_timing(True)
    tr.step(*batch, schedule)
    tr.sync()
    return {(r["kind"], r["block"], r["layer"], r["tile_m"]) for r in tr.read_timing()[1:]}


def _cross_cfg(batch, d, w):
    layers = [("cross", d, d), ("cross", d, d), ("linear_relu", d, w), ("linear_relu", w, d)]
    return synth.custom("bf16", batch, d, [{"input": "x", "layers": layers, "lam": 1.0}], label_p=0.2)


def _chain_cfg():
    blocks = [{"input": "x", "layers": [("linear_relu", 500, 900)], "lam": 1.0},
              {"input": "prev", "layers": [("linear_relu", 900, 500), ("linear_relu", 500, 700)], "lam": 0.5}]
    return synth.custom("bf16", 20000, 500, blocks, label_p=0.2)


@pytest.mark.parametrize("name,cfg,schedule,want", [
    ("cross 256", _cross_cfg(16300, 1000, 1000), "overlap",
     {("fwd_gemm", 0, 0, 256), ("fwd_gemm", 0, 2, 256), ("bwd_gemm", 0, 1, 256), ("bwd_gemm", 0, 2, 256),
      ("bwd_gemm", 0, 3, 256), ("wgrad_gemm", 0, 0, 128)}),
    ("cross 128", _cross_cfg(3700, 700, 650), "overlap",
     {("fwd_gemm", 0, 0, 128), ("fwd_gemm", 0, 2, 128), ("bwd_gemm", 0, 1, 128), ("bwd_gemm", 0, 2, 128),
      ("bwd_gemm", 0, 3, 128)}),
    ("chain 128", _chain_cfg(), "undetached", {("fwd_gemm", 0, 0, 128), ("bwd_gemm", 1, 0, 128)}),
])
def test_wide_tiles_vs_oracle(name, cfg, schedule, want):
    print(f"[wide] {name} {schedule}", flush=True)
    params, batches = synth.make_workload(cfg, 3, 1)
    _, g = run_gpu(cfg, params, batches, schedule)
    if schedule == "overlap":
        assert_bit_identical(g, run_gpu(cfg, params, batches, "serial")[1])
    check_bf16(cfg, g, params, batches, detach=schedule != "undetached")
    tr = erase.Trainer(cfg, params)
    got = _tiles(tr, *tr.device_batch(*batches[0]), schedule=schedule)
    tr.close()
    assert want <= got, (sorted(want - got), sorted(got))


@pytest.mark.parametrize("n,batch,d,w", [(1, 12001, 1937, 1457), (6, 19990, 1697, 437)])
def test_wide_wgrad_alone(n, batch, d, w):
    """The 256x256 weight gradient without an input gradient beside it, split,
    in a launch of one block and in launches of two (units of six blocks)."""
    layers = [("linear_relu", d, w)]
    cfg = synth.custom("bf16", batch, d, [{"input": "x", "layers": layers, "lam": 1.0 + 0.1 * i} for i in range(n)],
                       label_p=0.2)
    params, batches = synth.make_workload(cfg, 4, 1)
    print(f"[wide] wgrad {n} x {batch} {d} {w}", flush=True)
    _, g = run_gpu(cfg, params, batches, "overlap")
    assert_bit_identical(g, run_gpu(cfg, params, batches, "serial")[1])
    check_bf16(cfg, g, params, batches)
    tr = erase.Trainer(cfg, params)
    got = _tiles(tr, *tr.device_batch(*batches[0]), schedule="overlap")
    tr.close()
    assert ("wgrad_gemm", 0, 0, 256) in got, sorted(got)


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
    got = _tiles(tr, tr.device_tokens(batches[0]), schedule="serial")
    tr.close()
    big = {(k, b, w) for (k, b, w, t) in got if t in (128, 256)}
    want = {("fwd_gemm", b, w) for w in (0, 1, 2, 3) for b in (0, 1)} | {("dgrad_gemm", b, 3) for b in (0, 1)}
    assert want <= big, (sorted(want - big), sorted(got, key=str))
    assert np.isfinite(a[0]["losses"]).all()

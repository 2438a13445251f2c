"""Blocks of equal shape share launches: the same bits as when a block of
another shape between them keeps their launches apart, in every schedule.

Widths are odd, so every tile, chunk and segment has a remainder; the blocks'
lambdas differ.  "256" and "128" run those tiles, "256" with a first-layer
weight gradient that leaves Adam a launch of its own.  (Two blocks there: they
share launches in the schedules on one stream, and tiles are chosen for one.)
"""
import numpy as np
import pytest

from paper_2608_18469_amd import erase, synth
from tests.gpu_util import run_gpu

pytestmark = pytest.mark.gpu

CROSS = [("cross", 150, 150), ("cross", 150, 150), ("linear_relu", 150, 75), ("linear_relu", 75, 140)]
CASES = {
    "bf16 fused head": ("bf16", 333, 150, [("linear_relu", 150, 131), ("linear_relu", 131, 65)]),
    "bf16 cross": ("bf16", 777, 150, CROSS),
    "f32 fused head": ("f32", 333, 150, [("linear_relu", 150, 70), ("linear_relu", 70, 33)]),
    "f32 cross": ("f32", 200, 150, CROSS),
    "128": ("bf16", 3700, 700, [("cross", 700, 700), ("linear_relu", 700, 650), ("linear_relu", 650, 700)]),
    "256": ("bf16", 16300, 1000, [("cross", 1000, 1000), ("linear_relu", 1000, 1000), ("linear_relu", 1000, 1000)]),
}


def _say(*a):
    print(*a, flush=True)


def _bits(a, b, idx):
    """Blocks of run a against blocks idx of run b."""
    for ra, rb in zip(a, b):
        assert np.array_equal(ra["losses"].view(np.uint32), rb["losses"][idx].view(np.uint32))
        for k in ("params", "m", "v", "grads"):
            for i, j in enumerate(idx):
                assert np.array_equal(np.asarray(ra[k][i]).view(np.uint32), np.asarray(rb[k][j]).view(np.uint32)), (k, i)


def _kinds(cfg, params, batch, schedule):
    tr = erase.Trainer(cfg, params)
    tr.set_timing(True)
    tr.step(*tr.device_batch(*batch), schedule)
    tr.sync()
    n = len(tr.read_timing()) - 1
    tr.close()
    return n


@pytest.mark.parametrize("name", list(CASES))
def test_equal_blocks_share_launches(name):
    dtype, batch, in_dim, layers = CASES[name]
    n = 2 if name in ("128", "256") else 7  # seven: groups of two (three units and one block) in the ERASE schedules
    block = lambda i: {"input": "x", "layers": layers, "lam": 1.0 + 0.25 * i}
    other = {"input": "x", "layers": [("linear_relu", in_dim, 17)], "lam": 1.0}
    apart = [b for i in range(n) for b in (block(i), other)]
    cfg = synth.custom(dtype, batch, in_dim, [block(i) for i in range(n)], label_p=0.3)
    ref_cfg = synth.custom(dtype, batch, in_dim, apart, label_p=0.3)
    ref_params, batches = synth.make_workload(ref_cfg, 21, 1 if n == 2 else 2)
    params = ref_params[::2]
    _say(f"[shared] {name}: apart")
    ref = run_gpu(ref_cfg, ref_params, batches, "serial")[1]
    for sched in ("serial", "overlap", "pipeline", "overlap_adam_end", "serial_graph", "undetached"):
        _say(f"[shared] {name}: {sched}")
        _bits(run_gpu(cfg, params, batches, sched, bwd_streams=2)[1], ref, list(range(0, 2 * n, 2)))
    if n > 2:
        assert _kinds(cfg, params, batches[0], "serial") * 3 < _kinds(ref_cfg, ref_params, batches[0], "serial")


@pytest.mark.parametrize("dtype,width", [("bf16", 150), ("bf16", 65), ("f32", 150), ("f32", 33)])
def test_chained_blocks_share_backward_launches(dtype, width):
    """A chain of equal blocks (standalone and fused heads): the serial
    schedule shares the backward over all of them, the ERASE ones in units,
    and with a chain cut into single-block units by blocks of other widths in
    between, each block's backward runs alone; the undetached step shares
    heads and Adam.  Every detached schedule gives the same bits; graphs and
    eager steps too."""
    blocks = [{"input": "x" if i == 0 else "prev", "layers": [("linear_relu", width, 90), ("linear_relu", 90, width)],
               "lam": 1.0 + 0.1 * i} for i in range(9)]
    cfg = synth.custom(dtype, 600, width, blocks, label_p=0.3)
    params, batches = synth.make_workload(cfg, 23, 2)
    _say(f"[shared] chain {dtype} {width}: serial")
    ref = run_gpu(cfg, params, batches, "serial")[1]
    for sched in ("overlap", "pipeline", "overlap_adam_end", "overlap_graph"):
        _say(f"[shared] chain {dtype} {width}: {sched}")
        _bits(run_gpu(cfg, params, batches, sched, bwd_streams=2)[1], ref, list(range(9)))
    _say(f"[shared] chain {dtype} {width}: undetached")
    a = run_gpu(cfg, params, batches, "undetached")[1]
    _bits(run_gpu(cfg, params, batches, "undetached_graph")[1], a, list(range(9)))
    # alone: each block as a network of its own on the activations it read is
    # the same launch with one job; here the first blocks of shorter chains,
    # whose groups have other sizes, give the same bits
    for n in (1, 2, 3):
        sub = synth.custom(dtype, 600, width, blocks[:n], label_p=0.3)
        got = run_gpu(sub, params[:n], batches, "serial")[1]
        cut = [{k: (v[:n] if k == "losses" else v[:n]) for k, v in r.items()} for r in ref]
        _bits(got, cut, list(range(n)))

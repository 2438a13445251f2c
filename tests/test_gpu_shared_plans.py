"""Blocks whose plan depends on how many of them share a launch: networks whose
ERASE units are of unequal size, at sizes beyond the GEMM core's tiles.  Every
schedule gives the serial schedule's bits, and that one matches the oracle."""
import pytest

from paper_2608_18469_amd import synth
from tests.gpu_util import assert_bit_identical, check_bf16, run_gpu

pytestmark = pytest.mark.gpu

LIN = "linear_relu"
CASES = {
    "chain 6": (4096, 512, 6, [(LIN, 512, 512), (LIN, 512, 512)], True),
    "chain 9": (1651, 512, 9, [(LIN, 512, 508), (LIN, 508, 512)], True),
    "x 7": (4096, 512, 7, [(LIN, 512, 512), (LIN, 512, 512)], False),
    "ctr 10": (4096, 1677, 10, [(LIN, 1677, 512), (LIN, 512, 256), (LIN, 256, 128)], False),
    "dcn 7": (4096, 1677, 7, [("cross", 1677, 1677), (LIN, 1677, 1024), (LIN, 1024, 512)], False),
}


@pytest.mark.parametrize("name", list(CASES))
def test_uneven_units(name):
    batch, in_dim, n, layers, chain = CASES[name]
    blocks = [{"input": "prev" if chain and b else "x", "layers": layers, "lam": 1.0 + 0.1 * b} for b in range(n)]
    cfg = synth.custom("bf16", batch, in_dim, blocks, label_p=0.2)
    params, batches = synth.make_workload(cfg, 31, 1)
    print(f"[plans] {name}: serial", flush=True)
    ref = run_gpu(cfg, params, batches, "serial")[1]
    for sched in ("serial_graph", "overlap", "overlap_graph", "pipeline", "overlap_adam_end"):
        print(f"[plans] {name}: {sched}", flush=True)
        assert_bit_identical(run_gpu(cfg, params, batches, sched, bwd_streams=2)[1], ref)
    check_bf16(cfg, ref, params, batches)
    print(f"[plans] {name}: undetached", flush=True)
    und = run_gpu(cfg, params, batches, "undetached")[1]
    if chain:
        check_bf16(cfg, und, params, batches, detach=False)
    else:
        assert_bit_identical(und, ref)


@pytest.mark.parametrize("batch,width,mid", [(4096, 512, 1024), (3343, 608, 1326)])
def test_undetached_long_first_layer(batch, width, mid):
    """An input gradient across a cut with a contraction of 1024 and more into
    few columns, below the 128x128 tiles' range."""
    blocks = [{"input": "x", "layers": [(LIN, width, width)], "lam": 1.0}]
    blocks += [{"input": "prev", "layers": [(LIN, width, mid), (LIN, mid, width)], "lam": 0.5}] * 2
    cfg = synth.custom("bf16", batch, width, blocks, label_p=0.2)
    params, batches = synth.make_workload(cfg, 33, 1)
    print(f"[plans] undetached {batch} {width} {mid}", flush=True)
    check_bf16(cfg, run_gpu(cfg, params, batches, "undetached")[1], params, batches, detach=False)

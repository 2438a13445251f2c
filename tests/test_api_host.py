"""Host-only checks of the C ABI: the library loads, exports every entry
point the header declares, and validates configurations before any HIP call
(no GPU needed: nothing here launches device work)."""
import ctypes
import os
import re

import pytest

from paper_2608_18469_amd import erase, synth

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared_functions():
    with open(os.path.join(ROOT, "include", "erase.h")) as f:
        text = f.read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(erase_[a-z_]+)\s*\(", text)))


def test_library_exports_every_declared_symbol():
    L = erase.lib()
    names = _declared_functions()
    assert len(names) >= 13
    for n in names:
        assert hasattr(L, n), n
    assert set(names) == set(erase.SIGNATURES), set(names) ^ set(erase.SIGNATURES)


def test_library_hides_its_internal_host_functions():
    """Built with hidden visibility: the host-side launchers and planners are
    not exported, only the C entry points (and the kernels, which the HIP
    runtime registers)."""
    L = erase.lib()
    for internal in ("_ZN5erase11launch_gemmEiiRKNS_8GemmDescERKNS_9EpiParamsEP12ihipStream_tRKNS_8LaunchEvEPKNS_5BatchE",
                     "_ZN5erase11launch_adamEiRKNS_8AdamArgsEP12ihipStream_tRKNS_8LaunchEvEPKNS_5BatchE",
                     "_ZN5erase11launch_gemmEiiRKNS_8GemmDescERKNS_9EpiParamsEP12ihipStream_tRKNS_8LaunchEvE",
                     "_ZN5erase11launch_adamEiRKNS_8AdamArgsEP12ihipStream_tRKNS_8LaunchEvE"):
        assert not hasattr(L, internal), internal


def test_status_strings():
    L = erase.lib()
    for s in range(0, -8, -1):
        assert L.erase_status_str(s) and L.erase_status_str(s) != b"unknown status"
    assert L.erase_status_str(42) == b"unknown status"


def _ncfg(cfg, **kw):
    return erase.NativeConfig(cfg, **kw)


def test_param_count_matches_generator():
    for name in ("tiny", "ctr_mlp", "ctr_dcn", "deep_chain"):
        cfg = synth.config(name)
        nc = _ncfg(cfg)
        total = sum(erase.param_count(nc, b) for b in range(len(cfg["blocks"])))
        assert total == synth.param_count(cfg)
    assert synth.param_count(synth.config("ctr_mlp")) == 6140934
    assert synth.param_count(synth.config("ctr_dcn")) == 53527182
    assert synth.param_count(synth.config("deep_chain")) == 1582092


def test_pack_unpack_roundtrip():
    cfg = synth.config("tiny")
    params, _ = synth.make_workload(cfg, 0, 1)
    for blk, p in zip(cfg["blocks"], params):
        flat = erase.pack_block(p)
        q = erase.unpack_block(blk, flat)
        for (W, b), (W2, b2) in zip(p["layers"], q["layers"]):
            assert (W == W2).all() and (b == b2).all()
        assert (q["head"][0] == p["head"][0]).all() and (q["head"][1] == p["head"][1]).all()


def test_workspace_bytes_positive_and_monotone_in_batch():
    a = erase.workspace_bytes(_ncfg(synth.config("ctr_mlp", batch=1024)))
    b = erase.workspace_bytes(_ncfg(synth.config("ctr_mlp")))
    assert 0 < a < b
    # full CTR-MLP: activations in two layouts, gradients, partials; well under 1 GiB
    assert b < (1 << 30)


def _status_ws(cfg_mut):
    cfg = synth.config("tiny")
    nc = _ncfg(cfg)
    cfg_mut(nc)
    n = ctypes.c_size_t(0)
    return erase.lib().erase_workspace_bytes(nc.ptr(), ctypes.byref(n))


@pytest.mark.parametrize("mut,code", [
    (lambda nc: setattr(nc.c, "n_blocks", 0), erase.ERR_SHAPE),
    (lambda nc: setattr(nc.c, "batch", 0), erase.ERR_SHAPE),
    (lambda nc: setattr(nc.c, "dtype", 7), erase.ERR_INVALID_ARG),
    (lambda nc: setattr(nc.c, "x_ld", 15), erase.ERR_SHAPE),
    (lambda nc: setattr(nc.c, "x_ld", 18), erase.ERR_SHAPE),  # 72 bytes: not a multiple of 16
    (lambda nc: setattr(nc.c, "lr", float("nan")), erase.ERR_INVALID_ARG),
    (lambda nc: setattr(nc.c, "beta1", 1.0), erase.ERR_INVALID_ARG),
    (lambda nc: setattr(nc.c, "eps", -1.0), erase.ERR_INVALID_ARG),
    (lambda nc: setattr(nc._blocks[0], "input_src", erase.IN_PREV), erase.ERR_INVALID_ARG),
    (lambda nc: setattr(nc._blocks[1], "input_src", 5), erase.ERR_INVALID_ARG),
    (lambda nc: setattr(nc._blocks[0], "loss", 3), erase.ERR_UNSUPPORTED),
    (lambda nc: setattr(nc._blocks[0], "n_layers", 0), erase.ERR_SHAPE),
    (lambda nc: setattr(nc._blocks[0], "lam", float("inf")), erase.ERR_INVALID_ARG),
    (lambda nc: setattr(nc._layers[0][0], "in_dim", 17), erase.ERR_SHAPE),
    (lambda nc: setattr(nc._layers[0][1], "in_dim", 31), erase.ERR_SHAPE),
    (lambda nc: setattr(nc._layers[0][1], "kind", 9), erase.ERR_INVALID_ARG),
    (lambda nc: setattr(nc._layers[0][1], "kind", erase.CROSS), erase.ERR_UNSUPPORTED),
])
def test_validation_errors(mut, code):
    assert _status_ws(mut) == code


def test_cross_must_keep_width_and_precede_linear():
    blocks = [{"input": "x", "layers": [("cross", 8, 8), ("linear_relu", 8, 4)], "lam": 1.0}]
    nc = _ncfg(synth.custom("f32", 16, 8, blocks))
    assert erase.workspace_bytes(nc) > 0
    bad = [{"input": "x", "layers": [("linear_relu", 8, 8), ("cross", 8, 8), ("linear_relu", 8, 4)], "lam": 1.0}]
    n = ctypes.c_size_t(0)
    assert erase.lib().erase_workspace_bytes(_ncfg(synth.custom("f32", 16, 8, bad)).ptr(), ctypes.byref(n)) \
        == erase.ERR_UNSUPPORTED
    bad = [{"input": "x", "layers": [("cross", 8, 6), ("linear_relu", 6, 4)], "lam": 1.0}]
    assert erase.lib().erase_workspace_bytes(_ncfg(synth.custom("f32", 16, 8, bad)).ptr(), ctypes.byref(n)) \
        == erase.ERR_SHAPE
    chain = [{"input": "x", "layers": [("linear_relu", 8, 6)], "lam": 1.0},
             {"input": "prev", "layers": [("linear_relu", 7, 4)], "lam": 1.0}]
    assert erase.lib().erase_workspace_bytes(_ncfg(synth.custom("f32", 16, 8, chain)).ptr(), ctypes.byref(n)) \
        == erase.ERR_SHAPE


def test_init_rejects_bad_arguments_before_any_hip_call():
    L = erase.lib()
    cfg = synth.config("tiny")
    nc = _ncfg(cfg)
    ctx = ctypes.c_void_p()
    bufs = (erase.BlockBuffers * 2)()
    # null buffers
    assert L.erase_init(nc.ptr(), bufs, ctypes.c_void_p(256), 1 << 20, ctypes.c_void_p(8), ctypes.c_void_p(16),
                        ctypes.byref(ctx)) == erase.ERR_INVALID_ARG
    for b in range(2):
        bufs[b] = erase.BlockBuffers(256, 512, 768, None)
    # same stream twice
    assert L.erase_init(nc.ptr(), bufs, ctypes.c_void_p(256), 1 << 20, ctypes.c_void_p(8), ctypes.c_void_p(8),
                        ctypes.byref(ctx)) == erase.ERR_INVALID_ARG
    # backward-stream arrays: repeated, null, too many, none
    for arr in ([16, 16], [16, 0], list(range(16, 16 + 9 * 8, 8)), []):
        sb = (ctypes.c_void_p * max(1, len(arr)))(*arr)
        assert L.erase_init_streams(nc.ptr(), bufs, ctypes.c_void_p(256), 1 << 20, ctypes.c_void_p(8), sb, len(arr),
                                    ctypes.byref(ctx)) == erase.ERR_INVALID_ARG
    # misaligned / null / small workspace
    assert L.erase_init(nc.ptr(), bufs, ctypes.c_void_p(100), 1 << 20, ctypes.c_void_p(8), ctypes.c_void_p(16),
                        ctypes.byref(ctx)) == erase.ERR_WORKSPACE
    assert L.erase_init(nc.ptr(), bufs, None, 1 << 20, ctypes.c_void_p(8), ctypes.c_void_p(16),
                        ctypes.byref(ctx)) == erase.ERR_WORKSPACE
    assert L.erase_init(nc.ptr(), bufs, ctypes.c_void_p(256), 16, ctypes.c_void_p(8), ctypes.c_void_p(16),
                        ctypes.byref(ctx)) == erase.ERR_WORKSPACE
    assert ctx.value is None
    # step/sync on a NULL context
    assert L.erase_step(None, None, None, 0, None) == erase.ERR_INVALID_ARG
    assert L.erase_sync(None) == erase.ERR_INVALID_ARG
    assert L.erase_set_dispatch(None, erase.DISPATCH_WORKER) == erase.ERR_INVALID_ARG
    assert L.erase_destroy(None) == erase.OK


def test_gemm_flop_count_of_ctr_mlp():
    # 26.51 MFLOP per sample: forward and weight gradient of every layer, input
    # gradient of every layer but the first of each block
    f = synth.gemm_flops_per_step(synth.config("ctr_mlp"))
    assert abs(f / 4096 / 1e6 - 26.51) < 0.01


def test_embed_bags_validation():
    """Shape, pointer and alignment checks of erase_embed_bags happen on the
    host before anything is enqueued (fake pointers are never dereferenced)."""
    L = erase.lib()
    good = dict(batch=8, n_dense=13, n_tables=2, dim=64, rows=100, nnz=10, dtype=erase.F32, x_ld=144)

    def call(cfg=None, **ptrs):
        c = dict(good)
        c.update(cfg or {})
        bc = erase.BagConfig(c["batch"], c["n_dense"], c["n_tables"], c["dim"], c["rows"], c["nnz"], c["dtype"],
                             c["x_ld"])
        p = dict(dense=256, offsets=512, indices=768, tables=1024, x=2048, status=None)
        p.update(ptrs)
        return L.erase_embed_bags(ctypes.byref(bc), p["dense"], p["offsets"], p["indices"], p["tables"], p["x"],
                                  p["status"], None)

    assert L.erase_embed_bags(None, None, None, None, None, None, None, None) == erase.ERR_INVALID_ARG
    for bad in ({"batch": 0}, {"n_dense": -1}, {"n_dense": 5000}, {"n_tables": 0}, {"dim": 0}, {"dim": 6},
                {"dim": 260}, {"rows": 0}, {"rows": 1 << 31}, {"nnz": -1}, {"x_ld": 140}, {"x_ld": 145},
                {"batch": 1 << 20, "n_tables": 4096}):
        assert call(bad) == erase.ERR_SHAPE, bad
    assert call({"dtype": 5}) == erase.ERR_INVALID_ARG
    for bad in (dict(dense=None), dict(offsets=None), dict(offsets=516), dict(indices=None), dict(indices=770),
                dict(tables=None), dict(tables=1032), dict(x=None), dict(x=2056), dict(status=258)):
        assert call(**bad) == erase.ERR_INVALID_ARG, bad


def test_embed_bags_backward_validation():
    """erase_embed_bags_backward: shape, pointer, alignment and scratch checks
    on the host before anything is enqueued (fake pointers never dereferenced)."""
    L = erase.lib()
    good = dict(batch=8, n_dense=13, n_tables=2, dim=64, rows=100, nnz=10, dtype=erase.F32, x_ld=144)

    def cfg_of(c):
        return erase.BagConfig(c["batch"], c["n_dense"], c["n_tables"], c["dim"], c["rows"], c["nnz"], c["dtype"],
                               c["x_ld"])

    need = ctypes.c_size_t(0)
    gc = cfg_of(good)
    assert L.erase_embed_bags_backward_scratch_bytes(ctypes.byref(gc), ctypes.byref(need)) == erase.OK
    # count, start per table row; bucket, row id, owner, slot, large- and
    # small-row lists per entry (int32, padded to 64); the lists' counters;
    # two scan totals per 4096 rows
    assert need.value == 4 * (2 * 256 + 6 * 64 + 64 + 2 * 64)

    def call(cfg=None, **ptrs):
        c = dict(good)
        c.update(cfg or {})
        bc = cfg_of(c)
        p = dict(offsets=512, indices=768, dx=2048, grad=4096, scratch=8192, nbytes=need.value, status=None)
        p.update(ptrs)
        return L.erase_embed_bags_backward(ctypes.byref(bc), p["offsets"], p["indices"], p["dx"], p["grad"],
                                           p["scratch"], p["nbytes"], p["status"], None)

    assert L.erase_embed_bags_backward(None, None, None, None, None, None, 0, None, None) == erase.ERR_INVALID_ARG
    for bad in ({"batch": 0}, {"n_tables": 0}, {"dim": 6}, {"dim": 260}, {"rows": 0}, {"nnz": -1}, {"x_ld": 140},
                {"rows": 1 << 30, "n_tables": 2}):
        assert call(bad) == erase.ERR_SHAPE, bad
    for bad in (dict(offsets=None), dict(offsets=516), dict(indices=None), dict(dx=None), dict(dx=2056),
                dict(grad=None), dict(grad=4100), dict(status=258)):
        assert call(**bad) == erase.ERR_INVALID_ARG, bad
    for bad in (dict(scratch=None), dict(scratch=8200), dict(nbytes=need.value - 4)):
        assert call(**bad) == erase.ERR_WORKSPACE, bad


def test_embed_bags_backward_noalloc_validation():
    """The allocation-free variant checks shapes and pointers like the scratch
    entry point and rejects shapes whose scratch exceeds its static array,
    all before any HIP call (fake pointers never dereferenced)."""
    L = erase.lib()
    ok = dict(batch=8, n_dense=13, n_tables=2, dim=64, rows=100, nnz=10, dtype=erase.F32, x_ld=144)

    def call(ptrs=None, **over):
        c = dict(ok)
        c.update(over)
        bc = erase.BagConfig(c["batch"], c["n_dense"], c["n_tables"], c["dim"], c["rows"], c["nnz"], c["dtype"],
                             c["x_ld"])
        p = dict(offsets=512, indices=768, dx=2048, grad=4096, status=None)
        p.update(ptrs or {})
        return L.erase_embed_bags_backward_noalloc(ctypes.byref(bc), p["offsets"], p["indices"], p["dx"], p["grad"],
                                                   p["status"], None)

    assert L.erase_embed_bags_backward_noalloc(None, None, None, None, None, None, None) == erase.ERR_INVALID_ARG
    for bad in ({"batch": 0}, {"dim": 6}, {"x_ld": 140}):
        assert call(**bad) == erase.ERR_SHAPE, bad
    for bad in (dict(offsets=None), dict(dx=2056), dict(grad=4100)):
        assert call(bad) == erase.ERR_INVALID_ARG, bad
    # 26 tables of 1,000,000 rows: about 312 MB of counters, past the 64 MiB array
    big = dict(n_tables=26, rows=1_000_000, x_ld=13 + 26 * 64 + 3)
    need = ctypes.c_size_t(0)
    bc = erase.BagConfig(8, 13, 26, 64, 1_000_000, 10, erase.F32, big["x_ld"])
    assert L.erase_embed_bags_backward_scratch_bytes(ctypes.byref(bc), ctypes.byref(need)) == erase.OK
    assert need.value > erase.BAG_SCRATCH_MAX
    assert call(**big) == erase.ERR_WORKSPACE


def test_x_in_place_validation_and_workspace():
    """x read in place: x_ld and batch must be multiples of 128, the flag 0 or
    1, and the workspace has no padded copy of x."""
    L = erase.lib()
    cfg = synth.config("ctr_mlp")
    copy = _ncfg(cfg)
    inplace = _ncfg(cfg, x_ld=1792, x_in_place=True)
    assert erase.workspace_bytes(inplace) < erase.workspace_bytes(copy)
    for over in (dict(x_ld=1680), dict(batch=4000)):
        nc = _ncfg(dict(cfg, batch=over.get("batch", cfg["batch"])), x_ld=over.get("x_ld", 1792), x_in_place=True)
        n = ctypes.c_size_t(0)
        assert L.erase_workspace_bytes(nc.ptr(), ctypes.byref(n)) == erase.ERR_SHAPE, over
    bad = _ncfg(cfg, x_ld=1792, x_in_place=True)
    bad.c.x_in_place = 2
    n = ctypes.c_size_t(0)
    assert L.erase_workspace_bytes(bad.ptr(), ctypes.byref(n)) == erase.ERR_INVALID_ARG

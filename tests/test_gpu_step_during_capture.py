"""A step enqueued on streams of its own while another stream is captured, by
the same thread or another, in the global and the thread-local mode: the capture
holds what it recorded, and the step gives its usual results."""
import threading

import numpy as np
import pytest

from paper_2608_18469_amd import erase, synth

pytestmark = pytest.mark.gpu


def test_step_beside_a_capture():
    import torch
    cfg = synth.config("tiny")
    params, batches = synth.make_workload(cfg, 0, 1)
    ref, tr = erase.Trainer(cfg, params), erase.Trainer(cfg, params)
    x, y = tr.device_batch(*batches[0])
    ref.step(x, y)
    tr.step(x, y)
    ref.sync()
    tr.sync()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()
    buf = torch.zeros(1024, device="cuda")
    torch.cuda.synchronize()
    total = 0
    for mode in ("global", "thread_local"):
        for other in ("same thread", "other thread", "other thread, default stream"):
            print(f"[capture] {mode}, {other}", flush=True)
            failed = []

            def go():
                try:
                    with torch.cuda.stream(torch.cuda.default_stream() if "default" in other else s2):
                        tr.step(x, y)
                except Exception as e:  # reported below, after the capture has ended
                    failed.append(e)

            graph = torch.cuda.CUDAGraph()
            with torch.cuda.graph(graph, stream=s1, capture_error_mode=mode):
                buf.add_(1)
                if other == "same thread":
                    go()
                else:
                    t = threading.Thread(target=go)
                    t.start()
                    t.join()
                buf.add_(1)
            assert not failed, failed
            graph.replay()
            torch.cuda.synchronize()
            total += 2
            assert buf[0].item() == total
            ref.step(x, y)
            ref.sync()
            tr.sync()
            assert np.array_equal(ref.losses.cpu().numpy(), tr.losses.cpu().numpy())
            for a, b in zip(ref.flat_state()[0], tr.flat_state()[0]):
                assert np.array_equal(np.asarray(a).view(np.uint32), np.asarray(b).view(np.uint32))
    ref.close()
    tr.close()

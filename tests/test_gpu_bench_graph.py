"""bench.time_gpu times graph replays: whatever the warm-up, the timed steps replay the captured
ten-step graph and launch only what is left over, and the captured run leaves the history as the
same steps without a graph (bitwise)."""
import os

import pytest
import torch

import bench
import paper_1009_3308_amd as pkg

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("steps,warmup", [(20, 5), (20, 0), (35, 20), (60, 2), (7, 5)])
def test_timed_steps_replay_the_graph(steps, warmup):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    if not os.path.exists(pkg.LIB_PATH):
        from paper_1009_3308_amd import build
        build.build()
    print(f"case: bench steps={steps} warmup={warmup}", flush=True)
    info = {}
    s, h, *_ = bench.time_gpu(pkg, torch, 31, 1e-4, steps, warmup, info=info)
    # the start-up steps (k <= order) are launched one by one
    chunks = (steps - max(0, s.order + 1 - warmup)) // 10
    captured, launched = s.graph_counts()
    assert captured == 1 and launched >= chunks
    assert info["graphs_launched"] == chunks and info["capture_call_steps"] == 10
    e, he, *_ = bench.time_gpu(pkg, torch, 31, 1e-4, steps, warmup, graph=False)
    assert e.graph_counts() == (0, 0)
    assert torch.equal(h, he)
    s.close()
    e.close()

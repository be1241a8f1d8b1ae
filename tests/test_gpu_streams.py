"""Calls on one stream while another stream's kernel holds compute units."""
import statistics
import time

import pytest
import torch

from paper_2603_06619_amd.stage import LossStage

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def inputs(n, H, V):
    hidden = torch.randn((n, H), device=DEV).to(torch.bfloat16)
    W = torch.empty((V, H), device=DEV, dtype=torch.bfloat16)
    for v in range(0, V, 1024):
        W[v:v + 1024] = 0.01 * torch.randn((min(1024, V - v), H), device=DEV)
    return hidden, W, torch.randint(0, V, (n,), device=DEV, dtype=torch.int32), n


def test_logits_beside_a_kernel_that_holds_compute_units():
    # 32 workgroups of 8192 k-slices hold 32 of 256 compute units for about 5 ms; the log-probs beside them (74 tiles per compute
    # unit, 2 ms) lose those, 1.14 times the time, and a little at the end: 1.2 to 1.3.  Were a workgroup dealt its whole
    # share in advance, the shares of the 32 would run after all others: 1.9
    held, short = LossStage(DEV), LossStage(DEV)
    y, x = inputs(256, 262144, 32 * 256), inputs(8192, 1024, 151936)
    event = lambda: torch.cuda.Event(enable_timing=True)

    def run(sa, sb):
        torch.cuda.synchronize()
        start, end, b_end = event(), event(), event()
        if sb is not None:
            with torch.cuda.stream(sb):
                held.logp(*y)
                b_end.record()
            time.sleep(0.0007)                            # until its contraction runs
        with torch.cuda.stream(sa):
            start.record()
            short.logp(*x)
            end.record()
        torch.cuda.synchronize()
        return start.elapsed_time(end), sb is None or end.elapsed_time(b_end) > 0

    for _ in range(4):                                    # two streams that the runtime put on different queues
        sa, sb = torch.cuda.Stream(), torch.cuda.Stream()
        run(sa, None), run(sb, None)
        alone = statistics.median(run(sa, None)[0] for _ in range(5))
        beside = [run(sa, sb) for _ in range(7)]
        beside = [t for t, overlapped in beside if overlapped]
        if len(beside) >= 5:
            ratio = statistics.median(beside) / alone
            print("alone %.2f ms, beside the other kernel x%.2f" % (alone, ratio))
            assert ratio < 1.5
            return
    pytest.skip("the calls of the two streams did not run at the same time")

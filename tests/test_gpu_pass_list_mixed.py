"""The list of passing events in calls of several classes: one stage in turn (masks behind each class's
own staging) and one stage per class side by side, bitwise the events and totals of the same call with
|A|^2 of every event."""
import pytest
import torch

pytestmark = pytest.mark.gpu

FEW, ALL = ("weight", "obs", "pass", "acc"), ("weight", "obs", "pass", "acc", "amp2")


@pytest.mark.parametrize("mode", ["MIXED_SEQUENTIAL", "MIXED_CONCURRENT"])
def test_mixed_calls(gpu_lib, mode):
    classes = [(7, 32, 500077), (5, 32, 4001), (9, 64, 71500), (8, 64, 150001), (12, 32, 70003)]
    cfgs = [gpu_lib.config(n, prec=p, seed=40 + n, dynamic_scale=int(n == 9)) for n, p, _ in classes]
    counts = [N for _, _, N in classes]
    old = gpu_lib.get_mixed_launch()
    gpu_lib.set_mixed_launch(getattr(gpu_lib, mode))
    try:
        print("pass list,", mode, flush=True)
        for _ in range(2):
            got, ref = gpu_lib.generate(cfgs, counts, outputs=FEW), gpu_lib.generate(cfgs, counts, outputs=ALL)
            torch.cuda.synchronize()
            for c, g, r in zip(classes, got, ref):
                assert 0 < int(r["pass"].sum()) < c[2], c
                for k in FEW:
                    assert torch.equal(g[k], r[k]), (c, k)
    finally:
        gpu_lib.set_mixed_launch(old)

"""FP64 on groups of lanes in workgroups of several waves: generation on four lanes takes them where every
compute unit has three or four waves (8193 to 16384 events), bg_amp2 of n = 6 on two lanes as set.  Each
event is bitwise that of one-wave workgroups, and the totals are bg_generate_noalloc's."""
import pytest
import torch

pytestmark = pytest.mark.gpu

OUT = ("weight", "amp2", "acc")


@pytest.mark.parametrize("n", [10, 11, 12])
def test_generation_on_four_lanes(gpu_lib, n):
    old = gpu_lib.get_lanes(n, 64)
    gpu_lib.set_lanes(n, 64, 4)
    try:
        c = gpu_lib.config(n, prec=64, use_pdf=0, sqrt_s=1000.0, seed=51)
        full = gpu_lib.generate(c, 16500, outputs=OUT)
        for N in (8192, 8193, 8207, 10001, 16383, 16384, 16385):
            print("group blocks", n, N, flush=True)
            r = gpu_lib.generate(c, N, outputs=OUT)
            a = {k: torch.zeros_like(v) for k, v in r.items()}
            gpu_lib.generate_noalloc(c, N, a)
            for k in ("weight", "amp2"):
                assert torch.equal(r[k], full[k][:N]) and torch.equal(a[k], r[k]), (N, k)
            assert torch.equal(a["acc"], r["acc"]), N
            s = r["weight"].sum()
            assert abs(r["acc"][0] - s) <= 1e-12 * s
    finally:
        gpu_lib.set_lanes(n, 64, old)


def test_amp2_on_two_lanes(gpu_lib):
    n = 6
    old = gpu_lib.get_lanes(n, 64), gpu_lib.get_launch(n, 64)
    r = gpu_lib.generate(gpu_lib.config(n, prec=64, use_pdf=0, sqrt_s=1000.0, seed=52), 1027,
                         outputs=("momenta", "hel", "order"))
    try:
        gpu_lib.set_lanes(n, 64, 2)
        gpu_lib.set_launch(n, 64, 64, 1)
        want = gpu_lib.amp2(n, 64, r["momenta"], r["hel"], r["order"])
        for block in (128, 192, 256):
            print("group blocks, amp2", block, flush=True)
            gpu_lib.set_launch(n, 64, block, 1)
            for N in (1, 33, 64, 65, 96, 97, 127, 128, 129, 1027):
                a = gpu_lib.amp2(n, 64, *(r[k][:N].contiguous() for k in ("momenta", "hel", "order")))
                assert torch.equal(a, want[:N]), (block, N)
    finally:
        gpu_lib.set_lanes(n, 64, old[0])
        gpu_lib.set_launch(n, 64, *old[1])

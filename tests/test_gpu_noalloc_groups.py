"""bg_generate_noalloc of FP64 groups on both sides of 2^18 partials (their workgroups hold 64 lanes
whatever size is set): weights and totals are bitwise bg_generate's.  What it accepts goes by the set
workgroup size, and the shipped shapes accept 2^24 events at n = 9."""
import ctypes

import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.fixture
def shape(gpu_lib):
    old = {}

    def set_shape(n, lanes, block):
        old.setdefault(n, (gpu_lib.get_lanes(n, 64), gpu_lib.get_launch(n, 64)))
        gpu_lib.set_lanes(n, 64, lanes)
        gpu_lib.set_launch(n, 64, block, 1)
    yield set_shape
    for n, (lanes, launch) in old.items():
        gpu_lib.set_lanes(n, 64, lanes)
        gpu_lib.set_launch(n, 64, *launch)


# 2^18 partials: 2^22 events on four lanes, 2^23 on two
@pytest.mark.parametrize("n,lanes,N", [(10, 4, (1 << 22) - 3), (10, 4, (1 << 22) + 67), (9, 2, (1 << 23) + 129)])
def test_totals_past_2_18_partials(gpu_lib, shape, n, lanes, N):
    shape(n, lanes, 256)
    c = gpu_lib.config(n, prec=64, seed=31)
    print(f"noalloc groups n={n} N={N}", flush=True)
    out = {k: torch.zeros(s, dtype=torch.float64, device="cuda") for k, s in (("weight", N), ("amp2", N), ("acc", 4))}
    got = gpu_lib.generate_noalloc(c, N, out)
    ref = gpu_lib.generate(c, N, outputs=("weight", "amp2", "acc"))
    for k in out:
        assert torch.equal(got[k], ref[k]), k
    assert ref["acc"][0] > 0


def test_accepted_counts(gpu_lib, shape):
    def status(n, N):
        outs = gpu_lib.BgOutputs()
        acc = torch.zeros(4, dtype=torch.float64, device="cuda")
        outs.acc = acc.data_ptr()
        c = gpu_lib.config(n, prec=64, seed=1)
        st = gpu_lib.raw().bg_generate_noalloc(ctypes.byref(c), N, None, ctypes.byref(outs), None)
        torch.cuda.synchronize()
        return st
    print("noalloc groups, accepted counts", flush=True)
    assert status(9, 1 << 24) == gpu_lib.BG_OK
    for n, lanes, block, most in ((10, 4, 64, (1 << 22) + 16), (10, 4, 128, (1 << 23) + 32), (9, 2, 64, (1 << 23) + 32)):
        shape(n, lanes, block)
        assert status(n, most) == gpu_lib.BG_OK and status(n, most + 1) == gpu_lib.BG_EINVAL, (n, block)

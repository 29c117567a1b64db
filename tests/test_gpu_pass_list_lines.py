"""The list of passing events on both sides of the counts where it starts, for each staged form: every
output and the totals are bitwise those of a call that evaluates every event."""
import pytest
import torch

pytestmark = pytest.mark.gpu

FEW, ALL = ("weight", "obs", "pass", "acc"), ("weight", "obs", "pass", "acc", "amp2")
# (n, precision, lanes setting, first count: 60 us by the cost table, 2^17 lanes)
LINES = [(7, 32, 1, 260870), (8, 32, 1, 166667), (9, 32, 2, 80000), (10, 32, 2, 65536), (11, 32, 2, 65536),
         (7, 64, 2, 193549), (8, 64, 2, 131072), (9, 64, 2, 65536), (10, 64, 4, 38217), (10, 64, 2, 65536),
         (11, 64, 4, 32768), (12, 64, 4, 32768)]


@pytest.mark.parametrize("n,prec,lanes,first", LINES)
def test_both_sides(gpu_lib, n, prec, lanes, first):
    old = gpu_lib.get_lanes(n, prec)
    gpu_lib.set_lanes(n, prec, lanes)
    try:
        for kw in ({}, dict(use_pdf=0, sqrt_s=1000.0)):
            c = gpu_lib.config(n, prec=prec, seed=61, **kw)
            for N in (first - 1, first, first + 65):
                print("pass list lines", n, prec, lanes, N, flush=True)
                got, ref = gpu_lib.generate(c, N, outputs=FEW), gpu_lib.generate(c, N, outputs=ALL)
                assert 0 < int(ref["pass"].sum()) < N
                for k in FEW:
                    assert torch.equal(got[k], ref[k]), (N, k)
    finally:
        gpu_lib.set_lanes(n, prec, old)

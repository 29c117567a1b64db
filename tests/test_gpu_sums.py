"""Compensated totals where most waves hold only zero weights: the workgroup reduction skips
the exchange in such waves, so its result is compared with the exact sum of the weights."""
import math

import pytest

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -53


# one-wave workgroups (FP32 n <= 8), workgroups of several waves (FP64), two lanes per event
@pytest.mark.parametrize("n,prec", [(4, 32), (8, 32), (5, 64), (7, 64), (10, 32)])
@pytest.mark.parametrize("N", [1, 63, 64, 65, 257, 20011])
@pytest.mark.parametrize("pt_min", [20.0, 6000.0])
def test_totals_with_mostly_zero_weights(gpu_lib, n, prec, N, pt_min):
    c = gpu_lib.config(n, prec=prec, seed=99, pt_min=pt_min, tau_min=1e-4)
    print(f"totals n={n} prec={prec} N={N} pt_min={pt_min}", flush=True)
    r = gpu_lib.generate(c, N, outputs=("weight", "pass", "acc"))
    w, acc = r["weight"].cpu().numpy(), r["acc"].cpu().numpy()
    assert (w[r["pass"].cpu().numpy() == 0] == 0.0).all()
    if pt_min == 6000.0 and n > 4:   # three jets of 6 TeV exceed sqrt(S) = 14 TeV
        assert not w.any()
    # a TwoSum tree is within one rounding of the exact sum plus second-order terms
    for s, comp, x in ((acc[0], acc[1], w), (acc[2], acc[3], w * w)):
        exact = math.fsum(x.tolist())
        assert abs((s + comp) - exact) <= 4 * EPS * abs(exact)

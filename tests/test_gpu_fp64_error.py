"""The FP64 recursion's rounding against a plain evaluation of the printed formulas: the mean of the log
of the error ratio, GPU over the float64 oracle (both against the long-double oracle), over the events
of one class.  Bound: brackets summed as the formulas group them (two vectors) give 0.036, a sum in one
vector that ends with the span scalars' terms 0.087 (n = 8, either within 0.014); 0.06 lies between,
three times the spread of this many events from both."""
import numpy as np
import pytest

from tests.parity import oracle_amp2, popcount

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("count", [32000, 34000])   # two lanes per event, one
def test_error_of_the_plain_formulas(gpu_lib, count):
    n = 8
    print(f"fp64 error n={n} count={count}", flush=True)
    r = gpu_lib.generate(gpu_lib.config(n, prec=64, seed=81, use_pdf=0, sqrt_s=1000.0), count,
                         outputs=("momenta", "hel", "order"))
    got = gpu_lib.amp2(n, 64, r["momenta"], r["hel"], r["order"]).cpu().numpy()
    mom, order = r["momenta"].cpu().numpy(), r["order"].cpu().numpy()
    hel = r["hel"].cpu().numpy().astype(np.int64) & 0xFFFFFFFF
    pc = popcount(hel, n)
    live = (pc >= 2) & (pc <= n - 2)
    plain, exact = oracle_amp2(mom[live], hel[live], order[live])
    err = [np.maximum((np.abs(x - exact) / exact).astype(float), 1e-18) for x in (got[live], plain)]
    d = np.log(err[0] / err[1])
    assert len(d) > 25000
    assert d.mean() <= 0.06, (d.mean(), d.std() / np.sqrt(len(d)))

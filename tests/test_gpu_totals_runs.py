"""Totals of as many partials as fill one, some or all of the quarters of the one-launch reduction, and of
the first counts that take two launches: against the exact sum, alone and added to earlier totals."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("nparts", [1, 256, 257, 513, 1023, 1024, 1025, 1280, 2048])
def test_totals_against_the_exact_sum(gpu_lib, nparts):
    import math
    c = gpu_lib.config(4, prec=32, use_pdf=0, sqrt_s=1000.0, seed=17)
    print(f"totals of {nparts} partials", flush=True)
    r = gpu_lib.generate(c, 64 * nparts, outputs=("weight", "acc"))
    again = {"weight": torch.zeros_like(r["weight"]), "acc": r["acc"].clone()}
    gpu_lib.generate(c, 64 * nparts, outputs=("weight", "acc"), out_tensors=[again])   # totals are added to
    w, acc, twice = r["weight"].cpu().numpy(), r["acc"].cpu().numpy(), again["acc"].cpu().numpy()
    for s, x in ((0, w), (2, w * w)):
        exact = math.fsum(x.tolist())
        assert abs((acc[s] + acc[s + 1]) - exact) <= 4 * 2.0 ** -53 * exact
        assert abs((twice[s] + twice[s + 1]) - 2 * exact) <= 8 * 2.0 ** -53 * exact

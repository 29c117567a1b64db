"""Gradients of events whose ordering names a leg twice and leaves another out (not checked unless
BG_DEBUG): the absent leg's draws have derivative zero, the others are finite, and the well-formed events
around them keep their bits."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [4, 6, 8, 10])
def test_repeated_and_absent_legs(gpu_lib, n):
    N, bad = 130, [0, 31, 64, 129]
    c = gpu_lib.config(n, prec=64, seed=91, use_pdf=0, sqrt_s=1000.0)
    r = gpu_lib.generate(c, N, outputs=("uniforms", "x12", "hel", "order"))
    hel = torch.full_like(r["hel"], 0b0011)   # every event has |A|^2 > 0
    order = r["order"].clone()
    absent, twice = n - 1, 2
    legs = [0, 2, 1, 2] + list(range(3, n - 1))   # the two places apart: a pair of equal legs has K^2 = 0
    order[bad] = torch.tensor(legs, dtype=torch.uint8, device="cuda")
    print("gradients, malformed orders", n, flush=True)
    for prec in (64, 32):
        c = gpu_lib.config(n, prec=prec, seed=91, use_pdf=0, sqrt_s=1000.0)
        good = gpu_lib.amp2_grad(c, r["uniforms"], r["x12"], hel, r["order"])[0].cpu().numpy()
        got = gpu_lib.amp2_grad(c, r["uniforms"], r["x12"], hel, order)[0].cpu().numpy()
        keep = np.setdiff1d(np.arange(N), bad)
        assert np.array_equal(got[keep], good[keep])
        rows = got.reshape(N, n - 2, 4)[bad]
        assert not rows[:, absent - 2].any() and np.isfinite(rows).all()
        # n = 4: twice the same light-like momentum has no rest frame, the event is not finite: all zero
        assert rows[:, twice - 2].any(1).all() == (n > 4)

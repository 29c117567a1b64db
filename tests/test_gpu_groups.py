"""Two and four lanes per event: sizes around the 16 or 32 events of a wave give bitwise the events
of a larger call (the lanes past the end repeat the last event), an event that is not finite
leaves its neighbours in the wave alone, and the workgroup size changes nothing."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

OUT = ("weight", "amp2", "pass")
FORMS = [(6, 64, 2), (9, 64, 2), (10, 64, 2), (10, 64, 4), (11, 64, 4), (12, 64, 2), (12, 64, 4), (9, 32, 2), (12, 32, 2)]


@pytest.fixture
def form(gpu_lib, request):
    n, prec, lanes = request.param
    old = gpu_lib.get_lanes(n, prec), gpu_lib.get_launch(n, prec)
    gpu_lib.set_lanes(n, prec, lanes)
    yield n, prec, lanes
    gpu_lib.set_lanes(n, prec, old[0])
    gpu_lib.set_launch(n, prec, *old[1])


def host(r, keys=OUT):
    return {k: r[k].cpu().numpy() for k in keys}


@pytest.mark.parametrize("form", FORMS, indirect=True, ids=str)
def test_sizes_around_a_wave(gpu_lib, form):
    n, prec, lanes = form
    c = gpu_lib.config(n, prec=prec, use_pdf=0, sqrt_s=2000.0, seed=11)
    print("groups", form, flush=True)
    full = host(gpu_lib.generate(c, 197, outputs=OUT))
    r = gpu_lib.generate(c, 197, outputs=("momenta", "hel", "order"))
    ref = gpu_lib.amp2(n, prec, r["momenta"], r["hel"], r["order"]).cpu().numpy()
    for N in (1, 15, 16, 17, 31, 32, 33, 64, 65, 197):
        part = host(gpu_lib.generate(c, N, outputs=OUT))
        for k in OUT:
            assert np.array_equal(part[k], full[k][:N]), (N, k)
        got = gpu_lib.amp2(n, prec, r["momenta"][:N].contiguous(), r["hel"][:N].contiguous(), r["order"][:N].contiguous())
        assert np.array_equal(got.cpu().numpy(), ref[:N]), N
    for block in (64, 128, 256):
        gpu_lib.set_launch(n, prec, block, 1)
        again = host(gpu_lib.generate(c, 197, outputs=OUT))
        for k in OUT:
            assert np.array_equal(again[k], full[k]), (block, k)


@pytest.mark.parametrize("form", FORMS, indirect=True, ids=str)
def test_non_finite_event_stays_alone(gpu_lib, form):
    n, prec, lanes = form
    c = gpu_lib.config(n, prec=prec, use_pdf=0, sqrt_s=2000.0, seed=12)
    r = gpu_lib.generate(c, 96, outputs=("momenta", "hel", "order"))
    mom = r["momenta"]
    good = gpu_lib.amp2(n, prec, mom, r["hel"], r["order"]).cpu().numpy()
    bad = [0, 5, 17, 40, 95]
    mom[bad, 2] = torch.tensor([float("nan"), float("inf"), 1.0, -float("inf")], dtype=torch.float64, device="cuda")
    print("groups, events not finite", form, flush=True)
    got = gpu_lib.amp2(n, prec, mom, r["hel"], r["order"]).cpu().numpy()
    keep = np.setdiff1d(np.arange(96), bad)
    assert not np.isfinite(got[bad]).any() and np.array_equal(got[keep], good[keep])

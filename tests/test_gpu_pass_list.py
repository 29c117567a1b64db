"""Calls that ask for neither |A|^2 nor log w run the recursion on the events that pass the cuts only:
every output and the totals are bitwise those of a call that evaluates every event, at counts around
the first that takes the list, with ragged tails, none, few or all events passing, and past one
staging chunk."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

FEW, ALL = ("weight", "obs", "pass", "acc"), ("weight", "obs", "pass", "acc", "amp2")
# (n, precision, lanes, real polarisations, dynamic scale, first count that takes the list)
FORMS = [(7, 32, 1, 0, 0, 500000), (7, 32, 1, 1, 1, 500000), (8, 32, 1, 0, 1, 400000), (7, 64, 2, 0, 0, 166667),
         (8, 64, 2, 0, 0, 133334), (6, 64, 2, 0, 0, 212766), (9, 32, 2, 0, 0, 214286), (12, 32, 2, 0, 0, 65536),
         (9, 64, 2, 0, 1, 71429), (10, 64, 4, 0, 0, 37038)]


@pytest.fixture
def form(gpu_lib, request):
    n, prec, lanes = request.param[:3]
    if lanes > 1:
        old = gpu_lib.get_lanes(n, prec)
        gpu_lib.set_lanes(n, prec, lanes)
    yield request.param
    if lanes > 1:
        gpu_lib.set_lanes(n, prec, old)


def same(lib, c, N):
    got, ref = lib.generate(c, N, outputs=FEW), lib.generate(c, N, outputs=ALL)
    for k in FEW:
        assert np.array_equal(got[k].cpu().numpy(), ref[k].cpu().numpy()), (c.n, c.prec, N, k)
    return ref["pass"].cpu().numpy()


@pytest.mark.parametrize("form", FORMS, indirect=True, ids=str)
def test_list_gives_the_general_route(gpu_lib, form):
    n, prec, lanes, pol, dyn, first = form
    c = gpu_lib.config(n, prec=prec, seed=21, polarisation=pol, dynamic_scale=dyn)
    for N in (first - 1, first, first + 77):
        print("pass list", form, N, flush=True)
        p = same(gpu_lib, c, N)
        assert 0 < p.sum() < N


@pytest.mark.parametrize("n,prec", [(8, 32), (8, 64), (12, 32)])
def test_none_and_all_pass(gpu_lib, n, prec):
    N = 400005
    print("pass list, cuts", n, prec, flush=True)
    fixed = dict(prec=prec, seed=3, use_pdf=0, sqrt_s=3000.0)
    assert same(gpu_lib, gpu_lib.config(n, eta_max=1e-9, **fixed), N).sum() == 0
    loose = gpu_lib.config(n, pt_min=1e-9, eta_max=1e3, dr_min=0.0, **fixed)
    assert same(gpu_lib, loose, N).sum() == N


def test_past_one_chunk(gpu_lib):
    N = (1 << 22) + 1000
    print("pass list, two chunks", flush=True)
    p = same(gpu_lib, gpu_lib.config(7, prec=32, seed=5), N)
    assert p[1 << 22:].sum() > 0

"""Cuts and observables where the closest pair of jets and the |eta| cut are hard to decide:
tied pairs, |eta| within 1e-10 of the cut, jets along the beam.  The kernel ranks pairs in FP32
and evaluates the closest in FP64, so its decisions and R_min are compared with FP64 over all
pairs, formed here from the momenta the kernel returns."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu


def jets(mom):
    """(H_T, largest |eta|, R_min) of lab momenta [N, n, 4] over the outgoing legs."""
    p = mom[:, 2:]
    with np.errstate(divide="ignore", invalid="ignore"):
        pt = np.sqrt(p[..., 1] ** 2 + p[..., 2] ** 2)
        eta = np.copysign(np.log((p[..., 0] + np.abs(p[..., 3])) / pt), p[..., 3])
        phi = np.arctan2(p[..., 2], p[..., 1])
        i, j = np.triu_indices(p.shape[1], 1)
        dphi = np.abs(phi[:, i] - phi[:, j])
        dphi = np.where(dphi > np.pi, 2 * np.pi - dphi, dphi)
        d2 = (eta[:, i] - eta[:, j]) ** 2 + dphi ** 2
    return pt, eta, np.sqrt(np.nanmin(d2, axis=1))


def run(gpu_lib, n, prec, u, **kw):
    c = gpu_lib.config(n, prec=prec, use_pdf=0, sqrt_s=1000.0, seed=3, **kw)
    U = torch.tensor(u, device="cuda")
    r = gpu_lib.generate(c, len(u), inputs=dict(uniforms=U), outputs=("obs", "pass", "momenta"))
    return [r[k].cpu().numpy() for k in ("obs", "pass", "momenta")]


# three jets (all pairs in FP64), four (the first ranked form), 28 and 36 and 45 pairs (one and
# two words of pair flags); FP32 (split kernels) and FP64 (one kernel at n = 6)
SHAPES = [(5, 32), (6, 32), (6, 64), (8, 32), (10, 32), (11, 32), (12, 32)]


@pytest.mark.parametrize("n,prec", SHAPES)
def test_random_and_tied_pairs(gpu_lib, n, prec):
    rng = np.random.default_rng(n)
    N, nf = 2000 + 13, n - 2
    u = (rng.integers(0, 2 ** 32, (N, nf, 4)) + 0.5) * 2.0 ** -32
    # a ring: equal energies and polar angles, equal steps in azimuth (every neighbour ties)
    ring = slice(0, 500)
    u[ring, :, 0] = 0.5
    u[ring, :, 1] = (np.arange(nf)[None, :] / nf + u[ring, :1, 1]) % 1.0
    u[ring, :, 2:] = u[ring, :1, 2:]
    # near copies of one jet: several pairs at tiny distances
    close = slice(500, 1000)
    u[close, 1:3] = u[close, :1] + 1e-9 * rng.standard_normal((500, 2, 4))
    print(f"tied pairs n={n} prec={prec}", flush=True)
    obs, ok, mom = run(gpu_lib, n, prec, np.clip(u, 2.0 ** -33, 1 - 2.0 ** -33).reshape(N, -1))
    # all jets collinear (the near copies with three jets) is no phase-space point: M^2 is
    # rounding noise, and the momenta are not finite or not massless
    with np.errstate(invalid="ignore"):
        real = (np.abs(mom[..., 0] ** 2 - (mom[..., 1:] ** 2).sum(-1)) <= 1e-9 * mom[..., 0] ** 2).all(1)
    assert (n == 5 or real.all()) and real.sum() >= N - 500
    obs, ok, mom = obs[real], ok[real], mom[real]
    pt, eta, rmin = jets(mom)
    # eta and phi carry a few units of 2^-53 of at most 20; their differences no more
    assert np.all(np.abs(obs[:, 1] - rmin) <= 5e-14)
    assert np.all(np.abs(obs[:, 0] - pt.sum(1)) <= 1e-12 * pt.sum(1))
    want = (pt > 20).all(1) & (np.abs(eta) < 2.5).all(1) & (rmin > 0.4)
    sure = (np.abs(rmin - 0.4) > 1e-12) & (np.abs(pt - 20) > 1e-9).all(1) & (np.abs(np.abs(eta) - 2.5) > 1e-12).all(1)
    assert np.array_equal(ok[sure].astype(bool), want[sure]) and want.any() and sure.mean() > 0.99


@pytest.mark.parametrize("n,prec", SHAPES)
@pytest.mark.parametrize("delta", [1e-10, -1e-10, 1e-6, -1e-6])
def test_eta_cut_at_its_edge(gpu_lib, n, prec, delta):
    """The cut placed just above and just below one event's largest |eta|."""
    rng = np.random.default_rng(100 + n)
    u = ((rng.integers(0, 2 ** 32, (64, n - 2, 4)) + 0.5) * 2.0 ** -32).reshape(64, -1)
    print(f"eta edge n={n} prec={prec} delta={delta}", flush=True)
    _, eta, _ = jets(run(gpu_lib, n, prec, u)[2])
    top = np.abs(eta).max(1)
    for k in range(4):
        _, ok, _ = run(gpu_lib, n, prec, u, eta_max=float(top[k]) * (1 + delta), pt_min=0.0, dr_min=0.0)
        assert np.array_equal(ok.astype(bool), top < top[k] * (1 + delta)) and bool(ok[k]) == (delta > 0)


@pytest.mark.parametrize("n,prec", [(6, 32), (8, 32), (12, 32)])
def test_jets_along_the_beam(gpu_lib, n, prec):
    """|eta| beyond FP32's range of use, and a jet with pT = 0 in the RAMBO frame."""
    rng = np.random.default_rng(7 + n)
    N, nf = 300, n - 2
    u = (rng.integers(0, 2 ** 32, (N, nf, 4)) + 0.5) * 2.0 ** -32
    u[:100, 0, 0] = 1e-15
    u[100:200, 0, 0] = 1 - 2.0 ** -53
    u[200:, 0, 0] = 2.0 ** -60       # c rounds to -1
    # the others in pairs back to back across the beam, so that the boost keeps jet 0 on it
    for p in range(1, nf - 1, 2):
        u[:, p + 1] = u[:, p]
        u[:, p + 1, 1] = (u[:, p, 1] + 0.5) % 1.0
    print(f"beam jets n={n} prec={prec}", flush=True)
    obs, ok, mom = run(gpu_lib, n, prec, u.reshape(N, -1))
    pt, eta, rmin = jets(mom)
    far = np.isfinite(rmin) & (np.abs(eta).max(1) < 40)
    assert far.sum() > 100 and np.all(np.abs(obs[far, 1] - rmin[far]) <= 1e-13)
    assert not ok[np.abs(eta).max(1) > 3].any()

"""The gradient's adjoints beyond the recursion, checked on the CPU: the library's header compiled for
the host against long-double values of the same derivatives.  Their rms error is at most 1.05 of
that of the derivative's plain expression in float64 (both round each operation to nearest; 1.05
leaves room for the order of one or two operations)."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LD = np.longdouble
PI = LD("3.14159265358979323846264338327950288")


@pytest.fixture(scope="module")
def adjoints(tmp_path_factory):
    """run(tag, rows): the driver's output for each row of arguments."""
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("adjointcheck") / "adjoint_check")
    subprocess.run([HIPCC, "-O2", "--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", os.path.join(HERE, "native", "adjoint_check.hip"), "-o", exe],
                   check=True, capture_output=True)

    def run(tag, rows):
        inp = "\n".join(tag + " " + " ".join(float(x).hex() for x in r) for r in rows) + "\n"
        out = subprocess.run([exe], input=inp, check=True, capture_output=True, text=True).stdout.splitlines()
        return np.array([[float.fromhex(v) for v in l.split()] for l in out])
    return run


def rms(got, exact):
    """Per column, over its rms value."""
    return np.sqrt(((got - exact) ** 2).sum(0) / (exact ** 2).sum(0)).astype(float)


def q_adj(r, qb, t):
    """d(q . qb) of q = q0 (1, st cos phi, st sin phi, c) in the four draws, component by component."""
    r1, r2, r3, r4 = r.astype(t).T
    b0, b1, b2, b3 = qb.astype(t).T
    pi = PI if t is LD else np.float64(PI)
    c = 2 * r1 - 1
    st, phi, q0 = np.sqrt(1 - c * c), 2 * pi * r2, -np.log(r3 * r4)
    across = b1 * np.cos(phi) + b2 * np.sin(phi)
    b = b0 + b1 * st * np.cos(phi) + b2 * st * np.sin(phi) + b3 * c
    return np.stack([2 * (q0 * b3 - q0 * across * c / st), 2 * pi * q0 * st * (np.cos(phi) * b2 - np.sin(phi) * b1),
                     -b / r3, -b / r4], -1)


def test_rambo_q_adj(adjoints):
    rng = np.random.default_rng(5)
    r, qb = rng.random((40000, 4)), rng.normal(size=(40000, 4))
    r[:, 0] = 0.02 + 0.96 * r[:, 0]   # near the poles the angle's own rounding decides
    exact = q_adj(r, qb, LD)
    got, plain = rms(adjoints("Q", np.concatenate([r, qb], 1)), exact), rms(q_adj(r, qb, np.float64), exact)
    assert (got <= 1.05 * plain).all(), (got, plain)


def test_rambo_q_adj_at_the_edges(adjoints):
    """r1 = 0 and 1: the derivative in r1 is infinite, the others are finite; r3 = r4 = 1: q = 0, all
    are finite."""
    qb = [0.3, -1.1, 0.7, 0.4]
    rows = [[r1, 0.2, 0.3, 0.4] + qb for r1 in (0.0, 1.0)] + [[0.3, 0.2, 1.0, 1.0] + qb, [0.0, 0.2, 1.0, 1.0] + qb]
    got = adjoints("Q", rows)
    across = qb[1] * np.cos(0.4 * np.pi) + qb[2] * np.sin(0.4 * np.pi)
    assert np.isinf(got[:2, 0]).all() and (np.sign(got[:2, 0]) == np.sign(across) * np.array([1, -1])).all(), got
    assert np.isfinite(got[:3, 1:]).all() and np.isfinite(got[2]).all(), got
    want = [-(qb[0] + c * qb[3]) / 0.3 for c in (-1.0, 1.0)]
    assert np.allclose(got[:2, 2], want, rtol=1e-15, atol=0)


def source_adj(p, h, er, ei, t):
    """d(Re e . er + Im e . ei) of the helicity source e(p) in px, py, pz: the derivatives of the polar
    and azimuthal cosines and sines, each a quotient of products."""
    px, py, pz = p.astype(t).T
    e1, e2, e3 = er.astype(t).T
    i1, i2 = ei.astype(t).T
    r, h = np.sqrt(t(0.5)), h.astype(t)
    pt2 = px * px + py * py
    pa, pt = np.sqrt(pt2 + pz * pz), np.sqrt(pt2)
    ct, cf, sf = pz / pa, px / pt, py / pt
    ctb, stb = -h * r * (cf * e1 + sf * e2), h * r * e3
    cfb, sfb = -h * r * ct * e1 - r * i2, r * i1 - h * r * ct * e2
    pa3, pt3 = pa * pa * pa, pt2 * pt
    return np.stack([ctb * (-pz * px / pa3) + stb * (px * pz * pz / (pt * pa3)) + cfb * (py * py / pt3) + sfb * (-px * py / pt3),
                     ctb * (-pz * py / pa3) + stb * (py * pz * pz / (pt * pa3)) + cfb * (-px * py / pt3) + sfb * (px * px / pt3),
                     ctb * (pt2 / pa3) + stb * (-pt * pz / pa3)], -1)


def test_polarisation_adj(adjoints):
    rng = np.random.default_rng(6)
    p = rng.normal(size=(40000, 3)) * 100.0
    h, er, ei = rng.choice([-1.0, 1.0], 40000), rng.normal(size=(40000, 3)), rng.normal(size=(40000, 2))
    size = np.hypot(p[:, 0], p[:, 1])[:, None]   # the derivative falls as 1 / pT
    exact = source_adj(p, h, er, ei, LD) * size
    got = rms(adjoints("P", np.concatenate([p, h[:, None], er, ei], 1)) * size, exact)
    plain = rms(source_adj(p, h, er, ei, np.float64) * size, exact)
    assert (got <= 1.05 * plain).all(), (got, plain)


def init_adj(Q, rs, A, t):
    """Adjoint of b = -Q / M, gamma = Q0 / M, a = 1 / (1 + gamma), X = sqrt(s) / M in Q and sqrt(s)."""
    Q, rs, A = Q.astype(t), rs.astype(t), A.astype(t)
    bb, gb, ab, Xb = A[:, :3], A[:, 3], A[:, 4], A[:, 5]
    M = np.sqrt(Q[:, 0] ** 2 - Q[:, 1] ** 2 - Q[:, 2] ** 2 - Q[:, 3] ** 2)
    b, g, X = -Q[:, 1:] / M[:, None], Q[:, 0] / M, rs / M
    gb = gb - ab / ((1 + g) * (1 + g))
    Mb = -Xb * X / M - gb * g / M - (bb * b / M[:, None]).sum(1)
    m2 = Mb / (2 * M)
    return np.concatenate([(gb / M + 2 * Q[:, 0] * m2)[:, None], -bb / M[:, None] - 2 * Q[:, 1:] * m2[:, None],
                           (Xb / M)[:, None]], 1)


def test_rambo_init_adj(adjoints):
    rng = np.random.default_rng(7)
    q = rng.normal(size=(40000, 6, 3)) * rng.exponential(2.0, (40000, 6, 1))
    Q = np.concatenate([np.sqrt((q * q).sum(-1)).sum(1)[:, None], q.sum(1)], 1)
    rs, A = rng.uniform(200.0, 5000.0, 40000), rng.normal(size=(40000, 6))
    exact = init_adj(Q, rs, A, LD)
    got = rms(adjoints("I", np.concatenate([Q, rs[:, None], A], 1)), exact)
    plain = rms(init_adj(Q, rs, A, np.float64), exact)
    assert (got <= 1.05 * plain).all(), (got, plain)

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

"""The FP64 helicity sources, checked on the CPU: the library's header compiled for the host against
long-double values.  No word's rms error is larger than with correctly rounded square roots and
quotients (numpy's float64), but for 2%, the spread of the two over this many momenta."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
LD = np.longdouble


@pytest.fixture(scope="module")
def samples(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("sourcecheck") / "source_check")
    subprocess.run([HIPCC, "-O2", "--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", os.path.join(HERE, "native", "source_check.hip"), "-o", exe],
                   check=True, capture_output=True)
    out = subprocess.run([exe], check=True, capture_output=True, text=True).stdout.splitlines()
    return np.array([[float(l.split()[0])] + [float.fromhex(v) for v in l.split()[1:]] for l in out])


def words(plus, p, t):
    """re[1], im[1], re[2], im[2], re[3] of the sources, each operation rounded to the type t."""
    px, py, pz = p.astype(t).T
    pt2 = px * px + py * py
    beam = pt2 == 0
    pt, ipa = np.sqrt(pt2), 1 / np.sqrt(pt2 + pz * pz)
    ipt = 1 / np.where(beam, t(1), pt)
    ct, st = pz * ipa, pt * ipa
    cf, sf = np.where(beam, t(1), px * ipt), np.where(beam, t(0), py * ipt)
    r = np.sqrt(t(0.5))
    h = np.where(plus == 1, r, -r)
    return np.stack([-h * ct * cf, sf * r, -h * ct * sf, -cf * r, h * st], -1)


def test_sources_are_as_accurate_as_rounded_quotients(samples):
    plus, p, got = samples[:, 0], samples[:, 1:4], samples[:, 4:].reshape(-1, 4, 2)
    assert not got[:, 0].any() and not got[:, 3, 1].any()
    got = np.stack([got[:, 1, 0], got[:, 1, 1], got[:, 2, 0], got[:, 2, 1], got[:, 3, 0]], -1)
    exact, plain = words(plus, p, LD), words(plus, p, np.float64)
    beam = (p[:, 0] == 0) & (p[:, 1] == 0)
    assert beam.sum() == 400 and np.abs(got[beam] - exact[beam]).max() <= 2.0 ** -52
    rms = lambda x: np.sqrt(((x - exact) ** 2).mean(0) / (exact ** 2).mean(0)).astype(float)  # noqa: E731
    assert (rms(got) <= 1.02 * rms(plain)).all(), (rms(got), rms(plain))

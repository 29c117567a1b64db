"""The FP32 decision of the |eta| cut, checked on the CPU (the library's header compiled for the host): it
agrees with FP64 wherever it decides, leaves only values within its error of the cut undecided, and
decides every jet when there is no cut."""
import os
import shutil
import subprocess

import numpy as np
import pytest

HERE = os.path.dirname(os.path.abspath(__file__))
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")
ANGLE_ERR = 4e-6   # error of the FP32 pseudorapidities


@pytest.fixture(scope="module")
def side(tmp_path_factory):
    if not (os.path.exists(HIPCC) or shutil.which(HIPCC)):
        pytest.skip("hipcc not available")
    exe = str(tmp_path_factory.mktemp("cutscheck") / "cuts_check")
    subprocess.run([HIPCC, "-O2", "--offload-arch=gfx950", "-std=c++17", "-Xclang", "-target-feature", "-Xclang",
                    "-packed-fp32-ops", os.path.join(HERE, "native", "cuts_check.hip"), "-o", exe],
                   check=True, capture_output=True)

    def run(pairs):
        inp = "\n".join(f"{e!r} {m!r}" for e, m in pairs) + "\n"
        out = subprocess.run([exe], input=inp, check=True, capture_output=True, text=True).stdout.split()
        return np.array(out, dtype=int).reshape(-1, 2)
    return run


def test_decisions(side):
    rng = np.random.default_rng(9)
    pairs = []
    for m in (1e-9, 0.5, 2.5, 5.0, 20.0):
        for d in np.concatenate([rng.normal(size=200), rng.normal(size=200) * 3e-5, [0.0]]):
            pairs.append((float(np.float32(abs(m + d))), m))
    got = side(pairs)
    e, m = np.array(pairs).T
    assert (got[:, 0] == got[:, 1]).all()
    fails, passes = got[:, 0] == 1, got[:, 0] == -1
    assert (e[fails] > m[fails] + ANGLE_ERR).all() and (e[passes] < m[passes] - ANGLE_ERR).all()
    assert (np.abs(e - m)[got[:, 0] == 0] <= 2 * ANGLE_ERR + 4e-6 * np.maximum(m, 1.0)[got[:, 0] == 0]).all()


@pytest.mark.parametrize("no_cut", [float("inf"), 1e300, 1e35, 1e31])
def test_no_cut_decides_every_jet(side, no_cut):
    assert (side([(e, no_cut) for e in (0.0, 1e-3, 1.0, 20.0, 130.0)]) == -1).all()


def test_undecided(side):
    nan = float("nan")
    assert (side([(nan, 2.5), (1.0, nan), (nan, nan), (nan, float("inf"))]) == 0).all()

"""The one-lane kernels of n <= 8: one kernel up to n = 6, kinematics and recursion kernels at n = 7,
8, FP64 with leg momenta and span scalars in LDS.  Sizes around one workgroup of 64 events give
bitwise the events of a larger call, with and without the library's own workspace (values against
the oracle: test_gpu_amp2.py, test_gpu_generate.py, test_gpu_realpol.py)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

OUT = ("weight", "amp2", "obs", "pass", "logw", "hel", "order")


def host(r):
    return {k: r[k].cpu().numpy() for k in OUT}


@pytest.mark.parametrize("n,prec,pol", [(n, p, 0) for n in range(4, 9) for p in (32, 64)] +
                         [(4, 32, 1), (6, 32, 1), (7, 32, 1), (8, 32, 1), (6, 64, 1)])
def test_sizes_around_a_workgroup(gpu_lib, n, prec, pol):
    c = gpu_lib.config(n, prec=prec, use_pdf=0, sqrt_s=1000.0, seed=5, polarisation=pol)
    print(f"one-lane n={n} prec={prec} pol={pol}", flush=True)
    full = host(gpu_lib.generate(c, 261, outputs=OUT))
    assert full["pass"].any()
    for N in (1, 63, 64, 65, 128, 261):
        part = host(gpu_lib.generate(c, N, outputs=OUT))
        ws = gpu_lib.generate(c, N, outputs=OUT)
        for t in ws.values():
            t.zero_()
        alloc_free = host(gpu_lib.generate_noalloc(c, N, ws))
        for k in OUT:
            assert np.array_equal(part[k], full[k][:N], equal_nan=True), (N, k)
            assert np.array_equal(alloc_free[k], part[k], equal_nan=True), (N, k)


def test_fp64_lane_setting(gpu_lib):
    """n = 7, 8: the setting 2 alone, as before the one-lane kernels took its place."""
    for n in (7, 8):
        assert gpu_lib.get_lanes(n, 64) == 2
        gpu_lib.set_lanes(n, 64, 2)
        for bad in (1, 4):
            with pytest.raises(gpu_lib.BgError) as e:
                gpu_lib.set_lanes(n, 64, bad)
            assert e.value.status == gpu_lib.BG_ENOTSUP

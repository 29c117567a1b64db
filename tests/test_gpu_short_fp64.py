"""FP64 n = 7, 8: short calls take two lanes per event, longer ones one; both give the same bits."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
OUT = ("weight", "amp2", "logw", "pass", "acc")
PAIRS = 1 << 15   # the largest call with two lanes


@pytest.mark.parametrize("n", [7, 8])
def test_same_bits_either_side(gpu_lib, n):
    c = gpu_lib.config(n, prec=64, seed=9)
    print("short fp64", n, flush=True)
    full = {k: v.cpu().numpy() for k, v in gpu_lib.generate(c, PAIRS + 1, outputs=OUT).items()}
    r = gpu_lib.generate(c, PAIRS + 1, outputs=("momenta", "hel", "order"))
    ref = gpu_lib.amp2(n, 64, r["momenta"], r["hel"], r["order"]).cpu().numpy()
    for N in (1, 31, 33, 1000, PAIRS):
        part = gpu_lib.generate(c, N, outputs=OUT)
        for k in OUT[:4]:
            assert np.array_equal(part[k].cpu().numpy(), full[k][:N], equal_nan=True), (N, k)
        got = gpu_lib.amp2(n, 64, r["momenta"][:N].contiguous(), r["hel"][:N].contiguous(), r["order"][:N].contiguous())
        assert np.array_equal(got.cpu().numpy(), ref[:N]), N
    s = full["weight"][:PAIRS].sum()
    acc = part["acc"].cpu().numpy()
    assert abs(acc[0] + acc[1] - s) <= PAIRS * 2.0 ** -52 * np.abs(full["weight"]).max()

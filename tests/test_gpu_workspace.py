"""The small workspaces kept between calls: calls on several streams and threads at once, growing
and shrinking calls on one stream, and calls under graph capture give the results of calls made
one at a time."""
import threading

import pytest
import torch

pytestmark = pytest.mark.gpu

OUT = ("weight", "amp2", "acc")


def call(lib, n, prec, N, seed):
    return lib.generate(lib.config(n, prec=prec, seed=seed, use_pdf=0, sqrt_s=1000.0), N, outputs=OUT)


def same(a, b):
    return all(torch.equal(a[k], b[k]) for k in OUT)


# one kernel, two kernels (staged), two lanes per event
SHAPES = [(5, 64, 700), (8, 32, 900), (8, 64, 300), (10, 32, 200)]


def test_streams_and_threads(gpu_lib):
    want = {(i, r): call(gpu_lib, *SHAPES[r % 4], 10 * i + r) for i in range(4) for r in range(12)}
    torch.cuda.synchronize()
    print("workspace: 4 threads, 3 streams each", flush=True)
    got, errors = {}, []

    def work(i):
        try:
            streams = [torch.cuda.Stream() for _ in range(3)]
            for r in range(12):
                with torch.cuda.stream(streams[r % 3]):
                    got[i, r] = call(gpu_lib, *SHAPES[r % 4], 10 * i + r)
            for s in streams:
                s.synchronize()
        except Exception as e:   # shown by the assertion below
            errors.append(e)

    ts = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in ts:
        t.start()
    for t in ts:
        t.join()
    torch.cuda.synchronize()
    assert not errors and all(same(got[k], want[k]) for k in want)


def test_growing_and_shrinking_calls(gpu_lib):
    sizes = [1, 5000, 64, 70000, 300, 20000, 2, 70000]
    print("workspace: sizes", sizes, flush=True)
    got = [call(gpu_lib, 8, 32, N, 7) for N in sizes]
    torch.cuda.synchronize()
    full = got[3]
    for N, g in zip(sizes, got):
        assert torch.equal(g["amp2"], full["amp2"][:N]) and torch.equal(g["weight"], full["weight"][:N])
    assert torch.equal(got[3]["acc"], got[7]["acc"])


@pytest.mark.parametrize("nparts", [1, 255, 256, 257, 1024, 4095, 4096, 4097])
def test_totals_of_one_and_two_launches(gpu_lib, nparts):
    """Totals over up to 4096 partials come from one launch: against the exact sum."""
    import math
    c = gpu_lib.config(4, prec=32, use_pdf=0, sqrt_s=1000.0, seed=3)
    print(f"totals over {nparts} partials", flush=True)
    r = gpu_lib.generate(c, 64 * nparts - 5, outputs=("weight", "acc"))
    w, acc = r["weight"].cpu().numpy(), r["acc"].cpu().numpy()
    assert (w != 0).mean() > 0.5
    for s, comp, x in ((acc[0], acc[1], w), (acc[2], acc[3], w * w)):
        exact = math.fsum(x.tolist())
        assert abs((s + comp) - exact) <= 4 * 2.0 ** -53 * exact

"""Calls under graph capture (no workspace is kept for a capturing stream): replays, with eager calls of
other sizes and synchronisations between them, give the eager result each time."""
import pytest
import torch

pytestmark = pytest.mark.gpu

OUT = ("weight", "amp2", "obs", "pass", "acc")


def captured(fn):
    """fn recorded once (after a warm-up on a side stream, as torch asks for)."""
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        fn()
    torch.cuda.current_stream().wait_stream(s)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        fn()
    return g


def eager_between(lib):
    lib.generate(lib.config(8, prec=32, seed=9, use_pdf=0, sqrt_s=1000.0), 3000, outputs=("weight", "acc"))
    lib.generate(lib.config(5, prec=64, seed=9, use_pdf=0, sqrt_s=1000.0), 70000, outputs=("weight", "acc"))
    torch.cuda.synchronize()


# one kernel, two kernels, lane pairs, four lanes
@pytest.mark.parametrize("n,prec,N", [(5, 64, 700), (8, 32, 5000), (8, 64, 300), (10, 32, 2000), (12, 64, 300)])
@pytest.mark.parametrize("entry", ["generate", "generate_noalloc"])
def test_generate(gpu_lib, entry, n, prec, N):
    c = gpu_lib.config(n, prec=prec, seed=n, use_pdf=0, sqrt_s=1000.0)
    want = gpu_lib.generate(c, N, outputs=OUT)
    out = {k: torch.zeros_like(v) for k, v in want.items()}
    call = {"generate": lambda: gpu_lib.generate(c, N, outputs=OUT, out_tensors=[out]),
            "generate_noalloc": lambda: gpu_lib.generate_noalloc(c, N, out)}[entry]
    print("capture", entry, n, prec, N, flush=True)
    g = captured(call)
    for _ in range(4):
        for v in out.values():
            v.zero_()
        g.replay()
        torch.cuda.synchronize()
        for k in OUT:
            assert torch.equal(out[k], want[k]), k
        eager_between(gpu_lib)


@pytest.mark.parametrize("n,prec,N", [(6, 64, 500), (8, 32, 900)])
def test_matrix_elements_and_gradients(gpu_lib, n, prec, N):
    c = gpu_lib.config(n, prec=prec, seed=n, use_pdf=0, sqrt_s=1000.0)
    r = gpu_lib.generate(c, N, outputs=("momenta", "uniforms", "x12", "hel", "order"))
    res = {}

    def call():
        res["a"] = gpu_lib.amp2(n, prec, r["momenta"], r["hel"], r["order"])
        res["g"] = gpu_lib.amp2_grad(c, r["uniforms"], r["x12"], r["hel"], r["order"])
    call()
    want = [res["a"].clone()] + [t.clone() for t in res["g"]]
    print("capture, given points", n, prec, N, flush=True)
    g = captured(call)
    for _ in range(3):
        for t in (res["a"], *res["g"]):
            t.zero_()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip((res["a"], *res["g"]), want))
        eager_between(gpu_lib)

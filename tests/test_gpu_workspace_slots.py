"""Kept workspaces where they run out: more streams at once than there are slots, and a stream that comes
after the slots' streams have fallen silent."""
import pytest
import torch

pytestmark = pytest.mark.gpu

OUT = ("weight", "amp2", "acc")


def call(lib, seed, N=900):
    return lib.generate(lib.config(8, prec=32, seed=seed, use_pdf=0, sqrt_s=1000.0), N, outputs=OUT)


def same(a, b):
    return all(torch.equal(a[k], b[k]) for k in OUT)


def on(stream, fn):
    with torch.cuda.stream(stream):
        return fn()


def test_more_streams_than_slots(gpu_lib):
    want = [call(gpu_lib, s) for s in range(14)]
    torch.cuda.synchronize()
    print("workspace: 14 streams", flush=True)
    streams = [torch.cuda.Stream() for _ in range(14)]
    for _ in range(3):
        got = [on(s, lambda k=k: call(gpu_lib, k)) for k, s in enumerate(streams)]
        torch.cuda.synchronize()
        assert all(same(a, b) for a, b in zip(got, want))


def test_slot_of_a_silent_stream(gpu_lib):
    """4200 calls of one stream make every other slot a stale one; then nine new streams take them."""
    want = [call(gpu_lib, s, 300) for s in range(10)]
    torch.cuda.synchronize()
    print("workspace: 4200 calls, then new streams", flush=True)
    busy, out = torch.cuda.Stream(), call(gpu_lib, 0, 300)
    torch.cuda.synchronize()
    c = gpu_lib.config(8, prec=32, seed=0, use_pdf=0, sqrt_s=1000.0)
    with torch.cuda.stream(busy):
        for _ in range(4200):
            gpu_lib.generate(c, 300, outputs=("weight", "amp2"), out_tensors=[out])
    streams = [torch.cuda.Stream() for _ in range(9)]
    got = [on(s, lambda k=k: call(gpu_lib, k, 300)) for k, s in enumerate(streams)]
    torch.cuda.synchronize()
    assert all(same(a, b) for a, b in zip(got, want)) and torch.equal(out["weight"], want[0]["weight"])

"""First calls of the time-last kernels from several threads at once, each on a
stream of its own: what a kernel's launcher keeps (how many of its waves fit) is
shared by them.  Orders that no other test uses; every thread's results are those
of a later call.
"""
import threading

import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2501_14490_amd import mfpsn  # noqa: E402  (loads libmfpsn.so or raises)

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dtype,k", [("f32", 27), ("bf16", 21), ("q8_8", 13)])
def test_first_calls_from_several_threads(dtype, k):
    g = torch.Generator().manual_seed(k)
    T, N, C = 130, 3, 5
    desc = mfpsn.make_desc((T, N, C), k, 2, dtype, v_th=0.5, v_th_q=128)
    x, gs = (torch.randn(N, C, T, generator=g) for _ in range(2))
    if dtype == "q8_8":
        x, gs = ((v * 256).round().to(torch.int16) for v in (x, gs))
    x, gs = (v.to(mfpsn.STORAGE[desc.dtype]).to(DEV) for v in (x, gs))
    sign = (torch.randint(0, 2, (C, k), generator=g) * 2 - 1).to(torch.int8).to(DEV)
    shift = torch.randint(0, 8, (C, k), generator=g).to(torch.int8).to(DEV)
    bias = torch.zeros(C, dtype=mfpsn.BIAS[desc.dtype], device=DEV)
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(8)]
    got, go = [None] * len(streams), threading.Barrier(len(streams))

    def call(i):
        with torch.cuda.stream(streams[i]):
            go.wait(timeout=30)
            spikes = mfpsn.forward_time_last(desc, x, sign, shift, bias)
            got[i] = (spikes, *mfpsn.backward_time_last(desc, x, gs, sign, shift, bias))

    threads = [threading.Thread(target=call, args=(i,)) for i in range(len(streams))]
    for t in threads:
        t.start()
    for t in threads:
        t.join(timeout=60)
    torch.cuda.synchronize()
    want = (mfpsn.forward_time_last(desc, x, sign, shift, bias),
            *mfpsn.backward_time_last(desc, x, gs, sign, shift, bias))
    for out in got:
        assert out is not None and all(torch.equal(a, b) for a, b in zip(out, want))

"""MfPSNFunction around the orders where its backward stops recomputing the
surrogate factor and reads a saved one: gradients are those of the backward fed
with the saved factor, bit for bit, on both sides of the limit.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2501_14490_amd import mfpsn  # noqa: E402  (loads libmfpsn.so or raises)

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("shape", [(37, 3, 70), (29, 2, 5, 6), (23, 2, 5, 7)])
@pytest.mark.parametrize("dtype,k", [("f32", 1), ("f32", 16), ("f32", 17), ("bf16", 12), ("bf16", 13)])
def test_gradients_are_those_of_the_saved_factor(dtype, k, shape):
    g = torch.Generator().manual_seed(11)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    x, up = (torch.randn(shape, generator=g).to(tdt).to(DEV) for _ in range(2))
    C = shape[2]
    w = torch.randn(C, k, generator=g).to(DEV)
    b = (torch.randn(C, generator=g) * 0.1).to(DEV)
    leaves = [t.clone().requires_grad_() for t in (x, w, b)]
    spikes = mfpsn.MfPSNFunction.apply(*leaves, k, 2, 0.5, "atan", 2.0, 0, 7)
    got = torch.autograd.grad(spikes, leaves, up)
    desc = mfpsn.make_desc(shape, k, 2, dtype, "atan", 2.0, 0.5, 128, 0, 7)
    sign, shift = mfpsn.quantize(w, 0, 7)
    want_spikes, sg = mfpsn.forward(desc, x, sign, shift, b, want_sg=True)
    assert 0 < int(want_spikes.sum()) < want_spikes.numel()
    assert torch.equal(spikes.detach(), want_spikes.to(tdt))
    for have, want in zip(got, mfpsn.backward(desc, x, up, sign, shift, b, sg=sg)):
        assert torch.equal(have.reshape(want.shape), want)

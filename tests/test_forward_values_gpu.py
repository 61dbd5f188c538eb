"""mfpsn_forward_values on the GPU: the spikes it writes in the storage type are
what mfpsn_spikes_to_input makes of mfpsn_forward's bytes, and H and the
surrogate factor are mfpsn_forward's, bit for bit, in every lane mapping:
lane-channel, plane with one and two columns per lane, the flat mapping with
16- and 8-byte accesses, and tensors off the wide accesses' alignment.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2501_14490_amd import mfpsn  # noqa: E402  (loads libmfpsn.so or raises)

DEV = torch.device("cuda:0")


@pytest.mark.parametrize("dtype", ["f32", "bf16", "q8_8"])
@pytest.mark.parametrize("offset", [0, 1])
@pytest.mark.parametrize("shape,k,d", [
    ((19, 3, 130), 4, 2),         # lane-channel, a ragged channel group
    ((9, 2, 5, 7), 3, 1),         # plane, odd row
    ((13, 3, 3, 6), 5, 3),        # plane, two columns per lane
    ((33, 3, 9, 4, 4), 8, 2),     # flat, 16-byte accesses, a ragged last tile
    ((21, 2, 9, 4), 16, 1),       # flat, 8-byte accesses
    ((40, 2, 3, 8), 20, 1),       # plane, an order without two-column kernels
])
def test_values_are_the_spikes_in_the_storage_type(shape, k, d, offset, dtype):
    g = torch.Generator().manual_seed(7)
    desc = mfpsn.make_desc(shape, k, d, dtype, v_th=0.5, v_th_q=128)
    T, C, n = shape[0], shape[2], 1
    for v in shape:
        n *= v
    x = torch.randn(n, generator=g)
    x = (x * 256).round().to(torch.int16) if dtype == "q8_8" else x.to(mfpsn.STORAGE[desc.dtype])
    x = x.reshape(shape).to(DEV)
    sign = (torch.randint(0, 2, (C, k), generator=g) * 2 - 1).to(torch.int8).to(DEV)
    shift = torch.randint(0, 8, (C, k), generator=g).to(torch.int8).to(DEV)
    bias = torch.randn(C, generator=g) * 0.1
    bias = ((bias * 256).round().to(torch.int32) if dtype == "q8_8" else bias).to(DEV)
    spikes, h, sg = mfpsn.forward(desc, x, sign, shift, bias, want_h=True, want_sg=True)
    want = mfpsn.spikes_to_input(spikes, dtype)
    assert 0 < int(spikes.sum()) < n
    out = torch.full((n + offset + 8,), -1, dtype=x.dtype, device=DEV)
    h2, sg2 = torch.empty_like(h), torch.empty_like(sg)
    mfpsn.mfpsn_forward_values(desc, x, sign, shift, bias, None, out[offset:], h2, sg2)
    assert torch.equal(out[offset:offset + n].reshape(shape), want)
    assert bool((out[:offset] == -1).all()) and bool((out[offset + n:] == -1).all())
    assert torch.equal(h2.view(torch.int32), h.view(torch.int32))
    assert torch.equal(sg2.view(torch.int32), sg.view(torch.int32))
    assert torch.equal(mfpsn.forward(desc, x, sign, shift, bias, values=True), want)

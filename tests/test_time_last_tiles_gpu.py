"""Edges of the time-last tiles on the GPU (csrc/mfpsn_tl_tile.hip): the results
are those of the time-first entry points with the time axis moved last, bit
for bit for spikes, H and grad_x.  grad_w and grad_b are sums of exact
products in double rounded once to float (int64 for Q8.8): the two layouts add
them in different orders, so they agree to 1e-6 absolute + 1e-5 relative, the
bar of the other gradient tests, and exactly for Q8.8.

Shapes: padded rows (whole pieces, half pieces), odd tensors, one column per
tile with many chunks, rows of several channels cut by a tile, ragged blocks
of a row, more classes than lanes, dilations past the end (in the 20 KB of a
usual tile and above them), two and three segments with a ragged tail, tensors
1, 2 and 4 elements off 16-byte alignment, and the columns that go to a lane each.
"""
import pytest

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
if not torch.cuda.is_available():
    pytest.skip("no GPU", allow_module_level=True)

from paper_2501_14490_amd import mfpsn  # noqa: E402  (loads libmfpsn.so or raises)

DEV = torch.device("cuda:0")


def place(t, offset):
    """A contiguous copy of t that starts `offset` elements into a buffer."""
    buf = torch.empty(t.numel() + offset, dtype=t.dtype, device=DEV)
    view = buf[offset:].view(t.shape)
    view.copy_(t)
    return view


@pytest.mark.parametrize("dtype", ["f32", "bf16", "q8_8"])
@pytest.mark.parametrize("offset", [0, 1, 2, 4])
@pytest.mark.parametrize("T,N,C,S,k,d,lo", [
    (48, 3, 5, 9, 4, 1, 0),       # padded rows, ragged blocks of a row
    (20, 5, 7, 3, 3, 2, 0),       # half pieces (16-bit), channels cut by tiles
    (33, 3, 11, 1, 2, 1, 0),      # odd rows, several channels per tile
    (100, 2, 3, 5, 12, 7, -2),    # negative shifts
    (601, 1, 3, 1, 16, 1, 0),     # one column per tile, 64 chunks
    (150, 2, 3, 2, 2, 100, 0),    # more classes than lanes
    (70, 1, 4, 3, 4, 300, 0),     # dilation past the end
    (4100, 1, 2, 1, 4, 3, 0),     # segments, ragged tail
    (2000, 2, 3, 1, 8, 1, 0),     # few columns: short segments
    (5003, 1, 1, 2, 2, 1000, 0),  # long history between segments, more classes than lanes
    (2, 3, 70, 1, 32, 1, 0),      # two steps, the highest order
    (900, 2, 3, 1, 2, 1000, 0),   # a dilation past the end of a column too long for 20 KB
    (1020, 1, 2, 1, 2, 1024, 0),  # the same at the longest history
    (30, 2, 64, 9, 8, 3, 0),      # short columns: lane per column, whole blocks of 64
    (64, 3, 7, 11, 8, 32, 0),     # the longest, a ragged block, rows cut by blocks, a class of two steps
    (1, 5, 13, 1, 3, 1, 0),       # one step, several channels per block
    (9, 2, 5, 7, 32, 12, 0),      # a dilation past the end at the highest order
    (17, 4, 16, 3, 5, 2, -3),     # negative shifts
])
def test_tiles_equal_the_time_first_results(T, N, C, S, k, d, lo, offset, dtype):
    g = torch.Generator().manual_seed(11)
    shape = (T, N, C, S)
    if dtype == "q8_8":
        lo = max(lo, 0)
    desc = mfpsn.make_desc(shape, k, d, dtype, v_th=0.5, v_th_q=128, shift_lo=lo, shift_hi=7)

    def draw():
        v = torch.randn(shape, generator=g)
        return ((v * 256).round().to(torch.int16) if dtype == "q8_8" else v.to(mfpsn.STORAGE[desc.dtype])).to(DEV)

    x, gs = draw(), draw()
    sign = (torch.randint(0, 2, (C, k), generator=g) * 2 - 1).to(torch.int8).to(DEV)
    shift = torch.randint(lo, 8, (C, k), generator=g).to(torch.int8).to(DEV)
    bias = torch.randn(C, generator=g) * 0.1
    bias = ((bias * 256).round().to(torch.int32) if dtype == "q8_8" else bias).to(DEV)
    spikes, h = mfpsn.forward(desc, x, sign, shift, bias, want_h=True)
    gx, gw, gb = mfpsn.backward(desc, x, gs, sign, shift, bias)
    xl, gl = (place(t.movedim(0, -1), offset) for t in (x, gs))
    spikes_l, h_l = (torch.empty(spikes.numel() + offset, dtype=t, device=DEV)[offset:].view(xl.shape)
                     for t in (torch.uint8, h.dtype))
    mfpsn.mfpsn_forward_time_last(desc, xl, sign, shift, bias, spikes_l, h_l)
    spikes_n = torch.empty(spikes.numel() + offset, dtype=torch.uint8, device=DEV)[offset:].view(xl.shape)
    mfpsn.mfpsn_forward_time_last(desc, xl, sign, shift, bias, spikes_n)  # (kernels of their own)
    gx_l, gw_l, gb_l = mfpsn.backward_time_last(desc, xl, gl, sign, shift, bias)

    def same(a, b):
        b = b.movedim(0, -1).contiguous()
        bits = {2: torch.int16, 4: torch.int32}.get(b.element_size(), b.dtype)
        return torch.equal(a.contiguous().view(bits), b.view(bits))

    assert same(spikes_l, spikes) and same(spikes_n, spikes)
    assert same(h_l, h)
    assert same(gx_l, gx)
    for got, want in ((gw_l, gw), (gb_l, gb)):
        if dtype == "q8_8":
            assert torch.equal(got, want)
        else:
            assert bool(((got - want).abs() <= 1e-6 + 1e-5 * want.abs()).all())

"""Training of the small network on column slices of large feature-major
arrays: sixteen rows of a leading dimension of 71.6 million (FP32) span more
than 4 GiB, so row offsets need 64 bits.  The same bits as on contiguous
arrays, for tiles of 16 and of 32 samples."""
import pytest

import synth
from tests.helpers import make_handle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

WIDTHS = synth.NET_SMALL
HT = sum(WIDTHS[1:-1])


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


# the first leading dimension whose row 15 lies past 4 GiB, with the saved
# pre-activations (200 GB of address range, of which the slice is touched);
# without them one whose rows 8 to 15 do
@pytest.mark.parametrize("ld,save", [(71582789, True), (1 << 27, False)])
def test_column_slices_give_the_same_bits(ld, save):
    torch.cuda.empty_cache()
    need = 4 * ld * (3 * WIDTHS[0] + 3 * WIDTHS[-1] + (HT if save else 0))
    if torch.cuda.mem_get_info()[0] < need + (4 << 30):
        pytest.skip("not enough device memory")
    h = make_handle(synth.make_net(4, bias_scale=0.1), "fp32", max_batch=4200)
    p = h._params
    gen = torch.Generator("cuda").manual_seed(5)
    big_x = torch.empty((WIDTHS[0], ld), dtype=torch.float32, device="cuda")
    big_go = torch.empty((WIDTHS[-1], ld), dtype=torch.float32, device="cuda")
    big_z = torch.empty((HT, ld), dtype=torch.float32, device="cuda") if save else None
    for B in (33, 4200):
        print(f"case wide ld={ld} B={B} save={save}", flush=True)
        x = torch.randn((WIDTHS[0], B), device="cuda", generator=gen)
        go = torch.randn((WIDTHS[-1], B), device="cuda", generator=gen) / B
        z = torch.empty((HT, B), device="cuda") if save else None
        xw, gow = big_x[:, :B], big_go[:, :B]
        zw = big_z[:, :B] if save else None
        xw.copy_(x)
        gow.copy_(go)
        if save:
            zw.fill_(float("nan"))
        assert torch.equal(h.mlp_forward(xw, p, zw), h.mlp_forward(x, p, z))
        assert not save or torch.equal(zw, z)
        for saved, savedw in ((z, zw), (None, None)) if save else ((None, None),):
            ref = h.mlp_backward(x, p, saved, go, want_grad_x=True)
            got = h.mlp_backward(xw, p, savedw, gow, want_grad_x=True)
            assert torch.equal(got[0], ref[0]) and torch.equal(got[1], ref[1])
            del got
            assert torch.equal(h.mlp_backward(xw, p, savedw, gow)[0], ref[0])
    del big_x, big_go, big_z, xw, gow, zw
    torch.cuda.empty_cache()

"""The layer-by-layer path picks its tiles by the chunk's size; every choice
runs the same products in the same order, so a cell's result is the same bits
in a batch of any size.  Sizes around the tile edges, against a batch large
enough for the largest tiles (whose results the oracle tests check), and the
small ones against the FP64 oracle directly."""
import numpy as np
import pytest

import synth
from oracle import chem
from tests.helpers import dev_state, make_handle, rel_err

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BIG = 33000


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.fixture(scope="module")
def big():
    net = synth.make_net(6, bias_scale=0.1, out_stats=True)
    thermo = synth.make_thermo(6, 17)
    st = synth.make_state(6, BIG)
    return net, thermo, st


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
def test_every_batch_size_gives_the_same_bits(big, prec):
    net, thermo, st = big
    h = make_handle(net, prec, thermo=thermo)
    T, P, Y = dev_state(st)
    Yb, Tb = h.step(T, P, Y)
    torch.cuda.synchronize()
    o = 77                                   # (not on a block boundary)
    for n in (1, 15, 16, 17, 63, 65, 129, 255, 300, 511, 1000, 2049, 4097, 8300):
        print(f"case layer tiles {prec} n={n}", flush=True)
        Yn, Tn = h.step(T[o:o + n].contiguous(), P[o:o + n].contiguous(), Y[:, o:o + n].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(Yn, Yb[:, o:o + n]) and torch.equal(Tn, Tb[o:o + n]), n


@pytest.mark.parametrize("n", [1, 33, 129])
def test_small_batches_match_the_oracle(big, n):
    """FP32, the bar of the larger batches (1e-5 relative on Y_new and T_new)."""
    net, thermo, _ = big
    st = synth.make_state(6, n)
    h = make_handle(net, "fp32", thermo=thermo)
    Yn, Tn = h.step(*dev_state(st))
    torch.cuda.synchronize()
    ref = chem.step(st.T, st.P, st.Y, net, thermo=thermo)
    assert rel_err(Yn.cpu().numpy(), ref["Y_new"]) <= 1e-5
    assert rel_err(Tn.cpu().numpy(), ref["T_new"], floor=1.0) <= 1e-5
    assert np.isfinite(Tn.cpu().numpy()).all()

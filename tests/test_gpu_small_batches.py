"""A fused network's batch leaves a rest behind whole rounds of the fused
kernel's tiles; a small rest of a large network runs layer by layer.  The
products, their order and every rounding are the fused kernel's, so a cell's
result is the same bits as in a batch that the fused kernel takes whole: at the
edges of the cell-blocks and of the limits, and for a rest behind a round."""
import pytest

import synth
from tests.helpers import dev_state, make_handle
from tests.test_gpu_prop import _handle as make_prop

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BIG = 16384            # whole rounds of every fused tile size on 256 CUs


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def bits(t):
    return t.contiguous().view(torch.int64)


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
def test_chemistry_rests_give_the_same_bits(prec):
    net = synth.make_net(2, bias_scale=0.1, out_stats=True)
    h = make_handle(net, prec, thermo=synth.make_thermo(2, 29), molar_mass=synth.make_molar_masses(2, 29))
    T, P, Y = dev_state(synth.make_state(2, BIG))
    Y[3, 5] = float("nan")
    Yb, Tb, ob = h.step_source(T, P, Y, 1e-6)
    for n in (1, 15, 17, 64, 255, 1000, 4096, 4097, 6144, 6145):
        print(f"case rest {prec} n={n}", flush=True)
        nb = torch.zeros(1, dtype=torch.int32, device="cuda")
        Yn, Tn, on = h.step_source(T[:n].clone(), P[:n].clone(), Y[:, :n].contiguous(), 1e-6, n_bad=nb)
        assert torch.equal(bits(Yn), bits(Yb[:, :n])) and torch.equal(bits(Tn), bits(Tb[:n])), n
        assert torch.equal(bits(on), bits(ob[:, :n])) and int(nb) == (n > 5), n
    # one round, then a rest, in place
    n = BIG + 37
    T2, P2, Y2 = torch.cat([T, T[:37]]), torch.cat([P, P[:37]]), torch.cat([Y, Y[:, :37]], 1).contiguous()
    nb = torch.zeros(1, dtype=torch.int32, device="cuda")
    Yn, Tn = h.step(T2, P2, Y2, Y_out=Y2, n_bad=nb)
    assert torch.equal(bits(Yn), bits(torch.cat([Yb, Yb[:, :37]], 1))) and int(nb) == 2
    assert torch.equal(bits(Tn), bits(torch.cat([Tb, Tb[:37]])))


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
def test_property_rests_give_the_same_bits(prec):
    net = synth.make_prop_net(7, bias_scale=0.1)
    h = make_prop(net, prec)
    x = torch.tensor(synth.make_prop_inputs(7, BIG), device="cuda")
    yb = h.eval(x)
    for n in (1, 16, 33, 255, 256, 257, 1000, 6144, 6145):
        print(f"case property rest {prec} n={n}", flush=True)
        assert torch.equal(bits(h.eval(x[:, :n].contiguous())), bits(yb[:, :n])), n
    y2 = h.eval(torch.cat([x, x[:, :37]], 1).contiguous())
    assert torch.equal(bits(y2), bits(torch.cat([yb, yb[:, :37]], 1)))


def test_fp8_tiles_give_the_same_bits():
    """FP8 chooses tiles of 64 or 48 cells by the batch's size: edges of both
    tiles and of the ranges against a batch in tiles of 64."""
    net = synth.make_net(2, bias_scale=0.1, out_stats=True)
    h = make_handle(net, "fp8", thermo=synth.make_thermo(2, 29), act_amax=[6.0, 4.0, 4.0, 4.0])
    T, P, Y = dev_state(synth.make_state(2, 2 * BIG))
    Yb, Tb = h.step(T, P, Y)
    for n in (1, 47, 48, 49, 63, 65, 1000, 12288, 12289, 16384, 16385, 24577):
        print(f"case fp8 tiles n={n}", flush=True)
        Yn, Tn = h.step(T[:n].clone(), P[:n].clone(), Y[:, :n].contiguous())
        assert torch.equal(bits(Yn), bits(Yb[:, :n])) and torch.equal(bits(Tn), bits(Tb[:n])), n

"""The rest of a fused batch on fields inside larger arrays (leading dimension
past the cells) and with outputs in place (Y_out = Y, T_out = T): the bits of the
contiguous, out-of-place call, and nothing written past the cells."""
import pytest

import synth
from tests.helpers import dev_state, make_handle
from tests.test_gpu_prop import _handle as make_prop

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _same(a, b):
    return torch.equal(a.contiguous().view(torch.int64), b.contiguous().view(torch.int64))


def _padded(t, pad):
    """t [rows][n] inside rows of n + pad, -7 past the cells."""
    big = torch.full((t.shape[0], t.shape[1] + pad), -7.0, dtype=torch.float64, device="cuda")
    big[:, :t.shape[1]] = t
    return big


# a rest alone, and one behind whole rounds of the fused tiles
@pytest.mark.parametrize("n", [37, 1000, 16384 + 37])
@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16"])
def test_chemistry(prec, n):
    print(f"case rest fields {prec} n={n}", flush=True)
    net = synth.make_net(2, bias_scale=0.1, out_stats=True)
    h = make_handle(net, prec, thermo=synth.make_thermo(2, 29), molar_mass=synth.make_molar_masses(2, 29))
    T, P, Y = dev_state(synth.make_state(2, n))
    Yr, Tr, orr = h.step_source(T, P, Y, 1e-6)
    for pad in (1, 501):
        big, om = _padded(Y, pad), _padded(torch.zeros_like(Y), pad)
        Yw, T2 = big[:, :n], T.clone()
        Yn, Tn, on = h.step_source(T2, P, Yw, 1e-6, Y_out=Yw, T_out=T2, omega=om[:, :n])
        assert _same(Yn, Yr) and _same(Tn, Tr) and _same(on, orr)
        assert Yn.data_ptr() == big.data_ptr() and Tn.data_ptr() == T2.data_ptr()
        assert (big[:, n:] == -7.0).all() and (om[:, n:] == -7.0).all()
        # out of place, from a padded state
        out = torch.full_like(big, -7.0)
        Yn, Tn = h.step(T, P, _padded(Y, pad)[:, :n], Y_out=out[:, :n])
        assert _same(Yn, Yr) and _same(Tn, Tr) and (out[:, n:] == -7.0).all()


@pytest.mark.parametrize("prec,n", [("fp32", 1000), ("fp32", 8192 + 37), ("bf16", 200), ("fp16", 16384 + 37)])
def test_property(prec, n):
    print(f"case property rest fields {prec} n={n}", flush=True)
    h = make_prop(synth.make_prop_net(7, bias_scale=0.1), prec)
    x = torch.tensor(synth.make_prop_inputs(7, n), device="cuda")
    ref = h.eval(x)
    out = torch.full((1, n + 501), -7.0, dtype=torch.float64, device="cuda")
    y = h.eval(_padded(x, 501)[:, :n], out[:, :n])
    assert _same(y, ref) and (out[:, n:] == -7.0).all()

"""The rest of a fused network's batch runs layer by layer: inputs whose
Z-scores lie just past a tie of the operand format, where rounding once and
rounding through FP32 differ, become the same operands as in the fused kernel.
(The fused kernel's roundings are what the compiler makes of its conversions:
one for the property networks' inputs, two for temperature and pressure.)"""
import numpy as np
import pytest

import synth

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

BIG = 16384            # whole rounds of every fused tile size on 256 CUs


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def _past_ties(rng, shape, bits):
    """Values of [1, 2): `bits` significant bits, half an ulp, and 2^-40 more or less."""
    m = 1.0 + rng.integers(0, 1 << (bits - 1), shape) * 2.0 ** (1 - bits)
    return m + 2.0 ** -bits + np.where(rng.random(shape) < 0.5, 1.0, -1.0) * 2.0 ** -40


def _same(a, b):
    return torch.equal(a.contiguous().view(torch.int64), b.contiguous().view(torch.int64))


@pytest.mark.parametrize("prec,bits", [("bf16", 8), ("fp16", 11), ("fp32", 24)])
def test_property_inputs(prec, bits):
    from paper_2508_18969_amd import PropNet
    net = synth.make_prop_net(7, bias_scale=0.1)
    h = PropNet(net.widths, prec, torch.tensor(net.flat_params(), device="cuda"), np.zeros(3), np.ones(3))
    rng = np.random.default_rng(3)
    x = torch.tensor(_past_ties(rng, (3, BIG), bits) * rng.choice([-1.0, 1.0], (3, BIG)), device="cuda")
    yb = h.eval(x)
    for n in (1, 200, 256, 300):           # (300: tiles of 48 cells in 16 bits)
        print(f"case property inputs {prec} n={n}", flush=True)
        assert _same(h.eval(x[:, :n].contiguous()), yb[:, :n]), n
    y = h.eval(torch.cat([x, x[:, :100]], 1).contiguous())
    assert _same(y, torch.cat([yb, yb[:, :100]], 1))


@pytest.mark.parametrize("prec,bits", [("bf16", 8), ("fp16", 11), ("fp32", 24)])
def test_temperature_and_pressure(prec, bits):
    from paper_2508_18969_amd import ChemDNN
    net = synth.make_net(2, bias_scale=0.1, out_stats=True)
    mean, std = np.array(net.in_mean), np.array(net.in_std)
    mean[:2], std[:2] = 0.0, 1.0
    h = ChemDNN(net.widths, prec, torch.tensor(net.flat_params(), device="cuda"), mean, std, net.out_mean,
                net.out_std, lam=net.lam)
    rng = np.random.default_rng(4)
    T, P = torch.tensor(_past_ties(rng, (2, BIG), bits), device="cuda")
    Y = torch.tensor(synth.make_state(2, BIG).Y, device="cuda")
    yb, _ = h.step(T, P, Y)
    for n in (1, 200, 4096):
        print(f"case temperature and pressure {prec} n={n}", flush=True)
        y, _ = h.step(T[:n].clone(), P[:n].clone(), Y[:, :n].contiguous())
        assert _same(y, yb[:, :n]), n

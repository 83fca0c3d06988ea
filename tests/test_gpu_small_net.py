"""The small network's kernel (weights resident, tiles of one, two or four
cell-blocks by the batch's size): a cell's result is the same bits in a batch
of any size, at the edges of the cell-blocks and of the tiles' ranges, and the
species counts at the edges of its five-slot layout (18 at most; more run in the
fused kernel) match the FP64 oracle."""
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


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16", "fp8"])
def test_every_batch_size_gives_the_same_bits(prec):
    net = synth.make_net(1, bias_scale=0.1, out_stats=True)
    h = make_handle(net, prec, thermo=synth.make_thermo(1, 17), molar_mass=synth.make_molar_masses(1, 17),
                    act_amax=np.array([6.0, 4.0, 4.0, 4.0]) if prec == "fp8" else None)
    T, P, Y = dev_state(synth.make_state(1, BIG))
    Yb, Tb, ob = h.step_source(T, P, Y, 1e-6)
    torch.cuda.synchronize()
    o = 77                                   # (not on a block boundary)
    for n in (1, 15, 17, 1000, 4096, 4097, 8191, 8192, 8193, 16385):
        print(f"case small net {prec} n={n}", flush=True)
        Yn, Tn, on = h.step_source(T[o:o + n].contiguous(), P[o:o + n].contiguous(),
                                   Y[:, o:o + n].contiguous(), 1e-6)
        torch.cuda.synchronize()
        assert torch.equal(Yn, Yb[:, o:o + n]) and torch.equal(Tn, Tb[o:o + n]), n
        assert torch.equal(on, ob[:, o:o + n]), n


@pytest.mark.parametrize("S", [2, 13, 14, 15, 18, 19, 30])
def test_species_counts(S):
    """FP32, the bar of the 17-species net (1e-5 relative on Y_new and T_new)."""
    widths = (S + 2, 400, 200, 100, S)
    net = synth.make_net(1, widths=widths)
    thermo = synth.make_thermo(1, S)
    h = make_handle(net, "fp32", thermo=thermo)
    for n in (33, 4500):
        print(f"case small net species={S} n={n}", flush=True)
        st = synth.make_state(1, n, S=S)
        T, P, Y = dev_state(st, ld=n + 3)
        Yn, Tn = h.step(T, P, Y, Y_out=torch.empty(S, n + 3, dtype=torch.float64, device="cuda")[:, :n])
        torch.cuda.synchronize()
        ref = chem.step(st.T, st.P, st.Y, net, thermo=thermo)
        assert rel_err(Yn.cpu().numpy()[:, :n], ref["Y_new"]) <= 1e-5
        assert rel_err(Tn.cpu().numpy(), ref["T_new"], floor=1.0) <= 1e-5


@pytest.mark.parametrize("prec,gelu", [("fp32", "table"), ("bf16", "table16"), ("fp8", "table")])
def test_tables_give_the_same_bits_at_every_size(prec, gelu):
    """The tabulated GELU in the same kernel (its values against the oracle:
    test_gpu_step.py)."""
    net = synth.make_net(1, bias_scale=0.1, out_stats=True)
    h = make_handle(net, prec, gelu=gelu, act_amax=np.array([6.0, 4.0, 4.0, 4.0]) if prec == "fp8" else None)
    T, P, Y = dev_state(synth.make_state(1, BIG))
    Yb, _ = h.step(T, P, Y)
    torch.cuda.synchronize()
    o = 77
    for n in (1, 17, 4096, 4097, 8193):
        print(f"case small net {gelu} {prec} n={n}", flush=True)
        Yn, _ = h.step(T[o:o + n].contiguous(), P[o:o + n].contiguous(), Y[:, o:o + n].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(Yn, Yb[:, o:o + n]), n

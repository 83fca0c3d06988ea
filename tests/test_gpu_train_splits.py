"""Weight-gradient splits of the small network's training at their limits: the
allocation-free step at the largest batches of its static scratch, and batches
and chunks on both sides of the change from 27 to 34 splits (293 blocks of 32
samples)."""
import numpy as np
import pytest

import synth
from oracle import train
from tests.helpers import dev_state, make_handle

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

WIDTHS = synth.NET_SMALL


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


@pytest.mark.parametrize("S,B,chunk", [(2, 9360, 0), (9, 9280, 0), (13, 9232, 0), (13, 20000, 9232),
                                       (17, 9184, 0), (17, 1000, 16)])
def test_noalloc_takes_the_largest_batches(S, B, chunk):
    """The step of a handle with its own scratch, bit for bit."""
    print(f"case noalloc S={S} B={B} chunk={chunk}", flush=True)
    net = synth.make_net(1, widths=(S + 2, 400, 200, 100, S))
    T, P, Y = dev_state(synth.make_state(1, B, S=S))
    target = 0.1 * torch.randn((S, B), device="cuda", generator=torch.Generator("cuda").manual_seed(S))
    out = []
    for noalloc in (False, True):
        h = make_handle(net, "fp32", max_batch=0 if noalloc else B, recompute_chunk=chunk)
        p = h._params.clone()
        g, m, v = torch.full_like(p, float("nan")), torch.zeros_like(p), torch.zeros_like(p)
        loss = (h.train_step_noalloc if noalloc else h.train_step)(T, P, Y, target, p, g, m, v, 1)
        torch.cuda.synchronize()
        out.append([t.clone() for t in (loss, p, g, m, v)])
    assert all(torch.equal(a, b) for a, b in zip(*out)) and torch.isfinite(out[0][2]).all()


def _rel(got, ref):
    return float(np.linalg.norm(got - ref) / max(np.linalg.norm(ref), 1e-30))


@pytest.mark.parametrize("B,chunk", [(9376, 0), (9377, 0), (18500, 9392)])
def test_split_edges_match_fp64(B, chunk):
    """1e-4 relative per tensor, the bar of the other batches."""
    print(f"case train splits B={B} chunk={chunk}", flush=True)
    net = synth.make_net(4, bias_scale=0.1)
    rng = np.random.default_rng(B)
    x = rng.standard_normal((WIDTHS[0], B)).astype(np.float32)
    go = (rng.standard_normal((WIDTHS[-1], B)) / B).astype(np.float32)
    h = make_handle(net, "fp32", max_batch=B, recompute_chunk=chunk)
    gp, _ = h.mlp_backward(torch.tensor(x, device="cuda"), h._params, None, torch.tensor(go, device="cuda"))
    p64 = net.flat_params().astype(np.float64)
    _, zs = train.forward(x.astype(np.float64), p64, WIDTHS)
    g_ref, _ = train.backward(x.astype(np.float64), p64, WIDTHS, zs, go.astype(np.float64))
    got, ref = train.unflatten(gp.cpu().numpy().astype(np.float64), WIDTHS), train.unflatten(g_ref, WIDTHS)
    for a, b in zip(got[0] + got[1], ref[0] + ref[1]):
        assert _rel(a, b) <= 1e-4

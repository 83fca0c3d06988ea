"""The small network's training path works on tiles of 16 or 32 samples and
fixed batch splits; batches at the edges of both, with padded leading
dimensions and odd chunks, against the FP64 oracle (1e-4 relative per tensor,
the bar of the larger batches: FP32-accurate products over K <= 400 and sums
over the batch carry a few 1e-7)."""
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


def _rel(got, ref):
    return float(np.linalg.norm(got - ref) / max(np.linalg.norm(ref), 1e-30))


def _padded(a, pad):
    """a [rows][B] float32 on the device inside rows of B + pad (NaN past B)."""
    t = torch.full((a.shape[0], a.shape[1] + pad), float("nan"), dtype=torch.float32, device="cuda")
    t[:, :a.shape[1]] = torch.tensor(a, dtype=torch.float32)
    return t[:, :a.shape[1]]


# one sample; 16-sample tiles and their halves of a 32-sample block; the last
# batch of one round of 16-sample tiles on 256 CUs and the first after it; the
# last batch with 24 weight-gradient splits and the first after it
@pytest.mark.parametrize("B,pad,chunk", [(1, 0, 0), (1, 3, 0), (15, 0, 0), (16, 5, 0), (17, 0, 0), (33, 1, 0),
                                         (63, 0, 16), (100, 7, 48), (4096, 0, 0), (4097, 3, 0),
                                         (9216, 0, 0), (9217, 2, 4112)])
def test_edges_match_fp64(B, pad, chunk):
    print(f"case train tiles B={B} pad={pad} chunk={chunk}", flush=True)
    net = synth.make_net(4, bias_scale=0.1)
    rng = np.random.default_rng(B)
    x = rng.standard_normal((WIDTHS[0], B)).astype(np.float32)
    go = (rng.standard_normal((WIDTHS[-1], B)) / B).astype(np.float32)
    h = make_handle(net, "fp32", max_batch=B, recompute_chunk=chunk)
    p = torch.tensor(net.flat_params(), device="cuda")
    p64 = net.flat_params().astype(np.float64)
    xd, god = _padded(x, pad), _padded(go, pad)
    saved = _padded(np.zeros((sum(WIDTHS[1:-1]), B), np.float32), pad)
    out = h.mlp_forward(xd, p, saved)
    out2 = h.mlp_forward(xd, p)
    gp, gx = h.mlp_backward(xd, p, saved, god, want_grad_x=True)
    gp2, gx2 = h.mlp_backward(xd, p, None, god, want_grad_x=True)
    gp3, _ = h.mlp_backward(xd, p, saved, god)
    torch.cuda.synchronize()
    o_ref, zs = train.forward(x.astype(np.float64), p64, WIDTHS)
    g_ref, gx_ref = train.backward(x.astype(np.float64), p64, WIDTHS, zs, go.astype(np.float64))
    assert torch.equal(out, out2) and torch.equal(gp, gp2) and torch.equal(gx, gx2) and torch.equal(gp, gp3)
    assert _rel(out.cpu().numpy(), o_ref) <= 1e-4
    row, sv = 0, saved.cpu().numpy()
    for z in zs[:3]:
        assert _rel(sv[row:row + z.shape[0]], z) <= 1e-4
        row += z.shape[0]
    got, ref = train.unflatten(gp.cpu().numpy().astype(np.float64), WIDTHS), train.unflatten(g_ref, WIDTHS)
    for a, b in zip(got[0] + got[1], ref[0] + ref[1]):
        assert _rel(a, b) <= 1e-4
    assert _rel(gx.cpu().numpy(), gx_ref) <= 1e-4


def test_gradients_are_no_further_off_than_fp32_products():
    """Batch 40,000 of normal output gradients, whose bias gradients cancel to
    1/200 of their terms' sum: a rounding bias of a tenth of an ulp would show
    there.  FP32 products are within 5e-7 per tensor; so is this path."""
    B = 40000
    net = synth.make_net(4, bias_scale=0.1)
    rng = np.random.default_rng(1)
    x = rng.standard_normal((WIDTHS[0], B)).astype(np.float32)
    go = (rng.standard_normal((WIDTHS[-1], B)) / B).astype(np.float32)
    h = make_handle(net, "fp32", max_batch=B)
    p = torch.tensor(net.flat_params(), device="cuda")
    gp, _ = h.mlp_backward(torch.tensor(x, device="cuda"), p, None, torch.tensor(go, device="cuda"))
    p64 = net.flat_params().astype(np.float64)
    _, zs = train.forward(x.astype(np.float64), p64, WIDTHS)
    g_ref, _ = train.backward(x.astype(np.float64), p64, WIDTHS, zs, go.astype(np.float64))
    got, ref = train.unflatten(gp.cpu().numpy().astype(np.float64), WIDTHS), train.unflatten(g_ref, WIDTHS)
    for a, b in zip(got[0] + got[1], ref[0] + ref[1]):
        assert _rel(a, b) <= 5e-7


def test_first_training_call_under_capture():
    """A handle made without training sets its training kernels up with its
    first training call; that call may be the one that is captured."""
    net = synth.make_net(4)
    n = 300
    st = synth.make_state(4, n)
    h = make_handle(net, "fp32", max_batch=0)
    T, P, Y = dev_state(st)
    target = 0.1 * torch.randn(17, n, device="cuda", generator=torch.Generator("cuda").manual_seed(1))
    start = h._params.clone()
    p, g, m, v = start.clone(), torch.empty_like(start), torch.zeros_like(start), torch.zeros_like(start)
    loss = torch.empty(1, device="cuda")

    def step():
        return h.train_step_noalloc(T, P, Y, target, p, g, m, v, 1, loss=loss)

    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        step()
    seen = []
    for k in range(4):                      # three replays, then the eager call
        p.copy_(start)
        m.zero_()
        v.zero_()
        g.fill_(-1.0)
        loss.fill_(-1.0)
        graph.replay() if k < 3 else step()
        torch.cuda.synchronize()
        seen.append([t.clone() for t in (p, g, m, v, loss)])
    for s in seen[:3]:
        assert all(torch.equal(a, b) for a, b in zip(s, seen[3]))
    assert float(seen[3][4]) > 0.0

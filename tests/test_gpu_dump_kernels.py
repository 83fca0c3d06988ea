"""The layer dump (chem_dnn_debug_layers) runs the kernels of chem_dnn_step:
the two calls are captured, and the kernels of their graphs compared (names,
grids, workgroups); the checks of the layers then hold for the kernels in use."""
import ctypes as C
import re

import numpy as np
import pytest

import synth
from oracle import chem
from paper_2508_18969_amd import binding
from tests.helpers import dev_state, make_handle
from tests.test_gpu_layers import _layer_checks

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

AMAX = np.array([6.0, 4.0, 4.0, 4.0], np.float32)


@pytest.fixture(scope="module", autouse=True)
def _gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


class KernelNode(C.Structure):
    """hipKernelNodeParams"""
    _fields_ = [("block", C.c_uint32 * 3), ("extra", C.c_void_p), ("func", C.c_void_p),
                ("grid", C.c_uint32 * 3), ("params", C.c_void_p), ("shared", C.c_uint32)]


@pytest.fixture(scope="module")
def hip():
    torch.cuda.init()
    path = next(l.split()[-1] for l in open("/proc/self/maps") if "libamdhip64" in l)
    lib = C.CDLL(path)
    lib.hipKernelNameRefByPtr.restype = C.c_char_p
    lib.hipKernelNameRefByPtr.argtypes = [C.c_void_p, C.c_void_p]
    return lib


def _kernels(hip, call):
    """(kernel, operand format, grid, workgroup) of the kernels that `call`
    launches; it is captured, not run."""
    stream = torch.cuda.Stream()
    raw, graph, count = C.c_void_p(stream.cuda_stream), C.c_void_p(), C.c_size_t()
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):
        assert hip.hipStreamBeginCapture(raw, 2) == 0          # relaxed
        try:
            call()
        finally:
            st = hip.hipStreamEndCapture(raw, C.byref(graph))
    assert st == 0 and hip.hipGraphGetNodes(graph, None, C.byref(count)) == 0
    nodes = (C.c_void_p * count.value)()
    assert hip.hipGraphGetNodes(graph, nodes, C.byref(count)) == 0
    out = []
    for node in nodes:
        kind, p = C.c_int(), KernelNode()
        assert hip.hipGraphNodeGetType(C.c_void_p(node), C.byref(kind)) == 0 and kind.value == 0
        assert hip.hipGraphKernelNodeGetParams(C.c_void_p(node), C.byref(p)) == 0
        name = hip.hipKernelNameRefByPtr(p.func, None).decode()
        base = re.search(r"[a-z_]+_kernel", name).group(0)
        fmt = re.search(r"Op(F32|BF16|F16|F8)", name).group(0)
        out.append((base, fmt, tuple(p.grid), tuple(p.block)))
    hip.hipGraphDestroy(graph)
    return out


@pytest.mark.parametrize("config,prec,S", [
    (1, "fp32", 17), (1, "bf16", 17), (1, "fp16", 17), (1, "fp8", 17), (1, "bf16", 19), (1, "fp8", 30),
    (2, "fp32", 29), (2, "bf16", 29), (2, "fp16", 29), (2, "fp8", 29), (6, "bf16", 17)])
def test_dump_runs_the_kernels_of_the_step(hip, config, prec, S):
    widths = {1: (S + 2, 400, 200, 100, S)}.get(config)
    net = synth.make_net(config, widths=widths) if widths else synth.make_net(config)
    h = make_handle(net, prec, act_amax=AMAX if prec == "fp8" else None)
    for n in (1, 200, 4096):
        print(f"case dump kernels config={config} {prec} S={S} n={n}", flush=True)
        T, P, Y = dev_state(synth.make_state(config, n, S=S))
        Yo = torch.empty_like(Y)
        q = torch.empty((sum(net.widths[:-1]), n), device="cuda")
        a = torch.empty((sum(net.widths[1:]), n), device="cuda")
        step = _kernels(hip, lambda: h.step(T, P, Y, Y_out=Yo))
        dump = _kernels(hip, lambda: binding._check(binding.lib().chem_dnn_debug_layers(
            h._h, n, n, binding._ptr(T), binding._ptr(P), binding._ptr(Y), binding._ptr(q),
            binding._ptr(a), binding._stream()), "chem_dnn_debug_layers"))
        assert step and step == [k for k in dump if k[0] != "frag_decode_kernel"]


@pytest.mark.parametrize("prec", ["fp32", "bf16", "fp16", "fp8"])
@pytest.mark.parametrize("S,n", [(2, 33), (18, 200), (19, 200)])
def test_layers_at_the_edges_of_the_small_kernel(prec, S, n):
    """Its fewest and most species, and the fused kernel's first."""
    print(f"case dump layers {prec} S={S} n={n}", flush=True)
    net = synth.make_net(1, widths=(S + 2, 400, 200, 100, S), bias_scale=0.1, out_stats=True)
    act_s = w_s = amax = None
    if prec == "fp8":
        cal = synth.make_state(1, 1 << 12, S=S, stream="calibration")
        amax = chem.layer_input_amax(cal.T, cal.P, cal.Y, net).astype(np.float32)
        act_s, w_s = chem.pow2_scale(amax.astype(np.float64)), chem.pow2_scale(chem.weight_amax(net))
    h = make_handle(net, prec, act_amax=amax)
    _layer_checks(h, net, synth.make_state(1, n, S=S), prec, act_s, w_s)


@pytest.mark.parametrize("prec,n", [("fp8", 33), ("fp8", 333), ("bf16", 333), ("fp32", 33)])
def test_layers_of_ragged_tiles(prec, n):
    """The large network: last tiles of one, two and three cell-blocks."""
    print(f"case dump layers 29 species {prec} n={n}", flush=True)
    net = synth.make_net(2, bias_scale=0.1, out_stats=True)
    act_s = w_s = amax = None
    if prec == "fp8":
        cal = synth.make_state(2, 1 << 12, stream="calibration")
        amax = chem.layer_input_amax(cal.T, cal.P, cal.Y, net).astype(np.float32)
        act_s, w_s = chem.pow2_scale(amax.astype(np.float64)), chem.pow2_scale(chem.weight_amax(net))
    h = make_handle(net, prec, act_amax=amax)
    _layer_checks(h, net, synth.make_state(2, n), prec, act_s, w_s)


@pytest.mark.parametrize("config,prec", [(c, p) for c in (1, 2) for p in ("bf16", "fp16", "fp8")])
def test_the_dumped_output_is_the_steps(config, prec):
    """The output accumulators through the FP64 post-processing are Y_new to
    the FP32 inverse transform's error (1e-5, the bar of FP32 operands)."""
    print(f"case dump output config={config} {prec}", flush=True)
    net = synth.make_net(config, bias_scale=0.1, out_stats=True)
    thermo = synth.make_thermo(config, net.widths[-1])
    h = make_handle(net, prec, thermo=thermo, act_amax=AMAX if prec == "fp8" else None)
    st = synth.make_state(config, 333)
    T, P, Y = dev_state(st)
    _, acc = h.debug_layers(T, P, Y)
    Yn, _ = h.step(T, P, Y)
    torch.cuda.synchronize()
    o = acc[-1].cpu().numpy().astype(np.float64)
    if prec == "fp8":
        a, w = h.scales()
        o = o * (float(a[3]) * float(w[3])) + np.asarray(net.b[3], np.float64)[:, None]
    y, _, _ = chem.post(o, st.T, st.Y, net.out_mean, net.out_std, net.lam, thermo)
    assert np.max(np.abs(Yn.cpu().numpy() - y) / np.maximum(np.abs(y), 1e-10)) <= 1e-5

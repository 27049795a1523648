"""Forwards that read the packed arrays as they are leave the workspace alone: programs give one buffer to such calls on two streams, or the workspace that a
kept state waits in.

Sizes: the matrix-vector kernels, and k_gemm_mid with 64, 96 and 128 tokens a tile, few tiles and more than one round of them, ragged tokens, rows and columns.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
import paper_2407_11062_amd as eq
from paper_2407_11062_amd import synth

pytestmark = pytest.mark.gpu
TOL = 2e-2          # bf16 activations, as max|got - ref| / max|ref|

# (tokens, in, out, bits, group)
SIZES = [
    (1, 4096, 1024, 2, 64),
    (8, 5120, 520, 3, 128),
    (40, 1024, 1024, 4, 32),
    (128, 4096, 4096, 2, 64),
    (70, 8192, 1000, 3, 128),
    (100, 11008, 1288, 4, 32),
    (256, 4096, 4096, 2, -1),
    (257, 3424, 2560, 3, 32),                   # the last step has 96 columns of 256
    (333, 11008, 4096, 4, 128),
    (333, 4096, 11008, 2, 64),                  # 344 tiles
    (1000, 4096, 4096, 2, 128),
    (130, 2080, 1016, 4, 32),                   # nine steps, the last of 32 columns
]


def npf(t):
    return t.detach().float().cpu().numpy()


def layer(T, I, O, bits, g):
    W = synth.normal((O, I), 0.02, synth.seed_of("leaves workspace", I, O), torch.bfloat16)
    X = synth.normal((T, I), 1.0, synth.seed_of("leaves workspace", T, I), torch.bfloat16)
    s, z = oracle.init_minmax(npf(W), bits, g)
    Wp, zp = eq.eqat_pack(W.cuda(), torch.from_numpy(s).cuda(), torch.from_numpy(z).cuda(), bits, g)
    return X, s, z, Wp, zp


def route(d, source):
    out = (ctypes.c_int32 * 3)()
    assert eq.lib().eqat_fwd_route(ctypes.byref(d), source, out) == 0
    return out[0]


@pytest.mark.parametrize("T,I,O,bits,g", SIZES)
def test_not_a_byte_of_it_changes(T, I, O, bits, g):
    X, s, z, Wp, zp = layer(T, I, O, bits, g)
    d = eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16)
    assert route(d, 1) not in (0, 7) and route(d, 2) not in (0, 7)         # neither the tiled GEMM nor codes re-laid first
    Xd, sd, zd = X.cuda(), torch.from_numpy(s).cuda(), torch.from_numpy(z).cuda()
    ws = torch.empty(max(eq.lib().eqat_workspace_bytes(ctypes.byref(d), op) for op in range(6)), dtype=torch.uint8, device="cuda").random_(0, 256)
    before = ws.clone()
    Y = eq.eqat_qlinear_fwd(Xd, Wp, sd, zp, bits, g, ws=ws)
    Yz = eq.eqat_qlinear_fwd_z(Xd, Wp, sd, zd, bits, g, ws=ws)
    assert torch.equal(ws, before)
    ref = oracle.qlinear_fwd(npf(X), Wp.cpu().numpy(), s, zp.cpu().numpy(), bits, g)
    assert np.abs(npf(Y) - ref).max() <= TOL * np.abs(ref).max()
    assert torch.equal(Y, Yz)
    if T > 16:
        assert torch.equal(Y, eq.eqat_qlinear_fwd_prepared(Xd, eq.eqat_qlinear_prepare(Wp, zp, I, bits, g), sd, O, bits, g))


@pytest.mark.parametrize("g", [64, 256])          # 256: wider than a dW tile, and the backward's workspace has another layout
def test_a_kept_state_survives_a_forward_of_the_packed_arrays(g):
    T, I, O, bits = 333, 4096, 4096, 4
    X, s, z, Wp, zp = layer(T, I, O, bits, g)
    Xd, sd = X.cuda(), torch.from_numpy(s).cuda()
    dY = synth.normal((T, O), 1.0, synth.seed_of("leaves workspace", T, O), torch.bfloat16).cuda()
    d = eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16)
    ws = eq.workspace(d, eq.OP_Q_BWD, Xd.device)
    first = eq.eqat_qlinear_fwd(Xd, Wp, sd, zp, bits, g, ws=ws, keep=True)
    between = eq.eqat_qlinear_fwd(Xd, Wp, sd, zp, bits, g, ws=ws)
    want = eq.eqat_qlinear_bwd(Xd, Wp, sd, zp, dY, I, bits, g)
    for ask in (("dX",), ("dX", "ds"), ("dX",)):
        out = {"dX": torch.full((T, I), float("nan"), dtype=torch.bfloat16, device="cuda")}
        got = eq.eqat_qlinear_bwd(Xd, Wp, sd, zp, dY, I, bits, g, want=ask, out=out, ws=ws, kept=True)
        alone = eq.eqat_qlinear_bwd(Xd, Wp, sd, zp, dY, I, bits, g, want=ask)
        assert all(torch.equal(got[k], alone[k]) for k in ask)
        eq.eqat_qlinear_fwd(Xd, Wp, sd, zp, bits, g, ws=ws)
    assert torch.equal(first, between) and torch.equal(got["dX"], alone["dX"])
    some = np.arange(0, T, 37)
    ref = oracle.qlinear_bwd(npf(X)[some], Wp.cpu().numpy(), s, zp.cpu().numpy(), npf(dY)[some], I, bits, g)["dX"]
    assert np.abs(npf(want["dX"])[some] - ref).max() <= TOL * np.abs(ref).max()


def test_two_streams_and_replays_with_one_workspace():
    T, I, O, bits, g = 100, 11008, 1288, 4, 32
    X, s, z, Wp, zp = layer(T, I, O, bits, g)
    sd = torch.from_numpy(s).cuda()
    Xs = [X.cuda(), -X.cuda()]
    want = [eq.eqat_qlinear_fwd(x, Wp, sd, zp, bits, g) for x in Xs]
    ws = eq.workspace(eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16), eq.OP_Q_FWD, torch.device("cuda"))
    got = [[torch.full_like(want[k], float("nan")) for _ in range(8)] for k in range(2)]
    x, Y, graph = Xs[0].clone(), torch.empty_like(want[0]), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        eq.eqat_qlinear_fwd(x, Wp, sd, zp, bits, g, Y=Y, ws=ws)
    streams = [torch.cuda.Stream() for _ in range(2)]
    torch.cuda.synchronize()
    for n in range(8):                                    # two launches at a time
        for k, stream in enumerate(streams):
            with torch.cuda.stream(stream):
                eq.eqat_qlinear_fwd(Xs[k], Wp, sd, zp, bits, g, Y=got[k][n], ws=ws)
        graph.replay()                                    # and a third
    torch.cuda.synchronize()
    assert all(torch.equal(y, want[k]) for k in range(2) for y in got[k])
    for k in (1, 0, 1):
        x.copy_(Xs[k])
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(Y, want[k])

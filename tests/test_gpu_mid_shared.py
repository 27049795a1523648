"""k_gemm_mid where several workgroups share a tile, a part of the contraction each, and meet in memory.

Sizes: two, three and four parts, K steps that do not divide by them, a last step cut short, ragged tokens and rows, whole tiles in front of the
shared ones, 64 and 96 tokens a tile.  The words that count arrivals lie in a workspace that holds anything.
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

# (tokens, in, out, bits, group, token tile, parts)
SIZES = [
    (128, 4096, 4096, 2, 64, 64, 3),            # 16 steps: 6, 5, 5
    (70, 8192, 1000, 3, 128, 64, 4),
    (100, 11008, 1288, 4, 32, 64, 4),           # 43 steps
    (256, 4096, 4096, 2, -1, 64, 2),
    (257, 3424, 2560, 3, 32, 64, 2),            # the last step has 96 columns of 256
    (333, 11008, 4096, 4, 128, 96, 2),
    (333, 4096, 11008, 2, 64, 96, 2),           # 256 whole tiles, then 88 shared ones
    (130, 2080, 1016, 4, 32, 64, 3),            # nine steps, the last of 32 columns
]


def npf(t):
    return t.detach().float().cpu().numpy()


def parts_bytes(d, op, ws_bytes):
    first, end = ctypes.c_size_t(), ctypes.c_size_t()
    assert eq.lib().eqat_plan_scratch(ctypes.byref(d), op, 0, 256, ws_bytes, ctypes.byref(first), ctypes.byref(end)) == 0
    return end.value - first.value


def layer(T, I, O, bits, g):
    W = synth.normal((O, I), 0.02, synth.seed_of("mid shared", I, O), torch.bfloat16)
    X = synth.normal((T, I), 1.0, synth.seed_of("mid shared", T, I), torch.bfloat16)
    s, z = oracle.init_minmax(npf(W), bits, g)
    Wp, zp = eq.eqat_pack(W.cuda(), torch.from_numpy(s).cuda(), torch.from_numpy(z).cuda(), bits, g)
    return X, s, z, Wp, zp


@pytest.mark.parametrize("T,I,O,bits,g,bm,parts", SIZES)
def test_shared_tiles_against_the_oracle_and_from_every_source(T, I, O, bits, g, bm, parts):
    X, s, z, Wp, zp = layer(T, I, O, bits, g)
    d = eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16)
    n = eq.lib().eqat_workspace_bytes(ctypes.byref(d), eq.OP_Q_FWD)
    tiles = -(-T // bm) * -(-O // 128)
    assert parts_bytes(d, eq.OP_Q_FWD, n) == 2048 + tiles % 256 * parts * bm * 128 * 4
    Xd, sd, zd = X.cuda(), torch.from_numpy(s).cuda(), torch.from_numpy(z).cuda()
    ref = oracle.qlinear_fwd(npf(X), Wp.cpu().numpy(), s, zp.cpu().numpy(), bits, g)
    ws = torch.empty(n, dtype=torch.uint8, device="cuda")
    first = None
    for fill in (0, 255, 1, None):                       # whatever the workspace holds, and what the launch before left in it
        if fill is not None:
            ws.fill_(fill)
        Y = eq.eqat_qlinear_fwd(Xd, Wp, sd, zp, bits, g, ws=ws)
        first = Y if first is None else first
        assert torch.equal(Y, first)
    assert np.abs(npf(first) - ref).max() <= TOL * np.abs(ref).max()
    assert torch.equal(eq.eqat_qlinear_fwd_z(Xd, Wp, sd, zd, bits, g), first)
    prepared = eq.eqat_qlinear_prepare(Wp, zp, I, bits, g)
    assert torch.equal(eq.eqat_qlinear_fwd_prepared(Xd, prepared, sd, O, bits, g), first)


def test_a_workspace_without_room_for_parts_is_taken():
    T, I, O, bits, g = 128, 4096, 4096, 2, 64
    X, s, z, Wp, zp = layer(T, I, O, bits, g)
    d, one = eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16), eq.make_desc(1, I, O, bits, g, eq.BF16, eq.BF16)
    small = eq.lib().eqat_workspace_bytes(ctypes.byref(one), eq.OP_Q_FWD)          # sized for one token
    assert parts_bytes(d, eq.OP_Q_FWD, small) == 0
    Xd, sd = X.cuda(), torch.from_numpy(s).cuda()
    ws = torch.empty(small + 4096, dtype=torch.uint8, device="cuda").fill_(7)
    Y = eq.eqat_qlinear_fwd(Xd, Wp, sd, zp, bits, g, ws=ws[:small])
    assert bool((ws[small:] == 7).all())
    shared = eq.eqat_qlinear_fwd(Xd, Wp, sd, zp, bits, g)
    assert (Y.float() - shared.float()).abs().max() <= 2 ** -7 * shared.float().abs().max()          # another order of the sums: a rounding


def test_replays_of_a_graph_and_two_streams():
    T, I, O, bits, g = 100, 11008, 1288, 4, 32
    X, s, z, Wp, zp = layer(T, I, O, bits, g)
    sd = torch.from_numpy(s).cuda()
    d = eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16)
    Xs = [X.cuda(), -X.cuda()]
    want = [eq.eqat_qlinear_fwd(x, Wp, sd, zp, bits, g) for x in Xs]
    x, Y, ws = Xs[0].clone(), torch.empty_like(want[0]), eq.workspace(d, eq.OP_Q_FWD, torch.device("cuda"))
    st, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph, stream=st):
        for _ in range(2):                                # the same workspace twice in a row
            eq.eqat_qlinear_fwd(x, Wp, sd, zp, bits, g, Y=Y, ws=ws)
    for k in (1, 0, 1, 0):
        x.copy_(Xs[k])
        graph.replay()
        eager = eq.eqat_qlinear_fwd(Xs[1 - k], Wp, sd, zp, bits, g)          # eager work between the replays
        torch.cuda.synchronize()
        assert torch.equal(Y, want[k]) and torch.equal(eager, want[1 - k])
    streams = [torch.cuda.Stream() for _ in range(2)]
    got = [[], []]
    for _ in range(6):                                    # two launches at a time, each with a workspace of its own
        for k, stream in enumerate(streams):
            with torch.cuda.stream(stream):
                got[k].append(eq.eqat_qlinear_fwd(Xs[k], Wp, sd, zp, bits, g))
    torch.cuda.synchronize()
    assert all(torch.equal(y, want[k]) for k in range(2) for y in got[k])

"""Prepared layers where k_gemm_mid computes the forward: it reads step sizes and zero points as they are and leaves the pairs that a backward wants, or
reads the pairs of a small launch in front of it (long contractions).

Sizes: every token tile, more pairs than one round of the launch's lanes, fewer than its lanes, one group to a row, ragged rows and columns; both sides of
the lines between the two.
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

# (tokens, in, out, bits, group, token tile)
SIZES = [
    (65, 896, 392, 3, 32, 64),
    (66, 28672, 128, 2, 32, 64),              # groups of 32: the pairs by themselves where a backward follows, else not
    (66, 6144, 1024, 2, 32, 64),              # 49152 quads of pairs, 8192 lanes
    (70, 6400, 264, 4, 128, 64),              # a step more than the forward without the small launch takes
    (400, 8192, 520, 3, -1, 64),              # one group to a row, at any length
    (300, 4096, 2048, 4, 64, 64),
    (515, 4096, 4096, 3, -1, 96),             # one pair to a row
    (1000, 4096, 4096, 2, 128, 128),
    (700, 1056, 1016, 3, 32, 64),
    (333, 1024, 8, 2, -1, 64),                # eight pairs
]


def npf(t):
    return t.detach().float().cpu().numpy()


@pytest.mark.parametrize("trained", [False, True])
@pytest.mark.parametrize("T,I,O,bits,g,bm", SIZES)
def test_forward_and_what_it_leaves(T, I, O, bits, g, bm, trained):
    W = synth.normal((O, I), 0.02, synth.seed_of("one launch", I, O), torch.bfloat16)
    X = synth.normal((T, I), 1.0, synth.seed_of("one launch", T, I), torch.bfloat16).cuda()
    dY = synth.normal((T, O), 1.0, synth.seed_of("one launch", T, O), torch.bfloat16).cuda()
    s, z = oracle.init_minmax(npf(W), bits, g)
    sd, zd = torch.from_numpy(s).cuda(), torch.from_numpy(z).cuda()
    Wp, zp = eq.eqat_pack(W.cuda(), sd, zd, bits, g)
    zt = zd + 0.25 if trained else None
    prepared = eq.eqat_qlinear_prepare(Wp, zp, I, bits, g)
    d = eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16)
    route = (ctypes.c_int32 * 3)()
    assert eq.lib().eqat_fwd_route(ctypes.byref(d), 0, route) == 0 and (route[0], route[1]) == (1, bm)       # k_gemm_mid
    ws = eq.workspace(d, eq.OP_QP_BWD, X.device)
    ws.fill_(255)                         # NaNs wherever a pair is not written
    Y = eq.eqat_qlinear_fwd_prepared(X, prepared, sd, O, bits, g, z=zt, ws=ws, keep=True)
    kept = eq.eqat_qlinear_bwd_prepared(X, prepared, sd, dY, I, bits, g, z=zt, want=("dX", "ds", "dz"), ws=ws, kept=True)
    alone = eq.eqat_qlinear_bwd_prepared(X, prepared, sd, dY, I, bits, g, z=zt, want=("dX", "ds", "dz"))
    assert all(torch.equal(kept[k], alone[k]) for k in alone)
    packed = eq.eqat_qlinear_fwd_z(X, Wp, sd, zt, bits, g) if trained else eq.eqat_qlinear_fwd(X, Wp, sd, zp, bits, g)
    assert torch.equal(Y, packed) and torch.equal(Y, eq.eqat_qlinear_fwd_prepared(X, prepared, sd, O, bits, g, z=zt))
    if not trained:
        ref = oracle.qlinear_fwd(npf(X), Wp.cpu().numpy(), s, zp.cpu().numpy(), bits, g)
        assert np.abs(npf(Y) - ref).max() <= TOL * np.abs(ref).max()


def test_replays_take_the_step_sizes_of_their_time():
    T, I, O, bits, g = 300, 1024, 1024, 3, 64
    W = synth.normal((O, I), 0.02, synth.seed_of("one launch", I, O), torch.bfloat16).cuda()
    X = synth.normal((T, I), 1.0, synth.seed_of("one launch", T, I), torch.bfloat16).cuda()
    dY = synth.normal((T, O), 1.0, synth.seed_of("one launch", T, O), torch.bfloat16).cuda()
    s, z = (torch.from_numpy(a).cuda() for a in oracle.init_minmax(npf(W), bits, g))
    prepared = eq.eqat_qlinear_prepare(*eq.eqat_pack(W, s, z, bits, g), I, bits, g)
    ws = eq.workspace(eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16), eq.OP_QP_BWD, X.device)
    now, Y, out = s.clone(), torch.empty((T, O), dtype=X.dtype, device="cuda"), {}

    def step(sd, w):
        eq.eqat_qlinear_fwd_prepared(X, prepared, sd, O, bits, g, Y=Y, ws=w, keep=True)
        return eq.eqat_qlinear_bwd_prepared(X, prepared, sd, dY, I, bits, g, out=out, ws=w, kept=True)
    step(now, ws)
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        step(now, ws)
    for k in (1.0, 1.5, 0.5, 2.0):
        now.copy_(s * k)
        graph.replay()
        torch.cuda.synchronize()
        got = [Y.clone(), out["dX"].clone(), out["ds"].clone()]
        want = [eq.eqat_qlinear_fwd_prepared(X, prepared, now, O, bits, g)]
        alone = eq.eqat_qlinear_bwd_prepared(X, prepared, now, dY, I, bits, g)
        assert all(torch.equal(a, b) for a, b in zip(got, want + [alone["dX"], alone["ds"]]))

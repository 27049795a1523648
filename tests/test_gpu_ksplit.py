"""fwd / dX with few output tiles (k_gemm_ksplit; 256 x 256 tiles shared by workgroups): two K groups in a workgroup and up to four workgroups per tile.  Contraction
lengths that end in either group's K tile, odd numbers of K-tile pairs, ragged tiles, one to four parts; against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_11062_amd as eq
from paper_2407_11062_amd import synth
from test_gpu_parity import TOL, dev, make_case, npf, relerr
from test_workspace_parts import parts

pytestmark = pytest.mark.gpu

# tokens, in, out, group: dX contracts over out (parts of its tiles in the comment), the forward over in
CASES = [(70, 96, 40, 32),          # one pair
         (300, 352, 200, 32),       # two
         (1000, 4096, 264, 64),     # three pairs, 256 tiles
         (129, 512, 1480, 64),      # 3 parts, K ends inside the second group's tile
         (130, 256, 2056, 32),      # 4 parts, K ends inside the first group's tile, no second one
         (256, 1024, 3000, -1),     # 4 parts
         (600, 2048, 4096, 128),    # 3 parts, a last tile of 88 tokens
         (2560, 2048, 5504, 64),    # 80 tiles of 256 x 256, three workgroups each (the tile kernel)
         (2590, 2528, 10256, 32)]   # 110 of them, two each; K ends inside a K tile


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("T,I,O,g", CASES)
def test_dx_and_forward_with_few_tiles(T, I, O, g, bits):
    X, W, s, z, dY = make_case(("ksplit", T, I, O), T, I, O, bits, g, torch.bfloat16, torch.bfloat16)
    Xd, Wd, sd, zd, dYd = dev(X), dev(W), dev(s), dev(z), dev(dY)
    some = sorted({t for t in (0, 31, 32, 63, 64, 100, 127, 128, 191, 255, 256, 511, 512, T // 2, T - 2, T - 1) if 0 <= t < T})
    ws = eq.workspace(eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16), eq.OP_FQ_BWD, Xd.device)
    Y = eq.eqat_fq_linear_fwd(Xd, Wd, sd, zd, bits, g, ws=ws, keep=True)
    dX = eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, want=("dX",), ws=ws, kept=True)["dX"]
    ref = oracle.fq_linear_bwd(None, npf(W), s.numpy(), z.numpy(), npf(dY)[some], bits, g, want=("dX",))["dX"]
    assert relerr(dX[some], ref) <= TOL[torch.bfloat16]
    assert relerr(Y[some], oracle.fq_linear_fwd(npf(X)[some], npf(W), s.numpy(), z.numpy(), bits, g)) <= TOL[torch.bfloat16]
    # the counters of shared tiles are back at zero, the sum of the parts does not depend on who came last
    for _ in range(3):
        again = eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, want=("dX",), ws=ws, kept=True)["dX"]
        assert torch.equal(dX, again)
    # a prepared layer, whose counters live with it; zero points rounded into their range are those of Eq. (1) here
    Wp, zp = eq.eqat_pack(Wd, sd, zd, bits, g)
    prepared = eq.eqat_qlinear_prepare(Wp, zp, I, bits, g)
    for _ in range(2):
        assert torch.equal(dX, eq.eqat_qlinear_bwd_prepared(Xd, prepared, sd, dYd, I, bits, g, want=("dX",))["dX"])
    # a non-finite token stays where it is
    dYb = dYd.clone()
    dYb[T // 2] = float("nan")
    rest = [t for t in range(T) if t != T // 2]
    assert torch.equal(eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYb, bits, g, want=("dX",), ws=ws, kept=True)["dX"][rest], dX[rest])


@pytest.mark.parametrize("T,I,O,g", [(130, 256, 2056, 32), (600, 2048, 4096, 128), (2560, 2048, 5504, 64)])
def test_without_room_for_parts_the_tiles_are_not_shared(T, I, O, g):
    """A workspace that was sized for another token count: the same results but for the order of the sums."""
    bits = 2
    X, W, s, z, dY = make_case(("noroom", T, I, O), T, I, O, bits, g, torch.bfloat16, torch.bfloat16)
    Xd, Wd, sd, zd, dYd = dev(X), dev(W), dev(s), dev(z), dev(dY)
    some = sorted({0, 31, 32, 63, 64, 127, T // 2, T - 1})
    ref = oracle.fq_linear_bwd(None, npf(W), s.numpy(), z.numpy(), npf(dY)[some], bits, g, want=("dX",))["dX"]
    Yref = oracle.fq_linear_fwd(npf(X)[some], npf(W), s.numpy(), z.numpy(), bits, g)
    first, end = parts(T, I, O, eq.OP_FQ_BWD, 1, 256, 1 << 30, bits, g)
    assert end > first
    for room in (0, (end - first) // 2):
        guard = torch.full((first + room + 4096,), 0xA5, dtype=torch.uint8, device=Xd.device)
        ws = guard[:first + room]
        Y = eq.eqat_fq_linear_fwd(Xd, Wd, sd, zd, bits, g, ws=ws, keep=True)
        dX = eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, want=("dX",), ws=ws, kept=True)["dX"]
        assert relerr(dX[some], ref) <= TOL[torch.bfloat16] and relerr(Y[some], Yref) <= TOL[torch.bfloat16]
        assert bool((guard[first + room:] == 0xA5).all())
        assert torch.equal(dX, eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, want=("dX",), ws=ws, kept=True)["dX"])

"""fwd / dX with few output tiles (k_gemm_ksplit; 256 x 256 tiles shared by workgroups): two K groups in a workgroup and up to four workgroups per tile.  Contraction
lengths that end in either group's K tile, odd numbers of K-tile pairs, ragged tiles, one to four parts; against the oracle."""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_11062_amd as eq
from paper_2407_11062_amd import synth
from test_fwd_route import TILES, WORK, route
from test_gpu_mid_dx import dx_route
from test_gpu_parity import TOL, dev, make_case, npf, relerr
from test_shared_tiles_plan import parts_of
from test_work_plan import items_of_launch
from test_workspace_parts import parts

pytestmark = pytest.mark.gpu

# tokens, in, out, group, and what dX asked for alone, which contracts over out, runs on: workgroups per tile of k_gemm_ksplit; the tile kernel (edge
# of its tiles, numbers of workgroups per tile that occur); or None: k_gemm_mid_dx, and the row is there for its forward
CASES = [(70, 96, 40, 32, None),       # the forward: one pair
         (300, 352, 200, 32, None),    # three
         (330, 1120, 256, 32, None),
         (1000, 4096, 40, 32, 1),      # one pair, 256 tiles
         (1000, 4096, 200, 32, 1),     # two
         (1000, 4096, 264, 64, 1),     # three
         (129, 512, 1480, 64, 3),      # K ends inside the second group's tile
         (130, 256, 2056, 32, 4),      # K ends inside the first group's tile, no second one
         (256, 1024, 3000, -1, 4),
         (600, 2048, 4096, 128, 3),    # a last tile of 88 tokens
         (200, 12000, 128, 32, (128, 1)),                   # two whole K tiles
         (1000, 4096, 256, 32, (128, 1)),                   # four
         (2560, 2048, 5504, 64, (256, 3)),                  # 80 tiles
         (2590, 2528, 10256, 32, (128, 1)),                 # 420 tiles; K ends inside a K tile
         (2590, 2528, 12296, 32, (256, 2)),                 # 110 tiles; K ends inside a K tile
         # more than 256 tiles: one each, the rest split; with pieces of a K tile and without; and in runs
         (4400, 4128, 2056, 32, (256, 1, 4, 5)), (4400, 4128, 2048, 32, (256, 1, 4, 5)), (4400, 5920, 1032, 32, (256, 1, 2)),
         (4096, 2048, 2304, 128, (128, 1)), (4400, 8224, 200, 32, (256, 1))]          # 512 small tiles; 594 big ones, several for a workgroup


def assert_way(T, I, O, gemm, bits, g, way):
    other = gemm == 1 and dx_route(T, I, O, bits, g, True)[0]
    if way is None:
        assert other
        return
    assert not other
    if isinstance(way, int):
        assert parts_of(T, I, O, gemm, bits, g) == way
    else:
        items, _, _, tiles_m, tiles_n = items_of_launch(T, I, O, gemm)
        edge, *parts = way
        assert parts_of(T, I, O, gemm, bits, g) == 0 and {it[4] for _, _, it in items} == set(parts)
        assert (tiles_m, tiles_n) == (-(-T // edge), -(-(I if gemm else O) // edge))


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("T,I,O,g,way", CASES)
def test_dx_and_forward_with_few_tiles(T, I, O, g, way, bits):
    assert_way(T, I, O, 1, bits, g, way)
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
    """A workspace that was sized for another token count: the same results but for the order of the sums.  dX of the first is shared by fewer
    workgroups in half the room; where none are shared, the first two run in k_gemm_mid_dx (at most 128 tiles of 128 x 128 are ever shared, which are at most 256 of
    its 64-token tiles, and those are always estimated faster than one workgroup of k_gemm_ksplit per tile), the third on 128 x 128 tiles."""
    bits = 2
    X, W, s, z, dY = make_case(("noroom", T, I, O), T, I, O, bits, g, torch.bfloat16, torch.bfloat16)
    Xd, Wd, sd, zd, dYd = dev(X), dev(W), dev(s), dev(z), dev(dY)
    some = sorted({0, 31, 32, 63, 64, 127, T // 2, T - 1})
    ref = oracle.fq_linear_bwd(None, npf(W), s.numpy(), z.numpy(), npf(dY)[some], bits, g, want=("dX",))["dX"]
    Yref = oracle.fq_linear_fwd(npf(X)[some], npf(W), s.numpy(), z.numpy(), bits, g)
    first, end = parts(T, I, O, eq.OP_FQ_BWD, 1, 256, 1 << 30, bits, g)
    assert end > first
    for room in (0, (end - first) // 2):
        at, past = parts(T, I, O, eq.OP_FQ_BWD, 1, 256, first + room, bits, g)
        assert at == first and past - at == (room if T == 130 else 0)
        guard = torch.full((first + room + 4096,), 0xA5, dtype=torch.uint8, device=Xd.device)
        ws = guard[:first + room]
        Y = eq.eqat_fq_linear_fwd(Xd, Wd, sd, zd, bits, g, ws=ws, keep=True)
        dX = eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, want=("dX",), ws=ws, kept=True)["dX"]
        assert relerr(dX[some], ref) <= TOL[torch.bfloat16] and relerr(Y[some], Yref) <= TOL[torch.bfloat16]
        assert bool((guard[first + room:] == 0xA5).all())
        assert torch.equal(dX, eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, want=("dX",), ws=ws, kept=True)["dX"])


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("T,I,O,g,way", [(1, 2048, 264, 64, 4), (16, 1056, 1032, 32, 2), (7, 544, 72, -1, 1), (3, 256, 136, 32, (128, 1))])
def test_forward_of_a_few_tokens_on_a_prepared_layer(T, I, O, g, way, bits):
    """Up to 16 tokens only the packed arrays have matrix-vector kernels: shared tiles, with an odd number of pairs and a row that ends
    inside a K tile; two pairs of whole K tiles in the tile kernel."""
    assert_way(T, I, O, 0, bits, g, way)
    X, W, s, z, _ = make_case(("fewprep", T, I, O), T, I, O, bits, g, torch.bfloat16, torch.bfloat16)
    Xd, sd = dev(X), dev(s)
    Wp, zp = eq.eqat_pack(dev(W), sd, dev(z), bits, g)
    prepared = eq.eqat_qlinear_prepare(Wp, zp, I, bits, g)
    Y = eq.eqat_qlinear_fwd_prepared(Xd, prepared, sd, O, bits, g)
    assert relerr(Y, oracle.qlinear_fwd(npf(X), Wp.cpu().numpy(), s.numpy(), zp.cpu().numpy(), bits, g)) <= TOL[torch.bfloat16]
    for _ in range(2):
        assert torch.equal(Y, eq.eqat_qlinear_fwd_prepared(Xd, prepared, sd, O, bits, g))


# the forward on 128 x 128 tiles of the tile kernel (257 to 512 of them that k_gemm_mid leaves), whole K tiles and pieces of one
@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("T,I,O,g", [(2200, 352, 2056, 32), (2048, 512, 2176, 64), (1100, 2016, 5640, 96), (1999, 1920, 3304, -1)])
def test_forward_on_128_by_128_tiles(T, I, O, g, bits):
    assert route(T, I, O, bits, g, WORK)[0] == TILES
    assert_way(T, I, O, 0, bits, g, (128, 1))
    X, W, s, z, _ = make_case(("small tiles", T, I, O), T, I, O, bits, g, torch.bfloat16, torch.bfloat16)
    Xd, Wd, sd, zd = dev(X), dev(W), dev(s), dev(z)
    Y = eq.eqat_fq_linear_fwd(Xd, Wd, sd, zd, bits, g)
    some = sorted({t for e in range(0, T + 1, 128) for t in (e - 1, e, e + 33) if 0 <= t < T} | {T - 1})
    assert relerr(Y[some], oracle.fq_linear_fwd(npf(X)[some], npf(W), s.numpy(), z.numpy(), bits, g)) <= TOL[torch.bfloat16]
    Wp, zp = eq.eqat_pack(Wd, sd, zd, bits, g)
    assert torch.equal(Y, eq.eqat_qlinear_fwd(Xd, Wp, sd, zp, bits, g))


@pytest.mark.parametrize("bits,I,g", [(2, 3072, 1024), (2, 3104, -1), (2, 6144, -1)])
def test_forward_on_few_more_than_512_small_tiles(bits, I, g):
    """544 of them on 512 workgroups: one each, the rest split eight ways, with whole K tiles and with a piece of one at the end.  Without room
    for the parts the big tiles take it."""
    T, O = 4350, 2040
    first, end = parts(T, I, O, eq.OP_FQ_FWD, 0, 256, 1 << 30, bits, g)
    assert end - first == 512 * 128 * 128 * 4
    X, W, s, z, _ = make_case(("544", I), T, I, O, bits, g, torch.bfloat16, torch.bfloat16)
    Xd, Wd, sd, zd = dev(X), dev(W), dev(s), dev(z)
    some = sorted({t for e in range(0, T + 1, 512) for t in (e - 1, e, e + 33) if 0 <= t < T} | {T - 1})
    ref = oracle.fq_linear_fwd(npf(X)[some], npf(W), s.numpy(), z.numpy(), bits, g)
    for n in (end, first):
        guard = torch.full((n + 4096,), 0xA5, dtype=torch.uint8, device=Xd.device)
        Y = eq.eqat_fq_linear_fwd(Xd, Wd, sd, zd, bits, g, ws=guard[:n])
        assert relerr(Y[some], ref) <= TOL[torch.bfloat16]
        assert torch.equal(Y, eq.eqat_fq_linear_fwd(Xd, Wd, sd, zd, bits, g, ws=guard[:n]))
        assert bool((guard[n:] == 0xA5).all())
    assert torch.equal(eq.eqat_fq_linear_fwd(Xd, Wd, sd, zd, bits, g), eq.eqat_fq_linear_fwd(Xd, Wd, sd, zd, bits, g, ws=torch.empty(end, dtype=torch.uint8, device=Xd.device)))

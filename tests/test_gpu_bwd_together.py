"""dX and dW of one backward in one launch, with every kernel that computes dX there: dX against the oracle; dW, ds and dz bitwise those of a call without dX
(which runs dW alone; tiles that it cuts along the tokens are cut alike in the common launch)."""
import pytest
import torch

import oracle
import paper_2407_11062_amd as eq
from test_gpu_mid_dx import dx_route
from test_gpu_parity import TOL, dev, make_case, npf, relerr
from test_work_plan import items_of_launch

pytestmark = pytest.mark.gpu

# tokens, in, out, group, what computes dX, whether dW cuts tiles
BLOCK_AP = [(269, 1280, 1072, 256, 64, False), (515, 4096, 2568, 32, 96, False), (864, 2208, 2384, 96, 128, False),
            (1710, 3328, 2072, 32, 1, False), (620, 8192, 2688, 128, 0, False), (2200, 4384, 4224, 32, 0, True), (2200, 4384, 4232, 32, 1, True)]
E2E = [(698, 1792, 3328, 128, 64, False), (515, 4096, 4096, -1, 96, False), (459, 4608, 5504, 32, 128, False),
       (277, 2304, 3464, 256, 64, False), (1090, 8704, 5376, 64, 0, False), (2926, 1536, 4304, 96, 1, False),
       (2448, 14112, 1392, 32, 1, True), (2200, 4384, 4224, 32, 0, True)]


def cuts_dw(T, I, O):
    return any(it[4] > 1 for _, _, it in items_of_launch(T, I, O, 2)[0])


@pytest.mark.parametrize("bits,wdt", [(2, torch.bfloat16), (3, torch.float32), (4, torch.bfloat16), (2, torch.float32), (4, torch.float32)])
@pytest.mark.parametrize("T,I,O,g,dx,cut", BLOCK_AP)
def test_block_ap(T, I, O, g, dx, cut, bits, wdt):
    assert (dx_route(T, I, O, bits, g, True, eq.F32 if wdt == torch.float32 else eq.BF16)[1], cuts_dw(T, I, O)) == (dx, cut)
    X, W, s, z, dY = make_case(("together", T, I, O), T, I, O, bits, g, torch.bfloat16, wdt)
    Xd, Wd, sd, zd, dYd = dev(X), dev(W), dev(s), dev(z), dev(dY)
    ws = eq.workspace(eq.make_desc(T, I, O, bits, g, eq.BF16, eq._dt(Wd)), eq.OP_FQ_BWD, Xd.device)
    alone = eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, want=("dW", "ds", "dz"), ws=ws)
    some = sorted({t for t in (0, 31, 63, 64, 95, 96, 127, 128, 255, 256, T // 2, T - 1) if t < T})
    ref = oracle.fq_linear_bwd(None, npf(W), s.numpy(), z.numpy(), npf(dY)[some], bits, g, want=("dX",))["dX"]
    for _ in range(2):                                # the counters of cut tiles are back at zero
        both = eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, ws=ws)
        assert all(torch.equal(both[k], alone[k]) for k in alone)
        assert relerr(both["dX"][some], ref) <= TOL[torch.bfloat16]


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("T,I,O,g,dx,cut", E2E)
def test_e2e(T, I, O, g, dx, cut, bits):
    assert (dx_route(T, I, O, bits, g, False)[1], cuts_dw(T, I, O)) == (dx, cut)
    X, W, s, z, dY = make_case(("together", T, I, O), T, I, O, bits, g, torch.bfloat16, torch.bfloat16)
    Xd, sd, dYd = dev(X), dev(s), dev(dY)
    Wp, zp = eq.eqat_pack(dev(W), sd, dev(z), bits, g)
    prepared = eq.eqat_qlinear_prepare(Wp, zp, I, bits, g)
    zf = (dev(z).clamp(0, 2 ** bits - 1) + 0.25).contiguous()
    some = sorted({t for t in (0, 31, 63, 64, 95, 96, 127, 128, 255, 256, T // 2, T - 1) if t < T})
    alone = eq.eqat_qlinear_bwd_prepared(Xd, prepared, sd, dYd, I, bits, g, z=zf, want=("ds", "dz"))
    both = eq.eqat_qlinear_bwd_prepared(Xd, prepared, sd, dYd, I, bits, g, z=zf, want=("dX", "ds", "dz"))
    ref = oracle.qlinear_bwd_z(None, Wp.cpu().numpy(), s.numpy(), npf(zf), npf(dY)[some], I, bits, g, want=("dX",))["dX"]
    assert torch.equal(both["ds"], alone["ds"]) and torch.equal(both["dz"], alone["dz"])
    assert relerr(both["dX"][some], ref) <= TOL[torch.bfloat16]
    again = eq.eqat_qlinear_bwd_prepared(Xd, prepared, sd, dYd, I, bits, g, z=zf, want=("dX", "ds", "dz"))
    assert all(torch.equal(again[k], both[k]) for k in both)


@pytest.mark.parametrize("g", [96, 256])
def test_few_partials_are_summed_alike_whatever_their_number(g):
    """ds and dz of a row do not depend on how many rows there are (one lane of k_reduce_partials per group or four), with three and eight partials."""
    T, I, O, few, bits = 40, 768, 24000, 1000, 2
    X, W, s, z, dY = make_case(("fewpartials", g), T, I, O, bits, g, torch.bfloat16, torch.bfloat16)
    Xd, Wd, sd, zd, dYd = dev(X), dev(W), dev(s), dev(z), dev(dY)
    for k in ("ds", "dz"):
        many = eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, want=(k,))[k]
        some = eq.eqat_fq_linear_bwd(Xd, Wd[:few].contiguous(), sd[:few].contiguous(), zd[:few].contiguous(), dYd[:, :few].contiguous(), bits, g, want=(k,))[k]
        ref = oracle.fq_linear_bwd(npf(X), npf(W)[:few], s.numpy()[:few], z.numpy()[:few], npf(dY)[:, :few], bits, g, want=(k,))[k]
        assert torch.equal(many[:few], some) and relerr(some, ref) <= TOL[torch.bfloat16]

"""dX for few output tiles (k_gemm_mid_dx) against the oracle: every token tile, in one round of workgroups and two, ragged in tokens, in-features and the
contraction (ends of a 128-wide step, of a wave's quarter of it, of 8), one step and many, groups inside, across and beyond a wave's 64 columns."""
import ctypes

import pytest
import torch

import oracle
import paper_2407_11062_amd as eq
from test_gpu_parity import TOL, dev, make_case, npf, relerr

pytestmark = pytest.mark.gpu

# tokens, in, out, group, token tile
CASES = [(1, 9216, 136, 32, 64), (65, 9216, 840, 64, 64), (1500, 1056, 264, 96, 64), (300, 5472, 1256, 32, 64), (130, 3232, 1096, -1, 64),
         (1040, 2176, 2056, 32, 96), (1041, 2208, 2160, 96, 96), (1000, 3584, 4104, 128, 128), (1000, 3616, 4216, 32, 128), (1000, 4096, 11016, 256, 128)]


def dx_route(T, I, O, bits, g, block_ap, w=eq.BF16):
    out = (ctypes.c_int32 * 2)()
    rc = eq.lib().eqat_dx_route(ctypes.byref(eq.make_desc(T, I, O, bits, g, eq.BF16, w)), int(block_ap), out)
    assert rc == 0, eq.lib().eqat_status_string(rc)
    return tuple(out)


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("T,I,O,g,tokens", CASES)
def test_dx_for_few_tiles(T, I, O, g, tokens, bits):
    assert dx_route(T, I, O, bits, g, True)[0] == tokens
    X, W, s, z, dY = make_case(("middx", T, I, O), T, I, O, bits, g, torch.bfloat16, torch.bfloat16)
    Wd, sd, zd, dYd = dev(W), dev(s), dev(z), dev(dY)
    some = sorted({t for t in (0, 31, 32, 63, 64, 95, 96, 127, 128, 255, 256, T // 2, T - 2, T - 1) if 0 <= t < T})
    ws = eq.workspace(eq.make_desc(T, I, O, bits, g, eq.BF16, eq.BF16), eq.OP_FQ_BWD, dYd.device)
    dX = eq.eqat_fq_linear_bwd(dev(X), Wd, sd, zd, dYd, bits, g, want=("dX",), ws=ws)["dX"]
    ref = oracle.fq_linear_bwd(None, npf(W), s.numpy(), z.numpy(), npf(dY)[some], bits, g, want=("dX",))["dX"]
    assert relerr(dX[some], ref) <= TOL[torch.bfloat16]
    Wp, zp = eq.eqat_pack(Wd, sd, zd, bits, g)
    prepared = eq.eqat_qlinear_prepare(Wp, zp, I, bits, g)
    out = torch.full((T + 1, I), 7.0, dtype=torch.bfloat16, device="cuda")           # nothing past the last row is written
    again = eq.eqat_qlinear_bwd_prepared(dev(X), prepared, sd, dYd, I, bits, g, want=("dX",), out={"dX": out[:T]})["dX"]
    assert torch.equal(dX, again) and bool((out[T] == 7.0).all())
    if T > 1:                                         # a non-finite token stays where it is, also where the next row begins inside a step
        dYb = dYd.clone()
        dYb[T // 2] = float("inf")
        rest = [t for t in range(T) if t != T // 2]
        got = eq.eqat_fq_linear_bwd(dev(X), Wd, sd, zd, dYb, bits, g, want=("dX",), ws=ws)["dX"]
        assert torch.equal(got[rest], dX[rest])

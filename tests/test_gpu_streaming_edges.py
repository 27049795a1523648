"""The streaming passes at the edges of what a lane, a wave and a workgroup take.

min/max: a piece of 16 bytes per lane (8 bf16, 4 fp32 weights), 4 or 8 runs of 64 pieces a wave, groups of 4 to 128 pieces; codes:
8 weights a lane, 8192 a workgroup.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_11062_amd as eq
from paper_2407_11062_amd import synth

pytestmark = pytest.mark.gpu


def npf(t):
    return t.detach().float().cpu().numpy()


# (out, in): less than one wave's pieces; a workgroup less, exactly and more than one; a last workgroup that is nearly empty
@pytest.mark.parametrize("wdt", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("g", [32, 64, 128, 256, 512])
@pytest.mark.parametrize("O,I", [(1, 512), (15, 512), (16, 512), (33, 512), (5, 7 * 512)])
def test_minmax_and_codes_exact(O, I, g, wdt):
    W = synth.normal((O, I), 0.02, synth.seed_of("edges", O, I, g), wdt)
    W.view(-1)[:: 97] = 0.0
    for bits in (2, 3, 4):
        s, z = eq.eqat_init_minmax(W.cuda(), bits, g)
        s_ref, z_ref = oracle.init_minmax(npf(W), bits, g)
        assert np.array_equal(npf(s), s_ref) and np.array_equal(npf(z), z_ref)
        zf = z_ref + 0.4
        got = eq.eqat_pack(W.cuda(), s, torch.from_numpy(zf).cuda(), bits, g)
        for a, b in zip(got, oracle.pack(npf(W), s_ref, zf, bits, g)):
            assert np.array_equal(a.cpu().numpy(), b)


@pytest.mark.parametrize("zbar", [0.0, 1.0, 3.0])
def test_codes_of_quotients_beyond_every_code(zbar):
    """|w / s| far past the code range, up to where the quotient is no longer an integer the float can tell from its neighbours, and infinite."""
    big = [2.0 ** k for k in range(0, 40)] + [2.0 ** 22 + 0.5, 2.0 ** 23 + 1.0, 3e38, np.inf]
    w = np.array(big + [-b for b in big] + [0.0, -0.0, 0.5, 1.5, 2.5, -0.5, -1.5, -2.5], np.float32)
    w = np.concatenate([w, np.zeros(-len(w) % 32, np.float32)])
    s, z = np.ones((1, 1), np.float32), np.full((1, 1), zbar, np.float32)
    Wp, zp = eq.eqat_pack(torch.from_numpy(w[None]).cuda(), torch.from_numpy(s).cuda(), torch.from_numpy(z).cuda(), 2, -1)
    codes = eq.eqat_unpack(Wp, zp, len(w), 2, -1)[0].cpu().numpy()[0]
    assert np.array_equal(codes, np.clip(np.rint(w) + zbar, 0, 3).astype(np.int32))

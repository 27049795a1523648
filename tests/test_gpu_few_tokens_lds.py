"""k_gemv_wide where a wave fetches its weights as row pieces straight into LDS (up to 8 tokens, long rows), and beside it
where the lanes fetch them.

Rows of a run less, a piece more, several runs a wave; the last run cut anywhere; row blocks cut; every number of groups in a run; zero points packed and as
floats, in words that begin in the middle of a run's.
"""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_11062_amd as eq
from paper_2407_11062_amd import synth

pytestmark = pytest.mark.gpu
TOL = 2e-2          # bf16 activations, as max|got - ref| / max|ref|


def npf(t):
    return t.detach().float().cpu().numpy()


# in-features: 512 a run; eight waves at most: 4608 is nine runs, two of them a wave's second
@pytest.mark.parametrize("T,bits", [(7, 2), (8, 2), (7, 3), (8, 4), (12, 3), (16, 3), (27, 3)])
@pytest.mark.parametrize("I,O,g", [(512, 16, 32), (480, 24, 32), (544, 40, 32), (576, 8, 64), (4608, 72, 64), (5120, 104, 128), (4736, 56, 128), (4864, 56, 256),
                                   (4608, 72, -1), (10752, 16, 384)])
def test_against_the_oracle(T, bits, I, O, g):
    W = synth.normal((O, I), 0.02, synth.seed_of("lds", I, O, g), torch.bfloat16)
    X = synth.normal((T, I), 1.0, synth.seed_of("lds", T, I), torch.bfloat16)
    s, z = oracle.init_minmax(npf(W), bits, g)
    Wp, zp = eq.eqat_pack(W.cuda(), torch.from_numpy(s).cuda(), torch.from_numpy(z).cuda(), bits, g)
    Xd, sd = X.cuda(), torch.from_numpy(s).cuda()
    Y = eq.eqat_qlinear_fwd(Xd, Wp, sd, zp, bits, g)
    ref = oracle.qlinear_fwd(npf(X), Wp.cpu().numpy(), s, zp.cpu().numpy(), bits, g)
    assert np.abs(npf(Y) - ref).max() <= TOL * np.abs(ref).max()
    assert torch.equal(Y, eq.eqat_qlinear_fwd(Xd, Wp, sd, zp, bits, g))
    assert torch.equal(Y, eq.eqat_qlinear_fwd_z(Xd, Wp, sd, torch.from_numpy(z).cuda(), bits, g))


def test_what_follows_a_row_never_counts():
    """infinite step sizes and zero points in the rows behind, which the last run of a row reaches into"""
    T, I, O, bits, g = 8, 544, 48, 3, 32
    W = synth.normal((O, I), 0.02, 3, torch.bfloat16)
    X = synth.normal((T, I), 1.0, 4, torch.bfloat16).cuda()
    s, z = oracle.init_minmax(npf(W), bits, g)
    Wp, _ = eq.eqat_pack(W.cuda(), torch.from_numpy(s).cuda(), torch.from_numpy(z).cuda(), bits, g)
    clean = eq.eqat_qlinear_fwd_z(X, Wp, torch.from_numpy(s).cuda(), torch.from_numpy(z).cuda(), bits, g)
    for bad in (np.inf, -np.inf, np.nan):
        s2, z2 = s.copy(), z.copy()
        s2[1::2], z2[1::2] = bad, bad
        Y = eq.eqat_qlinear_fwd_z(X, Wp, torch.from_numpy(s2).cuda(), torch.from_numpy(z2).cuda(), bits, g)
        assert torch.equal(Y[:, 0::2], clean[:, 0::2])


@pytest.mark.parametrize("I,g", [(8192, 32), (8192, 64), (8192 + 128, 128), (9216, -1)])
def test_large_matrices_of_4_bit_codes_as_their_parts(I, g):
    """codes as row pieces in the whole (more than 2^26 weights), by the lanes in the parts: the same sums"""
    T, O, bits = 8, (1 << 26) // I // 8 * 8 + 24, 4
    gen = torch.Generator(device="cuda").manual_seed(7)
    W = (torch.randn((O, I), generator=gen, device="cuda") * 0.02).bfloat16()
    X = torch.randn((T, I), generator=gen, device="cuda").bfloat16()
    s, z = eq.eqat_init_minmax(W, bits, g)
    Wp, zp = eq.eqat_pack(W, s, z, bits, g)
    Y = eq.eqat_qlinear_fwd(X, Wp, s, zp, bits, g)
    for a, b in ((0, 40), (O - 24, O)):
        assert torch.equal(Y[:, a:b], eq.eqat_qlinear_fwd(X, Wp[a:b].contiguous(), s[a:b].contiguous(), zp[a:b].contiguous(), bits, g))
    assert torch.equal(Y, eq.eqat_qlinear_fwd_z(X, Wp, s, z, bits, g))


# where 2- and 3-bit codes go through LDS: four runs or more, groups of 32 and 3 bit with float zero points in large matrices only.  Rows of whole runs and a segment, two, a piece more;
# row blocks cut; eight waves at most: 4608 is nine runs
@pytest.mark.parametrize("T,bits", [(7, 2), (8, 2), (7, 3), (8, 3)])
@pytest.mark.parametrize("I,O,g", [(2016, 24, 32), (2048, 16, 64), (2080, 24, 32), (2112, 40, 64), (2176, 8, -1), (2560, 56, 128), (4608, 72, 256), (8192, 24, 128), (8320, 40, 64),
                                   (10752, 16, 384), (4096, 8184, 32), (4096, 8200, 32), (4128, 8216, 32), (5120, 8200, 128)])
def test_both_ways_against_the_oracle(T, bits, I, O, g):
    test_against_the_oracle(T, bits, I, O, g)

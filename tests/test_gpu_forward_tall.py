"""Forward on 128-token tiles (k_gemm_mid_tall): edges of its tiles, of its 128-wide K steps and of the four steps whose step sizes
are fetched together, every way to find a group.  All tokens at tile edges against the oracle, every entry point bitwise."""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_11062_amd as eq
from paper_2407_11062_amd import synth
from test_fwd_route import FLOATZ, MID, PACKED, WORK, route
from test_gpu_parity import TOL, dev, make_case, npf, relerr

pytestmark = pytest.mark.gpu

CASES = [  # tokens, in, out, group: I % 128 = 0, 32, 64, 96 and I % 512 != 0; ragged last tiles of tokens and rows
    (1024, 4096, 4096, 64), (1001, 1696, 4000, 32), (2040, 1728, 2048, 64), (900, 1760, 4096, 32), (200, 2048, 16376, 128),
    (1024, 1536, 4096, 256), (1000, 2304, 4096, 384), (1010, 2688, 4000, -1),
]


@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("T,I,O,g", CASES)
def test_forward_on_128_token_tiles(T, I, O, g, bits):
    for source in (WORK, PACKED, FLOATZ):
        assert route(T, I, O, bits, g, source) == (MID, 128, 128)
    X, W, s, z, _ = make_case(("tall", T, I, O), T, I, O, bits, g, torch.bfloat16, torch.bfloat16)
    Xd, Wd, sd, zd = dev(X), dev(W), dev(s), dev(z)
    Wp, zp = eq.eqat_pack(Wd, sd, zd, bits, g)
    zf = (z + synth.uniform(tuple(z.shape), -0.6, 0.6, synth.seed_of("tall", T))).contiguous()
    prepared = eq.eqat_qlinear_prepare(Wp, zp, I, bits, g)
    Y, Yz = eq.eqat_qlinear_fwd(Xd, Wp, sd, zp, bits, g), eq.eqat_qlinear_fwd_z(Xd, Wp, sd, dev(zf), bits, g)
    assert torch.equal(Y, eq.eqat_fq_linear_fwd(Xd, Wd, sd, zd, bits, g))
    assert torch.equal(Y, eq.eqat_qlinear_fwd_prepared(Xd, prepared, sd, O, bits, g))
    assert torch.equal(Yz, eq.eqat_qlinear_fwd_prepared(Xd, prepared, sd, O, bits, g, z=dev(zf)))
    # the oracle on tokens at the edges of blocks and tiles; What, a bf16 rounding of 2^-9, enters every product
    some = sorted({t for e in range(0, T + 1, 128) for t in (e - 1, e, e + 33) if 0 <= t < T} | {T - 1})[:24] + [T - 1]
    Xs, Wpn = npf(X)[some], Wp.cpu().numpy()
    assert relerr(Y[some], oracle.qlinear_fwd(Xs, Wpn, s.numpy(), zp.cpu().numpy(), bits, g)) <= TOL[torch.bfloat16]
    assert relerr(Yz[some], oracle.qlinear_fwd_z(Xs, Wpn, s.numpy(), zf.numpy(), bits, g)) <= TOL[torch.bfloat16]
    # a non-finite token, and a non-finite step size, stay where they are
    Xb = Xd.clone()
    Xb[T // 2] = float("inf")
    rest = [t for t in range(T) if t != T // 2]
    assert torch.equal(eq.eqat_qlinear_fwd(Xb, Wp, sd, zp, bits, g)[rest], Y[rest])
    sb = sd.clone()
    sb[1::2] = float("nan")
    assert torch.equal(eq.eqat_qlinear_fwd(Xd, Wp, sb, zp, bits, g)[:, 0::2], Y[:, 0::2])


@pytest.mark.parametrize("bits,g", [(2, 32), (3, 96), (4, 64)])
@pytest.mark.parametrize("T,O", [(1281, 1016), (1345, 136), (1850, 1016), (1990, 1000), (2700, 776)])
def test_forward_in_bands_of_token_tiles(T, O, bits, g):
    """More than 20 token tiles, in bands of unequal height: every tile is written once, at its own place."""
    I = 2880
    kind, tokens, _ = route(T, I, O, bits, g, PACKED)
    assert kind == MID and -(-T // tokens) > 20
    X, W, s, z, _ = make_case(("bands", T, O), T, I, O, bits, g, torch.bfloat16, torch.bfloat16)
    Xd, sd = dev(X), dev(s)
    Wp, zp = eq.eqat_pack(dev(W), sd, dev(z), bits, g)
    Y = eq.eqat_qlinear_fwd(Xd, Wp, sd, zp, bits, g)
    some = sorted({t for e in range(0, T + 1, 64) for t in (e - 1, e) if 0 <= t < T} | {T - 1})
    assert relerr(Y[some], oracle.qlinear_fwd(npf(X)[some], Wp.cpu().numpy(), s.numpy(), zp.cpu().numpy(), bits, g)) <= TOL[torch.bfloat16]
    # few tokens at a time have no bands; sums in another order differ by fp32 roundings before the one to bf16 (2^-8 of an output)
    for t in range(0, T, 640):
        few = eq.eqat_qlinear_fwd(Xd[t:t + 640], Wp, sd, zp, bits, g).float()
        assert (Y[t:t + 640].float() - few).abs().max() <= 2.0 ** -7 * few.abs().max()

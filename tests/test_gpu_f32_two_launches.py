"""The fp32 backward in two launches (few tiles, What beside dWhat in the workspace) against the same call in a workspace without room for What,
which takes the four launches in a row: the same sums in the same order, bitwise."""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_11062_amd as eq
from test_gpu_parity import dev, make_case, npf, relerr

pytestmark = pytest.mark.gpu

# remainders of the 32 x 32 tiles, the smallest out-feature count that reads What from memory, 240 and 256 tiles of 64 x 64 (the last one: four launches)
SHAPES = [(1, 32, 33, 32), (31, 96, 40, 96), (65, 160, 72, 32), (257, 512, 520, 128), (960, 1024, 64, -1), (1024, 1024, 64, 256)]


@pytest.mark.parametrize("T,I,O,g", SHAPES)
@pytest.mark.parametrize("bits,wdt", [(2, torch.float32), (3, torch.bfloat16), (4, torch.float32)])
def test_two_launches_equal_four(T, I, O, g, bits, wdt):
    X, W, s, z, dY = make_case(("f32two", T, I, O, bits), T, I, O, bits, g, torch.float32, wdt)
    s[::5, 0] = 2.0 ** -127                           # a denormal step size: quotients divided out, in both ways (that they are right: test_codes_near_rounding_ties)
    Xd, Wd, sd, zd, dYd = dev(X), dev(W), dev(s), dev(z), dev(dY)
    full = eq.workspace(eq.make_desc(T, I, O, bits, g, eq.F32, eq._dt(Wd)), eq.OP_FQ_BWD, Xd.device)
    room = O * I * 4
    assert (full.numel() > room + 256) == (T != 1024)
    small = full[:(room + 255) // 256 * 256].clone()
    full.fill_(0xFF)
    small.fill_(0xFF)
    got = eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, ws=full)
    want = eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, ws=small)
    for k in ("dX", "dW", "ds", "dz"):
        assert torch.equal(got[k], want[k]), k
    s[::5, 0] = s[::5, -1] if s.shape[1] > 1 else 0.01
    sd = dev(s)
    got = eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, ws=full)
    if T * I * O < 1 << 25:
        ref = oracle.fq_linear_bwd(npf(X), npf(W), s.numpy(), z.numpy(), npf(dY), bits, g)
        for k in ("dX", "ds", "dz"):
            assert relerr(got[k], ref[k]) <= 1e-5, k
        assert relerr(got["dW"], ref["dW"]) <= (1e-5 if wdt == torch.float32 else 2e-2)
        assert relerr(eq.eqat_fq_linear_fwd(Xd, Wd, sd, zd, bits, g), oracle.fq_linear_fwd(npf(X), npf(W), s.numpy(), z.numpy(), bits, g)) <= 1e-5
    Wp, zp = eq.eqat_pack(Wd, sd, zd, bits, g)
    got = eq.eqat_qlinear_bwd(Xd, Wp, sd, zp, dYd, I, bits, g)
    ws = eq.workspace(eq.make_desc(T, I, O, bits, g, eq.F32, eq.BF16), eq.OP_Q_BWD, Xd.device)
    less = ws[: ws.numel() - room].clone() if T != 1024 else ws
    want = eq.eqat_qlinear_bwd(Xd, Wp, sd, zp, dYd, I, bits, g, ws=less)
    assert torch.equal(got["dX"], want["dX"]) and torch.equal(got["ds"], want["ds"])


# contractions of one, three and five blocks of 32 per wave (eight waves), whole and with a remainder, along the tokens (dW) and the rows (dX)
@pytest.mark.parametrize("T,I,O", [(545, 64, 40), (768, 32, 250), (40, 64, 545), (256, 32, 768), (1025, 96, 36), (36, 96, 1025)])
def test_blocks_loaded_ahead(T, I, O):
    X, W, s, z, dY = make_case(("f32ahead", T, I, O), T, I, O, 3, 32, torch.float32, torch.float32)
    got = eq.eqat_fq_linear_bwd(dev(X), dev(W), dev(s), dev(z), dev(dY), 3, 32)
    ref = oracle.fq_linear_bwd(npf(X), npf(W), s.numpy(), z.numpy(), npf(dY), 3, 32)
    for k in ("dX", "dW", "ds", "dz"):
        assert relerr(got[k], ref[k]) <= 1e-5, k


@pytest.mark.parametrize("wdt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("bits", [2, 3, 4])
def test_codes_near_rounding_ties(bits, wdt):
    """Forward and dX multiply by a reciprocal and divide only near a tie: weights on every tie of their group and a few ulp beside it, and step sizes whose
    reciprocal is no normal number.  One-hot tokens (a power of two) bring single weights out: each must be the one of the exact quotient, to the bit."""
    I, O, g, qmax = 256, 72, 32, 2 ** bits - 1
    rng = np.random.default_rng(40 + bits)
    z = rng.integers(0, qmax + 1, (O, I // g)).astype(np.float32)
    k = (rng.integers(-1, qmax + 1, (O, I)) - np.repeat(z, g, 1) + 0.5).astype(np.float32)       # the ties around codes -1 .. qmax + 1
    scale = np.exp2(rng.integers(-14, -4, (O, I // g))).astype(np.float32)
    if wdt == torch.bfloat16:                         # bf16 holds k s exactly for step sizes of 3 bits: these are moved
        s = rng.integers(4, 8, (O, I // g)).astype(np.float32) * scale
        W = k * np.repeat(s, g, 1)
        s = (s.view(np.int32) + rng.integers(-2, 3, s.shape).astype(np.int32)).view(np.float32)
    else:
        s = rng.uniform(1, 2, (O, I // g)).astype(np.float32) * scale
        W = k * np.repeat(s, g, 1)
        W = (W.view(np.int32) + rng.integers(-2, 3, W.shape).astype(np.int32)).view(np.float32)
    assert torch.equal(torch.from_numpy(W).to(wdt).float(), torch.from_numpy(W))
    sw = np.repeat(s, g, 1)
    off = np.rint(W * (np.float32(1) / sw)) != np.rint(W / sw)
    assert off.mean() > 0.01                          # what the reciprocal alone would round the other way
    # no normal reciprocal: a denormal step size, and ones beyond 2^126 (of zero point 0 and code 1 at most, so that the weight is finite)
    s[3, 1], s[5, 2], s[7, 3] = 2.0 ** -127, 1.5 * 2.0 ** 126, 2.0 ** 127
    for o, j in ((3, 1), (5, 2), (7, 3)):
        z[o, j] = 0.0
        W[o, j * g:(j + 1) * g] = np.linspace(-1.25, 1.25, g).astype(np.float32).round(2) * s[o, j]
    W = torch.from_numpy(W).to(wdt)
    codes, _ = oracle.quantize(npf(W), s, z, bits, g)
    assert all(set(codes[o, j * g:(j + 1) * g]) == {0, 1} for o, j in ((3, 1), (5, 2), (7, 3)))
    one = np.full((O, 1), 2.0 ** -30, np.float32)     # of the token that brings row o out; the products of denormal weights are normal ones
    one[3] = 2.0 ** 100
    what = (codes - np.repeat(z, g, 1)).astype(np.float32) * np.repeat(s, g, 1)
    Wd, sd, zd = dev(W), dev(torch.from_numpy(s)), dev(torch.from_numpy(z))
    dX = eq.eqat_fq_linear_bwd(torch.zeros((O, I), device="cuda"), Wd, sd, zd, dev(torch.from_numpy(np.diag(one[:, 0]))), bits, g)["dX"]
    Y = eq.eqat_fq_linear_fwd(dev(torch.eye(I) * 2.0 ** -30), Wd, sd, zd, bits, g)
    assert np.array_equal(dX.cpu().numpy(), what * one)
    rows = [o for o in range(O) if o != 3]
    assert np.array_equal(Y.cpu().numpy().T[rows], what[rows] * np.float32(2.0 ** -30))

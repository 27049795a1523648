"""dW, ds and dz where the choice between its two tiles changes (270-odd big tiles of short batches, 130 to 159 of longer ones), with
ragged edges, groups inside a tile and across tiles; against the oracle on rows at the edges of tiles."""
import pytest
import torch

import oracle
import paper_2407_11062_amd as eq
from test_gpu_parity import TOL, dev, make_case, npf, relerr
from test_work_plan import items_of_launch

pytestmark = pytest.mark.gpu

CASES = [  # tokens, in, out, group, tile
    (515, 2592, 6600, 32, 128),        # 286 big tiles, 1092 small ones
    (65, 2816, 6000, 128, 128),        # 264; one pair of K tiles, the second of one token
    (2048, 4096, 4352, -1, 128),       # 272, the most tokens; 64 small ones are split
    (2049, 4096, 4352, 64, 256),
    (300, 4096, 5128, 64, 256),        # 336
    (576, 2816, 3000, 256, 128),       # 132
    (577, 2816, 3000, 256, 256),
    (2049, 2784, 3064, 96, 128),       # 132, long; 16 small ones are split
    # W rows past the caches from more than 24 MB on: bf16, then fp32
    (90, 3072, 4096, 64, 256),
    (90, 3072, 4104, 64, 256),
    (90, 2048, 3072, 64, 128),
    (90, 2048, 3080, 64, 128),
]


@pytest.mark.parametrize("bits,wdt", [(2, torch.bfloat16), (3, torch.float32), (4, torch.bfloat16)])
@pytest.mark.parametrize("T,I,O,g,tile", CASES)
def test_weight_gradients_on_either_tile(T, I, O, g, tile, bits, wdt):
    assert items_of_launch(T, I, O, 2)[3] == -(-I // tile)
    X, W, s, z, dY = make_case(("dwtiles", T, I, O), T, I, O, bits, g, torch.bfloat16, wdt)
    Xd, Wd, sd, zd, dYd = dev(X), dev(W), dev(s), dev(z), dev(dY)
    got = eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, want=("dW", "ds", "dz"))
    rows = sorted({r for e in range(0, O + 1, 128) for r in (e - 1, e, e + 40) if 0 <= r < O} | {O - 1})
    ref = oracle.fq_linear_bwd(npf(X), npf(W)[rows], s.numpy()[rows], z.numpy()[rows], npf(dY)[:, rows], bits, g, want=("dW", "ds", "dz"))
    for k in ("dW", "ds", "dz"):
        assert relerr(got[k][rows], ref[k]) <= TOL[torch.bfloat16], k
    # the split tiles' counters are back at zero
    again = eq.eqat_fq_linear_bwd(Xd, Wd, sd, zd, dYd, bits, g, want=("dW", "ds", "dz"))
    assert all(torch.equal(got[k], again[k]) for k in got)
    # step sizes alone, on a prepared layer
    Wp, zp = eq.eqat_pack(Wd, sd, zd, bits, g)
    prepared = eq.eqat_qlinear_prepare(Wp, zp, I, bits, g)
    ds = eq.eqat_qlinear_bwd_prepared(Xd, prepared, sd, dYd, I, bits, g, want=("ds",))["ds"]
    want = oracle.qlinear_bwd(npf(X), Wp.cpu().numpy()[rows], s.numpy()[rows], zp.cpu().numpy()[rows], npf(dY)[:, rows], I, bits, g, want=("ds",))["ds"]
    assert relerr(ds[rows], want) <= TOL[torch.bfloat16]

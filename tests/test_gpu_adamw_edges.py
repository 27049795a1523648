"""AdamW at the edges of its workgroups, 2048 elements each, four to an access, and of the size from which accesses pass the caches by."""
import numpy as np
import pytest
import torch

import oracle
import paper_2407_11062_amd as eq
from paper_2407_11062_amd import synth

pytestmark = pytest.mark.gpu


def npf(t):
    return t.detach().float().cpu().numpy()


@pytest.mark.parametrize("wdt", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("O,I", [(1, 32), (63, 32), (64, 32), (65, 32), (67, 96)])
def test_adamw_where_workgroups_end(O, I, wdt):
    g = 32
    t = {k: synth.normal((O, I), std, synth.seed_of("adam edge", O, I, k)) for k, std in (("W", 0.02), ("dW", 1e-2), ("mW", 1e-3))}
    W, dW, m = t["W"].to(wdt), t["dW"].to(wdt), t["mW"]
    v = m.square() + 1e-8
    f = lambda x: float(np.float32(x))          # the constants as the C ABI takes them
    ref = oracle.adamw(npf(W), npf(dW), npf(m), npf(v), f(1e-3), f(0.9), f(0.999), f(1e-8), f(0.1), 3)
    Wd, md, vd = W.cuda(), m.cuda(), v.cuda()
    eq.eqat_block_ap_update(eq.AdamW(1e-3, 1e-4, 0.9, 0.999, 1e-8, 0.1, 0.0, 3), 2, g, W=Wd, dW=dW.cuda(), mW=md, vW=vd)
    for got, want, tol in ((Wd, ref[0], 1e-5 if wdt == torch.float32 else 2 ** -8), (md, ref[1], 1e-5), (vd, ref[2], 1e-5)):
        assert np.abs(npf(got) - want).max() <= tol * np.abs(want).max()


# one group to a row: as many step sizes as rows.  Less than four; the last four cut; a workgroup less, exactly and more than one; the last access of a workgroup alone
@pytest.mark.parametrize("O", [1, 3, 5, 1023, 1024, 1025, 1030, 2047, 2048, 2051, 3073])
def test_step_sizes_and_zero_points_where_workgroups_end(O):
    t = {k: synth.normal((O, 1), std, synth.seed_of("adam groups", O, k)) for k, std in (("ds", 1e-2), ("ms", 1e-3), ("dz", 1e-2), ("mz", 1e-3))}
    p = {"s": synth.uniform((O, 1), 0.01, 0.05, synth.seed_of("adam groups", O, "s")), "z": synth.uniform((O, 1), 0.0, 3.0, synth.seed_of("adam groups", O, "z"))}
    f = lambda x: float(np.float32(x))
    d = {k: v.cuda() for k, v in {**t, **p, "vs": t["ms"].square() + 1e-8, "vz": t["mz"].square() + 1e-8}.items()}
    eq.eqat_block_ap_update(eq.AdamW(1e-3, 1e-4, 0.9, 0.999, 1e-8, 0.1, 0.0, 3), 2, -1, shape=(O, 32), **d)
    for k in "sz":
        m = t["m" + k]
        ref = oracle.adamw(npf(p[k]), npf(t["d" + k]), npf(m), npf(m.square() + 1e-8), f(1e-4), f(0.9), f(0.999), f(1e-8), f(0.0), 3, f(1e-10) if k == "s" else -np.inf)
        for got, want in zip((d[k], d["m" + k], d["v" + k]), ref):
            assert np.abs(npf(got) - want).max() <= 1e-5 * np.abs(want).max()


# Parameters, gradients and moments of 88 MB in all, 16 bytes a weight (bf16: 12), are where accesses begin to pass the caches by.
@pytest.mark.parametrize("wdt,below,above", [(torch.float32, 2401, 2403), (torch.bfloat16, 3203, 3205)])
def test_update_on_both_sides_of_the_size_that_passes_the_caches_by(wdt, below, above):
    I, limit, each = 2400, 88 << 20, 16 if wdt == torch.float32 else 12
    assert below * I * each <= limit < above * I * each
    gen = torch.Generator(device="cuda").manual_seed(11)
    W = (torch.randn((above, I), generator=gen, device="cuda") * 0.02).to(wdt)
    dW = (torch.randn((above, I), generator=gen, device="cuda") * 1e-2).to(wdt)
    m = torch.randn((above, I), generator=gen, device="cuda") * 1e-3
    v = m.square() + 1e-8
    start = [t.clone() for t in (W, m, v)]
    h = eq.AdamW(1e-3, 1e-4, 0.9, 0.999, 1e-8, 0.1, 0.0, 3)
    eq.eqat_block_ap_update(h, 2, 32, W=W, dW=dW, mW=m, vW=v)
    for rows in (slice(0, below), slice(below, above), slice(1, 38)):      # the same rows by a call below that size
        Wp, mp, vp = (t[rows].clone() for t in start)
        eq.eqat_block_ap_update(h, 2, 32, W=Wp, dW=dW[rows].clone(), mW=mp, vW=vp)
        assert torch.equal(Wp, W[rows]) and torch.equal(mp, m[rows]) and torch.equal(vp, v[rows])
    f = lambda x: float(np.float32(x))
    rows = slice(above - 40, above)
    ref = oracle.adamw(*(npf(t[rows]) for t in (start[0], dW, start[1], start[2])), f(1e-3), f(0.9), f(0.999), f(1e-8), f(0.1), 3)
    for got, want, tol in ((W, ref[0], 1e-5 if wdt == torch.float32 else 2 ** -8), (m, ref[1], 1e-5), (v, ref[2], 1e-5)):
        assert np.abs(npf(got[rows]) - want).max() <= tol * np.abs(want).max()

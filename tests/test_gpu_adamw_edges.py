"""AdamW at the edges of its workgroups: 2048 elements each, the last one element by element."""
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

"""What bench.py reckons per launch: the GEMM classes of a step add up to the flop of the step, whichever linears run dX and dW in one launch."""
import pytest
import torch

import bench
import paper_2407_11062_amd as eq
from paper_2407_11062_amd import synth


@pytest.mark.parametrize("name", ["llama2_7b_block_ap_w2g64", "llama2_13b_w3g128", "llama2_70b_w2g64", "llama2_7b_w4g128"])
@pytest.mark.parametrize("block_ap", [True, False])
def test_classes_add_up_to_the_step(name, block_ap):
    wl = synth.WORKLOADS[name]
    empty = torch.empty(0, dtype=torch.bfloat16)
    layers = [{"O": lin.out_features, "I": lin.in_features, "X": empty, "W": empty} for lin in wl.layers]
    flop = bench.gemm_flop(eq, layers, wl.tokens, wl.bits, wl.group, block_ap)
    one = sum(2.0 * wl.tokens * L["O"] * L["I"] for L in layers)
    assert flop["gemm_fwd"] * len(layers) == one
    merged = [2.0 * 2 * wl.tokens * L["O"] * L["I"] for L in layers if _together(wl, L, block_ap)]
    apart = len(layers) - len(merged)
    assert sum(merged) + apart * (flop.get("gemm_dx", 0.0) + flop.get("gemm_dw", 0.0)) == pytest.approx(2 * one, rel=1e-12)
    assert ("gemm_bwd" in flop) == bool(merged) and ("gemm_dx" in flop) == bool(apart)
    if merged:
        assert flop["gemm_bwd"] * len(merged) == pytest.approx(sum(merged), rel=1e-12)
    table = bench.kernel_table({k: (1.0, 2) for k in (*flop, "quantize")}, flop, {})
    assert all("tflops" in table[k] for k in flop) and "tflops" not in table["quantize"]


def _together(wl, L, block_ap):
    from test_gpu_mid_dx import dx_route
    return dx_route(wl.tokens, L["I"], L["O"], wl.bits, wl.group, block_ap)[1] >= 0

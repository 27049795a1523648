"""The work that users of the quantized-linear library have it do, as measurable cases.

A case is a dict of plain values:
  op      "serve"     eqat_qlinear_fwd on packed layers: decoding and prompt processing (one token to a few thousand)
          "block_ap"  one Block-AP training pass: Eq.(1), forward, backward with dX, dW, ds, dz
          "e2e"       one E2E-QP training pass on prepared layers: forward, backward with dX and ds (trained_z: and dz)
          "rtn"       step sizes and zero points from min/max, then the codes packed (round-to-nearest model, and the two
                      memory-bound ends of Block-AP)
          "update"    the step glue: reconstruction loss of the block's output, then AdamW on W, s, z of every linear
  shape   "block": the seven linears of a decoder block (hidden, inter, kv);  "linear": one linear (inf -> outf)
  tokens, bits, group (-1: one group per output row), act and w ("bf16" or "f32"), trained_z.

Every pass goes through the public functions of the package with outputs and workspaces that are allocated once, as the
training loop of a user's program (and this repository's benchmark) keeps them.
"""
from __future__ import annotations

import math

import torch

import paper_2407_11062_amd as eq
from paper_2407_11062_amd import synth

DTYPE = {"bf16": torch.bfloat16, "f32": torch.float32}


def _case(op, tokens, bits, group, *, hidden=0, inter=0, kv=0, inf=0, outf=0, act="bf16", w="bf16", trained_z=False):
    c = {"op": op, "shape": "block" if hidden else "linear", "tokens": tokens, "bits": bits, "group": group, "act": act, "w": w,
         "trained_z": trained_z}
    c.update({"hidden": hidden, "inter": inter, "kv": kv} if hidden else {"inf": inf, "outf": outf})
    return c


def listed():
    named = {
        # one token through a decoder block: the latency of interactive decoding (2 bit, the setting the method is for)
        "serve_4096_w2g64_1tok": _case("serve", 1, 2, 64, hidden=4096, inter=11008, kv=4096),
        # eight sequences decoded together, 3 bit
        "serve_5120_w3g128_8tok": _case("serve", 8, 3, 128, hidden=5120, inter=13824, kv=5120),
        # a prompt of a few hundred tokens, 4 bit, a length that no tile divides
        "serve_4096_w4g128_333tok": _case("serve", 333, 4, 128, hidden=4096, inter=11008, kv=4096),
        # the all-fp32 linear: the smallest training call
        "block_ap_512_f32_w4g128_256tok": _case("block_ap", 256, 4, 128, inf=512, outf=512, act="f32", w="f32"),
        # fp32 master weights, a short ragged batch, 4 bit
        "block_ap_4096_w4g128_f32w_1000tok": _case("block_ap", 1000, 4, 128, hidden=4096, inter=11008, kv=4096, w="f32"),
        # the headline step: 8192 tokens, 2 bit, group 64
        "block_ap_4096_w2g64_8192tok": _case("block_ap", 8192, 2, 64, hidden=4096, inter=11008, kv=4096),
        # the next larger block at 4096 tokens, 3 bit, group 128
        "block_ap_5120_w3g128_4096tok": _case("block_ap", 4096, 3, 128, hidden=5120, inter=13824, kv=5120),
        # E2E-QP at 4096 tokens, 2 bit
        "e2e_4096_w2g64_4096tok": _case("e2e", 4096, 2, 64, hidden=4096, inter=11008, kv=4096),
        # one short ragged sequence with trained zero points and one group per output row
        "e2e_4096_w3_perchannel_z_515tok": _case("e2e", 515, 3, -1, hidden=4096, inter=11008, kv=4096, trained_z=True),
        # the largest block, grouped-query attention (k and v are 1024 rows)
        "e2e_8192gqa_w2g64_4096tok": _case("e2e", 4096, 2, 64, hidden=8192, inter=28672, kv=1024),
        # both memory-bound ends of Block-AP on one block
        "rtn_4096_w2g64": _case("rtn", 0, 2, 64, hidden=4096, inter=11008, kv=4096),
        # loss and optimizer step of one block with fp32 master weights
        "update_4096_f32w_8192tok": _case("update", 8192, 2, 64, hidden=4096, inter=11008, kv=4096, w="f32"),
    }
    return [dict(c, name=n) for n, c in named.items()]


# ---- drawn cases ---------------------------------------------------------------------------------------------------------
MOST_FLOPS = 6 * 4096 * (2 * 8192 * 8192 + 2 * 1024 * 8192 + 3 * 8192 * 28672)      # the largest listed case


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _multiple(v, m):
    return max(1, round(v / m)) * m


def draw(rng):
    op = rng.choices(["serve", "block_ap", "e2e", "rtn", "update"], [40, 20, 22, 9, 9])[0]
    bits, group = rng.choice([2, 3, 4]), rng.choice([32, 64, 64, 128, 128, 256, -1])
    unit = 32 if group == -1 else group
    act = "f32" if op in ("block_ap", "e2e") and rng.random() < 0.2 else "bf16"
    w = "f32" if act == "f32" or rng.random() < 0.3 else "bf16"
    tokens = {"serve": (1, 2048), "block_ap": (256, 8192), "e2e": (256, 8192), "rtn": (1, 1), "update": (256, 8192)}[op]
    tokens = round(_log(rng, *tokens)) if op != "rtn" else 0
    trained_z = op == "e2e" and rng.random() < 0.4
    if act == "f32":            # fp32 activations: single linears of modest size
        c = _case(op, min(tokens, 2048), bits, group, inf=_multiple(_log(rng, 256, 2048), unit), outf=_multiple(_log(rng, 256, 2048), 8),
                  act=act, w=w, trained_z=trained_z)
    elif rng.random() < 0.5:
        hidden = _multiple(_log(rng, 1024, 8192), max(unit, 32))
        kv = hidden if rng.random() < 0.6 else _multiple(hidden / rng.choice([2, 4, 8]), 8)
        c = _case(op, tokens, bits, group, hidden=hidden, inter=_multiple(hidden * rng.uniform(2.5, 3.5), max(unit, 32)), kv=kv, w=w,
                  trained_z=trained_z)
    else:
        inf = _multiple(_log(rng, 1024, 28672), max(unit, 32))
        c = _case(op, tokens, bits, group, inf=inf, outf=_multiple(_log(rng, 1024, min(28672, 8192 * 28672 / inf)), 8), w=w,
                  trained_z=trained_z)
    while work(c)["flops"] > MOST_FLOPS:
        c["tokens"] //= 2
    return c


# ---- inputs --------------------------------------------------------------------------------------------------------------
def _linears(case):
    """[(name of the input it shares, out features, in features)]"""
    if case["shape"] == "linear":
        return [("x", case["outf"], case["inf"])]
    shared = {"q": "attn", "k": "attn", "v": "attn", "gate": "mlp", "up": "mlp"}
    return [(shared.get(l.name, l.name), l.out_features, l.in_features) for l in synth.llama_block(case["hidden"], case["inter"], case["kv"])]


def prepare(case, seed):
    dev = torch.device("cuda")
    gen = torch.Generator(device=dev)
    gen.manual_seed(seed)
    op, T, bits, g = case["op"], case["tokens"], case["bits"], case["group"]
    act, wdt = DTYPE[case["act"]], DTYPE[case["w"]]
    qmax = 2 ** bits - 1

    def normal(shape, std, dtype):
        return torch.empty(shape, dtype=torch.float32, device=dev).normal_(0.0, std, generator=gen).to(dtype)

    st = {"case": dict(case), "linears": []}
    inputs = {}
    for src, O, I in _linears(case):
        L = {"O": O, "I": I}
        W = normal((O, I), 0.02, wdt)
        s, z = eq.eqat_init_minmax(W, bits, g)
        if op != "rtn":                  # a trained state: some weights are clamped
            s = s * torch.empty_like(s).uniform_(0.7, 1.1, generator=gen)
            z = (z + torch.randint(-1, 2, z.shape, generator=gen, device=dev).float()).clamp_(0, qmax)
        L.update(W=W, s=s, z=z)
        if op in ("serve", "block_ap", "e2e"):
            if src not in inputs:
                inputs[src] = normal((T, I), 1.0, act)
            L["X"] = inputs[src]
            L["Y"] = torch.empty((T, O), dtype=act, device=dev)
        if op in ("block_ap", "e2e"):
            L["dY"] = normal((T, O), 1.0, act)
        d = eq.make_desc(T, I, O, bits, g, eq.BF16 if case["act"] == "bf16" else eq.F32, eq._dt(W))
        L["desc"] = d
        if op == "block_ap":
            L["out"] = {"dX": torch.empty((T, I), dtype=act, device=dev), "dW": torch.empty_like(W), "ds": torch.empty_like(s),
                        "dz": torch.empty_like(z)}
            L["ws"] = eq.workspace(d, eq.OP_FQ_BWD, dev)
        elif op == "serve":
            L["Wp"], L["zp"] = eq.eqat_pack(W, s, z, bits, g)
            L["ws"] = eq.workspace(d, eq.OP_Q_FWD, dev)
            del L["W"]
        elif op == "e2e":
            Wp, zp = eq.eqat_pack(W, s, z, bits, g)
            L["prepared"] = eq.eqat_qlinear_prepare(Wp, zp, I, bits, g, act_dtype=d.act_dtype)
            L["s"] = s * torch.empty_like(s).uniform_(0.95, 1.05, generator=gen)             # step sizes train on
            L["z"] = z + torch.empty_like(z).uniform_(-0.4, 0.4, generator=gen) if case["trained_z"] else None
            L["want"] = ("dX", "ds", "dz") if case["trained_z"] else ("dX", "ds")
            L["out"] = {"dX": torch.empty((T, I), dtype=act, device=dev), "ds": torch.empty_like(s)}
            if case["trained_z"]:
                L["out"]["dz"] = torch.empty_like(s)
            L["ws"] = eq.workspace(d, eq.OP_QP_BWD, dev)
            del L["W"], W, Wp, zp
        elif op == "rtn":
            L["Wp"], L["zp"] = eq.eqat_pack(W, s, z, bits, g)                                # output buffers
        elif op == "update":
            L["grads"] = {"dW": normal((O, I), 1e-3, wdt), "ds": normal(tuple(s.shape), 1e-2, torch.float32),
                          "dz": normal(tuple(s.shape), 1e-3, torch.float32)}
        st["linears"].append(L)
    Ls = st["linears"]
    if op == "rtn":
        st["batch"] = eq.Batch([L["desc"] for L in Ls], W=[L["W"] for L in Ls], s=[L["s"] for L in Ls], z=[L["z"] for L in Ls],
                               Wpacked=[L["Wp"] for L in Ls], zpacked=[L["zp"] for L in Ls])
    elif op == "block_ap" and case["shape"] == "block":
        st["batch"] = eq.Batch([L["desc"] for L in Ls], W=[L["W"] for L in Ls], s=[L["s"] for L in Ls], z=[L["z"] for L in Ls],
                               ws=[L["ws"] for L in Ls])
    elif op == "update":
        n_out = Ls[-1]["O"]
        st["Y"] = normal((T, n_out), 1.0, act)
        st["Yref"] = (st["Y"].float() + normal((T, n_out), 0.1, torch.float32)).to(act)
        st["loss"], st["dY"] = torch.empty(1, dtype=torch.float32, device=dev), torch.empty_like(st["Y"])
        st["ws"] = torch.empty(eq.lib().eqat_recon_loss_workspace_bytes(), dtype=torch.uint8, device=dev)
        # first and second moments of all parameters of the block, in two flat arrays
        sizes = [n for L in Ls for n in (L["W"].numel(), L["s"].numel(), L["z"].numel())]
        st["m"], st["v"] = normal((sum(sizes),), 1e-3, torch.float32), normal((sum(sizes),), 1e-3, torch.float32).square_()
        ms, vs = st["m"].split(sizes), st["v"].split(sizes)
        for k, L in enumerate(Ls):
            L["moments"] = {"mW": ms[3 * k], "vW": vs[3 * k], "ms": ms[3 * k + 1], "vs": vs[3 * k + 1], "mz": ms[3 * k + 2],
                            "vz": vs[3 * k + 2]}
        st["hyper"] = eq.AdamW(2e-5, 1e-4, 0.9, 0.999, 1e-8, 0.0, 0.0, 20)
    return st


def run(st):
    case, Ls = st["case"], st["linears"]
    op, bits, g = case["op"], case["bits"], case["group"]
    if op == "serve":
        return [eq.eqat_qlinear_fwd(L["X"], L["Wp"], L["s"], L["zp"], bits, g, Y=L["Y"], ws=L["ws"]) for L in Ls]
    if op == "block_ap":
        if "batch" in st:
            eq.eqat_fq_quantize_batched(st["batch"])
        for L in Ls:
            once = {"kept": True} if "batch" in st else {"keep": True}
            eq.eqat_fq_linear_fwd(L["X"], L["W"], L["s"], L["z"], bits, g, Y=L["Y"], ws=L["ws"], **once)
            eq.eqat_fq_linear_bwd(L["X"], L["W"], L["s"], L["z"], L["dY"], bits, g, out=L["out"], ws=L["ws"], kept=True)
        return [dict(L["out"], Y=L["Y"]) for L in Ls]
    if op == "e2e":
        for L in Ls:
            eq.eqat_qlinear_fwd_prepared(L["X"], L["prepared"], L["s"], L["O"], bits, g, z=L["z"], Y=L["Y"], ws=L["ws"], keep=True)
            eq.eqat_qlinear_bwd_prepared(L["X"], L["prepared"], L["s"], L["dY"], L["I"], bits, g, z=L["z"], want=L["want"], out=L["out"],
                                         ws=L["ws"], kept=True)
        return [dict(L["out"], Y=L["Y"]) for L in Ls]
    if op == "rtn":
        eq.eqat_init_minmax_batched(st["batch"])
        eq.eqat_pack_batched(st["batch"])
        return [(L["s"], L["z"], L["Wp"], L["zp"]) for L in Ls]
    eq.eqat_recon_loss(st["Y"], st["Yref"], loss=st["loss"], dY=st["dY"], ws=st["ws"])
    for L in Ls:
        eq.eqat_block_ap_update(st["hyper"], bits, g, W=L["W"], s=L["s"], z=L["z"], **L["grads"], **L["moments"])
    return [st["loss"], st["dY"], st["m"], st["v"]] + [(L["W"], L["s"], L["z"]) for L in Ls]


def work(case):
    """What one pass cannot do without: every distinct input once, every output once."""
    op, T, bits, g = case["op"], case["tokens"], case["bits"], case["group"]
    a, w = (2 if case[k] == "bf16" else 4 for k in ("act", "w"))
    nbytes, flops, seen = 0, 0, set()
    for src, O, I in _linears(case):
        n, groups = O * I, O * (1 if g == -1 else I // g)
        x_bytes = 0 if src in seen else T * I * a
        seen.add(src)
        packed = n * bits / 8 + groups * bits / 8
        if op == "serve":
            nbytes += packed + 4 * groups + x_bytes + T * O * a
            flops += 2 * T * n
        elif op == "block_ap":       # W, s, z, X, dY in; Y, dX, dW, ds, dz out
            nbytes += 2 * n * w + 16 * groups + x_bytes + (2 * T * O + T * I) * a
            flops += 6 * T * n
        elif op == "e2e":            # codes, s, z, X, dY in; Y, dX, ds (, dz) out
            nbytes += packed + (16 if case["trained_z"] else 8) * groups + x_bytes + (2 * T * O + T * I) * a
            flops += 6 * T * n
        elif op == "rtn":
            nbytes += n * w + 8 * groups + packed
        else:                        # p, g in, p out; two moments in and out
            nbytes += n * (3 * w + 16) + 2 * groups * 28
    if op == "update":
        nbytes += 3 * T * _linears(case)[-1][1] * a
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    if case["op"] == "rtn":
        return "exact"
    # Four times the distance to the same path in 64 bits: bf16 activations 2.4e-3 (What and the results are rounded to 8
    # bits), fp32 activations 1.1e-6.  The update is elementwise; a bf16 W may round the other way where a tie is near.
    return {"rel": 1e-5} if case["op"] == "update" else {"rel": 5e-6} if case["act"] == "f32" else {"rel": 1e-2}

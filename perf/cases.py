"""The work that users of this framework have it do, as cases whose speed can be measured.

Every case goes through the framework's executors (SwinBlock, SwinChain, AttnBlock, DecodeStep, CswinBlock) in the layout-elided
mode, the way a program uses them: the object is built once around the weights, then called with activations.  The listed cases are
the configurations that the benchmark runs and, for the same models, the small and the ragged calls that serving makes (one image, a
short prompt of odd length, one sequence with a short cache); draw() spreads over the sizes between and around them.

Values: activations and cached keys / values N(0, 1); Linear weights N(0, 1 / fan-in), so that every branch has the size of the
stream it is added to, as in a trained network; norm gains 1 + N(0, 0.02); biases and norm shifts N(0, 0.02); relative-position
tables N(0, 0.5), the 3 x 3 weights of the positional encoding N(0, 0.2).
"""
import math

import torch

from paper_2404_13528_amd import binding as sm

BF16, F32 = torch.bfloat16, torch.float32
DEPTHS = {96: (2, 2, 6, 2), 128: (2, 2, 18, 2)}      # of the hierarchical window-attention nets, by width of the first stage
HEAD = 32                                            # their head size
N_CLS = 1000


def listed():
    return [
        # one block alone in fp32 on one image: a user who checks or runs a block at full precision
        {"name": "swin_block_f32", "family": "swin_block", "dtype": "f32", "B": 1, "H": 56, "C": 96, "shift": 3},
        # a stage of six blocks on a batch of images: part of a detector's or classifier's backbone
        {"name": "swin_stage_b32", "family": "swin_stage", "B": 32, "H": 14, "C": 384, "depth": 6},
        # classification of a full batch of images by the whole net: throughput; the largest case
        {"name": "swin_net_b64", "family": "swin_net", "embed": 128, "B": 64},
        # the same net on one image: what an interactive user waits for
        {"name": "swin_net_b1", "family": "swin_net", "embed": 128, "B": 1},
        # the small net (widths 96 to 768) on an odd handful of images, as a server collects them
        {"name": "swin_net_small_b5", "family": "swin_net", "embed": 96, "B": 5},
        # a decoder layer over a long prompt
        {"name": "llama_s2048", "family": "llama", "B": 1, "S": 2048, "E": 4096},
        # ... and over a short prompt of odd length
        {"name": "llama_s333", "family": "llama", "B": 1, "S": 333, "E": 4096},
        # the spatial transformer of a diffusion net at its highest resolution, conditional and unconditional half together
        {"name": "sd_64x64_b2", "family": "sd", "B": 2, "C": 320, "H": 64, "W": 64},
        # an encoder block over 14 x 14 patches and the class token, a batch of images
        {"name": "vit_b32_s197", "family": "vit", "B": 32, "S": 197, "E": 768},
        # one new token for each of eight conversations with long histories
        {"name": "decode_b8_l2047", "family": "decode", "B": 8, "L": 2047},
        # one new token for one user early in a conversation; the smallest case
        {"name": "decode_b1_l150", "family": "decode", "B": 1, "L": 150},
        # a block of cross-shaped window attention on a batch of images
        {"name": "cswin_block_b64", "family": "cswin", "B": 64, "H": 14, "C": 256, "heads": 8, "sw": 7},
    ]


def _log(rng, lo, hi):
    """A whole number from lo to hi, spread over its logarithm."""
    return min(hi, max(lo, int(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    family = rng.choice(["swin_block", "swin_stage", "swin_net", "llama", "sd", "vit", "decode", "cswin"])
    if family == "swin_block":
        H, C = rng.choice([(56, 96), (28, 192), (14, 384), (7, 768)])
        return {"family": family, "dtype": rng.choice(["f32", "bf16"]), "B": _log(rng, 1, 16), "H": H, "C": C,
                "shift": rng.choice([0, 3]) if H > 7 else 0}
    if family == "swin_stage":
        H, C = rng.choice([(56, 128), (28, 192), (28, 256), (14, 384), (14, 512), (7, 768), (7, 1024)])
        return {"family": family, "B": _log(rng, 1, 64), "H": H, "C": C, "depth": rng.randint(2, 6)}
    if family == "swin_net":
        return {"family": family, "embed": rng.choice([96, 128]), "B": _log(rng, 1, 64)}
    if family == "llama":
        B = rng.choice([1, 1, 2, 4])
        return {"family": family, "B": B, "S": _log(rng, 16, 2048 // B), "E": rng.choice([1024, 2048, 4096])}
    if family == "sd":
        return {"family": family, "B": rng.randint(1, 4), "C": rng.choice([320, 640]), "H": rng.randint(8, 64), "W": rng.randint(8, 64)}
    if family == "vit":
        return {"family": family, "B": _log(rng, 1, 64), "S": rng.choice([50, 197, 257, 577]), "E": rng.choice([384, 768, 1024])}
    if family == "decode":
        return {"family": family, "B": _log(rng, 1, 32), "L": _log(rng, 16, 2047)}
    H, C, heads, sw = rng.choice([(56, 64, 2, 1), (28, 128, 4, 2), (14, 256, 8, 7), (7, 512, 16, 7)])
    return {"family": family, "B": _log(rng, 1, 64), "H": H, "C": C, "heads": heads, "sw": sw}


# ---- sizes that follow from a case -------------------------------------------------------------------------------------

def _ffn(E):
    return {4096: 11008, 2048: 5632, 1024: 2816}[E]         # gated MLP width of the decoder layer


SD_SC, SD_DC, SD_GROUPS, SD_HEADS = 77, 768, 32, 8           # the text context of the diffusion block, its norm groups and heads
NEOX = {"E": 2048, "heads": 8, "F": 8192, "rot": 64}         # the decode step's layer


def _stages(case):
    """[(C, heads, depth, H, W)] of a net case."""
    out, C, H = [], case["embed"], 56
    for depth in DEPTHS[case["embed"]]:
        out.append((C, C // HEAD, depth, H, H))
        C, H = 2 * C, H // 2
    return out


# ---- inputs -------------------------------------------------------------------------------------------------------------

class _Draw:
    def __init__(self, seed, dtype):
        self.g = torch.Generator(device="cuda").manual_seed(seed)
        self.dtype = dtype

    def normal(self, *shape, std=1.0, mean=0.0):
        t = torch.randn(*shape, generator=self.g, device="cuda", dtype=torch.float32)
        return (t.mul_(std).add_(mean) if (std, mean) != (1.0, 0.0) else t).to(self.dtype)

    def matrix(self, n_out, n_in):
        return self.normal(n_out, n_in, std=n_in ** -0.5)

    def vector(self, n):
        return self.normal(n, std=0.02)

    def gain(self, n):
        return self.normal(n, std=0.02, mean=1.0)


def _swin_params(dr, C):
    return {"ln1_g": dr.gain(C), "ln1_b": dr.vector(C), "wqkv": dr.matrix(3 * C, C), "bqkv": dr.vector(3 * C),
            "rpb_table": dr.normal(13 * 13, C // HEAD, std=0.5), "wproj": dr.matrix(C, C), "bproj": dr.vector(C),
            "ln2_g": dr.gain(C), "ln2_b": dr.vector(C), "w1": dr.matrix(4 * C, C), "b1": dr.vector(4 * C),
            "w2": dr.matrix(C, 4 * C), "b2": dr.vector(C)}


def _net_params(dr, stages):
    net = {"embed": {"w": dr.matrix(stages[0][0], 48), "b": dr.vector(stages[0][0]), "ln_g": dr.gain(stages[0][0]),
                     "ln_b": dr.vector(stages[0][0])}, "stages": [], "merges": []}
    for i, (C, _, depth, _, _) in enumerate(stages):
        net["stages"].append([_swin_params(dr, C) for _ in range(depth)])
        if i + 1 < len(stages):
            net["merges"].append({"ln_g": dr.gain(4 * C), "ln_b": dr.vector(4 * C), "w": dr.matrix(2 * C, 4 * C)})
    C = stages[-1][0]
    net["head"] = {"ln_g": dr.gain(C), "ln_b": dr.vector(C), "w": dr.matrix(N_CLS, C), "b": dr.vector(N_CLS)}
    return net


def _neox_params(dr, E, F):
    return {"ln1_g": dr.gain(E), "ln1_b": dr.vector(E), "wqkv": dr.matrix(3 * E, E), "bqkv": dr.vector(3 * E),
            "wdense": dr.matrix(E, E), "bdense": dr.vector(E), "ln2_g": dr.gain(E), "ln2_b": dr.vector(E),
            "w1": dr.matrix(F, E), "b1": dr.vector(F), "w2": dr.matrix(E, F), "b2": dr.vector(E)}


def prepare(case, seed):
    family = case["family"]
    dr = _Draw(seed, F32 if case.get("dtype") == "f32" else BF16)
    B = case["B"]
    if family == "swin_block":
        H, C = case["H"], case["C"]
        x, p = dr.normal(B, H * H, C), _swin_params(dr, C)
        return {"call": sm.SwinBlock(B, H, H, C, C // HEAD, 7, case["shift"], p, dr.dtype), "args": (x,)}
    if family == "swin_stage":
        H, C, depth = case["H"], case["C"], case["depth"]
        x, net = dr.normal(B, H * H, C), {"stages": [[_swin_params(dr, C) for _ in range(depth)]]}
        return {"call": sm.SwinChain(B, [(C, C // HEAD, depth, H, H)], 7, net, BF16), "args": (x,)}
    if family == "swin_net":
        stages = _stages(case)
        x, net = dr.normal(B, 3, 224, 224), _net_params(dr, stages)
        return {"call": sm.SwinChain(B, stages, 7, net, BF16, img=224, n_cls=N_CLS), "args": (x,)}
    if family == "llama":
        S, E, F = case["S"], case["E"], _ffn(case["E"])
        x = dr.normal(B, S, E)
        p = {"rms1_g": dr.gain(E), "wq": dr.matrix(E, E), "wk": dr.matrix(E, E), "wv": dr.matrix(E, E), "wo": dr.matrix(E, E),
             "rms2_g": dr.gain(E), "wgate": dr.matrix(F, E), "wup": dr.matrix(F, E), "wdown": dr.matrix(E, F)}
        return {"call": sm.AttnBlock("llama", p, BF16, B=B, S=S, E=E, heads=E // 128, F=F), "args": (x,)}
    if family == "sd":
        C, H, W, F = case["C"], case["H"], case["W"], 4 * case["C"]
        x, ctx = dr.normal(B, C, H, W), dr.normal(B, SD_SC, SD_DC)
        p = {"gn_g": dr.gain(C), "gn_b": dr.vector(C), "win": dr.matrix(C, C), "bin": dr.vector(C)}
        for i, n in ((1, C), (2, SD_DC)):
            p.update({"ln%d_g" % i: dr.gain(C), "ln%d_b" % i: dr.vector(C), "a%d_wq" % i: dr.matrix(C, C), "a%d_wk" % i: dr.matrix(C, n),
                      "a%d_wv" % i: dr.matrix(C, n), "a%d_wo" % i: dr.matrix(C, C), "a%d_bo" % i: dr.vector(C)})
        p.update({"ln3_g": dr.gain(C), "ln3_b": dr.vector(C), "ff_w1": dr.matrix(2 * F, C), "ff_b1": dr.vector(2 * F),
                  "ff_w2": dr.matrix(C, F), "ff_b2": dr.vector(C), "wout": dr.matrix(C, C), "bout": dr.vector(C)})
        return {"call": sm.AttnBlock("sd", p, BF16, B=B, E=C, heads=SD_HEADS, F=F, Hs=H, Ws=W, groups=SD_GROUPS, Sc=SD_SC, Dc=SD_DC),
                "args": (x, ctx)}
    if family == "vit":
        S, E = case["S"], case["E"]
        x, p = dr.normal(B, S, E), _neox_params(dr, E, 4 * E)
        p["wo"], p["bo"] = p.pop("wdense"), p.pop("bdense")
        return {"call": sm.AttnBlock("vit", p, BF16, B=B, S=S, E=E, heads=E // 64, F=4 * E), "args": (x,)}
    if family == "decode":
        E, h, F, L = NEOX["E"], NEOX["heads"], NEOX["F"], case["L"]
        x, p = dr.normal(B, E), _neox_params(dr, E, F)
        k, v = dr.normal(B, h, L + 1, E // h), dr.normal(B, h, L + 1, E // h)      # room for the new token's row
        return {"call": sm.DecodeStep(p, B, E, h, F, NEOX["rot"]), "args": (x, k, v, L), "updated": (k, v)}
    H, C = case["H"], case["C"]
    x, p = dr.normal(B, H * H, C), _swin_params(dr, C)
    p["lepe_w"], p["lepe_b"] = dr.normal(C, 3, 3, std=0.2), dr.vector(C)
    return {"call": sm.CswinBlock(B, H, H, C, case["heads"], case["sw"], p), "args": (x,)}


def run(state):
    y = state["call"](*state["args"])
    return (y,) + state["updated"] if "updated" in state else y


# ---- what a pass cannot do without ----------------------------------------------------------------------------------------

def _swin_work(T, C, window=49):
    """(flops, weights) of a block on T tokens of C channels whose queries see `window` keys each."""
    return T * (24.0 * C * C + 4.0 * window * C), 12 * C * C + 13 * C


def work(case):
    family, B = case["family"], case["B"]
    es = 4 if case.get("dtype") == "f32" else 2
    if family == "swin_block":
        T = B * case["H"] ** 2
        fl, w = _swin_work(T, case["C"])
        return {"bytes": es * (2.0 * T * case["C"] + w + 169 * case["C"] // HEAD), "flops": fl}
    if family == "swin_stage":
        T = B * case["H"] ** 2
        fl, w = _swin_work(T, case["C"])
        return {"bytes": 2.0 * (2 * T * case["C"] + case["depth"] * (w + 169 * case["C"] // HEAD)), "flops": case["depth"] * fl}
    if family == "swin_net":
        stages = _stages(case)
        C0, CL = stages[0][0], stages[-1][0]
        fl, w = B * 56 * 56 * 2.0 * 48 * C0 + B * 2.0 * CL * N_CLS, 48 * C0 + 3 * C0 + CL * N_CLS + 2 * CL + N_CLS
        for i, (C, h, depth, H, _) in enumerate(stages):
            f, n = _swin_work(B * H * H, C)
            fl, w = fl + depth * f, w + depth * (n + 169 * h)
            if i + 1 < len(stages):
                fl, w = fl + B * (H // 2) ** 2 * 16.0 * C * C, w + 8 * C * C + 8 * C
        return {"bytes": 2.0 * (B * 3 * 224 * 224 + B * N_CLS + w), "flops": fl}
    if family == "llama":
        S, E, F = case["S"], case["E"], _ffn(case["E"])
        w = 4 * E * E + 3 * E * F
        return {"bytes": 2.0 * (2 * B * S * E + w + 2 * E), "flops": 2.0 * B * S * w + 2.0 * B * S * (S + 1) * E}
    if family == "sd":
        C, S, F = case["C"], case["H"] * case["W"], 4 * case["C"]
        w_tok = 2 * C * C + 4 * C * C + 2 * C * C + 3 * C * F        # proj in / out, self q k v o, cross q o, gated MLP
        w_ctx = 2 * C * SD_DC
        fl = 2.0 * B * S * w_tok + 2.0 * B * SD_SC * w_ctx + 4.0 * B * S * (S + SD_SC) * C
        return {"bytes": 2.0 * (2 * B * S * C + B * SD_SC * SD_DC + w_tok + w_ctx + 13 * C + 2 * F), "flops": fl}
    if family == "vit":
        S, E = case["S"], case["E"]
        return {"bytes": 2.0 * (2 * B * S * E + 12 * E * E + 13 * E), "flops": 24.0 * B * S * E * E + 4.0 * B * S * S * E}
    if family == "decode":
        E, F, L = NEOX["E"], NEOX["F"], case["L"]
        w = 4 * E * E + 2 * E * F
        return {"bytes": 2.0 * (w + 10 * E + F + 2 * B * E + 2 * B * L * E + 2 * B * E), "flops": 2.0 * B * w + 4.0 * B * (L + 1) * E}
    T, C = B * case["H"] ** 2, case["C"]
    fl, w = _swin_work(T, C, window=case["H"] * case["sw"])
    return {"bytes": 2.0 * (2 * T * C + w + 10 * C), "flops": fl + 18.0 * T * C}


def tolerance(case):
    if case.get("dtype") == "f32":
        return {"rel": 2e-5}
    # bf16 activations between operators; a stage's output is its residual stream, rounded once or twice in each of its blocks (the
    # kernel-per-operator form of a six-block stage differs from the fused form by 8e-3; a net's head averages over its tokens: 4e-3)
    return {"rel": 1.5e-2} if case["family"] == "swin_stage" else {"rel": 1e-2}

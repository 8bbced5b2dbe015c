"""Benchmark of the layout-elided hot path on one MI355X.

Headline workload (benchmark configs[2], the largest single-GPU one): the full Swin-B-shaped net at 224x224,
bf16, B=64, patch 4, embed 128, depths (2,2,18,2), heads (4,8,16,32), window 7, patch merging between stages;
seeded synthetic image and random-init weights, resident in HBM before the timed region.  One step = one pass of
the whole chain (sm_run_chain, SM_ELIDED) over one batch of 64 images.

Prints ONE JSON line.  `value` = images/s of that chain.  `configs` holds, for each of the five configurations of
the benchmark spec, every variant timed the same way (elided / explicit-transpose chain, and for the Swin chains the
kernel-per-operator form beside the fused one, so that layout elimination and kernel fusion are reported apart):
ms per step, throughput, algorithmic HBM bytes, the per-kernel table from HIP events on the launch stream, the
dominant kernel and its roofline.  `roofline` (top level) is the headline chain's dominant kernel; `cpu_baseline`
is the CPU oracle on a bounded sample of the headline workload.

  python bench.py                       all five configurations and the extras 6-10 (about two minutes)
  python bench.py --config 3            one configuration (1-based, as in the benchmark's list; 6: ViT block, 7: Fig. 4
                                        graph, 8: decode step, 9: CSwin attention, 10: CSwin block)
  python bench.py --fold-microbench     the read- versus write-side folding micro-experiment (Sec. 3.2.2)
"""
import argparse
import json
import os
import re
import sys
import time

ROOT = os.path.dirname(os.path.abspath(__file__))
sys.path.insert(0, ROOT)

PEAK_HBM = 8.0e12          # B/s, MI355X published
PEAK_BF16 = 2.5e15         # FLOP/s dense bf16 MFMA, MI355X published
PEAK_F32 = 157.3e12        # FLOP/s fp32 (matrix and vector), MI355X published


def measured_traffic():
    """HBM bytes per launch from the committed rocprofv3 --pmc summaries (profiles/*_hbm_counters.md): table rows
    `| bench label | FETCH_SIZE KiB | WRITE_SIZE KiB | bytes |`, bytes = the two counters scaled by what they read for
    an identity copy of known size (factors stated in each file)."""
    out = {}
    pdir = os.path.join(ROOT, "profiles")
    for f in sorted(os.listdir(pdir)) if os.path.isdir(pdir) else []:
        if not f.endswith("_hbm_counters.md"):
            continue
        for line in open(os.path.join(pdir, f)):
            m = re.match(r"\|\s*`([^`]+)`\s*\|\s*([\d.]+)\s*\|\s*([\d.]+)\s*\|\s*(\d+)\s*\|", line)
            if m:
                out[m.group(1)] = int(m.group(4))
    return out


def kernel_model(label):
    """Algorithmic bytes and flops of one launch, from the kernel's timing label: tensor reads + writes at
    kernel-per-operator granularity with fused epilogues, weights and bias included; flops 2MNK for a Linear,
    4 nq nk d per (batch, head) for attention (halved when causal)."""
    e = 4 if "_f32" in label else 2
    m = re.match(r"(proj\+)?(ln\+)?mlp_\w+\[(\d+),(\d+),(\d+)\](\+ln)?(\+qkv)?", label)
    if m:      # fused MLP: X and the residual read, Y written, both weights, biases (and the norm's vectors);
        #        with the projection in front: its [C, C] weight and bias as well (A, x0 read, Y written);
        #        "+ln": the next block's LayerNorm as a second output
        M, Hd, C = int(m.group(3)), int(m.group(4)), int(m.group(5))
        by = 3 * M * C + 2 * Hd * C + Hd + C + (2 * C if m.group(2) else 0) + (C * C + C if m.group(1) else 0)
        by += (M * C + 2 * C) if m.group(6) and not m.group(7) else 0
        fl = 4.0 * M * Hd * C + (2.0 * M * C * C if m.group(1) else 0.0)
        if m.group(7):      # ... and the next block's QKV Linear on that norm: its weight, bias and [M, 3C] output
            by += 2 * C + 3 * C * C + 3 * C + 3 * M * C
            fl += 6.0 * M * C * C
        return by * e, fl
    m = re.match(r"decode_(ln\+qkv\+rope\|ln\+fc1\+gelu|dense\+sum\+res)_bf16\[(\d+),(\d+),(\d+)\]", label)
    if m:      # skinny Linears of the decode step: the weight once, the token rows in and out, biases / norm vectors
        B, N, K = int(m.group(2)), int(m.group(3)), int(m.group(4))
        extra = 4 * K if m.group(1).startswith("ln") else (N + B * N)          # two norms' gamma / beta | second bias, residual
        return (N * K + N + B * K + B * N + extra) * e, 2.0 * B * N * K
    m = re.match(r"decode_attention\|fc2_bf16\[(\d+),(\d+),(\d+),(\d+)\]\+\[(\d+),(\d+),(\d+)\]", label)
    if m:      # attention against the cache, and beside it W2 . hid (its fp32 parts are this form's own)
        B, h, n, d, _, N, K = [int(m.group(i)) for i in range(1, 8)]
        return (B * h * (2 * n * d + 2 * d) + N * K + B * K) * e, 4.0 * B * h * n * d + 2.0 * B * N * K
    m = re.match(r"cutgemm_bf16\[(\d+),(\d+),(\d+)\]", label)
    if m:      # cut over K: the operands (the fp32 parts are this form's own, as a fused operator's intermediates are)
        M, N, K = int(m.group(1)), int(m.group(2)), int(m.group(3))
        return (M * K + N * K) * e, 2.0 * M * N * K
    m = re.match(r"sum_parts_bf16\[(\d+),(\d+),\d+\]\+res(\+norm)?", label)
    if m:      # ... and its result and residual; with +norm the normalised rows are written as well
        M, N = int(m.group(1)), int(m.group(2))
        return (3 if m.group(3) else 2) * M * N * e, 0.0
    m = re.match(r"concat_bf16\[(\d+),(\d+),(\d+)\]", label)
    if m:
        return 2 * int(m.group(1)) * int(m.group(2)) * int(m.group(3)) * e, 0.0
    m = re.match(r"dwconv3x3_bf16\[(\d+),(\d+),(\d+),(\d+)\]", label)
    if m:      # depth-wise 3 x 3: the values read, the result written, 9 weights + bias per channel
        n, H, W, C = [int(m.group(i)) for i in range(1, 5)]
        return (2 * n * H * W * C + 10 * C) * e, 18.0 * n * H * W * C
    m = re.match(r"concat_bf16\[(\d+),(\d+)\]", label)
    if m:      # Concat along the channels: [rows, C] written, its two halves read
        return 2 * int(m.group(1)) * int(m.group(2)) * e, 0.0
    m = re.match(r"(?:ln\+|rms\+)?(?:p|split)?gemm_\w+\[(\d+),(\d+),(\d+)\](.*)", label)
    if m:
        M, N, K = int(m.group(1)), int(m.group(2)), int(m.group(3))
        n_out = N // 2 if "+glu" in m.group(4) else N
        by = (M * K + N * K + N + M * n_out + (M * n_out if "+res" in m.group(4) else 0) + (M * n_out if "+copy2" in m.group(4) else 0)) * e
        return by, 2.0 * M * N * K
    m = re.match(r"(layernorm|rmsnorm)_\w+\[(\d+),(\d+)\]", label)
    if m:
        R, C = int(m.group(2)), int(m.group(3))
        return (2 * R * C + 2 * C) * e, 8.0 * R * C
    m = re.match(r"attention_(\w+?)_\w+\[(\d+),(\d+),(\d+),(\d+),(\d+)\](\+acc)?", label)
    if m:      # q read, o written, k and v read ("+acc": o read as well)
        nb, h, nq, nk, d = [int(m.group(i)) for i in range(2, 7)]
        fl = 4.0 * nb * h * nq * nk * d * (0.5 if m.group(1) == "causal" else 1.0)
        return nb * h * ((3 if m.group(7) else 2) * nq + 2 * nk) * d * e, fl
    m = re.match(r"copy_\w+\[(\d+)\](.*)", label)
    if m:
        n = int(m.group(1))
        return (3 if "+add" in m.group(2) else 2) * n * e, 0.0
    m = re.match(r"groupnorm_\w+\[(\d+),(\d+),(\d+),(\d+)\]", label)
    if m:      # statistics pass reads x, apply pass reads x and writes y
        B, C, HW = int(m.group(1)), int(m.group(2)), int(m.group(3))
        return 3 * B * C * HW * e, 10.0 * B * C * HW
    m = re.match(r"mean_tokens_\w+\[(\d+),(\d+),(\d+)\]", label)
    if m:
        B, L, C = int(m.group(1)), int(m.group(2)), int(m.group(3))
        return (B * L * C + B * C) * e, float(B * L * C)
    m = re.match(r"reduce_(last|first)_\w+\[(\d+),(\d+)\]", label)
    if m:
        r, n = int(m.group(2)), int(m.group(3))
        return (r * n + r) * e, float(r * n)
    m = re.match(r"fill_row_tables?\[(\d+)\]", label)
    if m:
        return (4 * int(m.group(1)) if "table[" in label else 0), 0.0
    return 0, 0.0


def roofline_of(row, traffic):
    peak_f = PEAK_F32 if "_f32" in row["kernel"] else PEAK_BF16
    t_hbm, t_mfma = row["alg_bytes"] / PEAK_HBM, row["flops"] / peak_f
    if t_mfma >= t_hbm:
        r = {"bound": "mfma", "achieved": row["TFLOPs"], "peak": peak_f * 1e-12, "unit": "TFLOP/s"}
    else:
        r = {"bound": "hbm", "achieved": row["GBps"], "peak": PEAK_HBM * 1e-9, "unit": "GB/s"}
    r["frac"] = round(r["achieved"] / r["peak"], 4)
    r["traffic"] = traffic.get(row["kernel"])
    r["kernel"], r["avg_us"] = row["kernel"], row["avg_us"]
    return r


def fold_microbench(sm, torch, steps, warmup):
    """A transposition between two MatMuls, T = X . W1^T then Y = T^T . W2^T, three ways (the paper's micro-experiment
    "version a optimises reads, version b optimises writes", Sec. 3.2.2, for the MatMul operator):
    write_fold: the producer stores T transposed (strided stores), the consumer reads K-contiguous rows;
    read_fold:  the producer stores T as it comes, the consumer reads it transposed in place (K-strided loads);
    explicit:   the producer stores T as it comes, a copy kernel transposes it, the consumer reads the copy."""
    dt = torch.bfloat16
    out = {"experiment": "read- versus write-side folding of a transposition between two Linears (bf16)", "cases": []}
    for (M, N, K, N2) in ((2048, 2048, 512, 512), (6272, 1536, 384, 384)):
        g = torch.Generator().manual_seed(7)
        X = torch.randn(M, K, generator=g).to(dt).cuda()
        W1 = (torch.randn(N, K, generator=g) * K ** -0.5).to(dt).cuda()
        W2 = (torch.randn(N2, M, generator=g) * M ** -0.5).to(dt).cuda()
        T = torch.empty(M * N, dtype=dt, device="cuda")
        T2 = torch.empty(N, M, dtype=dt, device="cuda")
        Y = torch.empty(N, N2, dtype=dt, device="cuda")
        tmap = sm.Map.create((M, N), [("permute", (1, 0))])          # view [N, M] of T [M, N]

        def write_fold():
            sm.linear(X, W1, c_transposed_batch=M, out=T)             # T stored as [N, M]
            sm.linear(T, W2, out=Y, M=N)

        def read_fold():
            sm.linear(X, W1, out=T)
            sm.linear(T, W2, a_map=tmap, out=Y, M=N)

        def explicit():
            sm.linear(X, W1, out=T)
            tmap.gather(T.view(M, N), out=T2)
            sm.linear(T2, W2, out=Y, M=N)

        res, ref = {}, None
        for name, fn in (("write_fold", write_fold), ("read_fold", read_fold), ("explicit", explicit)):
            for _ in range(warmup):
                fn()
            torch.cuda.synchronize()
            t0 = time.perf_counter()
            for _ in range(steps):
                fn()
            torch.cuda.synchronize()
            res[name + "_us"] = round((time.perf_counter() - t0) / steps * 1e6, 2)
            y = Y.float().clone()
            ref = y if ref is None else ref
            res[name + "_max_diff"] = float((y - ref).abs().max())
        res.update(shape={"M": M, "N": N, "K": K, "N2": N2},
                   read_over_write=round(res["read_fold_us"] / res["write_fold_us"], 3),
                   explicit_over_write=round(res["explicit_us"] / res["write_fold_us"], 3))
        out["cases"].append(res)
    return out


SWIN_B = dict(depths=(2, 2, 18, 2), heads=(4, 8, 16, 32), embed=128, img=224, w=7)


def build_config(k, sm, torch, Wl):
    """-> (description, unit, units per step, {variant name: callable running one step}, oracle sample or None).
    Variants: "elided" and "explicit" always; Swin chains add "elided_per_op" / "explicit_per_op" (one kernel per
    surviving operator, fuse_mlp=False) so that elimination (per_op pair) and fusion (elided vs elided_per_op) are
    measured apart."""
    bf = torch.bfloat16
    dev = lambda p, dt: {n: v.to(dt).cuda() for n, v in p.items()}
    if k == 1:
        B, H, W, C, h, w, s = 1, 56, 56, 96, 3, 7, 3
        x, p = Wl.swin_block_case(B, H, W, C, h, w, seed=0)
        dp, xd = dev(p, torch.float32), x.cuda()
        y = torch.empty_like(xd)
        blk = {n: sm.SwinBlock(B, H, W, C, h, w, s, dp, torch.float32, m) for n, m in (("elided", sm.SM_ELIDED), ("explicit", sm.SM_EXPLICIT))}
        return ("configs[0]: one Swin block, fp32, B=1, 56x56 tokens, C=96, 3 heads, window 7, shift 3", "images/s", B,
                {n: (lambda b=b: b(xd, out=y)) for n, b in blk.items()}, None, "f32")
    if k == 2:
        B, H, W, C, h, w, depth = 32, 14, 14, 384, 12, 7, 6
        x, blocks = Wl.swin_stage_case(B, H, W, C, h, w, depth)
        net = {"stages": [[dev(p, bf) for p in blocks]]}
        xd = x.to(bf).cuda()
        y = torch.empty_like(xd)
        var = {}
        for n, m, f in (("elided", sm.SM_ELIDED, True), ("explicit", sm.SM_EXPLICIT, True),
                        ("elided_per_op", sm.SM_ELIDED, False), ("explicit_per_op", sm.SM_EXPLICIT, False)):
            ch = sm.SwinChain(B, [(C, h, depth, H, W)], w, net, bf, m, fuse_mlp=f)
            var[n] = (lambda ch=ch: ch(xd, out=y))
        return ("configs[1]: Swin stage-3 chain, bf16, B=32, 14x14 tokens, C=384, 12 heads, window 7, 6 blocks shift 0/3, MLP 4x",
                "images/s", B, var, None, "bf16")
    if k == 3:
        B = 64
        image, net = Wl.swin_net_case(B, img=SWIN_B["img"], embed=SWIN_B["embed"], depths=SWIN_B["depths"], heads=SWIN_B["heads"], w=SWIN_B["w"])
        dnet = {"embed": dev(net["embed"], bf), "stages": [[dev(p, bf) for p in st] for st in net["stages"]],
                "merges": [dev(m, bf) for m in net["merges"]], "head": dev(net["head"], bf)}
        stages, H, C = [], SWIN_B["img"] // 4, SWIN_B["embed"]
        for dep, hh in zip(SWIN_B["depths"], SWIN_B["heads"]):
            stages.append((C, hh, dep, H, H))
            H, C = H // 2, C * 2
        xd = image.to(bf).cuda()
        var = {}
        for n, m, f in (("elided", sm.SM_ELIDED, True), ("explicit", sm.SM_EXPLICIT, True),
                        ("elided_per_op", sm.SM_ELIDED, False), ("explicit_per_op", sm.SM_EXPLICIT, False)):
            ch = sm.SwinChain(B, stages, SWIN_B["w"], dnet, bf, m, img=SWIN_B["img"], n_cls=1000, fuse_mlp=f)
            y = torch.empty(B, 1000, dtype=bf, device="cuda")
            var[n] = (lambda ch=ch, y=y: ch(xd, out=y))
        return ("configs[2]: full Swin-B-shaped net at 224x224, bf16, B=64, patch 4, embed 128, depths (2,2,18,2), heads (4,8,16,32), "
                "window 7, patch merging, head 1000 classes", "images/s", B, var, (image, net), "bf16")
    if k == 4:
        B, S, E, h, F = 1, 2048, 4096, 32, 11008
        x, p = Wl.llama_case(B, S, E, F)
        dp, xd = dev(p, bf), x.to(bf).cuda()
        y = torch.empty_like(xd)
        blk = {n: sm.AttnBlock("llama", dp, bf, m, B=B, S=S, E=E, heads=h, F=F) for n, m in (("elided", sm.SM_ELIDED), ("explicit", sm.SM_EXPLICIT))}
        return ("configs[3]: Llama-style decoder layer prefill, bf16, B=1, seq 2048, hidden 4096, 32 heads x 128, RoPE, causal, SwiGLU 11008",
                "tokens/s", B * S, {n: (lambda b=b: b(xd, out=y)) for n, b in blk.items()}, None, "bf16")
    if k == 5:
        B, C, H, W, Sc, Dc, F, G, h = 2, 320, 64, 64, 77, 768, 1280, 32, 8
        x, ctx, p = Wl.sd_case(B, C, H, W, Sc, Dc, F)
        dp, xd, cd = dev(p, bf), x.to(bf).cuda(), ctx.to(bf).cuda()
        y = torch.empty_like(xd)
        blk = {n: sm.AttnBlock("sd", dp, bf, m, B=B, E=C, heads=h, F=F, Hs=H, Ws=W, groups=G, Sc=Sc, Dc=Dc)
               for n, m in (("elided", sm.SM_ELIDED), ("explicit", sm.SM_EXPLICIT))}
        return ("configs[4]: diffusion-UNet spatial transformer block, bf16, B=2, latent 64x64x320 NCHW, GroupNorm 32, self-attn 8 heads "
                "over 4096 tokens, cross-attn to 77x768, GEGLU 1280", "images/s", B,
                {n: (lambda b=b: b(xd, cd, out=y)) for n, b in blk.items()}, None, "bf16")
    if k == 6:     # a second workload from the paper's model list (Tables 1, 7), beyond the benchmark's five
        B, S, E, h, F = 32, 197, 768, 12, 3072
        x, p = Wl.vit_case(B, S, E, h, F)
        dp, xd = dev(p, bf), x.to(bf).cuda()
        y = torch.empty_like(xd)
        blk = {n: sm.AttnBlock("vit", dp, bf, m, B=B, S=S, E=E, heads=h, F=F) for n, m in (("elided", sm.SM_ELIDED), ("explicit", sm.SM_EXPLICIT))}
        return ("extra: ViT-B/16 encoder block, bf16, B=32, 197 tokens, 768 wide, 12 heads x 64, global attention, GELU MLP 3072",
                "images/s", B, {n: (lambda b=b: b(xd, out=y)) for n, b in blk.items()}, None, "bf16")
    if k == 7:     # the multi-consumer example of Sec. 3.2.2 (Fig. 4) with its redundant copy executed
        D1, D2, D3, Kin, Cout = 512, 64, 256, 256, 64
        a, w, wc = Wl.fanout_case(D1, D2, D3, Kin, Cout)
        ad, wd, wcd = a.to(bf).cuda(), w.to(bf).cuda(), wc.to(bf).cuda()
        gs = {"elided": sm.FanoutGraph(D1, D2, D3, Kin, Cout, bf, sm.SM_ELIDED, 1),          # two stored layouts (k = 1)
              "elided_one_layout": sm.FanoutGraph(D1, D2, D3, Kin, Cout, bf, sm.SM_ELIDED, 2),
              "explicit": sm.FanoutGraph(D1, D2, D3, Kin, Cout, bf, sm.SM_EXPLICIT, 1)}
        return ("extra: Fig. 4 graph MatMul -> Transpose -> Reshape -> {Reduce D3, Reduce' D1, Conv D3}, bf16, D1=512, D2=64, D3=256, "
                "Kin=256, Cout=64; redundant copy of %d bytes with k=1" % gs["elided"].plan["copy_bytes"], "graphs/s", 1,
                {n: (lambda g=g: g(ad, wd, wcd)) for n, g in gs.items()}, None, "bf16")
    if k == 8:     # the paper's decoder-only model (Pythia, Table 7) at a decode step: every Linear is a matrix-vector product
        B, E, h, L, F, rot = 8, 2048, 8, 2047, 8192, 64
        d = E // h
        x, p, kc, vc = Wl.neox_decode_case(B, E, h, L, F)
        dp, xd = dev(p, bf), x.to(bf).cuda()
        kbuf = torch.zeros(B, h, L + 1, d, dtype=bf, device="cuda")
        vbuf = torch.zeros_like(kbuf)
        kbuf[:, :, :L], vbuf[:, :, :L] = kc.to(bf).cuda(), vc.to(bf).cuda()
        st = {n: sm.DecodeStep(dp, B, E, h, F, rot, m) for n, m in (("elided", sm.SM_ELIDED), ("explicit", sm.SM_EXPLICIT))}
        return ("extra: Pythia-1B-shaped layer at a decode step, bf16, B=8 sequences, 1 new token each, hidden 2048, 8 heads x 256, "
                "64 rotary features, 2047 cached tokens, GELU MLP 8192, parallel residual", "tokens/s", B,
                {n: (lambda s_=s_: s_(xd, kbuf, vbuf, L)) for n, s_ in st.items()}, None, "bf16")
    if k == 9:     # CSwin (Tables 1, 7): cross-shaped window attention at the shape of CSwin-T's third stage
        B, H, W, C, h, sw = 64, 14, 14, 256, 8, 7
        qkv = Wl.cswin_qkv_case(B, H, W, C).to(bf).cuda()
        y = torch.empty(B, H * W, C, dtype=bf, device="cuda")
        pe = [t.to(bf).cuda() for t in Wl.cswin_lepe_params(C)]
        ops = {n: sm.CswinAttention(B, H, W, C, h, sw, m) for n, m in (("elided", sm.SM_ELIDED), ("explicit", sm.SM_EXPLICIT))}
        return ("extra: CSwin-style cross-shaped window attention with its positional encoding (depth-wise 3x3 on the values), bf16, "
                "B=64, 14x14 tokens, 256 channels, 8 heads x 32 (4 in vertical, 4 in horizontal stripes of width 7), from the fused "
                "q|k|v projection to the merged output", "images/s", B,
                {n: (lambda o=o: o(qkv, out=y, lepe=pe)) for n, o in ops.items()}, None, "bf16")
    if k == 10:    # ... and the whole CSwin block around it, at the same shape (third stage of CSwin-T)
        B, H, W, C, h, sw = 64, 14, 14, 256, 8, 7
        x, p = Wl.cswin_block_case(B, H, W, C)
        dp, xd = dev(p, bf), x.to(bf).cuda()
        y = torch.empty_like(xd)
        blk = {"elided": sm.CswinBlock(B, H, W, C, h, sw, dp, sm.SM_ELIDED), "explicit": sm.CswinBlock(B, H, W, C, h, sw, dp, sm.SM_EXPLICIT),
               "elided_per_op": sm.CswinBlock(B, H, W, C, h, sw, dp, sm.SM_ELIDED, fuse=False),
               "explicit_per_op": sm.CswinBlock(B, H, W, C, h, sw, dp, sm.SM_EXPLICIT, fuse=False)}
        return ("extra: one CSwin-T stage-3 block, bf16, B=64, 14x14 tokens, 256 channels, 8 heads x 32, stripes 7 wide, MLP 4x",
                "images/s", B, {n: (lambda b=b: b(xd, out=y)) for n, b in blk.items()}, None, "bf16")
    raise ValueError(k)


def measure(run, steps, warmup, sm, torch, traffic, tune):
    """Times `steps` calls between two synchronisations, then the same calls with per-launch HIP events.  tune: first
    one labelled pass to learn the chain's Linear shapes and the tuner on each of them (outside the timed region)."""
    tuned = None
    if tune:
        sm.timing_enable(True)
        run()
        torch.cuda.synchronize()
        labels = list(sm.timing_report().keys())
        sm.timing_enable(False)
        tuned = [t for t in sm.autotune_from_labels(labels, iters=10) if t["tile_rows"]]
    for _ in range(warmup):
        run()
    torch.cuda.synchronize()
    t0 = time.perf_counter()
    for _ in range(steps):
        run()
    torch.cuda.synchronize()
    sec = (time.perf_counter() - t0) / steps
    ev_steps = min(steps, 20)
    sm.timing_enable(True)
    for _ in range(ev_steps):
        run()
    seq = sm.timing_sequence()
    seq = seq[:len(seq) // ev_steps]      # one pass: the launch order a profiler's dispatch list is matched against
    sm.timing_calibrate(64)        # what an event pair adds to a kernel's own run time
    torch.cuda.synchronize()
    rep = sm.timing_report()
    sm.timing_enable(False)
    n, ms = rep.pop("empty_kernel")
    n2, ms2 = rep.pop("empty_pair")
    calib = {"empty_kernel_us": round(ms / n * 1e3, 3), "empty_pair_us": round(ms2 / n2 * 1e3, 3)}
    # avg_us: HIP-event time around each launch on the launch stream.  It contains the dispatch and the event records
    # themselves: a profiler's kernel duration is 2 to 3 us shorter (event_calibration: an event pair around an empty
    # kernel and around nothing)
    rows = []
    for label, (n, ms) in rep.items():
        by, fl = kernel_model(label)
        us = ms / n * 1e3
        rows.append({"kernel": label, "launches_per_step": round(n / ev_steps, 2), "avg_us": round(us, 3), "alg_bytes": by, "flops": fl,
                     "GBps": round(by / us * 1e-3, 1), "TFLOPs": round(fl / us * 1e-6, 1)})
    dom = max(rows, key=lambda r: r["avg_us"] * r["launches_per_step"])
    return {"ms_per_step": round(sec * 1e3, 4),
            "alg_bytes_per_step": int(sum(r["alg_bytes"] * r["launches_per_step"] for r in rows)),
            "flops_per_step": sum(r["flops"] * r["launches_per_step"] for r in rows),
            "launches_per_step": round(sum(r["launches_per_step"] for r in rows), 1),
            "kernel_us_per_step": round(sum(r["avg_us"] * r["launches_per_step"] for r in rows), 2),
            "roofline": roofline_of(dom, traffic), "event_calibration": calib, "kernels": rows, "launch_sequence": seq,
            "tuned_linears": None if tuned is None else [{"shape": list(t["shape"]), "tile_rows": t["tile_rows"], "stages": t["stages"],
                                                          "us": t["best_us"], "default_us": t["default_us"]} for t in tuned]}


def main():
    ap = argparse.ArgumentParser()
    ap.add_argument("--gpus", type=int, default=1)
    ap.add_argument("--steps", type=int, default=30)
    ap.add_argument("--warmup", type=int, default=5)
    ap.add_argument("--config", type=int, default=0, help="1..5: only this configuration of BASELINE.json (6: ViT block, 7: Fig. 4 graph, 8: decode step, 9: CSwin attention, 10: CSwin block); 0 = all")
    ap.add_argument("--variants", default="", help="comma-separated subset of the variants (elided, explicit, elided_per_op, explicit_per_op)")
    ap.add_argument("--kernels", action="store_true", help="include every variant's per-kernel table in the JSON line (long)")
    ap.add_argument("--no-autotune", action="store_true",
                    help="skip the tuner (sm_linear_autotune on every tiled-Linear shape of a chain before it is timed)")
    ap.add_argument("--no-cpu-baseline", action="store_true")
    ap.add_argument("--calibrate-copy", action="store_true",
                    help="also run an identity sm_gather_mapped copy of 256 MiB three times (counter calibration for rocprofv3 --pmc)")
    ap.add_argument("--fold-microbench", action="store_true",
                    help="instead of the chains: the read-versus-write folding micro-experiment of Sec. 3.2.2 on the mapped Linear")
    a = ap.parse_args()
    if a.gpus != 1:
        print("bench.py measures one GPU: this build has no multi-GPU path (--gpus %d refused)" % a.gpus, file=sys.stderr)
        sys.exit(2)

    import torch
    from paper_2404_13528_amd import binding as sm, workloads as Wl

    if a.fold_microbench:
        print(json.dumps(fold_microbench(sm, torch, a.steps, a.warmup)))
        return

    if a.calibrate_copy:
        n = 128 * 1024 * 1024                         # bf16 elements: 256 MiB read + 256 MiB written per launch
        src = torch.zeros(n, dtype=torch.bfloat16, device="cuda")
        ident = sm.Map.create((n // 1024, 1024), [])
        for _ in range(3):
            ident.gather(src.view(n // 1024, 1024))
        torch.cuda.synchronize()
        del src

    traffic = measured_traffic()
    HEAD = 3
    which = [a.config] if a.config else [3, 1, 2, 4, 5, 6, 7, 8, 9, 10]
    want = [v for v in a.variants.split(",") if v]
    configs, oracle_sample, calib = {}, None, None
    for k in which:
        desc, unit, units, variants, sample, dtype = build_config(k, sm, torch, Wl)
        if sample is not None:
            oracle_sample = sample
        entry = {"workload": desc, "unit": unit, "dtype": dtype, "variants": {}}
        for name, run in variants.items():
            if want and name not in want:
                continue
            r = measure(run, a.steps, a.warmup, sm, torch, traffic, not a.no_autotune)
            r["value"] = round(units / (r["ms_per_step"] * 1e-3), 1)
            calib = r.pop("event_calibration")
            if not a.kernels:
                del r["kernels"]
                del r["launch_sequence"]
            entry["variants"][name] = r
        v = entry["variants"]
        if "elided" in v and "explicit" in v:
            entry["elided_vs_explicit"] = {"speedup": round(v["explicit"]["ms_per_step"] / v["elided"]["ms_per_step"], 3),
                                           "alg_bytes_ratio": round(v["explicit"]["alg_bytes_per_step"] / v["elided"]["alg_bytes_per_step"], 3)}
        if "elided_per_op" in v and "explicit_per_op" in v:     # layout elimination alone (Sec. 4.3's breakdown): same kernels, copies removed
            entry["elimination_only"] = {"speedup": round(v["explicit_per_op"]["ms_per_step"] / v["elided_per_op"]["ms_per_step"], 3),
                                         "alg_bytes_ratio": round(v["explicit_per_op"]["alg_bytes_per_step"] / v["elided_per_op"]["alg_bytes_per_step"], 3)}
        if "elided" in v and "elided_per_op" in v:               # what the deeper fusion adds on top of elimination
            entry["fusion_on_top"] = {"speedup": round(v["elided_per_op"]["ms_per_step"] / v["elided"]["ms_per_step"], 3),
                                      "alg_bytes_ratio": round(v["elided_per_op"]["alg_bytes_per_step"] / v["elided"]["alg_bytes_per_step"], 3)}
        configs["config%d" % k] = entry
        del variants
        torch.cuda.empty_cache()

    hk = HEAD if ("config%d" % HEAD) in configs else which[0]
    head = configs["config%d" % hk]
    hv = head["variants"].get("elided") or next(iter(head["variants"].values()))
    out = {
        "metric": "Swin/attention block images(tokens)/s + HBM bytes vs explicit-transpose chain",
        "value": hv["value"], "unit": head["unit"],
        "n_gpus": 1, "steps": a.steps, "warmup": a.warmup,
        "ms_per_step": hv["ms_per_step"],
        "higher_is_better": True, "scaling": "weak", "vs_baseline": None,
        "dtype": head["dtype"], "data": "synthetic",
        "config": {"workload": head["workload"], "mode": "elided"},
        "roofline": hv["roofline"],
        "event_calibration": calib,
        "alg_bytes_are": "modelled from the shapes (kernel_model), not counters; roofline.traffic is the counter figure where profiles/ has one",
        "configs": configs,
    }

    if not a.no_cpu_baseline and oracle_sample is not None:
        from oracle import swin
        try:
            from threadpoolctl import threadpool_info
            cores = max([p.get("num_threads", 1) for p in threadpool_info()] or [1])
        except Exception:
            cores = os.cpu_count()
        image, net = oracle_sample
        nn = {"embed": {k: v.double().numpy() for k, v in net["embed"].items()},
              "stages": [[{k: v.double().numpy() for k, v in p.items()} for p in st] for st in net["stages"]],
              "merges": [{k: v.double().numpy() for k, v in m.items()} for m in net["merges"]],
              "head": {k: v.double().numpy() for k, v in net["head"].items()}}
        n_img, t0 = 0, time.perf_counter()
        while n_img < 2 or (time.perf_counter() - t0 < 12.0 and n_img < 64):          # about 12 s of host work
            swin.swin_net(image[n_img:n_img + 2].double().numpy(), nn, 4, SWIN_B["w"], SWIN_B["heads"])
            n_img += 2
        dt = time.perf_counter() - t0
        out["cpu_baseline"] = {"value": round(n_img / dt, 3), "unit": "images/s", "cores": cores, "kind": "oracle",
                               "sample": "%d of the 64 images of the headline workload through the whole net, two at a time, float64 numpy, %.2f s" % (n_img, dt)}
    print(json.dumps(out))


if __name__ == "__main__":
    main()

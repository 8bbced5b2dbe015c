"""GPU parity of sm_run_chain against the oracle: configuration 2 (bf16 Swin
stage-3 chain, B=32, 14x14, C=384, 12 heads, 6 blocks alternating shift 0/3) at
full size in the launch configuration the benchmark times; a reduced
Swin-B-shaped net (patch embedding, four stages, patch merging, head) in fp32
and bf16; and configuration 3 at full size with the feature map and the logits
both compared."""
import numpy as np
import pytest
import torch
from oracle import swin
from paper_2404_13528_amd import binding as sm, workloads as Wl
import functools
from util import to_np, np_params, dev, dev_params, rel_l2, assert_bf16_close

pytestmark = pytest.mark.gpu
MODES = [sm.SM_ELIDED, sm.SM_EXPLICIT]


def net_np(net):
    out = {"stages": [[np_params(b) for b in st] for st in net["stages"]]}
    if "embed" in net:
        out.update(embed=np_params(net["embed"]), merges=[np_params(m) for m in net["merges"]], head=np_params(net["head"]))
    return out


def net_dev(net, dtype):
    out = {"stages": [[dev_params(b, dtype) for b in st] for st in net["stages"]]}
    if "embed" in net:
        out.update(embed=dev_params(net["embed"], dtype), merges=[dev_params(m, dtype) for m in net["merges"]],
                   head=dev_params(net["head"], dtype))
    return out


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("fuse_mlp", [True, "mlp", False])
def test_config2_stage3_chain_full_size(mode, fuse_mlp):
    B, H, W, C, h, w, depth = 32, 14, 14, 384, 12, 7, 6
    x, blocks = Wl.swin_stage_case(B, H, W, C, h, w, depth)
    net = {"stages": [blocks]}
    chain = sm.SwinChain(B, [(C, h, depth, H, W)], w, net_dev(net, torch.bfloat16), torch.bfloat16, mode, fuse_mlp=fuse_mlp)
    y = chain(dev(x, torch.bfloat16))
    torch.cuda.synchronize()
    want = swin.swin_stage(to_np(x), net_np(net)["stages"][0], H, W, w, h)
    got = to_np(y)
    assert_bf16_close(got, want, "config-2 chain")
    assert rel_l2(got - to_np(x), want - to_np(x)) <= 3e-2
    # per block: LayerNorm-2, FC1, FC2 become one kernel; elided, the output projection joins them
    # and also computes the next block's LayerNorm-1 and QKV (the first block's run as one packed-weight Linear)
    n = 42 if not fuse_mlp else (13 if fuse_mlp is True and mode == sm.SM_ELIDED else 30)
    assert sm.launch_counts() == ((n, 0) if mode == sm.SM_ELIDED else (n, 3 * 4 + 3 * 6))


def small_net_case(dtype, mode, embed=32, heads=(1, 2), fuse_mlp=True):
    B, img, depths, w, ncls = 2, 112, (2, 2), 7, 24
    image, net = Wl.swin_net_case(B, img=img, embed=embed, depths=depths, heads=heads, w=w, n_cls=ncls,
                                  bf16=(dtype == torch.bfloat16))
    stages, H, C = [], img // 4, embed
    for dep, hh in zip(depths, heads):
        stages.append((C, hh, dep, H, H))
        H, C = H // 2, C * 2
    chain = sm.SwinChain(B, stages, w, net_dev(net, dtype), dtype, mode, img=img, n_cls=ncls, fuse_mlp=fuse_mlp)
    logits, feat = chain(dev(image, dtype), want_feat=True)
    torch.cuda.synchronize()
    f_want, l_want = swin.swin_net(to_np(image), net_np(net), 4, w, heads)
    return to_np(feat), f_want, to_np(logits), l_want


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_small_net_embed_merge_head(dtype, mode):
    f, fw, l, lw = small_net_case(dtype, mode)
    if dtype == torch.float32:
        assert np.abs(f - fw).max() <= 1e-4 * max(1.0, np.abs(fw).max()) and np.abs(l - lw).max() <= 1e-4
    else:
        assert_bf16_close(f, fw, "feature map")
        assert_bf16_close(l, lw, "logits")


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("fuse_mlp", [True, "mlp", False])
def test_small_net_with_fused_kernel_widths(mode, fuse_mlp):
    # stage widths 128 and 256 on 1568 and 392 tokens: the fused MLP / projection kernels are in play; elided and fully
    # fused, the second stage is few enough tokens for the chained tail (the row-owning one: test_gpu_split.py), and in
    # both stages block 0 also computes block 1's LayerNorm-1 and QKV through the composed reverse / shifted-partition map
    f, fw, l, lw = small_net_case(torch.bfloat16, mode, embed=128, heads=(4, 8), fuse_mlp=fuse_mlp)
    assert_bf16_close(f, fw, "feature map")
    assert_bf16_close(l, lw, "logits")
    if mode == sm.SM_ELIDED:
        # embed 2 + stage 1 (LayerNorm-1 folded into QKV: 3C <= 512) + merge 2 + stage 2 + head 3; fully fused, a
        # stage's first block is three kernels and its second starts at its attention kernel
        per_stage = {True: (3 + 2, 3 + 2), "mlp": (2 * 4, 2 * 5), False: (2 * 5, 2 * 7)}[fuse_mlp]
        assert sm.launch_counts()[0] == 2 + per_stage[0] + 2 + per_stage[1] + 3


@pytest.mark.parametrize("mode", MODES)
@pytest.mark.parametrize("fuse_mlp", [True, "mlp"])
def test_small_net_with_wide_rows(mode, fuse_mlp):
    # stage widths 256 and 512 on 1568 and 392 tokens: the second stage runs the chained tail when fully fused and elided
    # (the 64-token projection + MLP + next QKV kernel on more tokens: test_gpu_split.py), the 64-token MLP otherwise
    f, fw, l, lw = small_net_case(torch.bfloat16, mode, embed=256, heads=(8, 16), fuse_mlp=fuse_mlp)
    assert_bf16_close(f, fw, "feature map")
    assert_bf16_close(l, lw, "logits")
    if mode == sm.SM_ELIDED and fuse_mlp is True:
        assert sm.launch_counts()[0] == 2 + (3 + 2) + 2 + (3 + 2) + 3


CFG3_SAMPLE = list(range(0, 64, 4))          # 16 of the 64 images, spread over the batch (images are independent)


@functools.lru_cache(maxsize=1)
def config3_oracle():
    image, net = Wl.swin_net_case(64)
    return swin.swin_net(to_np(image[CFG3_SAMPLE]), net_np(net), 4, 7, (4, 8, 16, 32))


@pytest.mark.parametrize("mode", MODES)
def test_config3_swin_b_full_size(mode):
    B = 64
    depths, heads, w = (2, 2, 18, 2), (4, 8, 16, 32), 7
    image, net = Wl.swin_net_case(B)
    stages, H, C = [], 56, 128
    for dep, hh in zip(depths, heads):
        stages.append((C, hh, dep, H, H))
        H, C = H // 2, C * 2
    chain = sm.SwinChain(B, stages, w, net_dev(net, torch.bfloat16), torch.bfloat16, mode, img=224, n_cls=1000)
    img_d = dev(image, torch.bfloat16)
    logits_d, feat_d = chain(img_d, want_feat=True)
    torch.cuda.synchronize()
    logits, feat = to_np(logits_d), to_np(feat_d)
    f_want, l_want = config3_oracle()
    assert_bf16_close(feat[CFG3_SAMPLE], f_want, "config-3 feature map")
    assert_bf16_close(logits[CFG3_SAMPLE], l_want, "config-3 logits")
    assert np.isfinite(logits).all() and np.isfinite(feat).all()
    # the 48 images the oracle did not see: images are independent, so the batch rolled by r puts image i at the
    # position of image i + r; every position that was checked against the oracle (multiples of 4) then computes an
    # unchecked image, and its result must be exactly what that image's own position gave
    for r in (1, 2, 3):
        l_r, f_r = chain(torch.roll(img_d, r, 0).contiguous(), want_feat=True)
        torch.cuda.synchronize()
        assert torch.equal(torch.roll(f_r, -r, 0), feat_d), "feature maps depend on the batch position (roll %d)" % r
        assert torch.equal(torch.roll(l_r, -r, 0), logits_d), "logits depend on the batch position (roll %d)" % r

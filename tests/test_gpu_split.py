"""The column-split Linears (k_split.hip): single form against a torch fp64 Linear at the edges of its tiles (rows, columns
and K-tiles cut, resident panels and the ring of stages, both element types), the chained form (projection .. next QKV in
one launch) against the oracle's Swin stage."""
import pytest
import torch
from oracle import swin
from paper_2404_13528_amd import binding as sm, workloads as Wl
from util import assert_bf16_close, assert_close, dev, dev_params, np_params, to_np

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,N,K,norm,act,res", [
    (1, 8, 16, False, "none", False),            # one row, one chunk of columns, one k-step
    (31, 40, 48, True, "gelu", True),            # less than a row tile, a cut column tile, a cut K-tile
    (33, 1000, 96, False, "none", False),        # one row of a second tile, a classifier's width
    (49, 3072, 1024, True, "gelu", False),       # the widest normalised row (bf16): 32-column panels
    (65, 96, 1040, False, "gelu", True),         # K past the panels: ring of stages, its last one cut
    (196, 512, 2048, False, "none", True),       # ring, four and more stages
    (500, 520, 320, True, "none", True),         # 64-row tiles, both ends cut
    (97, 128, 384, True, "none", True),
    (33, 64, 512, True, "none", False),          # bf16: the longest row whose gamma and beta travel under its statistics,
    (33, 64, 528, True, "gelu", True),           # and the next, which asks for them piece by piece
    (257, 4104, 2064, False, "none", True),      # more 64-row tiles than CUs, a long K, all ends cut
])
def test_split_linear(M, N, K, norm, act, res, dtype):
    g = torch.Generator().manual_seed(M + N + K)
    A, W = (torch.randn(M, K, generator=g) + 0.3).to(dtype), (torch.randn(N, K, generator=g) * K ** -0.5).to(dtype)
    b, R = torch.randn(N, generator=g).to(dtype), torch.randn(M, N, generator=g).to(dtype)
    gam, bet = (1 + 0.1 * torch.randn(K, generator=g)).to(dtype), (0.1 * torch.randn(K, generator=g)).to(dtype)
    x = A.double()
    if norm:
        x = torch.nn.functional.layer_norm(x, (K,), gam.double(), bet.double(), 1e-5)
        if dtype == torch.bfloat16:
            x = x.to(dtype).double()             # the normalised row is rounded as a norm kernel would store it
    want = x @ W.double().t() + b.double()
    if act == "gelu":
        want = torch.nn.functional.gelu(want)
    if res:
        want = want + R.double()
    got = sm.linear(A.cuda(), W.cuda(), b.cuda(), residual=R.cuda() if res else None, act=act,
                    norm=("layer", gam.cuda(), bet.cuda(), 1e-5) if norm else None)
    got = got.double().cpu()
    err = (got - want).abs().max().item()
    assert err <= (2e-5 if dtype == torch.float32 else 1.2e-2) * max(1.0, want.abs().max().item()), err


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("M,K", [(31, 96), (97, 384), (65, 768), (49, 1024)])
def test_split_linear_norm_of_rows_with_a_large_mean(M, K, dtype):
    """Rows of 100 with a few elements one bf16 step (0.5) up: exact inputs whose variance, 3e-4 to 6e-2, is far below the
    rounding of the square of their mean.  The result is the normalised row itself (W = the identity)."""
    g = torch.Generator().manual_seed(K)
    A = torch.full((M, K), 100.0)
    for r in range(M):
        A[r, torch.randperm(K, generator=g)[:1 + r % 16]] = 100.5
    gam, bet = torch.ones(K), torch.zeros(K)
    want = torch.nn.functional.layer_norm(A.double(), (K,), gam.double(), bet.double(), 1e-5)
    got = sm.linear(A.to(dtype).cuda(), torch.eye(K, dtype=dtype).cuda(), norm=("layer", gam.to(dtype).cuda(), bet.to(dtype).cuda(), 1e-5))
    # fp32 statistics: the mean (100, of fp32 sums) is off by up to 8 roundings of 2^-18 against a spread of 0.018 and more;
    # bf16: the row rounded once for the product and its result once more, 2^-9 each
    tol = (8 * 2.0 ** -18 / 0.018 if dtype == torch.float32 else 2.0 ** -8 + 8 * 2.0 ** -18 / 0.018)
    err = ((got.double().cpu() - want).norm(dim=1) / want.norm(dim=1)).max().item()
    assert err <= tol, err


@pytest.mark.parametrize("B,H,C,depth", [
    (1, 14, 512, 3),       # 32-row tiles: one per XCD but one
    (3, 14, 512, 2),       # 64-row tiles, two per group for some
    (1, 14, 384, 4),
    (2, 14, 256, 2),
    (1, 7, 1024, 2),       # a width without a fused kernel; two row tiles
    (5, 7, 768, 2),        # 245 rows: the last tile is cut
])
def test_split_chain_matches_the_oracle(B, H, C, depth):
    h = C // 32
    x, blocks = Wl.swin_stage_case(B, H, H, C, h, 7, depth, seed=B + C)
    net = {"stages": [[dev_params(p, torch.bfloat16) for p in blocks]]}
    chain = sm.SwinChain(B, [(C, h, depth, H, H)], 7, net, torch.bfloat16)
    want = swin.swin_stage(to_np(x), [np_params(p) for p in blocks], H, H, 7, h)
    for _ in range(2):                           # the counters are cleared by every call
        y = chain(dev(x, torch.bfloat16))
        torch.cuda.synchronize()
        assert_bf16_close(y, want, "stage", x=to_np(x))
    assert sm.launch_counts() == (1 + 2 * depth, 0)      # LayerNorm + QKV, then attention and one chained launch per block


def _labels(f):
    sm.timing_enable(True)
    try:
        f()
        torch.cuda.synchronize()
        return sm.timing_sequence()
    finally:
        sm.timing_enable(False)


@pytest.mark.parametrize("C,T,chained", [(128, 49, False), (128, 98, False), (256, 49, True), (96, 49, True), (192, 98, True),
                                         (256, 588, False), (384, 1274, True), (384, 1323, False), (512, 2303, True), (512, 2352, False),
                                         (768, 245, True), (768, 294, False)])
def test_which_blocks_run_the_chained_tail(C, T, chained):
    x, p = Wl.swin_block_case(T // 49, 7, 7, C, C // 32, 7, seed=C, bf16=True, std=0.1)
    blk = sm.SwinBlock(T // 49, 7, 7, C, C // 32, 7, 0, dev_params(p, torch.bfloat16), torch.bfloat16)
    x = dev(x, torch.bfloat16)
    y = []
    labels = _labels(lambda: y.append(blk(x)))
    assert any(l.startswith("split_proj+ln+mlp") for l in labels) == chained, labels
    if T < 600:
        assert_bf16_close(y[0], swin.swin_block(to_np(x), np_params(p), 7, 7, 7, C // 32, 0), "block", x=to_np(x))


BF16, F32 = torch.bfloat16, torch.float32


@pytest.mark.parametrize("M,N,K,dtype,norm,split", [
    (500, 1024, 1024, BF16, True, True),         # LayerNorm over a wide row: two rounds of 32 x 32 tiles
    (245, 2304, 768, BF16, True, True),          # a little more
    (300, 3072, 768, BF16, True, False),
    (300, 1728, 576, BF16, True, False),
    (196, 3072, 1024, BF16, True, True),         # three rounds over a wider one
    (784, 1024, 1024, BF16, True, False),
    (2560, 320, 512, F32, True, True),           # fp32: four
    (1066, 1536, 288, F32, True, False),
    (256, 4096, 4096, BF16, False, True),        # one round of 64 x 64 tiles, more
    (257, 4096, 4096, BF16, False, False),
    (500, 4096, 4096, BF16, False, False),
    (3072, 960, 192, F32, False, True),          # fp32: three rounds of 64 x 64 tiles
    (6400, 512, 768, F32, False, False),
    (57600, 32, 192, F32, False, True),          # a narrow result: four
    (66000, 32, 192, F32, False, False),
    (196, 1536, 512, BF16, True, True),          # rows that fit
    (784, 1536, 512, BF16, True, False),
])
def test_which_linears_are_split(M, N, K, dtype, norm, split):
    g = torch.Generator().manual_seed(M + K)
    A, W = torch.randn(M, K, generator=g).to(dtype), (torch.randn(N, K, generator=g) * K ** -0.5).to(dtype)
    x, nm = A.double(), None
    if norm:
        nm = ("layer", torch.ones(K, dtype=dtype).cuda(), torch.zeros(K, dtype=dtype).cuda(), 1e-5)
        x = torch.nn.functional.layer_norm(x, (K,), eps=1e-5).to(dtype).double()
    got = []
    labels = _labels(lambda: got.append(sm.linear(A.cuda(), W.cuda(), norm=nm)))
    assert labels[0].startswith("%s%sgemm_" % ("ln+" if norm else "", "split" if split else "")), labels
    want = x @ W.double().t()
    err = (got[0].double().cpu() - want).norm().item() / want.norm().item()
    assert err <= (2e-6 if dtype == F32 else 4e-3), err      # fp32 sums of K products; bf16: the result rounded once, 2^-9, and a few flips of the normalised row


@pytest.mark.parametrize("C,ratio,B,H", [(160, 3, 1, 14), (96, 4, 1, 7), (512, 3, 1, 14), (384, 2, 1, 14), (384, 6, 3, 14), (640, 1, 1, 14), (1024, 5, 5, 7)])
def test_a_block_alone_with_the_chained_tail(C, ratio, B, H):
    """sm_swin_block's own use of the chain, widths and MLP widths around the usual ones: against the oracle, on the static
    workspace, in place, replayed from a graph; the same bits every time."""
    h, shift = C // 32, 3 if H > 7 else 0
    x, p = Wl.swin_block_case(B, H, H, C, h, 7, seed=C + ratio, bf16=True, std=0.1)
    g = torch.Generator().manual_seed(C)
    p = dict(p, w1=(0.1 * torch.randn(ratio * C, C, generator=g)).bfloat16().to(p["w1"].dtype), b1=(0.1 * torch.randn(ratio * C, generator=g)).bfloat16().to(p["b1"].dtype),
             w2=(0.1 * torch.randn(C, ratio * C, generator=g)).bfloat16().to(p["w2"].dtype))
    blk = sm.SwinBlock(B, H, H, C, h, 7, shift, dev_params(p, torch.bfloat16), torch.bfloat16, mlp_ratio=ratio)
    xd, got = dev(x, torch.bfloat16), []
    labels = _labels(lambda: got.append(blk(xd)))
    assert any(l.startswith("split_proj+ln+mlp") for l in labels), labels
    assert_bf16_close(got[0], swin.swin_block(to_np(x), np_params(p), H, H, 7, h, shift), "block", x=to_np(x))
    assert torch.equal(sm.swin_block_static(blk, xd), got[0])
    static, out = xd.clone(), torch.empty_like(xd)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        blk(static, out=out)
    for i in range(3):
        x2 = xd if i != 1 else -xd
        static.copy_(x2)
        graph.replay()
        torch.cuda.synchronize()
        want = blk(x2)
        torch.cuda.synchronize()
        assert torch.equal(out, want)
        assert i == 1 or torch.equal(want, got[0])
    assert torch.equal(blk(xd, out=xd), got[0])          # in place


@pytest.mark.parametrize("B,H,C", [(1, 28, 256), (12, 14, 512)])
def test_row_owning_tail_above_the_chain(B, H, C):
    """The projection + MLP + next LayerNorm + QKV kernels of 32 and 64 tokens, at the first batch above the chain's sizes."""
    h = C // 32
    x, blocks = Wl.swin_stage_case(B, H, H, C, h, 7, 2, seed=C)
    chain = sm.SwinChain(B, [(C, h, 2, H, H)], 7, {"stages": [[dev_params(p, torch.bfloat16) for p in blocks]]}, torch.bfloat16)
    got, xd = [], dev(x, torch.bfloat16)
    labels = _labels(lambda: got.append(chain(xd)))
    assert "proj+ln+mlp_bf16[%d,%d,%d]+ln+qkv" % (B * H * H, 4 * C, C) in labels, labels
    assert_bf16_close(got[0], swin.swin_stage(to_np(x), [np_params(p) for p in blocks], H, H, 7, h), "stage", x=to_np(x))


@pytest.mark.parametrize("ratio", [18, 19])
def test_row_owning_tail_with_a_very_wide_hidden_layer(ratio):
    """C = 512: the kernel's vectors in LDS, and beside a hidden layer whose bias takes their place."""
    B, H, C, h = 12, 14, 512, 16
    dr = Wl.Draw(ratio, True)
    x = dr.normal(B, H * H, C)
    blocks = [Wl.swin_block_params(dr, C, h, 7, ratio) for _ in range(2)]
    chain = sm.SwinChain(B, [(C, h, 2, H, H)], 7, {"stages": [[dev_params(p, torch.bfloat16) for p in blocks]]}, torch.bfloat16, mlp_ratio=ratio)
    got, xd = [], dev(x, torch.bfloat16)
    labels = _labels(lambda: got.append(chain(xd)))
    assert "proj+ln+mlp_bf16[%d,%d,%d]+ln+qkv" % (B * H * H, ratio * C, C) in labels, labels
    assert_bf16_close(got[0], swin.swin_stage(to_np(x), [np_params(p) for p in blocks], H, H, 7, h), "stage", x=to_np(x))


@pytest.mark.parametrize("M,N,K,dtype,norm,act,res", [
    (1100, 1000, 128, BF16, None, "gelu", True),         # LDS-DMA staging, ragged rows and columns
    (1100, 1000, 104, BF16, None, "gelu", True),         # register staging, a cut K-tile
    (1100, 1000, 104, BF16, "layer", "gelu", True),
    (6500, 520, 72, F32, None, "gelu", True),
    (6500, 520, 72, F32, "layer", "none", False),
    (70, 100, 64, BF16, None, "gelu", True),             # columns that the column-split kernel does not take
    (33, 40, 48, BF16, "layer without shift", "gelu", True),
    (33, 40, 48, F32, "rms", "none", True),
])
def test_tiled_linear_beside_the_split_one(M, N, K, dtype, norm, act, res):
    g = torch.Generator().manual_seed(M + K)
    A, W = (torch.randn(M, K, generator=g) + 0.3).to(dtype), (torch.randn(N, K, generator=g) * K ** -0.5).to(dtype)
    b, R = torch.randn(N, generator=g).to(dtype), torch.randn(M, N, generator=g).to(dtype)
    gam, bet = (1 + 0.1 * torch.randn(K, generator=g)).to(dtype), (0.1 * torch.randn(K, generator=g)).to(dtype)
    x, nm = A.double(), None
    if norm == "rms":
        x, nm = x / torch.sqrt((x * x).mean(1, keepdim=True) + 1e-5) * gam.double(), ("rms", gam.cuda(), None, 1e-5)
    elif norm:
        with_shift = norm == "layer"
        x = torch.nn.functional.layer_norm(x, (K,), gam.double(), bet.double() if with_shift else None, 1e-5)
        nm = ("layer", gam.cuda(), bet.cuda() if with_shift else None, 1e-5)
    if norm and dtype == BF16:
        x = x.to(dtype).double()                 # the normalised row is rounded as a norm kernel would store it
    want = x @ W.double().t() + b.double()
    if act == "gelu":
        want = torch.nn.functional.gelu(want)
    if res:
        want = want + R.double()
    got = []
    labels = _labels(lambda: got.append(sm.linear(A.cuda(), W.cuda(), b.cuda(), residual=R.cuda() if res else None, act=act, norm=nm)))
    assert len(labels) == 1 and "splitgemm" not in labels[0], labels
    err = (got[0].double().cpu() - want).abs().max().item()
    assert err <= (2e-5 if dtype == torch.float32 else 1.2e-2) * max(1.0, want.abs().max().item()), err      # as above


@pytest.mark.parametrize("C,T,form", [(128, 2352, "ln+splitgemm"), (128, 2744, "ln+pgemm"), (256, 2548, "ln+gemm"), (256, 2940, "ln+pgemm"),
                                      (384, 3528, "ln+gemm"), (384, 3724, "ln+pgemm"), (512, 784, "ln+gemm")])
def test_which_form_the_first_qkv_has(C, T, form):
    x, p = Wl.swin_block_case(T // 49, 7, 7, C, C // 32, 7, seed=C, bf16=True, std=0.1)
    p, x = dev_params(p, torch.bfloat16), dev(x, torch.bfloat16)
    blk = sm.SwinBlock(T // 49, 7, 7, C, C // 32, 7, 0, p, torch.bfloat16)
    labels = _labels(lambda: blk(x))
    assert any(l.startswith("%s_bf16[%d,%d,%d]" % (form, T, 3 * C, C)) for l in labels), labels
    # a 7 x 7 grid: the windows are the tokens' order
    want = sm.linear(x, p["wqkv"], p["bqkv"], norm=("layer", p["ln1_g"], p["ln1_b"], 1e-5))
    got = sm.swin_block_intermediates(blk)["qkv"].reshape(T, 3 * C)
    assert (got.float() - want.reshape(T, 3 * C).float()).norm() <= 4e-3 * want.float().norm()      # bf16: rounded once each


def test_per_operator_blocks_on_few_tokens_run_split_linears():
    """fuse_mlp=False at a fused width: one kernel per operator, the projection with its row table among the split ones."""
    x, p = Wl.swin_block_case(1, 14, 14, 256, 8, 7, seed=9, bf16=True, std=0.1)
    blk = sm.SwinBlock(1, 14, 14, 256, 8, 7, 3, dev_params(p, BF16), BF16, fuse_mlp=False)
    xd, got = dev(x, BF16), []
    labels = _labels(lambda: got.append(blk(xd)))
    for want in ("splitgemm_bf16[196,768,256]", "splitgemm_bf16[196,256,256]+res+scatter", "splitgemm_bf16[196,1024,256]+gelu", "splitgemm_bf16[196,256,1024]+res"):
        assert want in labels, (want, labels)
    assert_bf16_close(got[0], swin.swin_block(to_np(x), np_params(p), 14, 14, 7, 8, 3), "block", x=to_np(x))


def _few_tokens_block(C, **kw):
    x, p = Wl.swin_block_case(1, 14, 14, C, C // 32, 7, seed=C + 1, bf16=True)
    blk = sm.SwinBlock(1, 14, 14, C, C // 32, 7, 3, dev_params(p, torch.bfloat16), torch.bfloat16, **kw)
    return blk, dev(x, torch.bfloat16), to_np(x), np_params(p)


@pytest.mark.parametrize("offset", [None, 8])
@pytest.mark.parametrize("names", [("wqkv",), ("wproj",), ("w1", "w2"), ("wqkv", "wproj", "w1", "w2")])
def test_row_major_weights_may_be_absent_where_packed_ones_are_given(names, offset):
    """A caller who packed the weights need not keep the row-major matrices (absent, or at an address that no kernel may read)."""
    blk, x, x_np, p = _few_tokens_block(512)
    packed = sm.linear_pack(blk.params["wqkv"])
    blk.w.qkv_packed = packed.data_ptr()
    for n in names:
        setattr(blk.w, n, None if offset is None else getattr(blk.w, n) + offset)
    assert_bf16_close(blk(x), swin.swin_block(x_np, p, 14, 14, 7, 16, 3), "block", x=x_np)


@pytest.mark.parametrize("names", [("bqkv",), ("bproj", "b2"), ("b1",), ("ln1_b",), ("ln2_b",)])
def test_absent_biases_of_a_block_on_few_tokens(names):
    """A width without a fused kernel: biases and norm shifts may be absent."""
    blk, x, x_np, p = _few_tokens_block(768)
    for n in names:
        setattr(blk.w, n, None)
        p[n] = 0 * p[n]
    assert_bf16_close(blk(x), swin.swin_block(x_np, p, 14, 14, 7, 24, 3), "block", x=x_np)


@pytest.mark.parametrize("dtype,C", [(torch.float32, 192), (torch.bfloat16, 192), (torch.bfloat16, 768)])
def test_blocks_with_eps_zero(dtype, C):
    """The separate norm kernels take eps = 0 (here: every row has a spread)."""
    h = C // 32
    x, p = Wl.swin_block_case(1, 14, 14, C, h, 7, seed=C + 2, bf16=dtype == torch.bfloat16)
    y = sm.SwinBlock(1, 14, 14, C, h, 7, 3, dev_params(p, dtype), dtype, eps=0.0)(dev(x, dtype))
    want = swin.swin_block(to_np(x), np_params(p), 14, 14, 7, h, 3)      # eps 1e-5 beside variances of 1: 5e-6 of the norm's output
    if dtype == torch.float32:
        assert_close(y, want, dtype, "block")
    else:
        assert_bf16_close(y, want, "block", x=to_np(x))


def test_eps_zero_is_refused_by_the_fused_kernels():
    blk, x, _, _ = _few_tokens_block(512, eps=0.0)
    with pytest.raises(sm.SmError, match="eps > 0"):
        blk(x)


NEEDED = [(C, n) for C in (512, 768) for n in ("ln1_g", "ln2_g")] + [(768, n) for n in ("wqkv", "wproj", "w1", "w2")] + \
    [(512, n) for n in ("ln2_b", "bproj", "b1", "b2")]


@pytest.mark.parametrize("C,name,absent", [n + (a,) for n in NEEDED for a in (True, False)] +
                         [(512, n, False) for n in ("mlp_packed", "proj_packed", "qkv_packed")])
def test_missing_or_misaligned_weights_of_a_block_on_few_tokens_are_refused(C, name, absent):
    blk, x, _, _ = _few_tokens_block(C)
    setattr(blk.w, name, None if absent else getattr(blk.w, name) + 8)
    with pytest.raises(sm.SmError, match="null pointer|aligned"):
        blk(x)
    torch.cuda.synchronize()


@pytest.mark.parametrize("H,W,C,shift", [(14, 14, 192, 3), (7, 7, 768, 0), (14, 14, 1024, 3)])
def test_intermediates_of_a_block_with_the_chained_tail(H, W, C, shift):
    """Widths without a fused kernel: one kernel per operator or the chain leave x1 and the hidden activation in token order."""
    h = C // 32
    x, p = Wl.swin_block_case(1, H, W, C, h, 7, seed=C, bf16=True)
    blk = sm.SwinBlock(1, H, W, C, h, 7, shift, dev_params(p, torch.bfloat16), torch.bfloat16, fuse_mlp=False)
    y = blk(dev(x, torch.bfloat16))
    torch.cuda.synchronize()
    got = {k: to_np(v) for k, v in sm.swin_block_intermediates(blk).items()}
    want = swin.swin_block(to_np(x), np_params(p), H, W, 7, h, shift, want_all=True)
    for name in ("qkv", "o", "x1", "hid"):
        assert_bf16_close(got[name], want[name], name)
    assert_bf16_close(to_np(y), want["y"], "y", x=to_np(x))


@pytest.mark.parametrize("M,N,K,act", [
    (70, 2112, 1088, "swiglu"),        # 64-row tiles, cut ends, the shortest long K
    (257, 5696, 1088, "swiglu"),       # 64- or 128-row tiles, more than one round of the smaller
    (520, 22016, 1088, "swiglu"),      # several rounds
    (1025, 6152, 1152, "none"),        # 256-row tiles, a cut row tile
    (1652, 5120, 1152, "none"),        # 64-row tiles, two stages
    (1059, 3080, 1536, "none"),        # 128-row tiles, three stages
    (2300, 576, 1984, "swiglu"),       # 64-row tiles, three stages
])
def test_long_k_tiles(M, N, K, act):
    g = torch.Generator().manual_seed(M + N)
    A, W = torch.randn(M, K, generator=g).bfloat16(), (torch.randn(N, K, generator=g) * K ** -0.5).bfloat16()
    z = A.cuda().float() @ W.cuda().float().t()
    want = torch.nn.functional.silu(z[:, :N // 2]) * z[:, N // 2:] if act == "swiglu" else z
    got = sm.linear(A.cuda(), W.cuda(), None, act=act).float()
    assert (got - want).norm().item() <= 4e-3 * want.norm().item()      # bf16 result: relative rounding 2^-9, fp32 sums


@pytest.mark.parametrize("B,C,single", [(20, 384, False), (21, 384, True), (21, 512, True)])
def test_chains_of_more_than_two_row_tiles_per_xcd_run_single_linears(B, C, single):
    """980 and 1029 tokens, 21 windows: the last tiles of 64 rows are cut."""
    h = C // 32
    x, blocks = Wl.swin_stage_case(B, 7, 7, C, h, 7, 2, seed=B)
    chain = sm.SwinChain(B, [(C, h, 2, 7, 7)], 7, {"stages": [[dev_params(p, torch.bfloat16) for p in blocks]]}, torch.bfloat16)
    got, xd = [], dev(x, torch.bfloat16)
    labels = _labels(lambda: got.append(chain(xd)))
    assert any(l.startswith("split_proj+ln+mlp") for l in labels) != single and any("mlp_bf16" in l for l in labels) != single, labels
    assert_bf16_close(got[0], swin.swin_stage(to_np(x), [np_params(p) for p in blocks], 7, 7, 7, h), "stage", x=to_np(x))

"""The large-tile Linear (k_tile.hip) against gemm_kernel's 64-row form, which sums in the same order: the results are the same
bits.  Every case names the tile that its shape is to run in: each of the seven, rows and columns cut, one round of tiles and
several, K-tiles from 12 to 64, odd counts among them."""
import pytest
import torch
from paper_2404_13528_amd import binding as sm, workloads as Wl
from util import dev, dev_params

pytestmark = pytest.mark.gpu


def labelled(f):
    """f's result and the labels of the kernels it launched"""
    sm.timing_enable(True)
    try:
        return f(), sm.timing_sequence()
    finally:
        sm.timing_enable(False)


@pytest.mark.parametrize("M,N,K,act,res,rope,tile", [
    (4147, 928, 1088, "none", True, None, "128x192"),
    (834, 4672, 1088, "swiglu", False, None, "128x192"),
    (1292, 5440, 1280, "gelu", False, None, "128x256"),
    (4685, 832, 1088, "none", True, None, "192x128"),
    (5705, 656, 1088, "gelu", True, None, "192x128"),
    (1677, 4680, 1088, "gelu", False, None, "192x192"),
    (3335, 2368, 1088, "geglu", True, None, "192x192"),
    (2148, 4096, 1088, "swiglu", False, None, "192x256"),
    (5436, 1544, 1088, "gelu", True, None, "256x192"),
    (2041, 6144, 1088, "none", False, (4096, 128, 700, 10000.0), "256x192"),
    (2041, 8184, 2048, "none", True, None, "256x256"),                          # one round
    (1025, 12288, 4096, "none", False, (8192, 128, 1025, 10000.0), "256x256"),
    (4100, 9984, 2048, "swiglu", True, None, "256x256"),                        # several rounds
    (333, 11264, 2048, "swiglu", False, None, "192x128"),                       # few rows
    (1025, 4096, 4096, "none", True, None, "192x128"),                          # 64 K-tiles
    (6304, 2304, 768, "none", False, None, "256x256"),                          # 12
])
def test_tile_linear_is_the_tiled_kernel(M, N, K, act, res, rope, tile):
    g = torch.Generator().manual_seed(M + N + K)
    A, W = torch.randn(M, K, generator=g).bfloat16().cuda(), (torch.randn(N, K, generator=g) * K ** -0.5).bfloat16().cuda()
    b = None if rope else torch.randn(N, generator=g).bfloat16().cuda()
    R = torch.randn(M, N // 2 if "glu" in act else N, generator=g).bfloat16().cuda() if res else None
    run = lambda: sm.linear(A, W, b, residual=R, act=act, rope=rope)
    got, labels = labelled(run)
    assert len(labels) == 1 and labels[0].endswith("+tile" + tile), labels
    again = run()
    try:
        sm.gemm_tuning(64, 2)
        want, labels = labelled(run)
    finally:
        sm.gemm_tuning(0, 0)
    assert len(labels) == 1 and "+tile" not in labels[0], labels
    assert torch.isfinite(want.float()).all()
    assert torch.equal(got, want) and torch.equal(again, want)


@pytest.mark.parametrize("M,N,K,act,res,rope", [
    (33, 3072, 1024, "none", False, (2048, 128, 33, 10000.0)),      # 16 tiles: a fifth and more slower there than in gemm_kernel
    (241, 3072, 1024, "none", False, (2048, 128, 241, 10000.0)),    # 32
    (577, 4096, 11008, "none", True, None),                         # 110
    (354, 6464, 10240, "swiglu", False, None),                      # 102
    (14848, 640, 640, "none", True, None),                          # a short K and a residual
    (4702, 5184, 1088, "gelu", False, None),                        # near ties
    (1661, 4096, 11008, "none", True, None),
])
def test_large_tiles_only_where_they_are_faster(M, N, K, act, res, rope):
    A, W = torch.zeros(M, K, device="cuda").bfloat16(), torch.zeros(N, K, device="cuda").bfloat16()
    R = torch.zeros(M, N, device="cuda").bfloat16() if res else None
    _, labels = labelled(lambda: sm.linear(A, W, residual=R, act=act, rope=rope))
    assert len(labels) == 1 and labels[0].startswith("gemm_bf16[") and "+tile" not in labels[0], labels


@pytest.mark.parametrize("B,C,tile", [
    (65, 704, "192x256"),       # one round, the last row of tiles and the last column of them cut
    (130, 960, "256x192"),      # 500 tiles: a workgroup's second one
])
def test_result_and_residual_by_a_row_table(B, C, tile):
    """The output projection of a Swin block stores its rows in token order and adds the residual there."""
    H, w, h = 14, 7, C // 32
    g = torch.Generator(device="cuda").manual_seed(C)
    rnd = lambda *s, std=1.0, mean=0.0: (torch.randn(*s, generator=g, device="cuda") * std + mean).bfloat16()
    p = {"ln1_g": rnd(C, std=0.1, mean=1.0), "ln1_b": rnd(C), "wqkv": rnd(3 * C, C, std=C ** -0.5), "bqkv": rnd(3 * C), "rpb_table": rnd(169, h),
         "wproj": rnd(C, C, std=C ** -0.5), "bproj": rnd(C), "ln2_g": rnd(C, std=0.1, mean=1.0), "ln2_b": rnd(C), "w1": rnd(4 * C, C, std=C ** -0.5),
         "b1": rnd(4 * C), "w2": rnd(C, 4 * C, std=(4 * C) ** -0.5), "b2": rnd(C)}
    x = rnd(B, H * H, C)
    blk = sm.SwinBlock(B, H, H, C, h, w, 3, p, torch.bfloat16)
    got, labels = labelled(lambda: blk(x))
    assert "gemm_bf16[%d,%d,%d]+res+scatter+tile%s" % (B * H * H, C, C, tile) in labels, labels
    try:
        sm.gemm_tuning(64, 2)
        want, labels = labelled(lambda: blk(x))
    finally:
        sm.gemm_tuning(0, 0)
    assert not any("+tile" in t for t in labels), labels
    assert torch.isfinite(want.float()).all() and torch.equal(got, want)


@pytest.mark.parametrize("kind,B,S,E,h,F,cut", [
    ("llama", 1, 333, 4096, 32, 11008, 2),      # both Linears with a residual
    ("llama", 3, 235, 2048, 16, 5696, 1),       # only the long one; 89 K-tiles, runs of unequal length
    ("vit", 2, 577, 1024, 16, 4096, 1),         # a bias
    ("llama", 1, 333, 1024, 8, 2816, 0),        # short K: never cut
])
def test_cut_linears_of_a_block(kind, B, S, E, h, F, cut):
    """The Linears with a residual cut over K against the same block with a workspace that has no room for their parts: the same
    products summed in another order and one rounding less, so outputs (O(1)) differ by roundings of x1 and of the result to bf16:
    at most 2^-8 each, a third of it in the mean square."""
    x, p = Wl.llama_case(B, S, E, F, seed=S, std=E ** -0.5) if kind == "llama" else Wl.vit_case(B, S, E, h, F, seed=S, std=E ** -0.5)
    x, p = dev(x, torch.bfloat16), dev_params(p, torch.bfloat16)
    blk = sm.AttnBlock(kind, p, torch.bfloat16, B=B, S=S, E=E, heads=h, F=F)
    got, labels = labelled(lambda: blk(x))
    assert len([t for t in labels if t.startswith("cutgemm_bf16")]) == cut, labels
    # a label stands for one kernel: a dispatch list of the same call can be matched to them
    assert len([t for t in labels if not t.startswith("fill_row_tables")]) == sum(sm.launch_counts()), labels
    again, full = blk(x), blk.ws
    assert torch.equal(got, again) and torch.isfinite(got.float()).all()
    blk.ws = full[:16]
    with pytest.raises(sm.SmError, match="needed") as e:      # the error names what every call needs
        blk(x)
    need = int(str(e.value).split(",")[-1].split()[0])
    assert need <= full.numel() and (need < full.numel()) == (cut > 0)
    blk.ws = full[:need - 1]
    with pytest.raises(sm.SmError):
        blk(x)
    blk.ws = full[:need]
    want, labels = labelled(lambda: blk(x))
    assert not any("cutgemm" in t or "sum_parts" in t for t in labels), labels
    err = ((got.float() - want.float()).norm() / want.float().norm()).item()
    assert err <= 2 * 2 ** -8, err


# the tiles and numbers of parts that the plan takes; runs of unequal length (88 K-tiles in five, 172 in three, eight), rows of half a
# step of the sum kernel, one, one and a part, and two, the last with either norm behind it
@pytest.mark.parametrize("kind,T,E,F,first,second", [
    ("llama", 333, 4096, 11008, "192x128x4", "192x128x4"),
    ("llama", 71, 4096, 11008, "128x192x8", "128x192x8"),
    ("llama", 600, 4096, 11008, "128x256x3", "128x256x3"),
    ("llama", 700, 4096, 11008, "192x128x2", "192x256x4"),
    ("llama", 530, 2048, 5632, None, "192x128x5"),
    ("vit", 300, 4096, 4096, "192x128x4", "192x128x4"),
    ("vit", 90, 4096, 4096, "128x192x8", "128x192x8"),
    ("vit", 1171, 2560, 10240, None, "256x256x5"),
    ("vit", 1170, 1024, 4096, None, "192x128x4"),
])
def test_cut_linears_against_float64(kind, T, E, F, first, second):
    """One token per sequence, so that attention returns its values, a part of the QKV Linear's result.  With an MLP of zeros the
    block returns x1 = v Wo^T + bo + x: where that Linear is cut, one rounding to bf16 (half a unit in the last of eight places)
    and sums in fp32 (K terms of about K^-1/2: below 1e-5), else a second rounding in front of the residual.  With it, y - x1
    is the MLP of the norm of that x1, within the roundings of the activation and of y: at most 2^-8 of each."""
    g = torch.Generator(device="cuda").manual_seed(T + E)
    rnd = lambda *s, std=1.0, mean=0.0: (torch.randn(*s, generator=g, device="cuda") * std + mean).bfloat16()
    mat = lambda n, k: rnd(n, k, std=k ** -0.5)
    llama, F1 = kind == "llama", F * (2 if kind == "llama" else 1)
    x, wqkv, wo, w1, w2 = rnd(T, 1, E), mat(3 * E, E), mat(E, E), mat(F1, E), mat(E, F)
    vec = lambda n: None if llama else rnd(n, std=0.5)
    g1, g2, be1, be2, bqkv, bo, b1, b2 = rnd(E, std=0.2, mean=1.0), rnd(E, std=0.2, mean=1.0), vec(E), vec(E), vec(3 * E), vec(E), vec(F), vec(E)
    if llama:
        p = {"rms1_g": g1, "wq": wqkv[:E], "wk": wqkv[E:2 * E], "wv": wqkv[2 * E:], "wo": wo, "rms2_g": g2, "wgate": w1[:F], "wup": w1[F:], "wdown": w2}
    else:
        p = {"ln1_g": g1, "ln1_b": be1, "wqkv": wqkv, "bqkv": bqkv, "wo": wo, "bo": bo, "ln2_g": g2, "ln2_b": be2, "w1": w1, "b1": b1, "w2": w2, "b2": b2}
    run = lambda q: labelled(lambda: sm.AttnBlock(kind, q, torch.bfloat16, B=T, S=1, E=E, heads=E // 128, F=F)(x))
    zero = {n: torch.zeros_like(p[n]) for n in (("wdown",) if llama else ("w2", "b2"))}
    y, labels = run(p)
    assert [t.split("+tile")[1] for t in labels if t.startswith("cutgemm_")] == [t for t in (first, second) if t], labels
    x1, _ = run({**p, **zero})
    x1, y = x1.view(T, E).double(), y.view(T, E).double()
    add = lambda t: 0 if t is None else t.double()
    n0 = sm.norm(x.view(T, E), g1, be1, eps=1e-5, rms=llama)
    qkv = sm.linear(n0, wqkv, bqkv, rope=(2 * E, 128, 1, 10000.0) if llama else None)      # as the block runs it: the same bits
    want = qkv[:, 2 * E:].double() @ wo.double().t() + add(bo) + x.view(T, E).double()
    half = lambda t: 2 ** -8 * torch.exp2(torch.floor(torch.log2(t.abs().clamp_min(1e-6))))
    assert ((x1 - want).abs() <= 1.01 * (half(want) + (0 if first else half(want - x.view(T, E).double()))) + 1e-5).all()
    d = x1 if llama else x1 - x1.mean(-1, keepdim=True)
    n = (d * (d.square().mean(-1, keepdim=True) + 1e-5).rsqrt() * g2.double() + add(be2)).bfloat16().double()
    h = n @ w1.double().t() + add(b1)
    h = torch.nn.functional.silu(h[:, :F]) * h[:, F:] if llama else torch.nn.functional.gelu(h)
    branch = h.bfloat16().double() @ w2.double().t() + add(b2)
    err = ((y - x1 - branch).norm() / branch.norm()).item()
    assert err <= 2 ** -8 * (1 + (y.norm() / branch.norm()).item()), err


def test_a_picked_tile_takes_the_place_of_the_cut():
    """A tile forced or remembered for the Linear that runs, and only for that one: the tuner's entry of a Linear without the
    residual is another shape's."""
    B, S, E, F = 1, 333, 4096, 11008
    x, p = Wl.llama_case(B, S, E, F, seed=5, std=E ** -0.5)
    x = dev(x, torch.bfloat16)
    blk = sm.AttnBlock("llama", dev_params(p, torch.bfloat16), torch.bfloat16, B=B, S=S, E=E, heads=32, F=F)
    cuts = lambda: sorted(int(t.split("[")[1].split("]")[0].split(",")[2]) for t in labelled(lambda: blk(x))[1] if t.startswith("cutgemm_"))
    assert cuts() == [E, F]
    try:
        sm.gemm_tuning(64, 2)
        assert cuts() == []
        sm.gemm_tuning(0, 0)
        picked = [sm.linear_autotune(S, E, K, residual=False, iters=5)["tile_rows"] for K in (E, F)]
        assert cuts() == [E, F], picked
        tuned = {K: sm.linear_autotune(S, E, K, residual=True, iters=5)["tile_rows"] for K in (E, F)}
        assert cuts() == [K for K in (E, F) if not tuned[K]], tuned
    finally:
        sm.gemm_tuning(0, 0)
        sm.lib().sm_linear_autotune_clear()

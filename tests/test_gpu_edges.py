"""Edges of the dispatch rules and tiles of the backward kernels, each layer through the tensor-level entry
points against the CPU oracle (tolerances per output tensor as in test_gpu_parity.py)."""
import numpy as np
import pytest
import torch

import paper_2301_00330_amd.binding as B
import paper_2301_00330_amd.torch_api as T
from test_gpu_parity import TOL, mk, odesc, randn, rel_err, to64

pytestmark = pytest.mark.gpu


def check_filtered(oracle, case, dtype, groups=1):
    N, Ci, Co, H, W, K, s, r = case
    d = mk(N, Ci, Co, H, W, K, s, K // 2, g=groups, r=r, dtype=dtype)
    od = odesc(oracle, d)
    sh = T.shapes(d)
    x, w = randn(sh["x"], 1, dtype, relu=True), randn(sh["w"], 2, dtype, scale=(2.0 * groups / (Ci * K * K)) ** 0.5)
    gy = randn(sh["g_y"], 3, dtype, scale=1e-2)
    x_u = T.pool_activation(d, x.cuda())
    g_w, g_x, gy_u = T.conv_bwd_filtered(d, gy.cuda(), x_u, w.cuda())
    n_w, n_x, none = T.conv_bwd_filtered(d, gy.cuda(), x_u, w.cuda(), want_gyu=False)
    torch.cuda.synchronize()
    r_w, r_x, _, r_gyu = oracle.gf_backward(od, to64(x), to64(w), to64(gy))
    assert none is None and torch.equal(g_w, n_w) and torch.equal(g_x, n_x)
    assert rel_err(g_w, r_w) <= TOL[dtype] and rel_err(g_x, r_x) <= TOL[dtype] and rel_err(gy_u, r_gyu) <= TOL[dtype]
    assert np.array_equal(to64(g_x), to64(T.conv_bwd_input(d, gy_u, w.cuda())))   # the separate entry, bit for bit


def check_reduced(case, dtype):
    """A reduced input gradient is the full-resolution one, a value per patch, bit for bit."""
    N, Ci, Co, H, W, K, s, r = case
    d = mk(N, Ci, Co, H, W, K, s, K // 2, r=r, dtype=dtype)
    sh = T.shapes(d)
    w, gyu = randn(sh["w"], 2, dtype).cuda(), randn(sh["gy_u"], 3, dtype).cuda()
    g_x, g_xu = T.conv_bwd_input(d, gyu, w), T.conv_bwd_input(d, gyu, w, reduced_out=True)
    assert torch.equal(g_x[:, :, ::r * s, ::r * s], g_xu)


# N, C_in, C_out, H, W, K, stride, r: ragged or unaligned maps with more than 64 patches or planes over 16 KB
BAND_CASES = [
    (2, 24, 40, 65, 65, 1, 1, 4),      # one image in several bands, ragged last patch row and column
    (1, 8, 8, 33, 129, 3, 1, 2),       # 65 patch columns: the 128-column tile
    (1, 40, 16, 6, 255, 1, 1, 2),      # 128 patch columns, the widest tile; two row tiles of c_i
    (1, 72, 9, 3, 300, 3, 1, 2),       # 150 patch columns: over the widest tile
    (3, 20, 13, 31, 37, 3, 1, 3),      # odd patch size, channels that are no vector multiple
    (1, 5, 3, 67, 61, 3, 1, 2),
    (2, 16, 24, 66, 70, 3, 2, 3),      # strided, r_x = 6
    (1, 8, 16, 130, 120, 1, 1, 16),    # few, large patches: a band's pixels limit its rows
    (1, 12, 20, 300, 17, 1, 1, 16),
    (70, 16, 16, 35, 35, 1, 1, 4),     # many images: bands of several patch rows
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", BAND_CASES)
def test_input_gradient_bands(oracle, case, dtype):
    check_filtered(oracle, case, dtype)


# N, C_in, C_out, H, W, K, stride, r: edges of the two-product launch on small and large maps
GEMM_CASES = [
    (1, 3, 5, 7, 7, 1, 1, 2),          # a tensor of a few vectors: every load is at the end of its tensor
    (1, 8, 8, 2, 2, 1, 1, 2),          # one patch per plane
    (3, 65, 67, 7, 7, 3, 1, 2),        # one row and a few past the 64-row tiles, odd channels
    (5, 72, 72, 14, 14, 1, 1, 2),      # 49 patches: the last vector of a plane is partial
    (33, 64, 128, 7, 7, 1, 1, 4),      # 4 patches: several images per column tile, a last tile that is not full
    (200, 24, 40, 28, 28, 1, 1, 2),    # long K, one tile: slabs summed in two levels
    (64, 512, 256, 8, 8, 1, 1, 2),     # K slabs on both products
    (2, 40, 136, 12, 12, 3, 1, 3),     # 16 patches of 9 pixels; K tail of the input gradient
    (1, 8, 16, 64, 64, 1, 1, 8),       # whole images of 4096 pixels per tile
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", GEMM_CASES)
def test_dense_products(oracle, case, dtype):
    check_filtered(oracle, case, dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_dense_slab_sums_repeat(oracle, dtype):
    """The block that adds a tile's slabs sees every slab complete: ten runs on the same inputs, with the launches of
    another layer in between, agree bit for bit (256 -> 512 channels, stride 2: slabs of the weight gradient finish
    within a microsecond of each other)."""
    d = mk(64, 256, 512, 14, 14, 3, 2, 1, r=2, dtype=dtype)
    o = mk(16, 320, 640, 7, 7, r=2, dtype=dtype)
    args = []
    for e, seed in ((d, 5), (o, 6)):
        sh = T.shapes(e)
        args.append((e, randn(sh["g_y"], seed, dtype).cuda(), randn(sh["x_u"], seed + 10, dtype).cuda(), randn(sh["w"], seed + 20, dtype).cuda()))
    first = T.conv_bwd_filtered(*args[0])
    for _ in range(10):
        T.conv_bwd_filtered(*args[1])
        again = T.conv_bwd_filtered(*args[0])
        assert all(torch.equal(a, b) for a, b in zip(first, again))


# N, C_in, C_out, H, W, K, stride, padding, dilation: edges of the vanilla launch (tile sizes, K slabs, phases, routes)
EXACT_CASES = [
    (1, 65, 65, 6, 6, 3, 1, 1, 1),      # one row past 64 on both sides: 128 x 64 tiles, almost empty
    (40, 129, 130, 14, 14, 3, 1, 1, 1),  # 128 x 128 tiles with a remainder of one, odd channels
    (64, 128, 192, 7, 7, 3, 2, 1, 1),   # 128 x 128 tiles on phase planes of 4 x 4
    (1, 512, 192, 4, 4, 3, 1, 1, 1),    # K slabs of the input gradient, summed inside the launch
    (2, 320, 96, 5, 5, 3, 2, 1, 1),     # K slabs over phases with different numbers of taps
    (1, 9, 7, 24, 24, 13, 1, 6, 1),     # 169 taps
    (2, 24, 40, 13, 13, 1, 2, 0, 1),    # strided pointwise: three of four phases that no tap reaches
    (3, 17, 33, 21, 19, 1, 1, 0, 1),    # pointwise: the two-product launch on the maps themselves, odd planes
    (2, 12, 20, 40, 130, 3, 4, 1, 1),   # stride 4, wide phase planes
    (300, 8, 16, 6, 6, 3, 1, 1, 1),     # many images, small maps: many slabs of one weight tile
    (2, 24, 40, 112, 112, 3, 2, 1, 1),  # strided on planes that no block can stage: gathered from the phase planes
    (1, 9, 7, 131, 77, 3, 2, 1, 1),     # ... of odd extents, pixels that are no whole vectors
    (1, 8, 16, 200, 198, 5, 4, 2, 1),   # ... 16 phases
    (3, 16, 24, 57, 57, 1, 2, 0, 1),    # ... pointwise
    (2, 3, 32, 40, 38, 3, 2, 1, 1),     # few input channels, a small map
    (1, 3, 8, 512, 560, 3, 1, 1, 1),    # ... a large one: weights over the column tensor
    (9, 7, 4, 150, 149, 5, 1, 2, 1),    # ... 175 columns
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", EXACT_CASES)
def test_vanilla_products(oracle, case, dtype):
    N, Ci, Co, H, W, K, s, p, dl = case
    d = mk(N, Ci, Co, H, W, K, s, p, dl, r=2, dtype=dtype)
    sh = T.shapes(d)
    x, w, gy = (randn(sh[k], i, dtype) for i, k in enumerate(("x", "w", "g_y"), 1))
    g_w, g_x = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda())
    o_w, _ = T.conv_bwd_exact(d, x.cuda(), None, gy.cuda(), want_gx=False)
    _, o_x = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda(), want_gw=False)
    r_w, r_x = oracle.bwd_exact(odesc(oracle, d), to64(x), to64(w), to64(gy))
    for a, b, r in ((g_w, o_w, r_w), (g_x, o_x, r_x)):
        assert rel_err(a, r) <= TOL[dtype] and torch.equal(a, b)


# N, C_in, C_out, H, W: fp32 pointwise layers of few channels on one side, one pass over the maps -- every tile, rows and runs
# that are not full, planes at any alignment, the last vectors of a tensor -- and the edges of the rule
PIXEL_CASES = [
    (12, 24, 144, 64, 64),     # 1536 runs of 32 pixels: the fewest
    (12, 24, 144, 64, 63),     # one run fewer per image: two products
    (3, 32, 33, 128, 160),     # one channel more than a tile
    (24, 3, 97, 47, 61),       # odd planes
    (6, 31, 192, 104, 80),     # the most channels
    (6, 31, 193, 104, 80),     # one more: two products
    (2, 34, 32, 200, 130),     # and the other way round
    (700, 128, 5, 9, 11),      # less than a vector in the last run of every image
    (1, 160, 9, 223, 331),     # one image
    (5, 161, 17, 100, 100),    # a run of 16 pixels at the end of an image
    (1, 192, 1, 250, 200),     # one output channel
]


# ... of many input channels: every tile, half lines at the ends of rows, a last run of 16 pixels, and the edges of the rule
PIXEL_CASES += [
    (24, 33, 32, 64, 64), (24, 64, 1, 60, 60), (128, 65, 31, 28, 28), (25, 128, 8, 44, 44), (7, 129, 24, 100, 84), (12, 160, 32, 64, 64),
    (24, 161, 16, 52, 52), (12, 192, 3, 64, 64), (24, 161, 17, 52, 52), (12, 64, 24, 64, 64), (25, 96, 24, 42, 46),
]


@pytest.mark.parametrize("case", PIXEL_CASES)
def test_vanilla_pointwise_one_pass(oracle, case):
    N, Ci, Co, H, W = case
    test_vanilla_products(oracle, (N, Ci, Co, H, W, 1, 1, 0, 1), "f32")


@pytest.mark.parametrize("kind", ["tiny", "large", "infinite"])
@pytest.mark.parametrize("case", [(12, 24, 144, 64, 64), (24, 65, 31, 47, 61)])
def test_vanilla_pointwise_of_extreme_values(oracle, case, kind):
    N, Ci, Co, H, W = case
    test_fp32_products_of_extreme_values(oracle, (N, Ci, Co, H, W, 1, 1, 0), kind)


# N, C_in, C_out, H, W: every tile of the pass, for what three bf16 terms do not hold
@pytest.mark.parametrize("kind", ["tiny", "large", "infinite", "x", "w"])
@pytest.mark.parametrize("case", [(24, 9, 40, 47, 61), (24, 3, 97, 47, 61), (12, 24, 130, 64, 64), (24, 31, 192, 47, 61),
                                  (24, 40, 20, 64, 64), (12, 100, 31, 64, 64), (12, 160, 17, 64, 64), (12, 192, 9, 64, 64)])
def test_vanilla_pointwise_second_pass(oracle, case, kind):
    N, Ci, Co, H, W = case
    if kind in ("tiny", "large", "infinite"):
        return test_fp32_products_of_extreme_values(oracle, (N, Ci, Co, H, W, 1, 1, 0), kind)
    d = mk(N, Ci, Co, H, W, 1, 1, 0)   # one operand alone: one gradient is formed again, the other stays
    sh = T.shapes(d)
    x, w, gy = randn(sh["x"], 1, "f32"), randn(sh["w"], 2, "f32"), randn(sh["g_y"], 3, "f32")
    first = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda())
    {"x": x, "w": w}[kind].mul_(2.0 ** -121)
    g_w, g_x = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda())
    r_w, r_x = oracle.bwd_exact(odesc(oracle, d), to64(x), to64(w), to64(gy))
    same_values(g_w, r_w, 1e-5), same_values(g_x, r_x, 1e-5)
    assert torch.equal(*((g_x, first[1]) if kind == "x" else (g_w, first[0])))


@pytest.mark.parametrize("Ci,Co", [(24, 144), (144, 24)])
def test_vanilla_pointwise_second_pass_time(Ci, Co):
    """Gradients that underflow are ordinary data: the second pass of every block costs a few passes, not dozens (with a
    product per lane and step instead of matrix instructions: 25 - 35)."""
    d = mk(32, Ci, Co, 56, 56, 1, 1, 0)
    sh = T.shapes(d)
    x, w, gy = (randn(sh[k], i, "f32").cuda() for i, k in enumerate(("x", "w", "g_y")))
    tiny = gy.clone()
    tiny.view(-1)[::997] = 1e-36
    e = [torch.cuda.Event(enable_timing=True) for _ in range(2)]

    def least(g):
        out = []
        for _ in range(8):
            e[0].record()
            for _ in range(8):
                T.conv_bwd_exact(d, x, w, g)
            e[1].record()
            torch.cuda.synchronize()
            out.append(e[0].elapsed_time(e[1]))
        return min(out)

    assert least(tiny) <= 8 * least(gy)


# N, C_in, C_out, H, W, K, stride, padding, dilation: bf16 layers whose operands are staged -- tiles and chunks of 64 channels
# and pixels that are not full, phases, slabs of either product -- and the edges of the rule
STAGED_CASES = [
    (1, 64, 64, 1, 1, 3, 1, 1, 1),       # one pixel
    (1, 48, 64, 5, 7, 3, 1, 1, 1),       # fewest channels on one side, less than a chunk of pixels
    (3, 47, 64, 8, 8, 3, 1, 1, 1),       # one channel fewer: not staged
    (3, 64, 96, 9, 9, 5, 1, 2, 1),       # 128 x 64 tiles that are not full on either side
    (2, 97, 127, 13, 11, 3, 2, 1, 1),    # odd channels, phase planes of odd extents
    (2, 50, 61, 16, 20, 3, 3, 1, 1),     # stride 3
    (2, 64, 64, 14, 14, 4, 2, 1, 1),     # even kernel, stride 2
    (2, 144, 192, 12, 10, 3, 1, 2, 2),   # dilation
    (4, 64, 64, 10, 12, 11, 1, 5, 1),    # 121 taps
    (1, 512, 256, 4, 4, 3, 1, 1, 1),     # K slabs of the input gradient, summed inside the launch
    (2, 320, 128, 5, 5, 3, 2, 1, 1),     # ... over phases with different numbers of taps
    (16, 192, 255, 28, 28, 3, 1, 1, 1),  # 128 x 128 tiles, a last one of 127 rows
    (33, 64, 64, 30, 30, 3, 1, 1, 1),    # many slabs, no multiple of eight
]


@pytest.mark.parametrize("case", STAGED_CASES)
def test_vanilla_staged_operands(oracle, case):
    test_vanilla_products(oracle, case, "bf16")
    N, Ci, Co, H, W, K, s, p, dl = case
    d = mk(N, Ci, Co, H, W, K, s, p, dl, r=1, dtype="bf16")
    sh = T.shapes(d)
    x, w, gy = (randn(sh[k], i, "bf16") for i, k in enumerate(("x", "w", "g_y"), 1))
    e_w, e_x = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda())
    f_w, f_x, _ = T.conv_bwd_filtered(d, gy.cuda(), x.cuda(), w.cuda())   # patches of one pixel: the same products
    assert torch.equal(e_w, f_w) and torch.equal(e_x, f_x)
    if H * W == 1:
        return   # (no finite value would be left)
    gy[0, Co - 1, 0, 0], x[N - 1, 0, H - 1, W - 1] = float("inf"), float("-inf")
    g_w, g_x = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda())
    with np.errstate(invalid="ignore", over="ignore"):
        r_w, r_x = oracle.bwd_exact(odesc(oracle, d), to64(x), to64(w), to64(gy))
    same_values(g_w, r_w, TOL["bf16"]), same_values(g_x, r_x, TOL["bf16"])


@pytest.mark.parametrize("H", [57, 56])
def test_vanilla_one_call_entry_within_the_static_scratch(H):
    """Layers whose staged operands do not fit the library's scratch: the one-call entry keeps the form that does, on its
    own scratch and on a workspace.  g_x is gf_conv_bwd_exact's bit for bit; so is g_w on planes of whole vectors, on
    others up to the order of the fp32 sums."""
    d = mk(40, 256, 256, H, H, 3, 1, 1, 1, r=1, dtype="bf16")
    assert B.gf_workspace_bytes(d, B.GF_OP_BWD_FILTERED) <= B.GF_STATIC_SCRATCH_BYTES < B.gf_workspace_bytes(d, B.GF_OP_BWD_EXACT)
    sh = T.shapes(d)
    x, w, gy = (randn(sh[k], i, "bf16").cuda() for i, k in enumerate(("x", "w", "g_y"), 1))
    e_w, e_x = T.conv_bwd_exact(d, x, w, gy)
    f_w, f_x, _ = T.conv_bwd_filtered(d, gy, x, w)
    s_w, s_x = torch.empty_like(f_w), torch.empty_like(f_x)
    B.gf_conv_bwd_filtered_static(d, B.ptr(gy), B.ptr(x), B.ptr(w), 0, B.ptr(s_w), B.ptr(s_x), torch.cuda.current_stream().cuda_stream)
    torch.cuda.synchronize()
    assert torch.equal(s_w, f_w) and torch.equal(s_x, f_x) and torch.equal(e_x, f_x)
    assert torch.equal(e_w, f_w) if H * H % 8 == 0 else rel_err(e_w, to64(f_w)) <= 1e-5


@pytest.mark.parametrize("case", [(38, 96, 128, 64, 64, 3, 1, 1, 1), (40, 128, 96, 63, 61, 3, 1, 1, 1)])
def test_vanilla_weight_gradient_alone_on_a_large_map(oracle, case):
    """Past 64 MiB the weight gradient alone of such a layer reads the maps themselves: the bits of the call for both."""
    N, Ci, Co, H, W, K, s, p, dl = case
    d = mk(*case, r=2, dtype="bf16")
    sh = T.shapes(d)
    x, w, gy = (randn(sh[k], i, "bf16") for i, k in enumerate(("x", "w", "g_y"), 1))
    g_w, g_x = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda())
    o_w, _ = T.conv_bwd_exact(d, x.cuda(), None, gy.cuda(), want_gx=False)
    _, o_x = T.conv_bwd_exact(d, None, w.cuda(), gy.cuda(), want_gw=False)
    assert torch.equal(g_w, o_w) and torch.equal(g_x, o_x)
    od = odesc(oracle, mk(N, 2, 1, H, W, K, s, p, dl, r=2, dtype="bf16"))
    r_w, _ = oracle.bwd_exact(od, to64(x[:, 31:33]), None, to64(gy[:, Co - 1:]), want_gx=False)
    assert rel_err(g_w[Co - 1:, 31:33], r_w) <= TOL["bf16"]
    od = odesc(oracle, mk(1, Ci, Co, H, W, K, s, p, dl, r=2, dtype="bf16"))
    _, r_x = oracle.bwd_exact(od, None, to64(w), to64(gy[N - 1:]), want_gw=False)
    assert rel_err(g_x[N - 1:], r_x) <= TOL["bf16"]


# N, C_in, C_out, H, W, K, stride, padding, dilation: input gradients of vanilla layers with few tiles -- slabs of sixteen steps, eight and
# four, phases with more taps than others, all taps in one phase
VANILLA_FEW_CASES = [
    (1, 64, 64, 9, 9, 3, 1, 1, 1),
    (2, 96, 40, 6, 6, 3, 1, 1, 1),
    (2, 40, 150, 7, 5, 5, 1, 2, 1),
    (3, 33, 70, 21, 18, 5, 2, 2, 1),
    (2, 24, 96, 15, 16, 3, 2, 1, 1),
    (2, 48, 72, 17, 19, 3, 2, 2, 2),
    (2, 20, 64, 22, 20, 5, 3, 2, 1),
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", VANILLA_FEW_CASES)
def test_vanilla_input_gradient_of_few_tiles(oracle, case, dtype):
    N, Ci, Co, H, W, K, s, p, dl = case
    d = mk(N, Ci, Co, H, W, K, s, p, dl, r=1, dtype=dtype)
    sh = T.shapes(d)
    x, w, gy = (randn(sh[k], i, dtype) for i, k in enumerate(("x", "w", "g_y"), 1))
    g_w, g_x = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda())
    r_w, r_x = oracle.bwd_exact(odesc(oracle, d), to64(x), to64(w), to64(gy))
    assert rel_err(g_w, r_w) <= TOL[dtype] and rel_err(g_x, r_x) <= TOL[dtype]


# N, C_in, C_out, H, W, K, stride, padding, dtype; bytes for both gradients, g_w, g_x without the forms that need more
@pytest.mark.parametrize("case,least", [
    ((16, 192, 255, 28, 28, 3, 1, 1, "bf16"), (14984192, 14102784, 883712)),
    ((2, 97, 127, 13, 11, 3, 2, 1, "bf16"), (813056, 509952, 304128)),
    ((12, 24, 144, 64, 64, 1, 1, 0, "f32"), (1769472, 1769472, 256)),
    ((2, 256, 88, 6, 6, 3, 1, 1, "f32"), (2016256, 812032, 1205248)),     # fewer slabs of few tiles
    ((10, 52, 26, 20, 20, 5, 2, 2, "f32"), (2748928, 1781504, 970496)),
    ((18, 445, 179, 5, 20, 5, 2, 2, "bf16"), (53734144, 9790464, 44154624)),
    ((10, 59, 967, 14, 28, 3, 2, 1, "bf16"), (13948160, 4572672, 9377536)),   # neither staged nor fewer slabs
])
def test_vanilla_layers_with_less_workspace(oracle, case, least):
    """Staged operands and the one pass over the maps: a call whose workspace holds what the unstaged form or the two products need,
    but not the copies and slabs, is taken; one byte less than the smallest is not."""
    N, Ci, Co, H, W, K, s, p, dtype = case
    d = mk(N, Ci, Co, H, W, K, s, p, r=1, dtype=dtype)
    sh = T.shapes(d)
    x, w, gy = (randn(sh[k], i, dtype) for i, k in enumerate(("x", "w", "g_y"), 1))
    r_w, r_x = oracle.bwd_exact(odesc(oracle, d), to64(x), to64(w), to64(gy))
    x, w, gy = x.cuda(), w.cuda(), gy.cuda()
    ws = torch.empty(B.gf_workspace_bytes(d, B.GF_OP_BWD_EXACT) + 4096, dtype=torch.uint8, device="cuda")
    st = torch.cuda.current_stream().cuda_stream

    def call(n, a, b):   # the outputs, or None: refused
        g_w, g_x = torch.zeros(sh["w"], device="cuda"), torch.zeros_like(x)
        ws[n:].fill_(77)
        try:
            B.gf_conv_bwd_exact(d, B.ptr(x), B.ptr(w), B.ptr(gy), B.ptr(g_w) if a else 0, B.ptr(g_x) if b else 0, B.ptr(ws), n, st)
        except B.GfError as e:
            assert e.status == B.GF_ERR_WORKSPACE
            return None
        assert (ws[n:] == 77).all()
        return g_w, g_x

    for (a, b), most in zip(((1, 1), (1, 0), (0, 1)), least):
        lo, hi = 0, most   # refused without one (g_x of pointwise layers is not), taken with what these calls always needed
        assert call(hi, a, b) is not None
        while hi - lo > 1:
            mid = (lo + hi) // 2
            lo, hi = (lo, mid) if call(mid, a, b) is not None else (mid, hi)
        full = call(ws.numel() - 4096, a, b)
        for n in (hi, most):
            g_w, g_x = call(n, a, b)
            assert not a or rel_err(g_w, r_w) <= TOL[dtype]
            assert not b or rel_err(g_x, r_x) <= TOL[dtype]
            assert not b or dtype == "f32" or torch.equal(g_x, full[1])   # (fp32: fewer slabs, or the products instead of the one pass)


# N, C, H, W, K, padding: both gradients of a depthwise layer in one pass (ragged groups of pixels, frames, image runs)
DW_EXACT_CASES = [
    (3, 5, 20, 20, 3, 1),
    (2, 3, 21, 23, 5, 2),       # odd rows: the last group of a row holds three pixels
    (9, 2, 23, 19, 3, 0),       # unpadded: smaller output map
    (1, 4, 57, 31, 3, 2),       # larger output map
    (2, 3, 20, 20, 5, 4),
    (2, 2, 112, 112, 3, 1),     # frame of 52 KB
    (40, 160, 20, 21, 3, 1),    # several images per block, a remainder of images in the last one
    (37, 130, 14, 14, 3, 1),    # ... and several planes at a time
    (5, 6, 7, 7, 3, 1),
    (3, 5, 1, 3, 3, 1),         # planes of fewer elements than a vector
    (2, 2, 2, 1, 5, 2),
    (2, 2, 130, 130, 3, 1),     # a frame past the LDS budget: the separate launches
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", DW_EXACT_CASES)
def test_vanilla_depthwise_one_pass(oracle, case, dtype):
    N, C, H, W, K, p = case
    d = mk(N, C, C, H, W, K, 1, p, g=C, r=1, dtype=dtype)
    sh = T.shapes(d)
    x, w, gy = (randn(sh[k], i, dtype) for i, k in enumerate(("x", "w", "g_y"), 1))
    g_w, g_x = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda())
    o_w, _ = T.conv_bwd_exact(d, x.cuda(), None, gy.cuda(), want_gx=False)
    _, o_x = T.conv_bwd_exact(d, None, w.cuda(), gy.cuda(), want_gw=False)
    r_w, r_x = oracle.bwd_exact(odesc(oracle, d), to64(x), to64(w), to64(gy))
    assert rel_err(g_w, r_w) <= TOL[dtype] and rel_err(g_x, r_x) <= TOL[dtype]
    assert torch.equal(o_w, g_w) and torch.equal(o_x, g_x)
    # an infinite activation in a corner reaches the taps that read it and no others
    x[0, 0, 0, 0] = float("inf")
    g_w, _ = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda())
    r_w, _ = oracle.bwd_exact(odesc(oracle, d), to64(x), to64(w), to64(gy))
    assert torch.equal(torch.isfinite(g_w.cpu()), torch.isfinite(torch.from_numpy(r_w)))
    # ... and an infinite gradient at the end of a row the pixels and taps that read it
    if H * W > 14000:   # (planes past the LDS budget: kernels that multiply the zeros around the map)
        return
    x[0, 0, 0, 0] = 1.0
    Hy, Wy = sh["g_y"][2:]
    for i, j in ((0, Wy - 1), (Hy // 2, Wy - 1), (Hy - 1, 0)):
        gi = gy.clone()
        gi[0, 0, i, j] = float("inf")
        g_w, g_x = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gi.cuda())
        r_w, r_x = oracle.bwd_exact(odesc(oracle, d), to64(x), to64(w), to64(gi))
        for got, ref in ((g_w, r_w), (g_x, r_x)):
            assert torch.equal(torch.isfinite(got.cpu()), torch.isfinite(torch.from_numpy(ref)))


# N, C, H, W, K, padding: the same with stride 2 -- maps of either parity, first rows and columns before the map, last ones
# past it, every padding, several images per block and planes at a time
DW_STRIDE2_CASES = [
    (3, 5, 20, 20, 3, 1),
    (2, 3, 21, 23, 5, 2),
    (3, 2, 14, 15, 3, 0),
    (2, 4, 15, 18, 3, 2),
    (2, 3, 17, 16, 5, 4),
    (2, 3, 16, 19, 5, 3),
    (2, 3, 12, 13, 5, 1),
    (2, 3, 9, 10, 5, 0),
    (3, 5, 1, 3, 3, 1),
    (2, 2, 2, 1, 5, 2),
    (37, 130, 14, 14, 3, 1),
    (40, 160, 21, 20, 5, 2),
    (2, 2, 200, 201, 3, 1),     # frame of 41 KB
    (2, 2, 260, 260, 3, 1),     # a frame past the LDS budget: other kernels
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", DW_STRIDE2_CASES)
def test_vanilla_depthwise_stride_2(oracle, case, dtype):
    N, C, H, W, K, p = case
    d = mk(N, C, C, H, W, K, 2, p, g=C, r=1, dtype=dtype)
    sh = T.shapes(d)
    x, w, gy = (randn(sh[k], i, dtype) for i, k in enumerate(("x", "w", "g_y"), 1))
    g_w, g_x = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda())
    o_w, _ = T.conv_bwd_exact(d, x.cuda(), None, gy.cuda(), want_gx=False)
    _, o_x = T.conv_bwd_exact(d, None, w.cuda(), gy.cuda(), want_gw=False)
    r_w, r_x = oracle.bwd_exact(odesc(oracle, d), to64(x), to64(w), to64(gy))
    assert rel_err(g_w, r_w) <= TOL[dtype] and rel_err(g_x, r_x) <= TOL[dtype]
    assert torch.equal(o_w, g_w) and torch.equal(o_x, g_x)
    # an infinite activation, gradient or kernel value reaches what reads it and nothing else
    Hy, Wy = sh["g_y"][2:]
    for t, at in ((x, (0, 0, 0, 0)), (x, (N - 1, C - 1, H - 1, W - 1)), (gy, (0, 0, 0, Wy - 1)), (gy, (0, 0, Hy - 1, 0)),
                  (w, (0, 0, 0, 0)), (w, (0, 0, K - 1, K - 1))):
        kept = t[at].clone()
        t[at] = float("inf")
        g_w, g_x = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda())
        r_w, r_x = oracle.bwd_exact(odesc(oracle, d), to64(x), to64(w), to64(gy))
        for got, ref in ((g_w, r_w), (g_x, r_x)):
            assert torch.equal(torch.isfinite(got.cpu()), torch.isfinite(torch.from_numpy(ref)))
        t[at] = kept


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(3, 2, 200, 203, 3, 1), (2, 2, 190, 185, 5, 0)])
def test_vanilla_depthwise_stride_2_without_a_workspace(oracle, case, dtype):
    """Planes too large for the kernels that stage x: every entry takes the call without a workspace as well."""
    N, C, H, W, K, p = case
    d = mk(N, C, C, H, W, K, 2, p, g=C, r=1, dtype=dtype)
    sh = T.shapes(d)
    x, w, gy = (randn(sh[k], i, dtype).cuda() for i, k in enumerate(("x", "w", "g_y"), 1))
    r_w, r_x = oracle.bwd_exact(odesc(oracle, d), to64(x), to64(w), to64(gy))
    st = torch.cuda.current_stream().cuda_stream
    px, pw, pg = (B.ptr(t) for t in (x, w, gy))
    for call in (lambda a, b: B.gf_conv_bwd_exact(d, px, pw, pg, a, b, 0, 0, st), lambda a, b: B.gf_conv_bwd_exact(d, px, pw, pg, a, 0, 0, 0, st),
                 lambda a, b: B.gf_conv_bwd_weight(d, px, pg, a, 0, 0, st), lambda a, b: B.gf_conv_bwd_filtered(d, pg, px, pw, 0, a, b, 0, 0, st),
                 lambda a, b: B.gf_conv_bwd_chained(d, pg, px, pw, a, b, False, 0, 0, 0, st)):
        g_w, g_x = torch.zeros(sh["w"], device="cuda"), torch.zeros_like(x)
        call(B.ptr(g_w), B.ptr(g_x))
        torch.cuda.synchronize()
        assert rel_err(g_w, r_w) <= TOL[dtype]
        assert not g_x.any() or rel_err(g_x, r_x) <= TOL[dtype]


def check_codes(oracle, case, dtype, groups=1):
    """The one-call backward on codes against the oracle's integer contractions of the same codes, bit for bit."""
    N, Ci, Co, H, W, K, s, r = case
    d = mk(N, Ci, Co, H, W, K, s, K // 2, g=groups, r=r, dtype=dtype)
    sh = T.shapes(d)
    x, w, gy = (randn(sh[k], i, dtype) for i, k in enumerate(("x", "w", "g_y"), 1))
    inv_x, inv_g, inv_w, sw, sx = 8.0, 60.0, 12.0, 2.5e-4, 3.5e-4
    x_q = T.pool_activation_q8(d, x.cuda(), inv_x)
    g_w, g_x, gy_q = T.conv_bwd_filtered_q8(d, gy.cuda(), inv_g, x_q, w.cuda(), inv_w, sw, sx, want_gyq=True)
    n_w, n_x = T.conv_bwd_filtered_q8(d, gy.cuda(), inv_g, x_q, w.cuda(), inv_w, sw, sx)
    w_q = T.kernel_sum_q8(d, w.cuda(), inv_w)
    assert torch.equal(gy_q, T.filter_grad_q8(d, gy.cuda(), inv_g))
    assert torch.equal(g_w, n_w) and torch.equal(g_x, n_x)
    od, nq = odesc(oracle, d), lambda t: t.cpu().numpy()
    assert torch.equal(g_w.cpu(), torch.from_numpy(oracle.bwd_weight_q8(od, nq(x_q), nq(gy_q), sw)))
    r_x = oracle.bwd_input_q8(od, nq(gy_q), nq(w_q), sx)
    assert torch.equal(g_x.cpu(), torch.from_numpy(r_x).to(g_x.dtype))
    assert torch.equal(T.conv_bwd_weight_q8(d, x_q, gy_q, sw), g_w) and torch.equal(T.conv_bwd_input_q8(d, gy_q, w_q, sx), g_x)


# N, C_in, C_out, H, W, K, stride, r: edges of the two-product launch on codes
CODE_CASES = [
    (2, 16, 16, 4, 4, 1, 1, 2),        # the fewest channels; planes of four codes
    (1, 15, 16, 8, 8, 3, 1, 2),        # one channel too few: the per-pair and per-patch kernels
    (3, 65, 67, 14, 14, 3, 1, 2),      # planes of 49 codes, tensors that end inside a vector, odd channels
    (5, 48, 136, 7, 7, 1, 1, 2),       # 16 codes per plane: several images per column tile
    (200, 24, 40, 28, 28, 1, 1, 2),    # long K, one tile: slabs summed in two levels
    (24, 16, 16, 160, 152, 1, 1, 2),   # more products per output than an int32 holds: slabs added in 64 bits
    (1, 24, 20, 6, 300, 3, 1, 2),      # 150 patch columns: reduced map and expansion
    (2, 200, 300, 33, 29, 3, 2, 4),    # strided, ragged patches
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CODE_CASES)
def test_dense_products_on_codes(oracle, case, dtype):
    check_codes(oracle, case, dtype)


@pytest.mark.parametrize("case", [
    (36, 1280, 1217, 63, 63, 1),   # 400 tiles: one slab each, were it not for what an int32 sum holds
    (60, 64, 64, 50, 50, 3),       # one 64 x 64 tile of many slabs, added in 64 bits
])
def test_code_sums_past_int32(case):
    """Codes that are constant over a plane: every sum is N P times a product of two codes, past 2^31 for most pairs."""
    N, Ci, Co, Hp, Wp, K = case
    d = mk(N, Ci, Co, 2 * Hp, 2 * Wp, K, 1, K // 2, r=2)
    g = torch.Generator().manual_seed(N)
    a, b = (torch.randint(120, 128, (c,), generator=g) * (2 * torch.randint(0, 2, (c,), generator=g) - 1) for c in (Ci, Co))
    x_q, gy_q = (v.to(torch.int8).cuda().view(1, -1, 1, 1).expand(N, -1, Hp, Wp).contiguous() for v in (a, b))
    want = (N * Hp * Wp * torch.outer(b, a)).to(torch.float32) * np.float32(2.5e-4)
    g_w = T.conv_bwd_weight_q8(d, x_q, gy_q, 2.5e-4).cpu()
    assert torch.equal(g_w, want.view(Co, Ci, 1, 1).expand(-1, -1, K, K))


# N, C_in, C_out, H, W, K, stride, r: weight gradients on 32 x 32 tiles -- their edges, chunks for one wave, for all four and
# for a second round, slabs -- and the 64 x 64 tiles from the same rule's other side on
SHORT_K_CASES = [
    (1, 32, 32, 8, 8, 1, 1, 2),        # one tile, less than a chunk
    (1, 33, 31, 8, 8, 3, 1, 2),        # a row and a column past the tile
    (3, 17, 97, 6, 6, 1, 1, 2),        # nine patches: every vector ends inside its plane
    (5, 65, 96, 7, 7, 3, 1, 4),        # four patches: planes shorter than a vector of 16-bit values or codes
    (17, 48, 40, 8, 8, 1, 1, 2),       # chunks for more than four waves, a last one that is not full
    (64, 64, 61, 12, 12, 1, 1, 2),     # slabs
    (30, 16, 48, 17, 16, 5, 1, 2),     # 25 taps
    (90, 20, 24, 14, 14, 3, 2, 3),     # slabs of ragged planes, stride 2
    (24, 512, 512, 16, 16, 1, 1, 2),   # 64 x 64 tiles, slabs of both products
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", SHORT_K_CASES)
def test_short_k_weight_gradient(oracle, case, dtype):
    check_filtered(oracle, case, dtype)
    check_codes(oracle, case, dtype)


# N, C_in, C_out, H, W, K, stride, r: input gradients on 32 x 32 tiles -- their edges, K of one round of the four waves and of several,
# a last chunk that is not full, slabs; whole images, bands of patch rows, planes of less than a vector
FEW_TILE_CASES = [
    (1, 32, 64, 8, 8, 1, 1, 2),        # one tile, two chunks of 32-bit values
    (1, 33, 129, 7, 7, 3, 1, 2),       # a row past the tile, a row of k past the chunk
    (2, 40, 257, 6, 6, 1, 1, 2),       # nine patches: every vector ends inside its plane
    (3, 70, 800, 9, 7, 1, 1, 2),       # slabs, fp32
    (2, 64, 1090, 14, 14, 3, 1, 2),    # bands of four and of three patch rows
    (1, 31, 2100, 10, 62, 1, 1, 2),    # a patch row per band, slabs
    (4, 36, 130, 5, 5, 3, 2, 2),       # strided
    (1, 24, 300, 33, 30, 1, 1, 4),     # ragged patches
    (9, 20, 150, 6, 4, 5, 1, 7),       # one patch per plane
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", FEW_TILE_CASES)
def test_few_tile_input_gradient(oracle, case, dtype):
    check_filtered(oracle, case, dtype)
    check_reduced(case, dtype)
    check_codes(oracle, case, dtype)
    N, Ci, Co, H, W, K, s, r = case
    d = mk(N, Ci, Co, H, W, K, s, K // 2, r=r, dtype=dtype)
    sh = T.shapes(d)
    w, gyu = randn(sh["w"], 2, dtype), randn(sh["gy_u"], 3, dtype)
    g_xu = T.conv_bwd_input(d, gyu.cuda(), w.cuda(), reduced_out=True)
    assert rel_err(g_xu, oracle.bwd_input(odesc(oracle, d), to64(gyu), to64(w), reduced_out=True)) <= TOL[dtype]
    # an infinite gradient reaches the pixels of its patch and no others
    gyu[N - 1, Co - 1, -1, -1] = float("inf")
    g_x = T.conv_bwd_input(d, gyu.cuda(), w.cuda())
    assert torch.equal(torch.isfinite(g_x.cpu()), torch.isfinite(torch.from_numpy(oracle.bwd_input(odesc(oracle, d), to64(gyu), to64(w)))))


# N, C_in, C_out, H, W, K, stride, r: input gradients on bands of three, five and more patch rows in tiles of 128 columns, and just not
WIDE_BAND_CASES = [
    (4, 768, 24, 65, 65, 1, 1, 2),
    (4, 705, 17, 66, 83, 3, 1, 2),     # 42 patch columns: two left over; one row of c_i in the last tile
    (47, 64, 33, 70, 66, 1, 1, 2),     # a last band of two rows
    (26, 200, 40, 49, 50, 1, 1, 2),    # 25 patch columns
    (4, 700, 24, 65, 65, 1, 1, 2),     # a tile row less than fills the chip
    (4, 768, 24, 65, 85, 1, 1, 2),     # 43 patch columns: two rows
    (128, 200, 40, 18, 25, 3, 1, 2),   # nine rows of 13: one band, three of 64 columns
    (103, 270, 33, 13, 34, 1, 1, 2),   # seven of 17
    (15, 440, 64, 50, 46, 1, 1, 2),    # 25 of 23: five bands, thirteen
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", WIDE_BAND_CASES)
def test_input_gradient_wide_bands(oracle, case, dtype):
    check_filtered(oracle, case, dtype)
    check_reduced(case, dtype)
    check_codes(oracle, case, dtype)


# N, C_in, C_out, H, W, K, stride, r: runs of input-gradient pixels that are less than a vector, one, end vectors alone, one whole between
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(3, 5, 9, 1, 3, 1, 1, 2), (3, 6, 9, 1, 7, 1, 1, 2), (2, 7, 16, 3, 3, 1, 1, 2), (3, 65, 12, 2, 7, 3, 1, 2), (2, 9, 12, 1, 19, 1, 1, 4),
                                  (2, 33, 20, 5, 5, 3, 1, 2), (1, 31, 8, 2, 133, 1, 1, 2)])
def test_input_gradient_run_ends(oracle, case, dtype):
    check_filtered(oracle, case, dtype)


# N, C_in, C_out, H, W, K, stride, r: large bf16 products: both gradients in one launch or in kernels of their own
LARGE_CASES = [
    (128, 768, 768, 13, 13, 1, 1, 2),  # cut patches, 49 to a plane
    (25, 640, 256, 64, 48, 1, 1, 2),   # whole patches and vectors, under 8 GFLOP
    (12, 1024, 432, 64, 48, 1, 1, 2),  # ... past it, but 512 output channels on the larger tiles
    (12, 1024, 432, 63, 48, 1, 1, 2),  # ... a cut patch row
    (13, 1024, 432, 64, 44, 1, 1, 2),  # ... rows that end inside a vector
    (12, 2048, 224, 64, 48, 3, 1, 2),  # kernel sums
    (14, 1024, 512, 48, 48, 1, 1, 2),  # kernels of their own
    (14, 1000, 512, 48, 48, 3, 1, 2),
    (13, 1024, 512, 48, 48, 1, 1, 2),  # too few tiles for them
    (220, 1024, 728, 16, 16, 1, 1, 2), # more than 20 GFLOP: on small planes too
]


@pytest.mark.parametrize("case", LARGE_CASES)
def test_large_dense_products(oracle, case):
    check_filtered(oracle, case, "bf16")
    check_reduced(case, "bf16")


# ... on patch rows that need tiles of 128 columns; K of one chunk, of an odd number, with a part left
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(2, 40, 24, 9, 140, 1, 1, 2), (1, 72, 96, 5, 255, 3, 1, 2), (2, 65, 113, 7, 210, 1, 1, 3)])
def test_reduced_input_gradient_of_wide_rows(case, dtype):
    check_reduced(case, dtype)


# N, C_in, C_out, H, W: fp32, slabs of 32 x 32 tiles with one chunk for each wave, one more, two for each, one more, two in all
@pytest.mark.parametrize("case", [(76, 92, 10, 14, 14), (77, 92, 10, 14, 14), (64, 96, 160, 16, 16), (63, 70, 90, 12, 12), (1, 90, 70, 14, 14)])
def test_short_k_sums_do_not_lean(case):
    """The matrix instruction rounds its sums towards minus infinity; signs that change from wave to wave take that out: the mean
    error of n independent sums is within 5 / sqrt(n) of their deviation (without: 25, 15 and 12 / sqrt(n) for
    the first, the second and the last)."""
    N, Ci, Co, H, W = case
    d = mk(N, Ci, Co, H, W, 1, 1, 0, r=2)
    sh = T.shapes(d)
    x_u, gy, w = randn(sh["x_u"], 1, "f32").cuda(), randn(sh["g_y"], 2, "f32").cuda(), randn(sh["w"], 3, "f32").cuda()
    g_w, _, gy_u = T.conv_bwd_filtered(d, gy, x_u, w)
    err = g_w.view(Co, Ci).cpu().double() - torch.einsum("ncp,nkp->ck", gy_u.cpu().double().flatten(2), x_u.cpu().double().flatten(2))
    assert abs(err.mean()) <= 5 * err.std() / err.numel() ** 0.5


# N, C, H, W, stride, r: edges of the fused depthwise launches
DW_CASES = [
    (1, 1, 2, 2, 1, 2),                # runs shorter than a vector
    (2, 5, 5, 5, 2, 2), (3, 7, 15, 13, 2, 3),     # strided: odd runs, vectors shared by neighbouring blocks
    (40, 33, 7, 7, 1, 2),              # odd planes, several per block
    (3, 6, 15, 14, 1, 2), (3, 6, 10, 12, 1, 4),   # whole patch rows as words, a ragged last one
    (60, 50, 28, 28, 2, 2),            # strided, the filter adds columns first
    (300, 40, 9, 9, 4, 2),             # stride 4
    (1, 3, 101, 90, 1, 3), (1, 2, 144, 143, 1, 2),   # a plane per block, as large as it fits
    (2, 24, 16, 24, 1, 8), (1, 3, 64, 64, 1, 4),     # register rows
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", DW_CASES)
def test_depthwise_launches(oracle, case, dtype):
    N, c, H, W, s, r = case
    check_filtered(oracle, (N, c, c, H, W, 3, s, r), dtype, groups=c)
    check_codes(oracle, (N, c, c, H, W, 3, s, r), dtype, groups=c)


@pytest.mark.parametrize("C,H,W", [(1024, 7, 7), (520, 14, 14), (1100, 6, 5), (330, 15, 16), (3000, 2, 3)])
def test_reductions_of_long_runs_of_planes(C, H, W):
    """bf16 maps: blocks that hold many planes give a lane one patch position; the same planes image by image, in blocks
    of few planes, take the other loop.  Same values, bit for bit."""
    N = 48
    d, d1 = (mk(n, C, C, H, W, 1, 1, 0, r=2, dtype="bf16") for n in (N, 1))
    x = randn((N, C, H, W), 3, "bf16").cuda()
    many, batch, codes = T.filter_grad(d, x), T.pool_activation_batch([d], [x])[0], T.filter_grad_q8(d, x, 40.0)
    for n in (0, 1, N - 1):
        one = x[n:n + 1].contiguous()
        assert torch.equal(many[n:n + 1], T.filter_grad(d1, one))
        assert torch.equal(batch[n:n + 1], T.pool_activation(d1, one))
        assert torch.equal(codes[n:n + 1], T.filter_grad_q8(d1, one, 40.0))


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [
    (3, 72, 40, 61, 47, 3, 1, 8),      # few tiles of large planes: bands of one patch row, ragged in both directions
    (2, 16, 24, 64, 48, 1, 2, 8),      # strided
    (256, 8, 8, 40, 40, 1, 1, 8),      # more tiles, still bands
    (400, 8, 8, 40, 40, 1, 1, 8),      # enough of them: whole images
])
def test_large_patches_of_few_images(oracle, case, dtype):
    check_filtered(oracle, case, dtype)


@pytest.mark.parametrize("N,Ci,Co,H,W,dtype", [(1, 16, 8, 6000, 6000, "bf16"), (2, 9, 7, 5501, 8001, "bf16"), (1, 8, 8, 7001, 5003, "f32")])
def test_large_maps_of_few_channels(N, Ci, Co, H, W, dtype):
    """Pointwise vanilla BP on maps where a chunk of k has more rows than the layer has channels and the rows that do
    not exist would start past 2^31: sampled pixels of g_x and all of g_w against 64-bit sums."""
    d = mk(N, Ci, Co, H, W, 1, 1, 0, r=1, dtype=dtype)
    g = torch.Generator(device="cuda").manual_seed(3)
    td = torch.bfloat16 if dtype == "bf16" else torch.float32
    x, w, gy = (torch.randn(s, generator=g, device="cuda").to(td) for s in ((N, Ci, H, W), (Co, Ci, 1, 1), (N, Co, H, W)))
    g_w, g_x = T.conv_bwd_exact(d, x, w, gy)
    P = H * W
    pos = torch.cat([torch.arange(512), torch.randint(0, P, (4096,), generator=torch.Generator().manual_seed(1)), torch.arange(P - 512, P)]).cuda()
    r_w = torch.zeros(Co, Ci, dtype=torch.float64, device="cuda")
    for n in range(N):
        fx, fg = x[n].reshape(Ci, P), gy[n].reshape(Co, P)
        want = w.double().reshape(Co, Ci).t().contiguous() @ fg[:, pos].double()
        assert rel_err(g_x[n].reshape(Ci, P)[:, pos], want.cpu().numpy()) <= TOL[dtype]
        for p in range(0, P, 1 << 22):
            r_w += fg[:, p:p + (1 << 22)].double() @ fx[:, p:p + (1 << 22)].double().t().contiguous()
    assert rel_err(g_w.reshape(Co, Ci), r_w.cpu().numpy()) <= TOL[dtype]


def same_values(got, ref, tol):
    """Infinities and NaN where the reference has them, the rest within tol of the largest finite value."""
    got, fin = to64(got), np.isfinite(ref)
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    assert np.abs(got[fin] - ref[fin]).max() <= tol * np.abs(ref[fin]).max()


# N, C_in, C_out, H, W, K, stride, padding: a small and a large reduced map, ragged planes, every tile of the vanilla launch
FP32_CASES = [
    (4, 64, 72, 14, 14, 1, 1, 0), (8, 72, 64, 8, 8, 3, 1, 1), (2, 24, 40, 66, 62, 1, 1, 0), (1, 16, 16, 20, 260, 3, 1, 1),
    (3, 65, 65, 6, 6, 3, 1, 1), (40, 129, 130, 14, 14, 3, 1, 1), (2, 40, 24, 21, 19, 3, 1, 1), (2, 24, 40, 14, 14, 3, 2, 1),
]


@pytest.mark.parametrize("kind", ["tiny", "large", "infinite"])
@pytest.mark.parametrize("case", FP32_CASES)
def test_fp32_products_of_extreme_values(oracle, case, kind):
    """fp32 products outside the range that three bf16 terms cover: gradients around 2^-121, values past the largest
    bf16 and infinities come out as fp32 multiplication gives them, in both directions and on both paths."""
    N, Ci, Co, H, W, K, s, p = case
    d = mk(N, Ci, Co, H, W, K, s, p, r=2)
    od, sh = odesc(oracle, d), T.shapes(d)
    x, w, gy = randn(sh["x"], 1, "f32"), randn(sh["w"], 2, "f32", scale=0.1), randn(sh["g_y"], 3, "f32")
    if kind == "tiny":
        gy *= 2.0 ** -121
    elif kind == "large":
        x[0, 1, 1, 1], gy[0, 0, 2, 2], w[1, 2, 0, 0] = 3.4e38, 1e3, -3.395e38
        gy *= 1e-6
    else:
        x[0, 1, 1, 1], x[N - 1, 0, H - 1, W - 1], gy[0, 2, 0, 0] = float("inf"), float("-inf"), float("inf")
    with np.errstate(invalid="ignore", over="ignore"):
        r_w, r_x = oracle.bwd_exact(od, to64(x), to64(w), to64(gy))
        f_w, f_x, _, _ = oracle.gf_backward(od, to64(x), to64(w), to64(gy))
    g_w, g_x = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda())
    same_values(g_w, r_w, 1e-5), same_values(g_x, r_x, 1e-5)
    g_w, g_x, _ = T.conv_bwd_filtered(d, gy.cuda(), T.pool_activation(d, x.cuda()), w.cuda())
    same_values(g_w, f_w, 1e-5), same_values(g_x, f_x, 1e-5)


def test_workspaces_of_other_kinds():
    """A workspace is any object whose get(bytes) returns an address and a size: one without a `buf`, and a subclass of
    Workspace that overrides get."""
    class Mine:
        def __init__(self):
            self.mem, self.asked = torch.empty(1 << 22, dtype=torch.uint8, device="cuda"), []

        def get(self, nbytes):
            self.asked.append(nbytes)
            return int(self.mem.data_ptr()), int(self.mem.numel())

    class Counted(T.Workspace):
        asked = 0

        def get(self, nbytes):
            self.asked += 1
            return super().get(nbytes)

    d = mk(8, 64, 72, 14, 14, 3, 1, 1)
    sh = T.shapes(d)
    args = [randn(sh[k], i, "f32").cuda() for i, k in enumerate(("g_y", "x_u", "w"))]
    want = T.conv_bwd_filtered(d, *args)
    mine, counted = Mine(), Counted()
    for ws in (mine, counted, counted):
        assert all(torch.equal(a, b) for a, b in zip(want, T.conv_bwd_filtered(d, *args, ws=ws)))
    assert len(mine.asked) == 1 and mine.asked[0] > 0 and counted.asked == 2
    with pytest.raises(TypeError):
        Mine.get = lambda self, nbytes: None
        T.conv_bwd_filtered(d, *args, ws=Mine())


# N, C_in, C_out, H, W, K, stride, r: dense layers on codes; reduced maps, patch rows of 4 k patches, others
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(4, 64, 72, 14, 14, 3, 1, 2), (2, 40, 24, 16, 16, 1, 1, 2), (1, 32, 300, 8, 8, 3, 2, 2), (1, 16, 16, 4, 270, 1, 1, 2)])
def test_input_gradient_on_codes_without_workspace(oracle, case, dtype):
    """The reduced input gradient on codes takes a null workspace on every layer, the full one where patch rows are whole
    runs and otherwise with the reduced map as workspace: bit for bit what the workspace of gf_workspace_bytes gives."""
    N, Ci, Co, H, W, K, s, r = case
    d = mk(N, Ci, Co, H, W, K, s, K // 2, r=r, dtype=dtype)
    sh = T.shapes(d)
    rng = np.random.default_rng(5)
    gy_q, w_q = (torch.from_numpy(rng.integers(-127, 128, z).astype(np.int8)).cuda() for z in (sh["gy_u"], sh["w"][:2]))
    p = lambda t: int(t.data_ptr())  # noqa: E731
    for reduced in (True, False):
        want = T.conv_bwd_input_q8(d, gy_q, w_q, 1e-3, reduced_out=reduced)
        got = torch.full_like(want, 7.0)
        free = reduced or (sh["gy_u"][3] % 4 == 0 and r * s in (2, 4) and W == sh["gy_u"][3] * r * s)
        least = 0 if free else 4 * N * Ci * sh["x_u"][2] * sh["x_u"][3]
        mem = torch.empty(max(least, 1), dtype=torch.uint8, device="cuda")
        B.gf_conv_bwd_input_q8(d, p(gy_q), p(w_q), 1e-3, p(got), reduced, p(mem) if least else 0, least, torch.cuda.current_stream().cuda_stream)
        assert torch.equal(got, want), reduced


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(2, 64, 72, 14, 14), (1, 512, 16, 4, 4), (3, 20, 13, 31, 37), (1, 8, 600, 9, 7)])
def test_pointwise_input_gradient_without_workspace(oracle, case, dtype):
    """The input gradient alone of a pointwise layer, vanilla BP: a null workspace is taken."""
    N, Ci, Co, H, W = case
    d, u = mk(N, Ci, Co, H, W, r=1, dtype=dtype), mk(N, Ci, Co, 2 * H, 2 * W, r=2, dtype=dtype)   # u: d on its patch grid
    sh = T.shapes(d)
    w, gy = randn(sh["w"], 1, dtype), randn(sh["g_y"], 2, dtype)
    _, ref = oracle.bwd_exact(odesc(oracle, d), np.zeros(sh["x"]), to64(w), to64(gy))
    wg, gg, st = w.cuda(), gy.cuda(), torch.cuda.current_stream().cuda_stream
    for call in (lambda o: B.gf_conv_bwd_exact(d, 0, int(wg.data_ptr()), int(gg.data_ptr()), 0, o, 0, 0, st),
                 lambda o: B.gf_conv_bwd_input(d, int(gg.data_ptr()), int(wg.data_ptr()), o, False, 0, 0, st),
                 lambda o: B.gf_conv_bwd_unique(u, int(gg.data_ptr()), 0, int(wg.data_ptr()), 0, o, True, 0, 0, st)):
        out = torch.empty(sh["x"], dtype=gy.dtype, device="cuda")
        call(int(out.data_ptr()))
        assert rel_err(out, ref) <= TOL[dtype]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [
    (1, 40, 30, 18, 18, 1, 1, 2),      # K of a few chunks: one launch
    (1, 8, 16, 24, 44, 3, 1, 2),       # ... and 3 x 3 taps: 5 chunks in bf16, past the rule's edge; 9 in fp32
    (1, 24, 40, 16, 32, 3, 1, 2),      # 2 and 4 chunks
    (8, 64, 128, 56, 56, 3, 2, 2),     # several slabs, aligned planes: contraction and slab sums apart
    (3, 5, 9, 30, 34, 3, 1, 2),        # ... planes and channels that are no whole vectors
    (4, 296, 8, 52, 52, 1, 1, 2),
])
def test_weight_gradient_alone(oracle, case, dtype):
    N, Ci, Co, H, W, K, s, r = case
    d = mk(N, Ci, Co, H, W, K, s, K // 2, r=r, dtype=dtype)
    sh = T.shapes(d)
    x_u, gy_u = randn(sh["x_u"], 1, dtype), randn(sh["gy_u"], 2, dtype)
    g_w = T.conv_bwd_weight(d, x_u.cuda(), gy_u.cuda())
    assert rel_err(g_w, oracle.bwd_weight(odesc(oracle, d), to64(x_u), to64(gy_u))) <= 1e-5   # fp32 sums of either type


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [
    (1, 40, 24, 32, 32, 3, 1, 2),      # two slabs in fp32: added inside the launch
    (6, 24, 40, 32, 32, 3, 1, 2),      # three in bf16, 12 in fp32: apart
    (9, 70, 72, 40, 34, 3, 1, 2),      # four tiles with ragged edges
    (2, 130, 129, 40, 34, 3, 1, 2),    # nine tiles of five slabs in fp32: inside
    (3, 5, 9, 150, 134, 5, 2, 2),      # channels that are no whole vectors
    (33, 12, 20, 30, 30, 1, 1, 2),     # 1 x 1: 59 slabs in fp32 apart with a reduced map only, 15 in bf16 inside
    (40, 12, 20, 30, 30, 1, 1, 2),     # ... 71 apart, 18 apart with a reduced map only
])
def test_slab_sums_inside_and_apart(oracle, case, dtype):
    check_filtered(oracle, case, dtype)
    N, Ci, Co, H, W, K, s, r = case
    d = mk(N, Ci, Co, H, W, K, s, K // 2, r=r, dtype=dtype)
    sh = T.shapes(d)
    x_u, gy_u, w = randn(sh["x_u"], 1, dtype), randn(sh["gy_u"], 2, dtype), randn(sh["w"], 3, dtype)
    ref = oracle.bwd_weight(odesc(oracle, d), to64(x_u), to64(gy_u))
    for reduced in (True, False):
        g_w, g_x = T.conv_bwd_chained(d, gy_u.cuda(), x_u.cuda(), w.cuda(), reduced_out=reduced)
        assert rel_err(g_w, ref) <= 1e-5   # fp32 sums of either type
        assert rel_err(g_x, to64(T.conv_bwd_input(d, gy_u.cuda(), w.cuda(), reduced_out=reduced))) <= TOL[dtype]
    gy_u[0, 0, 0, 0] = float("inf")       # in one slab of one row
    g_w, _ = T.conv_bwd_chained(d, gy_u.cuda(), x_u.cuda(), w.cuda())
    assert not torch.isfinite(g_w[0]).any() and rel_err(g_w[1:], ref[1:]) <= 1e-5


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", [(6, 130, 24, 64, 130, 3, 1), (8, 72, 8, 78, 78, 3, 1), (8, 72, 8, 79, 80, 3, 1), (9, 200, 16, 131, 66, 3, 2)])
def test_vanilla_input_gradient_alone(oracle, case, dtype):
    """Few output channels, on both sides of the size from which g_x alone has larger tiles: the bits of the call for both in
    bf16, in fp32 the same products in partial sums of 16 instead of 32."""
    N, Ci, Co, H, W, K, s = case
    d = mk(N, Ci, Co, H, W, K, s, 1, r=1, dtype=dtype)
    sh = T.shapes(d)
    x, w, gy = randn(sh["x"], 1, dtype), randn(sh["w"], 2, dtype, scale=0.1), randn(sh["g_y"], 3, dtype)
    _, only = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda(), want_gw=False)
    _, both = T.conv_bwd_exact(d, x.cuda(), w.cuda(), gy.cuda())
    _, ref = oracle.bwd_exact(odesc(oracle, d), to64(x), to64(w), to64(gy))
    assert rel_err(only, ref) <= TOL[dtype] and rel_err(both, ref) <= TOL[dtype]
    assert torch.equal(only, both) if dtype == "bf16" else rel_err(only, to64(both)) <= 1e-6

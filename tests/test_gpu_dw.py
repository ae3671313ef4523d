"""GPU parity of the fused backward step of a linear layer (weight gradient on the matrix cores,
consumed by the update in the same kernel).  Two-stage check, because the gradient is a long fp32
accumulation while the update decides integer codes:
  1. the gradient the kernel used (dW_out) against the oracle's fp64 X^T dY, to the GEMM tolerance;
  2. codes, (s, b) and optimizer state against the oracle's step fed with exactly that gradient: bit for bit.
Every case is run a second time on its own copies of the buffers with dW_out = NULL -- the call a training loop
makes, where the gradient is not written anywhere -- and must leave the same codes, (s, b) and state, bit for bit."""
import numpy as np
import pytest
import torch

from oracle import omc_oracle as orc
from paper_2205_03494_amd import omc, synth
from gpu_util import bits_equal, dw_route, pair, to_dev
from test_gpu_gemm import check

pytestmark = pytest.mark.gpu


def run_case(EM, M, N, K, kind, lr, use_pvt=True, steps=2, grad_scale=1.0, rows=None, w_scale=0.05):
    want_dw = True
    of, gf = pair(*EM)
    n = K * N
    W = synth.normal_f32(n, w_scale, 2)
    packed, sb = orc.compress(W, of, use_pvt=use_pvt)
    st0 = np.zeros(n, np.float32) if kind >= 1 else None
    st1 = np.zeros(n, np.float32) if kind == 2 else None
    codes_d, sb_d = to_dev(packed), to_dev(sb)
    st0_d = None if st0 is None else to_dev(st0)
    st1_d = None if st1 is None else to_dev(st1)
    ws = torch.empty(omc.omc_dw_update_workspace_bytes(gf, M, N, K), dtype=torch.uint8, device="cuda")
    dW_d = torch.full((K, N), float("nan"), device="cuda") if want_dw else None
    # the same steps without a gradient copy, on separate buffers (workspace included)
    codes_n, sb_n = codes_d.clone(), sb_d.clone()
    st0_n = None if st0_d is None else st0_d.clone()
    st1_n = None if st1_d is None else st1_d.clone()
    ws_n = torch.empty_like(ws)
    for t in range(1, steps + 1):
        X = synth.to_bf16_bits(synth.normal_f32(M * K, 1.0, 10 + t))
        dY = synth.to_bf16_bits(synth.normal_f32(M * N, grad_scale / M, 20 + t))
        X_d, dY_d = to_dev(X), to_dev(dY)
        omc.omc_dw_update_recompress(X_d, dY_d, codes_d, gf, sb_d, use_pvt, st0_d, st1_d,
                                     omc.opt(kind, lr, t=t), dW_d, M, N, K, ws)
        omc.omc_dw_update_recompress(X_d, dY_d, codes_n, gf, sb_n, use_pvt, st0_n, st1_n,
                                     omc.opt(kind, lr, t=t), None, M, N, K, ws_n)
        torch.cuda.synchronize()
        assert torch.equal(codes_n, codes_d), f"dW_out = NULL: codes differ at step {t}"
        assert torch.equal(sb_n.view(torch.int32), sb_d.view(torch.int32)), f"dW_out = NULL: (s, b) differ at step {t}"
        if st0_d is not None:
            assert torch.equal(st0_n.view(torch.int32), st0_d.view(torch.int32)), f"dW_out = NULL: state0 differs at step {t}"
        if st1_d is not None:
            assert torch.equal(st1_n.view(torch.int32), st1_d.view(torch.int32)), f"dW_out = NULL: state1 differs at step {t}"
        g = dW_d.cpu().numpy()
        assert np.all(np.isfinite(g))
        if rows is None:
            check(g, orc.gemm_dw(X, dY, M, N, K, threads=8), (0, K))
        else:
            for r0 in rows:
                check(g, orc.gemm_dw(X, dY, M, N, K, rows=(r0, r0 + 16), threads=8), (r0, r0 + 16))
        orc.step_quantized(packed, n, of, sb, g.ravel(), st0, st1, orc.Opt(kind=kind, lr=lr, t=t), use_pvt=use_pvt)
        assert np.array_equal(codes_d.cpu().numpy(), packed), f"codes differ at step {t}"
        assert bits_equal(sb_d.cpu().numpy(), sb), (sb_d.cpu().numpy(), sb)
        if st0 is not None:
            assert bits_equal(st0_d.cpu().numpy(), st0)
        if st1 is not None:
            assert bits_equal(st1_d.cpu().numpy(), st1)


@pytest.mark.parametrize("kind,lr", [(0, 0.05), (1, 0.05), (2, 1e-3)])
@pytest.mark.parametrize("EM", [(4, 3), (5, 2), (3, 4), (4, 3, 4)])
def test_small_shapes(EM, kind, lr):
    run_case(EM, 96, 128, 256, kind, lr)


@pytest.mark.parametrize("shape", [(32, 128, 256), (160, 256, 512), (64, 384, 256)])
def test_tile_grid_and_minimal_contraction(shape):
    M, N, K = shape
    run_case((4, 3), M, N, K, 0, 0.05)


@pytest.mark.parametrize("M,kind,lr", [(1024, 0, 0.05), (4096, 1, 0.05), (2048, 2, 1e-3)])
def test_contraction_split_between_workgroups(M, kind, lr):
    """Few tiles and many rows: the M rows are shared out between workgroups, which leave partial sums, or between teams of waves of one
    workgroup; either way they are added in a fixed order.  Two runs must agree bit for bit with each other (run_case compares the
    second step too) and with the oracle's step on the gradient that was used."""
    run_case((4, 3), M, 128, 256, kind, lr, steps=2)
    run_case((4, 3), M, 256, 512, kind, lr, steps=1)


def test_without_the_transformation_and_with_saturating_updates():
    run_case((4, 3), 64, 128, 256, 0, 0.05, use_pvt=False)
    run_case((2, 5), 64, 128, 256, 0, 50.0, grad_scale=100.0)      # most weights end at the format's limits


def test_config5_layer_sampled_gradient_rows():
    # the feed-forward layer of the benchmark shape: X [8192 x 1024], W [1024 x 4096]
    run_case((4, 3), 8192, 4096, 1024, 0, 0.01, steps=1, rows=(0, 300, 500, 700, 1008))   # every 256-row tile, full width


@pytest.mark.parametrize("kind,lr", [(0, 0.05), (1, 0.05), (2, 1e-3)])
@pytest.mark.parametrize("EM", [(3, 7), (2, 3), (5, 7), (4, 14), (8, 7), (5, 10)])
def test_other_code_widths_take_the_two_kernel_path(EM, kind, lr):
    """6-, 11-, 13-, 16- and 19-bit formats: the gradient passes through the workspace as partial sums and a second kernel adds them and
    updates 2048 weights per wave; same two-stage check."""
    run_case(EM, 96, 128, 256, kind, lr)


def test_other_code_widths_with_split_contraction_and_several_tiles():
    run_case((3, 7), 2048, 256, 512, 1, 0.05, steps=2)
    run_case((2, 3), 1024, 128, 256, 0, 0.05, steps=2, grad_scale=20.0)


@pytest.mark.parametrize("EM", [(4, 18), (5, 23), (8, 16)])
def test_wide_mantissa_formats_keep_exact_fit_sums(EM):
    """16 and more mantissa bits: the update kernel carries the rounding errors of the fit's sums like the streaming
    kernels of these formats do, so (s, b) still match the oracle bit for bit."""
    run_case(EM, 96, 128, 256, 1, 0.05)
    run_case(EM, 1024, 256, 512, 0, 0.05, steps=1)


def test_fp32_as_a_format_is_plain_sgd():
    """S1E8M23 stores fp32 itself; without the transformation the fused step must equal w - lr * dW in fp32."""
    M, N, K = 64, 128, 256
    gf = omc.fmt(8, 23)
    W = synth.normal_f32(K * N, 0.05, 2)
    codes = to_dev(W.view(np.uint8).copy())
    sb = torch.tensor([1.0, 0.0], device="cuda")
    X = synth.to_bf16_bits(synth.normal_f32(M * K, 1.0, 11))
    dY = synth.to_bf16_bits(synth.normal_f32(M * N, 1.0 / M, 21))
    ws = torch.empty(omc.omc_dw_update_workspace_bytes(gf, M, N, K), dtype=torch.uint8, device="cuda")
    dW = torch.zeros((K, N), device="cuda")
    omc.omc_dw_update_recompress(to_dev(X), to_dev(dY), codes, gf, sb, False, None, None, omc.opt(0, 0.05), dW, M, N, K, ws)
    torch.cuda.synchronize()
    g = dW.cpu().numpy().ravel()
    step = (np.float32(0.05) * g).astype(np.float32)
    want = (W - step).astype(np.float32)
    assert bits_equal(codes.cpu().numpy().view(np.float32), want)
    assert sb.cpu().numpy().tolist() == [1.0, 0.0]


def test_large_matrix_is_updated_in_the_products_epilogue():
    # 4096 x 4096 weights = 1024 tiles of 128 x 128: no split, the update runs in the product kernel's epilogue
    assert dw_route(8, 64, 4096, 4096) == (True, 1, 1)
    run_case((4, 3), 64, 4096, 4096, 1, 0.05, steps=1, rows=(0, 2000, 4080))


@pytest.mark.parametrize("EM,kind,lr", [((4, 3), 0, 0.05), ((3, 7), 1, 0.05), ((2, 3), 2, 1e-3)])
def test_long_contraction_on_a_small_grid(EM, kind, lr):
    """4096 rows on 2048 x 1024 weights: 8-bit codes are updated by two teams of waves on 128 x 128 tiles in one kernel, the others from two partial
    sums."""
    run_case(EM, 4096, 2048, 1024, kind, lr, steps=2, rows=(0, 16, 320, 1008))


@pytest.mark.parametrize("EM", [(4, 3), (3, 7)])
@pytest.mark.parametrize("shape", [(160, 2048, 1024), (2080, 1024, 512), (2048, 2048, 512), (1056, 2048, 1024), (544, 4096, 2048),
                                   (1056, 4096, 4096), (4128, 384, 512)])
def test_every_tile_of_the_product_and_uneven_shares(EM, shape):
    """Tiles of 64 x 64 (one, two and four teams of waves) and 128 x 128 (one and two), in the kernel that updates 8-bit codes in its epilogue and
    in the one that leaves partial sums, there also 256 x 128; 65 or 33 steps of 32 rows do not share out evenly."""
    M, N, K = shape
    run_case(EM, M, N, K, 1, 0.05, steps=1, rows=None if K * N <= 1 << 20 else (0, 16, K // 2 - 16, K - 16))


@pytest.mark.parametrize("kind,lr", [(0, 0.05), (2, 1e-3)])
@pytest.mark.parametrize("shape", [(8192, 1024, 4096), (4096, 128, 256)])
def test_contraction_in_two_and_in_eight_parts(kind, lr, shape):
    """Room for two copies of the gradient: 8-bit codes are updated by two teams of waves in one kernel; for eight: teams and splits."""
    M, N, K = shape
    run_case((4, 3), M, N, K, kind, lr, steps=1, rows=(0, K - 16))


@pytest.mark.parametrize("kind,lr", [(0, 2.0 ** 45), (1, 2.0 ** 45), (2, 0.6 * 2.0 ** 105)])
@pytest.mark.parametrize("M", [96, 4096])
def test_eight_bit_format_whose_top_binades_need_the_wide_rounding(M, kind, lr):
    """S1E7M0 with a bias below 23 holds values above 2^105, which the rounding by add and subtract cannot reach.  96 rows: updated
    in the product's epilogue; 4096: by the second kernel, from partial sums."""
    run_case((7, 0, 10), M, 128, 256, kind, lr, steps=1, grad_scale=2.0 ** 60, w_scale=2.0 ** 107)


def test_epilogue_combines_its_waves_sums_without_rounding():
    """Two weights of +-2^80 in rows of two waves of a 64-row tile, ones in the rows of the wave between them: whoever adds the waves' sums in
    plain fp64 loses the ones, and with them their share of b.  V = Vt + 0.25 for the ones and V = Vt elsewhere (the zeros
    become codes of 0.25), so that what a wave loses beside +-2^80 it loses from both sums: s = 1, b = 0.25 x share of the ones, exactly."""
    of, gf = pair(7, 0, 40)
    M, N, K = 32, 128, 256
    assert dw_route(8, M, N, K) == (True, 4, 1)             # 64 x 64 tiles, eight waves of four rows in turn
    ones = (np.arange(K) % 8) >= 4                          # rows of the odd waves; the others hold zeros
    codes = np.where(ones[:, None], 40, 0) * np.ones((1, N), np.int64)
    codes[0, 0], codes[8, 0] = 120, 0x80 | 120
    packed, sb = orc.pack(codes.ravel().astype(np.uint32), 8), np.array([1.0, 0.25], np.float32)
    codes_d, sb_d = to_dev(packed), to_dev(sb)
    X, dY = torch.zeros((M, K), dtype=torch.int16, device="cuda"), torch.zeros((M, N), dtype=torch.int16, device="cuda")
    ws = torch.empty(omc.omc_dw_update_workspace_bytes(gf, M, N, K), dtype=torch.uint8, device="cuda")
    omc.omc_dw_update_recompress(X, dY, codes_d, gf, sb_d, True, None, None, omc.opt(0, 0.0), None, M, N, K, ws)
    orc.step_quantized(packed, K * N, of, sb, np.zeros(K * N, np.float32), None, None, orc.Opt(kind=0, lr=0.0))
    assert sb.tolist() == [1.0, 0.125]                      # (half of the rows)
    assert np.array_equal(codes_d.cpu().numpy(), packed)
    assert bits_equal(sb_d.cpu().numpy(), sb), (sb_d.cpu().numpy(), sb)


# in one kernel or through partial sums, tile, splits
ROUTES = {
    ((4, 3), (1024, 1408, 3840)): (True, 0, 1), ((4, 3), (96, 768, 4352)): (True, 1, 1), ((4, 3), (384, 896, 2816)): (True, 2, 1),
    ((4, 3), (32, 2944, 256)): (True, 3, 1), ((4, 3), (32, 128, 256)): (True, 4, 1), ((4, 3), (2048, 128, 1024)): (True, 5, 1),
    ((4, 3), (4096, 256, 4352)): (False, 0, 5), ((4, 3), (8192, 256, 4352)): (False, 1, 4), ((4, 3), (4096, 128, 4096)): (False, 2, 5),
    ((4, 3), (4096, 128, 2048)): (False, 5, 3), ((3, 7), (4096, 256, 4352)): (False, 0, 5), ((3, 7), (96, 768, 4352)): (False, 1, 1),
    ((3, 7), (384, 896, 2816)): (False, 2, 1), ((3, 7), (32, 2944, 256)): (False, 3, 1), ((3, 7), (4096, 128, 2048)): (False, 5, 3),
    ((3, 7), (1024, 128, 256)): (False, 4, 2), ((3, 7), (2048, 128, 1280)): (False, 4, 3), ((3, 7), (2048, 128, 256)): (False, 4, 4),
    ((3, 7), (4096, 128, 1024)): (False, 4, 5), ((3, 7), (4096, 128, 768)): (False, 4, 6), ((3, 7), (4352, 128, 512)): (False, 4, 7),
    ((3, 7), (4096, 128, 256)): (False, 4, 8), ((3, 7), (8192, 4096, 1024)): (False, 0, 2),
}


@pytest.mark.parametrize("EM,shape,route", [(EM, shape, route) for (EM, shape), route in ROUTES.items()])
def test_every_tile_in_both_routes_and_every_number_of_splits(EM, shape, route):
    """Tiles of both routes, and one to eight partial sums, also such as cut the steps into runs of unequal length (3, 5, 6, 7) under two teams."""
    M, N, K = shape
    assert dw_route(1 + sum(EM), M, N, K) == route
    run_case(EM, M, N, K, 1, 0.05, steps=1, rows=None if M * N * K <= 1 << 28 else (0, 16, K // 2 - 16, K - 16))

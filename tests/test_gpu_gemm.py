"""GPU parity of the dequant-fused forward GEMM against the oracle's fp64 GEMM on the decompressed
weights.  Tolerance (the reading of "relative tolerance 1e-3"): |C - C_ref| <= 1e-3 |C_ref| + 1e-3 rms(C_ref)."""
import numpy as np
import pytest
import torch

from oracle import omc_oracle as orc
from paper_2205_03494_amd import omc, synth
from gpu_util import gemm_sums, gemm_tile, pair, to_dev

pytestmark = pytest.mark.gpu


def run_gemm(A_bits, packed, gf, sb, M, N, K):
    C = torch.full((M, N), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(omc.omc_dequant_gemm_workspace_bytes(M), dtype=torch.uint8, device="cuda")
    omc.omc_dequant_gemm(to_dev(A_bits), to_dev(packed), gf, None if sb is None else to_dev(sb), C, M, N, K, ws)
    torch.cuda.synchronize()
    return C.cpu().numpy()


def tile_sample_rows(M, seed, tile=256, per_quarter=1):
    """Rows to check at full size: from every 256 rows of the output one row (or several) out of each 64-row quarter, which is the least that
    a tile covers, at seeded offsets."""
    rng = np.random.default_rng(seed)
    rows = [t * tile + 64 * q + int(rng.integers(0, 64)) for t in range(M // tile) for q in range(4) for _ in range(per_quarter)]
    return np.array(sorted(set(rows)))


def check_rows(C, ref, rows):
    """check() on a list of rows: ref holds the oracle's result for exactly those rows, in order."""
    return check(C[rows], ref, (0, len(rows)))


def check(C, ref, rows):
    ref = np.asarray(ref)
    got = C[rows[0]:rows[1]].astype(np.float64)
    rms = np.sqrt(np.mean(ref ** 2))
    err = np.abs(got - ref)
    assert np.all(err <= 1e-3 * np.abs(ref) + 1e-3 * rms), float((err / (np.abs(ref) + rms)).max())
    return float(np.linalg.norm(got - ref) / np.linalg.norm(ref))


@pytest.mark.parametrize("EM", [(4, 3), (5, 2), (3, 4), (2, 3), (3, 7), (8, 7), (4, 3, 4)])
@pytest.mark.parametrize("shape", [(256, 128, 32), (256, 256, 96), (512, 128, 160), (256, 128, 2048), (512, 256, 2112)])
def test_small_shapes_all_rows(EM, shape):
    of, gf = pair(*EM)
    M, N, K = shape
    A = synth.to_bf16_bits(synth.normal_f32(M * K, 1.0, 1))
    W = synth.normal_f32(K * N, 1 / np.sqrt(K), 2)
    packed, sb = orc.compress(W, of)
    C = run_gemm(A, packed, gf, sb, M, N, K)
    rel = check(C, orc.dequant_gemm(A, packed, of, sb, M, N, K, threads=8), (0, M))
    assert rel < 1e-5
    # without the transformation
    C = run_gemm(A, packed, gf, None, M, N, K)
    check(C, orc.dequant_gemm(A, packed, of, None, M, N, K, threads=8), (0, M))


# One size for every kernel of the products, by tile and chains of sums (a test without a GPU holds that); nearly all contractions end on half a step.
FP8_KERNELS = {(0, 1): (3584, 3584, 2976), (1, 1): (2560, 3328, 224), (2, 1): (5632, 768, 416), (3, 1): (1792, 1792, 224), (4, 1): (9472, 128, 288),
               (4, 2): (8448, 128, 288), (5, 1): (256, 2048, 32), (5, 2): (256, 2816, 224), (5, 4): (256, 128, 32), (6, 2): (6400, 128, 608),
               (6, 4): (256, 128, 480), (7, 4): (256, 128, 4000)}
BITS_KERNELS = {(0, 1): (3328, 3840, 224), (1, 1): (3328, 1920, 672), (2, 1): (1792, 3584, 544), (3, 1): (12544, 256, 160), (3, 2): (1280, 1664, 2592),
                (4, 1): (1792, 2944, 96), (5, 1): (768, 2176, 32), (5, 2): (256, 128, 32), (6, 2): (256, 128, 96), (6, 4): (256, 128, 160),
                (7, 4): (256, 128, 672)}


@pytest.mark.parametrize("EM", [(2, 3), (5, 2), (2, 3, 2), (5, 2, 14), (3, 4)])
@pytest.mark.parametrize("shape", [(256, 128, 64), (512, 256, 96), (2048, 2048, 512), (7936, 1024, 1536), (8192, 4096, 1024)] + list(BITS_KERNELS.values()))
def test_every_code_is_converted_exactly(EM, shape):
    """Formats that the hardware converts (S1E2M3 with bias 1, S1E5M2 with bias 15, whose top exponent the hardware reads as Inf and NaN) beside others of the same width:
    with one-hot rows of A the product is the weights' values, every code among them, in both directions and in every tile."""
    of, gf = pair(*EM)
    M, N, K = shape
    for tile, sums in [k for k in BITS_KERNELS if BITS_KERNELS[k] == shape]:
        assert (gemm_tile(EM, M, N, K), gemm_sums(EM, M, N, K)) == (tile, sums)
    bits = 1 + EM[0] + EM[1]
    rng = np.random.default_rng(bits)
    codes = np.concatenate([np.arange(1 << bits), rng.integers(0, 1 << bits, K * N - (1 << bits))]).astype(np.uint32)
    packed = to_dev(orc.pack(codes, bits))
    W = to_dev(orc.decode(codes, of))
    ws = torch.empty(omc.omc_dequant_gemm_workspace_bytes(M), dtype=torch.uint8, device="cuda")
    rows = torch.arange(M, device="cuda")
    for product, m, n, k in ((omc.omc_dequant_gemm, M, N, K), (omc.omc_dequant_gemm_dx, M, N, K), (omc.omc_dequant_gemm_dx, M, K, N)):
        transposed = product is omc.omc_dequant_gemm_dx
        width, columns = (n, k) if transposed else (k, n)
        if transposed and columns % 128 != 0:
            continue                                          # refused in this direction
        A = torch.zeros(m, width, dtype=torch.bfloat16, device="cuda")
        A[rows, rows % width] = 1.0
        C = torch.full((m, columns), float("nan"), device="cuda")
        product(A, packed, gf, None, C, m, n, k, ws)
        assert torch.equal(C, (W.reshape(k, n).t() if transposed else W.reshape(k, n))[rows % width])


def test_identity_pattern_pins_the_tile_layout():
    # A = one-hot rows, W = distinct representable values: C must reproduce W's rows exactly
    of, gf = pair(4, 3)
    M, N, K = 256, 128, 64
    A = np.zeros((M, K), np.float32)
    A[np.arange(M), np.arange(M) % K] = 1.0
    codes = (np.arange(K * N) * 7 + 3) % 120 + 1
    W = orc.decode(codes.astype(np.uint32), of)
    packed = orc.pack(codes.astype(np.uint32), 8)
    C = run_gemm(synth.to_bf16_bits(A.ravel()), packed, gf, None, M, N, K)
    want = W.reshape(K, N)[np.arange(M) % K]
    assert np.array_equal(C, want)


@pytest.mark.parametrize("shape", [(8192, 4096, 1024), (8192, 1024, 4096)])
def test_config5_shapes_sampled_rows(shape):
    M, N, K = shape
    of, gf = pair(4, 3)
    A = synth.to_bf16_bits(synth.normal_f32(M * K, 1.0, 11))
    W = synth.normal_f32(K * N, 1 / np.sqrt(K), 12)
    packed, sb = orc.compress(W, of)
    C = run_gemm(A, packed, gf, sb, M, N, K)
    assert np.all(np.isfinite(C))
    # rows of C depend on their own row of A only: the oracle multiplies the sampled rows as a matrix of their own
    rows = tile_sample_rows(M, seed=K)
    assert rows.size == 4 * (M // 256)
    ref = orc.dequant_gemm(np.ascontiguousarray(A.reshape(M, K)[rows]).ravel(), packed, of, sb, rows.size, N, K, threads=8)
    assert check_rows(C, ref, rows) < 1e-5
    for r0 in (0, M - 24):                                      # and two runs of consecutive rows at the ends
        ref = orc.dequant_gemm(A, packed, of, sb, M, N, K, rows=(r0, r0 + 24), threads=8)
        assert check(C, ref, (r0, r0 + 24)) < 1e-5


SMALL_KERNELS = {256: (5, 4), 2048: (6, 4), 4000: (7, 4)}    # of 256 x 128 results over so many products: 64 x 64 by one, two and four teams


@pytest.mark.parametrize("K", list(SMALL_KERNELS))
@pytest.mark.parametrize("top_at", [None, 0, -1, 12345])
def test_every_byte_code_exact_with_and_without_the_top_code(top_at, K):
    """S1E4M3 / bias 7 takes the hardware FP8 conversion, which reads a top code (value 480) as NaN; a tile whose sums show one anywhere in
    the stream is computed again, and both conversions must give the exact code values."""
    of, gf = pair(4, 3)
    M, N = 256, 128
    assert (gemm_tile((4, 3), M, N, K), gemm_sums((4, 3), M, N, K)) == SMALL_KERNELS[K]
    A = np.zeros((M, K), np.float32)
    pick = (np.arange(M) * 7 + 3) % K
    A[np.arange(M), pick] = 1.0
    codes = ((np.arange(K * N, dtype=np.int64) * 37 + 11) % 254).astype(np.uint32)
    codes = np.where(codes >= 127, codes + 1, codes)          # 0..126, 128..254: no top code, both signs, subnormals
    if top_at is not None:
        codes[top_at] = 0x7F if top_at != -1 else 0xFF
    W = orc.decode(codes, of)
    C = run_gemm(synth.to_bf16_bits(A.ravel()), orc.pack(codes, 8), gf, None, M, N, K)
    want = W.reshape(K, N)[pick]
    assert np.array_equal(C, want)


def run_gemm_dx(dY_bits, packed, gf, sb, M, N, K):
    dX = torch.full((M, K), float("nan"), dtype=torch.float32, device="cuda")
    ws = torch.empty(omc.omc_dequant_gemm_workspace_bytes(M), dtype=torch.uint8, device="cuda")
    omc.omc_dequant_gemm_dx(to_dev(dY_bits), to_dev(packed), gf, None if sb is None else to_dev(sb), dX, M, N, K, ws)
    torch.cuda.synchronize()
    return dX.cpu().numpy()


@pytest.mark.parametrize("EM", [(4, 3), (5, 2), (2, 3), (3, 7), (8, 7), (4, 3, 4)])
@pytest.mark.parametrize("shape", [(256, 32, 128), (256, 96, 256), (512, 160, 128), (256, 2048, 128), (512, 2112, 256)])
def test_dx_small_shapes_all_rows(EM, shape):
    of, gf = pair(*EM)
    M, N, K = shape
    dY = synth.to_bf16_bits(synth.normal_f32(M * N, 1.0, 5))
    W = synth.normal_f32(K * N, 1 / np.sqrt(K), 2)
    packed, sb = orc.compress(W, of)
    dX = run_gemm_dx(dY, packed, gf, sb, M, N, K)
    rel = check(dX, orc.dequant_gemm_dx(dY, packed, of, sb, M, N, K, threads=8), (0, M))
    assert rel < 1e-5
    dX = run_gemm_dx(dY, packed, gf, None, M, N, K)
    check(dX, orc.dequant_gemm_dx(dY, packed, of, None, M, N, K, threads=8), (0, M))


@pytest.mark.parametrize("N", [64] + list(SMALL_KERNELS))   # (64: one step, by one team)
@pytest.mark.parametrize("top_at", [None, 777])
def test_dx_identity_pattern_pins_the_transposed_layout(top_at, N):
    # dY = one-hot rows: dX must reproduce columns of W exactly, with and without a top code (both conversions)
    of, gf = pair(4, 3)
    M, K = 256, 128
    assert gemm_tile((4, 3), M, K, N) == SMALL_KERNELS.get(N, (5, 4))[0]
    dY = np.zeros((M, N), np.float32)
    pick = (np.arange(M) * 5 + 1) % N
    dY[np.arange(M), pick] = 1.0
    codes = ((np.arange(K * N, dtype=np.int64) * 37 + 11) % 254).astype(np.uint32)
    codes = np.where(codes >= 127, codes + 1, codes)
    if top_at is not None:
        codes[top_at] = 0x7F
    W = orc.decode(codes, of).reshape(K, N)
    dX = run_gemm_dx(synth.to_bf16_bits(dY.ravel()), orc.pack(codes, 8), gf, None, M, N, K)
    want = W[:, pick].T
    assert np.array_equal(dX, want)


@pytest.mark.parametrize("shape", [(8192, 4096, 1024), (8192, 1024, 4096)])
def test_dx_config5_shapes_sampled_rows(shape):
    M, N, K = shape
    of, gf = pair(4, 3)
    dY = synth.to_bf16_bits(synth.normal_f32(M * N, 1.0, 13))
    W = synth.normal_f32(K * N, 1 / np.sqrt(K), 12)
    packed, sb = orc.compress(W, of)
    dX = run_gemm_dx(dY, packed, gf, sb, M, N, K)
    assert np.all(np.isfinite(dX))
    rows = tile_sample_rows(M, seed=N)
    ref = orc.dequant_gemm_dx(np.ascontiguousarray(dY.reshape(M, N)[rows]).ravel(), packed, of, sb, rows.size, N, K, threads=8)
    assert check_rows(dX, ref, rows) < 1e-5
    for r0 in (0, M - 24):
        ref = orc.dequant_gemm_dx(dY, packed, of, sb, M, N, K, rows=(r0, r0 + 24), threads=8)
        assert check(dX, ref, (r0, r0 + 24)) < 1e-5


@pytest.mark.parametrize("shape", [(256, 128, 32), (512, 256, 160), (256, 128, 4096), (256, 2048, 128)])
def test_large_offset_makes_the_row_sum_term_count(shape):
    """With the fitted (s, b) of zero-mean weights b is tiny and the b * rowsum(A) term hides inside the tolerance;
    a hand-made pair with a large offset makes both GEMMs depend on their row sums."""
    of, gf = pair(4, 3)
    M, N, K = shape
    A = synth.to_bf16_bits(synth.normal_f32(M * K, 1.0, 1) + np.float32(0.5))
    W = synth.normal_f32(K * N, 1 / np.sqrt(K), 2)
    packed, _ = orc.compress(W, of)
    sb = np.array([0.75, 0.125], np.float32)
    C = run_gemm(A, packed, gf, sb, M, N, K)
    check(C, orc.dequant_gemm(A, packed, of, sb, M, N, K, threads=8), (0, M))
    dY = synth.to_bf16_bits(synth.normal_f32(M * N, 1.0, 5) + np.float32(0.5))
    dX = run_gemm_dx(dY, packed, gf, sb, M, N, K) if K % 128 == 0 else None
    if dX is not None:
        check(dX, orc.dequant_gemm_dx(dY, packed, of, sb, M, N, K, threads=8), (0, M))


def both_directions(EM, M, N, K, rows, sb=None, seed=0):
    """A [M x K] times W stored [K x N] and times the transpose of W stored [N x K]: the same tiles in both directions."""
    of, gf = pair(*EM)
    A = synth.to_bf16_bits(synth.normal_f32(M * K, 1.0, seed + 1) + np.float32(0.25))
    packed, fitted = orc.compress(synth.normal_f32(K * N, 1 / np.sqrt(K), seed + 2), of)
    sb = fitted if sb is None else sb
    sub = np.ascontiguousarray(A.reshape(M, K)[rows]).ravel()
    worst = check_rows(run_gemm(A, packed, gf, sb, M, N, K), orc.dequant_gemm(sub, packed, of, sb, rows.size, N, K, threads=8), rows)
    dX = run_gemm_dx(A, packed, gf, sb, M, K, N)            # the same stream read as a weight matrix of N rows, K columns
    ref = orc.dequant_gemm_dx(sub, packed, of, sb, rows.size, K, N, threads=8)
    return max(worst, check_rows(dX, ref, rows))


@pytest.mark.parametrize("EM", [(1, 0), (2, 0), (2, 1), (3, 1), (3, 2), (2, 3), (3, 3), (4, 3), (5, 2), (4, 4), (2, 7), (3, 7),
                                (4, 7), (5, 7), (6, 7), (7, 7), (8, 7)])
@pytest.mark.parametrize("shape", [(256, 128, 96), (256, 256, 1056)])
def test_every_code_width_half_steps_and_teams(EM, shape):
    """All widths 2 .. 16 (odd ones start a thread's codes in the middle of a dword), contractions that end on half a step, and
    workgroups of one team and of several.  1e-5: fp32 sums of 1056 products, each within 2^-24 of the last partial sum."""
    M, N, K = shape
    assert both_directions(EM, M, N, K, np.arange(M), sb=np.array([0.75, 0.125], np.float32)) < 1e-5


HALF_STEP = [(256, 256, 2080), (2304, 896, 544), (4096, 1024, 288), (4096, 2048, 96), (4096, 4096, 288), (8192, 1024, 2080)]
HALF_STEP_SHAPES = {                                        # every tile of the two dispatch tables
    (4, 3): HALF_STEP + [(3584, 3584, 2976), (1536, 4352, 1312), (512, 4864, 544), (256, 2816, 224), (256, 128, 1056), (256, 128, 4000)],
    (3, 7): HALF_STEP + [(2560, 3328, 1056), (1536, 4608, 1056), (1792, 3584, 544), (512, 3968, 1056), (256, 1408, 1056)],
}


@pytest.mark.parametrize("EM,shape", [(EM, shape) for EM, shapes in HALF_STEP_SHAPES.items() for shape in shapes])
def test_every_tile_size_ends_on_half_a_step(EM, shape):
    """At least one shape per tile of the two dispatch tables (a test without a GPU holds that), 64 x 64 up to 256 x 256, rows of every
    tile."""
    M, N, K = shape
    assert both_directions(EM, M, N, K, tile_sample_rows(M, seed=K, per_quarter=4)) < 1e-5


@pytest.mark.parametrize("EM,kernel", [((4, 3), k) for k in FP8_KERNELS] + [(EM, k) for EM in ((2, 3), (5, 2), (3, 7), (4, 7), (5, 7)) for k in BITS_KERNELS])
def test_every_kernel_with_a_visible_offset(EM, kernel):
    """Both directions of every kernel in 6, 8, 11, 12 and 13 bits (odd widths start a thread's codes in the middle of a dword), with an offset whose row
    sums count for more than the products do.  1e-5: fp32 sums of at most 4000 products."""
    M, N, K = (FP8_KERNELS if EM == (4, 3) else BITS_KERNELS)[kernel]
    assert both_directions(EM, M, N, K, tile_sample_rows(M, seed=K + N), sb=np.array([0.75, 0.125], np.float32)) < 1e-5


@pytest.mark.parametrize("shape,bound", [((512, 512, 512), 3.7e-8), ((5120, 256, 1472), 5.8e-8), ((512, 512, 4096), 6.6e-8)])
def test_small_products_against_64_bits(shape, bound):
    """S1E4M3 codes without a transformation: every product is exact, what is off are the fp32 sums.  Dealt into two or four chains they
    are 3.4e-8, 5.2e-8 and 6.0e-8 off; in half or a quarter as many 4.0e-8, 6.5e-8 and 7.2e-8.  The bounds lie between the two."""
    of, gf = pair(4, 3)
    M, N, K = shape
    A = synth.to_bf16_bits(synth.normal_f32(M * K, 1.0, 3))
    packed, _ = orc.compress(synth.normal_f32(K * N, 1 / np.sqrt(K), 4), of)
    for got, want in ((run_gemm(A, packed, gf, None, M, N, K), orc.dequant_gemm(A, packed, of, None, M, N, K, threads=8)),
                      (run_gemm_dx(A, packed, gf, None, M, K, N), orc.dequant_gemm_dx(A, packed, of, None, M, K, N, threads=8))):
        assert np.linalg.norm(got.astype(np.float64) - want) <= bound * np.linalg.norm(want)


# A long contraction for the tiles that can be asked for one: (format, tile, chains) -> size
LONG_CONTRACTIONS = {((4, 3), 0, 1): (3072, 3072, 8192), ((4, 3), 1, 1): (6144, 3072, 8192), ((4, 3), 2, 1): (1536, 3072, 8192), ((4, 3), 3, 1): (4096, 640, 8192),
                     ((4, 3), 4, 1): (3072, 640, 8192), ((4, 3), 6, 4): (1024, 1024, 8192), ((4, 3), 7, 4): (256, 128, 8192), ((3, 7), 0, 1): (3072, 3072, 8192),
                     ((3, 7), 1, 1): (1536, 3072, 8192), ((3, 7), 3, 1): (6144, 640, 8192), ((3, 7), 3, 2): (1536, 1536, 8192), ((3, 7), 4, 1): (8192, 768, 4096),
                     ((3, 7), 6, 2): (1536, 768, 8192), ((3, 7), 7, 4): (256, 128, 8192)}


@pytest.mark.parametrize("kernel", list(LONG_CONTRACTIONS))
def test_row_sums_against_64_bits(kernel):
    """Weights of zero and an offset of one: the product is the row sums of A, here of one sign, whose error grows with the length of a chain of fp32 sums.  In two chains
    they are 11.5e-8 off over 8192 and 6.4e-8 over 4096; in the four and more that a row has, at most 5.2e-8 and 4.1e-8.  The bounds lie between the two."""
    EM, tile, sums = kernel
    M, N, K = LONG_CONTRACTIONS[kernel]
    assert (gemm_tile(EM, M, N, K), gemm_sums(EM, M, N, K)) == (tile, sums)
    gf = omc.fmt(*EM)
    A = torch.from_numpy(synth.normal_f32(M * K, 1.0, 5)).cuda().abs().bfloat16().reshape(M, K)
    want = A.double().sum(1)
    codes = torch.zeros(omc.omc_packed_bytes(gf, K * N), dtype=torch.uint8, device="cuda")
    sb = torch.ones(2, device="cuda")
    ws = torch.empty(omc.omc_dequant_gemm_workspace_bytes(M), dtype=torch.uint8, device="cuda")
    for product, sizes in ((omc.omc_dequant_gemm, (M, N, K)), (omc.omc_dequant_gemm_dx, (M, K, N))):
        C = torch.full((M, N), float("nan"), device="cuda")
        product(A, codes, gf, sb, C, *sizes, ws)
        assert torch.equal(C, C[:, :1].expand(M, N))
        assert (C[:, 0].double() - want).norm() <= (7e-8 if K == 8192 else 5.2e-8) * want.norm()


@pytest.mark.parametrize("shape", [(4096, 2048, 160), (256, 256, 544)])
def test_top_codes_in_some_tiles_only(shape):
    """A tile that meets the code that the FP8 conversion reads as NaN is computed again; its neighbours are not."""
    of, gf = pair(4, 3)
    M, N, K = shape
    A = np.zeros((M, K), np.float32)
    pick = (np.arange(M) * 7 + 3) % K
    A[np.arange(M), pick] = 1.0
    codes = ((np.arange(K * N, dtype=np.int64) * 37 + 11) % 254).astype(np.uint32)
    codes = np.where(codes >= 127, codes + 1, codes)
    codes[3 * N + 5] = 0x7F                                 # the first tile's columns, an early k
    codes[(K - 1) * N + N - 1] = 0xFF                       # the last tile's, the last k
    W = orc.decode(codes, of)
    packed = orc.pack(codes, 8)
    assert np.array_equal(run_gemm(synth.to_bf16_bits(A.ravel()), packed, gf, None, M, N, K), W.reshape(K, N)[pick])
    got = run_gemm_dx(synth.to_bf16_bits(A.ravel()), packed, gf, None, M, K, N)
    assert np.array_equal(got, W.reshape(N, K)[:, pick].T)


TOP_CODE_SHAPES = [(3584, 3584, 2976), (2560, 3328, 1056), (7936, 1024, 1056), (1536, 4352, 1312), (1280, 2944, 1056), (768, 2688, 1056),
                   (512, 2816, 1056), (512, 4864, 544), (256, 2816, 1056), (256, 128, 1056), (256, 128, 4000)]     # every tile in turn


@pytest.mark.parametrize("where", ["early", "late", "everywhere"])
@pytest.mark.parametrize("shape", TOP_CODE_SHAPES)
def test_top_codes_along_a_long_contraction(shape, where):
    """The large tiles (256 x 256 and both of 128 x 256, the first four shapes) look for top codes after an eighth of the steps too and stop
    there; whether they do, find one at the end, or find none, every weight has its exact value."""
    of, gf = pair(4, 3)
    M, N, K = shape
    A = np.zeros((M, K), np.float32)
    pick = (np.arange(M) * 7 + 3) % K
    A[np.arange(M), pick] = 1.0
    A = synth.to_bf16_bits(A.ravel())
    codes = ((np.arange(K * N, dtype=np.int64) * 37 + 11) % 254).astype(np.uint32)
    codes = np.where(codes >= 127, codes + 1, codes)
    rows = {"early": slice(3, 11, 7), "late": slice(K - 8, K, 7), "everywhere": slice(0, K, 97)}[where]
    for trans in (False, True):                             # stored [K x N], or [N x K] for the input gradient
        W = codes.reshape(N, K).T.copy() if trans else codes.reshape(K, N).copy()
        W[rows, 5::1408] = 0x7F
        W[rows, N - 1] = 0xFF
        packed = orc.pack(np.ascontiguousarray(W.T if trans else W).ravel(), 8)
        got = run_gemm_dx(A, packed, gf, None, M, K, N) if trans else run_gemm(A, packed, gf, None, M, N, K)
        assert np.array_equal(got, orc.decode(np.ascontiguousarray(W).ravel(), of).reshape(K, N)[pick])

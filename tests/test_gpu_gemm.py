"""GPU parity: halo_gemm_i8 int32 accumulators bit-exact against the oracle's exact integer product."""
import numpy as np
import pytest
import torch

from oracle import halo_oracle as orc
from paper_2501_02625_amd import binding
from tests import gpu_util as gu

pytestmark = pytest.mark.gpu


# M, N, K: the configuration is the library's choice, ragged edges and a K tail.  test_gemm_plan.py holds the choice; a test
# that means a tile size names it (test_units_and_tile_edges, test_every_tile_configuration_gives_the_same_accumulators).
SHAPES = [
    (128, 512, 512),       # config c1 forward: 32x64 tiles
    (32, 32, 16),
    (1, 1, 64),
    (300, 200, 272),       # ragged M, N; K not a multiple of the 128-byte unit
    (257, 129, 1040),
    (2048, 4096, 256),     # 128x128 tiles, two rounds
    (4096, 4096, 128),     # 128x128 tiles, four rounds
    (4100, 3900, 80),      # 128x128 tiles with ragged edges
    (512, 14336, 64),
]
# M, N of test_small_products: the tile that one product takes, and that the pair takes at the longest K of the test
SMALL_SHAPES = {
    (1, 64): ("16x64", "32x64"), (16, 16): ("16x64", "32x64"), (17, 72): ("32x64", "32x64"), (31, 250): ("32x64", "32x64"),
    (48, 4100): ("32x64", "32x64"), (100, 4056): ("32x64", "64x64"), (200, 4056): ("64x64", "128x128"),
    (200, 4096 + 40): ("128x128", "128x128"),
}
SMALL_K = [16, 128, 400, 512, 1040, 2064]


# K around the 128-byte units of the main loop (a partial one, one, one and a bit, odd and even counts), M and N around the
# tile edges, every tile size: what lies beyond the matrix must enter as zeros and must not be stored.
@pytest.mark.parametrize("K", [16, 112, 128, 144, 384, 656])
@pytest.mark.parametrize("M,N,config", [(127, 112, 4), (129, 144, 4), (255, 128, 2), (272, 96, 2), (257, 272, 0), (240, 250, 0)])
@pytest.mark.parametrize("trans_b", [True, False])
def test_units_and_tile_edges(M, N, K, config, trans_b):
    step = {0: 64, 2: 128, 4: 16}[config]
    K = (K + step - 1) // step * step
    rng = np.random.default_rng(M + N + K)
    a = rand_codes(rng, (M, K)); b = rand_codes(rng, (N, K) if trans_b else (K, N))
    bd = torch.zeros((b.shape[0], (b.shape[1] + 15) // 16 * 16), dtype=torch.int8, device=gu.DEV)
    bd[:, :b.shape[1]] = gu.to_dev(b)
    acc = torch.full((M + 1, (N + 3) // 4 * 4 + 16), -7, dtype=torch.int32, device=gu.DEV)
    binding.halo_gemm_i8_desc(binding.gemm_desc(gu.to_dev(a), bd[:, :b.shape[1]], trans_b=trans_b, acc_out=acc[:M, :N],
                                                config=config))
    gu.assert_codes_equal(acc[:M, :N], orc.gemm_codes(a, b.T if trans_b else b), "accumulators")
    assert bool((acc[M:] == -7).all()) and bool((acc[:, N:] == -7).all())


# Scaled outputs of the tiled kernels, stored in pieces of 64 bytes that two column tiles (fp32) or two pairs of them (bf16)
# share: column counts that end inside such a piece, rows that end inside the eight of a request, pitches off the line.
@pytest.mark.parametrize("M,N", [(120, 16), (137, 48), (249, 80), (264, 112), (130, 208), (260, 272)])
@pytest.mark.parametrize("config", [0, 2, 4])
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_scaled_outputs_at_tile_edges(M, N, config, dtype):
    K = 256
    rng = np.random.default_rng(M + N + config)
    a = rand_codes(rng, (M, K)); b = rand_codes(rng, (N, K))
    rs = rng.uniform(1e-3, 1e-2, M).astype(np.float32); cs = rng.uniform(1e-3, 1e-2, N).astype(np.float32)
    out = torch.full((M + 1, N + 24), -7.0, dtype=dtype, device=gu.DEV)
    binding.halo_gemm_i8_desc(binding.gemm_desc(gu.to_dev(a), gu.to_dev(b), trans_b=True, row_scale=gu.to_dev(rs),
                                                col_scale=gu.to_dev(cs), out=out[:M, :N], config=config))
    want = orc.dequantize(orc.gemm_codes(a, b.T), rs, cs)
    (gu.assert_f32_identical if dtype == torch.float32 else gu.assert_bf16_within_one_ulp)(out[:M, :N], want, "scaled output")
    assert bool((out[M:] == -7).all()) and bool((out[:, N:] == -7).all())


# bf16 outputs on both sides of the rule for whole lines (bf16_whole_lines: 2 Mi elements with a pitch off the half lines, 7 Mi
# otherwise), every tile size, the edge tiles a few rows and columns wide.  The fp32 output of the same product is the same
# number before its one rounding.  rows, cols, pitch, whole lines
LINES = [(1033, 2032, 2048, False), (1033, 2032, 2056, True), (3595, 2048, 2048, True), (3583, 2048, 2080, False), (455, 16144, 16160, True)]


@pytest.mark.parametrize("M,N,pitch,whole", LINES)
@pytest.mark.parametrize("config", [0, 2, 4])
def test_bf16_outputs_in_whole_and_half_lines(M, N, pitch, whole, config):
    K = 128
    rng = np.random.default_rng(M + N)
    a, b = gu.to_dev(rand_codes(rng, (M, K))), gu.to_dev(rand_codes(rng, (N, K)))
    rs = gu.to_dev(rng.uniform(1e-3, 1e-2, M).astype(np.float32)); cs = gu.to_dev(rng.uniform(1e-3, 1e-2, N).astype(np.float32))
    outs = [torch.full((M + 1, pitch), -7.0, dtype=dtype, device=gu.DEV) for dtype in (torch.float32, torch.bfloat16)]
    for out in outs:
        binding.halo_gemm_i8_desc(binding.gemm_desc(a, b, trans_b=True, row_scale=rs, col_scale=cs, out=out[:M, :N], config=config))
    assert torch.equal(outs[1], outs[0].bfloat16())


# B as a column slice that ends with its allocation (K-strided: the last row's pitch reaches past the end): the tiled kernels
# and the split-K kernel, N below, at and beyond a tile.
@pytest.mark.parametrize("M,config", [(48, -1), (130, 4), (130, 2), (130, 0)])
@pytest.mark.parametrize("N", [40, 64, 200, 272])
def test_b_is_a_column_slice(M, N, config):
    K, c0 = 384, 64
    rng = np.random.default_rng(M + N)
    a = rand_codes(rng, (M, K)); wide = rand_codes(rng, (K, c0 + (N + 15) // 16 * 16))
    acc = torch.empty((M, (N + 3) // 4 * 4), dtype=torch.int32, device=gu.DEV)
    binding.halo_gemm_i8_desc(binding.gemm_desc(gu.to_dev(a), gu.to_dev(wide)[:, c0:c0 + N], trans_b=False, acc_out=acc[:, :N],
                                                config=config))
    gu.assert_codes_equal(acc[:, :N], orc.gemm_codes(a, wide[:, c0:c0 + N]), "accumulators")


# Tiles of 256 and of 192 columns in one launch (two_widths): M, N, K and the columns in wide tiles with bf16 and with fp32 out, -1 where
# one width is taken.  All narrow and mixed; last narrow tiles of 32, 80, 144 and 192 columns; odd rows; odd, even and ragged units.
TWO_WIDTHS = [(1845, 11168, 1040, 0, -1), (1363, 7760, 2064, 0, -1), (2048, 14336, 1168, 8192, 8192), (1923, 13840, 656, 6400, -1),
              (1536, 8016, 1680, 0, 0)]


@pytest.mark.parametrize("M,N,K", [t[:3] for t in TWO_WIDTHS])
@pytest.mark.parametrize("pad", [0, 24])
def test_tiles_of_two_widths(M, N, K, pad):
    rng = np.random.default_rng(M + N)
    a, b = gu.to_dev(rand_codes(rng, (M, K))), gu.to_dev(rand_codes(rng, (N, K)))
    rs = gu.to_dev(rng.uniform(1e-3, 1e-2, M).astype(np.float32)); cs = gu.to_dev(rng.uniform(1e-3, 1e-2, N).astype(np.float32))
    acc = torch.full((M + 1, N + pad), -7, dtype=torch.int32, device=gu.DEV)
    outs = [torch.full((M + 1, N + pad), -7.0, dtype=dtype, device=gu.DEV) for dtype in (torch.float32, torch.bfloat16)]
    for out in outs:
        binding.halo_gemm_i8_desc(binding.gemm_desc(a, b, trans_b=True, row_scale=rs, col_scale=cs, out=out[:M, :N]))
    binding.halo_gemm_i8_desc(binding.gemm_desc(a, b, trans_b=True, acc_out=acc[:M, :N]))
    # sums of codes are integers below 2^31 and exact in float64
    want = torch.cat([(a[i:i + 512].double() @ b.double().T).to(torch.int32) for i in range(0, M, 512)])
    assert torch.equal(acc[:M, :N], want)
    assert torch.equal(outs[0][:M, :N], want.float() * rs[:, None] * cs[None, :])
    assert torch.equal(outs[1][:M, :N], outs[0][:M, :N].bfloat16())
    for out in outs + [acc]:
        assert bool((out[M:] == -7).all()) and bool((out[:, N:] == -7).all())


# The split-K kernel for small products (16, 32 or 64 rows of a tile by 64 columns, K dealt to four wavefronts in units of
# 128) and the first shape beyond it: fewer units than wavefronts, partial units, several trips, ragged rows and columns;
# sums, scaled outputs and the pair.
@pytest.mark.parametrize("M,N", sorted(SMALL_SHAPES))
@pytest.mark.parametrize("K", SMALL_K)
@pytest.mark.parametrize("trans_b", [True, False])
def test_small_products(M, N, K, trans_b):
    rng = np.random.default_rng(M + N + K)
    a = rand_codes(rng, (M, K)); b = rand_codes(rng, (N, K) if trans_b else (K, N))
    bd = torch.full((b.shape[0], (b.shape[1] + 15) // 16 * 16), 77, dtype=torch.int8, device=gu.DEV)
    bd[:, :b.shape[1]] = gu.to_dev(b)
    ad, bd = gu.to_dev(a), bd[:, :b.shape[1]]
    rs = rng.uniform(1e-3, 1e-2, M).astype(np.float32); cs = rng.uniform(1e-3, 1e-2, N).astype(np.float32)
    want = orc.gemm_codes(a, b.T if trans_b else b)
    pitch = (N + 3) // 4 * 4 + 16
    acc = torch.full((M + 1, pitch), -7, dtype=torch.int32, device=gu.DEV)
    binding.halo_gemm_i8_desc(binding.gemm_desc(ad, bd, trans_b=trans_b, acc_out=acc[:M, :N]))
    gu.assert_codes_equal(acc[:M, :N], want, "accumulators")
    assert bool((acc[M:] == -7).all()) and bool((acc[:, N:] == -7).all())
    out = torch.zeros((M, (N + 7) // 8 * 8), dtype=torch.float32, device=gu.DEV)
    y, _ = binding.halo_gemm_i8(ad, bd, trans_b=trans_b, row_scale=gu.to_dev(rs), col_scale=gu.to_dev(cs), out=out[:, :N])
    gu.assert_f32_identical(y, orc.dequantize(want, rs, cs), "scaled output")
    y, _ = binding.halo_gemm_i8(ad, bd, trans_b=trans_b, row_scale=gu.to_dev(rs), col_scale=gu.to_dev(cs),
                                out=out.bfloat16()[:, :N])
    gu.assert_bf16_within_one_ulp(y, orc.dequantize(want, rs, cs), "scaled bf16 output")
    if not trans_b:                                   # a pair of unequal products, as in the layer's backward pass
        g = rand_codes(rng, (N, 48)); gd = gu.to_dev(g)
        acc2 = torch.full((K, 48), -7, dtype=torch.int32, device=gu.DEV)
        left = torch.zeros((K, (N + 15) // 16 * 16), dtype=torch.int8, device=gu.DEV)
        left[:, :N] = gu.to_dev(b)
        acc.fill_(-7)
        binding.halo_gemm_i8_pair(binding.gemm_desc(ad, bd, trans_b=False, acc_out=acc[:M, :N]),
                                  binding.gemm_desc(left[:, :N // 16 * 16], gd[:N // 16 * 16], trans_b=False, acc_out=acc2))
        gu.assert_codes_equal(acc[:M, :N], want, "accumulators, first of a pair")
        gu.assert_codes_equal(acc2, orc.gemm_codes(b[:, :N // 16 * 16], g[:N // 16 * 16]), "accumulators, second of a pair")


# M, N of test_small_products_narrow_tiles and the columns of the tile that the rule takes (test_gemm_plan.py)
NARROW_SHAPES = {(1, 16): 16, (16, 4090): 16, (16, 4104): 32, (13, 8200): 64, (17, 2040): 16, (32, 4088): 16, (32, 4104): 32,
                 (100, 500): 16, (128, 2030): 32}
# M, N, K, pitch: tiles of 32 columns that start at different K (small kernel), one unit per wavefront and several, fewer than the
# ring's stages and more
ROUND_SHAPES = [(16, 8192, 8192, 8192), (13, 8100, 512, 8192), (32, 5100, 1536, 16384), (48, 4096, 6656, 8192), (128, 2030, 4608, 8192)]


# The small kernel's tiles of 16, 32 and 64 columns (as many as run at once), with ragged rows and columns, K shorter than the
# ring and longer than one trip through it, every output.
@pytest.mark.parametrize("M,N", sorted(NARROW_SHAPES))
@pytest.mark.parametrize("K", [16, 656, 4368])
def test_small_products_narrow_tiles(M, N, K):
    rng = np.random.default_rng(M + N + K)
    a = rand_codes(rng, (M, K)); b = rand_codes(rng, (N, K))
    rs = rng.uniform(1e-3, 1e-2, M).astype(np.float32); cs = rng.uniform(1e-3, 1e-2, N).astype(np.float32)
    ad, bd = gu.to_dev(a), gu.to_dev(b)
    want = orc.gemm_codes(a, b.T)
    pitch = (N + 7) // 8 * 8 + 16
    acc = torch.full((M + 1, pitch), -7, dtype=torch.int32, device=gu.DEV)
    binding.halo_gemm_i8_desc(binding.gemm_desc(ad, bd, trans_b=True, acc_out=acc[:M, :N]))
    gu.assert_codes_equal(acc[:M, :N], want, "accumulators")
    assert bool((acc[M:] == -7).all()) and bool((acc[:, N:] == -7).all())
    for dtype, check in ((torch.float32, gu.assert_f32_identical), (torch.bfloat16, gu.assert_bf16_within_one_ulp)):
        out = torch.full((M + 1, pitch), -7.0, dtype=dtype, device=gu.DEV)
        binding.halo_gemm_i8(ad, bd, trans_b=True, row_scale=gu.to_dev(rs), col_scale=gu.to_dev(cs), out=out[:M, :N])
        check(out[:M, :N], orc.dequantize(want, rs, cs), "scaled output")
        assert bool((out[M:] == -7).all()) and bool((out[:, N:] == -7).all())


@pytest.mark.parametrize("M,N,K,pitch", ROUND_SHAPES)
def test_small_products_that_go_round_k(M, N, K, pitch):
    rng = np.random.default_rng(M + N + K)
    a = rand_codes(rng, (M, K)); b = rand_codes(rng, (N, K))
    bd = torch.full((N, pitch), 77, dtype=torch.int8, device=gu.DEV)
    bd[:, :K] = gu.to_dev(b)
    acc = torch.full((M, (N + 3) // 4 * 4), -7, dtype=torch.int32, device=gu.DEV)
    binding.halo_gemm_i8_desc(binding.gemm_desc(gu.to_dev(a), bd[:, :K], trans_b=True, acc_out=acc[:, :N]))
    gu.assert_codes_equal(acc[:, :N], orc.gemm_codes(a, b.T), "accumulators")


# Every tile configuration on shapes its K step divides (ragged M and N, several trips through the ring), through
# halo_gemm_i8_desc: the configurations differ in speed only.
@pytest.mark.parametrize("name", sorted(binding.HALO_GEMM_CONFIGS))
@pytest.mark.parametrize("trans_b", [True, False])
def test_every_tile_configuration_gives_the_same_accumulators(name, trans_b):
    cfg = binding.HALO_GEMM_CONFIGS[name]
    rng = np.random.default_rng(cfg + 10 * int(trans_b))
    M, N, K = 600, 520, 1024 + (16 if name.startswith("staged") else 0)
    a = rand_codes(rng, (M, K))
    b = rand_codes(rng, (N, K) if trans_b else (K, N))
    ldb = (b.shape[1] + 15) // 16 * 16
    bd = torch.zeros((b.shape[0], ldb), dtype=torch.int8, device=gu.DEV)
    bd[:, :b.shape[1]] = gu.to_dev(b)
    acc = torch.full((M, N), -7, dtype=torch.int32, device=gu.DEV)
    binding.halo_gemm_i8_desc(binding.gemm_desc(gu.to_dev(a), bd[:, :b.shape[1]], trans_b=trans_b, acc_out=acc, config=cfg))
    gu.assert_codes_equal(acc, orc.gemm_codes(a, b.T if trans_b else b), "accumulators, configuration " + name)


def test_tile_configuration_argument_errors():
    a = torch.zeros((64, 80), dtype=torch.int8, device=gu.DEV)
    b = torch.zeros((64, 80), dtype=torch.int8, device=gu.DEV)
    acc = torch.zeros((64, 64), dtype=torch.int32, device=gu.DEV)
    with pytest.raises(binding.HaloError) as e:       # K = 80 is not a multiple of the 64-byte K step
        binding.halo_gemm_i8_desc(binding.gemm_desc(a, b, trans_b=True, acc_out=acc, config=0))
    assert e.value.status == binding.HALO_ESHAPE
    with pytest.raises(binding.HaloError) as e:
        binding.halo_gemm_i8_desc(binding.gemm_desc(a, b, trans_b=True, acc_out=acc, config=9))
    assert e.value.status == binding.HALO_EINVAL
    binding.halo_gemm_i8_desc(binding.gemm_desc(a, b, trans_b=True, acc_out=acc, config=4))


def rand_codes(rng, shape, extreme=False):
    if extreme:
        return rng.choice(np.array([-127, 127], dtype=np.int8), size=shape)
    return rng.integers(-127, 128, size=shape, dtype=np.int8)


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("trans_b", [True, False])
def test_gemm_accumulators_bit_exact(M, N, K, trans_b):
    rng = np.random.default_rng(M * 7 + N * 3 + K)
    a = rand_codes(rng, (M, K))
    b = rand_codes(rng, (N, K) if trans_b else (K, N))
    ldb = (b.shape[1] + 15) // 16 * 16
    bd = torch.zeros((b.shape[0], ldb), dtype=torch.int8, device=gu.DEV)
    bd[:, :b.shape[1]] = gu.to_dev(b)
    _, acc = binding.halo_gemm_i8(gu.to_dev(a), bd[:, :b.shape[1]], trans_b=trans_b, out_dtype=None, want_acc=True,
                                  acc_out=torch.full((M, (N + 3) // 4 * 4), -7, dtype=torch.int32, device=gu.DEV)[:, :N])
    want = orc.gemm_codes(a, b.T if trans_b else b)
    gu.assert_codes_equal(acc, want, "accumulators")


@pytest.mark.parametrize("trans_b", [True, False])
def test_gemm_extreme_codes_longest_k(trans_b):
    """All +-127 at K = 14336: the largest magnitude the layer can produce, no int32 overflow."""
    rng = np.random.default_rng(5)
    M, N, K = 96, 160, 14336
    a = rand_codes(rng, (M, K), extreme=True)
    b = rand_codes(rng, (N, K) if trans_b else (K, N), extreme=True)
    a[0] = 127
    if trans_b:
        b[0] = 127
    else:
        b[:, 0] = 127
    _, acc = binding.halo_gemm_i8(gu.to_dev(a), gu.to_dev(b), trans_b=trans_b, out_dtype=None, want_acc=True)
    want = orc.gemm_codes(a, b.T if trans_b else b)
    assert want[0, 0] == 127 * 127 * K
    gu.assert_codes_equal(acc, want, "accumulators")


@pytest.mark.parametrize("odt", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("trans_b", [True, False])
def test_gemm_scaled_epilogue(odt, trans_b):
    rng = np.random.default_rng(6)
    M, N, K = 200, 328, 512
    a = rand_codes(rng, (M, K)); b = rand_codes(rng, (N, K) if trans_b else (K, N))
    rs = (np.abs(rng.standard_normal(M)) * 1e-2 + 1e-4).astype(np.float32)
    cs = (np.abs(rng.standard_normal(N)) * 1e-3 + 1e-5).astype(np.float32)
    ldc = (N + 7) // 8 * 8
    out = torch.zeros((M, ldc), dtype=odt, device=gu.DEV)
    ldb = (b.shape[1] + 15) // 16 * 16
    bd = torch.zeros((b.shape[0], ldb), dtype=torch.int8, device=gu.DEV)
    bd[:, :b.shape[1]] = gu.to_dev(b)
    bd = bd[:, :b.shape[1]]
    c, acc = binding.halo_gemm_i8(gu.to_dev(a), bd, trans_b=trans_b, row_scale=gu.to_dev(rs),
                                  col_scale=gu.to_dev(cs), out=out[:, :N], want_acc=True)
    want_acc = orc.gemm_codes(a, b.T if trans_b else b)
    want = orc.dequantize(want_acc, rs, cs)
    gu.assert_codes_equal(acc, want_acc, "accumulators")
    if odt == torch.float32:
        gu.assert_f32_identical(c, want, "scaled output")
    else:
        gu.assert_bf16_within_one_ulp(c, want, "scaled bf16 output")
    # row scale only / no scales
    c2, _ = binding.halo_gemm_i8(gu.to_dev(a), bd, trans_b=trans_b, row_scale=gu.to_dev(rs))
    gu.assert_f32_identical(c2, orc.dequantize(want_acc, rs), "row-scaled output")


def test_gemm_k_zero_writes_zeros_and_empty_is_noop():
    a = torch.empty((8, 0), dtype=torch.int8, device=gu.DEV)
    b = torch.empty((8, 0), dtype=torch.int8, device=gu.DEV)
    c, acc = binding.halo_gemm_i8(a, b, trans_b=True, want_acc=True)
    assert not c.any() and not acc.any()
    a = torch.empty((0, 64), dtype=torch.int8, device=gu.DEV)
    b = torch.empty((16, 64), dtype=torch.int8, device=gu.DEV)
    c, _ = binding.halo_gemm_i8(a, b, trans_b=True)
    assert c.shape == (0, 16)


def test_gemm_pair_matches_two_single_launches():
    """Both backward products in one launch give the same bits as two launches (config c2's shapes scaled down,
    ragged edges, one scaled bf16 output and one raw accumulator output)."""
    rng = np.random.default_rng(9)
    b, m, n = 384, 512, 640
    Eq = rand_codes(rng, (b, n)); Wq = rand_codes(rng, (n, m)); EqT = rand_codes(rng, (n, b)); Xq = rand_codes(rng, (b, m))
    s_e = (np.abs(rng.standard_normal(b)) * 1e-3 + 1e-5).astype(np.float32)
    dEq, dWq, dEqT, dXq = map(gu.to_dev, (Eq, Wq, EqT, Xq))
    ex = torch.zeros((b, m), dtype=torch.bfloat16, device=gu.DEV)
    acc_g = torch.zeros((n, m), dtype=torch.int32, device=gu.DEV)
    g1 = binding.gemm_desc(dEq, dWq, trans_b=False, row_scale=gu.to_dev(s_e), out=ex)
    g2 = binding.gemm_desc(dEqT, dXq, trans_b=False, acc_out=acc_g)
    binding.halo_gemm_i8_pair(g1, g2)
    want_ex = orc.dequantize(orc.gemm_codes(Eq, Wq), s_e)
    gu.assert_bf16_within_one_ulp(ex, want_ex, "paired E_X")
    gu.assert_codes_equal(acc_g, orc.gemm_codes(EqT, Xq), "paired G accumulators")
    ex1, _ = binding.halo_gemm_i8(dEq, dWq, trans_b=False, row_scale=gu.to_dev(s_e), out_dtype=torch.bfloat16)
    assert torch.equal(ex.view(torch.int16), ex1.contiguous().view(torch.int16))
    # a pair the shared configuration cannot take (K-contiguous B, ragged K) still works
    a = rand_codes(rng, (70, 80)); bb = rand_codes(rng, (50, 80))
    acc1 = torch.zeros((70, 52), dtype=torch.int32, device=gu.DEV)[:, :50]
    acc2 = torch.zeros((n, m), dtype=torch.int32, device=gu.DEV)
    binding.halo_gemm_i8_pair(binding.gemm_desc(gu.to_dev(a), gu.to_dev(bb), trans_b=True, acc_out=acc1),
                              binding.gemm_desc(dEqT, dXq, trans_b=False, acc_out=acc2))
    gu.assert_codes_equal(acc1, orc.gemm_codes(a, bb.T), "fallback pair, first")
    gu.assert_codes_equal(acc2, orc.gemm_codes(EqT, Xq), "fallback pair, second")


# Full-size products of configs c2 and c3 in the tile configuration the library picks for them: the steady state of
# the global->LDS ring (64..224 trips) on the large macro tiles.  Each runs twice into separate buffers: same bits
# both times, and the oracle's bits.
FULL = [
    ("c2 forward", 2048, 4096, 4096, True),
    ("c3 forward", 4096, 4096, 14336, True),
    ("c2 E_X", 2048, 4096, 4096, False),
    ("c2 G", 4096, 4096, 2048, False),
    ("c3 E_X / G", 4096, 14336, 4096, False),
]


@pytest.mark.parametrize("what,M,N,K,trans_b", FULL, ids=[f[0] for f in FULL])
def test_gemm_full_size_accumulators_bit_exact_and_repeatable(what, M, N, K, trans_b):
    rng = np.random.default_rng(M + 3 * N + 7 * K + int(trans_b))
    a = rand_codes(rng, (M, K))
    b = rand_codes(rng, (N, K) if trans_b else (K, N))
    da, db = gu.to_dev(a), gu.to_dev(b)
    _, acc1 = binding.halo_gemm_i8(da, db, trans_b=trans_b, out_dtype=None, want_acc=True)
    _, acc2 = binding.halo_gemm_i8(da, db, trans_b=trans_b, out_dtype=None, want_acc=True)
    assert torch.equal(acc1, acc2), "two runs of the same product differ"
    del acc2
    gu.assert_codes_equal(acc1, orc.gemm_codes(a, b.T if trans_b else b), what + " accumulators")


@pytest.mark.parametrize("b,m,n", [(2048, 4096, 4096), (4096, 14336, 4096)], ids=["c2", "c3"])
def test_gemm_pair_full_size_bit_exact_and_repeatable(b, m, n):
    """The paired backward launch at the sizes of configs c2 and c3: E_X = Eq Wq and G = EqT Xq accumulators."""
    rng = np.random.default_rng(b + m + n)
    Eq = rand_codes(rng, (b, n)); Wq = rand_codes(rng, (n, m)); EqT = rand_codes(rng, (n, b)); Xq = rand_codes(rng, (b, m))
    dEq, dWq, dEqT, dXq = map(gu.to_dev, (Eq, Wq, EqT, Xq))
    accs = []
    for _ in range(2):
        ax = torch.empty((b, m), dtype=torch.int32, device=gu.DEV)
        ag = torch.empty((n, m), dtype=torch.int32, device=gu.DEV)
        binding.halo_gemm_i8_pair(binding.gemm_desc(dEq, dWq, trans_b=False, acc_out=ax),
                                  binding.gemm_desc(dEqT, dXq, trans_b=False, acc_out=ag))
        accs.append((ax, ag))
    assert torch.equal(accs[0][0], accs[1][0]) and torch.equal(accs[0][1], accs[1][1]), "two runs differ"
    ax, ag = accs[0]
    del accs
    gu.assert_codes_equal(ax, orc.gemm_codes(Eq, Wq), "paired E_X accumulators")
    gu.assert_codes_equal(ag, orc.gemm_codes(EqT, Xq), "paired G accumulators")

"""GPU parity: W4A4 GEMM / GEMV (offq_w4a4_gemm) and weight packing vs the oracle."""
import numpy as np
import pytest
import torch

import paper_2606_07116_amd as offq
from oracle import gemm as OG
from oracle import quantizer as OQ
from paper_2606_07116_amd import inputs
from tests import parity as P

pytestmark = pytest.mark.gpu


def _layer(M, N, K, g, seed, layout="concentrated", n_out=4):
    x = inputs.activations(M, K, seed=seed, n_outliers=n_out, lo=50, hi=200, layout=layout, g=g)
    w = inputs.weights(N, K, seed=seed)
    (q, s, z), (codes, scale, zero) = P.rotate_quantize_and_check(x, g, True)
    q_w, sw, cs, packed = P.oracle_weights(w, g)
    wc, ws, wcs = P.upload_weights(packed, sw, cs)
    y, acc = offq.offq_w4a4_gemm(codes, scale, zero, wc, ws, wcs, g, debug=True)
    y2, _ = offq.offq_w4a4_gemm(codes, scale, zero, wc, ws, wcs, g, debug=False)
    torch.cuda.synchronize()
    assert torch.equal(y, y2)
    acc_ref = OG.int_gemm_groups(q, q_w, g)
    acc_gpu = P.host(acc)
    if not np.array_equal(acc_gpu, acc_ref):
        bad = np.argwhere(acc_gpu != acc_ref)
        raise AssertionError(f"accumulator mismatch at {bad[:5].tolist()} (of {len(bad)})")
    P.check_output(P.host(y.float()), acc_ref, s, z, sw, cs)
    return y


@pytest.mark.parametrize("M,N,K,g", [
    (17, 8, 256, 256), (128, 128, 512, 512), (130, 136, 1024, 256), (200, 250, 256, 64),
    (257, 384, 2048, 512), (64, 512, 4096, 4096), (40, 96, 8192, 8192), (33, 64, 512, 128),
    # groups of 8 and 16 steps of 128 k; 32 groups; g = 512 over a ragged grid
    (100, 136, 4096, 1024), (77, 64, 8192, 2048), (40, 64, 4096, 128), (300, 260, 3584, 512),
    # many groups: of one, two, four and sixteen steps, an odd number of them
    (257, 200, 14336, 128), (300, 136, 8192, 256), (100, 520, 16384, 512),
    (33, 130, 3712, 128), (64, 96, 65536, 2048),
])
def test_gemm_shapes(M, N, K, g):
    _layer(M, N, K, g, seed=M * 7 + N)


@pytest.mark.parametrize("M,N,K", [(4096, 6144, 4096), (4000, 6100, 1024)])
def test_wide_tile_gemm_accumulators(M, N, K):
    """One group per row on 384 tiles of 256 x 256: the form that the MLP up/gate
    projection and the 8192-row projection run. Every accumulator bit-exact, once on
    whole tiles and once ragged in M and N."""
    _layer(M, N, K, K, seed=M + N)


@pytest.mark.parametrize("M,N,K,g", [
    (4096, 8192, 1024, 1024), (4000, 8104, 512, 512),      # one group: 512 tiles of 256 x 256
    (4000, 8100, 512, 512),                                # ragged in M and N, N not a multiple of 8
    (4096, 4096, 2048, 256), (4001, 4000, 1024, 512),      # groups: 512 tiles of 256 x 128
    (4096, 4100, 3584, 512), (3900, 4096, 8192, 2048),     # odd group count; 16 stages per group
])
def test_large_gemm_shapes(M, N, K, g):
    """Prefill-sized grids (at least 512 tiles, several tiles per CU): every
    accumulator bit-exact and the output within the bar, on whole and ragged
    tile grids, with one group per row, 2 to 8 groups, an odd number of groups
    and long groups."""
    _layer(M, N, K, g, seed=M + N + g)


def test_out_must_cover_the_output():
    """The GEMM writes M x N values at the output's row stride: a short or a
    transposed output is refused before any launch."""
    M, N, K, g = 32, 64, 256, 256
    codes = torch.zeros((M, K // 2), dtype=torch.uint8, device=P.DEV)
    sc = torch.ones((M, 1), dtype=torch.float16, device=P.DEV)
    zp = torch.zeros((M, 1), dtype=torch.int16, device=P.DEV)
    wc = torch.zeros(offq.weight_codes_shape(N, K), dtype=torch.uint8, device=P.DEV)
    ws = torch.ones(N, dtype=torch.float16, device=P.DEV)
    cs = torch.zeros((1, N), dtype=torch.int32, device=P.DEV)
    short = torch.empty((M - 1, N), dtype=torch.bfloat16, device=P.DEV)
    trans = torch.empty((N, M), dtype=torch.bfloat16, device=P.DEV).t()
    for bad in (short, trans):
        with pytest.raises(ValueError):
            offq.offq_w4a4_gemm(codes, sc, zp, wc, ws, cs, g, out=bad)


@pytest.mark.parametrize("M", [1, 2, 4, 5, 16])
@pytest.mark.parametrize("K,g", [(256, 256), (2048, 512), (8192, 8192), (1024, 64),
                                 (4096, 128), (1536, 512), (2048, 1024)])
def test_gemv_shapes(M, K, g):
    _layer(M, 200, K, g, seed=M + K)


@pytest.mark.parametrize("N", [16, 33, 1030, 5000, 9000, 16400])
def test_gemv_channel_counts(N):
    """Single and ragged 16-channel tiles; one, two and four tiles per wave
    (the last with a ragged final workgroup)."""
    _layer(3, N, 4096, 512, seed=N)


@pytest.mark.parametrize("M,N,K,g", [(4, 4096, 14336, 128), (16, 4096, 14336, 512),
                                     (1, 20000, 5120, 128), (3, 8192, 6144, 256),
                                     (5, 8192, 6144, 1024)])
def test_gemv_parts_of_k(M, N, K, g):
    """K not a multiple of 4096: each wave's part of K is an odd number of
    batches, and with g = 1024 a part ends inside a group (the group's
    zero-point term is added once)."""
    _layer(M, N, K, g, seed=K + g)


@pytest.mark.parametrize("M,N,K,g", [
    (17, 100, 4096, 128), (32, 1000, 1024, 512),           # 32 x 16 tiles
    (33, 4096, 640, 128), (64, 2040, 14336, 128),          # 32 x 32, fewer steps than waves; 112 groups
    (64, 6150, 512, 256), (65, 4100, 3072, 1024),          # 64 x 32; parts of K that end inside a group
    (32, 24580, 384, 128), (20, 24600, 1024, 1024),        # 32 x 64
    (250, 4100, 1152, 128), (100, 8200, 2048, 2048),       # 64 x 64 by eight waves
    (250, 4100, 896, 128), (1270, 1030, 128, 128),         # ... by four: short K
    (333, 4096, 1536, 512), (257, 6145, 768, 256),         # 64 x 64 by four waves
])
def test_few_token_rows(M, N, K, g):
    """17 to a few hundred token rows: small tiles whose waves split K, each
    tile shape at ragged edges, with one and several groups per wave's part
    and parts that end inside a group."""
    _layer(M, N, K, g, seed=M + N + K)


@pytest.mark.parametrize("M,N,K,g", [
    (641, 6150, 128, 128), (1100, 3000, 384, 128),         # g = 128, 128 x 128 tiles: one, three stages
    (1030, 4098, 640, 128), (513, 8200, 4096, 128),
    (4096, 4096, 256, 128), (4001, 4090, 640, 128),        # g = 128, 256 x 256 tiles
    (4000, 4000, 1024, 1024), (3841, 4090, 512, 512),      # one group, 256 x 256 tiles
    (1800, 5000, 2048, 2048), (2100, 3722, 8192, 8192),    # ... long: the largest sums
    (2040, 4090, 512, 512), (2040, 4090, 256, 256),        # one group, 256 x 128 tiles on i8
    (2039, 4090, 2048, 2048),
    (2001, 2090, 1280, 256), (1990, 2100, 1536, 512),      # 5, 3 groups in LDS
    (1990, 2100, 3072, 1024),
    (1500, 6150, 8192, 256), (1300, 6200, 7936, 256),      # 32 and 31 groups of 256, streamed
    (2051, 2053, 14848, 512), (2049, 2058, 29696, 1024),   # 29 groups of 512, of 1024, streamed
])
def test_large_tile_forms(M, N, K, g):
    """Each large-tile kernel at ragged edges, with the smallest and odd stage
    counts."""
    _layer(M, N, K, g, seed=M + N + K)


@pytest.mark.parametrize("M,N,K,g", [
    (1, 17, 128, 128), (9, 30, 256, 256),                  # 16 channels by one wave
    (3, 16390, 640, 128), (5, 1030, 640, 128),             # by two, by four
    (16, 1000, 1792, 256), (2, 6150, 8192, 2048),          # by eight
    (7, 1030, 8320, 128), (4, 5130, 5120, 1024),           # by sixteen
    (4, 16390, 1280, 128), (3, 16390, 16384, 8192),        # M <= 4, wide: by four; by eight on long rows
    (16, 6150, 4224, 128), (5, 16400, 16512, 128),         # 32 channels by sixteen; 129 groups
    (16, 6150, 1024, 512), (9, 16400, 4608, 512),          # 32 by eight
    (9, 28690, 4608, 512),                                 # 64 by eight
    (2, 16384, 8192, 8192),                                # weights read front to back
    (16, 6150, 20480, 512), (3, 6160, 20480, 128),         # long rows, 160 groups
    (5, 6150, 20480, 2048), (6, 10250, 16384, 512),
    (7, 6150, 4224, 128), (5, 16390, 4096, 1024), (9, 16390, 4608, 512),
    (4, 16390, 640, 128), (16, 16390, 1024, 512),
])
def test_decode_shapes(M, N, K, g):
    """One to sixteen token rows: each split of K and channel tile, ragged."""
    _layer(M, N, K, g, seed=M + N + K)


def test_raw_layout_and_spikes():
    _layer(150, 192, 1024, 1024, seed=5, layout="raw", n_out=6)


@pytest.mark.parametrize("M,N,ld,off", [
    (140, 72, 100, 10),   # GEMM
    (16, 72, 100, 10),    # decode GEMV, output start not 8-byte aligned
    (16, 70, 101, 3),     # GEMV: odd row stride, N not a multiple of 4
    (5, 66, 99, 1),
])
def test_output_row_stride(M, N, ld, off):
    """The output is a view inside a larger matrix: the M x N values land at
    its row stride and offset, nothing around them is written."""
    K, g = 512, 256
    x = inputs.activations(M, K, seed=3, n_outliers=2, lo=50, hi=60, layout="concentrated", g=g)
    w = inputs.weights(N, K, seed=3)
    (q, s, z), (codes, scale, zero) = P.rotate_quantize_and_check(x, g, True)
    q_w, sw, cs, packed = P.oracle_weights(w, g)
    wc, ws, wcs = P.upload_weights(packed, sw, cs)
    big = torch.full((M, ld), 7.0, dtype=torch.bfloat16, device=P.DEV)
    offq.offq_w4a4_gemm(codes, scale, zero, wc, ws, wcs, g, out=big[:, off:off + N])
    torch.cuda.synchronize()
    yb = P.host(big.float())
    assert np.all(yb[:, :off] == 7.0) and np.all(yb[:, off + N:] == 7.0)
    P.check_output(yb[:, off:off + N], OG.int_gemm_groups(q, q_w, g), s, z, sw, cs)


def test_extreme_codes_and_zero_points():
    """All-15 activation codes against all -8 weights with large zero-points."""
    M, N, K, g = 130, 66, 1024, 512
    codes = torch.full((M, K // 2), 0xFF, dtype=torch.uint8, device=P.DEV)
    scale = torch.full((M, K // g), 0.5, dtype=torch.float16, device=P.DEV)
    zero = torch.full((M, K // g), -32768, dtype=torch.int16, device=P.DEV)
    q_w = np.full((N, K), -8, np.int8)
    sw = np.full(N, 0.25, np.float16)
    cs = OQ.colsum(q_w, g)
    wc, ws, wcs = P.upload_weights(OQ.pack_nibbles(q_w), sw, cs)
    y, acc = offq.offq_w4a4_gemm(codes, scale, zero, wc, ws, wcs, g, debug=True)
    torch.cuda.synchronize()
    acc_ref = OG.int_gemm_groups(np.full((M, K), 15, np.uint8), q_w, g)
    assert np.array_equal(P.host(acc), acc_ref)
    P.check_output(P.host(y.float()), acc_ref, P.host(scale), P.host(zero), sw, cs)


# one shape for each large-tile form: 6-bit 128 x 128 and 256 x 256 at g = 128 and with
# one group, i8 with one group, groups in LDS and streamed; M and N leave remainders
LARGE_TILES = [(645, 6150, 256, 128), (4001, 4090, 256, 128), (3841, 4090, 512, 512),
               (2040, 4090, 512, 512), (1990, 2100, 1024, 512), (2049, 2053, 7424, 256)]


def _random_product(M, N, K, g, z):
    """Random codes of both operands with the zero-points z: GPU operands and the
    oracle's accumulators, scales and column sums."""
    rng = np.random.default_rng(M + N)
    q = rng.integers(0, 16, (M, K), dtype=np.uint8)
    q_w = rng.integers(-8, 8, (N, K), dtype=np.int8)
    s = rng.uniform(0.05, 0.5, (M, K // g)).astype(np.float16)
    sw = rng.uniform(0.01, 0.1, N).astype(np.float16)
    cs = OQ.colsum(q_w, g)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(P.DEV)
    ops = (up(OQ.pack_nibbles(q)), up(s), up(z)) + P.upload_weights(OQ.pack_nibbles(q_w), sw, cs)
    return ops, (OG.int_gemm_groups(q, q_w, g), s, z, sw, cs)


@pytest.mark.parametrize("M,N,K,g", LARGE_TILES)
def test_large_tile_output_row_stride(M, N, K, g):
    """A strided output view off 16-byte boundaries, whole tiles and ragged ones:
    nothing around it is written, and its values are those of a dense output."""
    z = np.random.default_rng(1).integers(-40, 40, (M, K // g)).astype(np.int16)
    ops, _ = _random_product(M, N, K, g, z)
    dense, _ = offq.offq_w4a4_gemm(*ops, g)
    for ld, off in ((N + 29, 3), (N + 6, 0)):
        big = torch.full((M, ld), 7.0, dtype=torch.bfloat16, device=P.DEV)
        offq.offq_w4a4_gemm(*ops, g, out=big[:, off:off + N])
        torch.cuda.synchronize()
        assert torch.equal(big[:, off:off + N], dense)
        assert bool((big[:, :off] == 7.0).all()) and bool((big[:, off + N:] == 7.0).all())


@pytest.mark.parametrize("M,N,K,g", LARGE_TILES + [(2100, 3722, 8192, 8192), (333, 1000, 2048, 128),
                                                   (9, 1000, 2048, 128), (9, 6150, 20480, 512)])
def test_large_zero_points(M, N, K, g):
    """Zero-points over the whole int16 range and at both its ends: |z colsum| up to
    2^25 in a group of 128 and far beyond with one group, so that a group's term and
    its products no longer fit 24 bits together. The bar of the other tests holds (with
    one group: a bf16 neighbour of the exact value)."""
    z = np.random.default_rng(2).integers(-32768, 32768, (M, K // g)).astype(np.int16)
    z[::3] = 32767
    z[1::3] = -32768
    ops, ref = _random_product(M, N, K, g, z)
    y, acc = offq.offq_w4a4_gemm(*ops, g, debug=True)
    torch.cuda.synchronize()
    assert np.array_equal(P.host(acc), ref[0])
    P.check_output(P.host(y.float()), *ref)


@pytest.mark.parametrize("M,N,K,g", LARGE_TILES + [(2100, 3722, 8192, 8192)])
def test_largest_sums(M, N, K, g):
    """All-15 activation codes against all -8 weights: the largest accumulators and
    column sums of every large-tile form, with the largest zero-points."""
    q = np.full((M, K), 15, np.uint8)
    q_w = np.full((N, K), -8, np.int8)
    z = np.where(np.arange(M) % 2, 32767, -32768).astype(np.int16)[:, None].repeat(K // g, 1)
    s = np.full((M, K // g), 0.5, np.float16)
    sw = np.full(N, 0.25, np.float16)
    cs = OQ.colsum(q_w, g)
    up = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to(P.DEV)
    y, acc = offq.offq_w4a4_gemm(up(OQ.pack_nibbles(q)), up(s), up(z),
                                 *P.upload_weights(OQ.pack_nibbles(q_w), sw, cs), g, debug=True)
    torch.cuda.synchronize()
    # every row and column alike: one column's sums stand for all
    acc_ref = OG.int_gemm_groups(q[:2], q_w[:2], g)
    assert np.all(P.host(acc) == acc_ref[0, 0, 0])
    y_ref = OG.epilogue(np.broadcast_to(acc_ref[:, :1, :1], (K // g, M, 2)), s, z, sw[:2], cs[:, :2])
    y = P.host(y.float()).astype(np.float64)
    assert np.all(np.abs(y - y_ref[:, :1]) <= OG.bf16_ulp(y_ref[:, :1]))


def test_empty_m_is_noop():
    g, K, N = 256, 256, 8
    e = torch.empty((0, K // 2), dtype=torch.uint8, device=P.DEV)
    y, _ = offq.offq_w4a4_gemm(e, torch.empty((0, 1), dtype=torch.float16, device=P.DEV),
                               torch.empty((0, 1), dtype=torch.int16, device=P.DEV),
                               torch.zeros(offq.weight_codes_shape(N, K), dtype=torch.uint8,
                                           device=P.DEV),
                               torch.ones(N, dtype=torch.float16, device=P.DEV),
                               torch.zeros((1, N), dtype=torch.int32, device=P.DEV), g)
    assert y.shape == (0, N)


@pytest.mark.parametrize("N,K,g", [(7, 256, 64), (300, 4096, 4096), (64, 28672, 512), (33, 8192, 8192)])
def test_pack_weights(N, K, g):
    w = inputs.weights(N, K, seed=N)
    w[0] = 0.0                      # all-zero row -> scale 1
    w[1, 5] = 3.0                   # one large weight
    q_w, sw, cs, packed = P.oracle_weights(w, g)
    wc, ws, wcs = offq.offq_pack_weights(torch.from_numpy(w).to(P.DEV), g)
    torch.cuda.synchronize()
    assert np.array_equal(P.fp16_bits(P.host(ws)), P.fp16_bits(sw))
    assert tuple(wc.shape) == offq.weight_codes_shape(N, K)
    assert np.array_equal(offq.row_major_weight_codes(P.host(wc), N, K), packed)
    # the padding rows and k of the blocked layout hold zero codes
    assert int(P.host(wc).astype(np.int64).sum()) == int(packed.astype(np.int64).sum())
    assert np.array_equal(P.host(wcs), cs)

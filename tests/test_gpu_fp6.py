"""GPU parity of the FP6 kernels: every work-group shape of the tile kernel and every wave count of the split
kernel, at the edges of their tiles, against the CPU oracle.  Integer accumulators and 4-bit codes must match bit
for bit; fp32 outputs within 1e-5 relative.  The skinny kernel (int8) the same way."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DEV = "cuda:0"
SHAPES = list(range(1, 10))
# the dispatch record of each: the tile kernel's blocks per wave, waves along the rows, along the columns; the split kernels'
# waves and, on half tiles, blocks of 16 columns
TILES = {1: (4, 4, 1), 2: (2, 2, 2), 3: (2, 1, 4), 4: (2, 4, 1), 5: (1, 2, 1), 6: (1, 1, 4), 14: (4, 8, 1), 15: (2, 2, 1)}
TILES_JOINED = {20: (4, 4, 1), 21: (2, 1, 4), 22: (2, 4, 1), 23: (4, 8, 1), 24: (2, 2, 1)}
SPLITS = {7: (4, 0, 0), 8: (8, 0, 0), 9: (16, 0, 0), 16: (4, 1, 0), 17: (8, 1, 0), 18: (4, 2, 0), 19: (8, 2, 0)}


@pytest.fixture(scope="module")
def rm():
    import paper_2111_00153_amd as m
    assert torch.cuda.is_available(), "these tests need the GPU"
    yield m
    m.rmsmp_debug_set_wave_split(0, 0, 0, 0)


def _ran(rm, shape):
    """The last launch was of the shape that was asked for."""
    kernel, numbers = rm.rmsmp_debug_last_dispatch()
    if shape in TILES_JOINED:
        assert (kernel, numbers[:3], numbers[3] & 4) == ("fp6_tile", TILES_JOINED[shape], 4)
    else:
        assert (kernel, numbers[:3]) == (("fp6_tile", TILES[shape]) if shape in TILES else ("fp6_split", SPLITS[shape]))


def _to_dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _check_outputs(rm, oracle, call, p, M, N, ref, acc, z, bias, relu, bits=4):
    """int32, fp32, 4-bit and GELU outputs of call(Y, epilogue) against the oracle's epilogue of acc."""
    rs = oracle.rowsum(ref["wint"])
    bias_d = None if bias is None else _to_dev(bias)
    acc_c, y, _ = oracle.epilogue(acc, rs, z, ref["rowscale"], 0.05, bias, relu)
    Y = torch.full((M, N), -777, dtype=torch.int32, device=DEV)
    call(Y, rm.make_epilogue(0.05, z, bits, None, False, rm.OUT_INT32))
    Yf = torch.full((M, N), np.nan, dtype=torch.float32, device=DEV)
    call(Yf, rm.make_epilogue(0.05, z, bits, bias_d, relu, rm.OUT_FP32))
    torch.cuda.synchronize()
    assert np.array_equal(Y.cpu().numpy(), acc_c)
    assert np.all(np.abs(Yf.cpu().numpy() - y) <= 1e-5 * np.abs(y))
    if M % 2:
        return
    pos = y[y > 0]
    inv = np.float32(15.0 / max(float(np.percentile(pos, 99.0)) if pos.size else 1.0, 1e-6))
    _, _, q = oracle.epilogue(acc, rs, z, ref["rowscale"], 0.05, bias, relu, inv)
    Yq = torch.full((N, M // 2), 0xEE, dtype=torch.uint8, device=DEV)
    call(Yq, rm.make_epilogue(0.05, z, bits, bias_d, relu, rm.OUT_U4, inv))
    torch.cuda.synchronize()
    got = rm.unpack_u4(Yq.cpu().numpy())
    assert np.array_equal(got, np.ascontiguousarray(q[p.perm].T))
    _, y, _ = oracle.epilogue(acc, rs, z, ref["rowscale"], 0.05, bias, False)
    inv = float(np.float32(14.0 / max(float(np.percentile(np.abs(y), 99.0)), 1e-6)))
    _, q = oracle.epilogue_gelu(acc, rs, z, ref["rowscale"], 0.05, bias, inv, 1)
    Yq = torch.full((N, M // 2), 0xEE, dtype=torch.uint8, device=DEV)
    call(Yq, rm.make_epilogue(0.05, z, bits, bias_d, False, rm.OUT_GELU_U4, inv, 1))
    torch.cuda.synchronize()
    got = rm.unpack_u4(Yq.cpu().numpy())
    assert np.array_equal(got, np.ascontiguousarray(q[p.perm].T))


# one column / row more and less than a tile, K from one block to several chunks, ragged K, all row classes
GEMMS = [(34, 64, 65, (35, 60, 5)), (64, 576, 256, (35, 60, 5)), (130, 130, 33, (60, 35, 5)), (256, 384, 129, (0, 0, 100)), (257, 1002, 31, (100, 0, 0)),
         (98, 1600, 257, (0, 100, 0))]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("M,K,N,ratio", GEMMS)
def test_gemm_every_work_group_shape(rm, oracle, shape, M, K, N, ratio):
    rng = np.random.default_rng(M + K + N)
    W = si.weights_rowscaled(rng, M, K)
    scheme = si.scheme_permutation(rng, rm.rmsmp_ratio_counts(M, *ratio))
    x = si.act_codes_u4(rng, (N, K))
    bias = rng.normal(0.0, 0.3, M).astype(np.float32) if shape % 2 else None
    ref = oracle.quantize_rows(W, scheme)
    acc = oracle.gemm_acc(ref["wint"], x.astype(np.int32))
    p = rm.rmsmp_pack_weights(W, scheme, flags=rm.PACK_POT_AS_INT8 if shape == 2 else 0)
    X = _to_dev(rm.pack_u4(x))

    def call(Y, ep):
        rm.rmsmp_gemm(p, X, N, ep, Y)
        _ran(rm, 1 if shape in TILES_JOINED and ep.out_kind == rm.OUT_GELU_U4 else shape)
    rm.rmsmp_debug_set_wave_split(0, shape, 0, 0)
    try:
        _check_outputs(rm, oracle, call, p, M, N, ref, acc, (3 * shape) % 16, bias, shape % 3 == 0)
    finally:
        rm.rmsmp_debug_set_wave_split(0, 0, 0, 0)
        p.free()


# the tile kernel's shapes beyond those: 512 x 128 and 128 x 64 outputs, more rows than eight pairs of tiles, rows that leave
# the last pair half empty, Fixed-8 tiles by themselves
@pytest.mark.parametrize("shape", [14, 15])
@pytest.mark.parametrize("M,K,N,ratio", GEMMS + [(520, 192, 130, (35, 60, 5)), (610, 768, 129, (0, 40, 60)), (1024, 130, 70, (50, 50, 0))])
def test_gemm_further_work_group_shapes(rm, oracle, shape, M, K, N, ratio):
    test_gemm_every_work_group_shape(rm, oracle, shape, M, K, N, ratio)


# ragged channel counts, strides, padding beyond the filter, non-square and even filters, images that straddle tiles
CONVS = [((2, 24, 13, 11, 3, 3, 1, 1), 144), ((3, 50, 12, 10, 3, 3, 2, 1), 70), ((1, 64, 15, 17, 3, 3, 1, 1), 64), ((2, 6, 9, 9, 5, 5, 2, 2), 40),
         ((1, 22, 8, 9, 2, 4, 3, 2), 64), ((5, 160, 7, 5, 1, 1, 2, 0), 34), ((4, 96, 5, 5, 3, 3, 1, 0), 130)]


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("geom,M", CONVS)
def test_conv_every_work_group_shape(rm, oracle, shape, geom, M):
    B, C, H, Wd, KH, KW, stride, pad = geom
    rng = np.random.default_rng(sum(geom) + M)
    K = C * KH * KW
    W = si.weights_rowscaled(rng, M, K)
    scheme = si.scheme_permutation(rng, rm.rmsmp_ratio_counts(M, 35, 60, 5))
    x = si.act_codes_u4(rng, (B, H, Wd, C))
    bias = rng.normal(0.0, 0.3, M).astype(np.float32) if shape % 2 else None
    od = oracle.conv_desc(B, C, H, Wd, KH, KW, stride, pad)
    OH, OW = oracle.conv_out_hw(od)
    N = B * OH * OW
    z = (5 * shape) % 16
    ref = oracle.quantize_rows(W, scheme)
    acc = oracle.conv_acc(ref["wint"].reshape(M, C, KH, KW), x.astype(np.int32), od, zpad=z)
    p = rm.rmsmp_pack_weights(W, scheme, taps=KH * KW)
    d = rm.ConvDesc(B, C, H, Wd, KH, KW, stride, pad)
    X = _to_dev(rm.pack_u4(x))
    need = rm.rmsmp_conv2d_workspace_size(p, d, 4)
    ws = torch.empty((need,), dtype=torch.uint8, device=DEV) if need else None

    def call(Y, ep):
        rm.rmsmp_conv2d(p, X, d, ep, Y, ws)
        _ran(rm, 1 if shape in TILES_JOINED and ep.out_kind == rm.OUT_GELU_U4 else shape)
    rm.rmsmp_debug_set_wave_split(0, shape, 0, 0)
    try:
        _check_outputs(rm, oracle, call, p, M, N, ref, acc, z, bias, shape % 3 == 0)
    finally:
        rm.rmsmp_debug_set_wave_split(0, 0, 0, 0)
        p.free()


@pytest.mark.parametrize("shape", [14, 15])
@pytest.mark.parametrize("geom,M", CONVS)
def test_conv_further_work_group_shapes(rm, oracle, shape, geom, M):
    test_conv_every_work_group_shape(rm, oracle, shape, geom, M)


# neighbouring tiles joined in a wave (Fixed-8 rows, no GELU output): waves of two tiles in one part, of one in two parts, of both, of a
# tile that is left over; a last row block that is not full, a last tile that is not
JOINED = [20, 21, 22, 23, 24]


@pytest.mark.parametrize("shape", JOINED)
@pytest.mark.parametrize("M,K,N,ratio", [(64, 576, 256, (35, 60, 5)), (50, 64, 65, (0, 0, 100)), (256, 384, 129, (60, 35, 5)), (246, 130, 133, (0, 60, 40)), (320, 1002, 31, (40, 50, 10)), (96, 192, 65, (35, 60, 5)), (18, 330, 40, (0, 0, 100)), (846, 130, 70, (0, 0, 100)),
                                         (576, 192, 257, (60, 35, 5)), (1088, 320, 140, (0, 40, 60))])
def test_gemm_joined_tiles(rm, oracle, shape, M, K, N, ratio):
    test_gemm_every_work_group_shape(rm, oracle, shape, M, K, N, ratio)


@pytest.mark.parametrize("shape", JOINED)
@pytest.mark.parametrize("geom,M", CONVS + [((2, 64, 15, 13, 3, 3, 1, 1), 256), ((2, 24, 13, 11, 3, 3, 1, 1), 312)])
def test_conv_joined_tiles(rm, oracle, shape, geom, M):
    test_conv_every_work_group_shape(rm, oracle, shape, geom, M)


@pytest.mark.parametrize("shape", JOINED)
@pytest.mark.parametrize("scheme_code", [2])
def test_mixed_sums_just_below_what_fp32_holds_joined_tiles(rm, oracle, scheme_code, shape):
    test_mixed_sums_just_below_what_fp32_holds(rm, oracle, scheme_code, shape)


# the split kernel on half tiles: 4 and 8 waves, 16 and 32 columns; rows that end in a tile's first half, fewer K steps than
# waves, Fixed-8 tiles by themselves
HALVES = [16, 17, 18, 19]


@pytest.mark.parametrize("shape", HALVES)
@pytest.mark.parametrize("M,K,N,ratio", GEMMS + [(8, 64, 65, (35, 60, 5)), (520, 192, 130, (35, 60, 5)), (104, 4096, 66, (40, 50, 10)), (56, 2050, 79, (0, 40, 60))])
def test_gemm_half_tiles(rm, oracle, shape, M, K, N, ratio):
    test_gemm_every_work_group_shape(rm, oracle, shape, M, K, N, ratio)


@pytest.mark.parametrize("shape", HALVES)
@pytest.mark.parametrize("geom,M", CONVS + [((1, 512, 7, 7, 3, 3, 1, 1), 72)])
def test_conv_half_tiles(rm, oracle, shape, geom, M):
    test_conv_every_work_group_shape(rm, oracle, shape, geom, M)


# the patch kernel: column blocks per wave, K split, waves along the columns, pairs of tiles
PATCHES = {32: (2, 1, 2, 2), 33: (2, 2, 1, 2), 34: (2, 4, 1, 2), 35: (4, 1, 4, 1), 36: (2, 1, 4, 1), 37: (4, 2, 1, 2), 38: (4, 4, 1, 1), 39: (4, 1, 1, 4), 40: (4, 2, 2, 2),
           41: (2, 2, 1, 4)}


# ragged channel counts, strides (odd sides too: the next image begins before the row's end), no padding, non-square, even and
# large filters, images that straddle work-groups, more K steps than waves share and fewer; tiles in one part, in two, left over of either kind
@pytest.mark.parametrize("shape", sorted(PATCHES))
@pytest.mark.parametrize("geom,M,ratio", [((2, 24, 13, 11, 3, 3, 1, 1), 144, (35, 60, 5)), ((3, 26, 12, 10, 3, 3, 2, 1), 70, (0, 100, 0)), ((3, 32, 13, 11, 3, 3, 2, 1), 128, (60, 35, 5)),
                                          ((2, 6, 9, 9, 5, 5, 2, 2), 40, (0, 40, 60)), ((1, 22, 11, 9, 2, 4, 3, 1), 64, (35, 60, 5)), ((9, 96, 5, 5, 3, 3, 1, 0), 226, (0, 0, 100)),
                                          ((1, 64, 15, 17, 3, 3, 1, 1), 64, (35, 60, 5)), ((2, 34, 9, 10, 5, 6, 1, 2), 290, (40, 50, 10)), ((1, 160, 24, 23, 3, 3, 1, 1), 64, (100, 0, 0))])
def test_conv_patch_kernel(rm, oracle, shape, geom, M, ratio):
    B, C, H, Wd, KH, KW, stride, pad = geom
    rng = np.random.default_rng(sum(geom) + M)
    W = si.weights_rowscaled(rng, M, C * KH * KW)
    scheme = si.scheme_permutation(rng, rm.rmsmp_ratio_counts(M, *ratio))
    x = si.act_codes_u4(rng, (B, H, Wd, C))
    bias = rng.normal(0.0, 0.3, M).astype(np.float32) if shape % 2 else None
    od = oracle.conv_desc(*geom)
    OH, OW = oracle.conv_out_hw(od)
    z = (5 * shape) % 16
    ref = oracle.quantize_rows(W, scheme)
    acc = oracle.conv_acc(ref["wint"].reshape(M, C, KH, KW), x.astype(np.int32), od, zpad=z)
    p = rm.rmsmp_pack_weights(W, scheme, taps=KH * KW)
    d = rm.ConvDesc(*geom)
    X = _to_dev(rm.pack_u4(x))
    need = rm.rmsmp_conv2d_workspace_size(p, d, 4)
    ws = torch.empty((need,), dtype=torch.uint8, device=DEV) if need else None

    def call(Y, ep):
        rm.rmsmp_conv2d(p, X, d, ep, Y, ws)
        if ep.out_kind != rm.OUT_GELU_U4:  # (which this kernel does not have)
            assert rm.rmsmp_debug_last_dispatch() == ("fp6_patch", PATCHES[shape])
    rm.rmsmp_debug_set_wave_split(0, shape, 0, 0)
    try:
        _check_outputs(rm, oracle, call, p, M, B * OH * OW, ref, acc, z, bias, shape % 3 == 0)
    finally:
        rm.rmsmp_debug_set_wave_split(0, 0, 0, 0)
        p.free()


# rows whose sums are just below 2^24, as test_mixed_sums_just_below_what_fp32_holds has for the kernels that take GEMMs: 5 x 6 filters, whose K is deep
# enough (for PoT rows as many channels as the shape's patch has room for: 256 columns reach 0.93 of the bound, 512 reach 0.49)
@pytest.mark.parametrize("shape", sorted(PATCHES))
@pytest.mark.parametrize("rows", ["pot4", "fixed8", "both"])
def test_sums_just_below_what_fp32_holds_patch_kernel(rm, oracle, rows, shape):
    """Tiles in one part, in two, one of each in a wave, one left over: the largest and the smallest level in one instruction,
    small products on top of a large sum, a large sum and back to nothing, odd sums, both signs; the partial sums of waves that share K."""
    tn, _, wn, _ = PATCHES[shape]
    cols = 32 * tn * wn
    C = 288 if rows != "pot4" else 592 if cols <= 128 else 544 if cols == 256 else 288
    B, H, Wd, KH, KW, M = 2, 7, 11, 5, 6, 66 if rows != "both" else 64
    K = C * KH * KW
    rng = np.random.default_rng(240 + shape)
    limit = ((1 << 24) - 1) // 15
    scheme = np.full(M, 1 if rows == "pot4" else 2, np.uint8)
    if rows == "both":  # (a tile of each)
        scheme[:32] = 1
    Q = np.zeros((M, K), np.int64)
    for r in range(M):
        pot = scheme[r] == 1
        levels = np.array([0] + [s * 2 ** e for s in (-1, 1) for e in range(7)]) if pot else np.arange(-127, 128)
        q = np.full(K, 64 if pot else 127)
        kind = r % 32
        if kind == 1:
            q[::16] = 1
        elif kind == 2:
            q[::16] = -1
        elif kind == 3:
            q[K // 2:] *= -1
        elif kind == 4:
            q = -q
            q[1::32] = 1
        elif kind == 5:
            q[K - K // 8:] = 1
        elif kind == 6:
            q[: K // 8] = 1
        elif kind > 6:
            q = rng.choice(levels, K)
        h = (q + 8) >> 4
        cost = np.abs(q) if pot else 16 * np.abs(h) + np.abs(q - 16 * h)  # what the operands hold of a level
        q[np.cumsum(cost) > limit] = 0
        Q[r] = q
    W = (Q / np.where(scheme == 1, 64.0, 127.0)[:, None]).astype(np.float32)
    alpha = np.ones(M, np.float32)
    ref = oracle.quantize_rows(W, scheme, alpha=alpha)
    assert np.array_equal(ref["wint"], Q)
    x = si.act_codes_u4(rng, (B, H, Wd, C))
    x[0] = 15
    x[0, :, -1, 1::2] = 14
    od = oracle.conv_desc(B, C, H, Wd, KH, KW, 1, 2)
    OH, OW = oracle.conv_out_hw(od)
    acc = oracle.conv_acc(ref["wint"].reshape(M, C, KH, KW), x.astype(np.int32), od, zpad=0)
    reach = 0.98 if rows != "pot4" or cols <= 128 else 0.92 if cols == 256 else 0.49
    assert reach * (1 << 24) < int(np.abs(acc).max()) < 1 << 24 and (acc % 2).any()
    p = rm.rmsmp_pack_weights(W, scheme, alpha=alpha, taps=KH * KW)
    d = rm.ConvDesc(B, C, H, Wd, KH, KW, 1, 2)
    need = rm.rmsmp_conv2d_workspace_size(p, d, 4)
    ws = torch.empty((need,), dtype=torch.uint8, device=DEV) if need else None
    Y = torch.full((M, B * OH * OW), -777, dtype=torch.int32, device=DEV)
    rm.rmsmp_debug_set_wave_split(0, shape, 0, 0)
    try:
        rm.rmsmp_conv2d(p, _to_dev(rm.pack_u4(x)), d, rm.make_epilogue(0.05, 0, 4, None, False, rm.OUT_INT32), Y, ws)
        assert rm.rmsmp_debug_last_dispatch() == ("fp6_patch", PATCHES[shape])
    finally:
        rm.rmsmp_debug_set_wave_split(0, 0, 0, 0)
    torch.cuda.synchronize()
    assert np.array_equal(Y.cpu().numpy(), acc)
    p.free()


@pytest.mark.parametrize("shape", HALVES)
@pytest.mark.parametrize("scheme_code", [1, 2])
def test_mixed_sums_just_below_what_fp32_holds_half_tiles(rm, oracle, scheme_code, shape):
    test_mixed_sums_just_below_what_fp32_holds(rm, oracle, scheme_code, shape)


def test_scales_beyond_the_tile_kernels_multipliers(rm, oracle):
    """The tile kernel's multipliers are 32 times rowscale * act_scale: a scale that would take those to infinity goes to
    other kernels, with the same results as ever."""
    M, K, N = 64, 128, 130
    rng = np.random.default_rng(9)
    W = si.weights_rowscaled(rng, M, K)
    scheme = si.scheme_permutation(rng, rm.rmsmp_ratio_counts(M, 35, 60, 5))
    x = si.act_codes_u4(rng, (N, K))
    ref = oracle.quantize_rows(W, scheme)
    acc = oracle.gemm_acc(ref["wint"], x.astype(np.int32))
    p = rm.rmsmp_pack_weights(W, scheme)
    X = _to_dev(rm.pack_u4(x))
    top = float(np.abs(ref["rowscale"]).max())
    for scale, tiles in ((0.5e36 / top, True), (3e36 / top, False)):
        rm.rmsmp_debug_set_wave_split(0, 1, 0, 0)
        try:
            Y = torch.empty((M, N), dtype=torch.float32, device=DEV)
            rm.rmsmp_gemm(p, X, N, rm.make_epilogue(scale, 0, 4, None, False, rm.OUT_FP32), Y)
            assert (rm.rmsmp_debug_last_dispatch()[0] == "fp6_tile") == tiles
        finally:
            rm.rmsmp_debug_set_wave_split(0, 0, 0, 0)
        torch.cuda.synchronize()
        with np.errstate(over="ignore"):
            _, y, _ = oracle.epilogue(acc, oracle.rowsum(ref["wint"]), 0, ref["rowscale"], scale)
        got = Y.cpu().numpy()
        finite = np.isfinite(y)
        assert np.array_equal(got[~finite], y[~finite]) and np.all(np.abs(got[finite] - y[finite]) <= 1e-5 * np.abs(y[finite]))
    p.free()


# scales that cut the line of y into bins of one break point each, and scales that do not (many codes within 0.01, or break
# points far out on the falling branch)
@pytest.mark.parametrize("shape", [1, 4, 5, 15])
@pytest.mark.parametrize("s_out,z_out", [(0.18, 1), (0.18, 15), (0.05, 4), (1.0, 0), (0.011, 14), (1e-3, 7), (1e-4, 15), (40.0, 3)])
def test_gelu_codes_around_every_break_point(rm, oracle, shape, s_out, z_out):
    """Rows whose pre-activation is a break point of the code, its neighbours on the fp32 line, and the ends of that line."""
    inv = float(np.float32(1.0 / s_out))
    b = rm.rmsmp_debug_gelu_breakpoints(inv, z_out)
    at = np.array([v for v in [*b["rise"], *b["fall"], b["y_split"], 0.0, -0.0] if np.isfinite(v)], np.float32)
    y = np.concatenate([at, np.nextafter(at, np.float32(np.inf)), np.nextafter(at, np.float32(-np.inf)),
                        np.array([1e30, -1e30, 3e38, -3e38, 5.0, -5.0], np.float32)]).astype(np.float32)
    M, K, N = y.size + y.size % 2, 128, 33
    bias = np.zeros(M, np.float32)
    bias[:y.size] = y
    rng = np.random.default_rng(3)
    W, scheme = si.weights_rowscaled(rng, M, K), si.scheme_permutation(rng, rm.rmsmp_ratio_counts(M, 35, 60, 5))
    x = np.zeros((N, K), np.uint8)  # y is the bias
    ref = oracle.quantize_rows(W, scheme)
    _, q = oracle.epilogue_gelu(oracle.gemm_acc(ref["wint"], x.astype(np.int32)), oracle.rowsum(ref["wint"]), 0, ref["rowscale"], 0.05, bias, inv, z_out)
    p = rm.rmsmp_pack_weights(W, scheme)
    Y = torch.full((N, M // 2), 0xEE, dtype=torch.uint8, device=DEV)
    bias_d = _to_dev(bias)
    rm.rmsmp_debug_set_wave_split(0, shape, 0, 0)
    try:
        rm.rmsmp_gemm(p, _to_dev(rm.pack_u4(x)), N, rm.make_epilogue(0.05, 0, 4, bias_d, False, rm.OUT_GELU_U4, inv, z_out), Y)
        _ran(rm, shape)
    finally:
        rm.rmsmp_debug_set_wave_split(0, 0, 0, 0)
    torch.cuda.synchronize()
    assert np.array_equal(rm.unpack_u4(Y.cpu().numpy()), np.ascontiguousarray(q[p.perm].T))
    p.free()


# convolutions that the FP6 kernels decline where they lie (a tensor below 16 bytes, a side of 65536 and more): the
# lowered matrix has rows of the padded K, which is not taps * channels
LOWERED = [((1, 24, 1, 1, 3, 3, 1, 1), 66), ((1, 12, 1, 1, 3, 3, 1, 1), 34), ((1, 6, 2, 2, 2, 2, 1, 0), 64), ((1, 6, 1, 4, 1, 2, 1, 0), 40),
           ((1, 24, 1, 70000, 1, 9, 200, 0), 34)]


@pytest.mark.parametrize("geom,M", LOWERED)
def test_lowered_matrix_with_padded_columns(rm, oracle, geom, M):
    B, C, H, Wd, KH, KW, stride, pad = geom
    rng = np.random.default_rng(sum(geom) + M)
    K = C * KH * KW
    W = si.weights_rowscaled(rng, M, K)
    scheme = si.scheme_permutation(rng, rm.rmsmp_ratio_counts(M, 35, 60, 5))
    x = si.act_codes_u4(rng, (B, H, Wd, C))
    bias = rng.normal(0.0, 0.3, M).astype(np.float32)
    od = oracle.conv_desc(B, C, H, Wd, KH, KW, stride, pad)
    OH, OW = oracle.conv_out_hw(od)
    N, z = B * OH * OW, 5
    ref = oracle.quantize_rows(W, scheme)
    acc = oracle.conv_acc(ref["wint"].reshape(M, C, KH, KW), x.astype(np.int32), od, zpad=z)
    p = rm.rmsmp_pack_weights(W, scheme, taps=KH * KW)
    d = rm.ConvDesc(B, C, H, Wd, KH, KW, stride, pad)
    X = _to_dev(rm.pack_u4(x))
    ws = torch.empty((rm.rmsmp_conv2d_workspace_size(p, d, 4),), dtype=torch.uint8, device=DEV)
    _check_outputs(rm, oracle, lambda Y, ep: rm.rmsmp_conv2d(p, X, d, ep, Y, ws), p, M, N, ref, acc, z, bias, False)
    p.free()


# every column block and a column more and less, K steps that the waves do not share evenly, tiles cut off by the last
# row, a layer of more than 128 tiles, all row classes
SKINNY = [(34, 512, 1, (35, 60, 5)), (70, 576, 16, (35, 60, 5)), (64, 1088, 17, (100, 0, 0)), (98, 2112, 32, (0, 100, 0)), (33, 640, 33, (0, 0, 100)),
          (130, 1216, 48, (60, 35, 5)), (40, 4160, 64, (35, 60, 5)), (4130, 576, 49, (40, 50, 10)), (4130, 1088, 20, (40, 50, 10))]


@pytest.mark.parametrize("shape", [0, 10, 11, 12, 13])
@pytest.mark.parametrize("M,K,N,ratio", SKINNY)
def test_skinny_every_work_group_shape(rm, oracle, shape, M, K, N, ratio):
    rng = np.random.default_rng(M + K + N)
    W = si.weights_rowscaled(rng, M, K)
    scheme = si.scheme_permutation(rng, rm.rmsmp_ratio_counts(M, *ratio))
    x = si.act_codes_u4(rng, (N, K))
    bias = rng.normal(0.0, 0.3, M).astype(np.float32) if shape % 2 else None
    ref = oracle.quantize_rows(W, scheme)
    acc = oracle.gemm_acc(ref["wint"], x.astype(np.int32))
    p = rm.rmsmp_pack_weights(W, scheme, flags=rm.PACK_POT_AS_INT8 if shape == 12 else 0)
    X = _to_dev(rm.pack_u4(x))
    rm.rmsmp_debug_set_wave_split(0, shape, 0, 0)
    try:
        _check_outputs(rm, oracle, lambda Y, ep: rm.rmsmp_gemm(p, X, N, ep, Y), p, M, N, ref, acc, (3 * shape) % 16, bias, shape % 3 == 0)
        assert rm.rmsmp_debug_last_dispatch()[0] == "skinny"
    finally:
        rm.rmsmp_debug_set_wave_split(0, 0, 0, 0)
        p.free()


# 8-bit activations: the split kernel on int8 instructions with 8 and 16 waves, columns of 16 bytes and not, K steps that the
# waves do not share evenly, all row classes
@pytest.mark.parametrize("M,K,N,ratio,waves", [(34, 147, 33, (35, 60, 5), 8), (64, 512, 1, (0, 0, 100), 8), (130, 2050, 40, (60, 35, 5), 16),
                                               (1000, 512, 64, (0, 0, 100), 8), (70, 4112, 65, (35, 60, 5), 16), (96, 64, 320, (100, 0, 0), 8)])
def test_int8_split(rm, oracle, M, K, N, ratio, waves):
    rng = np.random.default_rng(M + K + N)
    W = si.weights_rowscaled(rng, M, K)
    scheme = si.scheme_permutation(rng, rm.rmsmp_ratio_counts(M, *ratio))
    x = si.act_codes_i8(rng, (N, K))
    bias = rng.normal(0.0, 0.3, M).astype(np.float32)
    ref = oracle.quantize_rows(W, scheme)
    acc = oracle.gemm_acc(ref["wint"], x.astype(np.int32))
    p = rm.rmsmp_pack_weights(W, scheme)
    X = _to_dev(x)
    _check_outputs(rm, oracle, lambda Y, ep: rm.rmsmp_gemm(p, X, N, ep, Y), p, M, N, ref, acc, -3, bias, True, 8)
    assert rm.rmsmp_debug_last_dispatch() == ("int8_split", (waves, 0, 0, 0 if K % 16 == 0 else 2))
    p.free()


@pytest.mark.parametrize("N", [8, 100, 300])
def test_a_bias_that_is_no_number_gives_code_15(rm, N):
    """Through the skinny, the split and the tile kernel as through the others: the upper clamp is what a NaN ends at."""
    M, K = 64, 512
    rng = np.random.default_rng(3)
    p = rm.rmsmp_pack_weights(si.weights_rowscaled(rng, M, K), np.ones(M, np.uint8))
    bias = torch.zeros(M, device=DEV)
    bias[5] = float("nan")
    Y = torch.empty((N, M // 2), dtype=torch.uint8, device=DEV)
    for shape in ([0] if N <= 64 else [2, 8]):
        rm.rmsmp_debug_set_wave_split(0, shape, 0, 0)
        rm.rmsmp_gemm(p, _to_dev(rm.pack_u4(si.act_codes_u4(rng, (N, K)))), N, rm.make_epilogue(0.05, 0, 4, bias, False, rm.OUT_U4, 1.0), Y)
        rm.rmsmp_debug_set_wave_split(0, 0, 0, 0)
        torch.cuda.synchronize()
        assert np.all(rm.unpack_u4(Y.cpu().numpy())[:, int(np.flatnonzero(p.perm == 5)[0])] == 15)
    p.free()


@pytest.mark.parametrize("shape", [1, 4, 6, 8, 9])
@pytest.mark.parametrize("scheme_code", [1, 2])
def test_mixed_sums_just_below_what_fp32_holds(rm, oracle, scheme_code, shape):
    """Rows whose weights are as large as a layer of the FP6 kernels may have: 15 times the sum of what the operands
    hold of a level is just below 2^24.  The largest and the smallest level in one instruction, large sums that small
    products are added to and large ones taken from, odd sums, both signs: every sum exact."""
    M, N = 34, 70
    rng = np.random.default_rng(24 + scheme_code)
    levels = np.array([0] + [s * 2 ** e for s in (-1, 1) for e in range(7)]) if scheme_code == 1 else np.arange(-127, 128)

    def cost(q):  # of a level q: |q|, or |16 h| + |l| of its two parts
        h = (q + 8) >> 4
        return np.abs(q) if scheme_code == 1 else 16 * np.abs(h) + np.abs(q - 16 * h)

    limit = ((1 << 24) - 1) // 15
    top = int(levels.max())
    K = 2 * (limit // int(cost(np.array([top, 1])).sum()))
    Q = np.zeros((M, K), np.int64)
    Q[0, 0::2], Q[0, 1::2] = top, 1                        # largest and smallest level by turns
    Q[1, : K // 2], Q[1, K // 2:] = top, 1                 # small products on top of a large sum
    Q[2, : K // 2], Q[2, K // 2:] = 1, top
    Q[3, 0::2], Q[3, 1::2] = top, -1
    Q[4, : K // 2: 2], Q[4, K // 2:: 2] = top, -top        # a large sum, then back to nothing
    Q[5] = -Q[0]
    Q[6, : K // 2] = -Q[1, : K // 2]
    for r in range(7, M):                                  # any levels, as many as the row may have
        q = rng.choice(levels, K)
        q[np.cumsum(cost(q)) > limit] = 0
        Q[r] = rng.permutation(q) if r % 2 else q
    assert cost(Q).sum(axis=1).max() <= limit and cost(Q[0]).sum() > 0.999 * limit
    W = (Q / float(top)).astype(np.float32)
    scheme, alpha = np.full(M, scheme_code, np.uint8), np.ones(M, np.float32)
    ref = oracle.quantize_rows(W, scheme, alpha=alpha)
    assert np.array_equal(ref["wint"], Q)
    x = si.act_codes_u4(rng, (N, K))
    x[:8] = 15
    x[4, -1] = 14
    x[5, ::2] = 1
    x[6, 1::2] = 1
    p = rm.rmsmp_pack_weights(W, scheme, alpha=alpha)
    rm.rmsmp_debug_set_wave_split(0, shape, 0, 0)
    try:
        Y = torch.full((M, N), -777, dtype=torch.int32, device=DEV)
        rm.rmsmp_gemm(p, _to_dev(rm.pack_u4(x)), N, rm.make_epilogue(0.05, 0, 4, None, False, rm.OUT_INT32), Y)
        _ran(rm, shape)
    finally:
        rm.rmsmp_debug_set_wave_split(0, 0, 0, 0)
    torch.cuda.synchronize()
    acc = oracle.gemm_acc(ref["wint"], x.astype(np.int32))
    # (127 is 128 - 1 in two parts: its sums end 1.5 % below those of the parts)
    assert int(np.abs(acc).max()) > 0.98 * (1 << 24) and (acc % 2).any()
    assert np.array_equal(Y.cpu().numpy(), acc)
    p.free()


def _pack_and_bytes(rm, W, scheme, flags):
    """The packed layer and the device memory it took."""
    torch.cuda.synchronize()
    before = torch.cuda.mem_get_info()[0]
    p = rm.rmsmp_pack_weights(W, scheme, flags=flags)
    torch.cuda.synchronize()
    return p, before - torch.cuda.mem_get_info()[0]


# a layer with all row classes whose rows are below the bound by their K, and one whose rows are beyond it
@pytest.mark.parametrize("M,K,beyond", [(4096, 2048, False), (2048, 17536, True)])
def test_device_memory_of_the_operand_form(rm, oracle, M, K, beyond):
    """The second copy of the weights is kept where calls can use it and the caller wants it, and nowhere else; the
    results do not depend on it."""
    N = 70
    rng = np.random.default_rng(9)
    slack = 8 << 20  # what an allocation may be rounded up by, and tables
    if beyond:
        W, scheme = np.full((M, K), 0.5, np.float32), np.ones(M, np.uint8)
        x = np.full((N, K), 15, np.uint8)
        x[3, :5] = 0
        blob, operand = M * K // 2, M * K * 3 // 4
    else:
        W, scheme = si.weights_rowscaled(rng, M, K), si.scheme_permutation(rng, rm.rmsmp_ratio_counts(M, 40, 50, 10))
        x = si.act_codes_u4(rng, (N, K))
        blob, operand = M * K * 55 // 100, M * K * 3 // 4 * 11 // 10
    rows = slice(0, M, 97)
    ref = oracle.quantize_rows(W[rows], scheme[rows])
    acc = oracle.gemm_acc(ref["wint"], x.astype(np.int32))
    X = _to_dev(rm.pack_u4(x))
    for flags in (0, rm.PACK_NO_OPERAND_FORM):
        p, took = _pack_and_bytes(rm, W, scheme, flags)
        want = blob + (operand if flags == 0 and not beyond else 0)
        assert want * 0.95 - slack // 4 <= took <= want * 1.05 + slack, (took, want)
        Y = torch.full((M, N), -777, dtype=torch.int32, device=DEV)
        rm.rmsmp_gemm(p, X, N, rm.make_epilogue(0.05, 0, 4, None, False, rm.OUT_INT32), Y)
        kernel = rm.rmsmp_debug_last_dispatch()[0]
        assert (kernel in ("fp6_split", "fp6_tile")) == (flags == 0 and not beyond), kernel
        torch.cuda.synchronize()
        assert np.array_equal(Y[rows].cpu().numpy(), acc)
        p.free()
    p = rm.rmsmp_pack_weights(W[:64], scheme[:64], flags=rm.PACK_NO_OPERAND_FORM | rm.PACK_POT_AS_INT8)
    p.free()


@pytest.mark.parametrize("scheme_code,K", [(1, 17536), (2, 8832), (1, 17472), (2, 8768)])
def test_rows_beyond_what_fp32_sums_hold_use_the_int8_kernels(rm, oracle, scheme_code, K):
    """Every weight at its row's maximum and every code 15: from a K on the sums pass 2^24 and the layer must not run
    through the FP6 kernels; just below it must still be exact."""
    M, N = 34, 70
    W = np.full((M, K), 0.5, np.float32)
    W[1] = -0.25
    scheme = np.full(M, scheme_code, np.uint8)
    ref = oracle.quantize_rows(W, scheme)
    x = np.full((N, K), 15, np.uint8)
    x[3, :5] = 0
    p = rm.rmsmp_pack_weights(W, scheme)
    Y = torch.full((M, N), -777, dtype=torch.int32, device=DEV)
    rm.rmsmp_gemm(p, _to_dev(rm.pack_u4(x)), N, rm.make_epilogue(0.05, 0, 4, None, False, rm.OUT_INT32), Y)
    torch.cuda.synchronize()
    assert np.array_equal(Y.cpu().numpy(), oracle.gemm_acc(ref["wint"], x.astype(np.int32)))
    p.free()

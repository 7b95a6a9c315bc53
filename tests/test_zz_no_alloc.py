"""rmsmp_conv2d_static_workspace (the entry point for callers that cannot allocate) against
rmsmp_conv2d with a caller workspace: same int32 accumulators, fp32 outputs and 4-bit codes, on two
calls in a row, the second with a smaller input; a layer too large for the static buffer is refused."""
import numpy as np
import pytest

import synth_inputs as si

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

DEV = "cuda:0"


@pytest.fixture(scope="module")
def rm():
    import paper_2111_00153_amd as m
    assert torch.cuda.is_available(), "these tests need the GPU"
    return m


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to(DEV)


def _both_ways(rm, B, C, H, M, k, stride, pad, seed, lowered):
    """All three output kinds of one layer through both entry points; returns the workspace size.  lowered: whether the
    matrix is to be found in the caller's workspace afterwards."""
    rng = np.random.default_rng(seed)
    K = C * k * k
    W = si.weights_rowscaled(rng, M, K)
    scheme = si.scheme_permutation(rng, rm.rmsmp_ratio_counts(M, 35, 60, 5))
    x = si.act_codes_u4(rng, (B, H, H, C))
    bias = _dev(rng.normal(0.0, 0.3, M).astype(np.float32))
    p = rm.rmsmp_pack_weights(W, scheme, taps=k * k)
    d = rm.ConvDesc(B, C, H, H, k, k, stride, pad)
    OH = (H + 2 * pad - k) // stride + 1
    N = B * OH * OH
    X = _dev(rm.pack_u4(x))
    need = rm.rmsmp_conv2d_workspace_size(p, d, 4)
    ws = torch.empty(max(need, 1), dtype=torch.uint8, device=DEV)
    for kind, shape, dtype in ((rm.OUT_INT32, (M, N), torch.int32), (rm.OUT_FP32, (M, N), torch.float32),
                               (rm.OUT_U4, (N, M // 2), torch.uint8)):
        ep = rm.make_epilogue(0.05, 3, 4, None if kind == rm.OUT_INT32 else bias, kind != rm.OUT_INT32, kind, 1.7)
        Ya = torch.zeros(shape, dtype=dtype, device=DEV)
        Yb = torch.ones(shape, dtype=dtype, device=DEV)
        ws.fill_(0xA5)
        rm.rmsmp_conv2d(p, X, d, ep, Ya, ws if need else None)
        rm.rmsmp_conv2d_static_workspace(p, X, d, ep, Yb)
        torch.cuda.synchronize()
        assert torch.equal(Ya, Yb), (kind, B, C, H)
        assert bool((ws != 0xA5).any()) == lowered
    p.free()
    return need


# 0: the library's choice, which reads such a layer where it lies; 1 and 2: the int8 kernels, the general kernel
@pytest.mark.parametrize("kernels", [0, 1, 2])
def test_static_workspace_matches_caller_workspace_twice(rm, kernels):
    rm.rmsmp_init()
    rm.rmsmp_debug_set_wave_split(0, 0, kernels, 0)
    try:
        # 24 input channels: not a multiple of 16, so the lowered matrix goes through the workspace
        big = _both_ways(rm, 3, 24, 20, 96, 3, 1, 1, 1, kernels != 0)
        assert 0 < big <= rm.STATIC_WORKSPACE_BYTES
        small = _both_ways(rm, 1, 24, 9, 96, 3, 2, 1, 2, kernels != 0)
        assert 0 < small < big
        # a layer that needs no workspace passes straight through
        assert _both_ways(rm, 2, 64, 10, 64, 3, 1, 1, 3, False) == 0
    finally:
        rm.rmsmp_debug_set_wave_split(0, 0, 0, 0)


def test_static_workspace_refuses_what_does_not_fit(rm):
    rng = np.random.default_rng(4)
    C, M, H, B = 24, 32, 56, 64
    W = si.weights_rowscaled(rng, M, C * 9)
    p = rm.rmsmp_pack_weights(W, np.zeros(M, np.uint8), taps=9)
    d = rm.ConvDesc(B, C, H, H, 3, 3, 1, 1)
    assert rm.rmsmp_conv2d_workspace_size(p, d, 4) > rm.STATIC_WORKSPACE_BYTES
    X = torch.zeros((B, H, H, C // 2), dtype=torch.uint8, device=DEV)
    Y = torch.zeros((M, B * H * H), dtype=torch.int32, device=DEV)
    with pytest.raises(rm.RmsmpError) as e:
        rm.rmsmp_conv2d_static_workspace(p, X, d, rm.make_epilogue(0.05, 0, 4, None, False, rm.OUT_INT32), Y)
    assert e.value.code == 6
    p.free()

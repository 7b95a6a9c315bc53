"""GPU parity of the training-side kernels (weight projection forward, straight-through backward)
against the oracle: fp32 outputs are compared bit for bit -- both sides use the same op order."""
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


@pytest.mark.parametrize("M,K", [(64, 576), (37, 130), (3, 1), (256, 2304), (5, 4099), (1000, 512), (6, 8192), (3, 8196), (9, 12)])
@pytest.mark.parametrize("with_alpha", [False, True])
def test_fake_quant_rows_matches_oracle_bitwise(rm, oracle, M, K, with_alpha):
    rng = np.random.default_rng(M * 31 + K)
    W = si.weights_rowscaled(rng, M, K)
    W[rng.integers(0, M)] = 0.0  # an all-zero row
    # values on rounding boundaries of both quantizers
    W[0, : min(K, 4)] = (np.abs(W[0]).max() * np.array([0.5, 2.0 ** -0.5, 2.0 ** -7, 1.5 / 7])[: min(K, 4)]).astype(np.float32)
    scheme = si.scheme_permutation(rng, oracle.ratio_counts(M, 35, 60, 5))
    alpha = (np.abs(W).max(axis=1) * 0.7 + 1e-3).astype(np.float32) if with_alpha else None
    ref, a_ref = oracle.project_rows_f32(W, scheme, alpha)
    Wd, out = _dev(W), torch.full((M, K), float("nan"), dtype=torch.float32, device=DEV)
    a_out = torch.empty(M, dtype=torch.float32, device=DEV)
    rm.rmsmp_fake_quant_rows(Wd, _dev(scheme), out, None if alpha is None else _dev(alpha), a_out)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.array_equal(got.view(np.uint32) & 0x7fffffff, ref.view(np.uint32) & 0x7fffffff)  # magnitudes, bit for bit
    assert np.array_equal(got, ref)  # and signs wherever the value is not zero
    assert np.array_equal(a_out.cpu().numpy(), a_ref)


# the largest and smallest rows of each way a row is held, 16-byte aligned and not, and scaling factors at and beyond the
# ends of the range in which the quotient is corrected instead of divided
# (the backward of rows that are no multiple of 16 bytes reads them 16 bytes at a time from 2^22 elements on: short rows, of which
# a work-group has many, rows of 2^k + 1 and 2^k - 1, a last read that ends with the tensor and one that does not)
ROWS = ([(M, K) for M in (3, 1026) for K in (1, 64, 65, 255, 256, 257, 1024, 1025, 1028, 2048, 2049, 4096, 4100, 8191, 8192, 8193)] +
        [(3, 32768), (3, 32772), (1024, 8196), (1026, 12292), (1024, 16384), (1024, 16388), (32515, 129), (8209, 513), (4099, 1023), (16383, 257), (129, 32771)])


@pytest.mark.parametrize("M,K", ROWS)
def test_projection_and_its_backward_at_every_row_length(rm, oracle, M, K):
    rng = np.random.default_rng(M + K)
    W = si.weights_rowscaled(rng, M, K)
    W[0] *= np.float32(2.0 ** 64)
    W[1] *= np.float32(2.0 ** -70)
    scheme = rng.integers(0, 3, M).astype(np.uint8)
    G = rng.normal(0.0, 1.0, (M, K)).astype(np.float32)
    Wd, Gd, out, dW, a_out = _dev(W), _dev(G), torch.empty((M, K), device=DEV), torch.empty((M, K), device=DEV), torch.empty(M, device=DEV)
    for alpha in (None, (np.abs(W).max(axis=1) * np.float32(0.7)).astype(np.float32)):
        ref, a_ref = oracle.project_rows_f32(W, scheme, alpha)
        ad = None if alpha is None else _dev(alpha)
        rm.rmsmp_fake_quant_rows(Wd, _dev(scheme), out, ad, a_out)
        rm.rmsmp_ste_backward(Gd, dW, None if ad is None else Wd, ad)
        torch.cuda.synchronize()
        assert np.array_equal(out.cpu().numpy(), ref)
        assert np.array_equal(a_out.cpu().numpy(), a_ref)
        assert np.array_equal(dW.cpu().numpy(), G if alpha is None else np.where(np.abs(W) > alpha[:, None], np.float32(0), G))


# rows enough for one or two waves a row: the first and last length of each way, numbers of rows that leave a work-group half empty
@pytest.mark.parametrize("M,K", [(1280, 260), (1281, 1024), (1281, 1028), (1283, 2048), (1281, 257), (1281, 512), (1283, 513), (2049, 1023), (2049, 510), (4096, 516), (4097, 768),
                                 (4097, 772), (4097, 129), (4099, 255), (4097, 257), (4101, 511), (8191, 1028), (8192, 1028), (8193, 2048)])
def test_projection_and_its_backward_of_many_rows(rm, oracle, M, K):
    test_projection_and_its_backward_at_every_row_length(rm, oracle, M, K)


def test_fake_quant_equals_what_the_packed_path_multiplies_with(rm, oracle):
    """The projected fp32 weight is rowscale * the integer the packed blob holds."""
    rng = np.random.default_rng(9)
    M, K = 96, 320
    W = si.weights_rowscaled(rng, M, K)
    scheme = si.scheme_permutation(rng, oracle.ratio_counts(M, 35, 60, 5))
    out = torch.empty((M, K), dtype=torch.float32, device=DEV)
    rm.rmsmp_fake_quant_rows(_dev(W), _dev(scheme), out)
    torch.cuda.synchronize()
    p = rm.rmsmp_pack_weights(W, scheme)
    wint = rm.rmsmp_unpack_codes(p).astype(np.float32)
    assert np.array_equal(out.cpu().numpy(), p.rowscale[:, None] * wint)
    p.free()


@pytest.mark.parametrize("M,K", [(64, 576), (37, 131), (5, 4099)])
def test_ste_backward_matches_oracle(rm, oracle, M, K):
    rng = np.random.default_rng(M + K)
    W = si.weights_rowscaled(rng, M, K)
    g = rng.standard_normal((M, K)).astype(np.float32)
    gd, out = _dev(g), torch.full((M, K), float("nan"), dtype=torch.float32, device=DEV)
    rm.rmsmp_ste_backward(gd, out)
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), oracle.ste_backward(W, g))
    alpha = (np.abs(W).max(axis=1) * 0.5).astype(np.float32)
    rm.rmsmp_ste_backward(gd, out, _dev(W), _dev(alpha))
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), oracle.ste_backward(W, g, alpha))


def test_qat_entry_points_reject_bad_arguments(rm):
    out = torch.empty((4, 8), dtype=torch.float32, device=DEV)
    with pytest.raises(rm.RmsmpError) as e:
        rm.rmsmp_ste_backward(out, out, None, torch.ones(4, device=DEV))  # alpha without W
    assert e.value.code == 1

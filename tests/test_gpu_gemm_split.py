"""The split-operand fp32 GEMM (soap_gemm_f32) against fp64 products: tile and
slab edges, every layout, operands at 4-byte alignment, operands whose
bfloat16 parts leave bfloat16's range, and long sums of one sign.

Tolerance.  The parts represent an operand exactly, the dropped partial
products are below 3 x 2^-27 of the product, and a sum of K products takes
ceil(K / 32) roundings of the accumulator plus the twelve matrix-instruction
additions of each slab, which cut off (up to 2^-23 of the slab's sum each,
observed far below): relative to sum |a||b| the error is at most
(ceil(K / 32) + 12) 2^-23, and for operands of random sign relative to the
result's norm about its square root; four times that is allowed.
"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def soap():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2607_20548_amd as soap
    soap.lib()
    return soap


def bound(K):
    return 4.0 * 2.0 ** -24 * np.sqrt(-(-K // 32) + 12)


def operand(rows, cols, pad, shift, seed, scale=1.0):
    """A rows x cols view with leading dimension cols + pad whose first element
    lies `shift` floats after a 16-byte boundary: (tensor, pointer, ld, fp64)."""
    import torch
    ld = cols + pad
    h = np.random.default_rng(seed).standard_normal((rows, ld)).astype(np.float32) * np.float32(scale)
    buf = torch.zeros(rows * ld + shift, device="cuda")
    buf[shift:] = torch.from_numpy(h.reshape(-1)).cuda()
    return buf, buf.data_ptr() + 4 * shift, ld, h[:, :cols].astype(np.float64)


@pytest.mark.parametrize("ta", [0, 1])
@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M,N,K,pad,shift", [
    (1, 1, 1, 0, 0), (2, 3, 5, 1, 1), (127, 129, 31, 0, 0), (128, 128, 32, 0, 0),
    (129, 127, 33, 0, 3), (130, 2, 64, 2, 2), (1, 257, 65, 0, 0), (255, 1, 100, 3, 1),
    (132, 260, 96, 4, 0), (64, 512, 2049, 0, 0),
    # more than 192 tiles of 128: the large tile
    (1801, 2051, 65, 1, 1), (2050, 1796, 96, 0, 0), (1920, 1665, 33, 0, 2),
])
def test_layouts_edges_and_alignment(soap, ta, tb, M, N, K, pad, shift):
    import torch
    A, pa, lda, ah = operand(*((K, M) if ta else (M, K)), pad, shift, 1)
    B, pb, ldb, bh = operand(*((N, K) if tb else (K, N)), pad, shift, 2)
    C, pc, ldc, ch = operand(M, N, pad, shift, 3)
    keep = C.clone()
    soap.soap_gemm_f32(ta, tb, M, N, K, -0.5, pa, lda, pb, ldb, 2.0, pc, ldc)
    torch.cuda.synchronize()
    got = C[shift:].view(M, ldc)
    want = -0.5 * (ah.T if ta else ah) @ (bh.T if tb else bh) + 2.0 * ch
    err = np.linalg.norm(got[:, :N].cpu().numpy().astype(np.float64) - want) / np.linalg.norm(want)
    assert err <= bound(K), err
    assert torch.equal(C[:shift], keep[:shift])                       # nothing outside C
    assert torch.equal(got[:, N:], keep[shift:].view(M, ldc)[:, N:])


@pytest.mark.parametrize("scale", [1e-30, 1e-34, 1e-37])
def test_tiny_operands(soap, scale):
    """Every element of one operand tiny, the other of order one."""
    import torch
    A, pa, lda, ah = operand(140, 96, 0, 0, 1, scale)
    B, pb, ldb, bh = operand(96, 130, 0, 0, 2)
    C = torch.empty(140, 130, device="cuda")
    soap.soap_gemm_f32(0, 0, 140, 130, 96, 1.0, pa, lda, pb, ldb, 0.0, C, 130)
    want = ah @ bh
    got = C.cpu().numpy().astype(np.float64)
    assert np.linalg.norm(got - want) / np.linalg.norm(want) <= bound(96)


@pytest.mark.parametrize("ta", [0, 1])
@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M,N,K", [(140, 130, 96), (1801, 2051, 65)])
def test_small_operands_beside_ordinary_ones(soap, ta, tb, M, N, K):
    """Rows of A from 1 down to fp32's subnormals, columns of B from 1 up to
    1e20, all in the same tiles: every element of the product is as exact as
    one of ordinary operands (relative to its own sum of |a||b|; a result
    below fp32's normal range may also be rounded to its last bit)."""
    import torch
    rng = np.random.default_rng(4)
    rows = np.array([1.0, 1e-36, 1e-30, 1e-38, 1e-41])[np.arange(M) % 5]
    cols = np.array([1.0, 1e10, 1e20])[np.arange(N) % 3]
    a = (rng.standard_normal((M, K)) * rows[:, None]).astype(np.float32)
    b = (rng.standard_normal((K, N)) * cols[None, :]).astype(np.float32)
    A = torch.from_numpy(np.ascontiguousarray(a.T if ta else a)).cuda()
    B = torch.from_numpy(np.ascontiguousarray(b.T if tb else b)).cuda()
    C = torch.empty(M, N, device="cuda")
    soap.soap_gemm_f32(ta, tb, M, N, K, 1.0, A, A.shape[1], B, B.shape[1], 0.0, C, N)
    a64, b64 = a.astype(np.float64), b.astype(np.float64)
    err = np.abs(C.cpu().numpy().astype(np.float64) - a64 @ b64)
    limit = (-(-K // 32) + 12) * 2.0 ** -23 * (np.abs(a64) @ np.abs(b64)) + 2.0 ** -149
    assert (err <= limit).all(), float((err / limit).max())


@pytest.mark.parametrize("ta", [0, 1])
@pytest.mark.parametrize("tb", [0, 1])
@pytest.mark.parametrize("M,N,K,shift", [(140, 130, 77, 1), (1, 3, 2, 0), (65, 64, 96, 0),
                                         (1801, 2051, 65, 3), (2048, 1792, 48, 0)])
def test_sums_past_the_scaled_range(soap, ta, tb, M, N, K, shift):
    """Sums near 1e30 and 1e36 (finite, but not when scaled) are taken on the
    fp32 instructions: every layout, whole and ragged groups of k."""
    import torch
    for scale in (1e15, 1e18):
        A, pa, lda, ah = operand(*((K, M) if ta else (M, K)), 0, shift, 1, scale)
        B, pb, ldb, bh = operand(*((N, K) if tb else (K, N)), 0, shift, 2, scale)
        C = torch.empty(M, N, device="cuda")
        soap.soap_gemm_f32(ta, tb, M, N, K, 1.0, pa, lda, pb, ldb, 0.0, C, N)
        want = (ah.T if ta else ah) @ (bh.T if tb else bh)
        got = C.cpu().numpy().astype(np.float64)
        # fp32 accumulation in order: sqrt(K) roundings of 2^-24, four times that
        assert np.linalg.norm(got - want) / np.linalg.norm(want) <= 4 * 2.0 ** -24 * K ** 0.5


def test_infinite_and_huge_operands(soap):
    """An infinity reaches its own row only, as an infinity; an operand that
    rounds past the largest bfloat16 stays finite."""
    import torch
    A, pa, lda, _ = operand(200, 64, 0, 0, 1)
    A.view(200, 64)[5, 7] = float("inf")
    A.view(200, 64)[150, 3] = 3.4e38
    B = torch.full((64, 140), 0.25, device="cuda")
    C = torch.empty(200, 140, device="cuda")
    soap.soap_gemm_f32(0, 0, 200, 140, 64, 1.0, pa, lda, B, 140, 0.0, C, 140)
    assert torch.isinf(C[5]).all() and (C[5] > 0).all()
    rest = torch.cat([C[:5], C[6:]])
    assert torch.isfinite(rest).all()
    assert abs(float(C[150, 0]) / (0.25 * 3.4e38) - 1) <= bound(64)


def test_long_sums_of_one_sign(soap):
    """K = 6144 products of one sign: each slab's sum is rounded into the
    accumulator once, so that the error stays below an eighth of the bound
    (K / 32 + 12) 2^-24 (a sixtieth of the K / 2 x 2^-24 that accumulating in
    order may lose)."""
    import torch
    K = 6144
    A = torch.rand(128, K, device="cuda") + 0.5
    B = torch.rand(128, K, device="cuda") + 0.5
    C = torch.empty(128, 128, device="cuda")
    soap.soap_gemm_f32(0, 1, 128, 128, K, 1.0, A, K, B, K, 0.0, C, 128)
    want = A.double() @ B.double().mT
    err = float(((C.double() - want) / want).abs().max())
    assert err <= (K // 32 + 12) * 2.0 ** -24 / 8, err

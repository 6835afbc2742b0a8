"""GPU parity of split reductions: the chunk sums of the GEMMs (both carriers) and of
the convolution weight gradient, added by split_reduce_kernel.

The shapes take every form of the reduction: few and many outputs, few and many
chunks, output counts that are not multiples of 4 (or of a workgroup's share), each
written to a 16-byte and to a 4-byte aligned buffer.  The GEMMs are compared bit for
bit with the fp32 epilogue applied to the exact integer sums of random codes
(float64 products, exact below 2^53); the two carriers split the same reduction into
different chunks.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import announce, host, epilogue_replica  # noqa: E402


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2112_10769_amd as lib
    return lib


def _codes(shape, values, gen):
    """Random codes of the given nibbles: packed bytes."""
    nib = torch.tensor(values, dtype=torch.uint8, device="cuda")[
        torch.randint(len(values), shape, device="cuda", generator=gen)]
    return (nib[:, 0::2] | (nib[:, 1::2] << 4)).contiguous()


def _decode(codes, table):
    nib = torch.stack([codes & 15, codes >> 4], dim=2).flatten(1).long()
    return torch.tensor(table, dtype=torch.float64, device="cuda")[nib]


LUQ = [0.0] + [2.0 ** (e - 1) for e in range(1, 8)] + [0.0] + [-2.0 ** (e - 1) for e in range(1, 8)]
INT4 = [float(q if q < 8 else q - 16) for q in range(16)]


@pytest.mark.parametrize("M,N,K", [
    (3, 5, 40000),        # 15 outputs
    (8, 8, 4096),         # 64 outputs, few chunks
    (64, 16, 131072),
    (37, 99, 65536),      # 3663 outputs, not a multiple of 4
    (130, 264, 16416),
    (300, 200, 33024),
    (512, 260, 65536),
    (725, 724, 20000),    # just past 2^19 outputs
    (1023, 515, 32800),   # past 2^19, not a multiple of 4
    (1040, 1040, 49152),
])
def test_gemm_split_sums(L, M, N, K):
    announce("split reduce", M, N, K)
    gen = torch.Generator(device="cuda").manual_seed(M * N + K)
    a = _codes((M, K), [n for n in range(16) if n != 8], gen)
    b = _codes((N, K), [n for n in range(16) if n != 8], gen)
    alpha = torch.full((1,), 0.0123, device="cuda")
    scale = torch.full((1,), 0.37, device="cuda")
    acc = host(_decode(a, LUQ) @ _decode(b, INT4).t().contiguous())
    want = epilogue_replica(np.rint(acc).astype(np.int64), host(alpha)[0], 1, host(scale)[0])
    for ns in (1, L.CARRIER_FP6 | 1):
        for skip in (0, 1):   # outputs skipped at the front of the buffer
            buf = torch.full((M * N + 8,), float("nan"), device="cuda")
            L.luq_gemm_dgrad(a, alpha, b, scale, True, M, N, K, n_samples=ns, dx=buf[skip:skip + M * N])
            got = host(buf)
            assert np.array_equal(got[skip:skip + M * N].reshape(M, N), want), (ns, skip)
            assert np.isnan(got[:skip]).all() and np.isnan(got[skip + M * N:]).all(), "wrote outside the output"


@pytest.mark.parametrize("B,H,W,C,Cout", [
    (64, 56, 56, 64, 64),      # 64 ranges, 36864 outputs
    (32, 14, 14, 256, 256),    # few ranges, 589824 outputs
    (32, 13, 13, 3, 32),       # general form, 864 outputs
    (32, 5, 5, 1, 1),          # 9 outputs
])
def test_conv_wgrad_split_sums_unaligned_output(L, B, H, W, C, Cout):
    announce("split reduce conv", B, H, W, C, Cout)
    gen = torch.Generator(device="cuda").manual_seed(B * H + C)
    T, n = B * H * W, Cout * 9 * C
    g = _codes((Cout, T), [i for i in range(16) if i != 8], gen)
    a = _codes((C, T), [i for i in range(16) if i != 8], gen)
    alpha = torch.full((1,), 0.0123, device="cuda")
    scale = torch.full((1,), 0.37, device="cuda")
    whole = torch.empty(n, device="cuda")
    L.luq_conv3x3_wgrad(g, alpha, a, scale, True, B, H, W, C, Cout, dw=whole)
    buf = torch.full((n + 8,), float("nan"), device="cuda")
    L.luq_conv3x3_wgrad(g, alpha, a, scale, True, B, H, W, C, Cout, dw=buf[1:1 + n])
    got = host(buf)
    assert np.array_equal(got[1:1 + n], host(whole))
    assert np.isnan(got[:1]).all() and np.isnan(got[1 + n:]).all(), "wrote outside the output"

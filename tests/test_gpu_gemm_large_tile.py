"""GPU parity of the 256 x 256 GEMM tile (eight waves, the INT4 operand read
straight into registers) through the C ABI.

LARGE holds shapes that the planner gives that tile (tests/test_gemm_plan_cpu.py
checks it without a GPU): ragged M and N, K a multiple of 128 (whole stages) and not
(a partly filled last stage).  Every A operand kind (LUQ, two SMP planes, the int8 SMP
sums, signed and unsigned INT4) runs on them with both INT4 signednesses of B, on
random codes; outputs are compared bit for bit with the fp32 epilogue applied to the
exact integer sums (float64 products, exact below 2^53).  Further large shapes, some of
them on the 128 x 256 tile, are compared with the oracle through the quantizers.  The
largest codes at the longest unsplit reduction (K = 2^18) and one stage past
it (a split reduction) check the int32 bound and the sign handling against
the closed form.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

import synth  # noqa: E402
from test_gpu_parity import _gemm_case, _wgrad_case, _fwd_case  # noqa: E402
from test_gpu_smp_sum import _dgrad_sum_case  # noqa: E402
from test_gpu_split_reduce import INT4, LUQ, _codes, _decode  # noqa: E402
from gpu_util import announce, host, epilogue_replica  # noqa: E402

LARGE = [(4096, 4096, 2048), (4090, 4052, 2080)]
UNSIGNED = [float(q) for q in range(16)]


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2112_10769_amd as lib
    return lib


@pytest.mark.parametrize("M,N,K", LARGE)
@pytest.mark.parametrize("bsig", [True, False])
@pytest.mark.parametrize("kind", ["luq", "planes", "sums", "int4", "uint4"])
def test_large_tile_operands(L, M, N, K, bsig, kind):
    announce("large tile operands", M, N, K, bsig, kind)
    gen = torch.Generator(device="cuda").manual_seed(M + N + K)
    every = list(range(16))
    luq = [n for n in every if n != 8]
    b = _codes((N, K), every if not bsig else luq, gen)
    B = _decode(b, INT4 if bsig else UNSIGNED).t().contiguous()
    alpha, scale = torch.full((1,), 0.0123, device="cuda"), torch.full((1,), 0.37, device="cuda")
    if kind in ("int4", "uint4"):
        a = _codes((M, K), luq if kind == "int4" else every, gen)
        A = _decode(a, INT4 if kind == "int4" else UNSIGNED)
        got = L.int4_gemm_fwd(a, alpha, kind == "int4", b, scale, bsig, M, N, K)
    elif kind == "sums":
        a = torch.randint(-64, 65, (M, K), device="cuda", generator=gen, dtype=torch.int8)
        A = a.double()
        got = L.luq_gemm_dgrad(a, alpha, b, scale, bsig, M, N, K, n_samples=L.SMP_SUM | 2)
    elif kind == "planes":
        low = [n for n in luq if n & 7 != 7]                    # two planes: levels up to 2^5
        planes = [_codes((M, K), low, gen) for _ in range(2)]
        a = torch.zeros(2 * L.plane_bytes(M * K), dtype=torch.uint8, device="cuda")
        for i, p in enumerate(planes):
            a[i * L.plane_bytes(M * K):][:p.numel()] = p.flatten()
        A = _decode(planes[0], LUQ) + _decode(planes[1], LUQ)
        got = L.luq_gemm_dgrad(a, alpha, b, scale, bsig, M, N, K, n_samples=2)
    else:
        a = _codes((M, K), luq, gen)
        A = _decode(a, LUQ)
        got = L.luq_gemm_dgrad(a, alpha, b, scale, bsig, M, N, K)
    acc = np.rint(host(A @ B)).astype(np.int64)
    ns = 2 if kind in ("sums", "planes") else 1
    assert np.array_equal(host(got), epilogue_replica(acc, host(alpha)[0], ns, host(scale)[0]))


@pytest.mark.parametrize("ns", [1, 2])
def test_large_tile_dgrad_ragged(L, ns):
    _gemm_case(L, 4100, 4104, 1056, ns, True, seed=17 + ns)


def test_large_tile_dgrad_whole_stages_unsigned(L):
    _gemm_case(L, 4096, 4096, 1024, 1, False, seed=23)


def test_large_tile_dgrad_smp_sum(L):
    _dgrad_sum_case(L, 4100, 4104, 1056, True, seed=29)


@pytest.mark.parametrize("signed", [False, True])
def test_large_tile_wgrad(L, signed):
    _wgrad_case(L, 1056, 4104, 4120, 1, signed=signed, seed=31)


@pytest.mark.parametrize("xsig,wsig", [(True, True), (False, True), (True, False), (False, False)])
def test_large_tile_fwd(L, xsig, wsig):
    _fwd_case(L, 4100, 4104, 1056, xsig, wsig, seed=37)


@pytest.mark.parametrize("K", [1 << 18, (1 << 18) + 128])
@pytest.mark.parametrize("signed", [True, False])
@pytest.mark.parametrize("neg", [False, True])
def test_large_tile_largest_products(L, K, signed, neg):
    """Every A code the top LUQ level of R = 6 (2^6, either sign) and every B
    code the largest INT4 (7 signed, 15 unsigned): each output is K * 2^6 * q
    in value units (its int32 carrier sum is at most 2^18 * 64 * 120 < 2^31)."""
    M = N = 4096
    announce("large tile largest products", K, signed, neg)
    byte_g = 0xFF if neg else 0x77   # field 7 with the sign bit set / clear
    byte_w = 0x77 if signed else 0xFF
    gc = torch.full((M * K // 2,), byte_g, dtype=torch.uint8, device="cuda:0")
    wct = torch.full((N * K // 2,), byte_w, dtype=torch.uint8, device="cuda:0")
    alpha = torch.tensor([2.0 ** -6], dtype=torch.float32, device="cuda:0")
    q = 7 if signed else 15
    s = torch.tensor([1.0 / q], dtype=torch.float32, device="cuda:0")
    dx = host(L.luq_gemm_dgrad(gc, alpha, wct, s, signed, M, N, K))
    del gc, wct
    acc = np.full((1,), (-1 if neg else 1) * K * 64 * q, np.int64)
    want = epilogue_replica(acc, np.float32(2.0 ** -6), 1, host(s)[0])[0]
    assert np.all(dx == want), (np.unique(dx)[:4], want)

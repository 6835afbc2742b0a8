"""GPU parity of every GEMM tile shape through the C ABI.

The planner picks a tile and a number of splits by predicted time; the shapes
below select each tile but the largest, which has a file of its own
(tests/test_gemm_plan_cpu.py checks that they do, without a GPU), with M and N at and just past tile edges, K a multiple
of the tile's stage depth (whole stages) and not (the last stage partly past the
end), one stage only, and split reductions whose last split is shorter.  Every A
operand kind (LUQ, two planes, the int8 sums, INT4) runs on every shape.  Outputs
are compared with the oracle within 1e-5 of sum |a b| and bit for bit with the
fp32 epilogue applied to the exact integer sums.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from test_gpu_parity import _gemm_case, _wgrad_case, _fwd_case  # noqa: E402
from test_gpu_smp_sum import _dgrad_sum_case  # noqa: E402
from gpu_util import announce, host  # noqa: E402


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2112_10769_amd as lib
    return lib


TILE_OF = {   # shape: the tile and the splits of a product of one code per k
    (4090, 4104, 2080): ("128x128", 1),
    (4096, 2048, 1024): ("128x256", 1),
    (4099, 2056, 1120): ("128x128", 1),
    (2050, 1032, 544): ("64x64k1", 1),
    (2048, 1024, 512): ("64x64k1", 1),
    (1060, 1032, 1056): ("64x128", 1),
    (1024, 1024, 1024): ("64x64", 1),
    (200, 264, 1056): ("32x64", 1),
    (1, 64, 512): ("32x64", 1),
    (33, 200, 2080): ("32x32", 1),
    (32, 64, 1024): ("32x32", 1),
    (520, 520, 96): ("64x64k1", 1),
    (130, 264, 16416): ("32x64", 9),
    (40, 72, 40000): ("32x32", 40),
    (2050, 3576, 1056): ("128x256", 1),
    (1060, 2072, 2048): ("64x128", 1),
    (2050, 200, 1120): ("64x64", 1),
    (2050, 1800, 128): ("128x128", 1),
    (1024, 2560, 512): ("64x64k1", 1),
    (33, 208, 4096): ("32x32", 1),
}
SHAPES = list(TILE_OF)


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("signed", [True, False])
def test_tile_luq(L, M, N, K, signed):
    _gemm_case(L, M, N, K, 1, signed, seed=M + N + K)


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_tile_two_planes(L, M, N, K):
    _gemm_case(L, M, N, K, 2, True, seed=M + N + K + 1)


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_tile_smp_sum(L, M, N, K):
    _dgrad_sum_case(L, M, N, K, True, seed=M + N + K + 2)


@pytest.mark.parametrize("M,N,K", SHAPES)
@pytest.mark.parametrize("xsig", [True, False])
def test_tile_fwd(L, M, N, K, xsig):
    # an odd number of output columns: scalar stores
    _fwd_case(L, M, N - 3, K, xsig, True, seed=M + N + K + 3)


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_tile_unaligned_output(L, M, N, K):
    """Outputs only 4-byte aligned (dword stores, whole and partial row blocks): the same
    values, and nothing written beside them.  One column and one row fewer in the second
    pass: rows that are not multiples of 16 bytes."""
    for m, n in ((M, N), (max(M - 1, 1), N - 1)):
        announce("unaligned output", m, n, K)
        gen = torch.Generator(device="cuda").manual_seed(m + n + K)
        a, b = (torch.randint(256, (rows * K // 2,), dtype=torch.uint8, device="cuda", generator=gen) for rows in (m, n))
        a &= 0x77
        alpha, scale = torch.full((1,), 0.0123, device="cuda"), torch.full((1,), 0.37, device="cuda")
        rows = -(-n // 4) * 4                      # the reference: the same product in rows of 16-byte multiples
        wide = torch.zeros(rows * K // 2, dtype=torch.uint8, device="cuda")
        wide[:b.numel()] = b
        want = host(L.luq_gemm_dgrad(a, alpha, wide, scale, True, m, rows, K))[:, :n]
        buf = torch.full((m * n + 8,), float("nan"), device="cuda")
        L.luq_gemm_dgrad(a, alpha, b, scale, True, m, n, K, dx=buf[1:1 + m * n])
        got = host(buf)
        assert np.array_equal(got[1:1 + m * n].reshape(m, n), want)
        assert np.isnan(got[:1]).all() and np.isnan(got[1 + m * n:]).all(), "wrote outside the output"


@pytest.mark.parametrize("T,Nout,Kin", [(1056, 1064, 520), (65568, 72, 40), (96, 1032, 264)])
def test_tile_wgrad(L, T, Nout, Kin):
    _wgrad_case(L, T, Nout, Kin, 1, signed=False, seed=T + Nout + Kin)

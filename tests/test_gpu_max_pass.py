"""GPU check of the quantizers' max pass: the maximum is found wherever it lies.

A max-pass thread takes a batch of groups of eight elements one grid stride apart and
what is left of a batch at the end.  The sizes leave every kind of rest: none, one
group, a few groups, a last group of one to seven elements; a single block and many;
tensors on either side of 16 MiB.  The maximum is put at the first and last element,
around each block's and stride's edge and at random places, one call each; maxabs and
the INT4 scale (signed and unsigned) must be exactly that element's.
"""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

from gpu_util import announce, host  # noqa: E402


@pytest.fixture(scope="module")
def L():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2112_10769_amd as lib
    return lib


GROUP = 8
BLOCK = 256 * GROUP
SIZES = [1, 7, 8, 9, BLOCK, BLOCK + 1, 4 * BLOCK - 8, 4 * BLOCK, 4 * BLOCK + 24, 12 * BLOCK + 3, 36 * BLOCK - 8,
         36 * BLOCK, 70000, 2082048, 4194304 + 8 * 37 + 5, 8388608 + 8 * 300 + 1]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_maximum_anywhere(L, n, dtype):
    announce("max pass", n, dtype)
    rng = np.random.default_rng(n)
    x = (torch.rand(n, device="cuda", generator=torch.Generator(device="cuda").manual_seed(n)) * 0.5).to(dtype)
    # the grid takes four, sixteen or eight groups a thread, in whole multiples of 8 blocks or not
    groups = -(-n // GROUP)
    edges = {0, n - 1, n - n % GROUP, n - n % GROUP - 1}
    for per in (4, 16):
        blocks = -(-groups // (256 * per))
        for b in (blocks, -(-blocks // 8) * 8):
            for k in range(1, per + 1):
                edges |= {k * b * BLOCK - 1, k * b * BLOCK}
    spots = sorted(p for p in edges if 0 <= p < n) + [int(p) for p in rng.integers(0, n, 12)]
    codes = torch.empty(n, dtype=torch.uint8, device="cuda")
    mx, al, sc = (torch.empty(1, device="cuda") for _ in range(3))
    got, want = [], []
    for i, p in enumerate(spots):
        keep = x[p].clone()
        value = 1.0 + i / 256.0                       # exact in bfloat16 up to 128 spots
        x[p] = -value if i % 2 else value
        v = float(x[p])
        L.luq_quantize_grad(x, codes=codes, maxabs=mx, alpha=al)
        got.append(mx.clone())
        want.append(np.float32(abs(v)))
        for signed in (True, False):
            if signed or v > 0:
                L.int4_quantize(x, is_signed=signed, codes=codes, scale=sc)
                got.append(sc.clone())
                want.append(np.float32(abs(v)) / np.float32(7 if signed else 15))
        x[p] = keep
    assert np.array_equal(host(torch.cat(got)), np.array(want, np.float32))

"""The GEMM planner, through the workspace it asks for (host only).

A split plan asks for one [M][N] int32 slab per split, so the split count can be
read back.  Every chunk's int32 sums must stay exact: |A| <= 64 and |B| <= 120 for
the LUQ products (chunks up to 2^18), 120 * 120 for INT4 times INT4 (2^17).
"""
import json
import os
import random
import shutil
import subprocess
import sys

import pytest

import paper_2112_10769_amd as luq

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _splits(op, M, N, K):
    d = (K, M, N) if op == luq.OP_GEMM_WGRAD else (M, N, K)
    ws = luq.workspace_size(op, *d)
    assert ws % (4 * M * N) == 0
    return ws // (4 * M * N)


@pytest.mark.parametrize("op,limit", [(luq.OP_GEMM_DGRAD, 1 << 18), (luq.OP_GEMM_WGRAD, 1 << 18),
                                      (luq.OP_GEMM_FWD, 1 << 17)])
def test_splits_keep_int32_sums_exact(op, limit):
    rng = random.Random(3)
    shapes = [(rng.randint(1, 9000), rng.randint(1, 9000), 32 * rng.randint(1, 60000)) for _ in range(400)]
    shapes += [(m, n, k) for m in (1, 64, 8192) for n in (1, 576, 4096)
               for k in (32, limit - 32, limit, limit + 32, 2 * limit, 2 * limit + 32, 5 * limit + 96)]
    for M, N, K in shapes:
        s = _splits(op, M, N, K)
        assert s != 1, (M, N, K)                       # one split needs no workspace
        assert s > 0 or K <= limit, (M, N, K, s)
        if s:                                          # chunks are whole stages of at most 1024
            assert -(-K // (s * 1024)) * 1024 <= limit and s <= -(-K // 128), (M, N, K, s)


def test_few_tiles_split_and_many_do_not():
    assert _splits(luq.OP_GEMM_WGRAD, 64, 576, 200704) > 1
    assert _splits(luq.OP_GEMM_DGRAD, 8192, 4096, 16384) == 0
    assert _splits(luq.OP_GEMM_DGRAD, 2048, 1024, 4096) == 0


GEMM_OPS = (luq.OP_GEMM_DGRAD, luq.OP_GEMM_WGRAD, luq.OP_GEMM_FWD, luq.OP_GEMM_DGRAD_FP6, luq.OP_GEMM_WGRAD_FP6)


def _query(M, N, K):
    """workspace_size of every GEMM, in a process of its own: a crash in it is one failure."""
    args = [(op, K, M, N) if op in (luq.OP_GEMM_WGRAD, luq.OP_GEMM_WGRAD_FP6) else (op, M, N, K) for op in GEMM_OPS]
    code = f"import paper_2112_10769_amd as l; print([l.workspace_size(*a) for a in {args}])"
    res = subprocess.run([sys.executable, "-c", code], capture_output=True, text=True, cwd=ROOT)
    assert res.returncode == 0, (M, N, K, res.returncode)
    return json.loads(res.stdout.splitlines()[-1])


# Sizes that every call refuses: tile counts that wrap to 0, split counts beyond 32
# bits, operands and split sums beyond any address, and one past the query's limits.
@pytest.mark.parametrize("M,N,K", [(1 << 40, 1 << 40, 1 << 20), (1 << 62, 1 << 62, 1 << 62), (1 << 36, 1 << 62, 1 << 36),
                                   (5, 7, 1 << 55), (1, 1, (1 << 62) + 5), (5, 7, 1 << 31), (1 << 30, 7, 32),
                                   ((1 << 30) - 1, (1 << 30) - 1, (1 << 31) - 1)])
def test_workspace_query_of_refused_sizes_is_zero(M, N, K):
    assert _query(M, N, K) == [0] * len(GEMM_OPS)


def test_workspace_query_at_its_limits():
    """The longest reduction a query plans for, K = 2^31 - 1."""
    K = (1 << 31) - 1
    for op, ws, limit in zip(GEMM_OPS, _query(5, 7, K), (1 << 18, 1 << 18, 1 << 17)):
        assert ws % (4 * 35) == 0 and ws // (4 * 35) >= -(-K // limit), op


# ---- which tile a shape gets ------------------------------------------------------

PLAN = r"""
#include <stdio.h>
#include "gemm_kernel.hpp"
int main() {
  long M, N, K, exact;
  int kind;
  while (scanf("%ld %ld %ld %ld %d", &M, &N, &K, &exact, &kind) == 5) {
    const luq::GemmPlan p = luq::search_plan(M, N, K, exact, (luq::PlanKind)kind);
    printf("%d %d\n", (int)p.tile, p.splits);
  }
}
"""
TILES = ["256x256", "128x256", "128x128", "64x128", "64x64", "32x64", "32x32", "64x64k1"]
DEPTH = dict(zip(TILES, (128, 128, 128, 256, 512, 512, 1024, 128)))


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    """The planner compiled for the host: (M, N, K, exact limit, two planes) -> (tile, splits)."""
    hipcc = shutil.which("hipcc") or "/opt/rocm/bin/hipcc"
    if not os.path.exists(hipcc):
        pytest.skip("no hipcc")
    d = tmp_path_factory.mktemp("plan")
    (d / "plan.hip").write_text(PLAN)
    pkg = os.path.join(ROOT, "paper_2112_10769_amd", "csrc")
    subprocess.run([hipcc, "--cuda-host-only", "-std=c++17", "-O1", "-I", pkg, "-I", os.path.join(ROOT, "include"),
                    str(d / "plan.hip"), "-o", str(d / "plan")], check=True, capture_output=True)

    def ask(shapes):
        text = "\n".join(" ".join(str(int(v)) for v in s) for s in shapes)
        out = subprocess.run([str(d / "plan")], input=text, check=True, capture_output=True, text=True).stdout
        return [(TILES[int(t)], int(s)) for t, s in (line.split() for line in out.splitlines())]
    return ask


LIMITS = [(1 << 18, 0), (1 << 18, 1), (1 << 17, 0)]   # LUQ and the sums, two planes, INT4


def test_large_tile_shapes_get_the_large_tile(plans):
    from test_gpu_gemm_large_tile import LARGE
    for limit in LIMITS:
        assert plans([(*s, *limit) for s in LARGE]) == [("256x256", 1)] * len(LARGE), limit
    assert {K % 128 == 0 for _, _, K in LARGE} == {True, False}


def test_tile_shapes_get_their_tiles(plans):
    """The shapes of the per-tile GPU tests select the tiles that they name, and for every
    operand kind each tile that it has is among them, on whole stages and on a partly
    filled last one (the largest tile: the test above)."""
    from test_gpu_gemm_tiles import SHAPES, TILE_OF
    got = plans([(*s, 1 << 18, 0) for s in SHAPES])
    assert got == [TILE_OF[s] for s in SHAPES]
    for limit in LIMITS:
        kinds = {(t, s[2] % DEPTH[t] == 0) for s, (t, _) in zip(SHAPES, plans([(*s, *limit) for s in SHAPES]))}
        tiles = [t for t in TILES[1:] if limit[1] == 0 or t not in ("64x64", "32x32")]
        missing = {(t, w) for t in tiles for w in (True, False)} - kinds
        assert not missing, (limit, missing)


def test_query_covers_both_plans(plans):
    """The workspace query answers for one plane, sums and two planes alike."""
    rng = random.Random(5)
    shapes = [(rng.randint(1, 3000), rng.randint(1, 3000), 32 * rng.randint(1, 4000)) for _ in range(300)]
    one, two = (plans([(*s, 1 << 18, kind) for s in shapes]) for kind in (0, 1))
    differ = 0
    for s, (_, a), (_, b) in zip(shapes, one, two):
        need = max(a if a > 1 else 0, b if b > 1 else 0)
        assert _splits(luq.OP_GEMM_DGRAD, *s) == need, s
        differ += a != b
    assert differ, "the shapes do not tell the two plans apart"


@pytest.mark.parametrize("d", [(1, 1, 1 << 40), (1 << 31, 1 << 31, 32), (1, 1, (1 << 62) + 5), (5, 7, 1)])
def test_workspace_query_takes_any_sizes(d):
    for op in (luq.OP_GEMM_DGRAD, luq.OP_GEMM_WGRAD, luq.OP_GEMM_FWD):
        assert luq.workspace_size(op, *d) >= 0

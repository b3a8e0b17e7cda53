"""The choice of GEMM tiles (host only): the launches that the 14B step is documented to make, the
choices that must never be made, and which tiles the GPU tests' shapes run in."""
import random

import pytest

from gemm_plans import TILES, plan

PAIRS = {("192x256", "128x256"), ("256x256", "128x256"), ("256x256", "192x256")}


# the 14B step's projections at 3152 rows; a 256-pixel camera's and one frame's rows
@pytest.mark.parametrize("M,N,K,bf16,fp8", [
    (3152, 15360, 5120, ("256x256", "128x256", 19), ("256x256", "128x256", 19)),   # QKV
    (3152, 13824, 5120, ("256x256", "192x256", 39), ("256x256", "192x256", 39)),   # FFN1
    (3152, 5120, 5120, ("128x256",), ("128x256",)),                                # O, cross-Q, cross-O
    (3152, 5120, 13824, ("128x256",), ("128x256",)),                               # FFN2
    (544, 13824, 5120, ("288x128",), ("192x256",)),
    (1560, 5120, 5120, ("288x128",), ("192x256",)),
])
def test_documented_plans(M, N, K, bf16, fp8):
    assert plan(M, N, K) == bf16
    assert plan(M, N, K, fp8=True) == fp8
    if N == 13824:  # FFN1 writes its output block-scaled
        assert plan(M, N, K, fp8=True, mx8=True) == fp8


def test_plans_are_launchable():
    """Tiles that a type or an output cannot take are never chosen, and of two column ranges both
    hold columns; over sizes far past the fitted ones, grouped products and other CU counts."""
    rng = random.Random(4)
    for _ in range(4000):
        M, N, K = (int(2 ** rng.uniform(0, b)) for b in (17, 15, 15))
        for fp8, mx8 in ((False, False), (True, False), (True, True)):
            n = (N + 127) // 128 * 128 if mx8 else N
            for ng, cus in ((1, 256), (rng.randint(2, 48), 256), (1, rng.choice([8, 64, 304]))):
                p = plan(M, n, K, fp8, mx8, ng, cus)
                assert p[0] in TILES
                if fp8:
                    assert "288x128" not in p
                if mx8:
                    assert "64x64" not in p and "192x128" not in p
                if len(p) == 3:
                    assert ng == 1 and p[:2] in PAIRS and 0 < p[2] < (n + 255) // 256


def test_gpu_shapes_cover_every_tile():
    """The GPU tests of the products run every tile and every pair of column ranges that a type
    and an output can take, with ragged last tiles."""
    import test_fp8_gpu as f8
    import test_gemm_tiles_gpu as tg
    import test_kernels_gpu as tk
    every = set((t,) for t in TILES) | PAIRS
    no288 = every - {("288x128",)}

    def ran(shapes, **kw):
        return {plan(*s, **kw)[:2] for s in shapes}

    assert ran(tg.TILE_SHAPES) == every
    assert ran(tg.TILE_SHAPES_FP8, fp8=True) == no288
    assert ran(tk.GEMM_SHAPES) >= PAIRS  # with row tails and every epilogue
    assert ran(f8.MXA_SHAPES, fp8=True) == no288
    assert ran(f8.MX8_SHAPES, fp8=True, mx8=True) == no288 - {("64x64",), ("192x128",)}

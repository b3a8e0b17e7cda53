"""GPU parity of the GEMM's tile choices at the edges of their tiles: products that leave most
of the chip idle in the largest tiles take smaller ones."""
import numpy as np
import pytest

import oracle
import synth
from dit_cases import BlockCase
from gpu_helpers import dev, host, log, rel_l2

pytestmark = pytest.mark.gpu


def lib():
    import paper_2602_15922_amd as w
    return w


# 64x64 tiles (one row; one past a tile; a K tail below one slice, of several slices), 128x128,
# 192x128, 288x128 and 128x256 tiles with a ragged last row and column tile
SHAPES = [(1, 64, 64), (65, 72, 520), (63, 16, 5120), (300, 520, 40), (545, 5120, 512), (513, 10248, 520),
          (500, 13824, 256), (570, 13824, 296), (289, 13832, 72), (575, 13832, 1032)]


@pytest.mark.parametrize("M,N,K", SHAPES)
def test_gemm_tile_edges(M, N, K):
    """bf16 output (one bf16 rounding: 3e-3) and the fp32 residual (fp32 sums: 1e-5) of every
    product against the fp64 oracle on the rows at the tiles' edges."""
    import torch
    w = lib()
    log(f"gemm tiles M={M} N={N} K={K}")
    A = synth.normal(21, "x", (M, K), 1.0, M)
    W = synth.normal(21, "w_o", (N, K), 0.05, N)
    x0 = synth.normal(21, "o_init", (M, N), 1.0, K, dtype="f32")
    rows = np.unique([r for e in (0, 32, 64, 128, 192, 256, 384, 512, M) for r in (e - 1, e) if 0 <= r < M])
    ref = oracle.linear(A.f64[rows], W.f64)
    out = torch.full((M + 1, N), -1.0, dtype=torch.bfloat16, device="cuda")
    w.wam_gemm_bf16(dev(A), dev(W), out[:M], w.WAM_EPI_BF16)
    res = dev(x0)
    w.wam_gemm_bf16(dev(A), dev(W), res, w.WAM_EPI_RESID_F32)
    torch.cuda.synchronize()
    assert rel_l2(host(out)[rows], ref) <= 3e-3
    assert (host(out[M]) == -1).all()
    assert rel_l2(host(res)[rows] - x0.f64[rows], ref) <= 1e-5


# a wide FFN and a short one, odd rows: products of few tiles and many K slices
@pytest.mark.parametrize("fp8", [False, True])
@pytest.mark.parametrize("d,H,ffn,Hl,Wl,A,Lc", [(512, 8, 2048, 10, 14, 3, 19), (1280, 10, 8960, 18, 34, 7, 33)])
def test_block_few_rows(d, H, ffn, Hl, Wl, A, Lc, fp8):
    """A block of few rows against the fp64 oracle (2e-2; FP8 projections of the unquantized
    model: 0.1), three runs bitwise equal."""
    wl = synth.WORKLOADS["block_d512"].replace(d=d, H=H, Dh=d // H, ffn=ffn, Hl=Hl, Wl=Wl, A=A, Lc=Lc, n_cached=1,
                                               mod_std=0.3)
    log(f"few-row block d={d} L={wl.L} fp8={fp8}")
    case = BlockCase(wl, bias_std=0.05)
    x, kc, vc = case.run_gpu(fp8=fp8)
    rx, _, _ = case.run_oracle()
    tol = 0.1 if fp8 else 2e-2
    assert rel_l2(host(x), rx) <= tol
    for _ in range(2):
        y, _, _ = case.run_gpu(fp8=fp8)
        assert np.array_equal(host(x), host(y))

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


# one row, one past a tile, K tails below one slice and of several slices, wide N with a short K
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


# one product per tile and pair of column ranges (test_gemm_plan.py holds the choice to that): ragged
# last row and column tiles, K tails, more slices than a ring's stages
TILE_SHAPES = [(65, 88, 584), (257, 6536, 584), (513, 6544, 648), (513, 13064, 2312), (778, 6536, 776), (1156, 6568, 584),
               (1741, 6544, 776), (770, 6584, 584), (1025, 14608, 584), (1798, 13080, 776), (2305, 8208, 1032)]
TILE_SHAPES_FP8 = [(65, 40, 1168), (259, 6600, 1168), (513, 6632, 1168), (769, 6552, 1584), (1156, 6560, 1168),
                   (1729, 6544, 1552), (769, 6552, 1168), (1038, 14480, 1168), (1795, 13120, 1552), (2314, 8200, 2064)]


def edge_rows(M):
    return np.unique([r for t in (64, 128, 192, 256, 288) for e in (*range(0, M, t), M) for r in (e - 1, e)
                      if 0 <= r < M and (e <= 2 * t or e > M - 2 * t)])


@pytest.mark.parametrize("M,N,K,fp8", [s + (False,) for s in TILE_SHAPES] + [s + (True,) for s in TILE_SHAPES_FP8])
def test_gemm_every_tile(M, N, K, fp8):
    """bf16 output (one bf16 rounding: 3e-3) and the gated fp32 residual (fp32 sums: 1e-5; the
    FP8 matrix instruction accumulates with fewer guard bits: 5e-5) of every tile against the
    fp64 product of the same operands on the rows at the tiles' edges; the row past the last
    untouched."""
    import torch
    w = lib()
    log(f"gemm every tile M={M} N={N} K={K} fp8={fp8}")
    A = synth.normal(22, "x", (M, K), 1.0, M)
    W = synth.normal(22, "w_o", (N, K), 0.05, N)
    bias = synth.normal(22, "b_o", (N,), 0.1, N, dtype="f32")
    gate = synth.normal(22, "mod6", (N,), 0.5, N, dtype="f32")
    rows = edge_rows(M)
    out = torch.full((M + 1, N), -1.0, dtype=torch.bfloat16, device="cuda")
    x0 = torch.randn((M + 1, N), generator=torch.Generator(device="cuda").manual_seed(K), device="cuda")
    res = x0.clone()
    if fp8:
        qa, qw = (torch.empty(t.shape, dtype=torch.uint8, device="cuda") for t in (A, W))
        sa, sw = torch.empty(M, device="cuda"), torch.empty(N, device="cuda")
        w.wam_quantize_rows_fp8(dev(A), qa, sa)
        w.wam_quantize_rows_fp8(dev(W), qw, sw)
        w.wam_gemm_fp8(qa, qw, out[:M], w.WAM_EPI_BF16, sa, sw, bias=dev(bias))
        w.wam_gemm_fp8(qa, qw, res[:M], w.WAM_EPI_RESID_F32, sa, sw, bias=dev(bias), gate_a=dev(gate))
        a64, w64 = (q.view(torch.float8_e4m3fn).double().cpu().numpy() * host(s)[:, None] for q, s in ((qa, sa), (qw, sw)))
    else:
        da, dw = dev(A), dev(W)
        w.wam_gemm_bf16(da, dw, out[:M], w.WAM_EPI_BF16, bias=dev(bias))
        w.wam_gemm_bf16(da, dw, res[:M], w.WAM_EPI_RESID_F32, bias=dev(bias), gate_a=dev(gate))
        a64, w64 = A.f64, W.f64
    torch.cuda.synchronize()
    ref = a64[rows] @ w64.T + bias.f64
    assert rel_l2(host(out)[rows], ref) <= 3e-3
    assert rel_l2(host(res)[rows] - host(x0)[rows], gate.f64 * ref) <= (5e-5 if fp8 else 1e-5)
    assert (host(out[M]) == -1).all() and torch.equal(res[M], x0[M])


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

"""Both sides of the rule that gives a product 32 x 128 tiles: a token's outputs are the same, bit for bit, whichever tile
its call runs on.  (Each kernel is checked against the oracle elsewhere.)"""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("bits", [3, 4, 8])
@pytest.mark.parametrize("M,N", [
    (1024, 3064), (2017, 1528), (96, 32760),
    (1024, 3200),                                              # 800 tiles: more than three per compute unit
    (190, 5376), (190, 5384), (64, 16384), (64, 16392),        # 252 tiles, 258; 256, 258
    (96, 27136), (96, 27640), (330, 4352), (290, 4992), (352, 8184), (600, 3328), (600, 3336),     # 636, 648; 374, 390; 704; 494, 513
])
def test_outputs_do_not_depend_on_the_tile(M, N, bits):
    import paper_2304_01089_amd as rp
    d, g, dev = 328, 9, dict(device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(M + N + bits)
    more = M + 32 * 400                                        # (well past 768 tiles)
    x = (torch.randn(more, d, generator=gen, **dev) * torch.exp(torch.randn(d, generator=gen, **dev))).bfloat16()
    cal = rp.calibrate_site([x[:256]], None, None, 1e-5, False, g, bits, seed=1)
    W = 0.02 * torch.randn(N, d, generator=gen, **dev)
    codes, _, rt = rp.ln_quant(cal, x, 1e-5)
    lin = rp.fold_linear(cal, W)
    for dtype in (torch.bfloat16, torch.float32):
        assert torch.equal(rp.cluster_gemm(cal, lin, codes, rt, M, dtype=dtype), rp.cluster_gemm(cal, lin, codes, rt, more, dtype=dtype)[:M])
    cw, sums = rp.fold_linear_cw(cal, W), rp.cluster_rowsums(cal, codes, more)
    assert torch.equal(rp.cluster_gemm_cw(cal, cw, codes, sums, M), rp.cluster_gemm_cw(cal, cw, codes, sums, more)[:M])
    nxt = rp.calibrate_site([(x[:256].float() @ W.T).bfloat16()], None, None, 1e-5, True, g, bits, seed=2)
    fused = rp.fold_linear(cal, W, next_site=nxt)
    c0, r0 = rp.cluster_gemm_quant(cal, fused, codes, rt, M, nxt)
    c1, r1 = rp.cluster_gemm_quant(cal, fused, codes, rt, more, nxt)
    assert torch.equal(c0, c1[: c0.numel()])
    # (fp64 sums per column tile of 128 or 256, rounded once to fp32)
    torch.testing.assert_close(r0, r1[:M], rtol=2.0 ** -23, atol=0.0)


@pytest.mark.parametrize("bits", [3, 4, 8])
@pytest.mark.parametrize("M,N", [
    (2048, 4608), (2017, 6296), (4070, 4200), (8190, 1248),    # 64 x 256 tiles: 512 + 64, 768 + 32, 1024 + 64, 512 + 128
])
def test_last_columns_on_small_tiles(M, N, bits):
    """More than two 64 x 256 tiles per compute unit and a few over: their columns run on 64 x 128 tiles in the same launch.
    Outputs, codes and row terms are those of calls of few rows, which run on other tiles throughout."""
    import paper_2304_01089_amd as rp
    d, g, dev, few = 328, 9, dict(device="cuda"), 160
    gen = torch.Generator(device="cuda").manual_seed(M + N + bits)
    x = (torch.randn(M, d, generator=gen, **dev) * torch.exp(torch.randn(d, generator=gen, **dev))).bfloat16()
    cal = rp.calibrate_site([x[:256]], None, None, 1e-5, False, g, bits, seed=1)
    W = 0.02 * torch.randn(N, d, generator=gen, **dev)
    codes, _, rt = rp.ln_quant(cal, x, 1e-5)
    parts = []
    for first in (0, M // 2, M - few):                          # (a copy: row starts are aligned anew)
        part, _, part_rt = rp.ln_quant(cal, x[first:first + few].clone(), 1e-5)
        parts.append((slice(first, first + few), part, part_rt))
    lin = rp.fold_linear(cal, W)
    for dtype in (torch.bfloat16, torch.float32):
        y = rp.cluster_gemm(cal, lin, codes, rt, M, dtype=dtype)
        assert all(torch.equal(y[at], rp.cluster_gemm(cal, lin, c, r, few, dtype=dtype)) for at, c, r in parts)
    cw = rp.fold_linear_cw(cal, W)
    y = rp.cluster_gemm_cw(cal, cw, codes, rp.cluster_rowsums(cal, codes, M), M)
    assert all(torch.equal(y[at], rp.cluster_gemm_cw(cal, cw, c, rp.cluster_rowsums(cal, c, few), few)) for at, c, _ in parts)
    nxt = rp.calibrate_site([(x[:256].float() @ W.T).bfloat16()], None, None, 1e-5, True, g, bits, seed=2)
    fused = rp.fold_linear(cal, W, next_site=nxt)
    c0, r0 = rp.cluster_gemm_quant(cal, fused, codes, rt, M, nxt)
    rows = c0.view(M, -1)
    for at, c, r in parts:
        c1, r1 = rp.cluster_gemm_quant(cal, fused, c, r, few, nxt)
        assert torch.equal(rows[at], c1.view(few, -1))
        # (fp64 sums per column tile of 128 or 256, rounded once to fp32)
        torch.testing.assert_close(r0[at], r1, rtol=2.0 ** -23, atol=0.0)

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


def small_tiles_behind(M, N):
    """The rule beyond 704 tiles of 64 x 256: so many of their columns go out as 64 x 128 tiles."""
    rows, cols = -(-M // 64), -(-N // 256)
    over = rows * cols % 256
    last = -(-over // rows)
    return last if rows * cols > 704 and 2 * last * rows <= 256 else 0


@pytest.mark.parametrize("bits", [3, 4, 8])
@pytest.mark.parametrize("M,N,d", [
    (2048, 8704, 328), (8190, 2100, 328),        # 1024 tiles of 64 x 256 and 64, 128 on 64 x 128: whole numbers per compute unit
    (2100, 8000, 328), (2900, 4099, 328),        # 33, 46 row tiles: walked row by row, a large part of 1023, 736
    (3072, 5600, 328), (1000, 18000, 328),       # 48, 16: blocks of 16 row tiles; seven columns, fourteen small ones: four walks
    (4070, 4200, 328), (2048, 7000, 328),
    (2100, 4500, 5128),                          # 594 tiles: at 8 bits over a long K 495 and 99; 64 x 128 tiles else
    (2100, 5000, 328),                           # 660 tiles: 64 x 128 tiles throughout
])
def test_last_columns_on_small_tiles(M, N, d, bits):
    """Whole rounds of 64 x 256 tiles and a few over: the columns of these run on 64 x 128 tiles in the same launch.  Every row's
    outputs, codes and row terms are those of calls of few rows, which run on other tiles throughout."""
    import paper_2304_01089_amd as rp
    g, dev, few = 9, dict(device="cuda"), 160
    behind = d == 328 and N != 5000
    assert bool(small_tiles_behind(M, N)) == behind
    gen = torch.Generator(device="cuda").manual_seed(M + N + bits)
    x = (torch.randn(M, d, generator=gen, **dev) * torch.exp(torch.randn(d, generator=gen, **dev))).bfloat16()
    cal = rp.calibrate_site([x[:256]], None, None, 1e-5, False, g, bits, seed=1)
    W = 0.02 * torch.randn(N, d, generator=gen, **dev)
    codes, _, rt = rp.ln_quant(cal, x, 1e-5)
    parts = []
    for first in range(0, M, few):                              # (copies: row starts are aligned anew)
        part, _, part_rt = rp.ln_quant(cal, x[first:first + few].clone(), 1e-5)
        parts.append((slice(first, min(M, first + few)), len(part_rt), part, part_rt))
    lin, cw, sums = rp.fold_linear(cal, W), rp.fold_linear_cw(cal, W), rp.cluster_rowsums(cal, codes, M)
    for dtype in (torch.bfloat16, torch.float32):
        y, yc = (torch.full((M + 1, N), 7.0, dtype=dtype, **dev) for _ in range(2))
        rp.cluster_gemm(cal, lin, codes, rt, M, y=y[:M])
        rp.cluster_gemm_cw(cal, cw, codes, sums, M, y=yc[:M])
        for at, n, c, r in parts:
            assert torch.equal(y[at], rp.cluster_gemm(cal, lin, c, r, n, dtype=dtype)), at
            assert torch.equal(yc[at], rp.cluster_gemm_cw(cal, cw, c, rp.cluster_rowsums(cal, c, n), n, dtype=dtype)), at
        assert (y[M:] == 7.0).all() and (yc[M:] == 7.0).all()
    W = W[: N // 8 * 8]                                         # (a site's width)
    nxt = rp.calibrate_site([(x[:256].float() @ W.T).bfloat16()], None, None, 1e-5, True, g, bits, seed=2)
    fused = rp.fold_linear(cal, W, next_site=nxt)
    assert bool(small_tiles_behind(M, fused.N)) == behind
    rows = torch.full((M + 1, fused.N * bits // 8), 0xab, dtype=torch.uint8, **dev)
    terms = torch.full((M + 1,), float("nan"), **dev)
    rp.cluster_gemm_quant(cal, fused, codes, rt, M, nxt, next_codes=rows[:M], next_rowterm=terms[:M])
    for at, n, c, r in parts:
        c1, r1 = rp.cluster_gemm_quant(cal, fused, c, r, n, nxt)
        assert torch.equal(rows[at], c1.view(-1)[: n * rows.shape[1]].view(n, -1)), at
        # (fp64 sums per column tile of 128 or 256, rounded once to fp32)
        torch.testing.assert_close(terms[at], r1[:n], rtol=2.0 ** -23, atol=0.0)
    assert (rows[M:] == 0xab).all() and terms[M:].isnan().all()

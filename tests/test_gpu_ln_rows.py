"""The LayerNorm + quantize kernel for few rows per compute unit against the pipelined one, at the edges of its rule: a
row's codes and row sum do not depend on how many rows share its call.  (The oracle's tests run both.)"""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def make_call(d, g, bits, M, seed=3, ln=True):
    import paper_2304_01089_amd as rp
    rng = np.random.default_rng(seed + d + g)
    cuts = np.sort(rng.choice(np.arange(1, d), g - 1, replace=False)) if g > 1 else []
    off = np.concatenate([[0], cuts, [d]]).astype(np.int32)
    s = np.exp(rng.normal(-1, 0.5, g)).astype(np.float32)
    inv = (1.0 / s.astype(np.float64)).astype(np.float32)
    z = rng.integers(-3, 4, g).astype(np.int32)
    z[0] = -(1 << 21)                                          # (the largest zero point: every code of the cluster saturates)
    kp = rp.rptq_padded_k(off)
    dev = dict(device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(seed)
    gamma, beta = torch.exp(0.3 * torch.randn(d, generator=gen, **dev)), 0.1 * torch.randn(d, generator=gen, **dev)
    perm_pad = torch.zeros(kp, dtype=torch.int32, **dev)
    gp, bp = (torch.zeros(kp, **dev) for _ in range(2)) if ln else (None, None)
    rp.rptq_fold_reorder(gamma if ln else None, beta if ln else None, d, rng.permutation(d).astype(np.int32), off, None, None,
                         None, 0, d, None, perm_pad, gp, bp, None, None, None, None, None)
    x = (torch.randn(M, d, generator=gen, **dev) * 2 + 0.5).bfloat16()
    x[0, : min(d, 5)] = torch.tensor([3e38, -3e38, 0.0, -0.0, 1e-40][: min(d, 5)], **dev).bfloat16()      # (far beyond every code range)

    def call(m, codes=None, rowterm=None):
        codes = torch.zeros((m, kp * bits // 8), dtype=torch.uint8, **dev) if codes is None else codes
        rowterm = torch.zeros(m, **dev) if rowterm is None else rowterm
        rp.rptq_ln_quant(x, m, d, gp, bp, 1e-5, not ln, perm_pad, off, s, inv, z, bits, codes, None, rowterm)
        return codes, rowterm
    return call


@pytest.mark.parametrize("ln", [True, False])
@pytest.mark.parametrize("bits", [3, 4, 8])
@pytest.mark.parametrize("d,g,most", [(8, 1, 128), (776, 64, 128), (2056, 9, 32), (5120, 32, 16), (8184, 32, 4), (12288, 33, 4)])
def test_few_rows_equal_many(d, g, most, bits, ln):
    import paper_2304_01089_amd as rp
    cus = rp.rptq_device_info()["compute_units"]
    many = cus * most + 1
    call = make_call(d, g, bits, many, ln=ln)
    codes, rowterm = call(many)
    for m in sorted({1, 2, 3, cus, cus + 1, 2 * cus, 2 * cus + 1, 2 * cus + 3, cus * most}):
        c, r = call(m)
        assert torch.equal(c, codes[:m]), m
        # (fp64 sums in two orders, each rounded once to fp32: one unit in the last place)
        torch.testing.assert_close(r, rowterm[:m], rtol=2.0 ** -23, atol=0.0, equal_nan=True)


def test_recorded_call_of_another_size():
    """Four wide rows per workgroup need more LDS than a kernel has by default; a call that is recorded before the limit
    was raised runs the other kernel."""
    d, bits = 12288, 4
    call = make_call(d, 32, bits, 2000)
    codes, rowterm = call(2000)
    m = 600
    c, r = torch.zeros_like(codes[:m]), torch.zeros_like(rowterm[:m])
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(m, c, r)
    for _ in range(3):
        c.zero_(), r.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(c, codes[:m])
        torch.testing.assert_close(r, rowterm[:m], rtol=2.0 ** -23, atol=0.0, equal_nan=True)
        call(m)

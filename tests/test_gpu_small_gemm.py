"""The product with K split over a workgroup's waves (few output tiles) against the integer form in float64, at the
edges of its tiles and of its rule (and past it): fewer K steps than waves, clusters that end inside and at the ends of the waves'
ranges, one cluster and 64, odd row and column counts; and against calls of other sizes, bit for bit."""
import numpy as np
import pytest

import packfmt

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("bits", [3, 4, 8])
@pytest.mark.parametrize("M,N,d,g", [
    (1, 1, 8, 8), (1, 33, 40, 9), (31, 1000, 1000, 8), (33, 70, 3000, 64), (32, 8192, 520, 13),     # K in 8
    (33, 4097, 264, 8), (100, 4097, 1032, 32), (32, 32768, 136, 10),                                # K in 4, and not split
    (64, 23040, 72, 8), (333, 4099, 1000, 16), (700, 2047, 2056, 11),
    (65, 15400, 520, 16), (1000, 2049, 1000, 8), (2100, 4500, 200, 9),                              # not split, 64 x 128 tiles
    (1000, 6401, 200, 9), (2100, 5700, 200, 9), (1000, 6403, 136, 3),                               # 416 and 759 tiles of 64 x 256
    (33, 70, 600, 7),
])
def test_split_product_against_float64(M, N, d, g, bits):
    import paper_2304_01089_amd as rp
    rng = np.random.default_rng(M * 7 + N + d + bits)
    cuts = np.sort(rng.choice(np.arange(1, d), g - 1, replace=False)) if g > 1 else []
    off = np.concatenate([[0], cuts, [d]]).astype(np.int32)
    s = np.exp(rng.normal(-3, 1, g)).astype(np.float32)
    z = rng.integers(-(1 << (bits - 1)), 1 << (bits - 1), g).astype(np.int32)
    q = rng.integers(-(1 << (bits - 1)), 1 << (bits - 1), (M, d)).astype(np.int8)
    kp = rp.rptq_padded_k(off)
    dev = dict(device="cuda")
    W = torch.from_numpy((0.02 * rng.standard_normal((N, d))).astype(np.float32)).cuda()
    perm_pad = torch.zeros(kp, dtype=torch.int32, **dev)
    Wq = torch.zeros(rp.rptq_weight_bytes(N, kp), dtype=torch.uint8, **dev)
    sW, ct = torch.zeros(N, **dev), torch.zeros(N, **dev)
    zW, wsum = torch.zeros(N, dtype=torch.int32, **dev), torch.zeros((N, g), dtype=torch.int32, **dev)
    rp.rptq_fold_reorder(None, None, d, rng.permutation(d).astype(np.int32), off, s, z, W, N, d, None, perm_pad, None, None,
                         Wq, sW, zW, wsum, ct)
    wq = torch.empty((N, d), dtype=torch.int8, **dev)
    rp.rptq_unpack_weights(Wq, N, off, wq)
    codes = torch.from_numpy(packfmt.pack_codes(q, off, bits)).cuda()
    rt = torch.from_numpy(rng.standard_normal(M).astype(np.float32)).cuda()
    y32 = torch.full((M + 2, N), 7.0, dtype=torch.float32, **dev)
    y16 = torch.full((M + 2, N), 7.0, dtype=torch.bfloat16, **dev)
    for y in (y32, y16):
        rp.rptq_cluster_gemm(codes, M, bits, Wq, N, off, s, sW, zW, ct, rt, y[:M])
    torch.cuda.synchronize()
    w64, q64 = wq.cpu().numpy().astype(np.float64), q.astype(np.float64)
    total, size = np.zeros((M, N)), np.zeros((M, N))
    pos = np.concatenate([[0], np.cumsum((np.diff(off) + 31) // 32 * 32)])       # padded start of every cluster
    for i in range(g):
        col = pos[i] + np.arange(off[i + 1] - off[i])
        for step in np.unique(col // 128):                # (a cluster is split at multiples of 128 padded positions)
            c = off[i] + np.flatnonzero(col // 128 == step)
            P = float(s[i]) * (q64[:, c] @ w64[:, c].T)
            total += P
            size += np.abs(P)
    f = lambda t: t.cpu().numpy().astype(np.float64)
    ref = f(sW) * ((total - f(ct)) - f(zW) * f(rt)[:, None])
    # one fp32 rounding per cluster (or part of one) in a wave's running sum, whose parts' magnitudes add up to at most
    # `size`; one rounding of each of the two differences and of the products (the unsplit kernel forms them in fp32)
    terms = size + np.abs(f(ct)) + np.abs(f(zW) * f(rt)[:, None])
    tol = 2.0 ** -24 * (f(sW) * ((g + 8) * size + 4 * terms) + 2 * np.abs(ref)) + 1e-30
    got = f(y32[:M])
    assert (np.abs(got - ref) <= tol).all()
    assert torch.equal(y16[:M], y32[:M].bfloat16())           # the same value, rounded once more
    assert (y32[M:] == 7.0).all() and (y16[M:] == 7.0).all()


# clusters of one slice and of many, few K steps and several periods of K (the clusters' sums do not all fit in LDS at once)
@pytest.mark.parametrize("d,g,bits", [(8, 8, 4), (600, 1, 8), (1000, 8, 3), (3000, 64, 4), (2048, 16, 4), (4096, 3, 8), (12288, 32, 3)])
def test_outputs_do_not_depend_on_the_size_of_the_call(d, g, bits):
    import paper_2304_01089_amd as rp
    M, N = 2900, 4099                                      # 46 x 17 tiles of 64 x 256
    rng = np.random.default_rng(d + g + bits)
    cuts = np.sort(rng.choice(np.arange(1, d), g - 1, replace=False)) if g > 1 else []
    off = np.concatenate([[0], cuts, [d]]).astype(np.int32)
    s = np.exp(rng.normal(-3, 1, g)).astype(np.float32)
    z = rng.integers(-(1 << (bits - 1)), 1 << (bits - 1), g).astype(np.int32)
    q = rng.integers(-(1 << (bits - 1)), 1 << (bits - 1), (M, d)).astype(np.int8)
    kp = rp.rptq_padded_k(off)
    dev = dict(device="cuda")
    W = torch.from_numpy((0.02 * rng.standard_normal((N, d))).astype(np.float32)).cuda()
    perm_pad = torch.zeros(kp, dtype=torch.int32, **dev)
    Wq = torch.zeros(rp.rptq_weight_bytes(N, kp), dtype=torch.uint8, **dev)
    sW, ct = torch.zeros(N, **dev), torch.zeros(N, **dev)
    zW, wsum = torch.zeros(N, dtype=torch.int32, **dev), torch.zeros((N, g), dtype=torch.int32, **dev)
    rp.rptq_fold_reorder(None, None, d, rng.permutation(d).astype(np.int32), off, s, z, W, N, d, None, perm_pad, None, None,
                         Wq, sW, zW, wsum, ct)
    codes = torch.from_numpy(packfmt.pack_codes(q, off, bits)).cuda()
    rt = torch.from_numpy(rng.standard_normal(M).astype(np.float32)).cuda()

    def product(m, n, dtype):                               # the first m tokens, the first n output channels
        y = torch.full((m + 1, n), 7.0, dtype=dtype, **dev)
        rp.rptq_cluster_gemm(codes, m, bits, Wq, n, off, s, sW, zW, ct, rt, y[:m])
        assert (y[m] == 7.0).all()
        return y[:m]

    for dtype in (torch.float32, torch.bfloat16):
        whole = product(M, N, dtype)
        for m, n in ((1, 1), (1, 33), (1, 4099), (7, 1000), (16, 256), (17, 4096), (31, 4099), (32, 2049), (33, 2050), (64, 1026),
                     (64, 4099), (130, 3000), (300, 800), (333, 4099), (2900, 64), (1500, 4099)):
            assert torch.equal(product(m, n, dtype), whole[:m, :n]), (m, n, dtype)

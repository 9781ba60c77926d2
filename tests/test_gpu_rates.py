"""Rules that pick a launch's shape, held against work on the same card of which the time is known, with wide margins: they
are there for sizes that the rule's own table may not have."""
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


def shortest(call, reps=5):
    """Shortest of a few timings of one call, in us."""
    call()
    times = []
    for _ in range(reps):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        b.synchronize()
        times.append(a.elapsed_time(b) * 1000)
    return min(times)


def test_calibration_of_many_rows_uses_the_chip():
    """Sixteen batches of 2048 rows x 12288 channels: 1.6 times as long as a copy of them on 256 workgroups, 4.3 times on 64
    (the number that is best for 512 rows)."""
    import paper_2304_01089_amd as rp
    d, dev = 12288, dict(device="cuda")
    x = torch.randn(16, 2048, d, dtype=torch.bfloat16, **dev)
    gamma, beta, out = torch.ones(d, **dev), torch.zeros(d, **dev), torch.zeros(2, d, **dev)
    ws = torch.zeros(rp.rptq_calibrate_workspace_bytes(d), dtype=torch.uint8, **dev)
    to = torch.empty_like(x)
    copy = shortest(lambda: to.copy_(x))
    assert shortest(lambda: rp.rptq_channel_minmax(list(x), gamma, beta, 1e-5, False, out[0], out[1], ws)) < 2.8 * copy


def test_product_of_a_tile_count_that_eight_does_not_divide():
    """192 tokens, K = 12288, weights from memory: 13568 columns take no longer than 13824 (on 32 x 128 tiles, 636 of them,
    every XCD fetches every weight: 73 us against 53)."""
    import numpy as np
    import paper_2304_01089_amd as rp
    M, K, g, bits, dev = 192, 12288, 32, 4, dict(device="cuda")
    off = (np.arange(g + 1) * (K // g)).astype(np.int32)
    sx = np.full(g, 0.01, np.float32)
    codes = torch.randint(0, 256, (rp.rptq_codes_bytes(M, K, bits),), dtype=torch.uint8, **dev)
    time = {}
    for N in (13568, 13824):
        W = [torch.randint(0, 256, (rp.rptq_weight_bytes(N, K),), dtype=torch.uint8, **dev) for _ in range(8)]
        sW, zW, ct, rt = torch.ones(N, **dev), torch.zeros(N, dtype=torch.int32, **dev), torch.zeros(N, **dev), torch.zeros(M, **dev)
        y = torch.empty(M, N, dtype=torch.bfloat16, **dev)

        def call():
            for Wq in W:
                rp.rptq_cluster_gemm(codes, M, bits, Wq, N, off, sx, sW, zW, ct, rt, y)
        time[N] = shortest(call)
        del W
    assert time[13568] < 1.2 * time[13824], time

"""Folding and packing of weight rows against the oracle, bit for bit, at the widths where the kernel's split
changes: eight, four, two and one rows in LDS; odd widths (no 16-byte chunks); output
counts that leave a partial row block; pad rows of an output index."""
import numpy as np
import pytest

from oracle import rptq_oracle as o

import packfmt

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("k,g,N,pads", [
    (40, 3, 5, False), (2048, 16, 70, True), (2333, 32, 33, False), (4096, 32, 40, True), (10232, 8, 9, False),
    (20480, 32, 6, True), (31999, 4, 3, False), (32768, 64, 3, True),
])
def test_fold_rows_bit_exact(k, g, N, pads, dtype):
    import paper_2304_01089_amd as rp
    rng = np.random.default_rng(k + g)
    W = (0.02 * rng.standard_normal((N, k))).astype(np.float32)
    if dtype == "bf16":
        W = torch.from_numpy(W).bfloat16().float().numpy()
    perm = rng.permutation(k).astype(np.int32)
    cuts = np.sort(rng.choice(np.arange(1, k), g - 1, replace=False))
    off = np.concatenate([[0], cuts, [k]]).astype(np.int32)
    s = (0.01 + rng.random(g)).astype(np.float32)
    z = rng.integers(-9, 9, g).astype(np.int32)
    out_rows = np.arange(N)
    if pads:                                              # rows in another order, a pad row (-1) in between
        out_rows = rng.permutation(np.concatenate([np.arange(N), [-1]]))
    n = len(out_rows)
    kp = rp.rptq_padded_k(off)
    dev = dict(device="cuda")
    perm_pad = torch.zeros(kp, dtype=torch.int32, **dev)
    Wq = torch.full((rp.rptq_weight_bytes(n, kp),), 0x5A, dtype=torch.uint8, **dev)
    sW, ct = torch.zeros(n, **dev), torch.full((n,), 7.0, **dev)
    zW, wsum = torch.zeros(n, dtype=torch.int32, **dev), torch.full((n, g), 7, dtype=torch.int32, **dev)
    Wd = torch.from_numpy(W).cuda()
    rp.rptq_fold_reorder(None, None, k, perm, off, s, z, Wd.bfloat16() if dtype == "bf16" else Wd, n, k,
                         out_rows.astype(np.int32) if pads else None, perm_pad, None, None, Wq, sW, zW, wsum, ct)
    torch.cuda.synchronize()
    wq, s_ref, _, z_ref = o.quantize_weights(W, perm, np.maximum(out_rows, 0))
    pad = out_rows < 0
    wq[pad], s_ref[pad], z_ref[pad] = 0, 1.0, 0
    got, extra = packfmt.unpack_weights(Wq.cpu().numpy(), n, off)
    assert np.array_equal(got, wq) and (extra == 0).all()
    n_p = (n + 255) // 256 * 256
    assert packfmt.unpack_weights(Wq.cpu().numpy(), n_p, off)[0][n:].any() == False        # rows added by rounding up
    assert np.array_equal(sW.cpu().numpy(), s_ref) and np.array_equal(zW.cpu().numpy(), z_ref)
    sums = np.add.reduceat(wq.astype(np.int64), off[:-1], axis=1)
    assert np.array_equal(wsum.cpu().numpy(), sums)
    ref = ((s.astype(np.float64) * z)[None, :] * sums).sum(axis=1)
    # one fp64 sum in another order, rounded once to fp32
    assert np.allclose(ct.cpu().numpy(), ref, rtol=2.0 ** -23, atol=1e-12 * np.abs((s * z)[None, :] * sums).sum(axis=1).max())


def test_fold_reports_bad_weights():
    import paper_2304_01089_amd as rp
    k, N = 4096, 40
    off = np.array([0, k], np.int32)
    dev = dict(device="cuda")
    perm_pad = torch.zeros(rp.rptq_padded_k(off), dtype=torch.int32, **dev)
    Wq = torch.zeros(rp.rptq_weight_bytes(N, k), dtype=torch.uint8, **dev)
    args = (torch.zeros(N, **dev), torch.zeros(N, dtype=torch.int32, **dev), torch.zeros(N, dtype=torch.int32, **dev), torch.zeros(N, **dev))
    for value in (float("nan"), float("-inf")):
        W = torch.full((N, k), 0.5, **dev)
        W[N - 1, k - 1] = value
        with pytest.raises(rp.RptqError) as e:
            rp.rptq_fold_reorder(None, None, k, np.arange(k, dtype=np.int32), off, [1.0], [0], W, N, k, None, perm_pad, None, None, Wq, *args)
        assert e.value.status == -6


def test_concurrent_folds_report_their_own_weights():
    """Two threads on two streams, one with a weight that is not finite: only its calls fail."""
    import threading

    import paper_2304_01089_amd as rp
    rp.load_library()
    k, N, rounds = 1024, 4096, 200
    off = np.array([0, k // 2, k], np.int32)
    dev = dict(device="cuda")
    bad_calls, errors = {True: 0, False: 0}, []
    start = threading.Barrier(2)

    def work(bad):
        try:
            stream = torch.cuda.Stream()
            with torch.cuda.stream(stream):
                W = torch.full((N, k), 0.5, **dev)
                if bad:
                    W[0, 0] = float("nan")
                perm_pad = torch.zeros(rp.rptq_padded_k(off), dtype=torch.int32, **dev)
                Wq = torch.zeros(rp.rptq_weight_bytes(N, k), dtype=torch.uint8, **dev)
                args = (torch.zeros(N, **dev), torch.zeros(N, dtype=torch.int32, **dev),
                        torch.zeros((N, 2), dtype=torch.int32, **dev), torch.zeros(N, **dev))
                stream.synchronize()
                start.wait(30)
                for _ in range(rounds):
                    try:
                        rp.rptq_fold_reorder(None, None, k, np.arange(k, dtype=np.int32), off, [1.0, 1.0], [0, 0], W, N, k, None,
                                             perm_pad, None, None, Wq, *args)
                    except rp.RptqError as e:
                        assert e.status == -6
                        bad_calls[bad] += 1
        except BaseException as e:
            errors.append(e)

    threads = [threading.Thread(target=work, args=(b,)) for b in (True, False)]
    for t in threads:
        t.start()
    for t in threads:
        t.join(60)
    assert not errors, errors
    assert bad_calls == {True: rounds, False: 0}


@pytest.mark.parametrize("cw", [False, True])
def test_fold_is_not_recorded(cw):
    """Under stream capture both folds are refused with nothing in the graph (they copy from host arrays and wait)."""
    import paper_2304_01089_amd as rp
    rp.load_library()
    k, N = 4096, 64
    off = np.array([0, 1000, k], np.int32)
    dev = dict(device="cuda")
    W = torch.full((N, k), 0.5, **dev)
    perm_pad = torch.full((rp.rptq_padded_k(off),), 7, dtype=torch.int32, **dev)
    Wq = torch.full((rp.rptq_weight_bytes(N, perm_pad.numel()),), 0x5A, dtype=torch.uint8, **dev)
    sW, zW, wsum = torch.zeros((N, 2), **dev), torch.full((N, 2), 7, dtype=torch.int32, **dev), torch.zeros((N, 2), dtype=torch.int32, **dev)
    ct, probe = torch.zeros(N, **dev), torch.zeros(1, **dev)
    tabs = [torch.zeros(n // 4, **dev) for n in (rp.rptq_cw_scale_bytes(N, 2), rp.rptq_cw_cross_bytes(N, 2))]
    perm = np.arange(k, dtype=np.int32)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        probe.add_(1.0)
        with pytest.raises(rp.RptqError) as e:
            if cw:
                rp.rptq_fold_reorder_cw(perm, off, [1.0, 1.0], [0, 0], W, N, k, np.arange(N, dtype=np.int32), perm_pad, Wq, sW, zW, wsum, *tabs, ct)
            else:
                rp.rptq_fold_reorder(None, None, k, perm, off, [1.0, 1.0], [0, 0], W, N, k, np.arange(N, dtype=np.int32), perm_pad,
                                     None, None, Wq, sW, zW, wsum, ct)
        assert e.value.status == -9
    graph.replay()
    torch.cuda.synchronize()
    assert probe.item() == 1.0
    assert (perm_pad == 7).all() and (Wq == 0x5A).all() and (zW == 7).all()

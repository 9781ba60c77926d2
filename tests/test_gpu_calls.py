"""The native marshalling of the serving entry points and the Python one behind it: the same calls, the same errors."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
import paper_2304_01089_amd as rp  # noqa: E402


def test_tensors_that_are_not_on_the_device_are_refused():
    rp.load_library()
    t = torch.zeros(4, 32, dtype=torch.bfloat16)
    for call in (lambda: rp.rptq_kv_quant(t, 4, 32, t, 4, t), lambda: rp.rptq_kv_dequant(None, 4, 32, t, 4, t),
                 lambda: rp.rptq_cluster_gemm(t, 4, 4, t, 8, [0, 32], [1.0], t, t, t, t, t),
                 lambda: rp.rptq_cluster_gemm_quant(t, 4, 4, t, 8, [0, 32], [1.0], t, t, t, t, 1, [0, 32], [1.0], [1.0], [0], 4, t, t, None)):
        with pytest.raises(ValueError):
            call()


@pytest.mark.gpu
def test_ordinary_and_other_arguments_give_the_same():
    d, M, N, g, bits, dev = 264, 5, 96, 4, 4, dict(device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(1)
    x = torch.randn(M, d, generator=gen, **dev).bfloat16()
    cal = rp.calibrate_site([x], None, None, 1e-5, True, g, bits, seed=1)
    lin = rp.fold_linear(cal, torch.randn(N, d, generator=gen, **dev))

    def step(off, s, inv, z, m, eps, relu, stream):
        codes = torch.zeros(rp.rptq_codes_bytes(M, cal.k_padded, bits), dtype=torch.uint8, **dev)
        rt, y = torch.zeros(M, **dev), torch.zeros(M, N, **dev)
        rp.rptq_ln_quant(x, m, d, None, None, eps, relu, cal.perm_pad, off, s, inv, z, bits, codes, None, rt, stream)
        rp.rptq_cluster_gemm(codes, m, bits, lin.Wq, N, off, s, lin.sW, lin.zW, lin.colterm, rt, y, stream)
        torch.cuda.synchronize()
        return codes, rt, y
    off, s, inv, z = cal.cluster_off, cal.s, cal.inv_s, cal.z
    want = step(off, s, inv, z, M, 1e-5, True, None)
    assert want[2].abs().max() > 0
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    for args in ((list(off), list(s), list(inv), list(z), M, 1, 1, None),
                 (off.astype(np.int64), s.astype(np.float64), np.repeat(inv, 2)[::2], z[None, :].astype(np.int16)[0], M, 1e-5, np.bool_(True), None),
                 (off, s, inv, z, M, 1e-5, True, stream), (off, s, inv, z, M, 1e-5, True, stream.cuda_stream)):
        got = step(*args)
        assert all(torch.equal(a, b) for a, b in zip(want, got))
    with torch.cuda.stream(stream):                            # the current stream is looked up on every call
        assert all(torch.equal(a, b) for a, b in zip(want, step(off, s, inv, z, M, 1e-5, True, None)))
    wrong = dict(dtype=torch.float32, **dev)
    with pytest.raises(ValueError, match="dtype"):
        rp.rptq_ln_quant(x.float(), M, d, None, None, 1e-5, True, cal.perm_pad, off, s, inv, z, bits, torch.zeros(1, **wrong))
    with pytest.raises(ValueError, match="contiguous"):
        rp.rptq_ln_quant(x[:, ::2], M, d, None, None, 1e-5, True, cal.perm_pad, off, s, inv, z, bits, torch.zeros(1, **wrong))
    with pytest.raises(ValueError, match="bf16 or fp32"):
        rp.rptq_cluster_gemm(want[0], M, bits, lin.Wq, N, off, s, lin.sW, lin.zW, lin.colterm, want[1], want[0])
    with pytest.raises(rp.RptqError):
        rp.rptq_ln_quant(x, M, d, None, None, 1e-5, True, cal.perm_pad, off, s, inv, z, 5, want[0])

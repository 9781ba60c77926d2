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


NAMES = ("ln_quant", "cluster_gemm", "cluster_gemm_quant", "cluster_rowsums", "cluster_gemm_cw", "kv_quant", "kv_dequant")


def test_the_native_marshalling_is_there():
    from paper_2304_01089_amd import binding
    rp.load_library()
    rp.rptq_padded_k([0, 32])                                  # (finds it if the library was loaded before torch)
    assert binding._CALLS is not None and all(hasattr(binding._CALLS, n) for n in NAMES)


def ordinary_calls():
    """The arguments of every entry point that is marshalled natively, as tensors and tables, with the tensors it writes."""
    d, M, N, g, bits, heads, dev = 264, 5, 96, 4, 4, 4, dict(device="cuda")
    gen = torch.Generator(device="cuda").manual_seed(2)
    x = torch.randn(M, d, generator=gen, **dev).bfloat16()
    W = torch.randn(N, d, generator=gen, **dev)
    gamma, beta = torch.exp(0.1 * torch.randn(d, generator=gen, **dev)), torch.randn(d, generator=gen, **dev)
    cal = rp.calibrate_site([x], gamma, beta, 1e-5, False, g, bits, seed=1)
    nxt = rp.calibrate_site([(x.float() @ W.T).bfloat16()], None, None, 1e-5, True, g, bits, seed=2)
    lin, fused, cw = rp.fold_linear(cal, W), rp.fold_linear(cal, W, next_site=nxt), rp.fold_linear_cw(cal, W)
    codes, xsum, rt = rp.ln_quant(cal, x, 1e-5, want_xsum=True)
    sums = rp.cluster_rowsums(cal, codes, M)
    y, y32 = torch.empty(M, N, dtype=torch.bfloat16, **dev), torch.empty(M, N, **dev)
    c2 = torch.empty(rp.rptq_codes_bytes(M, nxt.k_padded, bits), dtype=torch.uint8, **dev)
    r2, ws = torch.empty(M, **dev), torch.zeros(max(16, rp.rptq_cluster_gemm_quant_workspace_bytes(M, fused.N)), dtype=torch.uint8, **dev)
    width = 64
    xk = torch.randn(M, heads * width, generator=gen, **dev).bfloat16()
    table = torch.empty(rp.rptq_kv_table_bytes(heads * width), dtype=torch.uint8, **dev)
    s = np.full((heads, 2), 0.25, np.float32)
    rp.rptq_kv_tables(np.arange(heads * width, dtype=np.int32), np.tile(np.array([0, 20, width], np.int32), (heads, 1)), s, 1 / s,
                      np.zeros((heads, 2), np.int32), heads * width, heads, 2, table)
    ck = torch.empty(M * heads * width * bits // 8, dtype=torch.uint8, **dev)
    ck_in = torch.randint(0, 256, ck.shape, dtype=torch.uint8, generator=gen, **dev)
    back = torch.empty_like(xk)
    c1, x1, r1, sums1 = (torch.empty_like(t) for t in (codes, xsum, rt, sums))
    off, sx, inv, z = cal.cluster_off, cal.s, cal.inv_s, cal.z
    return [
        ("ln_quant", (x, M, d, cal.gamma_pad, cal.beta_pad, 1e-5, False, cal.perm_pad, off, sx, inv, z, bits, c1, x1, r1, None), (c1, x1, r1)),
        ("ln_quant", (x, M, d, cal.gamma_pad, cal.beta_pad, 1e-5, True, cal.perm_pad, off, sx, inv, z, bits, c1, None, r1, None), (c1, r1)),
        ("cluster_gemm", (codes, M, bits, lin.Wq, N, off, sx, lin.sW, lin.zW, lin.colterm, rt, y, None), (y,)),
        ("cluster_gemm", (codes, M, bits, lin.Wq, N, off, sx, lin.sW, lin.zW, lin.colterm, rt, y32, None), (y32,)),
        ("cluster_gemm_quant", (codes, M, bits, fused.Wq, fused.N, off, sx, fused.sW, fused.zW, fused.colterm, rt, True,
                                nxt.cluster_off, nxt.s, nxt.inv_s, nxt.z, bits, c2, r2, ws, None), (c2, r2)),
        ("cluster_rowsums", (codes, M, bits, off, sx, z, sums1, None), (sums1,)),
        ("cluster_gemm_cw", (codes, M, bits, cw.Wq, N, off, cw.scale_tab, cw.cross_tab, cw.colterm, sums, y, None), (y,)),
        ("cluster_gemm_cw", (codes, M, bits, cw.Wq, N, off, cw.scale_tab, cw.cross_tab, cw.colterm, sums, y32, None), (y32,)),
        ("kv_quant", (xk, M, heads * width, table, bits, ck, None), (ck,)),
        ("kv_dequant", (ck_in, M, heads * width, table, bits, back, None), (back,)),
    ]


@pytest.mark.gpu
def test_every_entry_point_marshals_natively_as_in_python(monkeypatch):
    """Ordinary arguments are taken (a status, and the outputs that the Python marshalling leads to), in every entry point;
    an argument out of the ordinary, whichever it is, is not (None, and no output touched)."""
    from paper_2304_01089_amd import binding
    calls, taken = ordinary_calls(), set()
    for name, args, outs in calls:
        native, entry = getattr(binding._CALLS, name), getattr(rp, "rptq_" + name)
        for t in outs:
            t.view(torch.uint8).fill_(0x5a)
        assert native(*args) == 0, name
        got = [t.clone() for t in outs]
        for t in outs:
            t.view(torch.uint8).fill_(0xa5)
        with monkeypatch.context() as m:
            m.setattr(binding, "_CALLS", None)
            m.setattr(binding, "_CALLS_SOUGHT", True)
            entry(*args)
        assert all(torch.equal(a.view(torch.uint8), b.view(torch.uint8)) for a, b in zip(got, outs)), name
        for t in outs:
            t.view(torch.uint8).fill_(0x3c)
        torch.cuda.synchronize()
        for i, a in enumerate(args):
            if isinstance(a, torch.Tensor):
                odd = [a.cpu(), torch.cat([a, a])[::2], 1]
                if a.dtype != torch.uint8:                     # (bytes: any type of element is taken)
                    odd.append(a.double())
                if name != "ln_quant" or i not in (3, 4, 14, 15):      # (NULL is an ordinary value there)
                    odd.append(None)
            elif isinstance(a, np.ndarray):
                odd = [a.tolist(), a.astype(a.dtype.str.replace("4", "8")), a.view(np.uint32), np.repeat(a, 2)[::2], a[None], a.tobytes(), None]
            elif a is None:
                odd = [torch.cuda.current_stream(), 1.0] if i == len(args) - 1 else [1]
            elif isinstance(a, bool):
                odd = [1, np.bool_(True)]
            elif isinstance(a, float):
                odd = [1, np.float32(1e-5)]
            else:
                odd = [float(a), np.int64(a), 1 << 80]
            for o in odd:
                assert native(*args[:i], o, *args[i + 1:]) is None, (name, i, o)
        assert native(*args[:-1]) is None and native(*args, None) is None, name
        torch.cuda.synchronize()
        assert all((t.view(torch.uint8) == 0x3c).all() for t in outs), name
        taken.add(name)
    assert taken == set(NAMES)

"""What a program may record without having run the very same call before: products of more than 32 rows after one such
product of any size, products of up to 32 rows at once.  Each case is a process of its own, since the driver set-up that
the first call of a process does is what matters."""
import os
import subprocess
import sys

import pytest

pytestmark = pytest.mark.gpu
pytest.importorskip("torch")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

PROGRAM = r"""
import sys
import numpy as np, torch
import paper_2304_01089_amd as rp
what = sys.argv[1]
d, N, g, bits, dev = 1024, 5376, 16, 4, dict(device="cuda")
gen = torch.Generator(device="cuda").manual_seed(3)
x = torch.randn(2900, d, generator=gen, **dev).bfloat16()
cal = rp.calibrate_site([x[:256]], None, None, 1e-5, False, g, bits, seed=1)
W = 0.02 * torch.randn(N, d, generator=gen, **dev)
codes, _, rt = rp.ln_quant(cal, x, 1e-5)

if what == "cw":
    lin = rp.fold_linear_cw(cal, W)
    sums = rp.cluster_rowsums(cal, codes, len(x))
    outs = lambda m: dict(y=torch.zeros(m, N, dtype=torch.bfloat16, **dev))
    call = lambda m, o: rp.cluster_gemm_cw(cal, lin, codes, sums, m, y=o["y"])
elif what == "quant":
    nxt = rp.calibrate_site([(x[:256].float() @ W.T).bfloat16()], None, None, 1e-5, True, g, bits, seed=2)
    lin = rp.fold_linear(cal, W, next_site=nxt)
    ws = torch.zeros(rp.rptq_cluster_gemm_quant_workspace_bytes(len(x), lin.N), dtype=torch.uint8, **dev)
    outs = lambda m: dict(c=torch.zeros(rp.rptq_codes_bytes(m, nxt.k_padded, bits), dtype=torch.uint8, **dev), r=torch.zeros(m, **dev))
    call = lambda m, o: rp.cluster_gemm_quant(cal, lin, codes, rt, m, nxt, relu=True, next_codes=o["c"], next_rowterm=o["r"], workspace=ws)
else:
    lin = rp.fold_linear(cal, W)
    dt = torch.float32 if what == "f32" else torch.bfloat16
    outs = lambda m: dict(y=torch.zeros(m, N, dtype=dt, **dev))
    call = lambda m, o: rp.cluster_gemm(cal, lin, codes, rt, m, y=o["y"])

first, sizes = (None, (32, 16, 1)) if what == "decode" else (40, (2900, 1500, 300, 33))
if first:
    call(first, outs(first))
torch.cuda.synchronize()
for m in sizes:
    o = outs(m)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        call(m, o)
    e = outs(m)
    call(m, e)
    for _ in range(2):
        for t in o.values():
            t.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(o[k], e[k]) for k in o), m
    print("recorded", what, m, flush=True)
print("ok")
"""


@pytest.mark.parametrize("what", ["bf16", "f32", "quant", "cw", "decode"])
def test_record_without_the_same_call_before(what):
    r = subprocess.run([sys.executable, "-u", "-c", PROGRAM, what], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr


@pytest.mark.parametrize("what", ["bf16", "f32", "quant"])
def test_record_the_first_product_of_a_process(what):
    """525 tiles of 64 x 256 (and 550 of the padded next site), 8-bit codes, K = 5120: where no call has raised the LDS limit of
    that tile, smaller ones serve a product of one to 1.4 rounds of it."""
    program = PROGRAM.replace("1024, 5376, 16, 4", "5120, 5376, 16, 8").replace("(40, (2900, 1500, 300, 33))", "(None, (1600,))")
    r = subprocess.run([sys.executable, "-u", "-c", program, what], cwd=ROOT, capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok") and "recorded %s 1600" % what in r.stdout, r.stdout + r.stderr

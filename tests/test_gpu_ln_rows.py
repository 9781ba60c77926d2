"""The LayerNorm + quantize kernel for few rows per compute unit against the pipelined one, at the edges of its rule: a
row's codes and row sum do not depend, bit for bit, on how many rows share its call.  (The oracle's tests run both.)"""
import os
import subprocess
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def rows_per_unit(d, bits, ln):
    """The rule: up to so many rows per compute unit."""
    if bits == 3:
        return 16 if d <= 3072 else 8 if d <= 5120 else 4
    if d <= 2048:
        return 64 if ln else 32 if d <= 640 else 64 if d <= 1792 else 128
    return 32 if d <= (4096 if bits == 4 else 3072) else 16 if d <= 5120 else 4


def make_call(d, g, bits, M, seed=3, ln=True):
    import paper_2304_01089_amd as rp
    rng = np.random.default_rng(seed + d + g)
    cuts = np.sort(rng.choice(np.arange(1, d), g - 1, replace=False)) if g > 1 else []
    off = np.concatenate([[0], cuts, [d]]).astype(np.int32)
    s = np.exp(rng.normal(-1, 0.5, g)).astype(np.float32)
    inv = (1.0 / s.astype(np.float64)).astype(np.float32)
    z = rng.integers(-3, 4, g).astype(np.int32)
    z[0] = -(1 << 21) if g > 1 else 0                          # (the largest zero point: every code of the cluster saturates)
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
@pytest.mark.parametrize("d,g", [(8, 1), (776, 64), (2048, 16), (2056, 9), (5120, 32), (8184, 32), (12288, 33), (15000, 8)])
def test_few_rows_equal_many(d, g, bits, ln):
    import paper_2304_01089_amd as rp
    most = rows_per_unit(d, bits, ln)
    cus = rp.rptq_device_info()["compute_units"]
    many = cus * most + 1
    call = make_call(d, g, bits, many, ln=ln)
    codes, rowterm = call(many)
    assert codes[1:].unique().numel() > 4 and rowterm[1:].unique().numel() > 4      # (rows that differ, none saturated throughout)
    for m in sorted({1, 2, 3, cus, cus + 1, 2 * cus, 2 * cus + 1, 2 * cus + 3, cus * most}):
        c, r = call(m)
        assert torch.equal(c, codes[:m]), m
        assert torch.equal(r, rowterm[:m]), m


@pytest.mark.parametrize("ln", [True, False])
@pytest.mark.parametrize("bits", [3, 4, 8])
@pytest.mark.parametrize("d,g", [(776, 8), (1536, 7), (2048, 16), (2560, 8), (4072, 32), (5120, 32), (8064, 4)])
def test_rows_of_a_workgroup(d, g, bits, ln):
    """One, two or four rows in a workgroup: either side of every line of that rule (rows per compute unit)."""
    import paper_2304_01089_amd as rp
    cus = rp.rptq_device_info()["compute_units"]
    most = min(12, rows_per_unit(d, bits, ln))
    call = make_call(d, g, bits, cus * most, ln=ln)
    codes, rowterm = call(cus * most)
    for m in (cus * line + k for line in range(1, most) for k in (-1, 0, 1)):
        c, r = call(m)
        assert torch.equal(c, codes[:m]) and torch.equal(r, rowterm[:m]), m


@pytest.mark.parametrize("ln", [True, False])
@pytest.mark.parametrize("bits", [3, 8])
@pytest.mark.parametrize("d", [264, 776, 2056, 5120, 12288])
def test_sums_that_show_their_order(d, bits, ln):
    """Rows whose 64-bit sums lose what is added while a pair of huge terms is open: with LayerNorm the mean of a few pairs
    +-2^58 among ordinary values (codes of the ordinary values follow it: scale 2^-58), without it the row sum over two
    outer clusters of scale 2^58.  The same bits still, in both kernels."""
    import paper_2304_01089_amd as rp
    dev, M, rng = dict(device="cuda"), rp.rptq_device_info()["compute_units"] * rows_per_unit(d, bits, ln) + 1, np.random.default_rng(d + bits)
    gen = torch.Generator(device="cuda").manual_seed(d)
    off = np.array([0, 40, d - 40, d], np.int32)
    big = 2.0 ** 58
    s = np.array([1, 1, 1] if ln else [big, 1, big], np.float32) / np.float32(big / d ** 0.5 if ln else 1)
    inv, z = (1.0 / s.astype(np.float64)).astype(np.float32), np.zeros(3, np.int32)
    perm_pad = torch.zeros(rp.rptq_padded_k(off), dtype=torch.int32, **dev)
    gp, bp = (torch.zeros(len(perm_pad), **dev) for _ in range(2)) if ln else (None, None)
    one, nil = (torch.ones(d, **dev), torch.zeros(d, **dev)) if ln else (None, None)
    perm = rng.permutation(d).astype(np.int32) if ln else np.arange(d, dtype=np.int32)
    rp.rptq_fold_reorder(one, nil, d, perm, off, None, None, None, 0, d, None, perm_pad, gp, bp, None, None, None, None, None)
    x = torch.randn(M, d, generator=gen, **dev) + 0.7
    ends = [np.arange(d)] * 2 if ln else [np.arange(40), np.arange(d - 40, d)]
    for sign, where in zip((1, -1), ends):                     # (the positive halves and the negative ones: disjoint)
        for k in range(4):
            lane = torch.from_numpy(where[(sign < 0) + 2 * k::8]).cuda()
            x[torch.arange(M, **dev), lane[torch.randint(len(lane), (M,), generator=gen, **dev)]] = sign * big
    x = x.bfloat16()

    def call(m):
        codes, rowterm = torch.zeros((m, len(perm_pad) * bits // 8), dtype=torch.uint8, **dev), torch.zeros(m, **dev)
        rp.rptq_ln_quant(x, m, d, gp, bp, 1e-5, False, perm_pad, off, s, inv, z, bits, codes, None, rowterm)
        return codes, rowterm
    codes, rowterm = call(M)
    for m in (1, 2, 3, 300, 600, M - 1):
        c, r = call(m)
        assert torch.equal(c, codes[:m]) and torch.equal(r, rowterm[:m]), m


PROGRAM = r"""
import sys
sys.path.insert(0, "tests")
import torch
from test_gpu_ln_rows import make_call
d, bits, first, m = (int(v) for v in sys.argv[1:])
call = make_call(d, 32, bits, 2000)
outs = [torch.zeros((m,) + t.shape[1:], dtype=t.dtype, device="cuda") for t in call(first)]
torch.cuda.synchronize()
graph = torch.cuda.CUDAGraph()
with torch.cuda.graph(graph):
    call(m, *outs)
codes, rowterm = call(2000)
for _ in range(3):
    for t in outs:
        t.zero_()
    graph.replay()
    torch.cuda.synchronize()
    assert torch.equal(outs[0], codes[:m]) and torch.equal(outs[1], rowterm[:m])
    call(m)
print("ok")
"""


@pytest.mark.parametrize("d,bits,first,m", [(12288, 4, 1, 600), (12288, 4, 2000, 600), (12288, 3, 300, 1), (5120, 8, 1, 2000)])
def test_recorded_call_of_another_size(d, bits, first, m):
    """Several wide rows per workgroup need more LDS than a kernel has by default.  A call that is recorded after one of
    another size (`first` rows, with either kernel) leaves the same bits.  Each case is a process of its own: raised limits
    last as long as it does."""
    r = subprocess.run([sys.executable, "-u", "-c", PROGRAM, str(d), str(bits), str(first), str(m)], cwd=ROOT,
                       capture_output=True, text=True, timeout=100)
    assert r.returncode == 0 and r.stdout.strip().endswith("ok"), r.stdout + r.stderr

"""The cases that the speed of this framework is measured on: what a program that serves (or prepares) an
RPTQ-quantized model calls, from one decoded token to the largest prefill, and the offline preparation.

A case is a dict of plain values; `kind` says which path it takes:

  linear   LayerNorm + quantize (rptq.ln_quant), then one linear layer (cluster_gemm): an attention or FFN input site
  ffn      LayerNorm + quantize, fc1 with the next site's quantizer in its output stage, fc2 on those codes
  cw       linear, with one weight parameter pair per (output channel, input cluster)
  kv       key and value cache of one layer: T new rows quantized and stored, S rows read back
  offline  calibration of a site and folding / quantizing of the weights that read it

Inputs follow the channel structure that the method is about: a few channels with a far wider range, ranges away
from zero; weights N(0, 0.02).  Everything comes from one torch generator seeded by the seed.
"""
from __future__ import annotations

import math
from types import SimpleNamespace

import numpy as np
import torch

import paper_2304_01089_amd as rp

EPS = 1e-5
CAL_ROWS = 128


def listed():
    return [
        # the smallest layer: a 768-wide model's first FFN layer on a short prompt, 8-bit activations
        dict(name="linear_m128_d768_a8", kind="linear", M=128, d=768, g=8, bits=8, N=3072, out="bf16"),
        # one sequence decoding one token on a 2048-wide layer: latency and launches
        dict(name="linear_m1_d2048_a4", kind="linear", M=1, d=2048, g=16, bits=4, N=8192, out="bf16"),
        # sixteen sequences decoding on the largest layer: the weights are streamed once
        dict(name="linear_m16_d12288_a3", kind="linear", M=16, d=12288, g=32, bits=3, N=49152, out="bf16"),
        # an ordinary prefill on a 2048-wide layer
        dict(name="linear_m2048_d2048_a4", kind="linear", M=2048, d=2048, g=16, bits=4, N=8192, out="bf16"),
        # a prompt of an odd length into an odd number of fp32 outputs
        dict(name="linear_m333_d4072_a3_f32", kind="linear", M=333, d=4072, g=32, bits=3, N=4099, out="f32"),
        # the largest prefill
        dict(name="linear_m8192_d12288_a3", kind="linear", M=8192, d=12288, g=32, bits=3, N=49152, out="bf16"),
        # a 5120-wide FFN: prefill, and a batch of thirty-two decoding sequences
        dict(name="ffn_m4096_d5120_a4", kind="ffn", M=4096, d=5120, dff=20480, g=32, bits=4, out="bf16"),
        dict(name="ffn_m32_d5120_a4", kind="ffn", M=32, d=5120, dff=20480, g=32, bits=4, out="bf16"),
        # the finer weight parameters on an attention output-sized layer
        dict(name="cw_m2048_d5120_a4", kind="cw", M=2048, d=5120, g=32, bits=4, N=5120, out="bf16"),
        # key/value cache: a whole prompt written and read, and a batch of sixteen sequences one token further
        dict(name="kv_t8192_d12288_b3", kind="kv", T=8192, S=8192, heads=96, width=128, g=4, bits=3),
        dict(name="kv_t16_d2048_b4", kind="kv", T=16, S=4096, heads=32, width=64, g=4, bits=4),
        # preparing a 2048-wide layer: calibration on sixteen batches, K-Means, weights folded and packed
        dict(name="offline_d2048_n8192_a4", kind="offline", d=2048, g=16, bits=4, N=8192, batches=16, cw=False),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _log_int(rng, lo, hi, step=1):
    return min(hi, max(lo, int(round(_log(rng, lo, hi) / step)) * step))


def _rows(rng, most):
    """Tokens of a call: decode batches, short and long prompts alike, round and ragged."""
    m = _log_int(rng, 1, most)
    return m if rng.random() < 0.6 or m < 48 else max(32, m // 32 * 32)


def draw(rng):
    kind = rng.choice(["linear", "linear", "linear", "linear", "ffn", "ffn", "cw", "kv", "kv", "offline"])
    bits = rng.choice([3, 4, 4, 8])
    out = rng.choice(["bf16", "bf16", "f32"])
    if kind == "kv":
        width = rng.choice([64, 128])
        heads = _log_int(rng, 768 // width, 12288 // width)
        heads += (heads * width) % 128 // 64                     # (whole 16-byte rows at 3 bits)
        T = _log_int(rng, 1, 8192)
        S = min(8192, max(T, _log_int(rng, 64, 8192)))
        return dict(kind="kv", T=T, S=S, heads=heads, width=width, g=4, bits=bits)
    if kind == "offline":
        d = _log_int(rng, 768, 5120, 8)
        return dict(kind="offline", d=d, g=rng.choice([8, 16, 32]), bits=bits, N=_log_int(rng, 512, 4 * d),
                    batches=rng.choice([4, 16]), cw=rng.random() < 0.3)
    if kind == "ffn":
        d = _log_int(rng, 768, 5120, 8)
        return dict(kind="ffn", M=_rows(rng, 4096), d=d, dff=min(20480, 4 * d), g=rng.choice([8, 16, 32]), bits=bits, out=out)
    top = 12288 if kind == "linear" else 5120
    d = _log_int(rng, 768, top, 8)
    g = 8 if d < 1024 else rng.choice([16, 32])
    N = _log_int(rng, 512, 4 * d)
    if rng.random() < 0.6:
        N = max(512, N // 64 * 64)
    return dict(kind=kind, M=_rows(rng, 8192 if kind == "linear" else 4096), d=d, g=g, bits=bits, N=N, out=out)


# ---- inputs ----------------------------------------------------------------------------------------
def _normal(gen, *shape):
    return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float32)


def _channels(gen, d):
    s_c = torch.exp(_normal(gen, d))
    wide = torch.randperm(d, generator=gen, device="cuda")[: round(0.01 * d)]
    s_c[wide] *= 30.0
    return _normal(gen, d) * (2.0 * s_c), s_c


def _batch(gen, m_c, s_c, rows):
    return (m_c + s_c * _normal(gen, rows, m_c.shape[0])).to(torch.bfloat16)


def _site(gen, case, batches=4):
    d = case["d"]
    m_c, s_c = _channels(gen, d)
    gamma = torch.exp(0.3 * _normal(gen, d))
    beta = 0.1 * _normal(gen, d)
    cal = [_batch(gen, m_c, s_c, CAL_ROWS) for _ in range(batches)]
    return m_c, s_c, gamma, beta, cal


def _weights(gen, N, K):
    return _normal(gen, N, K).mul_(0.02)


def _bytes(n):
    return torch.zeros(max(16, n), dtype=torch.uint8, device="cuda")


def _most_padded(d, g):
    """The padded width of a site depends on its clusters: buffers are made for the widest (then they have one size)."""
    return (d + 31 * g + 255) // 256 * 256


def _out(case, N):
    return torch.empty((case["M"], N), dtype=torch.float32 if case["out"] == "f32" else torch.bfloat16, device="cuda")


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed) * 1000003 + 17)
    kind = case["kind"]
    st = SimpleNamespace(kind=kind, case=case)
    if kind == "offline":
        d, g, N = case["d"], case["g"], case["N"]
        _, _, st.gamma, st.beta, st.cal = _site(gen, case, case["batches"])
        st.W = _weights(gen, N, d)
        st.seed = int(seed) & 0xffff
        st.scratch = _bytes(rp.rptq_calibrate_workspace_bytes(d))
        kp = _most_padded(d, g)
        st.perm_pad = torch.zeros(kp, dtype=torch.int32, device="cuda")
        st.gamma_pad, st.beta_pad = (torch.zeros(kp, dtype=torch.float32, device="cuda") for _ in range(2))
        per_row = N * g if case["cw"] else N
        st.Wq = _bytes(rp.rptq_weight_bytes(N, kp))
        st.sW, st.zW, st.wsum, st.colterm = (torch.zeros(n, dtype=t, device="cuda") for n, t in (
            (per_row, torch.float32), (per_row, torch.int32), (N * g, torch.int32), (N, torch.float32)))
        if case["cw"]:
            st.scale_tab = torch.zeros(rp.rptq_cw_scale_bytes(N, g) // 4, dtype=torch.float32, device="cuda")
            st.cross_tab = torch.zeros(rp.rptq_cw_cross_bytes(N, g) // 4, dtype=torch.float32, device="cuda")
        return st
    if kind == "kv":
        d, H, g, bits = case["heads"] * case["width"], case["heads"], case["g"], case["bits"]
        st.x, st.codes, st.tables, st.back, points = [], [], [], [], []
        for _ in range(3):                                       # queries, keys, values
            m_c, s_c = _channels(gen, d)
            cal = _batch(gen, m_c, s_c, 4 * CAL_ROWS).float()
            points.append((cal.amin(0).cpu().numpy() + np.float32(0), cal.amax(0).cpu().numpy() + np.float32(0), m_c, s_c))
        q, k, v = points
        shared = rp.rptq_cluster_heads([q[0], k[0]], [q[1], k[1]], H, g, bits, seed=int(seed) & 0xffff)
        alone = rp.rptq_cluster_heads([v[0]], [v[1]], H, g, bits, seed=(int(seed) + 1) & 0xffff)
        for hc, which, (_, _, m_c, s_c) in ((shared, 1, k), (alone, 0, v)):
            table = _bytes(rp.rptq_kv_table_bytes(d))
            rp.rptq_kv_tables(hc["perm"], hc["cluster_off"], hc["s"][which], hc["inv_s"][which], hc["z"][which], d, H, g, table)
            codes = torch.empty((case["S"], d * bits // 8), dtype=torch.uint8, device="cuda")
            rp.rptq_kv_quant(_batch(gen, m_c, s_c, case["S"]), case["S"], d, table, bits, codes)      # the context so far
            st.tables.append(table)
            st.codes.append(codes)
            st.x.append(_batch(gen, m_c, s_c, case["T"]))
            st.back.append(torch.empty((case["S"], d), dtype=torch.bfloat16, device="cuda"))
        st.new = [c[case["S"] - case["T"]:] for c in st.codes]   # where the new rows go
        return st
    M, bits, g, d = case["M"], case["bits"], case["g"], case["d"]
    m_c, s_c, gamma, beta, cal = _site(gen, case)
    st.cal = rp.calibrate_site(cal, gamma, beta, EPS, False, g, bits, seed=int(seed) & 0xffff)
    st.x = _batch(gen, m_c, s_c, M)
    st.codes = _bytes(rp.rptq_codes_bytes(M, _most_padded(d, g), bits))
    st.rowterm = torch.empty(M, dtype=torch.float32, device="cuda")
    if kind == "ffn":
        W1, W2 = _weights(gen, case["dff"], d), _weights(gen, d, case["dff"])
        hidden = [(torch.nn.functional.layer_norm(b.float(), (d,), gamma, beta, EPS) @ W1.T).to(torch.bfloat16) for b in cal]
        st.next = rp.calibrate_site(hidden, None, None, EPS, True, g, bits, seed=(int(seed) + 1) & 0xffff)
        st.fc1 = rp.fold_linear(st.cal, W1, next_site=st.next)
        st.fc2 = rp.fold_linear(st.next, W2)
        st.codes2 = _bytes(rp.rptq_codes_bytes(M, _most_padded(case["dff"], g), bits))
        st.rowterm2 = torch.empty(M, dtype=torch.float32, device="cuda")
        st.workspace = _bytes(rp.rptq_cluster_gemm_quant_workspace_bytes(M, st.fc1.N))
        st.y = _out(case, d)
    elif kind == "cw":
        st.lin = rp.fold_linear_cw(st.cal, _weights(gen, case["N"], d))
        st.rowsums = torch.empty(max(4, rp.rptq_cw_rowsum_bytes(M, st.cal.g_eff) // 4), dtype=torch.float32, device="cuda")
        st.y = _out(case, case["N"])
    else:
        st.lin = rp.fold_linear(st.cal, _weights(gen, case["N"], d))
        st.y = _out(case, case["N"])
    return st


# ---- one pass ----------------------------------------------------------------------------------------
def run(st):
    case = st.case
    if st.kind == "offline":
        d, N = case["d"], case["N"]
        r = rp.rptq_calibrate(st.cal, st.gamma, st.beta, EPS, False, case["g"], case["bits"], st.seed, workspace=st.scratch)
        perm, off, s, z = r["perm"], r["cluster_off"], r["s"], r["z"]
        none = None
        if case["cw"]:
            rp.rptq_fold_reorder(st.gamma, st.beta, d, perm, off, none, none, none, 0, d, none, st.perm_pad, st.gamma_pad,
                                 st.beta_pad, none, none, none, none, none)
            rp.rptq_fold_reorder_cw(perm, off, s, z, st.W, N, d, none, st.perm_pad, st.Wq, st.sW, st.zW, st.wsum,
                                    st.scale_tab, st.cross_tab, st.colterm)
        else:
            rp.rptq_fold_reorder(st.gamma, st.beta, d, perm, off, s, z, st.W, N, d, none, st.perm_pad, st.gamma_pad,
                                 st.beta_pad, st.Wq, st.sW, st.zW, st.wsum, st.colterm)
        out = dict(r, perm_pad=st.perm_pad, gamma_pad=st.gamma_pad, beta_pad=st.beta_pad,
                   Wq=st.Wq, sW=st.sW, zW=st.zW, wsum=st.wsum, colterm=st.colterm)
        if case["cw"]:
            out.update(scale_tab=st.scale_tab, cross_tab=st.cross_tab)
        return out
    if st.kind == "kv":
        d, bits = case["heads"] * case["width"], case["bits"]
        for x, new, table in zip(st.x, st.new, st.tables):
            rp.rptq_kv_quant(x, case["T"], d, table, bits, new)
        for codes, table, back in zip(st.codes, st.tables, st.back):
            rp.rptq_kv_dequant(codes, case["S"], d, table, bits, back)
        return dict(key=st.back[0], value=st.back[1], key_codes=st.new[0], value_codes=st.new[1])
    M = case["M"]
    codes, _, rowterm = rp.ln_quant(st.cal, st.x, EPS, codes=st.codes, rowterm=st.rowterm)
    if st.kind == "ffn":
        codes2, rowterm2 = rp.cluster_gemm_quant(st.cal, st.fc1, codes, rowterm, M, st.next, relu=True, next_codes=st.codes2,
                                                 next_rowterm=st.rowterm2, workspace=st.workspace)
        y = rp.cluster_gemm(st.next, st.fc2, codes2, rowterm2, M, y=st.y)
        return dict(y=y, codes=codes, rowterm=rowterm, codes2=codes2, rowterm2=rowterm2)
    if st.kind == "cw":
        rowsums = rp.cluster_rowsums(st.cal, codes, M, rowsums=st.rowsums)
        y = rp.cluster_gemm_cw(st.cal, st.lin, codes, rowsums, M, y=st.y)
        return dict(y=y, codes=codes, rowterm=rowterm, rowsums=rowsums)
    y = rp.cluster_gemm(st.cal, st.lin, codes, rowterm, M, y=st.y)
    return dict(y=y, codes=codes, rowterm=rowterm)


# ---- what a pass cannot do without -------------------------------------------------------------------
def work(case):
    kind, bits = case["kind"], case["bits"]
    if kind == "kv":
        d, T, S = case["heads"] * case["width"], case["T"], case["S"]
        return dict(bytes=2 * (T * d * (2 + bits / 8) + S * d * (2 + bits / 8) + 2 * 16 * d), flops=0)
    if kind == "offline":
        d, N = case["d"], case["N"]
        params = N * 4 * (3 * case["g"] if case["cw"] else 2 + case["g"]) + 4 * N
        return dict(bytes=case["batches"] * CAL_ROWS * d * 2 + N * d * 4 + N * d / 2 + params + 20 * d, flops=0)
    M, d = case["M"], case["d"]
    size = 4 if case["out"] == "f32" else 2
    site = M * d * 2 + M * d * bits / 8 + 12 * d + 4 * M                     # rows in, codes and row terms out
    if kind == "ffn":
        f = case["dff"]
        return dict(bytes=site + 2 * (d * f / 2) + 12 * (d + f) + M * f * bits / 8 + 4 * M + M * d * size, flops=2 * 2 * M * d * f)
    N = case["N"]
    params = N * 4 * 2 * case["g"] + M * 128 if kind == "cw" else 12 * N
    return dict(bytes=site + N * d / 2 + params + M * N * size, flops=2 * M * N * d)


def tolerance(case):
    """Whole numbers (codes, permutations, packed weights, cache values) are the same.  fp32 results: measured against
    the same integers in float64, 6e-8 to 6e-7 in norm and at most 6e-6 of the rms (8-bit codes).  bf16 results: up to
    4e-5 in norm from the few values that cross a rounding boundary, one step of bf16 (2^-7 of the value) where they do.
    ffn: such a crossing can move a code of the hidden layer by one (measured 2e-6 of the 8-bit codes)."""
    kind = case["kind"]
    if kind in ("kv", "offline"):
        return "exact"
    if case["out"] == "f32" and kind != "ffn":
        return {"rel": 2.5e-6, "max": 2.5e-5}
    if kind != "ffn":
        return {"rel": 1.6e-4, "max": 1e-2}
    return {"rel": 2.5e-4, "max": 1e-2, "differ": 1e-5}

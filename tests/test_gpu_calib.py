"""Per-channel minimum / maximum over calibration batches against the oracle, bit for bit, at the sizes where the
kernel's split can go wrong: one and several rows per workgroup, ragged and empty batches, more batches than one
launch takes, more rows than the workgroups of a launch take in one pass, one to four chunks per thread, the last width
with several rows per workgroup."""
import numpy as np
import pytest

import workloads as w
from oracle import rptq_oracle as o

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")
EPS = 1e-5


def dev_bf16(x):
    return torch.from_numpy(w.bf16_bits(x).view(np.int16)).cuda().view(torch.bfloat16)


@pytest.mark.parametrize("ln,relu", [(True, False), (False, False), (False, True)])
@pytest.mark.parametrize("d,rows", [
    (8, [1]), (520, [3, 0, 70]), (1032, [2] * 67), (2056, [129, 5]), (8064, [17]), (8072, [3, 2]), (16392, [5]),
    (8, [8200, 1, 9000]), (8064, [500, 0, 300]), (8072, [301]), (16392, [150, 1, 120]),       # several passes per workgroup
])
def test_channel_minmax_bit_exact(d, rows, ln, relu):
    import paper_2304_01089_amd as rp
    rng = np.random.default_rng(d + len(rows))
    sc = np.exp(rng.normal(0, 1, d))
    off = rng.normal(0, 2 * sc)
    batches = [w.round_to_bf16((off + sc * rng.standard_normal((r, d))).astype(np.float32)) for r in rows]
    gamma = np.exp(rng.normal(0, 0.3, d)).astype(np.float32) if ln else None
    beta = rng.normal(0, 0.1, d).astype(np.float32) if ln else None
    act = [o.site_activation(b, gamma, beta, EPS, relu) for b in batches if len(b)]
    assert not any(f.any() for _, f in act)               # (no row whose fp32 statistics could round either way)
    a = np.concatenate([x for x, _ in act])
    out = torch.full((2, d), 7.0, dtype=torch.float32, device="cuda")
    ws = torch.zeros(rp.rptq_calibrate_workspace_bytes(d), dtype=torch.uint8, device="cuda")
    up = lambda v: None if v is None else torch.from_numpy(v).cuda()
    rp.rptq_channel_minmax([dev_bf16(b) for b in batches], up(gamma), up(beta), EPS, relu, out[0], out[1], ws)
    torch.cuda.synchronize()
    got = out.cpu().numpy()
    assert np.array_equal(got[0], a.min(axis=0) + np.float32(0)) and np.array_equal(got[1], a.max(axis=0) + np.float32(0))

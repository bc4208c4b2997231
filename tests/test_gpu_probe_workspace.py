"""Probes with few sampled rows or none, given exactly the workspace that the size query returns, at
lengths whose two calls (scores, coverage) would choose different key ranges."""
import numpy as np
import pytest

from paper_2608_29058_amd import _rs

pytestmark = pytest.mark.gpu


def _layer(n, hq, hkv, d):
    import torch
    g = torch.Generator(device="cuda").manual_seed(n)
    return [torch.randn((h, n, d), generator=g, device="cuda").to(torch.bfloat16) for h in (hq, hkv, hkv)]


@pytest.mark.parametrize("n", [20000, 49500])
def test_block_means_alone(n):
    """Tolerance: the documented 2^-16 of sum_d |q_d k_d| x scale, and fp32 means of 64 values (2^-18)."""
    import torch
    hq, hkv, d = 32, 8, 128
    q, k, v = _layer(n, hq, hkv, d)
    qkv = _rs.make_qkv(q, k, v)
    units = _rs.make_units([(h, 0, n) for h in range(hq)])
    cfg = _rs.RsProbeCfg(r_rec=0, r_uni=0, r_bnd=0, bs_block=64, local_w=1024, flags=_rs.RS_PROBE_BLOCKMEAN)
    pb = _rs.ProbeBuffers(hq, 0, n, hq, blockmean=True)
    ws = _rs.workspace(_rs.rs_probe_workspace_size(qkv, units, hq, cfg))
    ws.fill_(0xff)
    _rs.rs_probe(qkv, units, hq, cfg, None, 0, None, ws, pb)
    torch.cuda.synchronize()
    nb = (n + 63) // 64
    low = torch.tril_indices(nb, nb, device="cuda")

    def means(x):
        x = torch.nn.functional.pad(x.double(), (0, 0, 0, nb * 64 - n)).view(nb, 64, d).sum(1)
        cnt = torch.full((nb, 1), 64.0, dtype=torch.float64, device="cuda")
        cnt[-1] = n - 64 * (nb - 1)
        return x / cnt

    for h in (0, 13, hq - 1):
        qm, km = means(q[h]), means(k[h // (hq // hkv)])
        ref = (qm @ km.T.contiguous()) / d ** 0.5
        bound = (qm.abs() @ km.abs().T.contiguous()) / d ** 0.5 * 2.0 ** -15
        err = (pb.lbs[h].double() - ref[low[0], low[1]]).abs()
        assert bool((err <= bound[low[0], low[1]] + 1e-12).all()), h


def test_one_sampled_row():
    """Probabilities of one row: fp32 sums of exponentials of fp32 logits, 1e-5 of the largest."""
    import torch
    n, hq, hkv, d = 12507, 32, 32, 128
    q, k, v = _layer(n, hq, hkv, d)
    qkv = _rs.make_qkv(q, k, v)
    units = _rs.make_units([(h, 0, n) for h in range(hq)])
    cfg = _rs.RsProbeCfg(r_rec=1, r_uni=0, r_bnd=0, bs_block=64, local_w=1024, flags=_rs.RS_PROBE_ROWS)
    pb = _rs.ProbeBuffers(hq, 1, n, hq)
    ws = _rs.workspace(_rs.rs_probe_workspace_size(qkv, units, hq, cfg))
    ws.fill_(0xff)
    _rs.rs_probe(qkv, units, hq, cfg, None, 0, None, ws, pb)
    torch.cuda.synchronize()
    for h in range(hq):
        p = torch.softmax(k[h].double() @ q[h, -1].double() / d ** 0.5, 0)
        assert float((pb.col[h].double() - p).abs().max()) <= 1e-5 * float(p.max())
        assert float((pb.diag[h].double() - p.flip(0)).abs().max()) <= 1e-5 * float(p.max())
    assert np.array_equal(pb.rows.cpu().numpy()[:, 0], np.full(hq, n - 1))

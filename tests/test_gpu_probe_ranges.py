"""The probe's key ranges (128 to 1024 keys, chosen by the size of the launch and the workspace) and
its wave tasks (1 to 4 units of a group over up to three row-block pairs): every range length
against the longest, and the coverage against the oracle.

Ranges move fp32 partial sums only.  col, diag and the coverage are sums of at most 1 per row over at
most 160 rows of probabilities below 1: 160 x 2^-23 x a few roundings < 1e-4 absolute; sums relative
to a row's maximum likewise, relative 1e-5."""
import numpy as np
import pytest

from oracle import attention as A
from oracle import patterns as P
from oracle import probe as PR
from paper_2608_29058_amd import _rs
from synth import gen as G

from gpu_helpers import dev

pytestmark = pytest.mark.gpu

GRID = [(_rs.RS_DENSE, 0, 0), (_rs.RS_ASHAPE, 64, 256), (_rs.RS_VSLASH, 50, 200), (_rs.RS_BSPARSE, 4, 64)]
NAMES = ("col", "diag", "row_max", "row_sum", "cov", "cov_rows", "entropy", "local")


@pytest.mark.parametrize("hq,hkv,rc", [(1, 1, (64, 64, 32)), (2, 1, (64, 16, 8)), (3, 1, (64, 64, 32)),
                                       (5, 1, (100, 16, 8)), (4, 4, (30, 0, 0))])
def test_ranges_and_wave_tasks(hq, hkv, rc):
    import torch
    n, d = 2811, 64
    r = np.random.default_rng(hq * 10 + hkv)
    q, k, v = (G.bf16_round(r.standard_normal((h, n, d)).astype(np.float32)) for h in (hq, hkv, hkv))
    bufs = [dev(x) for x in (q, k, v)]  # the descriptor does not own its arrays
    qkv = _rs.make_qkv(*bufs)
    units = [(h, s0, s1) for s0, s1 in ((0, 1300), (1300, n)) for h in range(hq)]
    U, rmax, C = len(units), sum(rc), len(GRID)
    u = _rs.make_units(units)
    cfg = _rs.RsProbeCfg(r_rec=rc[0], r_uni=rc[1], r_bnd=rc[2], bs_block=64, local_w=300,
                         flags=_rs.RS_PROBE_ROWS | _rs.RS_PROBE_BLOCKMEAN)
    g = _rs.make_grid(GRID)
    need = _rs.rs_probe_workspace_size(qkv, u, U, cfg)

    def bytes_of(rng):  # partial results of ranges of rng keys, without the arrays' alignment
        nch, nb = -(-n // rng), -(-n // 64)
        return 4 * (U * nch * (rng + rmax) + U * nch * rmax * 20 + (hq + hkv) * nb * d)

    out, ib = {}, None
    for rng in (1024, 512, 256, 128):
        # room for ranges of rng keys and not for the next shorter ones
        size = min(need, bytes_of(rng) + 8192 + 64 * U)
        if rng > 128:
            assert size < bytes_of(rng // 2)
        ws = _rs.workspace(size)
        ws.fill_(0xff)
        pb = _rs.ProbeBuffers(U, rmax, n, hq, C, blockmean=True)
        _rs.rs_probe(qkv, u, U, cfg, None, 0, None, ws, pb)
        if ib is None:
            ib = _rs.IndexBuffers(U, n, hq, GRID)
            _rs.rs_build_indices(pb, u, U, g, C, _rs.workspace(_rs.rs_build_indices_workspace_size(pb, g, C)), ib)
        x0 = {name: getattr(pb, name).clone() for name in ("row_max", "row_sum")}
        _rs.rs_probe(qkv, u, U, cfg, g, C, ib, ws, pb)
        torch.cuda.synchronize()
        got = {name: getattr(pb, name).cpu().numpy() for name in NAMES}
        got.update({"s_" + name: t.cpu().numpy() for name, t in x0.items()})
        out[rng] = got
    for rng in (512, 256, 128):
        for name, a in out[rng].items():
            np.testing.assert_allclose(a, out[1024][name], atol=1e-4, rtol=1e-5, err_msg=f"{name}, range {rng}")
    got = out[128]
    for ui, (h, s0, s1) in enumerate(units):
        kv = h // (hq // hkv)
        ref = PR.probe_unit(q[h], k[kv], s0, s1, *rc)
        rows, nr = ref["rows"], ref["rows"].size
        assert np.abs(got["col"][ui, :s1] - ref["col"]).max() <= 1e-4
        assert np.abs(got["diag"][ui, :s1] - ref["diag"]).max() <= 1e-4
        cnt = ib.vs_count[ui, 0].cpu().numpy()
        V, D = ib.vs_vsorted[ui, 0].cpu().numpy()[:cnt[0]], ib.vs_dsorted[ui, 0].cpu().numpy()[:cnt[1]]
        srt, bc = ib.bs_sorted[h, 0].cpu().numpy(), ib.bs_count[h, 0].cpu().numpy()
        for c, m in ((1, P.ashape_mask(rows, s1, 64, 256)), (2, P.vs_mask(rows, s1, V, D)),
                     (3, P.bs_mask(rows, s1, 64, lambda bq: srt[bq, :bc[bq]]))):
            assert np.abs(got["cov_rows"][ui, c, :nr] - A.retained_mass(ref["a"], m)).max() <= 1e-4, (ui, c)

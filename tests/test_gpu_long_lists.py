"""Unit lists of the probe and the index construction in every form that reaches the device: the
caller's unit tables (built on the host), kernel arguments (up to 128 units in the probe, 512 in the
index construction) and copies of longer lists.  All give the same bits."""
import numpy as np
import pytest

from paper_2608_29058_amd import _rs
from synth import gen as G

from gpu_helpers import dev

pytestmark = pytest.mark.gpu

GRID = [(0, 0, 0), (1, 16, 64), (2, 20, 30), (3, 4, 64)]
PROBE = ("rows", "subset", "nsub", "row_max", "row_sum", "col", "diag", "lbs", "cov_rows", "cov", "entropy", "local")
INDEX = ("vs_vsorted", "vs_dsorted", "vs_count", "vs_vbits", "vs_dbits", "bs_rank", "bs_sorted", "bs_count", "bs_bits")


@pytest.mark.parametrize("n,hq,hkv,seg,rc", [
    (2048, 2, 1, 32, (8, 8, 4)),       # 128 units: the arguments are full
    (2100, 1, 1, 16, (8, 8, 4)),       # 132: probe lists are copied
    (2048, 4, 2, 16, (8, 0, 4)),       # 512: as many as the index construction's arguments hold
    (1800, 2, 2, 7, (4, 3, 2)),        # 516, rows fewer than sampled: both copied
    (900, 3, 1, 100, (64, 64, 32)),    # sampled rows overlap
    (900, 3, 3, 130, (0, 100, 60)),    # no recent rows
    (777, 1, 1, 777, (5, 200, 51)),
])
def test_lists_in_every_form_give_the_same_bits(n, hq, hkv, seg, rc):
    import torch
    d, g = 64, _rs.make_grid(GRID)
    r = np.random.default_rng(n)
    t = [dev(G.bf16_round(r.standard_normal((h, n, d)).astype(np.float32))) for h in (hq, hkv, hkv)]
    ul = [(h, s, min(n, s + seg)) for s in range(0, n, seg) for h in range(hq)]
    U, rmax = len(ul), sum(rc)
    units = _rs.make_units([(*u, 0, i) for i, u in enumerate(ul)])
    cfg = _rs.RsProbeCfg(r_rec=rc[0], r_uni=rc[1], r_bnd=rc[2], bs_block=64, local_w=100,
                         flags=_rs.RS_PROBE_ROWS | _rs.RS_PROBE_BLOCKMEAN)
    got = []
    for tabled in (True, False):
        qkv = _rs.make_qkv(*t)
        pb = _rs.ProbeBuffers(U, rmax, n, hq, len(GRID), blockmean=True)
        if tabled:
            tab = _rs.UnitTable(qkv, units, U, cfg)
            qkv.tables = tab.ptr
            pb.c.tables = tab.ptr
        ib = _rs.IndexBuffers(U, n, hq, GRID)
        ws = _rs.workspace(max(_rs.rs_probe_workspace_size(qkv, units, U, cfg),
                               _rs.rs_build_indices_workspace_size(pb, g, len(GRID))))
        ws.fill_(0xff)
        _rs.rs_probe(qkv, units, U, cfg, None, 0, None, ws, pb)
        _rs.rs_build_indices(pb, units, U, g, len(GRID), ws, ib)
        _rs.rs_probe(qkv, units, U, cfg, g, len(GRID), ib, ws, pb)
        torch.cuda.synchronize()
        got.append({**{x: getattr(pb, x) for x in PROBE}, **{x: getattr(ib, x) for x in INDEX}})
    for name, a in got[0].items():
        b = got[1][name]
        if a.is_floating_point():
            a, b = a.view(torch.int32), b.view(torch.int32)
        assert torch.equal(a, b), name

"""Items split along the keys in lists with other units: a routed layer cut into segments, whose last
segment's dense and vertical-slash items are split, against one call per group (bitwise, as the rule
looks at the unit alone), and against a workspace without room for pieces: units that end before the
sequence are never split, so their rows are bitwise the same."""
import numpy as np
import pytest

from paper_2608_29058_amd import _rs
from synth import gen as G

from gpu_helpers import dev, fill_vs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d,n,seg", [(4, 2, 64, 2900, 1300), (5, 5, 128, 2111, 1000), (2, 1, 128, 1300, 128)])
def test_split_units_in_a_routed_layer(hq, hkv, d, n, seg):
    import torch
    r = np.random.default_rng(n)
    t = [dev(G.bf16_round(r.standard_normal((h, n, d)).astype(np.float32))) for h in (hq, hkv, hkv)]
    qkv = _rs.make_qkv(*t)
    grid = [(0, 0, 0), (1, 64, 256), (2, 200, 150)]
    g = _rs.make_grid(grid)
    segs = [(s, min(n, s + seg)) for s in range(0, n, seg)]
    ul = [(h, s0, s1) for s0, s1 in segs for h in range(hq)]
    U = len(ul)
    units = _rs.make_units([(*u, 0, i) for i, u in enumerate(ul)])
    ib = _rs.IndexBuffers(U, n, hq, grid)
    for i, (h, s0, s1) in enumerate(ul):
        fill_vs(ib, i, 0, np.sort(r.choice(s1, min(s1, 200), replace=False)),
                np.unique(np.concatenate([np.arange(20), r.choice(s1, min(s1, 100), replace=False)])))
    choice = [(0, 2, 1)[(i - (U - hq)) % 3] for i in range(U)]
    choice[1] = -1
    last = slice(U - hq, U)
    assert {0, 2} <= set(choice[last]), "both split families in the last segment"

    def outputs():
        return (torch.full((hq, n, d), float("nan"), dtype=torch.bfloat16, device="cuda"),
                torch.full((hq, n), float("nan"), dtype=torch.float32, device="cuda"))

    og, lg = outputs()
    for c in range(3):
        us = [i for i in range(U) if choice[i] == c]
        gu = _rs.make_units([(*ul[i], c, i) for i in us])
        ws = _rs.workspace(_rs.rs_attn_workspace_size(qkv, gu, len(us)))
        ws.fill_(0xff)
        if c == 0:
            _rs.rs_dense_attn_prefill(qkv, gu, len(us), og, lg, ws)
        else:
            _rs.rs_sparse_attn_prefill(qkv, gu, len(us), g, 3, ib, og, lg, ws)
        torch.cuda.synchronize()
    ch = torch.tensor(choice, dtype=torch.int32, device="cuda")
    need = _rs.rs_routed_attn_workspace_size(qkv, units, U)
    tiles = sum((s1 - 1) // 128 - s0 // 128 + 1 for _, s0, s1 in ul)
    bare = 16 * tiles + 4 * 48 * U + 32 * U + 4096
    assert need > bare + 2 * hq * 128 * d * 4, "the last segment may be split"
    got = []
    for nbytes in (need, bare):
        o, l = outputs()
        ws = _rs.workspace(nbytes)
        ws.fill_(0xff)
        _rs.rs_routed_attn_prefill(qkv, units, U, g, 3, ib, ch, o, l, ws)
        torch.cuda.synchronize()
        got.append((o, l))
    (o, l), (ob, lb) = got
    assert torch.equal(o.view(torch.int16), og.view(torch.int16)) and torch.equal(l.view(torch.int32), lg.view(torch.int32))
    h, s0, s1 = ul[1]
    assert bool(torch.isnan(o[h, s0:s1]).all())
    done = torch.ones((hq, n), dtype=torch.bool, device="cuda")
    done[h, s0:s1] = False
    assert bool(torch.isfinite(o[done]).all()) and bool(torch.isfinite(l[done]).all())
    s = segs[-1][0]
    assert torch.equal(o[:, :s].view(torch.int16), ob[:, :s].view(torch.int16))
    assert torch.equal(l[:, :s].view(torch.int32), lb[:, :s].view(torch.int32))
    # pieces move fp32 partial sums only: bf16 output rounding apart
    a, b = o[:, s:].float(), ob[:, s:].float()
    ok = done[:, s:]
    assert bool(((a - b).abs() <= 2.0 ** -8 * torch.maximum(a.abs(), b.abs()) + 2.0 ** -9)[ok].all())

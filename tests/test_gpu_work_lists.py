"""Work lists of the attention calls: up to 64 equal units in the kernel arguments, other lists in the
workspace.  A unit's result does not depend on the list it came in: every unit of a list, launched in
lists of different kinds and orders, gives the same bits, and every row is written."""
import numpy as np
import pytest

from paper_2608_29058_amd import _rs
from synth import gen as G

from gpu_helpers import dev, fill_bs, fill_vs

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fam", [_rs.RS_DENSE, _rs.RS_ASHAPE, _rs.RS_VSLASH, _rs.RS_BSPARSE])
@pytest.mark.parametrize("hq,hkv,heads", [
    (70, 10, None),             # more units than the arguments hold; key/value heads 8 and 9 share buckets
    (64, 8, None),              # as many as they hold
    (30, 10, None),             # buckets of different sizes: they drop out of the turns one by one
    (12, 12, (0, 3, 4, 11)),    # some buckets empty
    (4, 1, (1, 2)),             # one bucket; heads that are not mates of each other
    (1, 1, None),
])
def test_results_do_not_depend_on_the_work_list(fam, hq, hkv, heads):
    import torch
    n, d, s0 = 700, 64, 130
    r = np.random.default_rng(hq)
    heads = list(range(hq)) if heads is None else list(heads)
    t = [dev(G.bf16_round(r.standard_normal((h, n, d)).astype(np.float32))) for h in (hq, hkv, hkv)]
    qkv = _rs.make_qkv(*t)
    grid = [(_rs.RS_DENSE, 0, 0), (_rs.RS_ASHAPE, 70, 100), (_rs.RS_VSLASH, 30, 40), (_rs.RS_BSPARSE, 4, 64)]
    c = fam
    ib = _rs.IndexBuffers(len(heads), n, hq, grid)
    for x, h in enumerate(heads):
        fill_vs(ib, x, 0, np.sort(r.choice(n, 30, replace=False)),
                np.unique(np.concatenate([[0], r.choice(n, 3 + h % 37, replace=False)])))
    for h in range(hq):
        fill_bs(ib, h, 0, [sorted(set([b]) | set(r.integers(0, b + 1, 3).tolist())) for b in range((n + 63) // 64)])
    units = [(h, s0, n, c, x) for x, h in enumerate(heads)]

    def run(lists):
        o = torch.full((hq, n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full((hq, n), float("nan"), dtype=torch.float32, device="cuda")
        for us in lists:
            u = _rs.make_units(us)
            ws = _rs.workspace(_rs.rs_attn_workspace_size(qkv, u, len(us)))
            if fam == _rs.RS_DENSE:
                _rs.rs_dense_attn_prefill(qkv, u, len(us), o, lse, ws)
            else:
                _rs.rs_sparse_attn_prefill(qkv, u, len(us), _rs.make_grid(grid), len(grid), ib, o, lse, ws)
            torch.cuda.synchronize()
        return o, lse

    o, lse = run([units])
    assert bool(torch.isfinite(o[heads, s0:]).all()) and bool(torch.isnan(o[:, :s0]).all())
    others = [h for h in range(hq) if h not in heads]
    assert bool(torch.isnan(o[others]).all())
    # one by one; reversed; with a unit of other rows among them (a list in the workspace)
    first = (heads[0], 0, s0, c, 0)
    for lists in ([[u] for u in units[:6]], [units[::-1]], [units + [first]]):
        o2, lse2 = run(lists)
        hs = [u[0] for us in lists for u in us if u[1] == s0]
        assert torch.equal(o[hs, s0:].view(torch.int16), o2[hs, s0:].view(torch.int16))
        assert torch.equal(lse[hs, s0:].view(torch.int32), lse2[hs, s0:].view(torch.int32))

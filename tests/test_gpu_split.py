"""Items split along the keys (few query rows, long context): dense and vertical-slash against the
fp64 oracle, in one piece (a workspace that holds the work list only) and in several.

Tolerance: that of every attention output (max-abs 2e-2, relative Frobenius 1e-2); splitting
moves fp32 partial sums only, so the two runs agree to bf16 output rounding: 2^-8 of the larger
magnitude plus the bf16 spacing at the output's scale."""
import numpy as np
import pytest

from oracle import attention as A
from oracle import patterns as P
from paper_2608_29058_amd import _rs
from synth import gen as G

from gpu_helpers import check_close, dev, fill_vs, out_tensor, with_vt

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fam", ["dense", "vslash"])
@pytest.mark.parametrize("n,s0,hq,hkv,d,dtype,vt", [
    (4200, 4199, 2, 1, 128, "bf16", False),   # one row: one item, one valid row
    (4224, 3967, 3, 1, 128, "bf16", True),    # first and last item with one valid row, whole tiles
    (3001, 2871, 2, 2, 64, "bf16", False),    # odd length, rows across two items
    (2500, 0, 1, 1, 64, "f32", False),        # a whole prompt: early items have fewer tiles than pieces
    (1024, 1000, 1, 1, 128, "bf16", False),   # two pieces of the shortest length
])
def test_split_items_match_the_oracle(fam, n, s0, hq, hkv, d, dtype, vt):
    import torch
    r = np.random.default_rng(n + s0)
    q, k, v = (r.standard_normal((h, n, d)).astype(np.float32) for h in (hq, hkv, hkv))
    if dtype == "bf16":
        q, k, v = G.bf16_round(q), G.bf16_round(k), G.bf16_round(v)
    qd, kd, vd = dev(q, dtype), dev(k, dtype), dev(v, dtype)
    qkv = _rs.make_qkv(qd, kd, vd)
    if vt:
        qkv, _vt = with_vt(qkv)
    grid = [(_rs.RS_DENSE, 0, 0), (_rs.RS_VSLASH, 300, 400)]
    c = 0 if fam == "dense" else 1
    units = _rs.make_units([(h, s0, n, c, h) for h in range(hq)])
    ib, sets = None, []
    if c:
        # head 0: lines over the whole context; others: a short list (fewer pieces than allowed) with
        # no key in its lowest tiles, so that pieces hold rows without a kept key
        ib = _rs.IndexBuffers(hq, n, hq, grid)
        for h in range(hq):
            if h == 0:
                V = np.sort(r.choice(n, 300, replace=False))
                D = np.unique(np.concatenate([np.arange(100), r.choice(n, 300, replace=False)]))
            else:
                V, D = np.arange(n - 40, n - 30), np.arange(5)
            fill_vs(ib, h, 0, V, D)
            sets.append((V, D))
    need = _rs.rs_attn_workspace_size(qkv, units, hq)
    items = hq * ((n - 1) // 128 - s0 // 128 + 1)
    bare = 64 * hq + 4 * items + 1024   # holds the list of unsplit items, no partial results
    assert need > bare + items * 128 * d * 4, "the case is split"
    got = []
    for nbytes in (bare, need):
        o = out_tensor(hq, n, d)
        lse = torch.full((hq, n), float("nan"), dtype=torch.float32, device="cuda")
        ws = _rs.workspace(nbytes)
        ws.fill_(0xff)
        if c:
            _rs.rs_sparse_attn_prefill(qkv, units, hq, _rs.make_grid(grid), 2, ib, o, lse, ws)
        else:
            _rs.rs_dense_attn_prefill(qkv, units, hq, o, lse, ws)
        torch.cuda.synchronize()
        got.append((o.float().cpu().numpy(), lse.cpu().numpy()))
    rows, g = np.arange(s0, n), hq // hkv
    for h in range(hq):
        mask = P.vs_mask(rows, n, *sets[h]) if c else P.dense_mask(rows, n)
        ref, rl = A.masked_attention(q[h], k[h // g], v[h // g], rows, mask)
        for what, (o, lse) in zip(("one piece", "pieces"), got):
            check_close(o[h, s0:], ref, f"{what} h={h}")
            # fp32 inputs are rounded to bf16 on load: logits of a few units move by up to ~2^-8 of them
            np.testing.assert_allclose(lse[h, s0:], rl, atol=2e-3 if dtype == "bf16" else 3e-2, rtol=1e-4)
        if s0:
            assert np.isnan(got[1][0][h, :s0]).all() and np.isnan(got[1][1][h, :s0]).all()
    a, b = got[0][0][:, s0:], got[1][0][:, s0:]
    assert (np.abs(a - b) <= 2.0 ** -8 * np.maximum(np.abs(a), np.abs(b)) + 2.0 ** -9).all()

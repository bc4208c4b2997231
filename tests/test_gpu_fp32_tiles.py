"""fp32 inputs: rounded to bf16 copies once per call where the workspace has room, else per key tile.
The rounding is the same, so the results are the same bits: every family, head dimension, V layout
and launch (direct list, list in the workspace, one persistent launch of a layer, one per family), with
a workspace of the queried size and with one that holds the work lists only."""
import numpy as np
import pytest

from paper_2608_29058_amd import _rs

from gpu_helpers import dev, fill_bs, fill_vs, with_vt

pytestmark = pytest.mark.gpu


def _inputs(n, hq, hkv, d, layout):
    import torch
    r = np.random.default_rng(n + d)
    out = []
    for h in (hq, hkv, hkv):
        x = r.standard_normal((h, n, d)).astype(np.float32)
        if layout == "token":  # views of [n, heads, d]
            out.append(torch.from_numpy(np.ascontiguousarray(x.transpose(1, 0, 2))).cuda().transpose(0, 1))
        else:
            out.append(dev(x, "f32"))
    return out


def _fill(ib, i, h, s1, n, r):
    fill_vs(ib, i, 0, np.sort(r.choice(s1, min(s1, 90), replace=False)),
            np.unique(np.concatenate([np.arange(30), r.choice(s1, min(s1, 60), replace=False)])))
    fill_bs(ib, h, 0, [sorted(set([b]) | set(r.integers(0, b + 1, 10).tolist())) for b in range((n + 63) // 64)])


GRID = [(0, 0, 0), (1, 64, 2000), (2, 90, 90), (3, 64, 64)]


@pytest.mark.parametrize("fam", [0, 1, 2, 3])
@pytest.mark.parametrize("d,vt,layout", [(128, False, "head"), (128, True, "token"), (64, False, "token"), (64, True, "head")])
@pytest.mark.parametrize("units", [
    [(h, 130, 2200) for h in range(6)],                                  # equal rows: a list in the arguments
    [(1, 0, 1999), (4, 700, 2240), (5, 700, 2240), (5, 2240, 2299)],     # some heads, other rows: a list in memory
    [(0, 2100, 2250), (3, 2200, 2250)],                                  # few query rows over many keys
])
def test_copies_and_tiles_give_the_same_bits(fam, d, vt, layout, units):
    import torch
    n, hq, hkv = 2300, 6, 2  # no unit ends with the sequence: nothing is split
    t = _inputs(n, hq, hkv, d, layout)
    qkv = _rs.make_qkv(*t)
    if vt:
        qkv, _vt = with_vt(qkv)
    r = np.random.default_rng(5)
    U = len(units)
    ib = _rs.IndexBuffers(U, n, hq, GRID)
    for i, (h, s0, s1) in enumerate(units):
        _fill(ib, i, h, s1, n, r)
    u = _rs.make_units([(*x, fam, i) for i, x in enumerate(units)])
    tiles = 2 * sum((s1 - 1) // 128 - s0 // 128 + 1 for _, s0, s1 in units)
    bare = 64 * U + 4 * tiles + 1024
    need = _rs.rs_attn_workspace_size(qkv, u, U)
    got = []
    for nbytes in (need, bare):
        o = torch.full((hq, n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full((hq, n), float("nan"), dtype=torch.float32, device="cuda")
        ws = _rs.workspace(nbytes)
        ws.fill_(0xff)
        if fam == 0:
            _rs.rs_dense_attn_prefill(qkv, u, U, o, lse, ws)
        else:
            _rs.rs_sparse_attn_prefill(qkv, u, U, _rs.make_grid(GRID), len(GRID), ib, o, lse, ws)
        torch.cuda.synchronize()
        if nbytes == need:
            assert bool((ws[bare:nbytes] != 0xff).any()), "converted"
        got.append((o.view(torch.int16), lse.view(torch.int32)))
        for h, s0, s1 in units:
            assert bool(torch.isfinite(o[h, s0:s1]).all())
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])


def test_more_heads_than_one_conversion_launch_holds():
    import torch
    n, hq, hkv, d, s1 = 900, 200, 10, 64, 850
    t = _inputs(n, hq, hkv, d, "head")
    qkv = _rs.make_qkv(*t)
    r = np.random.default_rng(8)
    ib = _rs.IndexBuffers(hq, n, hq, GRID)
    V, D = np.sort(r.choice(s1, 90, replace=False)), np.unique(np.concatenate([[0], r.choice(s1, 89, replace=False)]))
    for h in range(hq):
        fill_vs(ib, h, 0, V, D)
    u = _rs.make_units([(h, 0, s1, 2, h) for h in range(hq)])
    need, bare = _rs.rs_attn_workspace_size(qkv, u, hq), 64 * hq + 32 * hq + 1024
    got = []
    for nbytes in (need, bare):
        o = torch.full((hq, n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        ws = _rs.workspace(nbytes)
        ws.fill_(0xff)
        _rs.rs_sparse_attn_prefill(qkv, u, hq, _rs.make_grid(GRID), len(GRID), ib, o, None, ws)
        torch.cuda.synchronize()
        if nbytes == need:
            assert bool((ws[bare:] != 0xff).any()), "converted"
        got.append(o.view(torch.int16))
        assert bool(torch.isfinite(o[:, :s1]).all())
    assert torch.equal(got[0], got[1])


@pytest.mark.parametrize("d,vt", [(128, True), (128, False), (64, True), (64, False)])
@pytest.mark.parametrize("events", [False, True])
def test_routed_copies_and_tiles_give_the_same_bits(d, vt, events):
    import torch
    n, hq, hkv, seg = 2900, 4, 2, 1300
    t = _inputs(n, hq, hkv, d, "head")
    qkv = _rs.make_qkv(*t)
    if vt:
        qkv, _vt = with_vt(qkv)
    r = np.random.default_rng(6)
    ul = [(h, s, min(n, s + seg)) for s in range(0, n, seg) for h in range(hq)]
    U = len(ul)
    units = _rs.make_units([(*x, 0, i) for i, x in enumerate(ul)])
    ib = _rs.IndexBuffers(U, n, hq, GRID)
    for i, (h, s0, s1) in enumerate(ul):
        _fill(ib, i, h, s1, n, r)
    choice = torch.tensor([(i + i // hq) % 4 for i in range(U)], dtype=torch.int32, device="cuda")
    tiles = sum((s1 - 1) // 128 - s0 // 128 + 1 for _, s0, s1 in ul)
    bare = 16 * tiles + 4 * 48 * U + 32 * U + 4096
    need = _rs.rs_routed_attn_workspace_size(qkv, units, U)
    got = []
    for nbytes in (need, bare):
        o = torch.full((hq, n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full((hq, n), float("nan"), dtype=torch.float32, device="cuda")
        ws = _rs.workspace(nbytes)
        ws.fill_(0xff)
        ev = [torch.cuda.Event(enable_timing=True) for _ in range(5)] if events else None
        _rs.rs_routed_attn_prefill(qkv, units, U, _rs.make_grid(GRID), len(GRID), ib, choice, o, lse, ws, events=ev)
        torch.cuda.synchronize()
        assert bool(torch.isfinite(o).all()) and bool(torch.isfinite(lse).all())
        got.append((o, lse))
    (a, la), (b, lb) = got
    s = ul[-1][1]
    assert torch.equal(a[:, :s].view(torch.int16), b[:, :s].view(torch.int16))
    assert torch.equal(la[:, :s].view(torch.int32), lb[:, :s].view(torch.int32))
    # the last segment's items have pieces where there is room: fp32 partial sums in another order
    x, y = a[:, s:].float(), b[:, s:].float()
    assert bool(((x - y).abs() <= 2.0 ** -8 * torch.maximum(x.abs(), y.abs()) + 2.0 ** -9).all())

"""A routed layer's attention as one launch of every family, and with timing events as one launch per
family: the same items through the same code, so O and LSE are bitwise equal."""
import numpy as np
import pytest

from paper_2608_29058_amd import _rs
from paper_2608_29058_amd.pipeline import RouteKnobs, RoutedLayer

from gpu_helpers import dev

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("hq,hkv,d,dtype,vt,fams", [
    (4, 2, 128, "bf16", True, (0, 1, 2, 3)),
    (6, 1, 64, "bf16", False, (0, 1, 2, 3)),
    (2, 2, 128, "f32", True, (0, 1, 2, 3)),
    (2, 2, 64, "f32", False, (0, 2)),        # families without queues
    (8, 8, 128, "bf16", True, (0, 1)),       # no index set read
])
def test_one_launch_equals_a_launch_per_family(hq, hkv, d, dtype, vt, fams):
    import torch
    n, seg = 3333, 1000
    r = np.random.default_rng(hq + d)
    q, k, v = (dev(r.standard_normal((h, n, d)).astype(np.float32), dtype) for h in (hq, hkv, hkv))
    grid = [g for g in [(0, 0, 0), (1, 64, 256), (2, 64, 128), (2, 128, 512), (3, 4, 64), (3, 8, 64)] if g[0] in fams]
    if not any(g[0] in (2, 3) for g in grid):
        index_grid = grid + [(3, 4, 64)]  # buffers for the unused family
    else:
        index_grid = grid
    RL = RoutedLayer(n, hq, hkv, d, seg, index_grid, r_rec=64, r_uni=16, r_bnd=8, use_vt=vt)
    qkv = RL.qkv(q, k, v)
    RL.probe_and_index(qkv)
    choice = torch.tensor([i % len(grid) for i in range(RL.nunits)], dtype=torch.int32, device="cuda")
    choice[3] = -1
    ws = _rs.workspace(_rs.rs_routed_attn_workspace_size(qkv, RL.units, RL.nunits))
    got = []
    for events in (None, [torch.cuda.Event(enable_timing=True) for _ in range(5)]):
        o = torch.full((hq, n, d), float("nan"), dtype=torch.bfloat16, device="cuda")
        lse = torch.full((hq, n), float("nan"), dtype=torch.float32, device="cuda")
        ws.fill_(0xff)
        _rs.rs_routed_attn_prefill(qkv, RL.units, RL.nunits, _rs.make_grid(grid), len(grid), RL.ib, choice, o, lse, ws,
                                   events=events)
        torch.cuda.synchronize()
        got.append((o.view(torch.int16), lse.view(torch.int32)))
    assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][1], got[1][1])
    h, s0, s1 = RL.unit_list[3]
    o = got[0][0].view(torch.bfloat16)
    assert bool(torch.isnan(o[h, s0:s1]).all())
    done = torch.ones((hq, n), dtype=torch.bool, device="cuda")
    done[h, s0:s1] = False
    assert bool(torch.isfinite(o[done]).all()), "every routed row is written"

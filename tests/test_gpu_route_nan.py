"""The device router on coverage that holds NaN (a probe of NaN inputs): every run gives the same route,
the one in which substitutions of undefined ratio come after all others, by unit and position."""
import numpy as np
import pytest

from paper_2608_29058_amd import _rs

pytestmark = pytest.mark.gpu

GRID = [(0, 0, 0), (1, 128, 1024), (1, 128, 4096), (2, 500, 256), (2, 1000, 512), (3, 50, 64), (3, 100, 64)]


def _route(t, R, T):
    """Greedy choices by the merged order of the units' moves (key: running maximum of the ratio)."""
    U, C = t.shape
    moves = []
    for u in range(U):
        cur, j, K = 0, 0, 0.0
        while True:
            best = None
            for c in range(C):
                if t[u, c] < t[u, cur]:
                    rho = (R[u, c] - R[u, cur]) / (t[u, cur] - t[u, c])
                    if best is None or rho < best[0]:
                        best = (rho, c)
            if best is None:
                break
            K = best[0] if j == 0 or best[0] > K else K
            moves.append((np.inf if np.isnan(K) else K, u, j, best[1]))
            cur, j = best[1], j + 1
    choice = [0] * U
    total = lambda: sum((t[u, choice[u]] for u in range(U)), 0.0)
    for _, u, _, c in sorted(moves):
        if total() <= T:
            break
        choice[u] = c
    return choice


@pytest.mark.parametrize("U,share", [(40, 0.1), (256, 0.5), (600, 0.02), (64, 1.0)])
def test_nan_coverage_routes_the_same_every_time(U, share):
    import torch
    r = np.random.default_rng(U)
    C = len(GRID)
    cov = np.repeat(r.uniform(0.5, 1.0, (U, C, 1)).astype(np.float32), 4, axis=2)
    cov[r.random((U, C)) < share] = np.nan
    cov[:, 0, :] = 1.0
    nsub = np.tile(np.array([64, 0, 0], np.int32), (U, 1))
    edges = np.array([16384, 32768], np.int32)
    s1 = r.choice(edges, U).astype(np.int32)
    tt = np.array([[512.0, 1024.0]] + [[float(r.integers(4, 200)), float(r.integers(4, 400))] for _ in range(C - 1)])
    t = tt[:, np.searchsorted(edges, s1)].T
    R = 1.0 - cov[:, :, 0].astype(np.float64)
    R[:, 0] = 0.0
    T = float(t[:, 0].sum() * 0.4)
    want = _route(t, R, T)
    cd, nd = torch.from_numpy(cov).cuda(), torch.from_numpy(nsub).cuda()
    for _ in range(5):
        rb = _rs.RouteDevBuffers(GRID, s1, tt, edges)
        _rs.rs_route_layer_device(rb, cd, nd, 0.0, T, 0.0, 1.0, 0.0, 0.0)
        torch.cuda.synchronize()
        assert rb.choice.cpu().tolist() == want

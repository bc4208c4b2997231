"""The work that a user of the library has it do, as cases that can be timed and compared.

A case is a dict of plain values:

  path    "dense", "ashape": attention over whole heads or over the last rows of a context;
          "vslash", "bsparse": scores, index construction and sparse attention of one layer;
          "routed": one whole layer through ``RoutedLayer`` (probe, indices, coverage, device
          route, one launch per family);
  n, s0   sequence length and first query row: s0 = 0 is a whole prompt, s0 > 0 a chunk of a
          chunked prefill (rows [s0, n) against keys [0, n));
  hq, hkv, d, dtype, layout
          heads, head dimension, "bf16" or "f32" inputs, and "head" ([heads, n, d]) or "token"
          (views of [n, heads, d], as a projection leaves them);
  vt      V is also laid out by ``rs_transpose_v`` (part of the pass: V is new in every layer);
  lse     the log-sum-exp of every row is written too (merging of chunks, audits);
  a, b    the budget: sink and window, columns and diagonals, or key blocks and block width;
  dense_heads
          heads of a vertical-slash layer that take the dense fallback;
  seg     rows per unit of a routed layer;
  inputs  "mixed": weak sinks, columns and a weak local band on every head; "regimes": every
          key/value head local, sink, vertical or diffuse, nearly all of its mass in that structure
          (what routing is for: of a "mixed" layer nearly every unit would fall back to dense).

Inputs are drawn on the GPU from the seed alone.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2608_29058_amd import _rs
from paper_2608_29058_amd.pipeline import RoutedLayer, RouteKnobs

DEV = "cuda"

# the candidate grid of the routed workload: dense, two A-shape, three vertical-slash and three
# block-sparse budgets
GRID = [(0, 0, 0), (1, 128, 1024), (1, 128, 4096), (2, 500, 256), (2, 1000, 512), (2, 2000, 2048),
        (3, 50, 64), (3, 100, 64), (3, 200, 64)]
# the same library at the budgets of a context of 4K to 32K tokens
GRID_SHORT = [(0, 0, 0), (1, 64, 256), (1, 128, 1024), (2, 128, 128), (2, 256, 256), (2, 500, 512),
              (3, 8, 64), (3, 16, 64), (3, 32, 64)]


def _case(name, path, n, hq=32, hkv=8, d=128, dtype="bf16", s0=0, layout="head", vt=True, lse=False, a=0, b=0,
          dense_heads=0, seg=0, inputs="regimes"):
    c = dict(path=path, n=n, s0=s0, hq=hq, hkv=hkv, d=d, dtype=dtype, layout=layout, vt=vt, lse=lse, a=a, b=b,
             dense_heads=dense_heads, seg=seg, inputs=inputs)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest call: one fp32 head of a 2K prompt through scores, indices and attention
        _case("vslash_2k_f32", "vslash", 2048, hq=1, hkv=1, d=64, dtype="f32", vt=False, a=64, b=256, inputs="mixed"),
        # a short prompt of odd length, dense, every head of a grouped-query layer
        _case("dense_777", "dense", 777, vt=False, lse=True),
        # an unaligned fp32 prompt with as many key/value heads as query heads and d = 64
        _case("dense_4000_f32", "dense", 4000, hq=16, hkv=16, d=64, dtype="f32", vt=False, layout="token"),
        # the last 512 tokens of a chunked prefill over a 64K context
        _case("dense_chunk_64k", "dense", 65536, s0=65024, vt=False, lse=True, layout="token"),
        # a whole dense layer at 32K: the fallback at its full rate
        _case("dense_32k", "dense", 32768),
        # an 8K layer, every head A-shape
        _case("ashape_8k", "ashape", 8192, a=128, b=1024, inputs="mixed"),
        # a 32K layer probed on its last 64 queries, vertical-slash, four heads on the dense fallback
        _case("vslash_32k", "vslash", 32768, vt=False, a=1000, b=6096, dense_heads=4, inputs="mixed"),
        # a chunk of 2048 tokens of a long prompt, vertical-slash, an odd context length
        _case("vslash_chunk_50k", "vslash", 50001, s0=47953, vt=False, lse=True, a=1000, b=512),
        # a 128K layer, block-sparse on every head
        _case("bsparse_128k", "bsparse", 131072, a=100, b=64),
        # a routed layer of a short prompt
        _case("routed_8k", "routed", 8192, seg=2048),
        # a routed layer of medium length, more query heads, an odd last segment
        _case("routed_30k", "routed", 30011, hq=40, hkv=8, seg=8192, lse=True),
        # the headline: a routed 128K layer in 16K segments
        _case("routed_128k", "routed", 131072, seg=16384),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng: random.Random):
    """One more case of the ranges above; half of the lengths are multiples of 64."""
    path = rng.choice(["dense", "dense", "dense", "ashape", "vslash", "vslash", "bsparse", "routed", "routed"])
    hq, hkv = rng.choice([(32, 8), (32, 8), (16, 16), (8, 2), (28, 4), (40, 8), (64, 8)])
    d = rng.choice([128, 128, 128, 64])
    dtype = "bf16"
    hi = {"dense": 32768, "ashape": 65536, "vslash": 32768, "bsparse": 131072, "routed": 98304}[path]
    lo = {"dense": 300, "ashape": 1000, "vslash": 1500, "bsparse": 2000, "routed": 4096}[path]
    # (as many pairs as 32 heads at the longest length, at most)
    n = _log_int(rng, lo, int(hi * math.sqrt(min(1.0, 32.0 / hq))))
    if rng.random() < 0.5:
        n = max(lo, n // 64 * 64)
    s0 = 0
    if path in ("dense", "vslash") and rng.random() < 0.35:  # a chunk of a chunked prefill
        n = max(n, 2 * lo)
        s0 = n - min(n // 2, _log_int(rng, 64, 4096))
    if path in ("dense", "vslash") and rng.random() < 0.2:
        dtype, n, s0 = "f32", min(n, 8192), s0 if n <= 8192 else 0
    a = b = seg = heads = 0
    if path == "ashape":
        a, b = rng.choice([(64, 512), (128, 1024), (128, 4096)])
    elif path == "vslash":
        a, b = rng.choice([(64, 256), (500, 256), (1000, 512), (2000, 2048), (1000, 6096)])
        heads = rng.choice([0, 0, 2, 4])
    elif path == "bsparse":
        a, b = rng.choice([16, 50, 100, 200]), 64
        if a == 200 or hq > 40:
            n = min(n, 65536)
    elif path == "routed":
        seg = rng.choice([2048, 4096]) if n <= 16384 else 8192 if n <= 65536 else 16384
        if hq > 32:
            n = min(n, 65536)
    return _case(None, path, n, hq=hq, hkv=hkv, d=d, dtype=dtype, s0=s0,
                 layout=rng.choice(["head", "head", "token"]),
                 vt=path in ("ashape", "bsparse", "routed") or (path == "dense" and s0 == 0 and rng.random() < 0.5),
                 lse=rng.random() < 0.5, a=a, b=b, dense_heads=heads, seg=seg,
                 inputs="regimes" if path == "routed" else rng.choice(["mixed", "regimes", "regimes"]))


# ---- inputs ------------------------------------------------------------------------------

def _inputs(case, seed):
    """q [hq, n, d], k, v [hkv, n, d]: unit normals, a local band before and sinks and columns
    after the rotary embedding (base 500000, rotate-half), rounded to the case's type."""
    n, hq, hkv, d = case["n"], case["hq"], case["hkv"], case["d"]
    g = torch.Generator(device=DEV).manual_seed(1000003 * seed + 17)
    r = random.Random(seed)
    dt = torch.bfloat16 if case["dtype"] == "bf16" else torch.float32
    half = d // 2
    theta = 500000.0 ** (-2.0 * torch.arange(half, dtype=torch.float64, device=DEV) / d)
    ang = torch.arange(n, dtype=torch.float64, device=DEV)[:, None] * theta[None, :]
    cos, sin = ang.cos().float(), ang.sin().float()
    del ang
    in_band = (theta >= 1e-3) & (theta <= 1e-1)
    band = torch.cat([in_band, in_band]).float()
    band = band / band.norm()
    dirs = torch.randn((d, 2), generator=g, device=DEV) * (band == 0)[:, None]
    dirs = torch.linalg.qr(dirs)[0].T.contiguous()
    amp = lambda x: math.sqrt(max(x, 0.0) * math.sqrt(d))

    def empty(h):
        if case["layout"] == "token":
            return torch.empty((n, h, d), dtype=dt, device=DEV).transpose(0, 1)
        return torch.empty((h, n, d), dtype=dt, device=DEV)

    def rope(x):
        x1, x2 = x[:, :half], x[:, half:]
        return torch.cat([x1 * cos - x2 * sin, x2 * cos + x1 * sin], 1)

    q, k, v = empty(hq), empty(hkv), empty(hkv)
    for kv in range(hkv):
        if case["inputs"] == "mixed":
            lam, sink, vert, nv = 4.0, 4.0, 3.0, 16
        else:
            reg = r.choices(["local", "sink", "vertical", "diffuse"], [0.35, 0.30, 0.28, 0.07])[0]
            lam = 0.0 if reg == "diffuse" else 17.0
            nv = 64
            sink = math.log(1.65 * n / 4) + 4.0 if reg == "sink" else 0.0
            vert = math.log(1.65 * n / nv) + 4.0 if reg == "vertical" else 0.0
        cols = torch.randint(4, n, (nv,), generator=g, device=DEV)
        grp = hq // hkv
        for h in range(kv * grp, (kv + 1) * grp):
            x = rope(torch.randn((n, d), generator=g, device=DEV) + amp(lam) * band)
            q[h] = (x + amp(sink) * dirs[0] + amp(vert) * dirs[1]).to(dt)
        x = rope(torch.randn((n, d), generator=g, device=DEV) + amp(lam) * band)
        x[:4] += amp(sink) * dirs[0]
        x[cols] += amp(vert) * dirs[1]
        k[kv] = x.to(dt)
        v[kv] = torch.randn((n, d), generator=g, device=DEV).to(dt)
    return q, k, v


def _pairs(s0, s1):
    """Causal (row, key) pairs of rows [s0, s1)."""
    return (s1 * (s1 + 1) - s0 * (s0 + 1)) // 2


def _segments(case):
    n, seg = case["n"], case["seg"]
    return [(s, min(n, s + seg)) for s in range(0, n, seg)]


def _grid(case):
    return GRID if case["n"] > 32768 else GRID_SHORT


def _latency_table(case):
    """Per-unit times in us of every candidate for each segment, as profiled offline once: rates
    of the families per million kept pairs on this card, the vertical-slash ones growing with the
    keys that their lines are spread over."""
    t = []
    for fam, a, b in _grid(case):
        row = []
        for s0, s1 in _segments(case):
            rows = s1 - s0
            if fam == 0:
                us = 0.45e-6 * _pairs(s0, s1)
            elif fam == 1:
                us = 0.76e-6 * rows * min(a + b, s1)
            elif fam == 2:
                us = rows / 16384.0 * (20.0 + 13.0 * math.log2(1.0 + s0 / rows)) * (0.5 * a / 500.0 + 0.5 * b / 256.0) ** 0.65
            else:
                us = 0.55e-6 * rows * min(64 * a, s1)
            row.append(us)
        t.append(row)
    return np.array(t)


# ---- state, pass -------------------------------------------------------------------------

class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.case = case
    s.q, s.k, s.v = _inputs(case, seed)
    n, hq, hkv, d = case["n"], case["hq"], case["hkv"], case["d"]
    s0, path = case["s0"], case["path"]
    # not read before a pass writes it; the rows that a chunk does not hold stay zero
    s.lse = torch.zeros((hq, n), dtype=torch.float32, device=DEV) if case["lse"] else None
    if path == "routed":
        s.rl = RoutedLayer(n, hq, hkv, d, case["seg"], _grid(case))
        t = _latency_table(case)
        s.rl.t_table = t
        s.rl.edges = np.array([e for _, e in _segments(case)], np.int32)
        dense = hq * t[0].sum()
        s.rl.t_probe_us = 0.035 * dense
        s.rl.knobs = RouteKnobs(T_layer_us=dense / 6.5, tau=0.95, alpha=1.0, beta=0.0, delta_q=0.03)
        s.rl.qkv(s.q, s.k, s.v)  # the layer's unit tables
        return s
    s.o = torch.zeros((hq, n, d), dtype=torch.bfloat16, device=DEV)
    s.qkv = _rs.make_qkv(s.q, s.k, s.v)
    s.vt = None
    if case["vt"]:
        s.vt = torch.empty(_rs.rs_vt_bytes(s.qkv), dtype=torch.uint8, device=DEV)
        s.qkv.vt = s.vt.data_ptr()
    fam = {"dense": 0, "ashape": 1, "vslash": 2, "bsparse": 3}[path]
    grid = [(0, 0, 0)] + ([(fam, case["a"], case["b"])] if fam else [])
    s.grid, s.ncand = _rs.make_grid(grid), len(grid)
    dense = set(range(0, 5 * case["dense_heads"], 5)) if path == "vslash" else set()
    if path == "dense":
        dense = set(range(hq))
    dense = sorted(h for h in dense if h < hq)
    sparse = [h for h in range(hq) if h not in dense]
    s.nd, s.ns = len(dense), len(sparse)
    s.ud = _rs.make_units([(h, s0, n) for h in dense])
    s.us = _rs.make_units([(h, s0, n, 1, i) for i, h in enumerate(sparse)])
    need = max(_rs.rs_attn_workspace_size(s.qkv, s.ud, s.nd), _rs.rs_attn_workspace_size(s.qkv, s.us, s.ns))
    if path in ("vslash", "bsparse"):
        vs = path == "vslash"
        r = min(64, n - s0) if vs else 0
        s.cfg = _rs.RsProbeCfg(r_rec=r, r_uni=0, r_bnd=0, bs_block=64, local_w=1024,
                               flags=_rs.RS_PROBE_ROWS if vs else _rs.RS_PROBE_BLOCKMEAN)
        s.pb = _rs.ProbeBuffers(s.ns, r, n, hq, blockmean=not vs)
        s.ib = _rs.IndexBuffers(s.ns, n, hq, grid)
        need = max(need, _rs.rs_probe_workspace_size(s.qkv, s.us, s.ns, s.cfg),
                   _rs.rs_build_indices_workspace_size(s.pb, s.grid, s.ncand))
    s.ws = _rs.workspace(need)
    return s


def run(s):
    case, path = s.case, s.case["path"]
    if path == "routed":
        s.rl.run(s.q, s.k, s.v, lse=s.lse, device_route=True)
        out = {"o": s.rl.o, "cov": s.rl.pb.cov, "choice": s.rl.rb.choice}
    else:
        if s.vt is not None:
            _rs.rs_transpose_v(s.qkv, s.vt)
        ib = None
        if path in ("vslash", "bsparse"):
            ib = s.ib
            _rs.rs_probe(s.qkv, s.us, s.ns, s.cfg, None, 0, None, s.ws, s.pb)
            _rs.rs_build_indices(s.pb, s.us, s.ns, s.grid, s.ncand, s.ws, ib)
        if s.ns:
            _rs.rs_sparse_attn_prefill(s.qkv, s.us, s.ns, s.grid, s.ncand, ib, s.o, s.lse, s.ws)
        if s.nd:
            _rs.rs_dense_attn_prefill(s.qkv, s.ud, s.nd, s.o, s.lse, s.ws)
        out = {"o": s.o[:, case["s0"]:]}
        if path == "vslash":
            out.update(col=s.pb.col, diag=s.pb.diag)
        if path == "bsparse":
            out["lbs"] = s.pb.lbs
    if s.lse is not None:
        out["lse"] = s.lse[:, case["s0"]:]
    return out


# ---- work and tolerance ------------------------------------------------------------------

def _kept(fam, a, b, s0, s1):
    """Kept pairs of rows [s0, s1) under a candidate (vertical-slash: columns and diagonals
    spread evenly over the keys)."""
    full = float(_pairs(s0, s1))
    i = np.arange(s0, s1, dtype=np.float64) + 1.0
    if fam == 0:
        return full
    if fam == 1:
        return float(np.minimum(i, a + b).sum())
    if fam == 2:
        return full * (1.0 - max(0.0, 1.0 - a / s1) * max(0.0, 1.0 - b / s1))
    return float(np.minimum(i, 64.0 * a).sum())


def work(case):
    n, s0, hq, hkv, d = case["n"], case["s0"], case["hq"], case["hkv"], case["d"]
    esz = 2 if case["dtype"] == "bf16" else 4
    byt = esz * d * (hq * (n - s0) + 2 * hkv * n) + 2 * hq * (n - s0) * d
    if case["lse"]:
        byt += 4 * hq * (n - s0)
    path, nb = case["path"], (n + 63) // 64
    if path == "routed":
        # sampled rows scored once, pooled scores, and attention at the mean of the sparse budgets
        rows = sum(min(160, e - s) * 0.75 * e for s, e in _segments(case))
        grid = _grid(case)[1:]
        pairs = sum(_kept(*g, s, e) for g in grid for s, e in _segments(case)) / len(grid)
        fl = hq * (2.0 * d * rows + 4.0 * d * pairs + 2.0 * d * nb * (nb + 1) / 2)
    else:
        fam = {"dense": 0, "ashape": 1, "vslash": 2, "bsparse": 3}[path]
        nd = hq if fam == 0 else min(case["dense_heads"], (hq + 4) // 5)
        fl = 4.0 * d * (nd * _pairs(s0, n) + (hq - nd) * (_kept(fam, case["a"], case["b"], s0, n) if fam else 0.0))
        if path == "vslash":
            fl += (hq - nd) * 2.0 * d * min(64, n - s0) * n
            byt += 4 * 2 * (hq - nd) * n
        if path == "bsparse":
            fl += hq * 2.0 * d * nb * (nb + 1) / 2
            byt += 4 * hq * nb * (nb + 1) / 2 + esz * d * hq * s0
    return {"bytes": float(byt), "flops": float(fl)}


def tolerance(case):
    # outputs are bf16 and P is rounded to bf16 before P V
    tol = {"rel": 1e-2}
    if case["path"] == "routed":
        # a unit whose coverage is within a few rounding errors of a threshold may route otherwise
        tol["differ"] = 1e-2
    return tol


# ---- the same results in 64 bits ---------------------------------------------------------

def _softmax_rows(lg, keep):
    """(probabilities, log-sum-exp) of the kept entries of each row."""
    lg = lg.masked_fill(~keep, -math.inf)
    m = lg.max(dim=-1, keepdim=True).values
    p = torch.exp(lg - m)
    z = p.sum(dim=-1, keepdim=True)
    return p / z, (m + torch.log(z)).squeeze(-1)


def _sample_rows(s0, s1, r_rec, r_uni, r_bnd):
    """Sampled rows of a unit (ascending) and their subset: 0 recent, 1 uniform, 2 boundary."""
    r0, ln = max(s0, s1 - r_rec), s1 - s0
    lab = {i: 0 for i in range(r0, s1)}
    for t in range(r_uni):
        i = s0 + ((2 * t + 1) * ln) // (2 * r_uni)
        if i < r0:
            lab.setdefault(i, 1)
    for t in range(r_bnd):
        i = max(s0, 64) + t
        if i < min(s1, r0):
            lab.setdefault(i, 2)
    rows = sorted(lab)
    return rows, [lab[i] for i in rows]


def _top(x, k):
    """Mask of the k largest entries of a vector."""
    m = torch.zeros(x.numel(), dtype=torch.bool, device=x.device)
    if k > 0:
        m[torch.topk(x, min(k, x.numel())).indices] = True
    return m


def _recent_scores(q, k, s0, s1, r_rec, scale):
    """col, diag over keys [0, s1) of the recent rows of one head (64 bits)."""
    rows = torch.arange(max(s0, s1 - r_rec), s1, device=DEV)
    keys = torch.arange(s1, device=DEV)
    p, _ = _softmax_rows(q[rows] @ k[:s1].T * scale, keys[None, :] <= rows[:, None])
    diag = torch.zeros(s1, dtype=torch.float64, device=DEV)
    for x, i in enumerate(rows.tolist()):
        diag[:i + 1] += p[x, :i + 1].flip(0)
    return p.sum(0), diag


def _vs_sets(col, diag, a, b):
    """Kept columns and diagonals as masks (diagonal 0 is always kept)."""
    dm = torch.zeros(diag.numel(), dtype=torch.bool, device=DEV)
    if b >= 1:
        dm[0] = True
        dm[1:] = _top(diag[1:], b - 1)
    return _top(col, a), dm


def _block_scores(q, k, scale):
    """Pooled logits of one head, [nb, nb]."""
    n, nb = q.shape[0], (q.shape[0] + 63) // 64
    def means(x):
        pad = torch.zeros((nb * 64, x.shape[1]), dtype=x.dtype, device=x.device)
        pad[:n] = x
        cnt = torch.full((nb, 1), 64.0, dtype=x.dtype, device=x.device)
        cnt[-1] = n - 64 * (nb - 1)
        return pad.view(nb, 64, -1).sum(1) / cnt
    return means(q) @ means(k).T * scale


def _bs_sets(l, a):
    """Selected key blocks of every query block, [nb, nb] mask: the diagonal and the a - 1 best."""
    nb = l.shape[0]
    eye = torch.eye(nb, dtype=torch.bool, device=DEV)
    low = torch.tril(torch.ones((nb, nb), dtype=torch.bool, device=DEV), -1)
    m = eye.clone()
    if a > 1 and nb > 1:
        x = l.masked_fill(~low, -math.inf)
        top = torch.topk(x, min(a - 1, nb), dim=1).indices
        m.scatter_(1, top, True)
    return m & (low | eye)


def _exact_attn(case, q, k, v, keep_of, heads, o, lse, step=2048):
    """Masked attention of `heads` in 64 bits; keep_of(h, rows, nk): mask [rows, nk] or None."""
    n, grp, scale = case["n"], case["hq"] // case["hkv"], 1.0 / math.sqrt(case["d"])
    for r0 in range(case["s0"], n, step):
        r1 = min(n, r0 + step)
        rows = torch.arange(r0, r1, device=DEV)
        causal = torch.arange(r1, device=DEV)[None, :] <= rows[:, None]
        rel = (rows[:, None] - torch.arange(r1, device=DEV)[None, :]).clamp_(min=0)
        for h in heads:
            kd, vd = k[h // grp, :r1].double(), v[h // grp, :r1].double()
            lg = q[h, r0:r1].double() @ kd.T * scale
            keep = keep_of(h, rows, rel)
            p, z = _softmax_rows(lg, causal if keep is None else causal & keep)
            o[h, r0 - case["s0"]:r1 - case["s0"]] = p @ vd
            lse[h, r0 - case["s0"]:r1 - case["s0"]] = z


def _exact_blocks(case, q, k, v, sel, h, o, lse):
    """Block-sparse attention of one head, 32 query blocks at a time over gathered key blocks."""
    n, grp, scale = case["n"], case["hq"] // case["hkv"], 1.0 / math.sqrt(case["d"])
    nb, ka = sel.shape[0], int(sel.sum(1).max())
    pad = lambda x: torch.cat([x.double(), torch.zeros((nb * 64 - n, x.shape[1]), dtype=torch.float64, device=DEV)])
    qd, kd, vd = pad(q[h]).view(nb, 64, -1), pad(k[h // grp]).view(nb, 64, -1), pad(v[h // grp]).view(nb, 64, -1)
    for b0 in range(0, nb, 32):
        b1 = min(nb, b0 + 32)
        w, blk = torch.sort(sel[b0:b1].to(torch.int8), dim=1, descending=True, stable=True)
        w, blk = w[:, :ka].bool(), blk[:, :ka]
        kk = kd[blk].reshape(b1 - b0, ka * 64, -1)
        vv = vd[blk].reshape(b1 - b0, ka * 64, -1)
        key = (blk[:, :, None] * 64 + torch.arange(64, device=DEV)).reshape(b1 - b0, 1, ka * 64)
        row = (torch.arange(b0, b1, device=DEV)[:, None] * 64 + torch.arange(64, device=DEV))[:, :, None]
        keep = (key <= row) & w.repeat_interleave(64, dim=1)[:, None, :]
        p, z = _softmax_rows(torch.bmm(qd[b0:b1], kk.transpose(1, 2).contiguous()) * scale, keep)
        r1 = min(n, b1 * 64)
        o[h, b0 * 64:r1] = torch.bmm(p, vv).reshape((b1 - b0) * 64, -1)[:r1 - b0 * 64]
        lse[h, b0 * 64:r1] = z.reshape(-1)[:r1 - b0 * 64]


def _exact_cov(case, q, k):
    """Subset means of the retained mass, [units, candidates, 4], of a routed layer."""
    n, hq, grp, scale = case["n"], case["hq"], case["hq"] // case["hkv"], 1.0 / math.sqrt(case["d"])
    grid, segs = _grid(case), _segments(case)
    cov = torch.zeros((len(segs) * hq, len(grid), 4), dtype=torch.float64, device=DEV)
    for h in range(hq):
        qd, kd = q[h].double(), k[h // grp].double()
        l = _block_scores(qd, kd, scale)
        bsel = {c: _bs_sets(l, g[1]) for c, g in enumerate(grid) if g[0] == 3}
        for si, (s0, s1) in enumerate(segs):
            col, diag = _recent_scores(qd, kd, s0, s1, 64, scale)
            rl, lab = _sample_rows(s0, s1, 64, 64, 32)
            rows, lab = torch.tensor(rl, device=DEV), torch.tensor(lab, device=DEV)
            keys = torch.arange(s1, device=DEV)
            causal = keys[None, :] <= rows[:, None]
            p, _ = _softmax_rows(qd[rows] @ kd[:s1].T * scale, causal)
            rel = (rows[:, None] - keys[None, :]).clamp_(min=0)
            for c, (fam, a, b) in enumerate(grid):
                if fam == 0:
                    mi = torch.ones(len(rl), dtype=torch.float64, device=DEV)
                else:
                    if fam == 1:
                        keep = (keys[None, :] < a) | (rel < b)
                    elif fam == 2:
                        vm, dm = _vs_sets(col, diag, a, b)
                        keep = vm[None, :] | dm[rel]
                    else:
                        keep = bsel[c][rows // 64][:, keys // 64]
                    mi = (p * (keep & causal)).sum(1)
                o = cov[si * hq + h, c]
                o[0] = mi.mean()
                for x in range(3):
                    if bool((lab == x).any()):
                        o[1 + x] = mi[lab == x].mean()
    return cov


def exact(case, seed):
    path, n, s0, hq, d = case["path"], case["n"], case["s0"], case["hq"], case["d"]
    grp, scale = hq // case["hkv"], 1.0 / math.sqrt(d)
    if path == "routed":
        # the route is a choice and the attention follows it: the coverage has an exact value
        if hq * n > 40 * 32768:
            return None
        q, k, _ = _inputs(case, seed)
        return {"cov": _exact_cov(case, q, k), "o": None, "choice": None, **({"lse": None} if case["lse"] else {})}
    if path == "ashape" and hq * n * n > 32 * 32768 ** 2:
        return None
    q, k, v = _inputs(case, seed)
    o = torch.zeros((hq, n - s0, d), dtype=torch.float64, device=DEV)
    lse = torch.zeros((hq, n - s0), dtype=torch.float64, device=DEV)
    out = {"o": o}
    a, b = case["a"], case["b"]
    if path == "dense":
        _exact_attn(case, q, k, v, lambda h, rows, rel: None, range(hq), o, lse)
    elif path == "ashape":
        keys = torch.arange(n, device=DEV)
        _exact_attn(case, q, k, v, lambda h, rows, rel: (keys[None, :rel.shape[1]] < a) | (rel < b), range(hq), o, lse)
    elif path == "vslash":
        dense = set(range(0, 5 * case["dense_heads"], 5))
        sparse = [h for h in range(hq) if h not in dense]
        col = torch.zeros((len(sparse), n), dtype=torch.float64, device=DEV)
        diag = torch.zeros_like(col)
        sets = {}
        for x, h in enumerate(sparse):
            col[x], diag[x] = _recent_scores(q[h].double(), k[h // grp].double(), s0, n, min(64, n - s0), scale)
            sets[h] = _vs_sets(col[x], diag[x], a, b)

        def keep_of(h, rows, rel):
            return None if h in dense else sets[h][0][None, :rel.shape[1]] | sets[h][1][rel]
        _exact_attn(case, q, k, v, keep_of, range(hq), o, lse)
        out.update(col=col, diag=diag)
    else:
        nb = (n + 63) // 64
        low = torch.tril_indices(nb, nb, device=DEV)
        out["lbs"] = torch.zeros((hq, nb * (nb + 1) // 2), dtype=torch.float64, device=DEV)
        for h in range(hq):
            l = _block_scores(q[h].double(), k[h // grp].double(), scale)
            out["lbs"][h] = l[low[0], low[1]]
            _exact_blocks(case, q, k, v, _bs_sets(l, a), h, o, lse)
    if case["lse"]:
        out["lse"] = lse
    return out

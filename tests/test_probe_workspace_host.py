"""The probe accepts a workspace of exactly the size that its query returns, for every length, head
count, number of sampled rows and flag, in scores and in coverage calls, and any workspace that an
earlier query's formula (ranges of 1024 keys) gave.

A call's workspace is checked before its first launch, so a process without a GPU sees either
RS_ERR_WORKSPACE (refused) or RS_ERR_HIP (accepted, nothing to launch on).  The calls run in a child
process that hides every GPU: the pointers are not memory, and no kernel may see them."""
import os
import subprocess
import sys

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))

CHILD = r"""
import ctypes as C
import random
from paper_2608_29058_amd import _rs

L = _rs.lib()
P = 1 << 20  # a 16-byte aligned address that nothing reads


def calls(n, hq, hkv, segs, rc, flags, dtype=0, d=128):
    seg = -(-n // segs)
    units = [(h, s, min(n, s + seg)) for s in range(0, n, seg) for h in range(hq)]
    U, nb, rmax = len(units), (n + 63) // 64, sum(rc)
    qkv = _rs.RsQkv(q=P, k=P, v=P, dtype=dtype, n=n, hq=hq, hkv=hkv, d=d, sq_h=n * d, sq_t=d, sk_h=n * d, sk_t=d,
                    sv_h=n * d, sv_t=d)
    u = _rs.make_units(units)
    cfg = _rs.RsProbeCfg(r_rec=rc[0], r_uni=rc[1], r_bnd=rc[2], bs_block=64, local_w=1024, flags=flags)
    grid = _rs.make_grid([(0, 0, 0), (1, 64, 256)])
    out = _rs.RsProbeOut(nunits=U, rmax=rmax, n=n, nb=nb, ncand=2, hq=hq, rows=P, subset=P, nsub=P, row_max=P,
                         row_sum=P, col=P, diag=P, entropy=P, local=P, lbs=P, cov_rows=P, cov=P)
    idx = _rs.RsIndexSet(nunits=U, n=n, nb=nb, hq=hq)
    need = L.rs_probe_workspace_size(C.byref(qkv), u, U, C.byref(cfg))
    up = lambda x: -(-x // 256) * 256
    nch = -(-n // 1024)
    part = U * nch * rmax * 4
    longest = (up(U * 32) + up(U * 16) + up(U * nch * (1024 + rmax) * 4) + 4 * up(part) + up(part * 16) + 256
               + (up(hq * nb * d * 4) + up(hkv * nb * d * 4) if flags & 2 else 0))
    bad = []
    for what, size in (("query", need), ("ranges of 1024", longest)):
        for cover in (False, True) if rmax else (False,):
            st = L.rs_probe(C.byref(qkv), u, U, C.byref(cfg), grid if cover else None, 2 if cover else 0,
                            C.byref(idx) if cover else None, C.c_void_p(P), size, C.byref(out), None)
            if st != _rs.RS_ERR_HIP:
                bad.append((what, cover, st, L.rs_last_error()))
    st = L.rs_probe(C.byref(qkv), u, U, C.byref(cfg), None, 0, None, C.c_void_p(P), 256, C.byref(out), None)
    if st != _rs.RS_ERR_WORKSPACE:
        bad.append(("256 bytes", st))
    return bad


r = random.Random(7)
heads = [(32, 8), (16, 16), (64, 8), (40, 8), (28, 4), (8, 2), (32, 32), (1, 1)]
cases = [(20000, 32, 8, 1, (0, 0, 0), 2), (49500, 32, 8, 1, (0, 0, 0), 2), (12507, 32, 32, 1, (1, 0, 0), 1),
         (1064, 32, 32, 8, (8, 4, 4), 1), (30, 32, 32, 1, (64, 64, 32), 3)]
for i in range(500):
    rc = r.choice([(0, 0, 0), (0, 0, 0), (1, 0, 0), (2, 0, 0), (8, 0, 0), (64, 0, 0), (64, 64, 32), (0, 8, 0), (100, 100, 56)])
    n = int(2 ** r.uniform(0, 18))
    if i % 2:
        n = max(1, n // 64 * 64)
    cases.append((n, *heads[i % len(heads)], r.choice([1, 1, 2, 5, 16]), rc, 2 if sum(rc) == 0 else r.choice([1, 3])))
for c in cases:
    bad = calls(*c)
    assert not bad, (c, bad)
print("checked", len(cases))
"""


def test_a_workspace_of_the_queried_size_is_accepted():
    env = dict(os.environ, HIP_VISIBLE_DEVICES="-1", ROCR_VISIBLE_DEVICES="-1", PYTHONPATH=ROOT)
    if os.path.exists("/dev/kfd"):
        pytest.skip("needs a machine without a GPU")
    p = subprocess.run([sys.executable, "-c", CHILD], capture_output=True, text=True, env=env, cwd=ROOT, timeout=600)
    assert p.returncode == 0 and "checked" in p.stdout, p.stdout[-500:] + p.stderr[-2000:]

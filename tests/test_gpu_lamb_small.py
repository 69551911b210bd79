"""GPU test of the one-launch LAMB step (shards of up to 1M elements, at most 8
layer pieces a workgroup) at the edges of its workgroups (1024, 2048 and 4096
elements), of its grids (256 workgroups of each size) and just past them, with
layers that end at, before and after those edges, one-element layers, a layer
over the whole shard, unequal array offsets, an overflow, and a table too fine
for it, which keeps the kernel sequence; zero_shard_last_step_stats tells which
ran.  Against the oracle (exact layer norms): every fp32 operation of the update
is correctly rounded in the oracle's order and a layer's fp32 step size comes from
fp64 norms, so the bound is the repository's 1e-6 and the observed difference is
zero bits."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import gpu_harness as H  # noqa: E402

from paper_1910_02054_amd import workloads  # noqa: E402

pytestmark = pytest.mark.gpu
HP = (1e-3, 0.9, 0.999, 1e-8, 0.01)
T = 1024
NONE, ALL = (0,) * 5, (3, 1, 1, 1, 2)


def _table(n, cuts):
    return np.unique(np.concatenate([[0], [c for c in cuts if 0 < c < n], [n]])).astype(np.int64)


@pytest.mark.parametrize("n,cuts,shifts,overflow,path", [
    (1, [], NONE, False, 1),
    (T - 1, [1, 2, 500], NONE, False, 1),
    (T, [T // 2], NONE, False, 1),
    (T + 1, [T - 1, T], ALL, False, 1),
    (3 * T + 2, [31, 32, T, T + 1, 2 * T + 1], ALL, False, 1),
    (256 * T, [5 * T, 100 * T + 7, 255 * T + 1], NONE, False, 1),
    (256 * T + 5, [T + 3, 256 * T + 4], NONE, True, 1),
    (512 * T, [2 * T, 2 * T + 1, 511 * T], ALL, False, 1),
    (512 * T + 9, [300 * T], NONE, False, 1),
    (1024 * T, [1, 4 * T - 1, 4 * T, 4 * T + 1, 700 * T], NONE, False, 1),
    (1024 * T, [], ALL, False, 1),
    (1024 * T + 40, [77], NONE, False, 0),
    (40 * T, [T + 10 * k for k in range(9)], NONE, False, 0),
])
def test_one_launch_lamb_step(n, cuts, shifts, overflow, path):
    import torch
    from paper_1910_02054_amd import binding as zb
    dts = (torch.float16, torch.float32, torch.float32, torch.float32, torch.float16)
    bufs = [H.Guarded(torch, n, dt, torch.device("cuda:0"), shift=s) for dt, s in zip(dts, shifts)]
    g16, theta, m, v = workloads.random_case(111, n)
    host = [g16, theta, m, v, workloads.p16_sentinel(n)]
    for b, a in zip(bufs, host):
        b.upload(a)
    ref = [a.copy() for a in host[1:]]
    seg = _table(n, cuts)
    with zb.LambPlan(seg) as plan:
        for t in (1, 2, 3):
            g = g16.copy()
            if overflow and t == 2:
                g[n - 1] = workloads.F16_QNAN
            bufs[0].upload(g)
            flag = zb.zero_lamb_step(plan, *(b.view for b in bufs), *HP, t, 2.0 ** 16, 1.0)
            skip, sc, _ = H.oracle_lamb_step(g, *ref, seg, *HP, t, 2.0 ** 16, 1.0)
            st = zb.zero_shard_last_step_stats()
            assert flag == skip == (1 if overflow and t == 2 else 0) and st.path == path, st.path
            assert skip or st.mult == sc.mult
            torch.cuda.synchronize()
    d = H.compare_state([b.download() for b in bufs[1:]], ref)
    assert all(b.guards_intact() for b in bufs)
    print("[gpu-lamb-small] n=%d layers=%d %s" % (n, seg.size - 1, d), flush=True)

"""GPU test of the LAMB layer sums at the edges of their two levels (1024 tile
pieces of 512 elements a chunk): layers of one chunk, of exactly one, of two and
of more than 64 chunks, next to one-element layers, called twice so that the
slots one call drained serve the next, and the split phase's sums in caller
memory.  The oracle's layer sums are exact; the kernels add fp64 squares, so
1e-13 bounds the relative difference (a few thousand additions a partial, each
off by at most 2^-53).  The asynchronous Adam update that derives its multiplier
in place is compared on both sides of its limit (8M elements) and with its flag
stored over the sum itself."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import gpu_harness as H  # noqa: E402

from paper_1910_02054_amd import workloads  # noqa: E402

pytestmark = pytest.mark.gpu
HP = (1e-3, 0.9, 0.999, 1e-8, 0.01)
C = 1024 * 512


@pytest.mark.parametrize("sizes", [[C - 1, 1, C], [C + 1, 3, 2 * C], [1, 66 * C + 5, 700]])
def test_layer_sums_across_chunks(sizes):
    import torch
    from paper_1910_02054_amd import binding as zb
    seg = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(seg[-1])
    dts = (torch.float16, torch.float32, torch.float32, torch.float32, torch.float16)
    bufs = [H.Guarded(torch, n, dt, torch.device("cuda:0")) for dt in dts]
    g16, theta, m, v = workloads.random_case(101, n)
    host = [g16, theta, m, v, workloads.p16_sentinel(n)]
    for b, a in zip(bufs, host):
        b.upload(a)
    ref = [a.copy() for a in host[1:]]
    out = torch.zeros(2 * len(sizes), dtype=torch.float64, device="cuda")
    with zb.LambPlan(seg) as plan:
        for t in (1, 2):
            views = [b.view for b in bufs]
            if t == 1:
                total = zb.zero_shard_stats(views[0])
                zb.zero_lamb_moments(plan, *views[:4], total, *HP[1:], t, 2.0 ** 16, 1.0, out)
                zb.zero_lamb_apply(plan, *views[1:], total, out, *HP, t)
            else:
                assert zb.zero_lamb_step(plan, *views, *HP, t, 2.0 ** 16, 1.0) == 0
            old = ref[0].astype(np.float64)
            H.oracle_lamb_step(g16, *ref, seg, *HP, t, 2.0 ** 16, 1.0)
            if t == 1:
                torch.cuda.synchronize()
                got = out.cpu().numpy().reshape(-1, 2)
                for k in range(len(sizes)):
                    want = float(np.sum(np.square(old[seg[k]:seg[k + 1]]).astype(np.longdouble)))
                    assert abs(got[k, 0] / want - 1.0) <= 1e-13, (k, got[k, 0], want)
        torch.cuda.synchronize()
    d = H.compare_state([b.download() for b in bufs[1:]], ref)
    assert all(b.guards_intact() for b in bufs)
    print("[gpu-lamb-sums] sizes=%s %s" % (sizes, d), flush=True)


@pytest.mark.parametrize("n,flag_on_sum", [(1000, False), (1000, True), (1 << 23, False), ((1 << 23) + 300, False)])
def test_async_update_takes_the_sum_where_it_lies(n, flag_on_sum):
    import torch
    from paper_1910_02054_amd import binding as zb
    dts = (torch.float16, torch.float32, torch.float32, torch.float32, torch.float16)
    bufs = [H.Guarded(torch, n, dt, torch.device("cuda:0")) for dt in dts]
    g16, theta, m, v = workloads.random_case(102, n)
    host = [g16, theta, m, v, workloads.p16_sentinel(n)]
    for b, a in zip(bufs, host):
        b.upload(a)
    ref = [a.copy() for a in host[1:]]
    total = torch.zeros(1, dtype=torch.float64, device="cuda")
    flag = total.view(torch.int32)[:1] if flag_on_sum else torch.full((1,), -1, dtype=torch.int32, device="cuda")
    for t in (1, 2):
        zb.zero_shard_stats_async(bufs[0].view, total)
        zb.zero_shard_apply_async(*(b.view for b in bufs), total, *HP, t, 2.0 ** 16, 1.0, skipped=flag)
        H.oracle_step(g16, *ref, *HP, t, 2.0 ** 16, 1.0)
        assert flag.item() == 0
    for bad in (float("nan"), -1.0, float("inf")):   # skipped: nothing may change
        total.fill_(bad)
        zb.zero_shard_apply_async(*(b.view for b in bufs), total, *HP, 3, 2.0 ** 16, 1.0, skipped=flag)
        assert flag.item() == 1
    d = H.compare_state([b.download() for b in bufs[1:]], ref)
    assert all(b.guards_intact() for b in bufs)
    print("[gpu-async] n=%d %s" % (n, d), flush=True)

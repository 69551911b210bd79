"""GPU test of what follows when a workgroup stops waiting for another one's sums.
build() makes the library a second time with waits that end at the first empty
slot, so that the closing workgroup of the statistics and of a layer's sums hands
over to a late one in nearly every launch (as it does after some thousand polls
when other work keeps a late workgroup off the device).  The sums are added in the same order
whichever workgroup closes them, so every result equals the ordinary library's bit
for bit, call after call: a slot that one call left filled, or a total that a call
gave up on, would show in the next.  Gradients change from call to call, with
overflows among them, so a sum of an earlier call is never the right one."""
import importlib.util
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import gpu_harness as H  # noqa: E402

from paper_1910_02054_amd import build as zbuild  # noqa: E402
from paper_1910_02054_amd import workloads  # noqa: E402

pytestmark = pytest.mark.gpu
HP = (1e-3, 0.9, 0.999, 1e-8, 0.01)
W = 64 * 4 * 8          # gradient elements a workgroup of the statistics reads per round
C = 1024 * 512          # elements whose LAMB layer sums one workgroup adds


@pytest.fixture(scope="module")
def libs():
    """The binding on the ordinary library, and a second one on the impatient build."""
    import torch
    from paper_1910_02054_amd import binding
    assert torch.cuda.is_available()
    ordinary = zbuild.LIB
    try:
        zbuild.LIB = zbuild.IMPATIENT_LIB
        spec = importlib.util.spec_from_file_location("paper_1910_02054_amd.binding_impatient", binding.__file__)
        other = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(other)
    finally:
        zbuild.LIB = ordinary
    assert other.LIB_PATH != binding.LIB_PATH
    return torch, binding, other


def _gradients(torch, n, seed, count=4):
    out = []
    for k in range(count):
        g16 = workloads.random_case(seed + k, n)[0]
        if k == count - 2:
            g16[(7919 * seed) % n] = workloads.F16_POS_INF
        out.append(torch.from_numpy(g16.view(np.int16)).cuda().view(torch.float16))
    return out


def _state(torch, n, seed):
    _, theta, m, v = workloads.random_case(seed, n)
    return [torch.from_numpy(a).cuda() for a in (theta, m, v)] + [torch.zeros(n, dtype=torch.float16, device="cuda")]


def _equal(torch, a, b):
    return all(torch.equal(x.view(torch.int16), y.view(torch.int16)) for x, y in zip(a, b))


@pytest.mark.parametrize("n", [W + 1, 64 * W, 64 * W + 8, 65 * W - 5, 2048 * W + 8, 9_000_017])
def test_statistics_closed_by_a_late_workgroup(libs, n):
    torch, zb, zi = libs
    grads = _gradients(torch, n, 301)
    want = [zb.zero_shard_stats(g) for g in grads]
    out = torch.zeros(1, dtype=torch.float64, device="cuda")
    for _ in range(25):
        for g, s in zip(grads, want):
            zi.zero_shard_stats_async(g, out)
            got = zi.zero_shard_stats(g)
            assert (got == s or not np.isfinite(s) and not np.isfinite(got)), (n, got, s)
            assert out.item() == got or not np.isfinite(got) and not np.isfinite(out.item()), (n, out.item(), got)


@pytest.mark.parametrize("n", [20_003, 3_000_017])
@pytest.mark.parametrize("graph", [False, True])
def test_resident_steps_closed_by_a_late_workgroup(libs, n, graph):
    torch, zb, zi = libs
    grads = _gradients(torch, n, 311)
    states = [_state(torch, n, 321) for _ in range(2)]
    records = [zb.resident_state(torch.device("cuda:0"), *HP, 1.0, 2.0 ** 16, window=5) for _ in range(2)]
    g16 = grads[0].clone()
    if graph:
        captured = torch.cuda.CUDAGraph()
        with torch.cuda.graph(captured):
            zi.zero_shard_step_resident(g16, *states[1], records[1])
    for k in range(40):
        g16.copy_(grads[k % 4])
        zb.zero_shard_step_resident(g16, *states[0], records[0])
        if graph:
            captured.replay()
        else:
            zi.zero_shard_step_resident(g16, *states[1], records[1])
        assert torch.equal(*records), (k, zb.read_resident_state(records[1]).skipped)
    assert zb.read_resident_state(records[1]).steps == 40 and zb.read_resident_state(records[1]).t == 31
    assert _equal(torch, *states)
    torch.cuda.synchronize()
    zb.zero_resident_release(records[0])
    zi.zero_resident_release(records[1])


def test_fused_and_asynchronous_steps_closed_by_a_late_workgroup(libs):
    torch, zb, zi = libs
    n = 2_500_009
    grads = _gradients(torch, n, 331)
    states = [_state(torch, n, 341) for _ in range(2)]
    total = torch.zeros(1, dtype=torch.float64, device="cuda")
    flag = torch.zeros(1, dtype=torch.int32, device="cuda")
    for k in range(40):
        g = grads[k % 4]
        skip = zb.zero_shard_step(g, *states[0], *HP, k + 1, 2.0 ** 16, 1.0)
        assert skip == (k % 4 == 2)
        if k % 3 == 0:
            got = zi.zero_shard_step(g, *states[1], *HP, k + 1, 2.0 ** 16, 1.0)
        elif k % 3 == 1:
            got = zi.zero_shard_step_noalloc(g, *states[1], *HP, k + 1, 2.0 ** 16, 1.0)
        else:
            zi.zero_shard_stats_async(g, total)
            zi.zero_shard_apply_async(g, *states[1], total, *HP, k + 1, 2.0 ** 16, 1.0, skipped=flag)
            got = flag.item()
        assert got == skip, (k, got, skip)
    assert _equal(torch, *states)


@pytest.mark.parametrize("sizes", [[C + 1, 3, 2 * C], [1, 66 * C + 5, 700]])
def test_layer_sums_closed_by_a_late_workgroup(libs, sizes):
    torch, zb, zi = libs
    seg = np.concatenate([[0], np.cumsum(sizes)]).astype(np.int64)
    n = int(seg[-1])
    grads = _gradients(torch, n, 351, count=2)      # the first one overflows
    states = [_state(torch, n, 361) for _ in range(2)]
    sums = [torch.zeros(2 * len(sizes), dtype=torch.float64, device="cuda") for _ in range(2)]
    with zb.LambPlan(seg) as plan, zi.LambPlan(seg) as impatient:
        for k in range(24):
            g = grads[k % 5 != 1]
            for lib, p, state, out in ((zb, plan, states[0], sums[0]), (zi, impatient, states[1], sums[1])):
                if k % 2 == 0:
                    total = zb.zero_shard_stats(g)
                    lib.zero_lamb_moments(p, g, *state[:3], total, *HP[1:], k + 1, 2.0 ** 16, 1.0, out)
                    lib.zero_lamb_apply(p, *state, total, out, *HP, k + 1)
                else:
                    assert lib.zero_lamb_step(p, g, *state, *HP, k + 1, 2.0 ** 16, 1.0) == (k % 5 == 1)
            assert torch.equal(*sums), (k, sums)
            if k % 8 == 7:
                assert _equal(torch, *states), k
        torch.cuda.synchronize()


@pytest.mark.parametrize("entry", ["step", "noalloc", "lamb"])
def test_one_launch_steps_that_stop_waiting(libs, entry):
    # a one-launch step that gives its exchange up has written nothing, and the kernel sequence takes
    # the step; LAMB's layers run on from workgroup to workgroup
    torch, zb, zi = libs
    n = 200 * 1024
    grads = _gradients(torch, n, 371)
    states = [_state(torch, n, 381) for _ in range(2)]
    seg = np.unique(np.concatenate([[0], np.arange(1, n, 256), [n]])).astype(np.int64)
    paths = [0, 0]
    with zb.LambPlan(seg) as plan, zi.LambPlan(seg) as impatient:
        for k in range(200):
            for lib, p, state in ((zb, plan, states[0]), (zi, impatient, states[1])):
                args = (grads[k % 4], *state, *HP, k + 1, 2.0 ** 16, 1.0)
                if entry == "lamb":
                    skip = lib.zero_lamb_step(p, *args)
                else:
                    skip = (lib.zero_shard_step if entry == "step" else lib.zero_shard_step_noalloc)(*args)
                assert skip == (k % 4 == 2), k
            assert zb.zero_shard_last_step_stats().path == 1
            paths[zi.zero_shard_last_step_stats().path] += 1
            assert _equal(torch, *states), (k, paths)
        torch.cuda.synchronize()
    print("[gpu-handover] %s: %d of 200 one-launch steps given up" % (entry, paths[0]), flush=True)
    assert paths[0] > 0

"""GPU test of the update direction at the limits of its short division and
square-root sequences: moments drawn over all fp32 magnitudes, just inside and
just outside the range that takes them, zeros, subnormals, infinities and NaN
among them, and bias corrections too small for them.  Both sequences are
correctly rounded, so the fp32 state equals the oracle's bit for bit (a NaN is
compared as a NaN)."""
import os
import sys

import numpy as np
import pytest

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
import gpu_harness as H  # noqa: E402

from paper_1910_02054_amd import workloads  # noqa: E402

pytestmark = pytest.mark.gpu


def _moments(kind, n, rng):
    def mag(lo, hi):
        return np.ldexp(1.0 + rng.random(n), rng.integers(lo, hi, n)).astype(np.float32)
    if kind == "usual":
        m, v = mag(-78, 38), mag(-98, 58)
    elif kind == "edges":
        m, v = mag(-83, -77), mag(-103, -97)
        m[::2], v[1::3] = mag(38, 42)[::2], mag(58, 62)[1::3]
    else:
        m, v = mag(-149, 127), mag(-149, 127)
        m[::7], v[::11] = 0.0, 0.0
        m[5::97], v[9::101] = np.inf, np.inf
        m[11::211] = np.nan
    return np.where(rng.random(n) < 0.5, m, -m).astype(np.float32), v


@pytest.mark.parametrize("kind", ["usual", "edges", "any"])
@pytest.mark.parametrize("beta1,beta2,eps,t", [(0.9, 0.999, 1e-8, 1), (0.9, 0.999, 0.0, 3000), (0.0, 0.5, 1e-3, 7),
                                               (1.0 - 2.0 ** -30, 1.0 - 2.0 ** -28, 1e-8, 2)])
@pytest.mark.parametrize("n", [40_003, 1_700_003])
def test_direction_equals_the_general_operations(kind, beta1, beta2, eps, t, n):
    import torch
    from paper_1910_02054_amd import binding as zb
    rng = np.random.default_rng(131 + n)
    g16, theta, _, _ = workloads.random_case(132, n)
    m, v = _moments(kind, n, rng)
    dts = (torch.float16, torch.float32, torch.float32, torch.float32, torch.float16)
    bufs = [H.Guarded(torch, n, dt, torch.device("cuda:0")) for dt in dts]
    host = [g16, theta, m, v, workloads.p16_sentinel(n)]
    for b, a in zip(bufs, host):
        b.upload(a)
    ref = [a.copy() for a in host[1:]]
    hp = (1e-3, beta1, beta2, eps, 0.01, t)
    with np.errstate(all="ignore"):
        flag = zb.zero_shard_step(*(b.view for b in bufs), *hp, 2.0 ** 16, 1.0)
        skip, _ = H.oracle_step(g16, *ref, *hp, 2.0 ** 16, 1.0)
    torch.cuda.synchronize()
    assert flag == skip == 0
    for name, b, r in zip(("master", "m", "v"), bufs[1:4], ref[:3]):
        a = b.download()
        same = (a.view(np.uint32) == r.view(np.uint32)) | (np.isnan(a) & np.isnan(r))
        assert same.all(), (name, a[~same][:4], r[~same][:4], m[~same][:4], v[~same][:4])
    assert all(b.guards_intact() for b in bufs)
    print("[gpu-direction] %s n=%d beta1=%g eps=%g same" % (kind, n, beta1, eps), flush=True)

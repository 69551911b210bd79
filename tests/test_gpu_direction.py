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


@pytest.mark.parametrize("beta2,scale,lo,hi", [(2.0 ** -30, 0, -100, 60), (1.0 - 2.0 ** -24, 24, 36, 60)])
def test_square_root_of_every_float_of_the_short_sequence(beta2, scale, lo, hi):
    # every second moment w of the short sequence's range [2^-100, 2^60) as its own root's argument (1 - beta2
    # rounds to 1), and those that 1 - beta2 = 2^-24 takes to [2^60, 2^84).  The root s is seen through the
    # division by it: m is 1/16 of the correctly rounded root (numpy's, of two binades; the others are theirs
    # times a power of two), and m / s is 1/16 exactly if and only if s is that root, since a quotient of
    # different floats differs from 1 by at least 2^-24.
    import torch
    from paper_1910_02054_amd import binding as zb
    mant = 1 << 23
    one = np.float32(1.0).view(np.int32)
    root = [torch.from_numpy(np.sqrt(np.arange(one, one + mant, dtype=np.int32).view(np.float32) *
                                     np.float32(2 ** odd))).cuda() for odd in (0, 1)]
    bits = torch.arange(mant, dtype=torch.int32, device="cuda")
    per = 4                                                # binades a step
    n = per * mant
    g, p16 = (torch.zeros(n, dtype=torch.float16, device="cuda") for _ in range(2))
    theta, m, v = (torch.empty(n, dtype=torch.float32, device="cuda") for _ in range(3))
    for first in range(lo, hi, per):
        theta.zero_()
        for k in range(per):
            e, part = first + k, slice(k * mant, (k + 1) * mant)
            w = bits + ((e + 127) << 23)
            if scale:                                      # beta2 times the next float above w rounds to w
                v[part] = (w + 1).view(torch.float32)
                assert first > lo or torch.equal(v[part] * np.float32(beta2).item(), w.view(torch.float32))
            else:
                v[part] = w.view(torch.float32) * 2.0 ** 30
            # beta1 = 1/2: the kernel halves m, and the bias correction doubles it again
            m[part] = root[e % 2] * 2.0 ** ((e - e % 2 + scale) // 2 - 4)
        assert zb.zero_shard_step(g, theta, m, v, p16, 1.0, 0.5, beta2, 0.0, 0.0, 1, 1.0, 0.0) == 0
        wrong = torch.nonzero(theta != -0.0625)
        assert wrong.numel() == 0, (first, v[wrong[0]], theta[wrong[0]], wrong.numel())
    print("[gpu-direction] roots of %d floats equal" % ((hi - lo) * mant), flush=True)

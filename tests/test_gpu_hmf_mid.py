"""HMF passes at the edges of their particles a block (256 .. 2048), vector widths and
sums (in the pass or by a one-block kernel), against the oracle.

Tolerances: FP64 states 1e-11, products and sweeps 1e-10 (an O(N) sum reordered, terms of
order 1), the FP32 state 1e-5 (2^-24 a stage on angles and momenta of order 1).
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import dev, gpu_run, host
from paper_1212_0262_amd import inputs, md

pytestmark = pytest.mark.gpu


def shifted(a):
    """The array on the device at an address that is 8- but not 16-byte aligned."""
    t = torch.empty(a.size + 1, dtype=torch.float64, device="cuda")[1:].view(a.shape)
    return t.copy_(dev(a))


# block sizes change past 262144, 524288, 1048576 (in-pass sums up to 2097152)
@pytest.mark.parametrize("n", [8193, 262_144, 262_145, 262_147, 524_289, 1_048_577, 2_097_155])
@pytest.mark.parametrize("prec,tol", [(md.FP64, 1e-11), (md.MIXED_F32STATE, 1e-5)])
def test_steps(n, prec, tol):
    q, p = inputs.hmf_waterbag(n, seed=n)
    f = oracle.force(md.HMF, q)
    qo, po, fo = oracle.step(md.HMF, q, p, f, 0.1, 2, 0.0)
    qg, pg, fg, _ = gpu_run(md.HMF, prec, q, p, 0.0, 0.1, 2)
    for a, b in ((qg, qo), (pg, po), (fg, fo)):
        assert np.abs(a - b).max() < tol
    for a, b in zip((qg, pg, fg), gpu_run(md.HMF, prec, q, p, 0.0, 0.1, 2, chunks=2)):
        np.testing.assert_array_equal(a, b)
    ctx = md.md_init(md.HMF, prec, n)
    qs, ps, fs = shifted(q), shifted(p), shifted(np.zeros_like(q))
    md.md_force(ctx, qs, fs)
    md.md_step(ctx, qs, ps, fs, 0.1, 2)
    for a, b in ((qs, qo), (ps, po), (fs, fo)):
        assert np.abs(host(a) - b).max() < tol
    ctx.close()


def product(q, w):
    """H(q) w by the mean-field identity of eqs. 6-7 (the oracle's is O(N^2))."""
    c, s = np.cos(q), np.sin(q)
    return w * (c * c.mean() + s * s.mean()) - (c * (c * w).mean() + s * (s * w).mean())


def sweep(q, p, dt, steps, lq, lp):
    """The reverse sweep, stage by stage, over the oracle's coefficients."""
    b0, b1, d0, d1 = (x * dt for x in oracle.yoshida())
    q, p, f, at = q.copy(), p.copy(), oracle.force(md.HMF, q), []
    stages = [(b0, d0), (b1, d1), (b1, d0), (b0, 0.0)] * steps
    for kick, drift in stages:
        p += kick * f
        at.append(q.copy())
        if drift:
            q += drift * p
            f = oracle.force(md.HMF, q)
    for (kick, drift), x in zip(reversed(stages), reversed(at)):
        lp = lp + drift * lq
        lq = lq - kick * product(x, lp)
    return lq, lp


# block sizes of the product's passes change past 131072, 262144, 524288; the sums leave
# the pass past 1048576
@pytest.mark.parametrize("n", [500, 8193, 131_072, 131_075, 262_145, 524_289, 1_048_576, 1_048_577])
def test_products_and_sweep(n):
    q, p = inputs.hmf_waterbag(n, seed=n)
    rng = np.random.default_rng(n)
    lq, lp = rng.normal(size=(1, n)), rng.normal(size=(1, n))
    ctx = md.md_init(md.HMF, md.FP64, n)
    ho, want = product(q, lq), sweep(q, p, 0.1, 2, lq, lp)
    if n == 500:
        assert np.abs(ho - oracle.hvp(md.HMF, q, lq, 0.0)).max() < 1e-12
        for a, b in zip(want, oracle.step_vjp(md.HMF, q, p, 0.1, 2, lq, lp, 0.0)):
            assert np.abs(a - b).max() < 1e-12
    for move in (dev, shifted):
        assert np.abs(host(md.md_hvp(ctx, move(q), move(lq))) - ho).max() < 1e-10
        a, b = move(lq), move(lp)
        md.md_step_vjp(ctx, move(q), move(p), 0.1, 2, a, b)
        assert max(np.abs(host(x) - y).max() for x, y in zip((a, b), want)) < 1e-10
    ctx.close()

"""HMF systems that one workgroup takes whole (n <= 8192): every number of particles a
thread (1, 2, 4, 8, 32) and its edges, both states, against the oracle and, at the edge, the
form that larger systems take.

Tolerances: FP64 trajectories 1e-11 and energies 1e-12 of K + |V| + n/2, the FP32 state
1e-5 (positions and momenta of order 1, 2^-24 a stage), as the parity tests.
"""
import ctypes

import numpy as np
import pytest
import torch

import oracle
from gpu_helpers import dev, gpu_run, host
from paper_1212_0262_amd import inputs, md

pytestmark = pytest.mark.gpu
SIZES = [1, 2, 63, 64, 65, 256, 257, 512, 513, 1024, 1025, 2049, 4095, 4096, 4097, 8191, 8192, 8193]


@pytest.mark.parametrize("n", SIZES)
@pytest.mark.parametrize("prec,tol", [(md.FP64, 1e-11), (md.MIXED_F32STATE, 1e-5)])
def test_steps_force_energy(n, prec, tol):
    q, p = inputs.hmf_waterbag(n, seed=n)
    f = oracle.force(md.HMF, q)
    qo, po, fo = oracle.step(md.HMF, q, p, f, 0.1, 7, 0.0)
    eo = np.asarray(oracle.energy(md.HMF, qo, po))
    qg, pg, fg, eg = gpu_run(md.HMF, prec, q, p, 0.0, 0.1, 7)
    for a, b in ((qg, qo), (pg, po), (fg, fo)):
        assert np.abs(a - b).max() < tol
    assert np.abs(eg[-1] - eo).max() < max(1e-12, tol) * (abs(eo[0]) + abs(eo[1]) + n / 2)
    for chunks in (7, 2):  # one call or several: the same bits
        for a, b in zip((qg, pg, fg), gpu_run(md.HMF, prec, q, p, 0.0, 0.1, 7, chunks=chunks)):
            np.testing.assert_array_equal(a, b)


@pytest.mark.parametrize("n", SIZES)
def test_same_sums_everywhere(n):
    """The force after a step is md_force's, and md_force_noalloc's, bit for bit."""
    q, p = (dev(x) for x in inputs.hmf_waterbag(n, seed=n))
    ctx = md.md_init(md.HMF, md.FP64, n)
    f, g, h = (torch.empty_like(q) for _ in range(3))
    md.md_force(ctx, q, f)
    md.md_step(ctx, q, p, f, 0.1, 3)
    md.md_force(ctx, q, g)
    md.md_force_noalloc(md.HMF, md.FP64, q, 0.0, h)
    assert torch.equal(f, g) and torch.equal(f, h)
    m = host(md.md_magnetization(ctx, q))
    assert np.abs(m - np.asarray(oracle.magnetization(host(q)))).max() < 1e-14
    ctx.close()


@pytest.mark.parametrize("n", [1, 65, 257, 1000, 2049, 4096, 4097, 8191])
def test_derivatives(n):
    q, p = inputs.hmf_waterbag(n, seed=n)
    rng = np.random.default_rng(n)
    lq, lp = rng.normal(size=(1, n)), rng.normal(size=(1, n))
    ctx = md.md_init(md.HMF, md.FP64, n)
    hw = host(md.md_hvp(ctx, dev(q), dev(lq)))
    assert np.abs(hw - oracle.hvp(md.HMF, q, lq, 0.0)).max() < 1e-11
    for steps in (1, 4):
        want = oracle.step_vjp(md.HMF, q, p, 0.1, steps, lq, lp, 0.0)
        a, b = dev(lq), dev(lp)
        md.md_step_vjp(ctx, dev(q), dev(p), 0.1, steps, a, b)
        assert max(np.abs(host(x) - y).max() for x, y in zip((a, b), want)) < 1e-10
        qr, pr, f = dev(q), dev(p), torch.empty_like(a)
        md.md_force(ctx, qr, f)
        stage = md.md_step_record(ctx, qr, pr, f, 0.1, steps)
        c, d = dev(lq), dev(lp)
        md.md_step_vjp_recorded(ctx, dev(q), 0.1, steps, c, d, stage)
        assert torch.equal(a, c) and torch.equal(b, d)
    ctx.close()


def test_angles_beyond_the_reduction():
    q, p = inputs.hmf_waterbag(1500, seed=3)
    q[0, ::7] += 2.0 ** 31
    q[0, 1499] = -3e15
    fo = oracle.force(md.HMF, q)
    ctx = md.md_init(md.HMF, md.FP64, 1500)
    f = torch.empty_like(dev(q))
    md.md_force(ctx, dev(q), f)
    assert np.abs(host(f) - fo).max() < 1e-13
    ctx.close()


@pytest.mark.parametrize("bad", [np.nan, np.inf])
def test_not_finite(bad):
    q, p = inputs.hmf_waterbag(1500, seed=3)
    q[0, 1234] = bad
    ctx = md.md_init(md.HMF, md.FP64, 1500)
    for call in (lambda: md.md_magnetization(ctx, dev(q)), lambda: md.md_energy(ctx, dev(q), dev(p))):
        with pytest.raises(md.MDError):
            call()
    ctx.close()


def test_many_steps_and_graph():
    """More steps than one launch takes, and replays of a captured call."""
    q, p = (dev(x) for x in inputs.hmf_waterbag(100, seed=9))
    ctx = md.md_init(md.HMF, md.FP64, 100)
    f = torch.empty_like(q)
    md.md_force(ctx, q, f)
    a = [x.clone() for x in (q, p, f)]
    md.md_step(ctx, *a, 0.01, 4099)
    b = [x.clone() for x in (q, p, f)]
    md.md_step(ctx, *b, 0.01, 4096)
    md.md_step(ctx, *b, 0.01, 3)
    assert all(torch.equal(x, y) for x, y in zip(a, b))
    s = torch.cuda.Stream()
    md.md_set_stream(ctx, s)
    s.wait_stream(torch.cuda.current_stream())
    c = [x.clone() for x in (q, p, f)]
    g = torch.cuda.CUDAGraph()
    with torch.cuda.stream(s):
        with torch.cuda.graph(g, stream=s):
            md.md_step(ctx, *c, 0.01, 50)
    want = [x.clone() for x in (q, p, f)]
    torch.cuda.synchronize()
    md.md_set_stream(ctx, torch.cuda.current_stream())
    for _ in range(3):
        g.replay()
        torch.cuda.synchronize()
        md.md_step(ctx, *want, 0.01, 50)
        torch.cuda.synchronize()
        assert all(torch.equal(x, y) for x, y in zip(c, want))
    ctx.close()


def test_many_steps_recorded_and_swept():
    """More steps than one launch takes: the recording, the recomputation and the sweep, each against
    two halves of the run, bit for bit."""
    n, dt, head, tail = 100, 0.01, 4097, 4098
    q0, p0 = (dev(x) for x in inputs.hmf_waterbag(n, seed=9))
    ctx = md.md_init(md.HMF, md.FP64, n)
    lq, lp = (torch.randn(1, n, dtype=torch.float64, device=q0.device) for _ in range(2))
    whole = [q0.clone(), p0.clone(), md.md_force(ctx, q0, torch.empty_like(q0))]
    halves = [x.clone() for x in whole]
    stage = md.md_step_record(ctx, *whole, dt, head + tail)
    first = md.md_step_record(ctx, *halves, dt, head)
    mid = [x.clone() for x in halves]
    second = md.md_step_record(ctx, *halves, dt, tail)
    assert all(torch.equal(x, y) for x, y in zip(whole, halves))
    assert torch.equal(stage, torch.cat([first, second]))
    a, b, c, d, e, f = (x.clone() for x in (lq, lp) * 3)
    md.md_step_vjp_recorded(ctx, q0, dt, head + tail, a, b, stage)
    md.md_step_vjp_recorded(ctx, mid[0], dt, tail, c, d, second)
    md.md_step_vjp_recorded(ctx, q0, dt, head, c, d, first)
    md.md_step_vjp(ctx, q0, p0, dt, head + tail, e, f)
    assert torch.equal(a, e) and torch.equal(b, f)
    # the halves' sweeps apply the joint's two kicks from two equal products, the whole run's
    # from one: the same sums, the same bits
    assert torch.equal(a, c) and torch.equal(b, d)
    ctx.close()


@pytest.mark.parametrize("steps,launches", [(4096, 1), (4097, 2), (8193, 3)])
def test_a_launch_takes_a_bounded_number_of_steps(steps, launches):
    """The kernels of md_step and md_step_vjp_recorded, counted in a captured graph."""
    n = 64
    ctx = md.md_init(md.HMF, md.FP64, n)
    q, p = (dev(x) for x in inputs.hmf_waterbag(n, seed=9))
    f = md.md_force(ctx, q, torch.empty_like(q))
    stage = torch.zeros(md.md_record_stage_bytes(ctx, steps), dtype=torch.uint8, device=q.device)
    lq, lp = torch.zeros_like(q), torch.zeros_like(q)
    s = torch.cuda.Stream()
    md.md_set_stream(ctx, s)
    s.wait_stream(torch.cuda.current_stream())
    for call in (lambda: md.md_step(ctx, q, p, f, 1e-3, steps),
                 lambda: md.md_step_vjp_recorded(ctx, q, 1e-3, steps, lq, lp, stage)):
        g = torch.cuda.CUDAGraph(keep_graph=True)
        with torch.cuda.graph(g, stream=s):
            call()
        nodes = ctypes.c_size_t(0)
        assert md.load().hipGraphGetNodes(ctypes.c_void_p(g.raw_cuda_graph()), None, ctypes.byref(nodes)) == 0
        assert nodes.value == launches
    torch.cuda.synchronize()
    ctx.close()


@pytest.mark.parametrize("prec", [md.FP64, md.MIXED_F32STATE])
@pytest.mark.parametrize("n,kernel,launches", [(4096, "k_hmf_small_step", 1), (4097, "k_hmf_pass", 10),
                                               (8192, "k_hmf_pass", 10)])
def test_steps_leave_the_one_workgroup_where_it_is_slower(n, kernel, launches, prec):
    """Above 4096 particles the passes are ahead (12.0 against 12.3 us a step at 4097, 9.7 against 12.5
    at 8192)."""
    ctx = md.md_init(md.HMF, prec, n)
    q, p = (dev(x) for x in inputs.hmf_waterbag(n, seed=n))
    f = md.md_force(ctx, q, torch.empty_like(q))
    md.md_timing_begin(ctx, 16)
    md.md_step(ctx, q, p, f, 0.1, 3)
    _, count, name = md.md_timing_end(ctx)
    assert (name, count) == (kernel, launches)
    ctx.close()


@pytest.mark.parametrize("n", [4097, 6144, 6145, 8192, 8193])
def test_energies_and_products_between_the_limits(n):
    """Energies (one workgroup up to 8192) and products (up to 6144) beside steps by passes."""
    q, p = inputs.hmf_waterbag(n, seed=n)
    w = np.random.default_rng(n).normal(size=(1, n))
    ctx = md.md_init(md.HMF, md.FP64, n)
    e, eo = host(md.md_energy(ctx, dev(q), dev(p))), np.asarray(oracle.energy(md.HMF, q, p, 0.0))
    assert np.abs(e - eo).max() < 1e-12 * (abs(eo[0]) + abs(eo[1]) + n / 2)
    assert np.abs(host(md.md_hvp(ctx, dev(q), dev(w))) - oracle.hvp(md.HMF, q, w, 0.0)).max() < 1e-11
    ctx.close()

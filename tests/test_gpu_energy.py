"""Energies (md_energy) against their definitions at the edges of the pair sum's groups, windows
and ranges, for every form of the term.

Tolerance: a pair term (the logarithm of a product of r^2 + eps, or the refined inverse
root of a half-angle form) carries at most about 16 roundings of 2^-53 of max(1, |term|),
and the sums add theirs in blocks: 1e-14 of the sum of max(1, |term|) over the pairs / n
plus the kinetic energy, against extended-precision sums of the definitions.
"""
import math

import numpy as np
import pytest
import torch

from gpu_helpers import dev, host
from paper_1212_0262_amd import inputs, md

pytestmark = pytest.mark.gpu


def reference(model, q, p, eps):
    """(K, V, K + V) in extended precision from the definitions (eqs. 1 and 3, the Ring's
    1 - cos d as 2 sin^2(d/2): formed as written it loses 2^-53 / eps to cancellation,
    more than the tolerance below eps = 1e-2), and the tolerance's scale."""
    n = q.shape[-1]
    wide = np.longdouble if n < 6000 else np.float64  # rows added by math.fsum
    q, p, eps = q.astype(wide), p.astype(wide), wide(eps)
    rows, size = [], 0.0
    for i in range(n - 1):
        if model == md.GRAV2D:
            t = np.log((q[0, i] - q[0, i + 1:]) ** 2 + (q[1, i] - q[1, i + 1:]) ** 2 + eps)
        else:
            t = 1 / np.sqrt(2 * np.sin((q[0, i] - q[0, i + 1:]) / 2) ** 2 + eps)
        rows.append(t.sum())
        size += float(np.maximum(1, np.abs(t)).sum())
    total = wide(math.fsum(rows)) if rows else wide(0)
    v = total / n if model == md.GRAV2D else -total / (np.sqrt(wide(2)) * n)
    k = (p * p).sum() / 2
    return np.array([k, v, k + v]), float(k) + size / n


def check(model, q, p, eps, got):
    want, scale = reference(model, q, p, eps)
    err = float(np.abs(got - want).max()) / scale
    print(f"n={q.shape[-1]} eps={eps}: err {err:.2e}", flush=True)
    assert err < 1e-14, err


def energy(model, prec, q, p, eps):
    ctx = md.md_init(model, prec, q.shape[-1], eps)
    out = host(md.md_energy(ctx, dev(q), dev(p)))
    ctx.close()
    return out


# groups of 64 i (of 256 above n = 32768, below); windows of 64 j, ranges of 256 and up
@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 255, 256, 257, 321, 5003, 16384, 16385])
@pytest.mark.parametrize("model,eps", [(md.GRAV2D, 1e-3), (md.RING, 1e-2), (md.RING, 1e-5)])
def test_energy_sizes(n, model, eps):
    q, p = inputs.uniform_state(model, n, seed=n)
    check(model, q, p, eps, energy(model, md.FP64, q, p, eps))


@pytest.mark.parametrize("model,eps", [(md.GRAV2D, 1e-3), (md.RING, 1e-2), (md.RING, 1e-5)])
def test_energy_wide_groups(model, eps):
    n = 32_769
    q, p = inputs.uniform_state(model, n, seed=n)
    check(model, q, p, eps, energy(model, md.FP64, q, p, eps))


# both sides of the Ring's half-angle range; repeated and unwrapped angles
@pytest.mark.parametrize("eps", [1e-12, 9.9e-5, 1e-4, 1.0, 1e101])
def test_ring_energy_forms(eps):
    q, p = inputs.uniform_state(md.RING, 700, seed=5, qscale=40.0)
    q[0, 100:110] = q[0, 0]
    check(md.RING, q, p, eps, energy(md.RING, md.FP64, q, p, eps))


# 2D: the ends of the softening's range, and particles past the range of the product of
# four r^2 + eps, among the i, the j and both
@pytest.mark.parametrize("eps", [1e-75, 1e-3, 1e75])
@pytest.mark.parametrize("far", [[], [3], [650], [3, 299, 650]])
def test_grav2d_energy_range(eps, far):
    q, p = inputs.uniform_state(md.GRAV2D, 700, seed=6)
    q[:, 20] = q[:, 21]
    for k in far:
        q[:, k] = (1e40 * (k + 1), -3e150)
    check(md.GRAV2D, q, p, eps, energy(md.GRAV2D, md.FP64, q, p, eps))


@pytest.mark.parametrize("model", [md.GRAV2D, md.RING])
@pytest.mark.parametrize("bad", [np.inf, np.nan])
def test_energy_not_finite(model, bad):
    q, p = inputs.uniform_state(model, 5000, seed=7)
    q[0, 4321] = bad
    with pytest.raises(md.MDError):
        energy(model, md.FP64, q, p, 1e-2)


@pytest.mark.parametrize("model,eps", [(md.GRAV2D, 1e-3), (md.RING, 1e-2), (md.RING, 1e-5)])
def test_batch_energy_sizes(model, eps):
    sizes = [1, 2, 64, 65, 255, 256, 257, 700, 2048, 2049, 2305]
    parts = [inputs.uniform_state(model, n, seed=n) for n in sizes]
    off = np.concatenate([[0], np.cumsum(sizes)])
    ctx = md.md_batch_init(model, md.FP64, off, eps)
    q = np.concatenate([a for a, _ in parts], axis=1)
    p = np.concatenate([b for _, b in parts], axis=1)
    out = host(md.md_energy(ctx, dev(q), dev(p)))
    ctx.close()
    for (a, b), got in zip(parts, out):
        check(model, a, b, eps, got)
    again = md.md_batch_init(model, md.FP64, off, eps)
    assert torch.equal(md.md_energy(again, dev(q), dev(p)).cpu(), torch.from_numpy(out))
    again.close()


@pytest.mark.parametrize("eps", [1e-12, 1e-6, 1e-4, 1e-2, 1.0])
def test_ring_pair_energy_is_relative(eps):
    """One pair of every separation, 1e-7 to pi: V to 8 roundings of 2^-53 relative, however close
    the pair and small eps (a chord off by 2^-53 absolutely is 1e-14 out at eps = 1e-4).  The
    roundings: ti - tj 1, the chord 2, the root 2 with its operand, the sums' scale and the
    prefactor 2.5."""
    nb = 2000
    rng = np.random.default_rng(3)
    q = np.empty((1, 2 * nb))
    q[0, ::2] = rng.uniform(-np.pi / 2, np.pi / 2, nb)
    q[0, 1::2] = q[0, ::2] + 10 ** rng.uniform(-7, 0, nb) * np.sign(-q[0, ::2])
    q[0, 1::40] = -q[0, ::40] * rng.uniform(0, 1, nb // 20)
    wide = q.astype(np.longdouble)
    h = np.sin((wide[0, ::2] - wide[0, 1::2]) / 2)
    want = -1 / (np.sqrt(2 * h * h + np.longdouble(eps)) * np.sqrt(np.longdouble(2)) * 2)
    ctx = md.md_batch_init(md.RING, md.FP64, 2 * np.arange(nb + 1), eps)
    got = host(md.md_energy(ctx, dev(q), dev(np.zeros_like(q))))[:, 1]
    ctx.close()
    err = float(np.abs(got / want - 1).max())
    k = int(np.abs(got / want - 1).argmax())
    print(f"eps={eps}: err {err:.2e}", flush=True)
    assert err < 8 * 2.0 ** -53, err
    one = energy(md.RING, md.MIXED, q[:, 2 * k:2 * k + 2], np.zeros((1, 2)), eps)
    assert one[1] == got[k]


@pytest.mark.parametrize("angle", [2.0 ** 29 - 1, 2.0 ** 29 + 1, 2.0 ** 32])
def test_ring_energy_past_the_reduction(angle):
    """Angles on both sides of the range of the chord's reduction, among the i, the j and both
    (multiples of 2^-20: every difference is exact)."""
    q, p = inputs.uniform_state(md.RING, 700, seed=8)
    q = np.round(q * 2.0 ** 20) / 2.0 ** 20
    q[0, [3, 299, 650]] = (angle, -angle, angle)
    check(md.RING, q, p, 1e-2, energy(md.RING, md.FP64, q, p, 1e-2))

// energy_terms.h -- a wavefront's share of the potential's pair sum (eqs. 1 and 3,
// i < j), shared by the single-system (energy.hip) and ensemble (batch.hip) kernels.
//
// Always FP64.  Bound by FP64 issue: the library's log, or its sin, sqrt and divide,
// cost 250 to 1100 cycles a pair and wavefront, so neither is called per pair.
//   2D: sum of log s = log of the product of s.  Four s (j, j+1, j+2, j+3) are
//     multiplied, the product's exponent is added to an integer and its mantissa
//     multiplied into a running one; one log per lane and i at the end.  5.6 FP64
//     instructions a pair.  Each product is off by about sqrt(terms) 2^-53 relative,
//     less than the rounding of a running sum of logs.
//   Ring: 2 sin(d/2) of the rounded difference d = ti - tj by one reduction modulo 2 pi
//     and a polynomial (ring_chord), and the refined hardware inverse square root: 22
//     FP64 instructions and the seed.  As the library's sine of d/2, the chord's error is
//     relative however close the pair (a difference of products of each particle's sines and
//     cosines, 9 instructions, is off by 2^-53 absolutely: 1e-14 of 1/sqrt(2 sin^2 + eps)
//     at eps = 1e-4).
// Measured (MI355X), md_energy before and after: 2D N = 262,144 97.6 -> 5.9 ms (27
// cycles a pair and wavefront; the seven FP64-rate instructions' cost); Ring N = 16,384
// 0.91 -> 0.12 ms, 65,536 12.4 -> 1.71 (125 cycles, of 115 for its instructions).
#pragma once

#include <type_traits>

#include "device.h"

namespace md {

// The 2D product takes four s <= 8 kEnergyMaxPos^2 + eps and >= eps at a time: with
// |x|, |y| <= 1e37 and eps in [1e-75, 1e75] (the widest range md_init takes) it stays
// in [1e-300, 1e302].  Windows with a particle further out, or not finite, take the
// log of every pair instead.
constexpr double kEnergyMaxPos = 1e37;

// The Ring's chord: |ti|, |tj| up to 2^29 (the reduction's range) and eps up to 1e100 (the
// square root's operand within range).  Windows with a larger angle, or one that is not
// finite, and larger eps take the library's sine, root and divide for every pair.
constexpr double kEnergyMaxAngle = 536870912.0, kEnergyMaxEps = 1e100;

// 2 sin(d/2) for |d| <= 2^30, of either sign (it is squared).  d = 2 pi k + r with k = rint(d /
// 2 pi) and 2 pi in two parts: for k = 0 r is d, for k = +-1 the first step is exact.  Then r (1 +
// z S(z)), z = r^2 <= pi^2: S interpolates (2 sin(r/2)/r - 1)/z at the eight Chebyshev points
// of [0, pi^2]; with its coefficients rounded it is off by 3.6e-17 relative at most.
__device__ __forceinline__ double ring_chord(double d)
{
    const double k = __builtin_rint(d * 0.15915494309189535);
    double r = __builtin_fma(-k, 6.283185307179586, d);
    r = __builtin_fma(-k, 2.4492935982947064e-16, r);
    const double z = r * r;
    double s = 4.167853941492218e-20;
    s = __builtin_fma(s, z, -4.665509213968379e-17);
    s = __builtin_fma(s, z, 3.920648757920964e-14);
    s = __builtin_fma(s, z, -2.4464948844722537e-11);
    s = __builtin_fma(s, z, 1.0764577819985637e-08);
    s = __builtin_fma(s, z, -3.1001984126960897e-06);
    s = __builtin_fma(s, z, 0.0005208333333333322);
    s = __builtin_fma(s, z, -0.041666666666666664);
    return __builtin_fma(r * z, s, r);
}

// j of a wavefront's window, one per lane: the positions' rows (2D), the angles (Ring).
template <int MODEL>
struct EnergyWin {
    double r[MODEL == MD_GRAV2D ? 2 : 1][kWave];
};

// The operands of particle i: the position (2D) or the angle (Ring; b is not used).
template <int MODEL>
__device__ __forceinline__ void energy_operands(const double *__restrict__ q, size_t row, int i, double &a, double &b)
{
    a = q[i];
    b = MODEL == MD_GRAV2D ? q[row + i] : 0.0;
}

// Outside the ranges above.
template <int MODEL>
__device__ __forceinline__ bool energy_far(double a, double b)
{
    if (MODEL == MD_GRAV2D) return !(fabs(a) <= kEnergyMaxPos && fabs(b) <= kEnergyMaxPos);
    return !(fabs(a) <= kEnergyMaxAngle);
}

// Sum over the pairs i < j of i in [i0, min(i0 + 64 IPL, i1)), j in [j0, j1) of
// log(|r_i - r_j|^2 + eps) (2D) or 1/sqrt(2 sin^2((ti - tj)/2) + eps) (Ring), each
// lane's part, by one wavefront; win: its own LDS window.  row: stride between the
// rows of q.  i0, i1, j0, j1 uniform over the wavefront, all indices below the array's
// end.  The 64 j of a window go out with one coalesced load per lane and are
// read broadcast from LDS; windows that meet the diagonal or the end of the j
// range mask their pairs.
template <int MODEL, int IPL>
__device__ __forceinline__ double energy_wave(const double *__restrict__ q, size_t row, int i0, int i1, int j0, int j1,
                                              double eps, EnergyWin<MODEL> &win)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int ilast = min(i0 + kWave * IPL, i1) - 1;
    j0 = max(j0, i0 + 1);  // no j <= i0 has a partner here
    if (j0 >= j1) return 0.0;
    double a[IPL], b[IPL], m[IPL], acc = 0.0, chords = 0.0;  // chords: of 1/sqrt(2 (..)) (Ring)
    int ii[IPL], ex[IPL];
    bool far = MODEL == MD_RING && !(eps <= kEnergyMaxEps);
#pragma unroll
    for (int k = 0; k < IPL; ++k) {
        ii[k] = i0 + k * kWave + lane;
        energy_operands<MODEL>(q, row, min(ii[k], ilast), a[k], b[k]);
        far |= energy_far<MODEL>(a[k], b[k]);
        if (ii[k] > ilast) ii[k] = 0x7fffffff;  // beyond the last i: no j is above it
        m[k] = 1.0;
        ex[k] = 0;
    }
    double na, nb;
    energy_operands<MODEL>(q, row, min(j0 + lane, j1 - 1), na, nb);
    for (int jw = j0; jw < j1; jw += kWave) {
        const bool slow = __any(far || energy_far<MODEL>(na, nb));
        wave_sync();  // the previous window's reads are done
        win.r[0][lane] = na;
        if constexpr (MODEL == MD_GRAV2D) win.r[1][lane] = nb;
        wave_sync();
        if (jw + kWave < j1) energy_operands<MODEL>(q, row, min(jw + kWave + lane, j1 - 1), na, nb);
        const bool masked = jw <= i0 + kWave * IPL - 1 || jw + kWave > j1 || ilast < i0 + kWave * IPL - 1;
        auto counted = [&](int k, int u) { return jw + u > ii[k] && jw + u < j1; };
        // s of i = k, j = u of the window (2D); 1 for a pair that is not counted
        auto square = [&](int k, int u, auto mask) {
            const double dx = a[k] - win.r[0][u], dy = b[k] - win.r[MODEL == MD_GRAV2D][u];
            const double s = __builtin_fma(dx, dx, __builtin_fma(dy, dy, eps));
            return !decltype(mask)::value || counted(k, u) ? s : 1.0;
        };
        auto window = [&](auto mask) {
            if constexpr (MODEL == MD_GRAV2D) {
                if (decltype(mask)::value && slow) {
                    for (int u = 0; u < kWave; ++u)
#pragma unroll
                        for (int k = 0; k < IPL; ++k) acc += log(square(k, u, mask));
                    return;
                }
#pragma unroll (IPL == 1 ? 4 : 1)
                for (int u = 0; u < kWave; u += 4) {
#pragma unroll
                    for (int k = 0; k < IPL; ++k) {
                        const double p = (square(k, u, mask) * square(k, u + 1, mask)) *
                                         (square(k, u + 2, mask) * square(k, u + 3, mask));
                        m[k] *= __builtin_amdgcn_frexp_mant(p);
                        ex[k] += __builtin_amdgcn_frexp_exp(p);
                    }
                }
#pragma unroll
                for (int k = 0; k < IPL; ++k) {  // 16 mantissas in [1/2, 1): back to [1/2, 1)
                    ex[k] += __builtin_amdgcn_frexp_exp(m[k]);
                    m[k] = __builtin_amdgcn_frexp_mant(m[k]);
                }
            } else {
                double direct = 0.0, chord = 0.0;
                if (decltype(mask)::value && slow) {
                    for (int u = 0; u < kWave; ++u)
#pragma unroll
                        for (int k = 0; k < IPL; ++k) {
                            const double h = sin(0.5 * (a[k] - win.r[0][u]));
                            const double t = 1.0 / sqrt(2.0 * h * h + eps);
                            direct += counted(k, u) ? t : 0.0;
                        }
                } else {
#pragma unroll (IPL == 1 ? 4 : 1)
                    for (int u = 0; u < kWave; ++u) {
#pragma unroll
                        for (int k = 0; k < IPL; ++k) {
                            const double g = ring_chord(a[k] - win.r[0][u]);
                            const double t = rsq64(__builtin_fma(g, g, 2.0 * eps));
                            chord += !decltype(mask)::value || counted(k, u) ? t : 0.0;
                        }
                    }
                }
                acc += direct;
                chords += chord;
            }
        };
        if (masked || slow) window(std::true_type{});
        else window(std::false_type{});
    }
    if constexpr (MODEL == MD_GRAV2D) {
        int et = 0;
#pragma unroll
        for (int k = 0; k < IPL; ++k) {
            acc += log(m[k]);
            et += ex[k];
        }
        return __builtin_fma((double)et, 0.6931471805599453, acc);
    } else {
        return __builtin_fma(1.4142135623730951, chords, acc);
    }
}

// The block's four wavefronts take the four quarters of [j0, j1) (whole windows).
template <int MODEL, int IPL>
__device__ __forceinline__ double energy_block(const double *__restrict__ q, size_t row, int i0, int i1, int j0,
                                               int j1, double eps, EnergyWin<MODEL> (&win)[4])
{
    const int wave = threadIdx.x / kWave;
    const int len = ((j1 - j0 + 4 * kWave - 1) / (4 * kWave)) * kWave;
    const int ja = min(j1, j0 + wave * len), jb = min(j1, ja + len);
    return energy_wave<MODEL, IPL>(q, row, i0, i1, ja, jb, eps, win[wave]);
}

}  // namespace md

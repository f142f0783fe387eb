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
//   Ring: sin((ti - tj)/2) from each particle's half-angle sine and cosine (as the
//     FP32 force form, here in FP64) and the refined hardware inverse square root:
//     9 FP64 instructions and the seed.
// Measured (MI355X), md_energy before and after: 2D N = 262,144 97.6 -> 5.9 ms (27
// cycles a pair and wavefront; the seven FP64-rate instructions' cost); Ring N = 16,384
// 0.94 -> 0.10 ms.
#pragma once

#include <type_traits>

#include "device.h"

namespace md {

// The 2D product takes four s <= 8 kEnergyMaxPos^2 + eps and >= eps at a time: with
// |x|, |y| <= 1e37 and eps in [1e-75, 1e75] (the widest range md_init takes) it stays
// in [1e-300, 1e302].  Windows with a particle further out, or not finite, take the
// log of every pair instead.
constexpr double kEnergyMaxPos = 1e37;

// The Ring's half-angle form is off by about 2^-53 in sin((ti - tj)/2), absolutely
// (the operands' rounding), so a pair's 1/sqrt(2 sin^2 + eps) by up to 2^-54 / sqrt(eps)
// relative: at eps >= 1e-4 that is 1e-14 for the closest pairs and averages out
// (measured against 64-bit sums: no larger than the direct form's).  Smaller eps take
// the sine of the rounded difference itself, whose error is relative.
constexpr double kEnergyHalfMinEps = 1e-4, kEnergyHalfMaxEps = 1e100;

// j of a wavefront's window, one per lane.
template <int MODEL>
struct EnergyWin {
    double r0[kWave], r1[kWave];
};

// The operands of particle i: the position (2D), sqrt2 (sin, cos)(t/2) (Ring, half
// angles) or the angle (Ring, direct).
template <int MODEL, bool HALF>
__device__ __forceinline__ void energy_operands(const double *__restrict__ q, size_t row, int i, double &a, double &b)
{
    if constexpr (MODEL == MD_GRAV2D) {
        a = q[i];
        b = q[row + i];
    } else if constexpr (HALF) {
        double s, c;
        sincos64(0.5 * q[i], &s, &c);
        a = 1.4142135623730951 * s;
        b = 1.4142135623730951 * c;
    } else {
        a = q[i];
        b = 0.0;
    }
}

// Sum over the pairs i < j of i in [i0, min(i0 + 64 IPL, i1)), j in [j0, j1) of
// log(|r_i - r_j|^2 + eps) (2D) or 1/sqrt(2 sin^2((ti - tj)/2) + eps) (Ring), each
// lane's part, by one wavefront; win: its own LDS window.  row: stride between the
// rows of q.  i0, i1, j0, j1 uniform over the wavefront, all indices below the array's
// end.  The 64 j of a window go out with one coalesced load (and one sincos) per lane
// and are read broadcast from LDS; windows that meet the diagonal or the end of the j
// range mask their pairs.
template <int MODEL, int IPL, bool HALF>
__device__ __forceinline__ double energy_wave(const double *__restrict__ q, size_t row, int i0, int i1, int j0, int j1,
                                              double eps, EnergyWin<MODEL> &win)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int ilast = min(i0 + kWave * IPL, i1) - 1;
    j0 = max(j0, i0 + 1);  // no j <= i0 has a partner here
    if (j0 >= j1) return 0.0;
    double a[IPL], b[IPL], m[IPL], acc = 0.0;
    int ii[IPL], ex[IPL];
    bool far = false;  // 2D: a particle outside the product's range
#pragma unroll
    for (int k = 0; k < IPL; ++k) {
        ii[k] = i0 + k * kWave + lane;
        energy_operands<MODEL, HALF>(q, row, min(ii[k], ilast), a[k], b[k]);
        if (MODEL == MD_GRAV2D) far |= !(fabs(a[k]) <= kEnergyMaxPos && fabs(b[k]) <= kEnergyMaxPos);
        if (ii[k] > ilast) ii[k] = 0x7fffffff;  // beyond the last i: no j is above it
        m[k] = 1.0;
        ex[k] = 0;
    }
    const double e = MODEL == MD_RING && HALF ? 2.0 * eps : eps;
    double na, nb;
    energy_operands<MODEL, HALF>(q, row, min(j0 + lane, j1 - 1), na, nb);
    for (int jw = j0; jw < j1; jw += kWave) {
        const bool slow =
            MODEL == MD_GRAV2D && __any(far || !(fabs(na) <= kEnergyMaxPos && fabs(nb) <= kEnergyMaxPos));
        wave_sync();  // the previous window's reads are done
        win.r0[lane] = na;
        win.r1[lane] = nb;
        wave_sync();
        if (jw + kWave < j1) energy_operands<MODEL, HALF>(q, row, min(jw + kWave + lane, j1 - 1), na, nb);
        const bool masked = jw <= i0 + kWave * IPL - 1 || jw + kWave > j1 || ilast < i0 + kWave * IPL - 1;
        // s of i = k, j = u of the window; 1 for a pair that is not counted
        auto term = [&](int k, int u, auto mask) {
            if constexpr (MODEL == MD_GRAV2D) {
                const double dx = a[k] - win.r0[u], dy = b[k] - win.r1[u];
                const double s = __builtin_fma(dx, dx, __builtin_fma(dy, dy, e));
                return !decltype(mask)::value || (jw + u > ii[k] && jw + u < j1) ? s : 1.0;
            } else {
                double t;
                if constexpr (HALF) {
                    const double d = __builtin_fma(a[k], win.r1[u], -(b[k] * win.r0[u]));
                    t = rsq64(__builtin_fma(d, d, e));
                } else {
                    const double h = sin(0.5 * (a[k] - win.r0[u]));
                    t = 1.0 / sqrt(2.0 * h * h + e);
                }
                return !decltype(mask)::value || (jw + u > ii[k] && jw + u < j1) ? t : 0.0;
            }
        };
        auto window = [&](auto mask) {
            if constexpr (MODEL == MD_GRAV2D) {
                if (slow) {
                    for (int u = 0; u < kWave; ++u)
#pragma unroll
                        for (int k = 0; k < IPL; ++k) acc += log(term(k, u, mask));
                    return;
                }
#pragma unroll (IPL == 1 ? 4 : 1)
                for (int u = 0; u < kWave; u += 4) {
#pragma unroll
                    for (int k = 0; k < IPL; ++k) {
                        const double p = (term(k, u, mask) * term(k, u + 1, mask)) *
                                         (term(k, u + 2, mask) * term(k, u + 3, mask));
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
                double part = 0.0;
#pragma unroll (IPL == 1 ? 4 : 1)
                for (int u = 0; u < kWave; ++u)
#pragma unroll
                    for (int k = 0; k < IPL; ++k) part += term(k, u, mask);
                acc += part;
            }
        };
        if (masked) window(std::true_type{});
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
        return HALF ? 1.4142135623730951 * acc : acc;
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
    if (MODEL == MD_RING && !(eps >= kEnergyHalfMinEps && eps <= kEnergyHalfMaxEps))
        return energy_wave<MODEL, IPL, false>(q, row, i0, i1, ja, jb, eps, win[wave]);
    return energy_wave<MODEL, IPL, true>(q, row, i0, i1, ja, jb, eps, win[wave]);
}

}  // namespace md

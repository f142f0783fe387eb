// hmf_small.hip -- the HMF model (Sec. 3.1) for systems one workgroup can hold in
// registers: a whole md_step call, or a whole reverse sweep, in one launch.
//
// The magnetization joins every particle at each stage.  Across blocks that takes a
// kernel boundary a stage (hmf.hip), 3 to 4 us however few the particles: the
// launch, a memory round trip for (t, p), the sums' way through memory.  Here one block
// of up to 512 threads keeps t, p and the sincos of t of P particles a thread in
// registers for all stages of the call, so a stage is one sincos per particle (the
// kick reuses the sincos the previous stage summed), a register reduction and one
// barrier.  Bound by FP64 issue on one CU (36 instructions of sincos a particle) above
// about 1000 particles and by the chain sincos - reduction - barrier below.
// Measured (MI355X), us per step by hmf.hip's passes and so, FP64 / FP32 state: n = 100 11.8 /
// 8.7 and 1.6 / 1.6; 2001 11.9 / 9.1 and 3.8 / 4.2; 4096 12.0 / 9.1 and 6.0 / 4.9.  Four steps'
// md_step_vjp at n = 2001: 112 and 46 us.  (The limits are in md_internal.h.)
//
// Sums: each thread's particles t, t + threads, ... in order, then small_means.  md_force,
// md_magnetization, md_energy and the reverse sweep of these systems take the same sums, so
// they agree bit for bit.
#include "device.h"
#include "hmf_terms.h"
#include "md_internal.h"

namespace md {
namespace {

// Most threads of a block whose threads hold P particles: their t, p, sin and cos take 8 P
// registers, of 256 a thread in blocks of 512 and 512 in blocks of 256 (16 in blocks of
// 512 and 11 in blocks of 768 spill to memory).
constexpr int small_threads(int P) { return P > 8 ? 256 : 512; }
constexpr int kSmallWaves = 16;  // the wavefronts' sums: one row of lanes
static_assert(small_threads(1) <= kSmallWaves * kWave, "a lane per wavefront");

// The totals of K = 2 or 4 values over the block of B threads, divided by n, in every thread.  The
// first lane exchanges put the K values in different rows of lanes, so that one chain
// of moves and adds serves them all; the wavefronts' sums meet in lds (this stage's
// buffer: two alternate, as a wavefront may be a stage ahead), one row of lanes per
// value.  Every wavefront does this, so a block takes as few of them as fill its SIMDs.
template <int K>
__device__ __forceinline__ void small_means(double (&v)[K], double (&lds)[K][kSmallWaves], int B, double n)
{
    static_assert(K == 2 || K == 4, "");
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave, nw = B / kWave;
    double t;
    if constexpr (K == 2) t = wave_sum2(v[0], v[1]);
    else t = wave_sum4(v[0], v[1], v[2], v[3]);
    constexpr int kLanes = kWave / K;  // lanes of each value
    if (lane % kLanes == 0) lds[lane / kLanes][wave] = t;
    __syncthreads();
    const int w = lane & (kSmallWaves - 1);
    t = row_sum(w < nw ? lds[lane / kLanes][w] : 0.0);
    t /= n;
    v[0] = lane_value<0>(t);
    v[1] = lane_value<kLanes>(t);
    if constexpr (K == 4) {
        v[2] = lane_value<2 * kLanes>(t);
        v[3] = lane_value<3 * kLanes>(t);
    }
}

// sum cos, sum sin of the thread's particles below n.
template <typename T, int P>
__device__ __forceinline__ void small_sums(const T (&s)[P], const T (&c)[P], int n, int B, double (&v)[2])
{
    v[0] = v[1] = 0.0;
#pragma unroll
    for (int k = 0; k < P; ++k) {
        if ((int)(threadIdx.x + k * B) < n) {
            v[0] += (double)c[k];
            v[1] += (double)s[k];
        }
    }
}

// The block's threads: a constant where the registers are short.
template <int P>
__device__ __forceinline__ int small_block(int threads)
{
    return P > 8 ? small_threads(P) : threads;
}

// eq. 6
__device__ __forceinline__ double small_force(double s, double c, double mx, double my)
{
    return __builtin_fma(c, my, -(s * mx));
}
__device__ __forceinline__ float small_force(float s, float c, float mx, float my)
{
    return __builtin_fmaf(c, my, -(s * mx));
}

// Kicks b0, b1 and drifts d0, d1 (eq. 4) times dt.
struct StepCoef {
    double b0, b1, d0, d1;
};

// nsteps >= 1 Yoshida steps.  snap (nullable): the angles after each drift, stride apart.
// positions_only: nothing past the last of them.
template <typename T, int P>
__global__ __launch_bounds__(small_threads(P)) void k_hmf_small_step(double *__restrict__ q, double *__restrict__ p,
                                                                  double *__restrict__ f, int n, int threads, StepCoef a,
                                                                  int nsteps, double *__restrict__ snap, size_t stride,
                                                                  int positions_only)
{
    const int B = small_block<P>(threads);
    __shared__ double lds[2][2][kSmallWaves];
    const T b0 = (T)a.b0, b1 = (T)a.b1, d0 = (T)a.d0, d1 = (T)a.d1;
    T th[P], pp[P], s[P], c[P];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int i = threadIdx.x + k * B;
        const double qi = i < n ? q[i] : 0.0, pi = i < n ? p[i] : 0.0, fi = i < n ? f[i] : 0.0;
        th[k] = (T)qi;
        if constexpr (sizeof(T) == 4) th[k] = wrap_pi(th[k]);
        pp[k] = (T)pi;
        pp[k] += b0 * (T)fi;
    }
    const int last = 3 * nsteps - 1;
    T dr = d0;
    for (int m = 0, r = 0;; ++m, r = r == 2 ? 0 : r + 1) {
#pragma unroll
        for (int k = 0; k < P; ++k) {
            th[k] += dr * pp[k];
            if constexpr (sizeof(T) == 4) th[k] = wrap_pi(th[k]);
        }
        if (snap) {
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const int i = threadIdx.x + k * B;
                if (i < n) snap[(size_t)m * stride + i] = (double)th[k];
            }
        }
        if (positions_only && m == last) return;
        sincos_n(th, s, c);
        double v[2];
        small_sums(s, c, n, B, v);
        small_means(v, lds[m & 1], B, n);
        const T mx = (T)v[0], my = (T)v[1];
        const T k1 = r == 2 ? b0 : b1;
        T(&fm)[P] = s;  // the force, in the place of the sines
#pragma unroll
        for (int k = 0; k < P; ++k) {
            fm[k] = small_force(s[k], c[k], mx, my);
            pp[k] += k1 * fm[k];
        }
        if (m == last) {
#pragma unroll
            for (int k = 0; k < P; ++k) {
                const int i = threadIdx.x + k * B;
                if (i < n) {
                    q[i] = (double)th[k];
                    p[i] = (double)pp[k];
                    f[i] = (double)fm[k];
                }
            }
            return;
        }
        if (r == 2) {  // the end kick of a step, then the start kick of the next
#pragma unroll
            for (int k = 0; k < P; ++k) pp[k] += b0 * fm[k];
        }
        dr = r == 0 ? d1 : d0;
    }
}

// What one evaluation of the magnetization of q gives (each output nullable): M (the
// context's and out2), the force f, the energies of (q, p), and whether M or the
// energies are finite.
template <int P>
__global__ __launch_bounds__(small_threads(P)) void k_hmf_small_eval(const double *__restrict__ q,
                                                                  const double *__restrict__ p, int n, int threads,
                                                                  double *__restrict__ M, double *__restrict__ out2,
                                                                  double *__restrict__ f, double *__restrict__ out3,
                                                                  unsigned *__restrict__ flag)
{
    const int B = small_block<P>(threads);
    __shared__ double lds[2][2][kSmallWaves];
    double th[P], pp[P], s[P], c[P], k2[2] = {0.0, 0.0};
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int i = threadIdx.x + k * B;
        th[k] = i < n ? q[i] : 0.0;
        pp[k] = out3 && i < n ? p[i] : 0.0;
        k2[0] += pp[k] * pp[k];
    }
    sincos_n(th, s, c);
    double v[2];
    small_sums(s, c, n, B, v);
    small_means(v, lds[0], B, n);
    if (f) {
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const int i = threadIdx.x + k * B;
            if (i < n) f[i] = small_force(s[k], c[k], v[0], v[1]);
        }
    }
    if (out3) small_means(k2, lds[1], B, 1.0);
    if (threadIdx.x != 0) return;
    if (M) {
        M[0] = v[0];
        M[1] = v[1];
    }
    bool fine = isfinite(v[0]) && isfinite(v[1]);
    if (out2) {
        out2[0] = v[0];
        out2[1] = v[1];
    }
    if (out3) {
        const double kin = 0.5 * k2[0];
        const double pot = 0.5 * (double)n * (1.0 - v[0] * v[0] - v[1] * v[1]);  // eq. 5
        out3[0] = kin;
        out3[1] = pot;
        out3[2] = kin + pot;
        fine = isfinite(kin) && isfinite(pot) && isfinite(kin + pot);
    }
    if (flag) *flag = fine ? 0u : 1u;
}

// The four means (Mx, My, Cw, Sw) of the product H(t) w (hmf.hip).
template <int P>
__device__ __forceinline__ void small_hvp_means(const double (&s)[P], const double (&c)[P], const double (&w)[P],
                                                int n, int B, double (&lds)[4][kSmallWaves], double (&v)[4])
{
#pragma unroll
    for (int k = 0; k < 4; ++k) v[k] = 0.0;
#pragma unroll
    for (int k = 0; k < P; ++k) {
        if ((int)(threadIdx.x + k * B) < n) {
            v[0] += c[k];
            v[1] += s[k];
            v[2] += c[k] * w[k];
            v[3] += s[k] * w[k];
        }
    }
    small_means(v, lds, B, n);
}

__device__ __forceinline__ double small_hw(double s, double c, double w, const double (&v)[4])
{
    return w * (c * v[0] + s * v[1]) - (c * v[2] + s * v[3]);
}

// out = H(q) w.
template <int P>
__global__ __launch_bounds__(small_threads(P)) void k_hmf_small_hvp(const double *__restrict__ q,
                                                                 const double *__restrict__ w, int n, int threads,
                                                                 double *__restrict__ out)
{
    const int B = small_block<P>(threads);
    __shared__ double lds[4][kSmallWaves];
    double th[P], wk[P], s[P], c[P], v[4];
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int i = threadIdx.x + k * B;
        th[k] = i < n ? q[i] : 0.0;
        wk[k] = i < n ? w[i] : 0.0;
    }
    sincos_n(th, s, c);
    small_hvp_means(s, c, wk, n, B, lds, v);
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int i = threadIdx.x + k * B;
        if (i < n) out[i] = small_hw(s[k], c[k], wk[k], v);
    }
}

// The reverse sweep over nsteps recorded steps (reverse_hmf in api.hip): products at
// P_3n, .., P_1, then at q0 (the position before the first drift), each followed by its
// kick(s) and, but for the last, the drift before it.  pos: P_1 .. P_3n, stride apart.
// A run of many steps is cut into several sweeps, the last steps' first: last says whether
// P_3n ends the run (else the kick of the step after it comes too); with q0 null the run
// starts earlier and the product there is the next sweep's first.
template <int P>
__global__ __launch_bounds__(small_threads(P)) void k_hmf_small_vjp(const double *__restrict__ q0,
                                                                 const double *__restrict__ pos, size_t stride, int n,
                                                                 int threads, StepCoef a, int nsteps, int last,
                                                                 double *__restrict__ lq, double *__restrict__ lp)
{
    const int B = small_block<P>(threads);
    __shared__ double lds[2][4][kSmallWaves];
    double x[P], w[P], th[P], s[P], c[P], v[4];
    const int top = 3 * nsteps, bottom = q0 ? 0 : 1;
    auto load = [&](int m) {  // positions m (0 = q0), for the next product
        const double *__restrict__ src = m > 0 ? pos + (size_t)(m - 1) * stride : q0;
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const int i = threadIdx.x + k * B;
            th[k] = i < n ? src[i] : 0.0;
        }
    };
    load(top);
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int i = threadIdx.x + k * B;
        x[k] = i < n ? lq[i] : 0.0;
        w[k] = i < n ? lp[i] : 0.0;
    }
    int r = 0;  // m mod 3
    for (int m = top; m >= bottom; --m, r = r == 0 ? 2 : r - 1) {
        sincos_n(th, s, c);
        if (m > bottom) load(m - 1);  // in flight under the sums
        small_hvp_means(s, c, w, n, B, lds[m & 1], v);
        const double kick = r == 0 ? a.b0 : a.b1;
        const bool two = r == 0 && m > 0 && (m < top || !last);  // the kicks of two steps at one position
#pragma unroll
        for (int k = 0; k < P; ++k) {
            const double hw = small_hw(s[k], c[k], w[k], v);
            x[k] -= kick * hw;
            if (two) x[k] -= kick * hw;
        }
        if (m > 0) {
            const double dr = r == 2 ? a.d1 : a.d0;  // the drift that led to P_m
#pragma unroll
            for (int k = 0; k < P; ++k) w[k] += dr * x[k];
        }
    }
#pragma unroll
    for (int k = 0; k < P; ++k) {
        const int i = threadIdx.x + k * B;
        if (i < n) {
            lq[i] = x[k];
            lp[i] = w[k];
        }
    }
}

// Particles a thread: four wavefronts, one a SIMD, with 1, 2, 4, then 8 particles each,
// up to eight wavefronts of 8, then four of 32: each wavefront repeats the reduction, so
// fewer, fuller ones are faster while the registers last.  Measured, us per FP64 step:
// n = 1000 2.55 (4 wavefronts of 4 a lane; 16 of 1 4.39, with the reduction of each sum by
// itself); n = 4096 5.81 (8 of 8; 4 of 16 6.62); n = 8192 12.2 (4 of 32, products and energies only).
int small_per_thread(int64_t n)
{
    if (n > 8 * small_threads(8)) return 32;
    int p = 1;
    while (p < 8 && n > (int64_t)4 * kWave * p) p *= 2;
    return p;
}
static_assert(kHmfSmallN <= 8 * small_threads(8), "up to 8 particles a thread in steps and sweeps");
static_assert(kHmfSmallHvpN <= 32 * small_threads(32) && kHmfSmallEnergyN <= 32 * small_threads(32), "a thread each");

// Launches K_(particles a thread), of MOST_ at most.
#define MD_SMALL(MOST_, K_, ...)                                                                       \
    do {                                                                                               \
        const int per = small_per_thread(c->n);                                                        \
        const int64_t waves = (c->n + (int64_t)kWave * per - 1) / ((int64_t)kWave * per);              \
        const int B = per > 8 ? small_threads(per) : (int)(waves * kWave);                             \
        const dim3 block((unsigned)B);                                                                 \
        switch (per) {                                                                                 \
        case 1: hipLaunchKernelGGL((K_(1)), dim3(1), block, 0, c->stream, __VA_ARGS__); break;         \
        case 2: hipLaunchKernelGGL((K_(2)), dim3(1), block, 0, c->stream, __VA_ARGS__); break;         \
        case 4: hipLaunchKernelGGL((K_(4)), dim3(1), block, 0, c->stream, __VA_ARGS__); break;         \
        case 8: hipLaunchKernelGGL((K_(8)), dim3(1), block, 0, c->stream, __VA_ARGS__); break;         \
        default: hipLaunchKernelGGL((K_(MOST_)), dim3(1), block, 0, c->stream, __VA_ARGS__); break;    \
        }                                                                                              \
    } while (0)

}  // namespace

hipError_t launch_hmf_small_steps(md_ctx *c, double b0, double b1, double d0, double d1, int64_t nsteps, double *q,
                                  double *p, double *f, double *snap, size_t snap_stride, bool positions_only)
{
    const StepCoef a{b0, b1, d0, d1};
    const int n = (int)c->n;
    hipError_t err = hipSuccess;
    for (int64_t done = 0; done < nsteps && err == hipSuccess;) {
        const int k = (int)(nsteps - done < kHmfSmallSteps ? nsteps - done : kHmfSmallSteps);
        double *sn = snap ? snap + (size_t)(3 * done) * snap_stride : nullptr;
        const int only = positions_only && done + k == nsteps;
        const int ts = timed_begin(c, "k_hmf_small_step");
#define K64(P_) k_hmf_small_step<double, P_>
#define K32(P_) k_hmf_small_step<float, P_>
        if (c->prec == MD_FP64) MD_SMALL(8, K64, q, p, f, n, B, a, k, sn, snap_stride, only);
        else MD_SMALL(8, K32, q, p, f, n, B, a, k, sn, snap_stride, only);
#undef K64
#undef K32
        err = hipGetLastError();
        timed_end(c, ts);
        done += k;
    }
    return err;
}

hipError_t launch_hmf_small_eval(md_ctx *c, const double *q, const double *p, double *out2, double *f, double *out3,
                                 unsigned *flag)
{
    const int n = (int)c->n;
#define K(P_) k_hmf_small_eval<P_>
    const int ts = timed_begin(c, "k_hmf_small_eval");
    MD_SMALL(32, K, q, p, n, B, c->scal, out2, f, out3, flag);
#undef K
    const hipError_t err = hipGetLastError();
    timed_end(c, ts);
    return err;
}

hipError_t launch_hmf_small_hvp(md_ctx *c, const double *q, const double *w, double *out)
{
    const int n = (int)c->n;
#define K(P_) k_hmf_small_hvp<P_>
    MD_SMALL(32, K, q, w, n, B, out);
#undef K
    return hipGetLastError();
}

hipError_t launch_hmf_small_vjp(md_ctx *c, double b0, double b1, double d0, double d1, int64_t nsteps,
                                const double *q0, const double *pos, size_t stride, double *lq, double *lp)
{
    const StepCoef a{b0, b1, d0, d1};
    const int n = (int)c->n;
    hipError_t err = hipSuccess;
    for (int64_t end = nsteps; end > 0 && err == hipSuccess;) {
        const int k = (int)(end < kHmfSmallSteps ? end : kHmfSmallSteps);
        const int64_t begin = end - k;
        const double *const from = begin == 0 ? q0 : nullptr;
        const double *const at = pos + (size_t)(3 * begin) * stride;
#define K(P_) k_hmf_small_vjp<P_>
        MD_SMALL(8, K, from, at, stride, n, B, a, k, (int)(end == nsteps), lq, lp);
#undef K
        err = hipGetLastError();
        end = begin;
    }
    return err;
}

}  // namespace md

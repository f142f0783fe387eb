// energy.hip -- diagnostic energies, always FP64 arithmetic and FP64 sums:
// K = (1/2) sum p^2; V of eq. 1 (Ring) and eq. 3 (2D) as the sum over pairs
// i < j; V of the HMF model through the magnetization (eq. 5).  The relative
// energy error |E - E0| / |E0| of Sec. 4 is formed from these on the host.
//
// Every sum is a per-thread FP64 partial over a fixed index set, a fixed
// block tree, and a one-block finalize in a fixed order: bitwise reproducible.
#include "device.h"
#include "energy_terms.h"
#include "md_internal.h"

namespace md {
namespace {

static_assert(kEnergyBlock == 4 * kWave, "energy_block: four wavefronts");
constexpr int64_t kEnergyBlocks = 65536;  // most pair partials
constexpr int64_t kEnergyManyBlocks = 8192;
static_assert(kEnergyBlocks <= kRedSlots / 2, "the pair partials have half of the reduction scratch");
constexpr int kKinGrid = 1024;    // most blocks of sum p^2
constexpr int kFinThreads = 1024;  // threads of the one-block finalize
constexpr int kFinBatch = 8;       // loads in flight per thread

// One block's part of sum p^2 over len values (block `block` of `blocks`, 256 threads,
// grid-stride).
__device__ __forceinline__ double sumsq_part(const double *__restrict__ p, int64_t len, int block, int blocks)
{
    double acc = 0.0;
    const int64_t stride = (int64_t)blocks * 256;
    for (int64_t k = (int64_t)block * 256 + threadIdx.x; k < len; k += stride) acc += p[k] * p[k];
    return acc;
}

// Block partials of the potential's pair sum and of sum p^2 (one launch).  Block t <
// ng nc takes the i group t mod ng (64 IPL particles) against the j range t / ng of
// jlen particles (the blocks below the diagonal have nothing to do and write 0); the
// nk blocks after them the grid-stride sum of p^2 over len values.
template <int MODEL, int IPL>
__global__ __launch_bounds__(kEnergyBlock) void k_energy_pairs(const double *__restrict__ q,
                                                               const double *__restrict__ p, int n, int64_t len,
                                                               int ng, int nc, int jlen, int nk, double eps,
                                                               double *__restrict__ redV, double *__restrict__ redK)
{
    __shared__ double lds[kEnergyBlock / kWave];
    __shared__ EnergyWin<MODEL> win[kEnergyBlock / kWave];
    const int t = (int)blockIdx.x;
    if (t < ng * nc) {
        const int i0 = (t % ng) * kWave * IPL, j0 = (t / ng) * jlen;
        const int64_t jend = (int64_t)j0 + jlen;
        const int j1 = jend < n ? (int)jend : n;
        double acc = 0.0;
        if (j1 > i0 + 1) acc = energy_block<MODEL, IPL>(q, (size_t)n, i0, n, j0, j1, eps, win);
        const double b = block_sum(acc, lds);
        if (threadIdx.x == 0) redV[t] = b;
        return;
    }
    const double b = block_sum(sumsq_part(p, len, t - ng * nc, nk), lds);
    if (threadIdx.x == 0) redK[t - ng * nc] = b;
}

// Block partials of sum p^2 over len values (HMF).
__global__ __launch_bounds__(256) void k_sumsq(const double *__restrict__ p, int64_t len, int blocks,
                                               double *__restrict__ red)
{
    __shared__ double lds[4];
    const double b = block_sum(sumsq_part(p, len, (int)blockIdx.x, blocks), lds);
    if (threadIdx.x == 0) red[blockIdx.x] = b;
}

// This thread's part of the sum of red[b stride], b < m, in a fixed order: kFinBatch
// loads at a time (one load, wait and add at a time leaves the one-block kernel bound
// by the memory latency: 65,536 partials took 256 of them in a row).
__device__ __forceinline__ double ordered_part(const double *__restrict__ red, int m, int stride)
{
    double acc = 0.0;
    for (int b0 = 0; b0 < m; b0 += kFinThreads * kFinBatch) {
        double v[kFinBatch];
#pragma unroll
        for (int k = 0; k < kFinBatch; ++k) {
            const int b = b0 + (int)threadIdx.x + kFinThreads * k;
            v[k] = b < m ? red[(size_t)b * stride] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < kFinBatch; ++k) acc += v[k];
    }
    return acc;
}

// out = {K, V, K + V} and the finiteness flag of the three (md_check).  redV: nv pair
// partials (Ring, 2D) or hmf_grid pairs of (sum cos, sum sin) (HMF).  redK: nk
// partials of sum p^2.
__global__ __launch_bounds__(kFinThreads) void k_energy_finalize(const double *__restrict__ redV, int nv,
                                                                 const double *__restrict__ redK, int nk, int model,
                                                                 int n, double *__restrict__ out,
                                                                 unsigned *__restrict__ flag)
{
    __shared__ double lds[3][kFinThreads / kWave];
    const double pk = ordered_part(redK, nk, 1);
    const double pv = ordered_part(redV, nv, model == MD_HMF ? 2 : 1);
    const double ps = model == MD_HMF ? ordered_part(redV + 1, nv, 2) : 0.0;
    const double k2 = block_sum<kFinThreads>(pk, lds[0]);
    const double sv = block_sum<kFinThreads>(pv, lds[1]);
    const double ss = block_sum<kFinThreads>(ps, lds[2]);
    if (threadIdx.x != 0) return;
    double v;
    if (model == MD_HMF) {
        const double mx = sv / (double)n, my = ss / (double)n;
        v = 0.5 * (double)n * (1.0 - mx * mx - my * my);
    } else {
        v = model == MD_GRAV2D ? sv / (double)n : -sv / (sqrt(2.0) * (double)n);
    }
    const double kin = 0.5 * k2;
    out[0] = kin;
    out[1] = v;
    out[2] = kin + v;
    *flag = isfinite(kin) && isfinite(v) && isfinite(kin + v) ? 0u : 1u;
}

// flag = 1 if any of v[0 .. count) is not finite, else 0 (one block).
__global__ __launch_bounds__(256) void k_finite_flag(const double *__restrict__ v, int count,
                                                     unsigned *__restrict__ flag)
{
    int bad = 0;
    for (int k = threadIdx.x; k < count; k += 256) bad |= !isfinite(v[k]);
    bad = __syncthreads_or(bad);
    if (threadIdx.x == 0) *flag = bad ? 1u : 0u;
}

}  // namespace

hipError_t launch_finite_flag(md_ctx *c, const double *vals, int count)
{
    hipLaunchKernelGGL(k_finite_flag, dim3(1), dim3(256), 0, c->stream, vals, count, finite_flag(c));
    return hipGetLastError();
}

// The i groups and j ranges of the pair sum: groups of 64 i (1 a lane) up to n = 32,768,
// where blocks are few, of 256 (4 a lane: a window's LDS read serves four) above, and
// j ranges of 256 (one 64-j window for each of a block's wavefronts) doubled while there
// are more than kEnergyManyBlocks blocks, up to 4096, and within kEnergyBlocks partials.
// Measured, md_energy in us, 1 / 4 a lane: 2D n = 4097 14.0 / 25.7, 8192 21.1 / 25.7,
// 16,384 47.2 / 54.3, 20,000 58.8 / 81.0, 32,768 132 / 146, 65,536 476 / 458; Ring 22.5 / 43.1,
// 39.8 / 59.3, 120 / 153, 171 / 204, 440 / 484, 1646 / 1705.  Blocks at most
// 8192 / 16,384 / 32,768 / 65,536 (4 a lane): 2D n = 65,536 490 / 512 / 545 / 622,
// 262,144 6856 / 6346 / 6139 / 6100.
struct EnergyGrid {
    int ipl, ng, nc, jlen;
};

EnergyGrid energy_grid(int64_t n)
{
    EnergyGrid g;
    g.ipl = n > 32768 ? 4 : 1;
    const int64_t per = (int64_t)kWave * g.ipl;
    const int64_t ng = (n + per - 1) / per;
    int64_t jlen = 4 * kWave;
    auto blocks = [&]() { return ng * ((n + jlen - 1) / jlen); };
    while ((blocks() > kEnergyManyBlocks && jlen < 4096) || blocks() > kEnergyBlocks) jlen *= 2;
    g.ng = (int)ng;
    g.nc = (int)((n + jlen - 1) / jlen);
    g.jlen = (int)jlen;
    return g;
}

// Layout of the reduction scratch: [0, kRedSlots/2) potential partials,
// [kRedSlots/2, kRedSlots/2 + kKinGrid) kinetic partials.
hipError_t launch_energy(md_ctx *c, const double *q, const double *p, double *out3)
{
    if (c->model == MD_HMF && hmf_small_energy(c))
        return launch_hmf_small_eval(c, q, p, nullptr, nullptr, out3, finite_flag(c));
    const int n = (int)c->n;
    const int64_t len = (int64_t)dims(c->model) * n;
    double *redV = c->red;
    double *redK = c->red + kRedSlots / 2;
    const int64_t kb = (len + 1023) / 1024;  // 4 values a thread at least
    const int nk = (int)(kb < kKinGrid ? kb : kKinGrid);
    int nv;
    if (c->model == MD_HMF) {
        // block partials of sum cos, sum sin of q (added here in FP64, in a fixed order; the pass's
        // fixed-point sums are not read)
        hipError_t e = launch_hmf_pass(c, 0, HMF_REDUCE, 0.0, 0.0, 0.0, const_cast<double *>(q), nullptr, nullptr, false);
        if (e != hipSuccess) return e;
        nv = hmf_grid(c->n);
        redV = const_cast<double *>(hmf_partials(c));
        hipLaunchKernelGGL(k_sumsq, dim3((unsigned)nk), dim3(256), 0, c->stream, p, len, nk, redK);
    } else {
        const EnergyGrid g = energy_grid(c->n);
        const dim3 grid((unsigned)(g.ng * g.nc + nk));
        nv = g.ng * g.nc;
#define MD_ENERGY(M_, I_)                                                                                          \
    hipLaunchKernelGGL((k_energy_pairs<M_, I_>), grid, dim3(kEnergyBlock), 0, c->stream, q, p, n, len, g.ng, g.nc, \
                       g.jlen, nk, c->eps, redV, redK)
        if (c->model == MD_GRAV2D) {
            if (g.ipl == 4) MD_ENERGY(MD_GRAV2D, 4);
            else MD_ENERGY(MD_GRAV2D, 1);
        } else {
            if (g.ipl == 4) MD_ENERGY(MD_RING, 4);
            else MD_ENERGY(MD_RING, 1);
        }
#undef MD_ENERGY
    }
    hipLaunchKernelGGL(k_energy_finalize, dim3(1), dim3(kFinThreads), 0, c->stream, redV, nv, redK, nk, c->model, n,
                       out3, finite_flag(c));
    return hipGetLastError();
}

hipError_t launch_magnetization(md_ctx *c, const double *q, double *out2)
{
    if (hmf_small(c)) return launch_hmf_small_eval(c, q, nullptr, out2, nullptr, nullptr, finite_flag(c));
    const hipError_t e =
        launch_hmf_pass(c, 0, HMF_REDUCE, 0.0, 0.0, 0.0, const_cast<double *>(q), nullptr, nullptr, false);
    if (e != hipSuccess) return e;
    return launch_hmf_magnetization(c, out2);
}

}  // namespace md

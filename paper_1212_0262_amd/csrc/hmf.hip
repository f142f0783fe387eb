// hmf.hip -- the Hamiltonian Mean Field model in O(N) (Sec. 3.1): the force
// f_i = cos(t_i) My - sin(t_i) Mx (eq. 6) from the magnetization
// (Mx, My) = (1/N) sum_i (cos t_i, sin t_i) (eq. 7).
//
// Unlike the paper's kernels, the cosines and sines are not stored: one pass
// over the particles reads (t, p) once, kicks with the current magnetization
// (recomputing sincos of the old angle), drifts, takes sincos of the new angle
// for the next magnetization, and writes (t, p) back.  Stored sines/cosines
// would add 32 B of HBM traffic per particle per stage to a bandwidth-bound
// pass; two sincos evaluations cost less.  The magnetization is a grid-wide
// dependency: each pass ends with FP64 block partials (lane exchanges, then a fixed
// serial order over wavefronts), which every block adds in fixed point (limbs of 2^-32
// and 2^-64, 64-bit integer atomics into kMSlots slots) to one of three buffers; every
// wavefront of the next pass sums the slots exactly, in integers, and converts the total
// once to FP64 (no launch between passes).  The second pass of a call takes the first's
// partials instead, as limbs again (partials_mean).
// Integer sums do not depend on the order of the atomics, so M is reproducible,
// and it is the exact sum of the FP64 block partials rounded once.  That is for
// grids of at most kHmfInPassM blocks (N <= 2.1e6); on larger ones every block
// re-deriving M costs more than a launch, so a one-block kernel sums the FP64
// block partials in a fixed order instead (M then differs in its last bits from
// the fixed-point total; either way it is fixed per N, so runs are
// reproducible).  The kernel boundary is the only synchronisation: no
// device-wide fences (on this GPU a device-scope release writes back the L2 of
// the issuing XCD).  The FP64 block partials are always stored (the energy sums
// them in its own fixed order).
//
// Memory access: each lane moves W consecutive elements (16-byte vector loads and
// stores: W = 2 in FP64, 4 in FP32), U vectors per grid-stride iteration, over a
// grid of one block per 256 to 2048 particles (hmf_block; at most 32768 blocks).
// Pointers that are not 16-byte aligned take W = 1.  The FP32 state is made from the
// FP64 arrays by a call's first pass and written back by its last.
//
// Also here: the O(N) Hessian-vector product of the HMF potential (the mean-field
// form of eqs. 6-7) and the passes of its reverse sweep.
#include "device.h"
#include "hmf_terms.h"
#include "md_internal.h"

namespace md {
namespace {

constexpr int kUnroll = 2;  // most vectors per thread per grid-stride iteration

// W consecutive values, aligned to their size (one vector load/store when W > 1).
template <typename T, int W>
struct alignas(sizeof(T) * W) Vec {
    T x[W];
};

// The work of one stage on E particles: kick (with f from f_in or from M), drift,
// and the sincos of the new angle into the partial sums (of the particles with
// ok[e]; in the order of e).  Each step runs over all E particles before the next,
// with no branch between them.
template <typename T, int E>
__device__ __forceinline__ void stage_n(T (&t)[E], T (&p)[E], const double (&fin)[E], double (&fout)[E],
                                        const bool (&ok)[E], T mx, T my, T k1, T k2, T dr, int flags, double &sc,
                                        double &ss)
{
    if (flags & (HMF_KICK_M | HMF_STORE_F)) {
        T s[E], c[E], f[E];
        sincos_n(t, s, c);
#pragma unroll
        for (int e = 0; e < E; ++e) f[e] = c[e] * my - s[e] * mx;
        if (flags & HMF_STORE_F) {
#pragma unroll
            for (int e = 0; e < E; ++e) fout[e] = (double)f[e];
        }
        if (flags & HMF_KICK_M) {
#pragma unroll
            for (int e = 0; e < E; ++e) p[e] += k1 * f[e];
            if (flags & HMF_KICK2) {
#pragma unroll
                for (int e = 0; e < E; ++e) p[e] += k2 * f[e];
            }
        }
    } else if (flags & HMF_KICK_F) {
#pragma unroll
        for (int e = 0; e < E; ++e) p[e] += k1 * (T)fin[e];
    }
    if (flags & HMF_DRIFT) {
#pragma unroll
        for (int e = 0; e < E; ++e) {
            t[e] += dr * p[e];
            if constexpr (sizeof(T) == 4) t[e] = wrap_pi(t[e]);
        }
    }
    if (flags & HMF_REDUCE) {
        T s[E], c[E];
        sincos_n(t, s, c);
#pragma unroll
        for (int e = 0; e < E; ++e) {
            if (ok[e]) {
                sc += (double)c[e];
                ss += (double)s[e];
            }
        }
    }
}

static_assert(kMSlots * kMLimbs == 256, "the 256 limb words: one per thread of the block that zeroes them");
static_assert(kMSlots == kWave && kMLimbs == 4, "one slot per lane of the wavefront that converts the sums");

// x = (hi + lo 2^-32) 2^-32, hi = floor(x 2^32), 0 <= lo <= 2^32: exact for |x| < 2^20
// down to 2^-64 (the bits below are rounded).
__device__ __forceinline__ void to_limbs(double x, long long &hi, long long &lo)
{
    const double y = x * 0x1p32;
    const double h = floor(y);
    hi = (long long)h;
    lo = (long long)rint((y - h) * 0x1p32);
}

// M = (the total of the limb sums) / n in every lane, by one wavefront whose lane l loads
// the limbs of slot l: the slots are added in 64-bit integers (exact, so in any order the
// same total) by lane exchanges, one chain for the four limbs, no LDS and no barrier.
__device__ __forceinline__ void limbs_mean(const long long *__restrict__ acc, int n, double &mx, double &my)
{
    const long long *__restrict__ a = acc + (threadIdx.x & (kWave - 1)) * kMLimbs;
    const long long t = wave_sum4(a[0], a[1], a[2], a[3]);
    mx = ((double)lane_value<0>(t) * 0x1p-32 + (double)lane_value<16>(t) * 0x1p-64) / (double)n;
    my = ((double)lane_value<32>(t) * 0x1p-32 + (double)lane_value<48>(t) * 0x1p-64) / (double)n;
}

// The same M from the g block partials (sum cos, sum sin) of a pass 0, by a block of 256
// (a barrier): each partial as its limbs, added in integers, so the same bits.  Pass 1 of a
// call takes it, so that no launch has to zero a limb buffer before pass 0.  Over the whole
// block, kMeanBatch loads a thread in flight: by each wavefront for itself the conversions
// cost more than that launch.  md_force, us, with it, by each wavefront, and so: N = 1e6
// 12.9, 17.8, 12.4; N = 16,384 11.3, 9.3, 8.9.
constexpr int kMeanBatch = 2;

__device__ __forceinline__ void partials_mean(const double *__restrict__ red, int g, int n, long long (&lds)[4][4],
                                              double &mx, double &my)
{
    long long a[4] = {0, 0, 0, 0};
    for (int b0 = threadIdx.x; b0 < g; b0 += 256 * kMeanBatch) {
        double x[kMeanBatch][2];
#pragma unroll
        for (int j = 0; j < kMeanBatch; ++j) {
            const int b = b0 + 256 * j;
#pragma unroll
            for (int k = 0; k < 2; ++k) x[j][k] = b < g ? red[2 * b + k] : 0.0;
        }
#pragma unroll
        for (int j = 0; j < kMeanBatch; ++j) {
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                long long hi, lo;
                to_limbs(x[j][k], hi, lo);
                a[2 * k] += hi;
                a[2 * k + 1] += lo;
            }
        }
    }
    const int lane = threadIdx.x & (kWave - 1);
    const long long t = wave_sum4(a[0], a[1], a[2], a[3]);
    if (lane % 16 == 0) lds[lane / 16][threadIdx.x / kWave] = t;
    __syncthreads();
    long long s[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) s[k] = (lds[k][0] + lds[k][1]) + (lds[k][2] + lds[k][3]);
    mx = ((double)s[0] * 0x1p-32 + (double)s[1] * 0x1p-64) / (double)n;
    my = ((double)s[2] * 0x1p-32 + (double)s[3] * 0x1p-64) / (double)n;
}

// One kick/drift/reduce pass over all particles (grid-stride over a grid fixed
// per n, so every partial sum is reproducible).  T: state type; W: elements per
// vector access; U: vectors per thread and iteration.  HMF_REDUCE writes the block
// partials (sum cos, sum sin) to red[2b], red[2b+1].  LIMBS (in-pass sums):
// HMF_KICK_M / HMF_STORE_F take the magnetization from the limb sums mrd, each
// wavefront by itself (block 0 also stores it to M), HMF_REDUCE adds the partials'
// limbs to mwr, and block 0 zeroes mzero for the next pass.
// Without LIMBS the kernel reads M[0..1] and leaves the partials to the one-block
// kernel (no code of the limbs).  Launched with 256 threads.
// f: read by HMF_KICK_F, written by HMF_STORE_F.  macc: the limb sums, three buffers
// [kMSlots][kMLimbs] in turn: buf is read, the next added to, the one after it zeroed.
// HMF_FIRST (pass 0): nothing is added.  HMF_SECOND (pass 1): M comes from pass 0's partials,
// 2 kHmfInPassM before this pass's red.
// FP32 state: HMF_IN64 takes the state from th64, p64 instead (angles wrapped),
// HMF_OUT64 writes it there.  FP64 state: the drifted angles also go to snap (both x64).
template <typename T, int W, int U, bool LIMBS>
__global__ __launch_bounds__(256) void k_hmf_pass(T *__restrict__ th, T *__restrict__ p,
                                                  long long *__restrict__ macc, double *__restrict__ M, int n,
                                                  int grid, int flags, int buf, double *__restrict__ f,
                                                  double *__restrict__ red, double kick1, double kick2, double drift,
                                                  double *__restrict__ x64, double *__restrict__ p64)
{
    __shared__ double lds[2][4];
    __shared__ long long mlds[4][4];
    double *__restrict__ th64 = x64;  // FP32 state
    double *__restrict__ snap = x64;  // FP64 state
    constexpr int B = kMSlots * kMLimbs;  // words per limb buffer; the three in turn: read, add, zero
    const long long *__restrict__ mrd = macc + buf * B;
    long long *__restrict__ mwr = macc + (buf == 2 ? 0 : buf + 1) * B;
    long long *__restrict__ mzero = macc + (buf == 0 ? 2 : buf - 1) * B;
    const T k1 = (T)kick1, k2 = (T)kick2, dr = (T)drift;
    const bool in64 = sizeof(T) == 4 && (flags & HMF_IN64), out64 = sizeof(T) == 4 && (flags & HMF_OUT64);
    const bool take_snap = sizeof(T) == 8 && snap && (flags & HMF_DRIFT);
    T mx = 0, my = 0;
    if (flags & (HMF_KICK_M | HMF_STORE_F)) {
        if constexpr (LIMBS) {
            double dmx, dmy;
            if (flags & HMF_SECOND) partials_mean(red - 2 * kHmfInPassM, grid, n, mlds, dmx, dmy);
            else limbs_mean(mrd, n, dmx, dmy);
            if (blockIdx.x == 0 && threadIdx.x == 0) {
                M[0] = dmx;
                M[1] = dmy;
            }
            mx = (T)dmx;
            my = (T)dmy;
        } else {
            mx = (T)M[0];
            my = (T)M[1];
        }
    }
    if (LIMBS && blockIdx.x == 0) mzero[threadIdx.x] = 0;
    const bool need_p = flags & (HMF_KICK_F | HMF_KICK_M | HMF_DRIFT);
    const bool write = flags & HMF_WRITE;
    double sc = 0.0, ss = 0.0;
    const int nvec = n / W;
    const int stride = grid * 256;
    using VT = Vec<T, W>;
    using VD = Vec<double, W>;
    constexpr int E = U * W;  // particles per thread and iteration: e = u W + w
    for (int base = blockIdx.x * 256 + threadIdx.x; base < nvec; base += stride * U) {
        VT t[U], q[U];
        VD fi[U];
        bool ok[E];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = base + u * stride;
            t[u] = VT{};
            q[u] = VT{};
            fi[u] = VD{};
            if (v < nvec) {
                if (in64) {  // the call's first pass: element loads, any alignment
#pragma unroll
                    for (int w = 0; w < W; ++w) {
                        if constexpr (sizeof(T) == 4) t[u].x[w] = wrap_pi((float)th64[v * W + w]);
                        q[u].x[w] = (T)p64[v * W + w];
                    }
                } else {
                    t[u] = reinterpret_cast<const VT *>(th)[v];
                    if (need_p) q[u] = reinterpret_cast<const VT *>(p)[v];
                }
                if (flags & HMF_KICK_F) fi[u] = reinterpret_cast<const VD *>(f)[v];
            }
#pragma unroll
            for (int w = 0; w < W; ++w) ok[u * W + w] = v < nvec;
        }
        T te[E], pe[E];
        double fe[E], fo[E];
#pragma unroll
        for (int e = 0; e < E; ++e) {
            te[e] = t[e / W].x[e % W];
            pe[e] = q[e / W].x[e % W];
            fe[e] = fi[e / W].x[e % W];
            fo[e] = 0.0;
        }
        stage_n(te, pe, fe, fo, ok, mx, my, k1, k2, dr, flags, sc, ss);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int v = base + u * stride;
            if (v >= nvec) continue;
            VT to, po;
            VD ff;
#pragma unroll
            for (int w = 0; w < W; ++w) {
                to.x[w] = te[u * W + w];
                po.x[w] = pe[u * W + w];
                ff.x[w] = fo[u * W + w];
            }
            if (flags & HMF_STORE_F) reinterpret_cast<VD *>(f)[v] = ff;
            if (write && out64) {
#pragma unroll
                for (int w = 0; w < W; ++w) {
                    th64[v * W + w] = (double)to.x[w];
                    p64[v * W + w] = (double)po.x[w];
                }
            } else if (write) {
                reinterpret_cast<VT *>(th)[v] = to;
                if (need_p) reinterpret_cast<VT *>(p)[v] = po;
            }
            if (take_snap) {
#pragma unroll
                for (int w = 0; w < W; ++w) snap[v * W + w] = to.x[w];
            }
        }
    }
    // the n mod W particles past the last full vector: block 0
    if (W > 1 && blockIdx.x == 0 && (int)threadIdx.x < n - nvec * W) {
        const int i = nvec * W + threadIdx.x;
        T t1[1], p1[1] = {T(0)};
        if (in64) {
            if constexpr (sizeof(T) == 4) t1[0] = wrap_pi((float)th64[i]);
            p1[0] = (T)p64[i];
        } else {
            t1[0] = th[i];
            if (need_p) p1[0] = p[i];
        }
        const double f1[1] = {(flags & HMF_KICK_F) ? f[i] : 0.0};
        double fo1[1] = {0.0};
        const bool ok1[1] = {true};
        stage_n(t1, p1, f1, fo1, ok1, mx, my, k1, k2, dr, flags, sc, ss);
        if (flags & HMF_STORE_F) f[i] = fo1[0];
        if (write && out64) {
            th64[i] = (double)t1[0];
            p64[i] = (double)p1[0];
        } else if (write) {
            th[i] = t1[0];
            if (need_p) p[i] = p1[0];
        }
        if (take_snap) snap[i] = t1[0];
    }
    if (flags & HMF_REDUCE) {
        // lane 0 of a wavefront has its sum cos, lane 32 its sum sin; the first
        // wavefront's then add the block's in order and their limbs
        const int lane = threadIdx.x & (kWave - 1), k = lane / 32;
        const double t = wave_sum2(sc, ss);
        if (lane % 32 == 0) lds[k][threadIdx.x / kWave] = t;
        __syncthreads();
        if (threadIdx.x < kWave && lane % 32 == 0) {
            const double b = ((lds[k][0] + lds[k][1]) + lds[k][2]) + lds[k][3];
            red[2 * blockIdx.x + k] = b;
            if (LIMBS && !(flags & HMF_FIRST)) {
                unsigned long long *w =
                    reinterpret_cast<unsigned long long *>(mwr + (blockIdx.x % kMSlots) * kMLimbs + 2 * k);
                long long hi, lo;
                to_limbs(b, hi, lo);
                atomicAdd(w, (unsigned long long)hi);  // two's complement: the signed sum, exactly
                atomicAdd(w + 1, (unsigned long long)lo);
            }
        }
    }
}

// M from the g block partials of a pass 0 (one block), to M[0..1] and (if given) out[0..1].
__global__ __launch_bounds__(256) void k_hmf_limbs_to_m(const double *__restrict__ red, int g, int n,
                                                          double *__restrict__ out, double *__restrict__ M)
{
    __shared__ long long lds[4][4];
    double mx, my;
    partials_mean(red, g, n, lds, mx, my);
    if (threadIdx.x == 0) {
        if (out) {
            out[0] = mx;
            out[1] = my;
        }
        M[0] = mx;
        M[1] = my;
    }
}

// M[0..1] = (sum of the g partial pairs) / n, in a fixed order (one block of
// 1024 threads; thread t adds partials t, t + 1024, ... in that order).  Loads go
// out kFinBatch per thread at a time, which keeps the kernel in registers (no
// private segment) at 1024 threads; g <= kHmfGrid takes at most 4 batches.
constexpr int kFinBatch = 8;

__global__ __launch_bounds__(1024) void k_hmf_finalize(const double *__restrict__ red, int g, int n,
                                                       double *__restrict__ M)
{
    __shared__ double lds[2][16];
    double c = 0.0, s = 0.0;
    for (int b0 = 0; b0 < g; b0 += 1024 * kFinBatch) {
        double vc[kFinBatch], vs[kFinBatch];
#pragma unroll
        for (int k = 0; k < kFinBatch; ++k) {
            const int b = b0 + threadIdx.x + 1024 * k;
            vc[k] = b < g ? red[2 * b] : 0.0;
            vs[k] = b < g ? red[2 * b + 1] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < kFinBatch; ++k) {
            c += vc[k];
            s += vs[k];
        }
    }
    // lane 0 of each wavefront has its sum cos, lane 32 its sum sin; then the first
    // wavefront's rows of lanes add the wavefronts'
    const int lane = threadIdx.x & (kWave - 1), k = lane / 32;
    const double t = wave_sum2(c, s);
    if (lane % 32 == 0) lds[k][threadIdx.x / kWave] = t;
    __syncthreads();
    if (threadIdx.x >= kWave) return;
    const double m = row_sum(lds[k][lane % 16]) / (double)n;
    if (lane % 32 == 0) M[k] = m;
}

// ------------------------------------------------------------------- adjoint --
// HMF Hessian-vector product, O(N): phi''(d) = cos(d)/N gives
//   (H w)_i = w_i (c_i Mx + s_i My) - (c_i Cw + s_i Sw),
// Mx, My the magnetization (eq. 7), Cw = (1/N) sum c_j w_j, Sw = (1/N) sum s_j w_j.

//
// A pass applies one product and takes the sums of the next (k_hmf_adj_pass): per
// product t of both positions, lq and lp read and lq, lp written once, 48 B a particle.
// Measured, md_step_vjp of four steps, us, before (a pass for the sums, a one-block kernel
// over up to 4096 partials, an elementwise kernel: 56 B a particle and three launches)
// and after: N = 16,384 235 -> 106; 100,003 256 -> 129; 1e6 533 -> 266; 4e6 1282 -> 913.

// sums[0..3] = (Mx, My, Cw, Sw) from the g block partials of each, by a block: thread t
// adds quadruples t, t + T, ..., kAdjBatch loads at a time, then wave_sum4 and the
// wavefronts in order.  In every thread (a barrier).  The passes of at most kAdjInPass
// blocks take it at their start; on larger grids it costs every block more than the
// one-block kernel.
constexpr int kAdjBatch = 2;
constexpr int kAdjInPass = 512;

template <int T>
__device__ __forceinline__ void adj_means(const double *__restrict__ part, int g, int n, double (&lds)[4][T / kWave],
                                          double (&v)[4])
{
    double a[4] = {0.0, 0.0, 0.0, 0.0};
    for (int b0 = 0; b0 < g; b0 += T * kAdjBatch) {
        double x[kAdjBatch][4];
#pragma unroll
        for (int k = 0; k < kAdjBatch; ++k) {
            const int b = b0 + (int)threadIdx.x + T * k;
#pragma unroll
            for (int j = 0; j < 4; ++j) x[k][j] = b < g ? part[4 * b + j] : 0.0;
        }
#pragma unroll
        for (int k = 0; k < kAdjBatch; ++k)
#pragma unroll
            for (int j = 0; j < 4; ++j) a[j] += x[k][j];
    }
    const int lane = threadIdx.x & (kWave - 1);
    const double t = wave_sum4(a[0], a[1], a[2], a[3]);
    if (lane % 16 == 0) lds[lane / 16][threadIdx.x / kWave] = t;
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < T / kWave; ++w) s += lds[j][w];
        v[j] = s / (double)n;
    }
}

__global__ __launch_bounds__(1024) void k_hmf_adj_finalize(const double *__restrict__ red, int g, int n,
                                                           double *__restrict__ sums)
{
    __shared__ double lds[4][1024 / kWave];
    double v[4];
    adj_means<1024>(red, g, n, lds, v);
    if (threadIdx.x == 0) {
#pragma unroll
        for (int j = 0; j < 4; ++j) sums[j] = v[j];
    }
}

// Elementwise (g blocks of 256 threads), with the product hw = H(th) lp from its sums
// (part_in, g blocks of them, or sums): out = hw (ADJ_OUT); lq -= h hw (ADJ_KICK), lq -= h2 hw (ADJ_KICK2);
// lp += a lq (ADJ_DRIFT).  Then, if th_next is given, the block partials of the sums of
// H(th_next) lp to part_out.  Grid-stride over a grid fixed per n.  W: elements per
// vector access; U: vectors per thread and iteration; IN: sums from part_in.
template <int W, int U, bool IN>
__global__ __launch_bounds__(256) void k_hmf_adj_pass(const double *__restrict__ th, const double *__restrict__ part_in,
                                                      const double *__restrict__ sums, int g, int flags, int n,
                                                      double h, double h2, double a, double *__restrict__ lq,
                                                      double *__restrict__ lp, double *__restrict__ out,
                                                      const double *__restrict__ th_next,
                                                      double *__restrict__ part_out)
{
    __shared__ double lds[2][4][4];
    using VD = Vec<double, W>;
    constexpr int E = U * W;
    const bool product = flags & (ADJ_OUT | ADJ_KICK);
    double v[4] = {0.0, 0.0, 0.0, 0.0};
    if (product) {
        if constexpr (IN) {
            adj_means<256>(part_in, g, n, lds[0], v);
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = sums[j];
        }
    }
    double sum[4] = {0.0, 0.0, 0.0, 0.0};
    // E particles: t of this product and of the next, lq, lp, hw; ok[e]: they exist
    auto stage = [&](auto &t, auto &tn, auto &x, auto &w, auto &hw, const auto &ok) {
        constexpr int N = sizeof(ok) / sizeof(ok[0]);
        double s[N], c[N];
        if (product) {
            sincos_n(t, s, c);
#pragma unroll
            for (int e = 0; e < N; ++e) {
                hw[e] = w[e] * (c[e] * v[0] + s[e] * v[1]) - (c[e] * v[2] + s[e] * v[3]);
                if (flags & ADJ_KICK) x[e] -= h * hw[e];
                if (flags & ADJ_KICK2) x[e] -= h2 * hw[e];
            }
        }
        if (flags & ADJ_DRIFT) {
#pragma unroll
            for (int e = 0; e < N; ++e) w[e] += a * x[e];
        }
        if (th_next) {
            sincos_n(tn, s, c);
#pragma unroll
            for (int e = 0; e < N; ++e) {
                if (ok[e]) {
                    sum[0] += c[e];
                    sum[1] += s[e];
                    sum[2] += c[e] * w[e];
                    sum[3] += s[e] * w[e];
                }
            }
        }
    };
    const bool need_x = flags & (ADJ_KICK | ADJ_DRIFT);
    const int nvec = n / W, stride = g * 256;
    for (int base = blockIdx.x * 256 + threadIdx.x; base < nvec; base += stride * U) {
        double t[E], tn[E], x[E], w[E], hw[E];
        bool ok[E];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = base + u * stride;
            const bool in = k < nvec;
            VD vt{}, vn{}, vx{}, vw{};
            if (in) {
                if (product) vt = reinterpret_cast<const VD *>(th)[k];
                if (th_next) vn = reinterpret_cast<const VD *>(th_next)[k];
                if (need_x) vx = reinterpret_cast<const VD *>(lq)[k];
                vw = reinterpret_cast<const VD *>(lp)[k];
            }
#pragma unroll
            for (int e = 0; e < W; ++e) {
                t[u * W + e] = vt.x[e];
                tn[u * W + e] = vn.x[e];
                x[u * W + e] = vx.x[e];
                w[u * W + e] = vw.x[e];
                hw[u * W + e] = 0.0;
                ok[u * W + e] = in;
            }
        }
        stage(t, tn, x, w, hw, ok);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int k = base + u * stride;
            if (k >= nvec) continue;
            VD vx, vw, vo;
#pragma unroll
            for (int e = 0; e < W; ++e) {
                vx.x[e] = x[u * W + e];
                vw.x[e] = w[u * W + e];
                vo.x[e] = hw[u * W + e];
            }
            if (flags & ADJ_OUT) reinterpret_cast<VD *>(out)[k] = vo;
            if (flags & ADJ_KICK) reinterpret_cast<VD *>(lq)[k] = vx;
            if (flags & ADJ_DRIFT) reinterpret_cast<VD *>(lp)[k] = vw;
        }
    }
    // the n mod W particles past the last full vector: block 0
    if (W > 1 && blockIdx.x == 0 && (int)threadIdx.x < n - nvec * W) {
        const int i = nvec * W + threadIdx.x;
        double t[1] = {product ? th[i] : 0.0}, tn[1] = {th_next ? th_next[i] : 0.0}, x[1] = {need_x ? lq[i] : 0.0},
               w[1] = {lp[i]}, hw[1] = {0.0};
        const bool ok[1] = {true};
        stage(t, tn, x, w, hw, ok);
        if (flags & ADJ_OUT) out[i] = hw[0];
        if (flags & ADJ_KICK) lq[i] = x[0];
        if (flags & ADJ_DRIFT) lp[i] = w[0];
    }
    if (th_next) {
        const int lane = threadIdx.x & (kWave - 1), j = lane / 16;
        const double t = wave_sum4(sum[0], sum[1], sum[2], sum[3]);
        if (lane % 16 == 0) lds[1][j][threadIdx.x / kWave] = t;
        __syncthreads();
        if (threadIdx.x < kWave && lane % 16 == 0)
            part_out[4 * blockIdx.x + j] = ((lds[1][j][0] + lds[1][j][1]) + lds[1][j][2]) + lds[1][j][3];
    }
}

}  // namespace

// Vector width of the accesses for this context (1 when a pointer is not 16-byte aligned).
static int vec_width(bool f32, const void *a, const void *b, const void *c, const void *d = nullptr)
{
    const uintptr_t m = (uintptr_t)a | (uintptr_t)b | (uintptr_t)c | (uintptr_t)d;
    if (m & 15u) return 1;
    return f32 ? 4 : 2;
}

// Particles of a pass block: 2048 (two grid-stride iterations of W = 2 at U = 2) at large
// n; measured at N = 1e7 against 1024 (7% slower: each block's closing reduction is
// amortised over fewer particles) and 4096 (2% slower).  Below, as few as keep the
// grid within kHmfInPassM blocks, 256 at least: a thread's particles are a serial
// chain, and 2048 a block leaves most CUs idle (49 blocks at N = 1e5).
// Measured, us per step before (2048 a block, M by a barrier and LDS in every block) and
// after, FP64 / FP32 state: N = 16,384 21.5 / 19.4 -> 12.0 / 11.4; 100,003 22.6 / 20.0 ->
// 13.6 / 12.4; 400,000 24.5 / 21.0 -> 19.1 / 16.0; 1e6 33.0 / 26.3 -> 27.7 / 19.8 (and with
// the cheaper launches of device.h 9.9 / 9.2, 11.3 / 10.6, 17.4 / 15.2, 26.2 / 19.1).
static int64_t hmf_block(int64_t n)
{
    int64_t per = 256;
    while (per < 256 * kUnroll * 2 * 2 && n > per * kHmfInPassM) per *= 2;
    return per;
}

// Blocks of an HMF pass.  At most kHmfGrid (N = 6.7e7); above that the grid strides.
// Capping at 16384 instead made N = 5e7 8% slower.
int hmf_grid(int64_t n)
{
    const int64_t per_block = hmf_block(n);
    const int64_t b = (n + per_block - 1) / per_block;
    return (int)(b < kHmfGrid ? (b < 1 ? 1 : b) : kHmfGrid);
}

const double *hmf_partials(const md_ctx *c) { return c->red; }

// The passes of this context sum M in fixed point (small grids) rather than
// through the one-block kernel over the FP64 partials.
static bool hmf_in_pass(const md_ctx *c) { return hmf_grid(c->n) <= kHmfInPassM; }  // n <= 2,097,152

hipError_t launch_hmf_pass(md_ctx *c, int k, int flags, double kick1, double kick2, double drift, double *th,
                           double *p, double *f, bool f32state, double *snap)
{
    if (!f32state) flags &= ~(HMF_IN64 | HMF_OUT64);
    const int n = (int)c->n;
    const int g = hmf_grid(c->n);
    // Small grids: M from the limb sums inside the pass, no other launch.  Large
    // ones: the one-block kernel over the FP64 partials after a reducing pass, and
    // M read from c->scal.
    const bool in_pass = hmf_in_pass(c);
    // the partials alternate between two halves of the scratch when a pass reads them; the
    // energy and the one-block kernels take the first half's
    static_assert(4 * kHmfInPassM <= kRedSlots, "two halves of block partials");
    double *red = in_pass && k == 1 ? c->red + 2 * kHmfInPassM : c->red;
    const int buf = (k + 2) % 3;
    if (k < 2) flags |= k == 0 ? HMF_FIRST : HMF_SECOND;
    const bool vec = (f32state ? vec_width(true, c->th32, c->p32, f) : vec_width(false, th, p, f)) > 1;
    // the vector and unroll that give a thread hmf_block / 256 particles (two iterations
    // of kUnroll 16-byte vectors at most); W = 1 where a pointer is not 16-byte aligned
    const int per = (int)(hmf_block(c->n) / 256);
    const int ts = timed_begin(c, "k_hmf_pass");
#define MD_HMF_PASS(T_, W_, U_, L_, TH_, P_, X_)                                                                 \
    hipLaunchKernelGGL((k_hmf_pass<T_, W_, U_, L_>), dim3(g), dim3(256), 0, c->stream, TH_, P_, c->macc, c->scal, n, \
                       g, flags, buf, f, red, kick1, kick2, drift, X_, p)
#define MD_HMF_FORM(T_, V_, TH_, P_, X_)                                                     \
    do {                                                                                     \
        if (!in_pass && vec) MD_HMF_PASS(T_, V_, kUnroll, false, TH_, P_, X_);               \
        else if (!in_pass) MD_HMF_PASS(T_, 1, kUnroll, false, TH_, P_, X_);                  \
        else if (vec && per >= V_ * kUnroll) MD_HMF_PASS(T_, V_, kUnroll, true, TH_, P_, X_); \
        else if (vec && per >= V_) MD_HMF_PASS(T_, V_, 1, true, TH_, P_, X_);                \
        else if (per >= kUnroll) MD_HMF_PASS(T_, 1, kUnroll, true, TH_, P_, X_);             \
        else MD_HMF_PASS(T_, 1, 1, true, TH_, P_, X_);                                       \
    } while (0)
    if (f32state) MD_HMF_FORM(float, 4, c->th32, c->p32, th);
    else MD_HMF_FORM(double, 2, th, p, snap);  // snap: element stores, any alignment
#undef MD_HMF_FORM
#undef MD_HMF_PASS
    hipError_t e = hipGetLastError();
    timed_end(c, ts);
    if (e == hipSuccess && !in_pass && (flags & HMF_REDUCE)) {
        hipLaunchKernelGGL(k_hmf_finalize, dim3(1), dim3(1024), 0, c->stream, c->red, g, n, c->scal);
        e = hipGetLastError();
    }
    return e;
}

hipError_t launch_hmf_magnetization(md_ctx *c, double *out2)
{
    if (!hmf_in_pass(c))  // the reducing pass's one-block kernel left M in c->scal
        return hipMemcpyAsync(out2, c->scal, 2 * sizeof(double), hipMemcpyDeviceToDevice, c->stream);
    hipLaunchKernelGGL(k_hmf_limbs_to_m, dim3(1), dim3(256), 0, c->stream, c->red, hmf_grid(c->n), (int)c->n, out2,
                       c->scal);
    return hipGetLastError();
}

// One pass of the product (k_hmf_adj_pass), the k-th of a call: its sums come from pass
// k - 1, the next product's (th_next, nullable) go to pass k + 1.  The block partials
// alternate between two halves of the scratch; with more than kAdjInPass blocks a
// one-block kernel turns them into the context scalars c->scal[4..7].
hipError_t launch_hmf_adj_pass(md_ctx *c, int k, const double *th, int flags, double h, double h2, double a,
                               double *lq, double *lp, double *out, const double *th_next)
{
    const int n = (int)c->n;
    // 256 to 2048 particles a block (1, 2, 4 or 8 a thread), as few as keep the grid
    // within kAdjInPass; above, 2048 and a grid-stride loop
    int64_t per = 256;
    while (per < 2048 && c->n > per * kAdjInPass) per *= 2;
    int64_t blocks = (c->n + per - 1) / per;
    if (blocks > kHmfGrid) blocks = kHmfGrid;
    const bool in = blocks <= kAdjInPass;
    static_assert(4 * kHmfGrid <= kRedSlots && 8 * kAdjInPass <= kRedSlots, "the partials fit the scratch");
    double *part[2] = {c->red, in ? c->red + 4 * kAdjInPass : c->red};
    const double *pin = part[(k + 1) & 1];
    double *pout = part[k & 1];
    const bool vec = vec_width(false, th, lq, lp, out) > 1 && ((uintptr_t)th_next & 15u) == 0 && per >= 512;
    const dim3 grid((unsigned)blocks), block(256);
#define MD_ADJ_PASS(W_, U_, IN_)                                                                                  \
    hipLaunchKernelGGL((k_hmf_adj_pass<W_, U_, IN_>), grid, block, 0, c->stream, th, pin, c->scal + 4, (int)blocks, \
                       flags, n, h, h2, a, lq, lp, out, th_next, pout)
    if (!in) {
        if (vec) MD_ADJ_PASS(2, 2, false);
        else MD_ADJ_PASS(1, 2, false);
    } else if (per == 256) MD_ADJ_PASS(1, 1, true);
    else if (vec && per == 512) MD_ADJ_PASS(2, 1, true);
    else if (vec) MD_ADJ_PASS(2, 2, true);
    else MD_ADJ_PASS(1, 2, true);
#undef MD_ADJ_PASS
    hipError_t e = hipGetLastError();
    if (e == hipSuccess && th_next && !in) {
        hipLaunchKernelGGL(k_hmf_adj_finalize, dim3(1), dim3(1024), 0, c->stream, pout, (int)blocks, n, c->scal + 4);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace md

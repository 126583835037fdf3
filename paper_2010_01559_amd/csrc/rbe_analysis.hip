// rbe_analysis.hip -- analysis kernels that are not part of a time step.
//
// Pair-distance counts by charge class (Sec. 4.1: the pair correlations
// g_++ and g_+- of the charge-charge correlation rho(r) = g_++ - g_+-).  A pair
// at distance r < r_max falls in bin floor(r / dr), with r the square root of
// dx^2 + dy^2 + dz^2 of the minimum-image displacement in FP64, every
// operation rounded on its own (contraction into fused multiply-adds is
// switched off), so that the bin is the one the plain definition gives.
//
// All pairs i < j of a system are visited as jobs of 256 particles i against a
// chunk of particles j; blocks of 16 waves take jobs in turn, so that they end
// together, and add their LDS histogram (32-bit atomics) to the global int64
// counts at their end, and before that whenever the jobs since could have filled a
// counter (PairHistPlan::flush).  Each pair's bin first comes from 32-bit fixed-point box
// fractions in single precision (12 instructions and a square root); only where
// that value lies within its error bound of a bin edge, or a particle's
// coordinates are outside the range of the bound, is the FP64 definition
// evaluated: the counts are those of the definition for every pair.  Measured
// at N = 30001, 200 bins, r_max = 0.499 L: 9.7 ms with the definition for every
// pair (three divisions and a square root in FP64) on one block per 256
// particles, 430 us now (28 VALU instructions per 64 pairs by the counters, one of them a
// square root, and two LDS accesses).
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>

#include "rbe_device.h"
#include "rbe_internal.h"

namespace rbe {

constexpr int kHistTile = kPairHistTile;      // particles i of a job
constexpr int kHistBlock = 1024;              // four groups of 256 threads share the job's particles j
constexpr uint32_t kHistSlow = 0x80000000u;   // the record's fractions are not within the error bound

// LDS record of a particle: fixed-point box fractions and its class offset
// (nbins when q > 0), with kHistSlow.
__device__ __forceinline__ uint4 hist_record(double x, double y, double z, bool plus, const SysDev &S, int nbins)
{
    // fractions carry at most 2^-32 from x / L for |x| < 2^20 L; NaN fails the test
    const double lim = 1048576.0 * S.L;
    const bool ok = fabs(x) < lim && fabs(y) < lim && fabs(z) < lim;
    return make_uint4(to_fix(frac01(x * S.invL)), to_fix(frac01(y * S.invL)), to_fix(frac01(z * S.invL)),
                      (plus ? (uint32_t)nbins : 0u) | (ok ? 0u : kHistSlow));
}

// Bin of the definition, or -1.
__device__ __noinline__ int hist_exact(double xi, double yi, double zi, double xj, double yj, double zj, double L,
                                       double r_max, double dr, int nbins)
{
#pragma clang fp contract(off)
    double dx = xj - xi, dy = yj - yi, dz = zj - zi;
    dx = dx - L * rint(dx / L);
    dy = dy - L * rint(dy / L);
    dz = dz - L * rint(dz / L);
    const double r = sqrt(dx * dx + dy * dy + dz * dz);
    if (!(r < r_max)) return -1;
    const int b = (int)floor(r / dr);
    return b < nbins ? b : -1;
}

// jw: particles j of a job (16, 64 or 256); flush: jobs after which a counter could
// wrap; blocks of one system along x, systems along y.
template <typename T>
__global__ __launch_bounds__(kHistBlock) void k_pair_hist(const SysDev *__restrict__ sys, const T *__restrict__ pos,
                                                          const T *__restrict__ q, int64_t ntot, double r_max,
                                                          int nbins, int jw, int flush,
                                                          unsigned long long *__restrict__ counts)
{
    extern __shared__ unsigned int hist[];   // [3][nbins]
    __shared__ uint4 rec[kHistTile];
    __shared__ int any_slow;   // some particle j of the job is outside the range of the bound
    const SysDev S = sys[blockIdx.y];
    const int tid = threadIdx.x, lane256 = tid & 255, group = tid >> 8;
    for (int k = tid; k < 3 * nbins; k += kHistBlock) hist[k] = 0u;
    const int n = S.n;
    const T *px = pos + S.off, *py = px + ntot, *pz = py + ntot, *pq = q + S.off;
    const double L = S.L, dr = r_max / nbins;
    // bf = r / dr in single precision is within 5e-7 bf + e1 of the exact
    // quotient: 2^-24 for each conversion, product and the square root, and
    // four units of 2^-32 L per coordinate difference
    const float cs = (float)(L * (1.0 / 4294967296.0) / dr);
    const float e1 = 8.0f * cs;
    const float top = (float)nbins + 1.0f + 2.0f * e1;
    const uint32_t all_slow = e1 < 0.25f ? 0u : kHistSlow;   // bins finer than the fractions resolve
    const int T0 = (n + kHistTile - 1) / kHistTile, NC = (n + jw - 1) / jw, ratio = kHistTile / jw;
    // jobs of tile I: chunks J = I ratio .. NC - 1
    auto first_job = [&](int64_t I) { return I * NC - ratio * (I * (I - 1) / 2); };
    const int64_t jobs = first_job(T0);
    const int jper = jw >> 2;   // particles j of a group
    // (the first barrier of the next run of jobs is ahead of its counts)
    for (int64_t k = blockIdx.x; k < jobs;) {
        const int64_t run = min(jobs, k + (int64_t)flush * gridDim.x);
        for (; k < run; k += gridDim.x) {
            const double bq = (double)NC + 0.5 * ratio;
            int64_t I = (int64_t)((bq - sqrt(fmax(bq * bq - 2.0 * ratio * (double)k, 0.0))) / ratio);
            I = I < 0 ? 0 : (I >= T0 ? T0 - 1 : I);
            while (I > 0 && first_job(I) > k) --I;
            while (I + 1 < T0 && first_job(I + 1) <= k) ++I;
            const int J = (int)(I * ratio + (k - first_job(I)));
            const int i = (int)I * kHistTile + lane256, j0 = J * jw;
            const bool act = i < n;
            const int ic = act ? i : n - 1;
            const double xi = (double)px[ic], yi = (double)py[ic], zi = (double)pz[ic];
            const uint4 ri = hist_record(xi, yi, zi, pq[ic] > (T)0, S, nbins);
            __syncthreads();   // the job before has read rec
            if (tid == 0) any_slow = 0;
            __syncthreads();
            if (tid < jw && j0 + tid < n) {
                const int j = j0 + tid;
                const uint4 v = hist_record((double)px[j], (double)py[j], (double)pz[j], pq[j] > (T)0, S, nbins);
                rec[tid] = v;
                if (v.w & kHistSlow) any_slow = 1;
            }
            __syncthreads();
            if (!act) continue;
            // classes 0 ++, 1 +-, 2 --; a particle i outside the range of the bound
            // takes the definition for all its pairs
            const bool i_slow = (ri.w | all_slow) & kHistSlow;
            const int base = 2 * nbins - (int)(ri.w & ~kHistSlow);
            const float e1i = i_slow ? 1.0f : e1;
            const float topi = i_slow ? INFINITY : top;
            const int u0 = group * jper;
            auto exact = [&](int u) {
                return hist_exact(xi, yi, zi, (double)px[j0 + u], (double)py[j0 + u], (double)pz[j0 + u], L, r_max, dr,
                                  nbins);
            };
            // one pair, its bin quotient bf in single precision
            auto count = [&](const uint4 &rj, float bf, int u, bool slow) {
                if (!(bf < topi) && !slow) return;
                const float fl = floorf(bf);
                int b = (int)fl;
                if (fabsf(bf - fl - 0.5f) + fmaf(5e-7f, bf, e1i) > 0.5f || slow) b = exact(u);
                if ((uint32_t)b < (uint32_t)nbins) atomicAdd(&hist[base - (int)(rj.w & ~kHistSlow) + b], 1u);
            };
            auto quotient = [&](const uint4 &rj) {
                const float dx = (float)(int32_t)(rj.x - ri.x), dy = (float)(int32_t)(rj.y - ri.y),
                            dz = (float)(int32_t)(rj.z - ri.z);
                return __builtin_amdgcn_sqrtf(fmaf(dx, dx, fmaf(dy, dy, dz * dz))) * cs;
            };
            if (j0 >= (I + 1) * kHistTile && j0 + jw <= n && !any_slow) {
                // a whole chunk past the tile: four records at once, whose LDS
                // latency overlaps the arithmetic, and no test per pair
                for (int u = u0; u < u0 + jper; u += 4) {
                    uint4 rj[4];
                    float bf[4];
#pragma unroll
                    for (int t = 0; t < 4; ++t) rj[t] = rec[u + t];
#pragma unroll
                    for (int t = 0; t < 4; ++t) bf[t] = quotient(rj[t]);
#pragma unroll
                    for (int t = 0; t < 4; ++t) count(rj[t], bf[t], u + t, false);
                }
            } else {
                const int u1 = min(u0 + jper, n - j0);
                for (int u = max(u0, i + 1 - j0); u < u1; ++u) {
                    const uint4 rj = rec[u];
                    count(rj, quotient(rj), u, rj.w & kHistSlow);
                }
            }
        }
        __syncthreads();
        unsigned long long *out = counts + (int64_t)blockIdx.y * 3 * nbins;
        for (int b = tid; b < 3 * nbins; b += kHistBlock) {
            if (hist[b]) atomicAdd(&out[b], (unsigned long long)hist[b]);
            hist[b] = 0u;
        }
    }
}

PairHistPlan pair_hist_plan(int64_t max_n, int R)
{
    PairHistPlan p;
    // particles j of a job: fewer where the largest system would not give every
    // compute unit a job
    p.jw = max_n >= 8192 ? 256 : (max_n >= 2048 ? 64 : 16);
    const int64_t T0 = (max_n + kHistTile - 1) / kHistTile, NC = (max_n + p.jw - 1) / p.jw;
    // one block per compute unit (each adds its histogram to the global one,
    // whose counters all blocks share); 1024 threads, so that one fills it
    const int64_t most = std::max(256 / R, 4);
    p.blocks = (int)std::max<int64_t>(1, std::min(T0 * NC, most));
    // a job adds at most kHistTile jw to one counter
    p.flush = (int)((((int64_t)1 << 32) - 1) / ((int64_t)kHistTile * p.jw));
    return p;
}

hipError_t launch_pair_hist(const LaunchCfg &c, const Workspace &w, const void *pos, const void *q, double r_max,
                            int nbins, int64_t *counts)
{
    const size_t sm = sizeof(unsigned int) * 3 * (size_t)nbins;
    const PairHistPlan p = pair_hist_plan(c.max_n, c.R);
    const dim3 g((unsigned)p.blocks, c.R);
    auto out = reinterpret_cast<unsigned long long *>(counts);
    if (c.prec == RBE_FP64)
        launch_k(k_pair_hist<double>, g, kHistBlock, sm, c.stream, w.sys, (const double *)pos, (const double *)q, c.ntot,
                 r_max, nbins, p.jw, p.flush, out);
    else
        launch_k(k_pair_hist<float>, g, kHistBlock, sm, c.stream, w.sys, (const float *)pos, (const float *)q, c.ntot,
                 r_max, nbins, p.jw, p.flush, out);
    return hipGetLastError();
}

}  // namespace rbe

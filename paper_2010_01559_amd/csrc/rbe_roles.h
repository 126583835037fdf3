// Device roles of the launch that follows the staging launch (k_mid):
// structure-factor totals and per-mode force constants, the next step's
// modes, and the gated neighbour-list rebuild (binning, cell scan, scatter
// into cell order).  Loops that depend on the block size take their shape
// from blockDim.
#pragma once

#include <hip/hip_runtime.h>

#include <stdint.h>

#include <type_traits>

#include "rbe_device.h"
#include "rbe_internal.h"

namespace rbe {

// What the force constants of one mode take besides its structure factor:
// the mode, its weight and the system's constants, and its index o in the
// mode arrays.  The totals load these before the partial sums, so that their
// latency overlaps the sums.
struct KModeIn {
    double mx, my, mz, w, coulomb, L;
    int o, polar;
};

__device__ __forceinline__ KModeIn kmode_in(const SysDev &S, int moff, int l, const int32_t *modes,
                                            const double *mode_w, int mcap)
{
    KModeIn in;
    in.o = moff + l;
    in.mx = modes[in.o];
    in.my = modes[mcap + in.o];
    in.mz = modes[2 * mcap + in.o];
    in.w = mode_w[in.o];
    in.coulomb = S.coulomb;
    in.L = S.L;
    in.polar = S.polar;
    return in;
}

// Polar form of the structure factor c + i s: modulus A and phase
// t = u - v in revolutions (see KModeF), the phase within 1e-8.  It is straight-line code
// on the totals launch's critical path, where fetching instructions is what costs,
// so it is short: the phase is an eighth of a turn's multiple and an odd
// polynomial of degree 11 (Chebyshev fit of atan(z) / (2 pi z) in z^2,
// |z| <= tan(pi/8)).  The library's hypot and atan2 took 0.9 us more (launch
// of 100 modes at N = 3000).
__device__ __forceinline__ void polar(double c, double s, double &A, float &u, float &v)
{
    const double x = fabs(c), y = fabs(s), hi = fmax(x, y), lo = fmin(x, y);
    const double d2 = fma(hi, hi, lo * lo);
    const double r = __builtin_amdgcn_rsq(d2), a = d2 * r;
    const bool red = lo > 0.41421356237309503 * hi;
    float z = (float)((red ? lo - hi : lo) * __builtin_amdgcn_rcp(red ? lo + hi : hi));
    A = fma(fma(-a, a, d2), 0.5 * r, a);
    if (d2 == 0.0) {
        A = 0.0;
        z = 0.0f;
    }
    const float w = z * z;
    float p = fmaf(w, -0.00960183144f, 0.0168270133f);
    p = fmaf(w, p, -0.0226636175f);
    p = fmaf(w, p, 0.031828139f);
    p = fmaf(w, p, -0.0530516058f);
    p = fmaf(w, p, 0.159154937f);
    // t = e + k
    float e = p * z, k = red ? 0.125f : 0.0f;
    if (y > x) {
        e = -e;
        k = 0.25f - k;
    }
    if (c < 0.0) {
        e = -e;
        k = 0.5f - k;
    }
    if (s < 0.0) {
        e = -e;
        k = -k;
    }
    const float eh = rintf(e * 16777216.0f) * (1.0f / 16777216.0f);
    u = __builtin_amdgcn_fractf(k + eh);
    v = eh - e;
}

// Force coefficient of mode m without its factor m:
//   a_l = coulomb w_l 2 m_l / (L^2 |m_l|^2)   (eq. 3.6 with k = 2 pi m / L).
__device__ __forceinline__ double force_coefficient(const KModeIn &in)
{
    const double m2 = in.mx * in.mx + in.my * in.my + in.mz * in.mz;
    return in.coulomb * in.w * 2.0 / (in.L * in.L * m2);
}

// Force constants of mode in.o with structure factor c + i s, f its
// force_coefficient().
template <typename KM>
__device__ __forceinline__ KM kmode_of(const KModeIn &in, double f, double c, double s)
{
    const double mx = in.mx, my = in.my, mz = in.mz;
    KM k;
    if constexpr (sizeof(KM) == sizeof(KModeF)) {
        k.u = c;
        k.v = s;
        if (in.polar) {
            double A;
            polar(c, s, A, k.u, k.v);
            f *= -A;
        }
    } else {
        k.C = c;
        k.S = s;
    }
    k.m[0] = mx;
    k.m[1] = my;
    k.m[2] = mz;
    k.a[0] = f * mx;
    k.a[1] = f * my;
    k.a[2] = f * mz;
    return k;
}

// Structure factor totals and force constants of mode in.o, stored.
template <typename KM>
__device__ __forceinline__ void make_kmode(const KModeIn &in, double f, double c, double s, double *rho, KM *km)
{
    rho[2 * in.o] = c;
    rho[2 * in.o + 1] = s;
    km[in.o] = kmode_of<KM>(in, f, c, s);
}

// Gated list rebuild: binning blocks, then scan blocks, then scatter
// blocks, ordered by bounded device flags.
struct RebuildArgs {
    const SysDev *sys;
    int R;
    int32_t *ready;
    int32_t *count;
    int32_t *start;
    const Tile *part_tiles;
    int n_part_tiles;
    const int32_t *cellid;
    const int32_t *rank;
    const void *packed;     // records, or NULL: formed from the positions
    const void *pos, *q;
    int64_t ntot;
    int32_t *sorted_idx;
    void *sorted;
    int32_t *slot_of;
    void *ref;
    int32_t *overflow;
    int32_t *builds;
    int32_t *flag;
    int32_t *bins_done;     // binning blocks finished (reset by the staging launch)
    int n_bin;              // binning blocks of the launch
    int n_scan;             // scan blocks
    int32_t *poison;        // raised when a wait gives up, cleared by a complete scan
    int wait_limit;         // spin bound of every wait
    const double *diam;     // per-particle diameters, moved along when set
    double *dsorted;
};

// Record of particle i, as the staging launch forms it.
__device__ __forceinline__ void rebuild_record(const RebuildArgs &a, const SysDev &S, int64_t i, PackF &v)
{
    if (a.packed) {
        v = reinterpret_cast<const PackF *>(a.packed)[i];
        return;
    }
    const float *x = reinterpret_cast<const float *>(a.pos) + i;
    v = PackF{to_fix(frac01((double)x[0] * S.invL)), to_fix(frac01((double)x[a.ntot] * S.invL)),
              to_fix(frac01((double)x[2 * a.ntot] * S.invL)), reinterpret_cast<const float *>(a.q)[i]};
}

__device__ __forceinline__ void rebuild_record(const RebuildArgs &a, const SysDev &S, int64_t i, PartD &v)
{
    if (a.packed) {
        v = reinterpret_cast<const PartD *>(a.packed)[i];
        return;
    }
    const double *x = reinterpret_cast<const double *>(a.pos) + i;
    v = PartD{frac01(x[0] * S.invL), frac01(x[a.ntot] * S.invL), frac01(x[2 * a.ntot] * S.invL),
              reinterpret_cast<const double *>(a.q)[i]};
}

template <typename KM>
struct MidArgs {
    const SysDev *sys;
    int R, max_p;
    int n_final_blocks;   // blocks doing the structure-factor totals
    int single_p;         // single-system context: its mode count (else 0) ...
    int single_nt;        // ... and its structure-factor tile count
    int final_lw;         // log2 of the waves per mode of the totals (0 or 2)
    const double *partial;
    const int32_t *part_off;   // [2R]: partial offsets, then tile counts
    const int32_t *modes;
    const double *mode_w;
    int mcap;
    double *rho;
    KM *km;
    int32_t *count;
    int32_t *start;
    int do_scan;
    const int32_t *scan_gate;   // when set, the scan runs only if *scan_gate != 0
    // binning of a list rebuild (blocks after the totals), only if *bin_gate != 0
    const int32_t *bin_gate;
    int n_bin_blocks;
    const Tile *part_tiles;
    int n_part_tiles;
    int32_t *cellid;
    int32_t *rank;
    // the next step's modes (one block per system), and a flag to clear
    int n_sample_blocks;
    uint64_t sample_step;
    const double *cdf;
    int table_lds;
    int32_t *modes_next;
    double *mode_w_next;
    int32_t *clear_flag;
    const uint64_t *step_base;   // added to sample_step when set
    // list rebuild (gated by bin_gate): rb.n_scan scan blocks and n_reb_scatter
    // scatter blocks after all the others
    int reb;
    int n_reb_scatter;
    RebuildArgs rb;
};

// Up to 128 blocks, each striding over the 256-particle tiles: on the many
// steps where nothing is binned the launch costs only their dispatch.  A thread
// takes up to kRebBatch tiles at once: it loads all their records, then
// issues all the counter atomics, then stores the cell ids and ranks, so
// that the memory latencies of its particles overlap instead of adding up.
constexpr int kRebBatch = 4;

template <typename KM>
__device__ void mid_bin(const MidArgs<KM> &a, int b)
{
    const int k = threadIdx.x & 255;
    const int tpb = (int)(blockDim.x >> 8);   // 256-particle tiles per block and round
    const int stride = tpb * a.n_bin_blocks;
    for (int t0 = tpb * b + (int)(threadIdx.x >> 8); t0 < a.n_part_tiles; t0 += kRebBatch * stride) {
        int64_t idx[kRebBatch];
        int cell[kRebBatch];
#pragma unroll
        for (int u = 0; u < kRebBatch; ++u) {
            idx[u] = -1;
            cell[u] = 0;
            const int ti = t0 + u * stride;
            if (ti >= a.n_part_tiles) continue;
            const Tile t = a.part_tiles[ti];
            if (k >= t.count) continue;
            const SysDev &S = a.sys[t.sys];
            const int64_t i = S.off + t.start + k;
            int cx, cy, cz;
            if constexpr (sizeof(KM) == sizeof(KModeF)) {
                PackF v;
                rebuild_record(a.rb, S, i, v);
                cx = cell_of_fix(v.x, S.nc);
                cy = cell_of_fix(v.y, S.nc);
                cz = cell_of_fix(v.z, S.nc);
            } else {
                PartD v;
                rebuild_record(a.rb, S, i, v);
                cx = cell_of_frac(v.x, S.nc);
                cy = cell_of_frac(v.y, S.nc);
                cz = cell_of_frac(v.z, S.nc);
            }
            idx[u] = i;
            cell[u] = S.cell_off + (cz * S.nc + cy) * S.nc + cx;
        }
        int rk[kRebBatch];
#pragma unroll
        for (int u = 0; u < kRebBatch; ++u) rk[u] = idx[u] >= 0 ? atomicAdd(&a.count[cell[u]], 1) : 0;
#pragma unroll
        for (int u = 0; u < kRebBatch; ++u)
            if (idx[u] >= 0) {
                a.cellid[idx[u]] = cell[u];
                a.rank[idx[u]] = rk[u];
            }
    }
}


// Structure-factor totals, W = 2^final_lw waves per mode (1 or 4) and 16 / W
// modes per 1024-thread block: the wave of part q sums the tile partials of
// its mode in runs of 64 tiles q, q + W, q + 2W, ... (a lane its tile of
// each run, in order), the waves reduce across lanes, and the mode's first
// wave adds the W part sums in order and writes the force constants.  The
// partials of one mode sit a tile row apart (one cache line per tile), so
// four waves per mode quarter the chain of dependent load batches of a long
// tile list; a context whose systems all have at most 64 tiles takes one
// wave per mode and a quarter of the blocks.
int final_waves_log2(int max_tiles_per_system);

template <typename KM>
__device__ void mid_final(const MidArgs<KM> &a, int blk)
{
    __shared__ double2 q_sum[16];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    const int lw = a.final_lw, W = 1 << lw;
    const int gm = (blk << (4 - lw)) + (wave >> lw);
    const int q = wave & (W - 1);
    const int r = a.single_p ? (gm >= a.max_p ? a.R : 0) : gm / a.max_p, l = gm - r * a.max_p;
    // a single system's mode and tile counts come with the launch, so that
    // the partial loads do not wait for the system constants and offsets
    bool ok = r < a.R;
    int P = 0, nt = 0;
    const double *base = a.partial;
    if (ok) {
        P = a.single_p ? a.single_p : a.sys[r].p;
        ok = l < P;
        nt = a.single_p ? a.single_nt : a.part_off[a.R + r];
        base = a.partial + (a.single_p ? 0 : 2 * (int64_t)a.part_off[r]);
    }
    // the inputs of the force constants, loaded by the thread that forms them
    KModeIn in{};
    if (ok && q == 0 && lane == 0) {
        const SysDev &S = a.sys[r];
        in = kmode_in(S, a.single_p ? 0 : S.moff, l, a.modes, a.mode_w, a.mcap);
    }
    double c = 0.0, s = 0.0;
    if (ok) {
        // eight loads are issued before they are added, so their latencies overlap
        const int STRIDE = 64 * W;
        for (int t0 = 64 * q + lane; t0 < nt; t0 += 8 * STRIDE) {
            double2 v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int t = t0 + STRIDE * u;
                if (t < nt) v[u] = *reinterpret_cast<const double2 *>(base + 2 * ((int64_t)t * P + l));
            }
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (t0 + STRIDE * u < nt) {
                    c += v[u].x;
                    s += v[u].y;
                }
        }
        c = wave_sum(c);
        s = wave_sum(s);
    }
    // in every lane, without a branch: its divisions run under the sums
    const double f = force_coefficient(in);
    if (W > 1) {
        if (lane == 0) q_sum[wave] = make_double2(c, s);
        __syncthreads();
        c = s = 0.0;
        for (int k = 0; k < W; ++k) {
            c += q_sum[min(wave + k, 15)].x;
            s += q_sum[min(wave + k, 15)].y;
        }
    }
    if (ok && q == 0 && lane == 0) make_kmode<KM>(in, f, c, s, a.rho, a.km);
}

// Exclusive scan of one system's cell counts with NW waves (64 NW threads).
// Cells are processed in passes of NCH chunks x 256 NW; thread t owns cells
// [base + g*256 NW + 4t, +4) of chunk g.  Cell offsets are padded to
// multiples of 4 so the counts load as int4.  Fewer chunks per pass hold
// fewer registers.
constexpr int kScanChunks = 8;

template <int NW, int NCH = kScanChunks>
__device__ void mid_scan(const SysDev &S, int r, int32_t *count, int32_t *start)
{
    constexpr int CH = 256 * NW;              // cells per chunk
    constexpr int NT = NCH * NW;              // wave totals per pass (at most 128)
    static_assert(NT <= 128, "one wave prefixes the wave totals, two per lane");
    __shared__ int wtot[NT];
    __shared__ int gpre[NT + 1];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int32_t *cnt = count + S.cell_off;
    int32_t *st = start + S.cell_off + r;
    const int ncell = S.ncell;
    int carry = 0;
    for (int base = 0; base < ncell; base += NCH * CH) {
        int v[NCH][4];
        int s[NCH], incl[NCH];
#pragma unroll
        for (int g = 0; g < NCH; ++g) {
            const int idx = base + g * CH + 4 * tid;
            if (idx + 3 < ncell) {
                const int4 x = *reinterpret_cast<const int4 *>(cnt + idx);
                v[g][0] = x.x;
                v[g][1] = x.y;
                v[g][2] = x.z;
                v[g][3] = x.w;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j) v[g][j] = (idx + j < ncell) ? cnt[idx + j] : 0;
            }
            s[g] = v[g][0] + v[g][1] + v[g][2] + v[g][3];
        }
#pragma unroll
        for (int g = 0; g < NCH; ++g) {
            incl[g] = wave_incl_scan(s[g]);
            if (lane == 63) wtot[g * NW + wave] = incl[g];
        }
        __syncthreads();
        if (wave == 0) {
            // exclusive prefix of the NT wave totals in (chunk, wave) order
            const int x0 = 2 * lane < NT ? wtot[2 * lane] : 0;
            const int x1 = 2 * lane + 1 < NT ? wtot[2 * lane + 1] : 0;
            const int inc = wave_incl_scan(x0 + x1);
            if (2 * lane < NT) gpre[2 * lane] = inc - x0 - x1;
            if (2 * lane + 1 < NT) gpre[2 * lane + 1] = inc - x1;
            if (lane == 63) gpre[NT] = inc;
        }
        __syncthreads();
#pragma unroll
        for (int g = 0; g < NCH; ++g) {
            const int idx = base + g * CH + 4 * tid;
            const int run = S.off + carry + gpre[g * NW + wave] + incl[g] - s[g];
            const int o[4] = {run, run + v[g][0], run + v[g][0] + v[g][1], run + v[g][0] + v[g][1] + v[g][2]};
            if (idx + 3 < ncell) {
                // whole groups of four: 16-byte stores (the starts of system
                // r are shifted by r entries, so they are aligned when r % 4 == 0)
                *reinterpret_cast<int4 *>(cnt + idx) = make_int4(0, 0, 0, 0);
                if ((r & 3) == 0) {
                    *reinterpret_cast<int4 *>(st + idx) = make_int4(o[0], o[1], o[2], o[3]);
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) st[idx + j] = o[j];
                }
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (idx + j < ncell) {
                        st[idx + j] = o[j];
                        cnt[idx + j] = 0;
                    }
            }
        }
        carry += gpre[NT];
        __syncthreads();
    }
    if (tid == 0) st[ncell] = S.off + carry;
}

// ---------------------------------------------------------------------------
// List rebuild inside the totals launch (work only when the step's rebuild
// flag is set).  The binning blocks count their particles into the cells and
// then each adds one to bins_done; the scan blocks, which come after them in
// block order, wait for all of them, scan their systems' counts and each add one to
// `ready`; the scatter blocks, last in block order, wait for that and stride
// over the 256-particle tiles, moving records into cell order.  A block only
// waits for blocks of lower index, which are dispatched before it and do not
// wait for it, so every wait ends (with one block per compute unit the last
// scatter blocks of a large launch start when earlier blocks finish); the
// waits are bounded anyway.  A wait that reaches its bound gives up: it
// raises the timeout bit of the error word and the poison flag, and its
// block skips its work.  The
// force launch of that step then clears the cell counts (the scan that would
// have cleared them did not run) and the next step's staging launch asks for
// a rebuild; the cell pass of the failed step reads the previous cell starts,
// clamped to the system, so every access stays in bounds.  The staging
// launch of each step resets bins_done and ready.
// ---------------------------------------------------------------------------

// Thread 0 waits (at most `limit` polls) until *p reaches want; the block
// learns the outcome.  The polls are relaxed loads and one acquire follows
// the last: on gfx950 an agent-scope acquire invalidates the XCD's L2, so
// acquiring on every poll would keep evicting the data that the blocks still
// working on that XCD read.  The block's waves share thread 0's compute unit
// and L1, and the barrier orders their loads after its invalidation.
__device__ bool block_wait(int32_t *p, int want, int limit, int32_t *flag, int32_t *poison)
{
    __shared__ int s_ok;
    if (threadIdx.x == 0) {
        int ok = 0;
        for (int it = 0; it < limit; ++it) {
            if (__hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) >= want) {
                ok = 1;
                break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
        if (ok) {
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            __builtin_amdgcn_s_waitcnt(0);   // the invalidation is done before the barrier
        } else {
            atomicOr(flag, kFlagTimeout);
            atomicOr(poison, 1);
        }
        s_ok = ok;
    }
    __syncthreads();
    return s_ok != 0;
}

// Publishing a block's stores to the other blocks of the launch: every wave
// waits until its stores have reached the L2 (a workgroup barrier alone does
// not wait for them), then thread 0 alone writes the XCD's L2 back (an
// agent-scope release fence, which writes back every dirty line of that L2;
// issued by every wave, these write-backs took 15-30 us per hand-off).
// Thread 0 then raises the block's flag.
__device__ __forceinline__ void block_stores_done()
{
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __builtin_amdgcn_s_waitcnt(0);
    __atomic_signal_fence(__ATOMIC_SEQ_CST);
    __syncthreads();
    if (threadIdx.x == 0) {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
        __builtin_amdgcn_s_waitcnt(0);   // the write-back has completed before the flag
    }
}

// Scan block b of n_scan of a rebuild: waits for every binning block and turns the
// cell counts of its systems (every n_scan-th) into slot starts; the scatter
// blocks wait for all scan blocks.  The last one clears the overflow flag, counts the
// build and lowers the poison flag.  With one block scanning every system in
// turn the totals launch of a rebuild step of 64 replicas took 428 us, 84 us now.
template <int NW, int NCH = kScanChunks>
__device__ void rebuild_scan(const RebuildArgs &a, int b)
{
    if (!block_wait(a.bins_done, a.n_bin, a.wait_limit, a.flag, a.poison)) return;
    for (int r = b; r < a.R; r += a.n_scan) mid_scan<NW, NCH>(a.sys[r], r, a.count, a.start);
    block_stores_done();
    if (threadIdx.x == 0 &&
        __hip_atomic_fetch_add(a.ready, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == a.n_scan - 1) {
        *a.overflow = 0;
        *a.builds += 1;
        *a.poison = 0;
    }
}

// Scatter block b of nb: moves records into cell order once the scan is out,
// and records each particle's slot and list reference record.  As in the
// binning, a thread loads everything for up to kScatBatch tiles before it
// stores (fewer than there: each holds a whole record).
constexpr int kScatBatch = 4;

template <typename Rec>
__device__ void rebuild_scatter(const RebuildArgs &a, int b, int nb)
{
    if (!block_wait(a.ready, a.n_scan, a.wait_limit, a.flag, a.poison)) return;
    const int k = threadIdx.x & 255;
    const int tpb = (int)(blockDim.x >> 8);
    const int stride = tpb * nb;
    // records move as 16-byte words (PackF: one, PartD: two)
    constexpr int W = (int)(sizeof(Rec) / sizeof(uint4));
    for (int t0 = tpb * b + (int)(threadIdx.x >> 8); t0 < a.n_part_tiles; t0 += kScatBatch * stride) {
        int idx[kScatBatch], cell[kScatBatch], rk[kScatBatch], sys[kScatBatch];
        uint4 v[kScatBatch][W];
#pragma unroll
        for (int u = 0; u < kScatBatch; ++u) {
            idx[u] = -1;
            sys[u] = 0;
            cell[u] = 0;
            rk[u] = 0;
#pragma unroll
            for (int q = 0; q < W; ++q) v[u][q] = make_uint4(0, 0, 0, 0);
            const int ti = t0 + u * stride;
            if (ti < a.n_part_tiles) {
                const Tile t = a.part_tiles[ti];
                if (k < t.count) {
                    const int i = a.sys[t.sys].off + t.start + k;
                    idx[u] = i;
                    sys[u] = t.sys;
                    cell[u] = a.cellid[i];
                    rk[u] = a.rank[i];
                    Rec p;
                    rebuild_record(a, a.sys[t.sys], i, p);
                    __builtin_memcpy(v[u], &p, sizeof p);
                }
            }
        }
        int slot[kScatBatch];
#pragma unroll
        for (int u = 0; u < kScatBatch; ++u) slot[u] = idx[u] >= 0 ? a.start[cell[u] + sys[u]] + rk[u] : 0;
#pragma unroll
        for (int u = 0; u < kScatBatch; ++u)
            if (idx[u] >= 0) {
                // a slot outside the system can only come from stale counts
                const SysDev &S = a.sys[sys[u]];
                if (slot[u] < S.off || slot[u] >= S.off + S.n) {
                    atomicOr(a.flag, kFlagBounds);
                    continue;
                }
                a.sorted_idx[slot[u]] = idx[u];
                a.slot_of[idx[u]] = slot[u];
                if (a.diam) a.dsorted[slot[u]] = a.diam[idx[u]];
#pragma unroll
                for (int q = 0; q < W; ++q) {
                    reinterpret_cast<uint4 *>(a.sorted)[(int64_t)slot[u] * W + q] = v[u][q];
                    reinterpret_cast<uint4 *>(a.ref)[(int64_t)idx[u] * W + q] = v[u][q];
                }
            }
    }
}


// Wave tiles of the cell pass of a force, energy or adjoint call, written from
// the cell starts by the launch that scatters the particles into cell order:
// runs of at most ppw = 2^lg slots of one row of cells, so that a wave has one
// set of candidates (a run across two rows has two, and with every wave of a
// launch resident at once the launch lasted twice the average wave).  Row
// `row` of a system takes the entries from base = floor(a0 / ppw) + row, a0
// its first slot: one or two more than it needs at most, left empty, which
// spares a prefix sum over the rows.
struct RowTileArgs {
    const SysDev *sys;
    const Tile *rows;
    const int32_t *start;
    Tile *out;
    int n;    // row tiles
    int lg;   // log2 of the particles per wave tile
};

__device__ __forceinline__ void write_row_tiles(const RowTileArgs &a, int b)
{
    const Tile t = a.rows[b];
    if ((int)threadIdx.x >= t.count) return;
    const SysDev &S = a.sys[t.sys];
    const int row = t.start + threadIdx.x;
    const int32_t *st = a.start + S.cell_off + t.sys + row * S.nc;
    const int a0 = min(max(st[0] - S.off, 0), S.n), a1 = min(max(st[S.nc] - S.off, a0), S.n);
    const int base = S.ctile_off + (a0 >> a.lg) + row, end = S.ctile_off + (a1 >> a.lg) + row + 1;
    for (int e = base, s = a0; e < end; ++e, s += 1 << a.lg)
        a.out[e] = Tile{t.sys, min(s, a1), max(min(1 << a.lg, a1 - s), 0), 0};
}

inline RowTileArgs row_tile_args(const LaunchCfg &c, const Workspace &w)
{
    return RowTileArgs{w.sys, w.row_tiles, w.cell_start, w.cell_tiles, c.n_row_tiles, c.cell_ppw == 16 ? 4 : 3};
}

// Next step's modes of system b (exact sampler), drawn by one block; the
// cumulative table is read from tab when given (the caller has room for it in
// LDS), else from global memory.
template <typename KM>
__device__ void mid_sample(const MidArgs<KM> &a, int b, double *tab)
{
    const SysDev S = a.sys[b];
    const double *t = a.cdf + S.cdf_off;
    if (tab) {
        for (int k = threadIdx.x; k < 2 * S.M + 1; k += blockDim.x) tab[k] = t[k];
        __syncthreads();
        t = tab;
    }
    for (int l = threadIdx.x; l < S.p; l += blockDim.x) {
        int mx, my, mz;
        sample_mode(t, S.M, (uint32_t)l, S.seed, a.sample_step + (a.step_base ? *a.step_base : 0), mx, my, mz);
        const int o = S.moff + l;
        a.modes_next[o] = mx;
        a.modes_next[a.mcap + o] = my;
        a.modes_next[2 * a.mcap + o] = mz;
        a.mode_w_next[o] = S.S / (double)S.p;
    }
}

// Arguments of the totals and of the draw of the next step's modes.
template <typename KM>
inline void totals_args(MidArgs<KM> &a, const LaunchCfg &c, const Workspace &w, int sample_next, uint64_t sample_step,
                        const ListStep *ls)
{
    a.sys = w.sys;
    a.R = c.R;
    a.max_p = c.max_p;
    a.single_p = c.R == 1 ? c.max_p : 0;
    a.single_nt = c.n_rho_tiles;
    a.partial = w.partial;
    a.part_off = w.partial_off;
    a.modes = w.modes;
    a.mode_w = w.mode_w;
    a.mcap = c.mcap;
    a.rho = w.rho;
    a.km = (KM *)w.kmode;
    a.n_sample_blocks = sample_next ? c.R : 0;
    a.sample_step = sample_step;
    a.cdf = w.cdf;
    a.table_lds = sample_next && c.max_table <= 6144 ? 1 : 0;
    a.modes_next = w.modes_alt;
    a.mode_w_next = w.mode_w_alt;
    a.step_base = ls ? ls->step_base : nullptr;
}

}  // namespace rbe

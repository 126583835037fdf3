// rbe_real.hip -- real-space kernels of librbe (gfx950).
//
// Paper: Jin, Li, Xu & Zhao, arXiv:2010.01559: the truncated erfc sum of
// eq. (2.9) and the second term of eq. (2.11); the shifted Lennard-Jones
// repulsion of eq. (4.1), with r_off = 0 or, from per-particle diameters,
// r_off = (d_i + d_j)/2 - sigma (Sec. 4.2).  The paper leaves the neighbour
// search open; here it is a cell list with cells of side >= 1/nh of the search
// radius (the largest cutoff, + skin; nh = 1 to 3 by the particles within it), rebuilt
// for every stand-alone evaluation, and inside
// rbe_step a Verlet list of the pairs within cutoff + skin, rebuilt on the
// device whenever some particle has moved more than skin/2 since the last
// build (the rebuild step evaluates the forces on the cell list and writes
// the list in the same pass).
//
// Pair force on particle i: phi(r) d with d = r_j - r_i (minimum image),
//   phi = -coulomb q_i q_j (erfc(beta r)/r + 2 beta exp(-alpha r^2)/sqrt(pi)) / r^2
//         + 4 eps (6 (sigma/r)^6 - 12 (sigma/r)^12) / r^2        (r < R_c)
// with beta = sqrt(alpha); the Coulomb part acts for r <= r_c.
//
// Work decomposition of the cell pass (cell_pairs): a wave takes sixteen
// cell-sorted particles (eight in small systems); the cells around them are
// (2 nh + 1)^2 = 9, 25 or 49 rows of consecutive cells, contiguous ranges of the
// cell-sorted array (two where a row wraps in x, so up to 98).  The squared
// distances of the particles to their candidates come from the
// matrix cores (a conservative test in single precision); the partners that
// pass are listed in LDS and evaluated by four lanes per particle (eight) from the
// exact records, so the pair terms do not diverge on the distance test.  Calls of
// sparse systems test their few candidates one by one (sparse_body).  Each
// lane accumulates its FP32 pair terms exactly (on a fixed grid, see qterm),
// so the result does not depend on the order of the particles inside a cell
// (which comes from atomic counters) nor on the path (cell or list pass).
// Systems with fewer than three cells per side use all-pairs tiles, one
// particle per wave (allpairs_body).
//
// List pass: LPP lanes per particle walk its list in strides of LPP; the
// LPP partial sums are combined by a fixed butterfly.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <type_traits>

#include "rbe_device.h"
#include "rbe_internal.h"
#include "rbe_roles.h"

namespace rbe {

constexpr int RL_BS = 256;                  // threads per block: 4 waves
constexpr int RL_PPB = 64;                  // particles per cell-pass tile of a step (16 per wave)
constexpr int RL_ALLPAIRS = 4;              // particles per all-pairs tile: one per wave

int real_rows_per_tile() { return RL_PPB; }
int real_allpairs_per_tile() { return RL_ALLPAIRS; }

template <typename T>
struct RBT;
template <>
struct RBT<float> {
    using Rec = PackF;
};
template <>
struct RBT<double> {
    using Rec = PartD;
};

struct PairE {
    double e_real, e_lj;
};

// Single-precision pair terms are added on a fixed grid of 2^-32 (as integers
// held in double): every partial sum is exact, so a particle's real-space
// force does not depend on the order in which its partners are visited (cell
// ranks come from atomic counters; list and cell passes order partners
// differently).  This holds while partial sums stay below 2^21 in magnitude
// (an LJ wall at r = 0.45 sigma, far inside anything these systems reach);
// the grid is far below single-precision rounding of the forces.
// A pair's force component phi * d on that grid.  In single precision the
// scale is applied to phi first (a power of two, so (phi 2^32) d rounds to
// the same float as (phi d) 2^32), and the rounding to an integer is done in
// single precision, where it is exact: the same values as
// rint((double)(phi d) * 2^32) with fewer double-precision instructions.
__device__ __forceinline__ float qphi(float phi) { return phi * 0x1p32f; }

// Flags a single-precision partial sum (in units of 2^-32) that has reached
// 2^52, half the range in which the grid sums are exact (checked at the end
// of each lane's sum and after the lanes of a particle are combined): only
// particles pressed far into each other's LJ wall get there (a force of
// 2^20), and then the forces are reported as unusable instead of silently
// losing exactness.
__device__ __forceinline__ void range_check(double x, double y, double z, int32_t *flag)
{
    if (fmax(fabs(x), fmax(fabs(y), fabs(z))) >= 0x1p52) atomicOr(flag, kFlagRange);
}
__device__ __forceinline__ double qphi(double phi) { return phi; }
__device__ __forceinline__ double qterm(float scaled) { return (double)rintf(scaled); }
__device__ __forceinline__ double qterm(double v) { return v; }
template <typename T>
__device__ __forceinline__ double qscale()
{
    return sizeof(T) == 4 ? 0x1p-32 : 1.0;
}

// erfc(x) exp(x^2) = t * sum_k c_k t^k with t = 1/(1 + 0.47047 x), x >= 0: the
// form of Abramowitz & Stegun 7.1.26 refitted to degree 9 for a relative
// error of erfc below 4e-7 in single precision on [0, 8] (fit_erfc.py).
__device__ __forceinline__ float erfc_scaled_f32(float x)
{
    const float t = __builtin_amdgcn_rcpf(fmaf(0.47047f, x, 1.0f));
    float s = -4.859511559e-02f;
    s = fmaf(s, t, 2.750724646e-01f);
    s = fmaf(s, t, -5.785352996e-01f);
    s = fmaf(s, t, 4.823851487e-01f);
    s = fmaf(s, t, -1.365632976e-01f);
    s = fmaf(s, t, 2.525006764e-01f);
    s = fmaf(s, t, 2.213245585e-01f);
    s = fmaf(s, t, 2.670528048e-01f);
    s = fmaf(s, t, 2.653580831e-01f);
    return s * t;
}

// phi(r) of one pair in single precision (r2 = |d|^2 in box units); both
// terms are evaluated and selected, so a wave does not branch on the
// per-lane cutoff tests.  With ENERGY, half the pair energies are added to e.
template <bool ENERGY>
__device__ __forceinline__ float pair_phi(const PairConstF &c, float qi, float qj, float r2, PairE &e)
{
    const float rinv = __builtin_amdgcn_rsqf(r2);
    const float rinv2 = rinv * rinv;
    const bool in_c = r2 <= c.rc2;
    const bool in_lj = c.lj_on && r2 < c.lj_rc2;
    const float r = r2 * rinv;
    const float ex = __builtin_amdgcn_exp2f(c.nalpha_log2e * r2);   // exp(-alpha r^2)
    const float ec = erfc_scaled_f32(c.beta * r) * ex;               // erfc(beta r)
    const float g = fmaf(ec, rinv, c.two_beta_rsqrtpi * ex) * rinv2;
    const float cq = c.coulomb * qi * qj;
    const float sr2 = c.lj_sig2 * rinv2;
    const float sr6 = sr2 * sr2 * sr2;
    const float plj = c.eps4 * fmaf(-12.0f, sr6, 6.0f) * sr6 * rinv2;
    if constexpr (ENERGY) {
        if (in_c) e.e_real += 0.5 * (double)(cq * ec * rinv);
        if (in_lj) e.e_lj += 0.5 * ((double)c.eps4 * ((double)sr6 * sr6 - sr6) + c.lj_shift);
    }
    return (in_c ? -cq * g : 0.0f) + (in_lj ? plj : 0.0f);
}

// The same in double precision (libm erfc/exp).
template <bool ENERGY>
__device__ __forceinline__ double pair_phi(const SysDev &S, double qi, double qj, double r2, PairE &e)
{
    double phi = 0.0;
    if (r2 <= S.rc2) {
        const double r = sqrt(r2);
        const double ec = erfc(S.beta * r);
        const double ex = exp(-S.alpha * r2);
        const double g = (ec / r + 2.0 / 1.7724538509055160273 * S.beta * ex) / r2;
        const double cq = S.coulomb * qi * qj;
        phi = -cq * g;
        if constexpr (ENERGY) e.e_real += 0.5 * cq * ec / r;
    }
    if (S.lj_on && !S.diam_on && r2 < S.lj_rc2) {
        const double sr2 = S.lj_sig2 / r2;
        const double sr6 = sr2 * sr2 * sr2;
        phi += 4.0 * S.lj_eps * (6.0 * sr6 - 12.0 * sr6 * sr6) / r2;
        if constexpr (ENERGY) e.e_lj += 0.5 * (4.0 * S.lj_eps * (sr6 * sr6 - sr6) + S.lj_shift);
    }
    return phi;
}

// Shifted LJ of eq. (4.1) with r_off = (d_i + d_j)/2 - sigma from the two
// diameters, in double: s = r - r_off is a small difference of two
// distances that can be fifty times larger (a colloid against an ion), so r
// comes from the exact displacement and s is formed in double.  Returns
// dV/dr / r (the coefficient of d in the force on i) and adds half the pair
// energy when ENERGY.
template <bool ENERGY>
__device__ __forceinline__ double lj_offset(const SysDev &S, double di, double dj, double r2, PairE &e)
{
    const double r = sqrt(r2);
    const double sv = r - (0.5 * (di + dj) - S.lj_sig);
    if (!(sv < S.lj_rc)) return 0.0;
    const double sr2 = S.lj_sig2 / (sv * sv);
    const double sr6 = sr2 * sr2 * sr2;
    if constexpr (ENERGY) e.e_lj += 0.5 * (4.0 * S.lj_eps * (sr6 * sr6 - sr6) + S.lj_shift);
    return 4.0 * S.lj_eps * (6.0 * sr6 - 12.0 * sr6 * sr6) / (sv * r);
}

// Whether r^2 is beyond the reach of lj_offset, whose double-precision root and
// difference then need not be formed: the reach is R_c around r_off, so of a list of
// r_c = 40 hardly a pair is inside (with the diameters loaded in cell order beside
// the records instead of after the indices: step at N = 3101 21.5 -> 20.1 us).  The
// margin is far above the rounding of a single-precision r^2.
template <typename T>
__device__ __forceinline__ bool lj_far(const SysDev &S, double di, double dj, T r2)
{
    const T b = (T)(0.5 * (di + dj) + (S.lj_rc - S.lj_sig));
    return b < (T)0 || r2 > b * b * (T)1.00001;
}

// |d|^2 of two records in double: exact wrapped integer differences for
// PackF, the wrapped double difference for PartD.
__device__ __forceinline__ double r2_double(const PackF &a, const PackF &b, double L)
{
    const double u = L * (1.0 / 4294967296.0);
    const double dx = (double)(int32_t)(b.x - a.x) * u, dy = (double)(int32_t)(b.y - a.y) * u,
                 dz = (double)(int32_t)(b.z - a.z) * u;
    return dx * dx + dy * dy + dz * dz;
}

__device__ __forceinline__ double r2_double(const PartD &a, const PartD &b, double L)
{
    double sx = b.x - a.x, sy = b.y - a.y, sz = b.z - a.z;
    sx = (sx - rint(sx)) * L;
    sy = (sy - rint(sy)) * L;
    sz = (sz - rint(sz)) * L;
    return sx * sx + sy * sy + sz * sz;
}

// Displacement between two records.  rmax2 is the largest cutoff squared in
// the record's own units (fixed-point units for PackF).
struct Geo {
    float scale;     // PackF: box length of one fixed-point unit
    float rmax2u;    // PackF: search radius^2 in fixed-point units
    double rmax2;    // PartD: search radius^2
    double L;
};

template <typename T>
__device__ __forceinline__ Geo make_geo(const SysDev &S)
{
    return Geo{S.pair.scale, S.pair.rmax2u, S.rsearch2, S.L};
}

__device__ __forceinline__ bool near_test(const PackF &pa, const PackF &pb, const Geo &g)
{
    const float ux = (float)(int32_t)(pb.x - pa.x);
    const float uy = (float)(int32_t)(pb.y - pa.y);
    const float uz = (float)(int32_t)(pb.z - pa.z);
    return fmaf(ux, ux, fmaf(uy, uy, uz * uz)) <= g.rmax2u;
}

__device__ __forceinline__ void displacement(const PackF &pa, const PackF &pb, const Geo &g, float &dx, float &dy,
                                             float &dz, float &r2)
{
    dx = (float)(int32_t)(pb.x - pa.x) * g.scale;
    dy = (float)(int32_t)(pb.y - pa.y) * g.scale;
    dz = (float)(int32_t)(pb.z - pa.z) * g.scale;
    r2 = fmaf(dx, dx, fmaf(dy, dy, dz * dz));
}

__device__ __forceinline__ void displacement(const PartD &pa, const PartD &pb, const Geo &g, double &dx, double &dy,
                                             double &dz, double &r2)
{
    double sx = pb.x - pa.x, sy = pb.y - pa.y, sz = pb.z - pa.z;
    sx -= rint(sx);
    sy -= rint(sy);
    sz -= rint(sz);
    dx = sx * g.L;
    dy = sy * g.L;
    dz = sz * g.L;
    r2 = dx * dx + dy * dy + dz * dz;
}

__device__ __forceinline__ bool near_test(const PartD &pa, const PartD &pb, const Geo &g)
{
    double dx, dy, dz, r2;
    displacement(pa, pb, g, dx, dy, dz, r2);
    return r2 <= g.rmax2;
}

template <typename T>
__device__ __forceinline__ void cell_coords(const PackF &p, int nc, int &cx, int &cy, int &cz)
{
    cx = cell_of_fix(p.x, nc);
    cy = cell_of_fix(p.y, nc);
    cz = cell_of_fix(p.z, nc);
}

template <typename T>
__device__ __forceinline__ void cell_coords(const PartD &p, int nc, int &cx, int &cy, int &cz)
{
    cx = cell_of_frac(p.x, nc);
    cy = cell_of_frac(p.y, nc);
    cz = cell_of_frac(p.z, nc);
}

template <typename T>
struct RealArgs {
    const SysDev *sys;
    const Tile *tiles;       // steps: block tiles (aux = 0: RL_PPB sorted slots; 1: all pairs); calls: wave tiles
                             // (k_real_sparse: of kSparsePPW slots, in any cells)
    const Tile *wave_tiles;
    int single;              // single-system context
    const int32_t *start;
    const int32_t *sorted_idx;
    const void *sorted;
    const void *packed;      // original order (all-pairs tiles)
    const T *q;              // energies: charges in original order
    int64_t ntot;
    T *F;
    int accumulate;
    T *vel;                  // kick target (may be NULL); velocities for kinetic energy when ENERGY
    int32_t *flag;
    double *epart;           // ENERGY: [wave tiles][8]
    const void *km;          // per-mode force constants (KModeF / KModeD) for the fused Fourier force
    uint64_t kick_step;      // index of the step whose closing half kick is applied (its time step)
    const double *diam;      // per-particle diameters (original order) when some system has them
    const double *dsorted;   // the same in cell order (list steps)
};

// Neighbour-list state seen by the real-space pass of a step.
struct ListArgs {
    ListStep ls;
    int32_t *count;          // cell counts, cleared here after a rebuild gave up
    int ncell_tot;
    const Tile *list_tiles;
    int n_rows, n_list;      // tiles of the cell pass and of the list pass
    int32_t *nbr;            // [kmax][Ntot] partner slots, column k of slot s at k * Ntot + s
    int32_t *nnb;
    int kmax;
    int single_n, single_p;  // single-system context (SINGLE launches): its particle and mode counts
};

// Store (or add) the real-space force of particle i and apply the optional
// half kick; with ENERGY add the one-body sums to ev instead.
template <typename T, bool ENERGY>
__device__ __forceinline__ void finish_particle(const RealArgs<T> &a, const SysDev &S, int64_t i, double fxd,
                                                double fyd, double fzd, double *ev)
{
    if constexpr (ENERGY) {
        if (a.vel) {
            const double x = a.vel[i], y = a.vel[a.ntot + i], z = a.vel[2 * a.ntot + i];
            ev[3] += 0.5 * S.mass * (x * x + y * y + z * z);
        }
        const double qq = (double)a.q[i];
        ev[4] += qq * qq;
        ev[5] += qq;
        ev[6] += fabs(qq);
        return;
    }
    if (i < S.off || i >= (int64_t)S.off + S.n) {
        // the slot's particle index is stale (a rebuild gave up before its scatter)
        atomicOr(a.flag, kFlagBounds);
        return;
    }
    T fx = (T)fxd, fy = (T)fyd, fz = (T)fzd;
    if (!isfinite(fx + fy + fz)) atomicOr(a.flag, kFlagNonFinite);
    if (a.accumulate) {
        fx += a.F[i];
        fy += a.F[a.ntot + i];
        fz += a.F[2 * a.ntot + i];
    }
    a.F[i] = fx;
    a.F[a.ntot + i] = fy;
    a.F[2 * a.ntot + i] = fz;
    if (a.vel && i - S.off >= S.n_fixed) {
        // the same rounding as the deferred kick of the integrator
        const double h = S.anneal > 0.0 ? 0.5 * step_dt(S, a.kick_step) / S.mass : S.h_m;
        a.vel[i] = (T)fma(h, (double)fx, (double)a.vel[i]);
        a.vel[a.ntot + i] = (T)fma(h, (double)fy, (double)a.vel[a.ntot + i]);
        a.vel[2 * a.ntot + i] = (T)fma(h, (double)fz, (double)a.vel[2 * a.ntot + i]);
    }
}

template <typename T>
struct PairCT {
    using type = SysDev;
};
template <>
struct PairCT<float> {
    using type = PairConstF;
};

template <typename T>
__device__ __forceinline__ typename PairCT<T>::type pair_consts(const SysDev &S);
template <>
__device__ __forceinline__ PairConstF pair_consts<float>(const SysDev &S)
{
    return S.pair;
}
template <>
__device__ __forceinline__ SysDev pair_consts<double>(const SysDev &S)
{
    return S;
}

// ---------------------------------------------------------------------------
// Fourier force fused into the real-space pass of a step (eq. 3.6).  Wave w of
// the block sums the modes of quarter w, [w P/4, (w+1) P/4), for every particle of
// the tile and leaves the partial sum in LDS; the particle's lane adds
// the quarters in a fixed order when it finishes the particle.  The decomposition
// is the same on every tile shape, so the Fourier force of a particle does not
// depend on the real-space path.
// ---------------------------------------------------------------------------
constexpr int FT_MAX = 256;   // particles per tile, any shape

template <typename T>
struct KMT;
template <>
struct KMT<float> {
    using type = KModeF;
};
template <>
struct KMT<double> {
    using type = KModeD;
};

template <typename T>
using Four = T (*)[FT_MAX][3];

// Terms of the modes [l0, l1) of one lane's particle, as four sums f_j over the modes
// l0 + j, l0 + j + 4, ..., added as (f_0 + f_1) + (f_2 + f_3).  SUBS lanes of the
// wave share a particle (64 / SUBS apart), each with 4 / SUBS of the sums, so that
// small tiles, whose particles would leave lanes idle, walk a half or a quarter of the
// modes each (step at N = 3000 with 16 particles per tile 18.6 -> 17.5 us, N = 10001 in
// double precision with 32 30.3 -> 29.6).  Halves load four modes at a time whatever is
// left of the list, where an unrolled loop takes its remainder one load latency after the
// other (launch at N = 15000 with 8 lanes, P = 50 7.1 us with that, 6.6 now, 6.1 with 4
// lanes; in double precision 12.0 -> 11.3); for quarters that was no better (step at
// N = 10001 in double precision 27.9 -> 28.3 us).  With one lane per particle the mode constants
// are wave-uniform (scalar loads), and double precision, whose sums need not agree to the
// bit between tile shapes, has one sum and two modes at a time: the constants of four
// overflow the scalar registers (launch at N = 3e4, P = 1600 106 -> 113 us with them).
template <int SUBS, typename KM, typename Term>
__device__ __forceinline__ void fourier_subs(const KM *kk0, int l0, int l1, decltype(KM::m[0] + 0) f[3], Term &&term)
{
    using T = decltype(KM::m[0] + 0);
    constexpr int NS = 4 / SUBS;
    T s[NS][3];
#pragma unroll
    for (int j = 0; j < NS; ++j) s[j][0] = s[j][1] = s[j][2] = 0;
    if constexpr (SUBS == 1) {
        const auto kk = uniform_modes(kk0);
        l0 = __builtin_amdgcn_readfirstlane(l0);
        l1 = __builtin_amdgcn_readfirstlane(l1);
        int l = l0;
        if constexpr (sizeof(T) == 8) {
#pragma unroll 2
            for (; l < l1; ++l) term(load_mode(kk, l), s[0]);
        } else {
            for (; l + 4 <= l1; l += 4)
#pragma unroll
                for (int j = 0; j < 4; ++j) term(load_mode(kk, l + j), s[j]);
#pragma unroll
            for (int j = 0; j < 3; ++j)
                if (l + j < l1) term(load_mode(kk, l + j), s[j]);
        }
    } else if constexpr (SUBS == 2) {
        const int g = ((int)threadIdx.x & 63) / (64 / SUBS);
        for (int l = l0 + NS * g; l < l1; l += 8) {
            KM k[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) k[u] = kk0[min(l + 4 * (u >> 1) + (u & 1), l1 - 1)];
#pragma unroll
            for (int u = 0; u < 4; ++u)
                if (l + 4 * (u >> 1) + (u & 1) < l1) term(k[u], s[u & 1]);
        }
    } else {
        const int g = ((int)threadIdx.x & 63) / (64 / SUBS);
#pragma unroll 4
        for (int l = l0 + g; l < l1; l += 4) term(kk0[l], s[0]);
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        if constexpr (SUBS == 1) f[d] = (s[0][d] + s[1][d]) + (s[2][d] + s[3][d]);
        if constexpr (SUBS == 2) f[d] = lane_xor_sum<32>(s[0][d] + s[1][d]);
        if constexpr (SUBS == 4) f[d] = lane_xor_sum<32>(lane_xor_sum<16>(s[0][d]));
    }
}

template <typename T, int SUBS>
__device__ __forceinline__ void fourier_tile(const RealArgs<T> &a, const SysDev &S, const void *recs, int first,
                                             int count, Four<T> s4)
{
    using Rec = typename RBT<T>::Rec;
    using KM = typename KMT<T>::type;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int l0 = (S.p * wave) / 4, l1 = (S.p * (wave + 1)) / 4;
    const KM *kk = reinterpret_cast<const KM *>(a.km) + S.moff;
    const Rec *rp = reinterpret_cast<const Rec *>(recs) + first;
    constexpr int PART = 64 / SUBS;
    for (int p0 = 0; p0 < count; p0 += PART) {
        const int p = p0 + (lane & (PART - 1));
        T f[3] = {0, 0, 0};
        const Rec r = rp[min(p, count - 1)];
        if constexpr (sizeof(T) == 4) {
            float h[3], lo[3];
            split_fix(r.x, S, h[0], lo[0]);
            split_fix(r.y, S, h[1], lo[1]);
            split_fix(r.z, S, h[2], lo[2]);
            if (S.polar)
                fourier_subs<SUBS>(kk, l0, l1, f, [&](const KM &k, T g[3]) { fourier_term<true>(k, h, lo, g); });
            else
                fourier_subs<SUBS>(kk, l0, l1, f, [&](const KM &k, T g[3]) { fourier_term<false>(k, h, lo, g); });
        } else {
            const double s3[3] = {r.x, r.y, r.z};
            fourier_subs<SUBS>(kk, l0, l1, f, [&](const KM &k, T g[3]) { fourier_term(k, s3, g); });
        }
        if (p < count && lane < PART) {
            s4[wave][p][0] = f[0];
            s4[wave][p][1] = f[1];
            s4[wave][p][2] = f[2];
        }
    }
}

// Adds the Fourier force of tile particle k (charge qi) to (fx, fy, fz).
template <typename T>
__device__ __forceinline__ void add_fourier(Four<T> s4, int k, T qi, double &fx, double &fy, double &fz)
{
    T g[3];
    for (int d = 0; d < 3; ++d) g[d] = ((s4[0][k][d] + s4[1][k][d]) + s4[2][k][d]) + s4[3][k][d];
    fx += (double)(-qi * g[0]);
    fy += (double)(-qi * g[1]);
    fz += (double)(-qi * g[2]);
}

// Partner queue of the all-pairs waves of a block: the records (and, with
// per-particle diameters, the indices) of a wave's partners inside the search
// radius that have not been evaluated yet.
constexpr int kApUnroll = 2;                     // candidates per lane and round
constexpr int kApQueue = 64 * (kApUnroll + 1);   // at most 63 left over plus one round

template <typename T, bool DIAM>
struct PairQueue {
    typename RBT<T>::Rec r[RL_BS / 64][kApQueue];
    int32_t j[DIAM ? RL_BS / 64 : 1][DIAM ? kApQueue : 1];
};

// Orders the LDS accesses of one wave (its LDS instructions execute in order;
// this keeps the compiler from moving them).
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Tiles of a system whose totals the force launch of an all-pairs step forms by
// itself, and modes: see totals_in_force().
constexpr int kTotalTiles = 8, kTotalModes = 128;

// Fourier force of one particle (record pa) with a mode per lane, summed over
// the wave.  TOTALS: the lane first adds its modes' tile partials (in the order of the
// totals launch) and forms their constants; particle 0 stores them.
template <typename T, bool TOTALS>
__device__ __forceinline__ void fourier_lanes(const RealArgs<T> &a, const MidArgs<typename KMT<T>::type> *m, int sys,
                                              int il, const SysDev &S, const typename RBT<T>::Rec &pa, T g[3])
{
    using KM = typename KMT<T>::type;
    const KM *kk = reinterpret_cast<const KM *>(a.km) + S.moff;
    g[0] = g[1] = g[2] = 0;
    float h[3], lo[3];
    if constexpr (sizeof(T) == 4) {
        split_fix(pa.x, S, h[0], lo[0]);
        split_fix(pa.y, S, h[1], lo[1]);
        split_fix(pa.z, S, h[2], lo[2]);
    }
    for (int l = threadIdx.x & 63; l < S.p; l += 64) {
        KM k;
        if constexpr (TOTALS) {
            const KModeIn in = kmode_in(S, S.moff, l, m->modes, m->mode_w, m->mcap);
            const int nt = m->single_p ? m->single_nt : m->part_off[m->R + sys];
            const double2 *p = reinterpret_cast<const double2 *>(m->partial) + (m->single_p ? 0 : m->part_off[sys]) + l;
            double2 v[kTotalTiles];
#pragma unroll
            for (int t = 0; t < kTotalTiles; ++t) v[t] = t < nt ? p[(int64_t)t * S.p] : make_double2(0.0, 0.0);
            const double f = force_coefficient(in);
#pragma unroll
            for (int w = kTotalTiles / 2; w > 0; w >>= 1)
                for (int t = 0; t < w; ++t) {
                    v[t].x += v[t + w].x;
                    v[t].y += v[t + w].y;
                }
            k = kmode_of<KM>(in, f, v[0].x, v[0].y);
            if (il == 0) {
                m->rho[2 * in.o] = v[0].x;
                m->rho[2 * in.o + 1] = v[0].y;
                m->km[in.o] = k;
            }
        } else {
            k = kk[l];
        }
        if constexpr (sizeof(T) == 4) {
            if (S.polar)
                fourier_term<true>(k, h, lo, g);
            else
                fourier_term<false>(k, h, lo, g);
        } else {
            const double s3[3] = {pa.x, pa.y, pa.z};
            fourier_term(k, s3, g);
        }
    }
#pragma unroll
    for (int d = 0; d < 3; ++d) g[d] = wave_sum(g[d]);
}

// All-pairs real space of particle il of a one-cell system by one wave, its
// lanes 64 partners at a time in original order.  The partners inside the
// search radius go through the wave's LDS queue and are evaluated 64 at a
// time, so the pair terms run on full waves whatever share of the partners is
// inside.  With one particle per thread instead (256 per block, each walking
// all partners alone, two blocks at N = 300) the launch lasted as long as N
// dependent loads and pair terms of one lane: 79 us at N = 300 in single and
// 122 us at N = 200 in double precision, against about 5 us each now (a step
// of the 300 ions 105 -> 30 us then, 12 now in two launches).  FOURIER adds the Fourier force (a
// mode per lane).  DIAM compiles the per-particle-diameter LJ (only launches
// of contexts with diameters).
template <typename T, bool ENERGY, bool DIAM, bool FOURIER, bool TOTALS = false>
__device__ __forceinline__ void allpairs_body(const RealArgs<T> &a, int il, const SysDev &S, double *ev,
                                              PairQueue<T, DIAM> &qu, int sys = 0,
                                              const MidArgs<typename KMT<T>::type> *m = nullptr)
{
    using Rec = typename RBT<T>::Rec;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const Geo geo = make_geo<T>(S);
    const auto pc = pair_consts<T>(S);
    const Rec *pk = reinterpret_cast<const Rec *>(a.packed) + S.off;
    const int n = S.n;
    const Rec pa = pk[il];
    const double da = DIAM && S.diam_on ? a.diam[S.off + il] : 0.0;
    double fx = 0, fy = 0, fz = 0;
    PairE e{0, 0};
    Rec *qr = qu.r[wave];
    int32_t *qj = qu.j[DIAM ? wave : 0];
    int nq = 0;   // queued partners
    auto pair = [&](int k) {
        const Rec pb = qr[k];
        T dx, dy, dz, r2;
        displacement(pa, pb, geo, dx, dy, dz, r2);
        T phi = pair_phi<ENERGY>(pc, (T)pa.q, (T)pb.q, r2, e);
        if (DIAM && S.diam_on) {
            const double db = a.diam[S.off + qj[k]];
            if (!lj_far(S, da, db, r2)) phi += (T)lj_offset<ENERGY>(S, da, db, r2_double(pa, pb, S.L), e);
        }
        const T ph = qphi(phi);
        fx += qterm(ph * dx);
        fy += qterm(ph * dy);
        fz += qterm(ph * dz);
        if constexpr (ENERGY) ev[2] += 0.5 * (double)(phi * r2);
    };
    // a round's records are loaded a round ahead, the first ones under the Fourier force
    Rec pn[kApUnroll];
#pragma unroll
    for (int u = 0; u < kApUnroll; ++u) pn[u] = pk[min(64 * u + lane, n - 1)];
    T g[3];
    if constexpr (FOURIER) fourier_lanes<T, TOTALS>(a, m, sys, il, S, pa, g);
    for (int j0 = 0; j0 < n; j0 += 64 * kApUnroll) {
        Rec pb[kApUnroll];
#pragma unroll
        for (int u = 0; u < kApUnroll; ++u) {
            pb[u] = pn[u];
            pn[u] = pk[min(j0 + 64 * (kApUnroll + u) + lane, n - 1)];
        }
#pragma unroll
        for (int u = 0; u < kApUnroll; ++u) {
            const int j = j0 + 64 * u + lane;
            const bool in = j < n && j != il && near_test(pa, pb[u], geo);
            const uint64_t m = __ballot(in);
            if (in) {
                const int k = nq + __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32),
                                                             __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
                qr[k] = pb[u];
                if constexpr (DIAM) qj[k] = j;
            }
            nq += __builtin_popcountll(m);
        }
        wave_lds_order();
        while (nq >= 64) {
            nq -= 64;
            pair(nq + lane);
        }
        wave_lds_order();
    }
    if (lane < nq) pair(lane);
    if constexpr (ENERGY) {
        ev[0] += e.e_real;
        ev[1] += e.e_lj;
    }
    if constexpr (sizeof(T) == 4) range_check(fx, fy, fz, a.flag);
    fx = wave_sum(fx);
    fy = wave_sum(fy);
    fz = wave_sum(fz);
    if (lane != 0) return;
    if constexpr (sizeof(T) == 4) range_check(fx, fy, fz, a.flag);
    fx *= qscale<T>();
    fy *= qscale<T>();
    fz *= qscale<T>();
    if constexpr (FOURIER) {
        fx += (double)(-(T)pa.q * g[0]);
        fy += (double)(-(T)pa.q * g[1]);
        fz += (double)(-(T)pa.q * g[2]);
    }
    finish_particle<T, ENERGY>(a, S, S.off + il, fx, fy, fz, ev);
}

// ---------------------------------------------------------------------------
// Cell pass of one wave: every pair of its PPW (16 or 8) particles within the
// search radius.  Lane l works for particle l mod PPW: the 4 (8) lanes of a
// particle share its candidates.
//  1. The particles are taken in segments: runs that lie in one row of cells
//     and span few enough cells that the wrapped offsets from the segment's
//     centre are minimum images for every pair within the radius: they stay below
//     (nc - 1) / (2 nc) of the box, except with three cells along it, where they reach the
//     faces at +-1/2 and the rounding of the centre decides the sign.  If the cells are one
//     radius wide, such a candidate can be within reach on either side: it enters the test
//     by a bound of both (EDGE, a variant of its own: three more registers, which the step's
//     force launch would pay, N = 1e6 steps 1303 -> 1331 us for five.  Contexts with
//     lists have eight cells there).
//  2. The candidates of a segment, the parts of the rows of cells around it
//     that come within the radius, are numbered through and staged in LDS in
//     chunks of kCellChunk: the records, and the offsets (-2u, |u|^2) from
//     the segment's centre in box units.
//  3. One 16x16x4 FP32 matrix product per sixteen candidates gives
//     |u_i|^2 - R^2 + |u_j|^2 - 2 u_i.u_j, whose sign is the test: 256 pairs for
//     one matrix instruction and four sign shifts, where a lane that tests
//     its own particle's candidates takes about 15 instructions per pair of 64
//     (and walks candidates of other particles' rows in step).  R^2 carries
//     a margin above every rounding, so no pair is lost; what passes is
//     evaluated from the exact records, whose terms test the cutoffs.
//  4. Each lane appends its hits to its particle's list in LDS, and the lanes
//     of a particle evaluate that list.
// With eight particles per wave the matrix product has each of them in two
// columns, each column taking every second group of sixteen candidates: twice
// the waves and half the evaluations in each wave's chain, for launches that
// would leave most wave slots of the chip empty.
// ---------------------------------------------------------------------------
constexpr int kCellChunk = 128;   // candidates per chunk: one 32-bit mask per lane
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <typename Rec>
struct CellLds {
    union {
        float c[4][kCellChunk + 16];   // rows 16 banks apart: conflict-free operand reads
        uint8_t hit[16][kCellChunk + 4];
    };
    Rec rec[kCellChunk];
    int32_t slot[kCellChunk];
};

// Box fraction (x, y, z) of the segment's centre and a record's offset from it
// in box units, wrapped.
template <typename Rec>
struct CellOrigin;
template <>
struct CellOrigin<PackF> {
    uint32_t x, y, z;
};
template <>
struct CellOrigin<PartD> {
    double x, y, z;
};

// (any point near the centre will do: offsets of both sides are taken from it)
__device__ __forceinline__ void cell_origin(float x, float y, float z, CellOrigin<PackF> &o)
{
    o.x = __builtin_amdgcn_readfirstlane((uint32_t)(x * 4294967040.0f));
    o.y = __builtin_amdgcn_readfirstlane((uint32_t)(y * 4294967040.0f));
    o.z = __builtin_amdgcn_readfirstlane((uint32_t)(z * 4294967040.0f));
}
__device__ __forceinline__ void cell_origin(float x, float y, float z, CellOrigin<PartD> &o)
{
    o.x = x;
    o.y = y;
    o.z = z;
}
__device__ __forceinline__ void cell_offset(const PackF &p, const CellOrigin<PackF> &o, float u[3])
{
    u[0] = (float)(int32_t)(p.x - o.x) * 0x1p-32f;
    u[1] = (float)(int32_t)(p.y - o.y) * 0x1p-32f;
    u[2] = (float)(int32_t)(p.z - o.z) * 0x1p-32f;
}
// (a particle without a position, NaN in its record, is far from everything: its pairs,
// whose terms would be NaN for the other particle as well, do not pass the test)
constexpr float kNowhere = 1e10f;
__device__ __forceinline__ void cell_offset(const PartD &p, const CellOrigin<PartD> &o, float u[3])
{
    const double x = p.x - o.x, y = p.y - o.y, z = p.z - o.z;
    u[0] = (float)(x - rint(x));
    u[1] = (float)(y - rint(y));
    u[2] = (float)(z - rint(z));
    for (int d = 0; d < 3; ++d) u[d] = fabsf(u[d]) <= 1.0f ? u[d] : kNowhere;
}

// An offset of half the box, to within the roundings of the centre and of the offset.  The
// nearer image of such a candidate is 1/2 - a away from a particle at +-a of the
// centre, a <= 1/6, and (1/2 - a)^2 is at least a^2 + 1/12, whatever the sign.
constexpr float kCellEdge = 4e-6f;
__device__ __forceinline__ bool cell_edge(float u) { return fabsf(fabsf(u) - 0.5f) < kCellEdge; }

// Calls pair(record, slot, k) for every partner of the lane's particle pa
// (slot, active when act) that may lie within the search radius, split over
// the particle's lanes; k numbers the particle's partners from 0.
// Returns their number (the same on those lanes).  radius2: the search
// radius squared in box units; st: the system's cell starts.
template <typename T, int PPW, bool EDGE, typename F>
__device__ __forceinline__ int cell_pairs(const SysDev &S, const int32_t *st, const typename RBT<T>::Rec *gs,
                                          const typename RBT<T>::Rec &pa, int slot, bool act, float radius2,
                                          CellLds<typename RBT<T>::Rec> &w, F &&pair)
{
    using Rec = typename RBT<T>::Rec;
    const int lane = threadIdx.x & 63, i = lane & (PPW - 1), sub = lane >> 4;
    constexpr uint32_t kParticles = (1u << PPW) - 1;
    const int nc = __builtin_amdgcn_readfirstlane(S.nc), h = __builtin_amdgcn_readfirstlane(S.nh);
    const int slo = S.off, shi = S.off + S.n;
    int cx, cy, cz;
    cell_coords<T>(pa, nc, cx, cy, cz);
    const int row = cz * nc + cy;
    const int span = max(nc - 2 * h - 1, 1);   // most cells along x of a segment
    const int side = 2 * h + 1, nrows = side * side;
    const float cell = 1.0f / (float)nc;
    int listed = 0;
    uint32_t todo = (uint32_t)__ballot(act) & kParticles;
    while (todo) {
        const int lead = __builtin_ctz(todo);
        const int row0 = __builtin_amdgcn_readlane(row, lead), cx0 = __builtin_amdgcn_readlane(cx, lead);
        const bool in = ((todo >> i) & 1) && row == row0 && (uint32_t)(cx - cx0) < (uint32_t)span;
        const uint32_t seg = (uint32_t)__ballot(in) & kParticles;
        const int cx1 = __builtin_amdgcn_readlane(cx, 31 - __builtin_clz(seg));
        todo &= ~seg;
        const int cy0 = __builtin_amdgcn_readlane(cy, lead), cz0 = __builtin_amdgcn_readlane(cz, lead);
        // rows that wrap in x have two parts; part ids [0, nrows) are the
        // first parts, [nrows, 2 nrows) the second ones
        const int parts = (cx0 - h < 0 || cx1 + h >= nc) ? 2 * nrows : nrows;
        // matrix operand of the sixteen: (u, 1) by component `sub`
        CellOrigin<Rec> o;
        cell_origin(0.5f * (float)(cx0 + cx1 + 1) * cell, ((float)cy0 + 0.5f) * cell, ((float)cz0 + 0.5f) * cell, o);
        float ui[3];
        cell_offset(pa, o, ui);
        const float bop = sub == 0 ? ui[0] : (sub == 1 ? ui[1] : (sub == 2 ? ui[2] : 1.0f));
        // offsets are at most ex in x and ey in y and z, so the product's
        // terms stay below 4 (ex^2 + 2 ey^2); the margin covers their
        // roundings several times over
        const float ex = (0.5f * (float)(cx1 - cx0 + 1) + (float)h) * cell, ey = (0.5f + (float)h) * cell;
        const float r2m = radius2 + 1e-5f * (ex * ex + 2.0f * ey * ey);
        float ci = in ? fmaf(ui[0], ui[0], fmaf(ui[1], ui[1], ui[2] * ui[2])) - r2m : 1e30f;
        if constexpr (sizeof(T) == 8) ci = ci < kNowhere ? ci : 1e30f;
        const f32x4 cop = {ci, ci, ci, ci};
        for (int p0 = 0; p0 < parts; p0 += 64) {
            // candidate ranges: lane l has part p0 + l
            int rb = 0, rlen = 0;
            const int v = p0 + lane;
            const int q = v >= nrows ? v - nrows : v;
            if (v < parts) {
                const int qz = (q * (1024 / side + 1)) >> 10, qy = q - qz * side;   // q / side for q < 64, side <= 7
                const int dz = qz - h, dy = qy - h;
                int zz = cz0 + dz, yy = cy0 + dy;
                zz += zz < 0 ? nc : (zz >= nc ? -nc : 0);
                yy += yy < 0 ? nc : (yy >= nc ? -nc : 0);
                // the row is at least gy, gz away from every particle of the
                // segment: cells beyond the chord of the sphere are left out
                const float gy = fmaxf(fabsf((float)dy) - 1.0f, 0.0f), gz = fmaxf(fabsf((float)dz) - 1.0f, 0.0f);
                const float chord2 = radius2 * 1.00001f * (float)nc * (float)nc - (gy * gy + gz * gz);
                const int hx = min(h, (int)ceilf(sqrtf(fmaxf(chord2, 0.0f)) * 1.00001f));
                const int lo = cx0 - hx, hi = cx1 + hx;
                int xa, xb;   // cells xa .. xb - 1 of the row
                if (v < nrows) {
                    xa = max(lo, 0);
                    xb = min(hi, nc - 1) + 1;
                } else {
                    xa = lo < 0 ? lo + nc : 0;
                    xb = lo < 0 ? nc : max(hi - nc + 1, 0);
                }
                if (chord2 < 0.0f) xb = xa;
                const int base = (zz * nc + yy) * nc;
                // cell starts come from the last complete scan; clamped to the
                // system's slots every range stays in bounds whatever they hold
                rb = min(max(st[base + xa], slo), shi);
                rlen = min(max(st[base + xb], rb), shi) - rb;
            }
            const int incl = wave_incl_scan(rlen);
            const int pre = incl - rlen, del = rb - pre;   // candidate k of range r is slot k + del
            const int total = __builtin_amdgcn_readlane(incl, 63);
            // this particle's own number among the candidates (it is in its
            // own row, the middle one)
            int self = -1;
            for (int m = nrows / 2; m < parts; m += nrows) {
                const int r = m - p0;
                if (r < 0 || r >= 64) continue;
                const int b0 = __builtin_amdgcn_readlane(rb, r), n = __builtin_amdgcn_readlane(rlen, r);
                if ((uint32_t)(slot - b0) < (uint32_t)n) self = slot - __builtin_amdgcn_readlane(del, r);
            }
            int r0 = 0;   // first range of the chunk
            for (int c0 = 0; c0 < total; c0 += kCellChunk) {
                const int cnt = min(total - c0, kCellChunk);
                // slots of the chunk's candidates
                int d[2] = {0, 0}, r = r0;
                for (; r < 64; ++r) {
                    const int pr = __builtin_amdgcn_readlane(pre, r), dr = __builtin_amdgcn_readlane(del, r);
                    if (pr >= c0 + cnt) break;
                    d[0] = c0 + lane >= pr ? dr : d[0];
                    d[1] = c0 + lane + 64 >= pr ? dr : d[1];
                }
                r0 = r - 1;   // the range that the chunk ends in may go on
                Rec pb[2];
                int sl[2];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int k = c0 + lane + 64 * u;
                    sl[u] = k < total ? k + d[u] : -1;
                    pb[u] = gs[max(sl[u], slo)];
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    float x[3], edge2 = 0.0f;
                    cell_offset(pb[u], o, x);
                    if (EDGE && nc == 3)
                        for (int d = 0; d < 3; ++d)
                            if (cell_edge(x[d])) {
                                x[d] = 0.0f;
                                edge2 += 1.0f / 12.0f - kCellEdge;
                            }
                    const int k = lane + 64 * u;
                    const bool ok = sl[u] >= 0;
                    w.c[0][k] = ok ? -2.0f * x[0] : 0.0f;
                    w.c[1][k] = ok ? -2.0f * x[1] : 0.0f;
                    w.c[2][k] = ok ? -2.0f * x[2] : 0.0f;
                    const float x2 = fmaf(x[0], x[0], fmaf(x[1], x[1], x[2] * x[2]));
                    w.c[3][k] = ok ? (EDGE ? x2 + edge2 : x2) : 1e30f;
                    w.rec[k] = pb[u];
                    w.slot[k] = sl[u];
                }
                wave_lds_order();
                // lane (column, sub) gets candidates 16 g + 4 sub + t of group
                // g in register t; their signs enter the mask from the right:
                // candidate 16 g + 4 sub + t is bit 31 - (4 g + t)
                uint32_t m = 0;
#pragma unroll
                for (int g = 0; g < 8; g += 4) {
                    if (16 * g >= cnt) {
                        m <<= 16;
                        continue;
                    }
                    f32x4 y[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        y[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(w.c[sub][16 * (g + u) + (lane & 15)], bop, cop, 0, 0,
                                                                    0);
#pragma unroll
                    for (int u = 0; u < 4; ++u)
#pragma unroll
                        for (int t = 0; t < 4; ++t) m = __builtin_amdgcn_alignbit(m, __float_as_uint(y[u][t]), 31);
                }
                const int sk = self - c0;
                if ((uint32_t)sk < (uint32_t)kCellChunk && ((sk >> 2) & 3) == sub)
                    m &= ~(0x80000000u >> (4 * (sk >> 4) + (sk & 3)));
                // append to the particle's list, in the order of its lanes
                // (the lists take the place of the operands)
                wave_lds_order();
                int at = 0, n, part = sub;
                if constexpr (PPW == 8) {
                    const bool odd = lane & 8;
                    m &= odd ? 0x0F0F0F0Fu : 0xF0F0F0F0u;
                    n = __builtin_popcount(m);
                    const int both = lane_xor_sum<8>(n);
                    at = odd ? both - n : 0;
                    n = both;
                    part = 2 * sub + (odd ? 1 : 0);
                } else {
                    n = __builtin_popcount(m);
                }
                uint32_t lower, upper;
                lane_pair<16>((uint32_t)n, lower, upper);
                at += (sub & 1) ? (int)lower : 0;
                lane_pair<32>(lower + upper, lower, upper);
                at += (sub & 2) ? (int)lower : 0;
                n = (int)(lower + upper);
                while (m) {
                    const int b = __builtin_clz(m);
                    m &= ~(0x80000000u >> b);
                    w.hit[i][at++] = (uint8_t)(16 * (b >> 2) + 4 * sub + (b & 3));
                }
                wave_lds_order();
                constexpr int kLanes = 64 / PPW;
                for (int k = part; k < n; k += 2 * kLanes) {
                    const bool two = k + kLanes < n;
                    const int b0 = w.hit[i][k], b1 = w.hit[i][two ? k + kLanes : k];
                    const Rec p0 = w.rec[b0], p1 = w.rec[b1];
                    const int s0 = w.slot[b0], s1 = w.slot[b1];
                    pair(p0, s0, listed + k);
                    if (two) pair(p1, s1, listed + k + kLanes);
                }
                listed += n;
                wave_lds_order();   // the next chunk reuses the LDS
            }
        }
    }
    return listed;
}

// Adds a value over the lanes that share a particle in the cell pass.
template <int PPW>
__device__ __forceinline__ double cell_sum(double v)
{
    if constexpr (PPW == 8) v = lane_xor_sum<8>(v);
    return lane_xor_sum<32>(lane_xor_sum<16>(v));
}

// Cell pass of a wave over the cnt >= 1 slots from slot0 on of system `sys`.
// With BUILD the search radius is the list radius and every partner is also
// written to the particle's list.  The caller finishes the particles.
struct CellSum {
    double fx, fy, fz;
    int32_t iorig;
    bool first;   // the lane that finishes its particle
};

template <typename T, int PPW, bool ENERGY, bool BUILD, bool DIAM, bool EDGE>
__device__ __forceinline__ CellSum cells_body(const RealArgs<T> &a, const ListArgs *la, int sys, int slot0, int cnt,
                                              const SysDev &S, double *ev, CellLds<typename RBT<T>::Rec> &lds, typename RBT<T>::Rec &pa)
{
    using Rec = typename RBT<T>::Rec;
    const Geo geo = make_geo<T>(S);
    const auto pc = pair_consts<T>(S);
    const int lane = threadIdx.x & 63;
    CellSum c{0, 0, 0, 0, false};
    const int k = lane & (PPW - 1);
    const bool act = k < cnt;
    const int slot = slot0 + min(k, cnt - 1);
    const Rec *gs = reinterpret_cast<const Rec *>(a.sorted);
    pa = gs[slot];
    c.iorig = a.sorted_idx[slot];
    const double da = DIAM && S.diam_on ? a.diam[c.iorig] : 0.0;
    double fx = 0, fy = 0, fz = 0, vir = 0;
    PairE e{0, 0};
    const float r2 = BUILD ? S.pair.rlist2_box : S.pair.rsearch2_box;
    const int n = cell_pairs<T, PPW, EDGE>(S, a.start + S.cell_off + sys, gs, pa, slot, act, r2, lds,
                                [&](const Rec &pb, int b, int k) {
        if constexpr (BUILD)
            if (k < la->kmax) la->nbr[(int64_t)k * a.ntot + slot] = b;
        if (b == slot) return;   // only where stale cell starts name a slot twice
        T dx, dy, dz, d2;
        displacement(pa, pb, geo, dx, dy, dz, d2);
        T phi = pair_phi<ENERGY>(pc, (T)pa.q, (T)pb.q, d2, e);
        if (DIAM && S.diam_on) {
            const double db = BUILD ? a.dsorted[b] : a.diam[a.sorted_idx[b]];
            if (!lj_far(S, da, db, d2)) phi += (T)lj_offset<ENERGY>(S, da, db, r2_double(pa, pb, S.L), e);
        }
        const T ph = qphi(phi);
        fx += qterm(ph * dx);
        fy += qterm(ph * dy);
        fz += qterm(ph * dz);
        if constexpr (ENERGY) vir += 0.5 * (double)(phi * d2);
    });
    if constexpr (sizeof(T) == 4) range_check(fx, fy, fz, a.flag);
    c.fx = cell_sum<PPW>(fx);
    c.fy = cell_sum<PPW>(fy);
    c.fz = cell_sum<PPW>(fz);
    c.first = act && lane < PPW;
    if constexpr (sizeof(T) == 4)
        if (c.first) range_check(c.fx, c.fy, c.fz, a.flag);
    if constexpr (ENERGY) {
        ev[0] += e.e_real;
        ev[1] += e.e_lj;
        ev[2] += vir;
    }
    if constexpr (BUILD)
        if (c.first) {
            // an overflowing list is never read (the next step rebuilds)
            const bool ok = n <= la->kmax;
            la->nnb[slot] = ok ? n : 0;
            if (!ok) atomicOr(la->ls.overflow, 1);
        }
    c.fx *= qscale<T>();
    c.fy *= qscale<T>();
    c.fz *= qscale<T>();
    return c;
}

// The calling wave's tile (its own, so that a wave has one row of cells; see
// write_row_tiles), in XCD order over the blocks.
__device__ __forceinline__ int wave_tile(int nblocks)
{
    return 4 * xcd_tile((int)blockIdx.x, nblocks) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// Real space of force and energy calls, a wave tile per wave.  Bound by the
// VALU work of the pair terms and hit lists and, at small N, by the wave's chain of
// dependent loads.  Against one row of cells per lane (nine lanes a particle,
// tiles across rows, rows of more than 64 particles walked directly), force calls,
// trace times: N = 1e5 at density 0.1 48.5 -> 28 us, N = 3e4 23 -> 15 us,
// N = 3e4 with r_c = 13.6 (1060 partners) 778 -> 179 us; the step that builds the
// lists at N = 1e5 68 -> 45 us.
template <typename T, int PPW, bool ENERGY, bool DIAM, bool EDGE>
__global__ __launch_bounds__(RL_BS, sizeof(T) == 4 && !DIAM ? (ENERGY ? 6 : 7) : 1) void k_real_rows(RealArgs<T> a)
{
    // a wave runs one of the two bodies on its own part of either member
    __shared__ union {
        PairQueue<T, DIAM> pairs;
        CellLds<typename RBT<T>::Rec> cells[RL_BS / 64];
    } lds;
    const int wt = wave_tile((int)gridDim.x);
    const Tile t = a.tiles[wt];
    const SysDev S = a.sys[a.single ? 0 : t.sys];
    double ev[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (t.aux == 1) {
        allpairs_body<T, ENERGY, DIAM, false>(a, t.start, S, ev, lds.pairs);
    } else if (t.count > 0) {
        typename RBT<T>::Rec pa;
        const CellSum c = cells_body<T, PPW, ENERGY, false, DIAM, EDGE>(a, nullptr, t.sys, S.off + t.start, t.count, S, ev,
                                                                        lds.cells[threadIdx.x >> 6], pa);
        if (c.first) finish_particle<T, ENERGY>(a, S, c.iorig, c.fx, c.fy, c.fz, ev);
    }
    if constexpr (ENERGY) {
#pragma unroll
        for (int k = 0; k < 8; ++k) ev[k] = wave_sum(ev[k]);
        if ((threadIdx.x & 63) == 0)
            for (int k = 0; k < 8; ++k) a.epart[8 * (int64_t)wt + k] = ev[k];
    }
}

// ---------------------------------------------------------------------------
// Cell pass of sparse systems (sparse_pass): seven particles per wave, each on nine lanes,
// a lane per row of three cells.  A lane tests its row's few candidates one by one
// into a mask and evaluates those that pass.  With a candidate or two per
// row the chain of cell_pairs (ranges, staging, products, hit lists) costs more
// than the tests it saves: launch of 64 x 60 particles 10.3 us with it and 4.8 here,
// 64 x 461 17.6 and 8.2, 64 x 3679 at density 0.013 52 and 26.
// ---------------------------------------------------------------------------
constexpr int kSparsePPW = 7;
int sparse_per_tile() { return kSparsePPW; }

// Sum over the nine lanes of a particle, on its first lane.
__device__ __forceinline__ double row_sum(double v, int lane, int r)
{
    const double last = __shfl(v, lane + 8, 64);
    if (r == 0) v += last;
#pragma unroll
    for (int o = 4; o > 0; o >>= 1) {
        const double w = __shfl(v, lane + o, 64);
        if (r < o) v += w;
    }
    return v;
}

template <typename T, bool ENERGY, bool DIAM>
__device__ __forceinline__ void sparse_body(const RealArgs<T> &a, const Tile &t, const SysDev &S, double *ev)
{
    using Rec = typename RBT<T>::Rec;
    Geo geo = make_geo<T>(S);
    geo.rmax2u *= 1.00001f;   // the terms test the cutoffs, as on the other paths
    geo.rmax2 *= 1.00001;
    const auto pc = pair_consts<T>(S);
    const int lane = threadIdx.x & 63, p = lane / 9, r = lane - 9 * p;
    const bool act = p < t.count;
    const int slot = S.off + t.start + min(p, t.count - 1);
    const Rec *gs = reinterpret_cast<const Rec *>(a.sorted);
    const Rec pa = gs[slot];
    const int64_t iorig = a.sorted_idx[slot];
    const double da = DIAM && S.diam_on ? a.diam[iorig] : 0.0;
    const int nc = S.nc, slo = S.off, shi = S.off + S.n;
    const int32_t *st = a.start + S.cell_off + t.sys;
    int cx, cy, cz;
    cell_coords<T>(pa, nc, cx, cy, cz);
    int yy = cy + r % 3 - 1, zz = cz + r / 3 - 1;
    yy += yy < 0 ? nc : (yy >= nc ? -nc : 0);
    zz += zz < 0 ? nc : (zz >= nc ? -nc : 0);
    // cells cx - 1 .. cx + 1, and the one across the face; the starts clamped as in cell_pairs
    const int base = (zz * nc + yy) * nc, x0 = max(cx - 1, 0), x1 = min(cx + 2, nc);
    const int w = base + (cx == 0 ? nc - 1 : 0);
    const bool wrap = cx == 0 || cx == nc - 1;
    const int b0 = min(max(st[base + x0], slo), shi), n0 = min(max(st[base + x1], b0), shi) - b0;
    const int b1 = min(max(st[w], slo), shi), n1 = wrap ? min(max(st[w + 1], b1), shi) - b1 : 0;
    const int n = act ? n0 + n1 : 0;
    auto at = [&](int k) { return k < n0 ? b0 + k : b1 + k - n0; };
    double fx = 0, fy = 0, fz = 0, vir = 0;
    PairE e{0, 0};
    for (int c = 0; c < n; c += 64) {
        const int end = min(n, c + 64);
        uint64_t m = 0;
        for (int k = c; k < end; k += 2) {
            const int s0 = at(k), s1 = at(min(k + 1, n - 1));
            const Rec p0 = gs[s0], p1 = gs[s1];
            const uint32_t h0 = near_test(pa, p0, geo) && s0 != slot;
            const uint32_t h1 = near_test(pa, p1, geo) && s1 != slot && k + 1 < end;
            m |= (uint64_t)(h0 | h1 << 1) << (k - c);
        }
        while (m) {
            const int b = at(c + __builtin_ctzll(m));
            m &= m - 1;
            const Rec pb = gs[b];
            T dx, dy, dz, d2;
            displacement(pa, pb, geo, dx, dy, dz, d2);
            T phi = pair_phi<ENERGY>(pc, (T)pa.q, (T)pb.q, d2, e);
            if (DIAM && S.diam_on) {
                const double db = a.diam[a.sorted_idx[b]];
                if (!lj_far(S, da, db, d2)) phi += (T)lj_offset<ENERGY>(S, da, db, r2_double(pa, pb, S.L), e);
            }
            const T ph = qphi(phi);
            fx += qterm(ph * dx);
            fy += qterm(ph * dy);
            fz += qterm(ph * dz);
            if constexpr (ENERGY) vir += 0.5 * (double)(phi * d2);
        }
    }
    if constexpr (sizeof(T) == 4) range_check(fx, fy, fz, a.flag);
    fx = row_sum(fx, lane, r);
    fy = row_sum(fy, lane, r);
    fz = row_sum(fz, lane, r);
    if constexpr (ENERGY) {
        ev[0] += e.e_real;
        ev[1] += e.e_lj;
        ev[2] += vir;
    }
    if (!act || r != 0) return;
    if constexpr (sizeof(T) == 4) range_check(fx, fy, fz, a.flag);
    finish_particle<T, ENERGY>(a, S, iorig, fx * qscale<T>(), fy * qscale<T>(), fz * qscale<T>(), ev);
}

template <typename T, bool ENERGY, bool DIAM>
__global__ __launch_bounds__(RL_BS) void k_real_sparse(RealArgs<T> a)
{
    __shared__ PairQueue<T, DIAM> pairs;
    const int wt = wave_tile((int)gridDim.x);
    const Tile t = a.tiles[wt];
    const SysDev S = a.sys[a.single ? 0 : t.sys];
    double ev[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (t.aux == 1)
        allpairs_body<T, ENERGY, DIAM, false>(a, t.start, S, ev, pairs);
    else if (t.count > 0)
        sparse_body<T, ENERGY, DIAM>(a, t, S, ev);
    if constexpr (ENERGY) {
#pragma unroll
        for (int k = 0; k < 8; ++k) ev[k] = wave_sum(ev[k]);
        if ((threadIdx.x & 63) == 0)
            for (int k = 0; k < 8; ++k) a.epart[8 * (int64_t)wt + k] = ev[k];
    }
}

// Last launch of an energy call, a block per system: the sums of the wave tiles'
// partials in a fixed order (eight lanes per tile and one sum each), the Fourier
// energy and its virial from the modes, and the error word, all into memory of the host
// (kEnergyOut values per system, then the word).  With the sums over the modes on the
// host, five copies brought their inputs over, each with a wait of its own (energy and
// pair counts at N = 30001 553 -> 454 us, with two launches fewer).
__global__ __launch_bounds__(1024) void k_energy_sum(const SysDev *__restrict__ sys, int R, int n_tiles, int sparse,
                                                     const double *__restrict__ part, const int32_t *__restrict__ modes,
                                                     const double *__restrict__ mode_w, int mcap,
                                                     const double *__restrict__ rho, const int32_t *__restrict__ flag,
                                                     double *__restrict__ out)
{
    __shared__ double red[1024];
    __shared__ double2 wred[16];
    const int r = blockIdx.x, tid = threadIdx.x;
    const SysDev &S = sys[r];
    double ek = 0.0, wk = 0.0;
    for (int l = tid; l < S.p; l += 1024) {
        const int o = S.moff + l;
        const double mx = modes[o], my = modes[mcap + o], mz = modes[2 * (int64_t)mcap + o];
        const double m2 = mx * mx + my * my + mz * mz;
        const double rr = rho[2 * o] * rho[2 * o] + rho[2 * o + 1] * rho[2 * o + 1];
        // (2 pi/(V k^2)) |rho|^2 with k = 2 pi m/L  ==  |rho|^2 / (2 pi L |m|^2)
        const double el = mode_w[o] * rr / (2.0 * kPi * S.L * m2);
        ek += el;
        // lambda dE/dlambda under r -> lambda r, L -> lambda L at fixed alpha
        wk += el * (2.0 * kPi * kPi * m2 / (S.alpha * S.L * S.L) - 1.0);
    }
    ek = wave_sum(ek);
    wk = wave_sum(wk);
    if ((tid & 63) == 0) wred[tid >> 6] = make_double2(ek, wk);
    const auto first = [&](int k) { return k == R ? n_tiles : (sparse ? sys[k].stile_off : sys[k].ctile_off); };
    const int e1 = first(r + 1);
    double v = 0.0;
    int e = first(r) + (tid >> 3);
    for (; e + 3 * 128 < e1; e += 4 * 128) {
        double x[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) x[u] = part[8 * (int64_t)(e + 128 * u) + (tid & 7)];
#pragma unroll
        for (int u = 0; u < 4; ++u) v += x[u];
    }
    for (; e < e1; e += 128) v += part[8 * (int64_t)e + (tid & 7)];
    red[tid] = v;
    for (int w = 512; w >= 8; w >>= 1) {
        __syncthreads();
        if (tid < w) red[tid] += red[tid + w];
    }
    double *o = out + kEnergyOut * r;
    if (tid < 8) o[tid] = red[tid];
    if (tid == 8) {
        ek = wk = 0.0;
        for (int w = 0; w < 16; ++w) {
            ek += wred[w].x;
            wk += wred[w].y;
        }
        o[8] = S.coulomb * ek;
        o[9] = S.coulomb * wk;
    }
    if (r == 0 && tid == 9) out[kEnergyOut * R] = (double)*flag;
}

// List tile: LPP lanes per cell-sorted slot, U partners per lane and round.
constexpr int kListU = 4;

// What the list pass of a tile particle loads before its partners: its
// record, original index (where its force goes) and list length, and the
// raw partner slots of its first round.  None depends on the Fourier part,
// so the force launch issues these loads before it and their latency
// overlaps the Fourier arithmetic.  The first round's slots are read whatever
// the length (its columns are below 4 LPP; a clamp keeps them inside the list's
// kmax columns) and replaced by the particle's own slot
// past the length before any is used.
template <typename T>
struct ListHead {
    typename RBT<T>::Rec pa;
    int32_t iorig;
    int n, slot;
    int b[kListU];
};

template <typename T, int LPP>
__device__ __forceinline__ void list_head(const RealArgs<T> &a, const ListArgs &la, const Tile &t, const SysDev &S,
                                          ListHead<T> &h)
{
    using Rec = typename RBT<T>::Rec;
    const int tid = threadIdx.x;
    const int k = tid / LPP, sub = tid % LPP;
    h.n = 0;
    h.slot = 0;
    h.iorig = 0;
    h.pa = Rec{};
    if (k < t.count) {
        h.slot = S.off + t.start + k;
        h.pa = reinterpret_cast<const Rec *>(a.sorted)[h.slot];
        h.iorig = a.sorted_idx[h.slot];
        h.n = la.nnb[h.slot];
        const int32_t *nb = la.nbr + h.slot;
#pragma unroll
        for (int u = 0; u < kListU; ++u) h.b[u] = nb[(int64_t)min(sub + u * LPP, la.kmax - 1) * a.ntot];
    }
}

// Real-space force of tile particle k from its list, summed over the
// particle's LPP lanes (each of them holds the sum).
template <typename T, int LPP, bool DIAM>
__device__ __forceinline__ void list_pairs(const RealArgs<T> &a, const ListArgs &la, const Tile &t, const SysDev &S,
                                           const ListHead<T> &h, double &fx, double &fy, double &fz)
{
    using Rec = typename RBT<T>::Rec;
    const Geo geo = make_geo<T>(S);
    const auto pc = pair_consts<T>(S);
    const int tid = threadIdx.x;
    const int k = tid / LPP, sub = tid % LPP;
    fx = 0;
    fy = 0;
    fz = 0;
    const Rec pa = h.pa;
    const int slot = h.slot, n = h.n;
    if (k < t.count) {
        const Rec *gs = reinterpret_cast<const Rec *>(a.sorted);
        const double da = DIAM && S.diam_on ? a.diam[h.iorig] : 0.0;
        const int32_t *nb = la.nbr + slot;
        PairE e{0, 0};
        constexpr int U = kListU;
        int b[U];
#pragma unroll
        for (int u = 0; u < U; ++u) b[u] = sub + u * LPP < n ? h.b[u] : slot;
        for (int j = sub; j < n; j += U * LPP) {
            // this round's partner records, then the next round's partner
            // slots, so that those loads overlap this round's pairs
            Rec pb[U];
            double db[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                pb[u] = gs[b[u]];
                if constexpr (DIAM) db[u] = S.diam_on ? a.dsorted[b[u]] : 0.0;
            }
            int bn[U];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const int jj = j + U * LPP + u * LPP;
                bn[u] = jj < n ? nb[(int64_t)jj * a.ntot] : slot;
            }
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (j + u * LPP < n) {
                    T dx, dy, dz, r2;
                    displacement(pa, pb[u], geo, dx, dy, dz, r2);
                    T phi = pair_phi<false>(pc, (T)pa.q, (T)pb[u].q, r2, e);
                    if (DIAM && S.diam_on && !lj_far(S, da, db[u], r2))
                        phi += (T)lj_offset<false>(S, da, db[u], r2_double(pa, pb[u], S.L), e);
                    const T ph = qphi(phi);
                    fx += qterm(ph * dx);
                    fy += qterm(ph * dy);
                    fz += qterm(ph * dz);
                }
            }
#pragma unroll
            for (int u = 0; u < U; ++u) b[u] = bn[u];
        }
    }
    if constexpr (sizeof(T) == 4) range_check(fx, fy, fz, a.flag);
    fx = group_sum<LPP>(fx);
    fy = group_sum<LPP>(fy);
    fz = group_sum<LPP>(fz);
}

// Last step of a list particle (its first lane): scale of the real-space sum,
// the Fourier force from the tile's quarter sums, store.
template <typename T, int LPP>
__device__ __forceinline__ void list_finish(const RealArgs<T> &a, const Tile &t, const SysDev &S, const ListHead<T> &h,
                                            Four<T> s4, double fx, double fy, double fz)
{
    const int tid = threadIdx.x;
    const int k = tid / LPP, sub = tid % LPP;
    if (k < t.count && sub == 0) {
        if constexpr (sizeof(T) == 4) range_check(fx, fy, fz, a.flag);
        fx *= qscale<T>();
        fy *= qscale<T>();
        fz *= qscale<T>();
        add_fourier<T>(s4, k, (T)h.pa.q, fx, fy, fz);
        finish_particle<T, false>(a, S, h.iorig, fx, fy, fz, nullptr);
    }
}

// Slot of the calling wave on its SIMD: bits 3:0 (WAVE_ID) of the HW_ID
// hardware register, read with s_getreg_b32 (operand: (size - 1) << 11 |
// offset << 6 | register, HW_ID being register 4).  It only orders
// independent work; no result depends on it.
__device__ __forceinline__ int wave_slot() { return __builtin_amdgcn_s_getreg((4 - 1) << 11 | 0 << 6 | 4); }

// Force pass of one time step: the Fourier force plus the real-space force,
// on the cell list with list build when the step's rebuild flag is set, else
// on the list; then the closing half kick on the last step of a call.  Tiles
// are taken in XCD order (xcd_tile).  On the list, a particle's real-space sum
// stays in registers and its Fourier force in the tile's LDS quarter sums
// until the finish, which adds them in a fixed order, so the order of the
// two phases does not change any result.  SINGLE (a single-system context, which
// has no all-pairs tiles when it runs list steps) forms the tile from its
// index as the host builds it, and takes the system's particle and mode
// offsets (both 0) and its mode count from the launch, so that the record and
// mode-constant loads do not wait for the tile and the system constants.
// Seven waves per SIMD (72 registers, a few of the rebuild's in scratch): the list
// pass waits on its gathers, and 1792 blocks at once take N = 1e5 (1563) without a
// second round (N = 1e6 step 267 -> 263 us against six; eight spill into the list
// pass, 271 us).
// Double precision asks for two and reaches three (157 to 169 registers, no accumulation
// registers beside them): with three asked for, the compiler runs the two modes of the
// Fourier loop one after the other (launch at N = 3e4, P = 1000 70 -> 84 us), with one it
// takes 12 accumulation registers more and two waves (64 systems of 3000, P = 300
// 134 -> 151 us).
template <typename T, int LPP, bool DIAM, bool SINGLE>
__global__ __launch_bounds__(RL_BS, sizeof(T) == 8 ? 2 : (DIAM ? 1 : 7)) void k_real_step(RealArgs<T> a, ListArgs la)
{
    __shared__ union {
        T s4[4][FT_MAX][3];
        CellLds<typename RBT<T>::Rec> cells[RL_BS / 64];
        PairQueue<T, DIAM> pairs;
    } lds;
    auto &s4 = lds.s4;
    constexpr int SUBS = LPP <= 4 ? 1 : (LPP == 8 ? 2 : 4);   // list tiles of 256 / LPP particles
    // both flags are read before anything is stored, so that neither read
    // waits for the other
    const int poison = *la.ls.poison;
    const int rebuild = *la.ls.rebuild;
    // no launch of this kernel reads the step number: advance the replay's
    // base for the next steps
    if (la.ls.step_bump && blockIdx.x == 0 && threadIdx.x == 0) *la.ls.step_bump += la.ls.bump;
    if (poison) {
        // this step's rebuild gave up before its scan cleared the cell counts
        for (int k = blockIdx.x * RL_BS + threadIdx.x; k < la.ncell_tot; k += gridDim.x * RL_BS) la.count[k] = 0;
    }
    const int nb = rebuild ? la.n_rows : la.n_list;
    if ((int)blockIdx.x >= nb) return;
    const int ti = xcd_tile((int)blockIdx.x, nb);
    Tile t;
    if constexpr (SINGLE) {
        const int per = rebuild ? RL_PPB : 256 / LPP;
        t = Tile{0, ti * per, min(per, la.single_n - ti * per), rebuild ? 0 : 2};
    } else {
        t = rebuild ? a.tiles[ti] : la.list_tiles[ti];
    }
    // (a copy of a batch's constants crowds the modes out of the scalar registers, in single
    // precision; a reference costs double precision vector registers)
    using Sys = typename std::conditional<SINGLE || sizeof(T) == 8, SysDev, const SysDev &>::type;
    Sys S = a.sys[SINGLE ? 0 : __builtin_amdgcn_readfirstlane(t.sys)];
    if constexpr (SINGLE) {
        S.off = 0;
        S.moff = 0;
        S.p = la.single_p;
    }
    const bool allpairs = t.aux == 1;
    if (!allpairs && !rebuild) {
        ListHead<T> h;
        list_head<T, LPP>(a, la, t, S, h);
        double fx, fy, fz;
        // the two phases are independent until the finish: waves in odd
        // slots of their SIMD take the list pairs first, the others the
        // Fourier terms, so that the waves sharing a SIMD do not all wait on
        // loads at the same time
        if (wave_slot() & 1) {
            list_pairs<T, LPP, DIAM>(a, la, t, S, h, fx, fy, fz);
            fourier_tile<T, SUBS>(a, S, a.sorted, S.off + t.start, t.count, s4);
        } else {
            fourier_tile<T, SUBS>(a, S, a.sorted, S.off + t.start, t.count, s4);
            list_pairs<T, LPP, DIAM>(a, la, t, S, h, fx, fy, fz);
        }
        __syncthreads();
        list_finish<T, LPP>(a, t, S, h, s4, fx, fy, fz);
        return;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (allpairs) {
        if (wave < t.count) allpairs_body<T, false, DIAM, true>(a, t.start + wave, S, nullptr, lds.pairs);
        return;
    }
    // rebuild step: the pairs first, then the Fourier force, whose quarter sums
    // take the LDS of the pairs
    typename RBT<T>::Rec pa;
    CellSum c{0, 0, 0, 0, false};
    if (16 * wave < t.count)
        c = cells_body<T, 16, false, true, DIAM, false>(a, &la, t.sys, S.off + t.start + 16 * wave, min(16, t.count - 16 * wave), S,
                                                 nullptr, lds.cells[wave], pa);
    __syncthreads();
    fourier_tile<T, 1>(a, S, a.sorted, S.off + t.start, t.count, s4);
    __syncthreads();
    if (c.first) {
        add_fourier<T>(s4, 16 * wave + (int)(threadIdx.x & 15), (T)pa.q, c.fx, c.fy, c.fz);
        finish_particle<T, false>(a, S, c.iorig, c.fx, c.fy, c.fz, nullptr);
    }
}

// Force pass of a time step of a context that has only one-cell systems:
// Fourier and all-pairs real-space force in one launch (there is no list and
// nothing to rebuild).  With TOTALS it also forms the structure-factor totals, every wave
// for itself, and blocks behind the particles' draw the next step's modes: a step is
// then two launches (50 steps and an energy of the 300-ion electrolyte 849 -> 690 us).
template <typename T, bool DIAM, bool TOTALS>
__global__ __launch_bounds__(RL_BS) void k_pairs_step(RealArgs<T> a, int n_blocks, int single_n, int single_p,
                                                      MidArgs<typename KMT<T>::type> m)
{
    extern __shared__ double pairs_tab[];
    __shared__ PairQueue<T, DIAM> qu;
    const int b = (int)blockIdx.x;
    if (TOTALS && b >= n_blocks) {
        mid_sample(m, b - n_blocks, m.table_lds ? pairs_tab : nullptr);
        return;
    }
    // a single system's tile, offsets and mode count come with the launch
    const Tile t = single_n ? Tile{0, b * RL_ALLPAIRS, min(RL_ALLPAIRS, single_n - b * RL_ALLPAIRS), 1} : a.tiles[b];
    SysDev S = a.sys[t.sys];
    if (single_n) {
        S.off = 0;
        S.moff = 0;
        S.n = single_n;
        S.p = single_p;
    }
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave < t.count) allpairs_body<T, false, DIAM, true, TOTALS>(a, t.start + wave, S, nullptr, qu, t.sys, &m);
}

// Stand-alone scatter into cell order (force and energy calls; a time step
// on the neighbour list scatters inside the totals launch), then blocks that
// write the wave tiles.
// With gF the gradient of the forces moves along (adjoint of the real space).
template <typename T>
__global__ __launch_bounds__(256) void k_scatter(const SysDev *__restrict__ sys, const Tile *__restrict__ tiles,
                                                 const int32_t *__restrict__ start, const int32_t *__restrict__ cellid,
                                                 const int32_t *__restrict__ rank, const void *__restrict__ packed,
                                                 int32_t *__restrict__ sorted_idx, void *__restrict__ sorted, int n_tiles,
                                                 RowTileArgs rt, const T *__restrict__ gF, T *__restrict__ gsorted,
                                                 int64_t ntot)
{
    if ((int)blockIdx.x >= n_tiles) {
        write_row_tiles(rt, blockIdx.x - n_tiles);
        return;
    }
    const Tile t = tiles[blockIdx.x];
    if ((int)threadIdx.x >= t.count) return;
    const int64_t i = sys[t.sys].off + t.start + threadIdx.x;
    const int slot = start[cellid[i] + t.sys] + rank[i];
    scatter_record<T>(i, slot, packed, sorted_idx, sorted);
    if (gF) store4(gsorted, slot, gF[i], gF[ntot + i], gF[2 * ntot + i]);
}

// ---------------------------------------------------------------------------
// Real-space and LJ adjoint.  With dG = G_i - G_j and the pair force phi d:
//   dLoss/dq_i += -coulomb sum_j q_j (G(r)/r) dG.d
//   dLoss/dr_i += sum_j [ -(phi'(r)/r)(dG.d) d - phi dG ]
// G(r)/r = erfc(beta r)/r^3 + 2 beta exp(-alpha r^2)/(sqrt(pi) r^2), whose
// derivative is -3 erfc/r^4 - 6 beta e/(sqrt(pi) r^3) - 4 beta^3 e/(sqrt(pi) r).
// Same decomposition as the force.
// ---------------------------------------------------------------------------
template <typename T>
__device__ __forceinline__ void vjp_pair(const SysDev &S, T qi, T qj, T dx, T dy, T dz, T r2, T Gx, T Gy, T Gz,
                                         double &dq, double &rx, double &ry, double &rz)
{
    T phi = 0, dphi_r = 0, gq = 0;   // phi, phi'(r)/r, and the charge term
    const T GD = Gx * dx + Gy * dy + Gz * dz;
    if (r2 <= (T)S.rc2) {
        const T r = sqrt(r2);
        const T beta = (T)S.beta;
        const T ec = erfc(beta * r);
        const T ex = exp(-(T)S.alpha * r2);
        const T isp = (T)(1.0 / 1.7724538509055160273);
        const T inv_r = (T)1 / r, inv_r2 = inv_r * inv_r;
        const T g = (ec * inv_r + (T)2 * beta * isp * ex) * inv_r2;
        const T dg = -(T)3 * ec * inv_r2 * inv_r2 - (T)6 * beta * isp * ex * inv_r2 * inv_r -
                     (T)4 * beta * beta * beta * isp * ex * inv_r;
        const T cq = (T)S.coulomb * qi * qj;
        phi = -cq * g;
        dphi_r = -cq * dg * inv_r;
        gq = -(T)S.coulomb * qj * g * GD;
    }
    if (S.lj_on && r2 < (T)S.lj_rc2) {
        const T sr2 = (T)S.lj_sig2 / r2;
        const T sr6 = sr2 * sr2 * sr2, sr12 = sr6 * sr6;
        const T eps4 = (T)(4.0 * S.lj_eps);
        phi += eps4 * ((T)6 * sr6 - (T)12 * sr12) / r2;
        dphi_r += eps4 * ((T)168 * sr12 - (T)48 * sr6) / (r2 * r2);
    }
    dq += (double)gq;
    rx -= (double)(dphi_r * GD * dx + phi * Gx);
    ry -= (double)(dphi_r * GD * dy + phi * Gy);
    rz -= (double)(dphi_r * GD * dz + phi * Gz);
}

template <typename T, int PPW, bool EDGE>
__global__ __launch_bounds__(RL_BS) void k_vjp_real(RealArgs<T> a, const T *__restrict__ gF,
                                                    const T *__restrict__ gsorted, T *__restrict__ gpos,
                                                    T *__restrict__ gq, int accumulate)
{
    using Rec = typename RBT<T>::Rec;
    __shared__ CellLds<typename RBT<T>::Rec> lds[RL_BS / 64];
    const Tile t = a.tiles[wave_tile((int)gridDim.x)];
    const SysDev S = a.sys[a.single ? 0 : t.sys];
    const Geo geo = make_geo<T>(S);
    const int tid = threadIdx.x;
    const int64_t ntot = a.ntot;
    auto finish = [&](int64_t i, double dq, double rx, double ry, double rz) {
        if (accumulate) {
            dq += gq[i];
            rx += gpos[i];
            ry += gpos[ntot + i];
            rz += gpos[2 * ntot + i];
        }
        gq[i] = (T)dq;
        gpos[i] = (T)rx;
        gpos[ntot + i] = (T)ry;
        gpos[2 * ntot + i] = (T)rz;
    };
    if (t.aux == 1) {
        // a particle per wave (as in allpairs_body), a partner per lane
        const Rec *pk = reinterpret_cast<const Rec *>(a.packed) + S.off;
        {
            const int il = t.start;
            const int64_t i = S.off + il;
            const Rec pa = pk[il];
            const T Gix = gF[i], Giy = gF[ntot + i], Giz = gF[2 * ntot + i];
            double dq = 0, rx = 0, ry = 0, rz = 0;
            for (int j = tid & 63; j < S.n; j += 64) {
                if (j == il) continue;
                const Rec pb = pk[j];
                if (!near_test(pa, pb, geo)) continue;
                T dx, dy, dz, r2;
                displacement(pa, pb, geo, dx, dy, dz, r2);
                const int64_t jj = S.off + j;
                vjp_pair<T>(S, (T)pa.q, (T)pb.q, dx, dy, dz, r2, Gix - gF[jj], Giy - gF[ntot + jj],
                            Giz - gF[2 * ntot + jj], dq, rx, ry, rz);
            }
            dq = wave_sum(dq);
            rx = wave_sum(rx);
            ry = wave_sum(ry);
            rz = wave_sum(rz);
            if ((tid & 63) == 0) finish(i, dq, rx, ry, rz);
        }
        return;
    }
    const int lane = tid & 63, k = lane & (PPW - 1);
    const bool act = k < t.count;
    if (t.count <= 0) return;
    const int slot = S.off + t.start + min(k, t.count - 1);
    const Rec *gs = reinterpret_cast<const Rec *>(a.sorted);
    const Rec pa = gs[slot];
    const int64_t i = a.sorted_idx[slot];
    T Gix, Giy, Giz;
    load4(gsorted, slot, Gix, Giy, Giz);
    double dq = 0, rx = 0, ry = 0, rz = 0;
    cell_pairs<T, PPW, EDGE>(S, a.start + S.cell_off + t.sys, gs, pa, slot, act, S.pair.rsearch2_box, lds[tid >> 6],
                       [&](const Rec &pb, int b, int) {
        T dx, dy, dz, r2;
        displacement(pa, pb, geo, dx, dy, dz, r2);
        T Gjx, Gjy, Gjz;
        load4(gsorted, b, Gjx, Gjy, Gjz);
        vjp_pair<T>(S, (T)pa.q, (T)pb.q, dx, dy, dz, r2, Gix - Gjx, Giy - Gjy, Giz - Gjz, dq, rx, ry, rz);
    });
    dq = cell_sum<PPW>(dq);
    rx = cell_sum<PPW>(rx);
    ry = cell_sum<PPW>(ry);
    rz = cell_sum<PPW>(rz);
    if (act && lane < PPW) finish(i, dq, rx, ry, rz);
}

__global__ void k_fill_zero(uint32_t *p, int64_t n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
hipError_t launch_fill_zero(hipStream_t s, void *ptr, int64_t nbytes)
{
    const int64_t n = nbytes / 4;
    if (n <= 0) return hipSuccess;
    launch_k(k_fill_zero, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (uint32_t *)ptr, n);
    return hipGetLastError();
}

template <typename T>
static void scatter_launch(const LaunchCfg &c, const Workspace &w, const void *gF)
{
    launch_k(k_scatter<T>, c.n_part_tiles + c.n_row_tiles, 256, 0, c.stream, w.sys, w.part_tiles, w.cell_start, w.cellid,
             w.rank, w.packed, w.sorted_idx, w.sorted, c.n_part_tiles, row_tile_args(c, w), (const T *)gF,
             (T *)w.gsorted, c.ntot);
}

hipError_t launch_scatter(const LaunchCfg &c, const Workspace &w, const void *gF)
{
    if (c.prec == RBE_FP64)
        scatter_launch<double>(c, w, gF);
    else
        scatter_launch<float>(c, w, gF);
    return hipGetLastError();
}

template <typename T>
static RealArgs<T> real_args(const LaunchCfg &c, const Workspace &w, void *force, int accumulate, void *vel,
                             const void *q, uint64_t kick_step = 0)
{
    RealArgs<T> a;
    a.kick_step = kick_step;
    a.sys = w.sys;
    a.tiles = w.real_tiles;
    a.wave_tiles = w.cell_tiles;
    a.single = c.R == 1;
    a.start = w.cell_start;
    a.sorted_idx = w.sorted_idx;
    a.sorted = w.sorted;
    a.packed = w.packed;
    a.q = (const T *)q;
    a.ntot = c.ntot;
    a.F = (T *)force;
    a.accumulate = accumulate;
    a.vel = (T *)vel;
    a.flag = w.flag;
    a.epart = w.energy_part;
    a.km = w.kmode;
    a.diam = w.diam;
    a.dsorted = w.dsorted;
    return a;
}

template <typename T, bool ENERGY>
static void real_rows_launch(const LaunchCfg &c, const Workspace &w, RealArgs<T> a)
{
    // the per-particle-diameter LJ only in launches that need it: it costs
    // the others registers (and with them resident blocks)
    if (c.n_sparse_tiles) {
        a.tiles = w.sparse_tiles;
        launch_k(a.diam ? k_real_sparse<T, ENERGY, true> : k_real_sparse<T, ENERGY, false>, c.n_sparse_tiles / 4, RL_BS, 0,
                 c.stream, a);
        return;
    }
    a.tiles = a.wave_tiles;
    const int nb = c.n_cell_tiles / 4;
    const auto go = [&](auto edge) {
        constexpr bool E = decltype(edge)::value;
        if (c.cell_ppw == 8)
            launch_k(a.diam ? k_real_rows<T, 8, ENERGY, true, E> : k_real_rows<T, 8, ENERGY, false, E>, nb, RL_BS, 0,
                     c.stream, a);
        else
            launch_k(a.diam ? k_real_rows<T, 16, ENERGY, true, E> : k_real_rows<T, 16, ENERGY, false, E>, nb, RL_BS, 0,
                     c.stream, a);
    };
    if (c.cell_edge)
        go(std::true_type{});
    else
        go(std::false_type{});
}

hipError_t launch_real(const LaunchCfg &c, const Workspace &w, void *force, int accumulate, void *vel_kick,
                       uint64_t kick_step)
{
    if (c.prec == RBE_FP64)
        real_rows_launch<double, false>(c, w, real_args<double>(c, w, force, accumulate, vel_kick, nullptr, kick_step));
    else
        real_rows_launch<float, false>(c, w, real_args<float>(c, w, force, accumulate, vel_kick, nullptr, kick_step));
    return hipGetLastError();
}

template <typename T, int LPP>
static void real_step_launch(const LaunchCfg &c, const RealArgs<T> &a, const ListArgs &la)
{
    const int nb = la.n_rows > la.n_list ? la.n_rows : la.n_list;
    if (c.R == 1) {
        if (a.diam)
            launch_k(k_real_step<T, LPP, true, true>, nb, RL_BS, 0, c.stream, a, la);
        else
            launch_k(k_real_step<T, LPP, false, true>, nb, RL_BS, 0, c.stream, a, la);
    } else {
        if (a.diam)
            launch_k(k_real_step<T, LPP, true, false>, nb, RL_BS, 0, c.stream, a, la);
        else
            launch_k(k_real_step<T, LPP, false, false>, nb, RL_BS, 0, c.stream, a, la);
    }
}

template <typename T>
static void real_step_dispatch(const LaunchCfg &c, const Workspace &w, const ListStep &ls, const PairsStep &ps,
                               const RealArgs<T> &a, const ListArgs &la)
{
    if (c.all_pairs) {
        MidArgs<typename KMT<T>::type> m{};
        totals_args(m, c, w, ps.totals && ps.draw_next, ps.draw_step, &ls);
        // with the partner queues (28 KB at most) the table stays below 64 KB of LDS
        m.table_lds = m.table_lds && c.max_table <= 4096;
        const size_t sm = m.table_lds ? sizeof(double) * c.max_table : 0;
        const auto kernel = ps.totals ? (a.diam ? k_pairs_step<T, true, true> : k_pairs_step<T, false, true>)
                                      : (a.diam ? k_pairs_step<T, true, false> : k_pairs_step<T, false, false>);
        launch_k(kernel, c.n_real_tiles + m.n_sample_blocks, RL_BS, sm, c.stream, a, c.n_real_tiles, la.single_n,
                 la.single_p, m);
        return;
    }
    switch (c.list_lanes) {
    case 1:
        real_step_launch<T, 1>(c, a, la);
        break;
    case 2:
        real_step_launch<T, 2>(c, a, la);
        break;
    case 8:
        real_step_launch<T, 8>(c, a, la);
        break;
    case 16:
        real_step_launch<T, 16>(c, a, la);
        break;
    case 32:
        real_step_launch<T, 32>(c, a, la);
        break;
    default:
        real_step_launch<T, 4>(c, a, la);
        break;
    }
}

// An all-pairs step forms its totals in the force launch while every wave can load
// a mode's partials at once and has at most two modes per lane.
int totals_in_force(const LaunchCfg &c)
{
    return c.all_pairs && c.max_sys_rho_tiles <= kTotalTiles && c.max_p <= kTotalModes;
}

hipError_t launch_real_step(const LaunchCfg &c, const Workspace &w, const ListStep &ls, const PairsStep &ps, void *force,
                            void *vel_kick, uint64_t kick_step)
{
    ListArgs la;
    la.ls = ls;
    la.list_tiles = w.list_tiles;
    la.n_rows = c.n_real_tiles;
    la.n_list = c.n_list_tiles;
    la.nbr = w.nbr;
    la.nnb = w.nnb;
    la.kmax = c.kmax;
    la.count = w.cell_count;
    la.ncell_tot = c.ncell_tot;
    la.single_n = c.R == 1 ? (int)c.ntot : 0;
    la.single_p = c.R == 1 ? c.max_p : 0;
    if (c.prec == RBE_FP64)
        real_step_dispatch<double>(c, w, ls, ps, real_args<double>(c, w, force, 0, vel_kick, nullptr, kick_step), la);
    else
        real_step_dispatch<float>(c, w, ls, ps, real_args<float>(c, w, force, 0, vel_kick, nullptr, kick_step), la);
    return hipGetLastError();
}

hipError_t launch_energy(const LaunchCfg &c, const Workspace &w, const void *q, const void *vel)
{
    if (c.prec == RBE_FP64)
        real_rows_launch<double, true>(c, w, real_args<double>(c, w, nullptr, 0, (void *)vel, q));
    else
        real_rows_launch<float, true>(c, w, real_args<float>(c, w, nullptr, 0, (void *)vel, q));
    return hipGetLastError();
}

hipError_t launch_energy_sum(const LaunchCfg &c, const Workspace &w, double *out)
{
    const int sparse = c.n_sparse_tiles ? 1 : 0;
    launch_k(k_energy_sum, c.R, 1024, 0, c.stream, w.sys, c.R, sparse ? c.n_sparse_tiles : c.n_cell_tiles, sparse, w.energy_part, w.modes, w.mode_w, c.mcap,
             w.rho, w.flag, out);
    return hipGetLastError();
}

template <typename T>
static void vjp_real_launch(const LaunchCfg &c, RealArgs<T> a, const void *gF, const void *gsorted, void *gpos, void *gq,
                            int accumulate)
{
    a.tiles = a.wave_tiles;
    const auto kernel = c.cell_edge ? (c.cell_ppw == 8 ? k_vjp_real<T, 8, true> : k_vjp_real<T, 16, true>)
                                    : (c.cell_ppw == 8 ? k_vjp_real<T, 8, false> : k_vjp_real<T, 16, false>);
    launch_k(kernel, c.n_cell_tiles / 4, RL_BS, 0, c.stream, a,
             (const T *)gF, (const T *)gsorted, (T *)gpos, (T *)gq, accumulate);
}

hipError_t launch_vjp_real(const LaunchCfg &c, const Workspace &w, const void *gF, void *gpos, void *gq,
                           int accumulate)
{
    if (c.prec == RBE_FP64)
        vjp_real_launch<double>(c, real_args<double>(c, w, nullptr, 0, nullptr, nullptr), gF, w.gsorted, gpos, gq, accumulate);
    else
        vjp_real_launch<float>(c, real_args<float>(c, w, nullptr, 0, nullptr, nullptr), gF, w.gsorted, gpos, gq, accumulate);
    return hipGetLastError();
}

}  // namespace rbe

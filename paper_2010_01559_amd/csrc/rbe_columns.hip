// rbe_columns.hip -- Fourier sums over dense mode lists (classical Ewald) on
// the matrix cores.
//
// A list that fills columns (m_x, m_y, m_z = -Z .. Z), as the ball of eq. (2.9)
// does, factorises: exp(i k.r) is the product of one factor per dimension, and
//   rho(m_x, m_y, m_z) = sum_j [q_j e(m_x x_j) e(m_y y_j)] e(m_z z_j),
//   e(m s) = exp(2 pi i m s),
// is a matrix product over the particles j: rows are the columns' products in
// brackets, columns the cosines and sines of n z, n = 0 .. Z.  The force (eq. 2.11,
// first term) is the transposed product, over the trigonometric rows of a
// particle, with the coefficients of k_col_final.  Modes +m and -m have
// conjugate structure factors and equal force terms, so one of a pair is formed,
// and n and -n share a cosine and a sine: two real multiply-adds per mode and
// particle in the structure factor and four in the force, where a sum mode by
// mode takes a sine, a cosine and about 15 instructions in each pass.
//
// The factors come from one sine and cosine per particle and dimension and
// their powers, all in double, and the products run on the FP64 matrix
// instruction (16x16x4; lane l holds row or column l mod 16 of operand A or B at
// depth l / 16, and rows 4 r + l / 16, column l mod 16 of the result in register r),
// for both precisions: half the rate of the FP32 one, no rounding to watch, and
// already far from what the sums by mode reach.  Measured at N = 30000 and
// 11752 modes in single precision (trace): 147 + 22 + 191 + 5 us by mode (partials,
// totals, force, sum of its parts), 52 + 7 + 86 us here, of which the matrix
// instructions alone are 16 and 31; the force's relative error against 64 bits
// 2.5e-7 -> 1.8e-7.
#include <hip/hip_runtime.h>

#include <stdint.h>

#include <algorithm>

#include "rbe_device.h"
#include "rbe_internal.h"
#include "rbe_roles.h"

namespace rbe {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kColsPerBlock = 64;    // structure-factor blocks: 4 waves x 2 row tiles x 8 columns
constexpr int kTrigPerBlock = 32;    // trigonometric rows of a structure-factor block: two tiles
constexpr int kColPad = 4;           // particles of padding per LDS table row: spreads rows over the banks

// Trigonometric row of cos(n z) and sin(n z): 0 is the constant, then cosine and
// sine of 1, of 2, ...
__device__ __forceinline__ int trig_cos(int n) { return n == 0 ? 0 : 2 * n - 1; }

// e(m s), m = 0 .. M, times `scale` into row m of tab (stride ld).
__device__ __forceinline__ void power_table(double s, double scale, int M, double2 *tab, int ld)
{
    double sn, cs;
    sincospi(2.0 * s, &sn, &cs);
    double2 e = make_double2(scale, 0.0);
    for (int m = 0;; ++m) {
        tab[m * ld] = e;
        if (m == M) break;
        e = make_double2(e.x * cs - e.y * sn, e.x * sn + e.y * cs);
    }
}

// Trigonometric rows [t0, t1) of one z into tab (row t0 first, stride ld).
__device__ __forceinline__ void trig_table(double s, int t0, int t1, double *tab, int ld)
{
    double sn, cs, c0, s0;
    sincospi(2.0 * s, &sn, &cs);
    const int n0 = t0 >> 1;
    sincospi(2.0 * wrap_rev((double)n0 * s), &s0, &c0);
    double2 e = make_double2(c0, s0);
    for (int n = n0; 2 * n - 1 < t1; ++n) {
        const int tc = trig_cos(n), ts = 2 * n;
        if (tc >= t0 && tc < t1) tab[(tc - t0) * ld] = e.x;
        if (n > 0 && ts >= t0 && ts < t1) tab[(ts - t0) * ld] = e.y;
        e = make_double2(e.x * cs - e.y * sn, e.x * sn + e.y * cs);
    }
}

// The lane's signed pair (p, q) of the y factor with which the x factor (xr, xi)
// gives xr p + xi q: the real part (comp 0) or the imaginary part (comp 1) of
// e(m_x x) e(m_y y), m_y = sgn |m_y|.
__device__ __forceinline__ double xy_part(const double2 &x, const double2 &y, int comp, double sgn)
{
    const double yi = sgn * y.y;
    return comp == 0 ? fma(x.x, y.x, -(x.y * yi)) : fma(x.x, yi, x.y * y.x);
}

struct ColArgs {
    const SysDev *sys;
    const ColumnDev *cols;
    int ncols, Rx, Ry, Zm;
    int64_t D;          // trigonometric slots of all columns
    double *part;       // [groups][D][2]
    int per;            // particles of a group
};

// Structure-factor partials of a group of particles (grid x) for 64 columns
// (grid y) and 32 trigonometric rows (grid z), in chunks of NB particles whose
// factors are tabulated in LDS.  Bound by the matrix cores (4 NB / 4
// instructions of 64 cycles per wave and chunk) and, for the largest lists' small
// chunks, by the tables.
template <typename T, int NB>
__global__ __launch_bounds__(256) void k_col_rho(ColArgs a, const T *__restrict__ pos, const T *__restrict__ q,
                                                 int64_t ntot)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int LD = NB + kColPad;
    double2 *ex = reinterpret_cast<double2 *>(smem);
    double2 *ey = ex + (a.Rx + 1) * LD;
    double *ez = reinterpret_cast<double *>(ey + (a.Ry + 1) * LD);   // [kTrigPerBlock][LD]
    const int tid = threadIdx.x, lane = tid & 63, row = lane & 15, depth = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int t0 = blockIdx.z * kTrigPerBlock;
    // columns are sorted by falling Z: nothing left when the first has no such row
    const int c_first = blockIdx.y * kColsPerBlock;
    if (2 * a.cols[c_first].Z < t0) return;
    const int n = a.sys[0].n;
    const double invL = a.sys[0].invL;
    // this lane's two columns (rows are (column, real or imaginary part))
    int mx[2], my[2], nt[2];
    double sgn[2];
    const int comp = row & 1;
#pragma unroll
    for (int u = 0; u < 2; ++u) {
        const int c0 = c_first + (2 * wave + u) * 8;
        const ColumnDev col = a.cols[min(c0 + (row >> 1), a.ncols - 1)];
        mx[u] = col.mx;
        my[u] = col.my < 0 ? -col.my : col.my;
        sgn[u] = col.my < 0 ? -1.0 : 1.0;
        const int rows_left = c0 < a.ncols ? 2 * a.cols[c0].Z + 1 - t0 : 0;   // of the tile's first column
        nt[u] = rows_left <= 0 ? 0 : (rows_left <= 16 ? 1 : 2);
    }
    f64x4 acc[2][2];
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int v = 0; v < 2; ++v) acc[u][v] = f64x4{0.0, 0.0, 0.0, 0.0};
    const int first = blockIdx.x * a.per, last = min(n, first + a.per);
    for (int j0 = first; j0 < last; j0 += NB) {
        __syncthreads();   // the chunk before has been read
        if (tid < 3 * NB) {
            const int d = tid / NB, j = tid % NB;
            const bool ok = j0 + j < last;
            const double s = ok ? frac01((double)pos[d * ntot + j0 + j] * invL) : 0.0;
            if (d == 0)
                power_table(s, ok ? (double)q[j0 + j] : 0.0, a.Rx, ex + j, LD);
            else if (d == 1)
                power_table(s, 1.0, a.Ry, ey + j, LD);
            else
                trig_table(s, t0, t0 + kTrigPerBlock, ez + j, LD);
        }
        __syncthreads();
#pragma unroll 2
        for (int k = depth; k < NB; k += 4) {
            const double b0 = ez[row * LD + k], b1 = ez[(16 + row) * LD + k];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                if (nt[u] == 0) continue;
                const double v = xy_part(ex[mx[u] * LD + k], ey[my[u] * LD + k], comp, sgn[u]);
                acc[u][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, b0, acc[u][0], 0, 0, 0);
                if (nt[u] > 1) acc[u][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(v, b1, acc[u][1], 0, 0, 0);
            }
        }
    }
    double *out = a.part + 2 * (int64_t)blockIdx.x * a.D;
#pragma unroll
    for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int c = c_first + (2 * wave + u) * 8 + ((4 * r + depth) >> 1);
            if (c >= a.ncols) continue;
            const ColumnDev col = a.cols[c];
#pragma unroll
            for (int v = 0; v < 2; ++v) {
                const int t = t0 + 16 * v + row;
                if (t <= 2 * col.Z) out[2 * (int64_t)(col.base + t) + (depth & 1)] = acc[u][v][r];
            }
        }
}

// Structure factors and force constants of the listed modes from the group
// partials, and the coefficient matrix of the force pass.  A thread quad per
// slot (column, n): a quarter of the groups each.
template <typename KM>
__global__ __launch_bounds__(256) void k_col_final(ColArgs a, int groups, const int32_t *__restrict__ slot_col,
                                                   const int4 *__restrict__ slot_mode, int nslots,
                                                   const double *__restrict__ mode_w, double *__restrict__ rho,
                                                   KM *__restrict__ km, double *__restrict__ coef)
{
    __shared__ double red[4][64][4];
    const int k = threadIdx.x & 63, part = threadIdx.x >> 6;
    const int s = blockIdx.x * 64 + k;
    const bool ok = s < nslots;
    ColumnDev col{};
    int n = 0;
    double v[4] = {0.0, 0.0, 0.0, 0.0};   // sums of (real, imaginary part) x (cosine, sine)
    if (ok) {
        col = a.cols[slot_col[s]];
        n = s - col.slot;
        const double2 *p = reinterpret_cast<const double2 *>(a.part) + col.base;
        const int tc = trig_cos(n), ts = 2 * n;
#pragma unroll 4
        for (int g = part; g < groups; g += 4) {
            const double2 c = p[g * a.D + tc];
            const double2 d = p[g * a.D + ts];
            v[0] += c.x;
            v[1] += c.y;
            v[2] += d.x;
            v[3] += d.y;
        }
    }
    for (int j = 0; j < 4; ++j) red[part][k][j] = v[j];
    __syncthreads();
    if (part != 0 || !ok) return;
    for (int j = 0; j < 4; ++j) v[j] = ((red[0][k][j] + red[1][k][j]) + red[2][k][j]) + red[3][k][j];
    if (n == 0) v[2] = v[3] = 0.0;
    // rho of (m_x, m_y, +n) and (m_x, m_y, -n)
    const double2 rp = make_double2(v[0] - v[3], v[1] + v[2]), rm = make_double2(v[0] + v[3], v[1] - v[2]);
    const SysDev &S = a.sys[0];
    const int4 l4 = slot_mode[s];
    const int l[4] = {l4.x, l4.y, l4.z, l4.w};
    double w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        w[e] = 0.0;
        if (l[e] < 0) continue;
        w[e] = mode_w[l[e]];
        // entries 0, 1: (m_x, m_y, +-n); 2, 3: their negatives
        const double sg = e < 2 ? 1.0 : -1.0, zn = (e & 1) ? -(double)n : (double)n;
        const double2 r = (e & 1) ? rm : rp;
        KModeIn in;
        in.o = l[e];
        in.mx = sg * col.mx;
        in.my = sg * col.my;
        in.mz = sg * zn;
        in.w = w[e];
        in.coulomb = S.coulomb;
        in.L = S.L;
        in.polar = S.polar;
        make_kmode<KM>(in, force_coefficient(in), r.x, sg * r.y, rho, km);
    }
    // g+- = f w rho / |m|^2, a pair's weights added; P = g+ + g-, Q = g+ - g-
    const double m2 = (double)col.mx * col.mx + (double)col.my * col.my + (double)n * n;
    const double f = m2 > 0.0 ? S.coulomb * 2.0 / (S.L * S.L * m2) : 0.0;
    const double fp = f * (w[0] + w[2]), fm = f * (w[1] + w[3]);
    const double2 P = make_double2(fp * rp.x + fm * rm.x, fp * rp.y + fm * rm.y);
    const double2 Q = make_double2(fp * rp.x - fm * rm.x, fp * rp.y - fm * rm.y);
    // sum over the signs of n of g e(-n z) = cos P - i sin Q, and with the factor
    // m_z: n (cos Q - i sin P); rows of the matrix are cosines and sines,
    // columns the real and imaginary part of the two
    double *o = coef + col.coef;
    const double dn = (double)n;
    double *oc = o + 16 * trig_cos(n);
    oc[0] = P.x;
    oc[1] = P.y;
    oc[2] = dn * Q.x;
    oc[3] = dn * Q.y;
    if (n > 0) {
        double *os = o + 16 * (2 * n);
        os[0] = Q.y;
        os[1] = -Q.x;
        os[2] = dn * P.y;
        os[3] = -dn * P.x;
    }
}

// Force of NB particles (grid x) from all columns: tiles of four columns x four
// sums (the real and imaginary parts of k_col_final's two) by sixteen
// particles; the waves take the column tiles in turn.  A result element times
// the real or imaginary part of its e(-m_x x - m_y y) adds to the force.
template <typename T, int NB>
__global__ __launch_bounds__(256) void k_col_force(ColArgs a, const int32_t *__restrict__ tile_rows,
                                                   const double *__restrict__ coef, const T *__restrict__ pos,
                                                   const T *__restrict__ q, int64_t ntot, T *__restrict__ F,
                                                   int accumulate, int32_t *__restrict__ flag)
{
    extern __shared__ __align__(16) unsigned char smem[];
    constexpr int LD = NB + kColPad, RT = NB / 16;
    const int KZ = (2 * a.Zm + 1 + 3) & ~3;
    double2 *ex = reinterpret_cast<double2 *>(smem);
    double2 *ey = ex + (a.Rx + 1) * LD;
    double *ez = reinterpret_cast<double *>(ey + (a.Ry + 1) * LD);   // [KZ][LD]
    const int tid = threadIdx.x, lane = tid & 63, col16 = lane & 15, depth = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = a.sys[0].n;
    const double invL = a.sys[0].invL;
    const int first = blockIdx.x * NB;
    if (tid < 3 * NB) {
        const int d = tid / NB, j = tid % NB;
        const double s = first + j < n ? frac01((double)pos[d * ntot + first + j] * invL) : 0.0;
        if (d == 0)
            power_table(s, 1.0, a.Rx, ex + j, LD);
        else if (d == 1)
            power_table(s, 1.0, a.Ry, ey + j, LD);
        else
            trig_table(s, 0, KZ, ez + j, LD);
    }
    __syncthreads();
    double a1[RT][4], a2[RT][4];
#pragma unroll
    for (int u = 0; u < RT; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) a1[u][r] = a2[u][r] = 0.0;
    const int comp = lane & 3;
    const int ntiles = (a.ncols + 3) / 4;
    for (int ct = wave; ct < ntiles; ct += 4) {
        const int K = tile_rows[2 * ct];
        const double *cf = coef + tile_rows[2 * ct + 1] + lane;   // row 4 s + depth, column col16
        f64x4 acc[RT];
#pragma unroll
        for (int u = 0; u < RT; ++u) acc[u] = f64x4{0.0, 0.0, 0.0, 0.0};
#pragma unroll 2
        for (int t = 0; t < K; t += 4) {
            const double b = cf[16 * t];
#pragma unroll
            for (int u = 0; u < RT; ++u)
                acc[u] = __builtin_amdgcn_mfma_f64_16x16x4f64(ez[(t + depth) * LD + 16 * u + col16], b, acc[u], 0, 0, 0);
        }
        const ColumnDev col = a.cols[min(4 * ct + (col16 >> 2), a.ncols - 1)];
        const int my = col.my < 0 ? -col.my : col.my;
        const double sgn = col.my < 0 ? -1.0 : 1.0;
        // Im(e(-phi) (re + i im)) = cos(phi) im - sin(phi) re
        const double f1 = comp < 2 ? (double)col.mx : 1.0, f2 = comp < 2 ? (double)col.my : 0.0;
#pragma unroll
        for (int u = 0; u < RT; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int i = 16 * u + 4 * r + depth;
                const double2 x = ex[col.mx * LD + i], y = ey[my * LD + i];
                const double part = (comp & 1) ? xy_part(x, y, 0, sgn) : -xy_part(x, y, 1, sgn);
                const double v = acc[u][r] * part;
                a1[u][r] = fma(f1, v, a1[u][r]);
                a2[u][r] = fma(f2, v, a2[u][r]);
            }
    }
    __syncthreads();   // the tables have been read
    // sums over the sixteen lanes of a particle, then over the waves
    double *red = reinterpret_cast<double *>(smem);   // [4][NB][3]
#pragma unroll
    for (int u = 0; u < RT; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            double x = comp < 2 ? a1[u][r] : 0.0, y = a2[u][r], z = comp < 2 ? 0.0 : a1[u][r];
#pragma unroll
            for (int o = 8; o > 0; o >>= 1) {
                x += __shfl_xor(x, o, 64);
                y += __shfl_xor(y, o, 64);
                z += __shfl_xor(z, o, 64);
            }
            if (col16 == 0) {
                double *p = red + 3 * (wave * NB + 16 * u + 4 * r + depth);
                p[0] = x;
                p[1] = y;
                p[2] = z;
            }
        }
    __syncthreads();
    if (tid >= NB || first + tid >= n) return;
    const int64_t i = first + tid;
    const double mq = -(double)q[i];
    T f[3];
#pragma unroll
    for (int d = 0; d < 3; ++d) {
        double v = 0.0;
        for (int w = 0; w < 4; ++w) v += red[3 * (w * NB + tid) + d];
        f[d] = (T)(mq * v);
    }
    if (!isfinite(f[0] + f[1] + f[2])) atomicOr(flag, kFlagNonFinite);
#pragma unroll
    for (int d = 0; d < 3; ++d) F[d * ntot + i] = accumulate ? F[d * ntot + i] + f[d] : f[d];
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
static ColArgs col_args(const LaunchCfg &c, const Workspace &w)
{
    const ColumnSet &s = c.cols;
    ColArgs a;
    a.sys = w.sys;
    a.cols = w.cols;
    a.ncols = s.ncols;
    a.Rx = s.Rx;
    a.Ry = s.Ry;
    a.Zm = s.Zm;
    a.D = s.D;
    a.part = w.partial;
    a.per = s.per;
    return a;
}

static size_t rho_lds(const ColumnSet &s, int nb)
{
    return (size_t)(nb + kColPad) * (16 * (size_t)(s.Rx + s.Ry + 2) + 8 * kTrigPerBlock);
}

static size_t force_lds(const ColumnSet &s, int nb)
{
    const size_t tables = (size_t)(nb + kColPad) * (16 * (size_t)(s.Rx + s.Ry + 2) + 8 * ((2 * (size_t)s.Zm + 4) & ~(size_t)3));
    return std::max(tables, (size_t)4 * nb * 3 * sizeof(double));
}

// Particles per block of the two passes, and the particle groups of the first:
// 64 where the tables of two blocks fit a compute unit's 160 KB of LDS, 32 for
// longer columns and, in the force pass, while 64 would give fewer blocks than compute
// units.  Returns whether the tables of 32 fit (modes up to about 97 in each
// dimension), and the partial sums of one group at least in `room` doubles.
bool column_shapes(ColumnSet &s, int64_t n, size_t room)
{
    constexpr size_t most = 160 * 1024, two = 80 * 1024;
    if (std::max(rho_lds(s, 32), force_lds(s, 32)) > most) return false;
    s.rho_nb = rho_lds(s, 64) <= two ? 64 : 32;
    s.force_nb = force_lds(s, 64) <= two && n > 16384 ? 64 : 32;
    // about two blocks per compute unit
    const int64_t blocks = (int64_t)((s.ncols + kColsPerBlock - 1) / kColsPerBlock);
    const int64_t chunks = (n + s.rho_nb - 1) / s.rho_nb;
    const int64_t most_groups = (int64_t)(room / (2 * (size_t)s.D));
    if (most_groups < 1) return false;
    int64_t groups = std::min<int64_t>(std::max<int64_t>(1, (512 + blocks - 1) / blocks), chunks);
    groups = std::min(groups, most_groups);
    s.per = (int)((chunks + groups - 1) / groups * s.rho_nb);
    s.groups = (int)((n + s.per - 1) / s.per);
    return true;
}

template <typename T>
static hipError_t col_rho(const LaunchCfg &c, const Workspace &w, const void *pos, const void *q)
{
    const ColumnSet &s = c.cols;
    const dim3 g(s.groups, (s.ncols + kColsPerBlock - 1) / kColsPerBlock, (2 * s.Zm + 1 + kTrigPerBlock - 1) / kTrigPerBlock);
    return launch_lds(s.rho_nb == 64 ? k_col_rho<T, 64> : k_col_rho<T, 32>, g, dim3(256), rho_lds(s, s.rho_nb), c.stream,
                      col_args(c, w), (const T *)pos, (const T *)q, c.ntot);
}

hipError_t launch_col_rho(const LaunchCfg &c, const Workspace &w, const void *pos, const void *q)
{
    return c.prec == RBE_FP64 ? col_rho<double>(c, w, pos, q) : col_rho<float>(c, w, pos, q);
}

template <typename KM>
static hipError_t col_final(const LaunchCfg &c, const Workspace &w)
{
    const ColumnSet &s = c.cols;
    launch_k(k_col_final<KM>, dim3((s.nslots + 63) / 64), dim3(256), 0, c.stream, col_args(c, w), s.groups,
             (const int32_t *)w.col_slot, (const int4 *)w.col_mode, s.nslots, (const double *)w.mode_w, w.rho,
             (KM *)w.kmode, w.col_coef);
    return hipGetLastError();
}

hipError_t launch_col_final(const LaunchCfg &c, const Workspace &w)
{
    return c.prec == RBE_FP64 ? col_final<KModeD>(c, w) : col_final<KModeF>(c, w);
}

template <typename T>
static hipError_t col_force(const LaunchCfg &c, const Workspace &w, const void *pos, const void *q, void *F, int acc)
{
    const ColumnSet &s = c.cols;
    const dim3 g((unsigned)((c.ntot + s.force_nb - 1) / s.force_nb));
    return launch_lds(s.force_nb == 64 ? k_col_force<T, 64> : k_col_force<T, 32>, g, dim3(256), force_lds(s, s.force_nb), c.stream,
                      col_args(c, w), (const int32_t *)w.col_tile, (const double *)w.col_coef, (const T *)pos,
                      (const T *)q, c.ntot, (T *)F, acc, w.flag);
}

hipError_t launch_col_force(const LaunchCfg &c, const Workspace &w, const void *pos, const void *q, void *force,
                            int accumulate)
{
    return c.prec == RBE_FP64 ? col_force<double>(c, w, pos, q, force, accumulate)
                              : col_force<float>(c, w, pos, q, force, accumulate);
}

}  // namespace rbe

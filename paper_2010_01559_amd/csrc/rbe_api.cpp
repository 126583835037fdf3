// rbe_api.cpp -- host side of librbe: validation, context and workspace
// management, and the C-ABI entry points declared in include/rbe.h.
//
// Paper: Jin, Li, Xu & Zhao, arXiv:2010.01559.
#include <dlfcn.h>
#include <hip/hip_runtime.h>

#include <algorithm>
#include <chrono>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <string>
#include <vector>

#include "rbe.h"
#include "rbe_internal.h"

using namespace rbe;

namespace rbe {
LaunchEvents &launch_events()
{
    thread_local LaunchEvents e;
    return e;
}
}  // namespace rbe

namespace {

// Message of the last failed call that has no context (creation, or the
// no-allocation entry point), in a fixed buffer so that setting it from the
// no-allocation path allocates nothing.
struct NullError {
    char buf[512] = "no error";
    NullError &operator=(const std::string &m) { return *this = m.c_str(); }
    NullError &operator=(const char *m)
    {
        std::snprintf(buf, sizeof buf, "%s", m);
        return *this;
    }
    const char *c_str() const { return buf; }
};
thread_local NullError g_create_error;

void null_errf(const char *f, ...)
{
    va_list ap;
    va_start(ap, f);
    std::vsnprintf(g_create_error.buf, sizeof g_create_error.buf, f, ap);
    va_end(ap);
}

const char *kKernelNames[K_COUNT] = {"sample", "stage",      "mid",        "kforce",   "scatter", "real",
                                     "energy", "vjp_reduce", "vjp_gather", "vjp_real", "misc"};

std::string fmt(const char *f, ...)
{
    char buf[512];
    va_list ap;
    va_start(ap, f);
    vsnprintf(buf, sizeof buf, f, ap);
    va_end(ap);
    return buf;
}

// 1-D factor of the normaliser (Sec. 3.1, eq. 3.2, direct form).
double normaliser_H(double alpha, double L)
{
    const double a = kPi * kPi / (alpha * L * L);
    double h = 1.0;
    for (long m = 1; m < 100000000L; ++m) {
        const double t = std::exp(-a * (double)m * (double)m);
        if (t == 0.0 || t < h * 1e-20) break;
        h += 2.0 * t;
    }
    return h;
}

// Half-width M of the 1-D mode table: the continuous Gaussian of eq. (3.4)
// has standard deviation sqrt(alpha L^2/(2 pi^2)); beyond 10 of them the
// mass is below exp(-50).
int table_half_width(double alpha, double L)
{
    const double sigma = std::sqrt(alpha * L * L / (2.0 * kPi * kPi));
    return (int)std::ceil(10.0 * sigma) + 1;
}

// Cumulative table of the 1-D weights exp(-pi^2 m^2/(alpha L^2)) for
// m = -M..M: running sums from m = -M upwards over the total.
void build_cdf(double alpha, double L, std::vector<double> &out)
{
    const int M = table_half_width(alpha, L);
    const int K = 2 * M + 1;
    const double a = kPi * kPi / (alpha * L * L);
    std::vector<double> w(K);
    for (int k = 0; k < K; ++k) {
        const double m = (double)(k - M);
        w[k] = std::exp(-a * m * m);
    }
    double tot = 0.0;
    for (int k = 0; k < K; ++k) tot += w[k];
    double run = 0.0;
    for (int k = 0; k < K; ++k) {
        run += w[k];
        out.push_back(run / tot);
    }
}

bool finite_pos(double x) { return std::isfinite(x) && x > 0.0; }

// Whether single-precision mode constants take the polar form (see KModeF).  It
// saves every particle-mode term a cosine and two products and costs the totals
// launch 0.5 us (N = 3000, P = 100: 20.2 -> 20.7 us a step), so it takes 2^23
// terms (N = 1e5, P = 100: 37.5 -> 37.2 us; 64 x 20000: 146 -> 142 us; force
// launch at N = 1e6, P = 200: 98 -> 86 us).
int polar_form(int64_t terms, int prec) { return prec == RBE_FP32 && terms >= (1 << 23) ? 1 : 0; }

// The constants of one system that the Fourier passes read: sizes, box,
// splitting, normaliser S = H^3 - 1 (eqs. 3.1-3.2), the mode table bound and
// the single-precision phase split (|m| <= 2M must satisfy |m| < 2^(22 - hi_bits)).
void fourier_constants(const rbe_params &p, SysDev &s)
{
    s.n = p.n;
    s.p = p.p;
    s.M = table_half_width(p.alpha, p.box);
    s.L = p.box;
    s.invL = 1.0 / p.box;
    s.alpha = p.alpha;
    s.beta = std::sqrt(p.alpha);
    s.coulomb = p.coulomb;
    const double H = normaliser_H(p.alpha, p.box);
    s.S = H * H * H - 1.0;
    int bm = 0;
    while ((1 << bm) <= 2 * s.M) ++bm;
    s.hi_bits = std::min(14, 22 - bm);
    s.hi_scale = std::ldexp(1.0f, s.hi_bits);
    s.hi_inv = std::ldexp(1.0f, -s.hi_bits);
}

// The single-precision pair constants from the double ones.
void pair_constants(SysDev &s)
{
    PairConstF &c = s.pair;
    c.rc2 = (float)s.rc2;
    c.lj_rc2 = (float)s.lj_rc2;
    c.beta = (float)s.beta;
    c.nalpha_log2e = (float)(-s.alpha * 1.4426950408889634074);
    c.two_beta_rsqrtpi = (float)(2.0 * s.beta / 1.7724538509055160273);
    c.coulomb = (float)s.coulomb;
    c.lj_sig2 = (float)s.lj_sig2;
    c.eps4 = (float)(4.0 * s.lj_eps);
    c.lj_shift = (float)s.lj_shift;
    c.lj_on = s.lj_on && !s.diam_on;
    c.scale = (float)(s.L * (1.0 / 4294967296.0));
    c.rmax2u = (float)(s.rsearch2 / ((double)c.scale * (double)c.scale));
    c.rsearch2_box = (float)(s.rsearch2 / (s.L * s.L) * (1.0 + 1e-6));
    c.rlist2_box = (float)(s.rlist2 / (s.L * s.L) * (1.0 + 1e-6));
}

// Structure-factor chunk of the calls without a context, and the largest for which
// rbe_reserve_modes leaves room: one (1024-thread) block per compute unit when the
// particles allow.
int default_rho_chunk(int64_t ntot)
{
    return (int)std::min<int64_t>(512, std::max<int64_t>(64, ((ntot + 255) / 256 + 7) / 8 * 8));
}

// Rounds that the busiest of a compute unit's four SIMDs spends on a block's sums over
// P modes: the waves with modes to sum, dealt to the SIMDs in turn, times
// the rounds of a lane (k_stage_rho).  512 threads and 347 modes are one group of
// particles on 6 waves, two on two of the SIMDs; 1024 threads two groups on 11.
int sum_rounds(int chunk, int block, int P, int prec)
{
    const bool two = prec == RBE_FP32 && P >= kRhoTwoModes && chunk >= kRhoTwoChunk;
    const int Pt = std::min(P, block), Pl = two ? (Pt + 1) / 2 : Pt, G = std::min(block / Pl, kRhoGroupsMax);
    const int per = G * (two ? kRhoUnroll / 2 : kRhoUnroll), rounds = (chunk + per - 1) / per;
    int total = 0;
    for (int m0 = 0; m0 < P; m0 += Pt) {
        int simd[4] = {0, 0, 0, 0};
        for (int w = 0; w < block / 64; ++w) {
            bool busy = false;
            for (int t = 64 * w; t < 64 * (w + 1) && !busy; ++t) busy = t / Pl < G && t % Pl < P - m0;
            simd[w & 3] += busy ? 1 : 0;
        }
        total += rounds * *std::max_element(simd, simd + 4);
    }
    return total;
}

// Default structure-factor shape of a context: particles per block, threads of a step's
// block and of a call's.  The step's block integrates its chunk from memory and then
// works on the chunk's sums; 512 threads leave room for a second block (256 threads for
// four more) whose loads run under them.  A call's block only reads its chunk; what it
// gains is waves at work.
// - Up to a block of 512 particles per compute unit, one block each.  A step's 512
//   threads cost less to synchronise than 1024 and cover a 64-particle chunk's
//   terms (N = 1e4 in double precision 32.2 -> 30.8 us a step); 256 do, in calls as well, where the
//   chunk has fewer than 4096 of them (N = 300, P = 10: 21.4 -> 20.4 us), and 1024
//   are better where 512 leave the SIMDs uneven (sum_rounds) or take a second
//   tile of modes for a few (staging and totals launches, N = 1e5 in double precision:
//   P = 171 54 and 47 us, P = 347 92 and 77, P = 256 57 and 58; N = 3e4 in single
//   precision: P = 600 20.1 and 17.3, P = 1934 41 and 36).  Calls take 1024 from 160 modes on
//   and, in double precision, for chunks that are not short (N = 1e5: P = 110 31 and 28, P = 171 55
//   and 41, P = 347 91 and 70).  Steps of
//   all-pairs contexts with few modes take 128 particles at least, so that the force
//   launch forms the totals of twice the system (see totals_in_force; N = 600, P = 60:
//   17.1 -> 13.4 us) from half the tiles (N = 300: 12.3 -> 12.0 us; with 100 modes in double
//   precision the staging launch of a force call is 4 us longer).
// - Beyond, lists of at least 160 modes, whose sums outweigh the loads, and double
//   precision take two blocks of 512 threads per compute unit and round (N = 1e6,
//   P = 200: 331 us a step with 512 particles on 1024 threads, 276 with 984 on
//   512, 285 with 512 on 256), shorter lists three of 256 (N = 1e6, P = 50: 249 and 214 us
//   with 1024 / 512, 201 with 512 / 256; 64 x 20000, P = 100: 177, 152, 146 us).  1024 here, too, where
//   512 are uneven by more than what the second block fills (64 x 6105 in double
//   precision, P = 347: 334 and 284 us) and in calls from 100 modes on (the same call 332 and
//   247), if the chunk leaves them room in the LDS.
void default_rho_shape(int64_t ntot, int max_p, int prec, int all_pairs, int *chunk, int *block, int *call)
{
    const auto per = [&](int64_t blocks) { return (int)(((ntot + blocks - 1) / blocks + 7) / 8 * 8); };
    const auto uneven = [&](double by) {
        return sum_rounds(*chunk, 512, max_p, prec) > by * sum_rounds(*chunk, 1024, max_p, prec);
    };
    if (ntot <= 256 * 512) {
        *chunk = std::max(all_pairs && max_p * (prec == RBE_FP64 ? 4 : 1) <= 64 ? 128 : 64, per(256));
        if ((int64_t)*chunk * max_p < 4096) {
            *block = *call = 256;
        } else {
            *block = max_p > 400 || uneven(1.06) ? 1024 : 512;
            *call = max_p < 160 && (prec == RBE_FP32 || *chunk < 160) ? 512 : 1024;
        }
    } else if (max_p >= 160 || prec == RBE_FP64) {
        *chunk = per(512 * ((ntot + 512 * 1024 - 1) / (512 * 1024)));
        const bool room = *chunk <= 896;   // 1024 threads within 64 KB of LDS
        *block = room && uneven(1.15) ? 1024 : 512;
        *call = room && max_p >= 100 ? 1024 : 512;
    } else {
        *chunk = std::min(512, per(768));
        *block = 256;
        *call = max_p < 100 ? 512 : 1024;
    }
}

// Four waves share a 64-particle tile in the force pass while the tiles alone
// would not fill the chip several times over, two beyond.
int default_force_split(int64_t ntot) { return ntot >= 500000 ? 2 : 4; }

// ---------------------------------------------------------------------------
// Tile cache: shapes picked by rbe_autotune, keyed by device architecture,
// precision, the power-of-two buckets of the total particle count and of the
// largest batch size, and whether the context holds several systems.  It is
// read at the first context creation from $RBE_TUNE_CACHE, or else from
// rbe_tiles.txt beside the library, and consulted by every creation;
// rbe_autotune adds its result and appends it to the file when it can.
// Lines: "arch precision n_bucket p_bucket batched rho_chunk rho_block
// force_split real_split"; '#' starts a comment.
// ---------------------------------------------------------------------------
struct TuneKey {
    std::string arch;
    int prec, nb, pb, batched;
    bool operator<(const TuneKey &o) const
    {
        if (arch != o.arch) return arch < o.arch;
        if (prec != o.prec) return prec < o.prec;
        if (nb != o.nb) return nb < o.nb;
        if (pb != o.pb) return pb < o.pb;
        return batched < o.batched;
    }
};

struct TuneCache {
    std::mutex mu;
    bool loaded = false;
    bool persist = false;   // rbe_autotune appends to the file (only one named by RBE_TUNE_CACHE)
    std::string path;
    std::map<TuneKey, rbe_tiles> m;
};

TuneCache &tune_cache()
{
    static TuneCache t;
    return t;
}

int log2_bucket(int64_t v)
{
    int b = 0;
    while (v > 1) {
        v >>= 1;
        ++b;
    }
    return b;
}

// The architecture name without its feature suffixes ("gfx950:sramecc+" -> "gfx950").
TuneKey tune_key(const char *arch, int prec, int64_t ntot, int max_p, int R)
{
    std::string a = arch;
    const size_t colon = a.find(':');
    if (colon != std::string::npos) a.resize(colon);
    return TuneKey{a, prec, log2_bucket(ntot), log2_bucket(max_p), R > 1 ? 1 : 0};
}

void tune_load_locked(TuneCache &t)
{
    if (t.loaded) return;
    t.loaded = true;
    if (const char *env = std::getenv("RBE_TUNE_CACHE")) {
        t.path = env;
        t.persist = true;
    } else {
        Dl_info info;
        if (dladdr((void *)&tune_cache, &info) && info.dli_fname) {
            std::string lib = info.dli_fname;
            const size_t slash = lib.rfind('/');
            t.path = (slash == std::string::npos ? std::string(".") : lib.substr(0, slash)) + "/rbe_tiles.txt";
        }
    }
    FILE *f = t.path.empty() ? nullptr : std::fopen(t.path.c_str(), "r");
    if (!f) return;
    char line[256];
    while (std::fgets(line, sizeof line, f)) {
        if (char *hash = std::strchr(line, '#')) *hash = 0;
        char arch[32];
        TuneKey k;
        rbe_tiles v;
        if (std::sscanf(line, "%31s %d %d %d %d %d %d %d %d", arch, &k.prec, &k.nb, &k.pb, &k.batched, &v.rho_chunk,
                        &v.rho_block, &v.force_split, &v.real_split) == 9) {
            k.arch = arch;
            t.m[k] = v;
        }
    }
    std::fclose(f);
}

bool tune_lookup(const TuneKey &k, rbe_tiles *out)
{
    TuneCache &t = tune_cache();
    std::lock_guard<std::mutex> lock(t.mu);
    tune_load_locked(t);
    auto it = t.m.find(k);
    if (it == t.m.end()) return false;
    *out = it->second;
    return true;
}

void tune_store(const TuneKey &k, const rbe_tiles &v)
{
    TuneCache &t = tune_cache();
    std::lock_guard<std::mutex> lock(t.mu);
    tune_load_locked(t);
    t.m[k] = v;
    if (!t.persist || t.path.empty()) return;
    if (FILE *f = std::fopen(t.path.c_str(), "a")) {
        std::fprintf(f, "%s %d %d %d %d %d %d %d %d\n", k.arch.c_str(), k.prec, k.nb, k.pb, k.batched, v.rho_chunk,
                     v.rho_block, v.force_split, v.real_split);
        std::fclose(f);
    }
}

// Whether a tile shape fits the kernels' dynamic LDS, 64 KB as the staging kernel is
// launched: 32 bytes per particle (plus 256 padding records) and 28 per thread (its
// table falls back to global memory when it does not fit).  The adjoint reduction stages
// 48 bytes per particle, 56 in double precision, and 16 per thread; its launch takes more
// than 64 KB where double precision needs it (launch_lds; at most 74 KB of the 160 here).
bool tiles_fit(const rbe_tiles &n)
{
    return n.rho_chunk >= 64 && n.rho_chunk <= 2048 && n.rho_chunk % 8 == 0 &&
           (n.rho_block == 256 || n.rho_block == 512 || n.rho_block == 1024) &&
           (n.force_split == 1 || n.force_split == 2 || n.force_split == 4) &&
           (n.real_split == 1 || n.real_split == 2 || n.real_split == 4 || n.real_split == 8) &&
           48 * (size_t)n.rho_chunk + 16 * (size_t)n.rho_block <= 64 * 1024 &&
           32 * ((size_t)n.rho_chunk + 256) + 28 * (size_t)n.rho_block <= 64 * 1024;
}

// Largest centre distance at which the shifted LJ of eq. (4.1) still acts:
// R_c without diameters (r_off = 0), else r_off + R_c of the pair of the two
// largest diameters, r_off = (d_i + d_j)/2 - sigma.
double lj_reach(const rbe_params &p)
{
    if (!p.diameter || p.n < 2) return p.lj_rcut;
    double d1 = -1e300, d2 = -1e300;
    for (int i = 0; i < p.n; ++i) {
        const double d = p.diameter[i];
        if (d > d1) {
            d2 = d1;
            d1 = d;
        } else if (d > d2) {
            d2 = d;
        }
    }
    return 0.5 * (d1 + d2) - p.lj_sigma + p.lj_rcut;
}

rbe_status validate(const rbe_params &p, std::string &err)
{
    if (p.n < 1) return err = fmt("n must be >= 1 (got %d)", p.n), RBE_ERR_INVALID;
    if (p.p < 1) return err = fmt("p must be >= 1 (got %d)", p.p), RBE_ERR_INVALID;
    if (!finite_pos(p.box)) return err = "box must be finite and > 0", RBE_ERR_INVALID;
    if (!finite_pos(p.alpha)) return err = "alpha must be finite and > 0", RBE_ERR_INVALID;
    if (!finite_pos(p.r_cut)) return err = "r_cut must be finite and > 0", RBE_ERR_INVALID;
    if (!std::isfinite(p.coulomb)) return err = "coulomb must be finite", RBE_ERR_INVALID;
    if (p.r_cut > 0.5 * p.box)
        return err = fmt("r_cut %.6g exceeds half the box %.6g (minimum image)", p.r_cut, 0.5 * p.box),
               RBE_ERR_CUTOFF;
    if (!std::isfinite(p.lj_eps) || p.lj_eps < 0.0) return err = "lj_eps must be finite and >= 0", RBE_ERR_INVALID;
    if (p.diameter)
        for (int i = 0; i < p.n; ++i)
            if (!finite_pos(p.diameter[i])) return err = fmt("diameter[%d] must be finite and > 0", i), RBE_ERR_INVALID;
    if (p.lj_eps > 0.0) {
        if (!finite_pos(p.lj_sigma) || !finite_pos(p.lj_rcut))
            return err = "lj_sigma and lj_rcut must be finite and > 0 when lj_eps > 0", RBE_ERR_INVALID;
        if (lj_reach(p) > 0.5 * p.box)
            return err = fmt("the LJ reach r_off + lj_rcut = %.6g exceeds half the box", lj_reach(p)), RBE_ERR_CUTOFF;
    }
    if (p.n_fixed < 0 || p.n_fixed > p.n) return err = fmt("n_fixed must be in [0, n] (got %d)", p.n_fixed), RBE_ERR_INVALID;
    if (p.reserved != 0) return err = "reserved must be 0", RBE_ERR_INVALID;
    if (!std::isfinite(p.kT) || p.kT < 0.0) return err = "kT must be finite and >= 0", RBE_ERR_INVALID;
    if (!std::isfinite(p.gamma) || p.gamma < 0.0) return err = "gamma must be finite and >= 0", RBE_ERR_INVALID;
    if (!std::isfinite(p.dt) || p.dt < 0.0) return err = "dt must be finite and >= 0", RBE_ERR_INVALID;
    if (!finite_pos(p.mass)) return err = "mass must be finite and > 0", RBE_ERR_INVALID;
    if (!std::isfinite(p.nu) || p.nu < 0.0) return err = "nu must be finite and >= 0", RBE_ERR_INVALID;
    if (!std::isfinite(p.skin) || p.skin < 0.0) return err = "skin must be finite and >= 0", RBE_ERR_INVALID;
    if (p.precision != RBE_FP32 && p.precision != RBE_FP64) return err = "unknown precision", RBE_ERR_INVALID;
    if (p.integrator != RBE_LANGEVIN_BAOAB && p.integrator != RBE_LEAPFROG_ANDERSEN)
        return err = "unknown integrator", RBE_ERR_INVALID;
    if (p.sampler != RBE_SAMPLER_EXACT && p.sampler != RBE_SAMPLER_MH && p.sampler != RBE_SAMPLER_FIXED)
        return err = "unknown sampler", RBE_ERR_INVALID;
    if (p.flags != 0) return err = "flags must be 0", RBE_ERR_INVALID;
    const double H = normaliser_H(p.alpha, p.box);
    if (1.0 / (H * H * H) > 0.5)
        return err = fmt("alpha L^2 = %.3g is too small: the zero mode would carry most of the mass",
                         p.alpha * p.box * p.box),
               RBE_ERR_INVALID;
    if (table_half_width(p.alpha, p.box) > (1 << 20)) return err = "alpha L^2 too large for the mode table", RBE_ERR_INVALID;
    if (p.precision == RBE_FP32 && table_half_width(p.alpha, p.box) > 4095)
        return err = fmt("alpha L^2 = %.3g needs modes beyond |m| = 8191, past the single-precision phase "
                         "split; use RBE_FP64", p.alpha * p.box * p.box),
               RBE_ERR_INVALID;
    return RBE_OK;
}

}  // namespace

struct rbe_ctx {
    int R = 0;
    int prec = RBE_FP32;
    int device = 0;
    std::string arch;               // gcnArchName of the device
    bool tiles_from_cache = false;  // creation took its tile shapes from the tile cache
    hipStream_t stream = nullptr;
    std::vector<rbe_params> prm;
    std::vector<SysDev> sysh;
    std::vector<int> ntiles_rho;   // per system
    int64_t ntot = 0;
    int mtot = 0;                  // active modes in total
    int mcap = 0;                  // capacity of the mode arrays
    int max_p = 0;
    bool modes_valid = false;
    bool list_valid = false;       // the neighbour list matches the cell order in `sorted`
    uint64_t list_gen = 0;         // steps taken in list mode (selects the rebuild flag)
    bool any_mh = false;
    bool fixed = false;            // rbe_step keeps the active mode list
    // rbe_sample_k with the exact sampler only records the draw; the next
    // structure-factor launch draws the modes itself (or a sampling launch
    // runs first where that launch cannot)
    bool sample_pending = false;
    uint64_t sample_step = 0;
    // The active modes are the exact sample of step cur_step (cur_drawn), and
    // the totals launch of a force call draws the sample of cur_step + 1 into
    // the alternate mode arrays (next_ready, next_step), so that an
    // rbe_sample_k for that step only swaps the arrays.
    bool cur_drawn = false;
    uint64_t cur_step = 0;
    bool next_ready = false;
    uint64_t next_step = 0;
    LaunchCfg cfg{};
    Workspace w{};
    size_t partial_cap = 0;        // doubles allocated for partial
    bool lanes_set = false;        // rbe_set_tiles gave real_split
    bool shape_set = false;        // the structure-factor shape comes from rbe_set_tiles or the tile cache
    int mean_list = 0;             // expected neighbours of a list particle (largest system)
    void *col_mem = nullptr;       // buffers of a dense mode list (one of allocs)
    size_t col_bytes = 0;
    std::vector<void *> allocs;
    std::string err = "no error";
    // profiling
    bool prof = false;
    struct Pend {
        int id;
        hipEvent_t a, b;
    };
    std::vector<Pend> pend;
    std::vector<hipEvent_t> pool;
    double prof_ms[K_COUNT] = {};
    int64_t prof_n[K_COUNT] = {};
    // host staging
    double *energy_h = nullptr;    // pinned: kEnergyOut sums per system, then the error word (first energy call)
    // graphs of steady-state list steps, keyed by everything their
    // kernel arguments were taken from
    bool graphs = false;
    hipStream_t cap_stream = nullptr;
    struct StepGraph {
        hipGraphExec_t exec = nullptr;
        LaunchCfg cfg{};
        Workspace w{};
        const void *pos, *vel, *q, *force;
        int par;
        bool andersen;
        uint64_t used;
    };
    std::vector<StepGraph> step_graphs;
    uint64_t graph_clock = 0;
};

namespace {

rbe_status set_err(rbe_ctx *c, rbe_status st, const std::string &m)
{
    if (c) c->err = m;
    return st;
}

rbe_status hip_fail(rbe_ctx *c, hipError_t e, const char *what)
{
    return set_err(c, RBE_ERR_HIP, fmt("%s: %s", what, hipGetErrorString(e)));
}

#define HIPCHK(ctx, call)                                    \
    do {                                                     \
        hipError_t e_ = (call);                              \
        if (e_ != hipSuccess) return hip_fail(ctx, e_, #call); \
    } while (0)

template <typename F>
rbe_status run(rbe_ctx *c, int id, F &&f)
{
    if (c->prof) {
        hipEvent_t a, b;
        if (c->pool.size() >= 2) {
            a = c->pool.back();
            c->pool.pop_back();
            b = c->pool.back();
            c->pool.pop_back();
        } else {
            HIPCHK(c, hipEventCreate(&a));
            HIPCHK(c, hipEventCreate(&b));
        }
        // the launches of f record a and b themselves (launch_k)
        LaunchEvents &le = launch_events();
        le = LaunchEvents{a, b, false};
        hipError_t e = f();
        const bool launched = le.started;
        le = LaunchEvents{};
        if (e != hipSuccess) return hip_fail(c, e, kKernelNames[id]);
        if (!launched) {
            c->pool.push_back(a);
            c->pool.push_back(b);
            return RBE_OK;
        }
        c->pend.push_back({id, a, b});
        if (c->pend.size() > 4096) {
            HIPCHK(c, hipStreamSynchronize(c->stream));
            for (auto &p : c->pend) {
                float ms = 0.f;
                (void)hipEventElapsedTime(&ms, p.a, p.b);
                c->prof_ms[p.id] += ms;
                c->prof_n[p.id] += 1;
                c->pool.push_back(p.a);
                c->pool.push_back(p.b);
            }
            c->pend.clear();
        }
        return RBE_OK;
    }
    hipError_t e = f();
    if (e != hipSuccess) return hip_fail(c, e, kKernelNames[id]);
    return RBE_OK;
}

#define RUN(ctx, id, expr)                                       \
    do {                                                         \
        rbe_status s_ = run(ctx, id, [&]() { return (expr); }); \
        if (s_ != RBE_OK) return s_;                             \
    } while (0)

template <typename T>
rbe_status dalloc(rbe_ctx *c, T **p, size_t bytes)
{
    if (bytes == 0) bytes = 16;
    void *q = nullptr;
    hipError_t e = hipMalloc(&q, bytes);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return set_err(c, RBE_ERR_OOM, fmt("hipMalloc of %zu bytes failed: %s", bytes, hipGetErrorString(e)));
    }
    c->allocs.push_back(q);
    *p = (T *)q;
    return RBE_OK;
}

void drop_graphs(rbe_ctx *c)
{
    for (auto &g : c->step_graphs) (void)hipGraphExecDestroy(g.exec);
    c->step_graphs.clear();
}

void free_all(rbe_ctx *c)
{
    drop_graphs(c);
    if (c->cap_stream) (void)hipStreamDestroy(c->cap_stream);
    c->cap_stream = nullptr;
    for (void *p : c->allocs) (void)hipFree(p);
    c->allocs.clear();
    if (c->energy_h) (void)hipHostFree(c->energy_h);
    c->energy_h = nullptr;
}

// Structure-factor tiles for the current chunk size, their partial offsets
// (in (C,S) pairs) and per-system tile counts.
void build_rho_tiles(rbe_ctx *c, std::vector<Tile> &tiles, std::vector<int32_t> &poff, int chunk, int pcap_of_sys0)
{
    tiles.clear();
    poff.assign(2 * c->R, 0);
    c->ntiles_rho.assign(c->R, 0);
    int64_t run = 0;
    for (int r = 0; r < c->R; ++r) {
        const int n = c->sysh[r].n;
        const int nt = (n + chunk - 1) / chunk;
        c->ntiles_rho[r] = nt;
        poff[r] = (int32_t)run;
        poff[c->R + r] = nt;
        for (int k = 0; k < nt; ++k) tiles.push_back(Tile{r, k * chunk, std::min(chunk, n - k * chunk), k});
        const int pc = (c->R == 1) ? pcap_of_sys0 : c->sysh[r].p;
        run += (int64_t)nt * pc;
    }
}

// Doubles held for partial sums: two per row (a tile's mode) for the structure
// factor, and four for the adjoint, which takes long lists of a single system in
// slices of the modes.  `twice` holds all of them at once; in any case a slice of one
// mode fits at the smallest chunk (tiles64 tiles of 64 particles).
size_t partial_room(int64_t rows, int64_t tiles64, bool twice)
{
    return (size_t)std::max<int64_t>(2 * rows * (twice ? 2 : 1), 4 * tiles64);
}

// Slices of an adjoint over `modes` modes whose partials fit `room` doubles (0: none do).
int vjp_slices(int64_t tiles, int modes, size_t room)
{
    if (4 * tiles > (int64_t)room) return 0;
    int k = 1;
    while (4 * tiles * ((modes + k - 1) / k) > (int64_t)room) ++k;
    return k;
}

// Whether a context of R systems and ntot particles holds the adjoint's sums of all modes:
// the chunks of a large single system are at least twice 64, unless the caller sets them.
bool partial_twice(int R, int64_t ntot) { return R > 1 || ntot < 65536; }

int64_t tiles64(const rbe_ctx *c)
{
    int64_t t = 0;
    for (const SysDev &s : c->sysh) t += (s.n + 63) / 64;
    return t;
}

size_t partial_need(rbe_ctx *c, int chunk)
{
    int64_t run = 0;
    for (int r = 0; r < c->R; ++r) {
        const int nt = (c->sysh[r].n + chunk - 1) / chunk;
        const int pc = (c->R == 1) ? c->mcap : c->sysh[r].p;
        run += (int64_t)nt * pc;
    }
    return (size_t)run * 2;
}

// Real-space tiles: runs of real_rows_per_tile() cell-sorted slots for systems with at least
// three cells per side (aux = 0), runs of real_allpairs_per_tile() particles in
// original order for the all-pairs systems (aux = 1).
void build_real_tiles(rbe_ctx *c, std::vector<Tile> &out)
{
    out.clear();
    for (int r = 0; r < c->R; ++r) {
        const SysDev &s = c->sysh[r];
        const int aux = s.nc == 1 ? 1 : 0;
        const int step = aux ? real_allpairs_per_tile() : real_rows_per_tile();
        for (int k = 0; k < s.n; k += step) out.push_back(Tile{r, k, std::min(step, s.n - k), aux});
    }
}

// Whether the force and energy calls of a context take the cell pass of sparse systems
// (sparse_body): cells of one radius with few particles each, in every system.  The
// lines (launch times by waves / here, us): up to 1000 particles the rows of cells are
// short, and the pass by waves needs many (N = 300 with 4.7 a cell 11.8 / 8.2, 64 systems
// of 130 with 4.8 14.9 / 9.8, N = 300 with 11 a cell 13.3 / 18.0; in double precision
// N = 300 with 4.7 16.1 / 15.6 and 11 a cell 18 / 31); beyond, with the chip to fill,
// N = 4000 with 3.0 8.2 / 7.3 and 5.5 8.0 / 8.3, N = 4e4 with 2.0 12.7 / 11.6 and 3.3
// 14 / 14.3, N = 1.5e5 with 1.0 23 / 20.5 and 2.0 24 / 29.5; double precision,
// whose tests are dearer, N = 1.2e4 with 1.1 9.4 / 7.8 and 2.1 10.2 / 11.2, N = 1.5e5
// with 0.5 39 / 27 and 1.0 41 / 43.
bool sparse_pass(const rbe_ctx *c)
{
    const bool fp64 = c->prec == RBE_FP64;
    bool any = false;
    for (const SysDev &s : c->sysh) {
        if (s.nc == 1) continue;
        double most = fp64 ? 5.0 : 6.5;
        if (s.n >= 1000) {
            if (fp64)
                most = c->ntot < 65536 ? 1.5 : 0.8;
            else
                most = c->ntot < 16384 ? 4.0 : (c->ntot < 65536 ? 2.5 : 1.5);
        }
        if (s.nh != 1 || s.n > most * s.ncell) return false;
        any = true;
    }
    return any;
}

// List-pass tiles: runs of 256/LPP cell-sorted slots (aux = 2) for list
// systems, all-pairs runs (aux = 1) for one-cell systems.
void build_list_tiles(rbe_ctx *c, int lpp, std::vector<Tile> &out)
{
    out.clear();
    for (int r = 0; r < c->R; ++r) {
        const SysDev &s = c->sysh[r];
        const int aux = s.nc == 1 ? 1 : 2;
        const int step = aux == 1 ? real_allpairs_per_tile() : 256 / lpp;
        for (int k = 0; k < s.n; k += step) out.push_back(Tile{r, k, std::min(step, s.n - k), aux});
    }
}

// Lanes per particle of the list pass.  real_split as the caller set it; the
// default of 4 becomes 8, 16 or 32 while that would leave compute units without a
// block and the lists are longer than the lanes: the launch then lasts as long as
// one lane's chain of list rounds (N = 3101, lists of 217: 36 us with 4 lanes,
// 12 us with 32).  The chains of double precision are ten times as long and
// worth more lanes a little beyond, up to 640 blocks (N = 10001 with 16 instead of 8
// 29.6 -> 28.6 us a step, N = 20000 with 8 instead of 4 36.0 -> 34.5; N = 14000 with 16, 875
// blocks, 30.2 -> 32.0; single precision at N = 18000 with 8, 562 blocks, 20.8 -> 22.0).
// The sums over a particle's list are exact in single
// precision, so the lanes do not change them.
int default_lanes(int prec, int64_t ntot, int mean_list)
{
    int lanes = 4;
    const int64_t blocks = prec == RBE_FP64 ? 321 : 256;
    while (lanes < 32 && ntot * lanes / 256 < blocks && 2 * lanes <= mean_list) lanes *= 2;
    return lanes;
}

int list_lanes(const rbe_ctx *c)
{
    const int lanes = c->cfg.real_split;
    return c->lanes_set || lanes != 4 ? lanes : default_lanes(c->prec, c->ntot, c->mean_list);
}

// Tiles of one system of n particles in the list pass (see build_list_tiles).
int64_t list_tiles(int n, bool one_cell, int lanes)
{
    const int step = one_cell ? real_allpairs_per_tile() : 256 / lanes;
    return ((int64_t)n + step - 1) / step;
}

// Room for the list tiles of a context: up to 8 lanes as a caller sets them, or the default.
int64_t list_tile_room(const rbe_ctx *c)
{
    const int lanes = std::max(8, default_lanes(c->prec, c->ntot, c->mean_list));
    int64_t n = 0;
    for (const SysDev &s : c->sysh) n += list_tiles(s.n, s.nc == 1, lanes);
    return n;
}

rbe_status upload_list_tiles(rbe_ctx *c)
{
    if (!c->cfg.list_on) return RBE_OK;
    std::vector<Tile> lt;
    c->cfg.list_lanes = list_lanes(c);
    build_list_tiles(c, c->cfg.list_lanes, lt);
    if ((int64_t)lt.size() > list_tile_room(c)) return set_err(c, RBE_ERR_STATE, "no room for the list tiles");
    c->cfg.n_list_tiles = (int)lt.size();
    HIPCHK(c, hipMemcpy(c->w.list_tiles, lt.data(), lt.size() * sizeof(Tile), hipMemcpyHostToDevice));
    return RBE_OK;
}

rbe_status upload_rho_tiles(rbe_ctx *c)
{
    std::vector<Tile> tiles;
    std::vector<int32_t> poff;
    build_rho_tiles(c, tiles, poff, c->cfg.rho_chunk, c->mcap);
    c->cfg.n_rho_tiles = (int)tiles.size();
    c->cfg.max_sys_rho_tiles = 0;
    for (int nt : c->ntiles_rho) c->cfg.max_sys_rho_tiles = std::max(c->cfg.max_sys_rho_tiles, nt);
    HIPCHK(c, hipMemcpy(c->w.rho_tiles, tiles.data(), tiles.size() * sizeof(Tile), hipMemcpyHostToDevice));
    HIPCHK(c, hipMemcpy(c->w.partial_off, poff.data(), poff.size() * sizeof(int32_t), hipMemcpyHostToDevice));
    return RBE_OK;
}

// By the modes in use, which rbe_set_k and the draws after it change: a call
// without a context (rbe_kspace_forces_noalloc) goes by its own list.
void set_polar(rbe_ctx *c)
{
    int64_t terms = 0;
    for (const SysDev &s : c->sysh) terms += (int64_t)s.n * s.p;
    for (SysDev &s : c->sysh) s.polar = polar_form(terms, c->prec);
}

rbe_status upload_sys(rbe_ctx *c)
{
    set_polar(c);
    HIPCHK(c, hipStreamSynchronize(c->stream));
    HIPCHK(c, hipMemcpy(c->w.sys, c->sysh.data(), c->sysh.size() * sizeof(SysDev), hipMemcpyHostToDevice));
    return RBE_OK;
}

// The default structure-factor shape follows the modes in use, which rbe_set_k and the
// draws after it change (a long list on a shape for few modes: 98 -> 112 us a
// step at N = 30000 with 1934 modes on a context of ten).
void refresh_shape(rbe_ctx *c)
{
    if (c->shape_set) return;
    int chunk, block, call;
    default_rho_shape(c->ntot, c->max_p, c->prec, c->cfg.all_pairs, &chunk, &block, &call);
    if (partial_need(c, chunk) > c->partial_cap) return;
    c->cfg.rho_chunk = chunk;
    c->cfg.rho_block = block;
    c->cfg.call_block = call;
}

void refresh_cfg_modes(rbe_ctx *c)
{
    c->mtot = 0;
    c->max_p = 0;
    for (auto &s : c->sysh) {
        c->mtot += s.p;
        c->max_p = std::max(c->max_p, s.p);
    }
    c->cfg.max_p = c->max_p;
    c->cfg.mcap = c->mcap;
    refresh_shape(c);
}

bool check_device_ptr(const void *p) { return p != nullptr; }

// Columns of a mode list (see rbe_columns.hip): worth it when at least half of
// the columns' slots are listed (a random batch fills few; its lists keep the
// sums by mode).  The set has ncols = 0 for any other list.
struct ColumnLists {
    ColumnSet set{};
    std::vector<ColumnDev> cols;
    std::vector<int32_t> slot_col, slot_mode, tiles;
    size_t coef = 0;   // doubles of the coefficient matrix
};

constexpr int kColumnMinModes = 512;
constexpr int kColumnMaxM = 128;

// Whether D column slots beat nm modes summed one by one for n particles (force
// call, us by mode and by columns; a whole list has D = nm / 2).
// - Few particles leave the columns a chain of table, product and tile that grows with the
//   list, 23 us and 4 us per 1000 modes, while the sums by mode are split over the chip.
//   Single precision, up to 3500 particles: N = 1000, 2968 modes 40.7 / 36.5, 4168 modes
//   40.6 / 41.7, 33400 modes 85 / 154; N = 3000, 7808 modes 57.6 / 60.4; N = 5000, 33400
//   modes 269 / 177.  Double precision: N = 300, 16662 modes 106 / 93, 33400 modes
//   141 / 156; N = 1000, 33400 modes 181 / 154.
// - Many particles make single precision's sums by mode cheap for short lists, as the
//   columns tabulate every particle's factors whatever the list: N = 30000, 514 modes
//   34 / 54, 1044 modes 50 / 55, 1934 modes 79 / 61, N = 1e5 65 / 107, 123 / 133,
//   196 / 155; N = 5000, 618 modes 27.5 / 27.1.  By these, .032 us a mode against
//   36 + .01 a slot.
bool columns_pay(int prec, int64_t n, int nm, int64_t D)
{
    if (prec == RBE_FP64) return n >= 512 || 2 * D <= 24576;
    if (n < 3500) return 2 * D <= 4096;
    return n <= 6000 || 10 * (int64_t)nm - 3 * D > 11000;
}

void build_columns(const int32_t *modes, int nm, int64_t n, int prec, size_t room, ColumnLists &out)
{
    if (nm <= kColumnMinModes) return;
    const int32_t *X = modes, *Y = modes + nm, *Z = modes + 2 * (size_t)nm;
    int R = 0;
    for (int l = 0; l < nm; ++l) {
        // (before any absolute value: that of -2^31 is undefined)
        const int lo = std::min(X[l], std::min(Y[l], Z[l])), hi = std::max(X[l], std::max(Y[l], Z[l]));
        if (lo < -kColumnMaxM || hi > kColumnMaxM) return;
        R = std::max(R, std::max(std::abs(X[l]), std::abs(Y[l])));
    }
    // of the columns (m_x, m_y) and -(m_x, m_y) the first is the one with m_x > 0, or
    // m_x = 0 and m_y >= 0
    const int W = 2 * R + 1;
    std::vector<int32_t> zmax((size_t)(R + 1) * W, -1), id((size_t)(R + 1) * W, -1);
    auto flip = [&](int l) { return X[l] < 0 || (X[l] == 0 && Y[l] < 0); };
    auto cell = [&](int l) { return (size_t)std::abs(X[l]) * W + (flip(l) ? -Y[l] : Y[l]) + R; };
    for (int l = 0; l < nm; ++l) zmax[cell(l)] = std::max(zmax[cell(l)], std::abs(Z[l]));
    int64_t D = 0;
    std::vector<ColumnDev> &cols = out.cols;
    for (int a = 0; a <= R; ++a)
        for (int b = -R; b <= R; ++b) {
            const int z = zmax[(size_t)a * W + b + R];
            if (z < 0) continue;
            cols.push_back(ColumnDev{a, b, z, 0, 0, 0});
            D += 2 * z + 1;
        }
    if (D > nm || !columns_pay(prec, n, nm, D)) return;   // a full set of columns and their negatives lists about 2 D modes
    std::stable_sort(cols.begin(), cols.end(), [](const ColumnDev &p, const ColumnDev &q) { return p.Z > q.Z; });
    ColumnSet s{};
    s.ncols = (int)cols.size();
    s.Rx = s.Ry = R;
    s.Zm = cols[0].Z;
    s.D = (int)D;
    int base = 0, slot = 0;
    for (int c = 0; c < s.ncols; ++c) {
        ColumnDev &k = cols[c];
        if (c % 4 == 0) {
            // a tile of four columns has the rows of its longest, in fours
            const int rows = (2 * k.Z + 1 + 3) & ~3;
            out.tiles.push_back(rows);
            out.tiles.push_back((int32_t)out.coef);
            out.coef += 16 * (size_t)rows;
        }
        k.base = base;
        k.slot = slot;
        k.coef = out.tiles[2 * (c / 4) + 1] + 4 * (c % 4);
        id[(size_t)k.mx * W + k.my + R] = c;
        for (int z = 0; z <= k.Z; ++z) out.slot_col.push_back(c);
        base += 2 * k.Z + 1;
        slot += k.Z + 1;
    }
    s.nslots = slot;
    if (out.coef > (size_t)1 << 30) return;
    out.slot_mode.assign(4 * (size_t)slot, -1);
    for (int l = 0; l < nm; ++l) {
        const bool f = flip(l);
        const int z = f ? -Z[l] : Z[l];
        int32_t &e = out.slot_mode[4 * (size_t)(cols[id[cell(l)]].slot + std::abs(z)) + (f ? 2 : 0) + (z < 0 ? 1 : 0)];
        if (e >= 0) return;   // a mode listed twice
        e = l;
    }
    if (!column_shapes(s, n, room)) return;
    out.set = s;
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

rbe_status rbe_normalizer(double alpha, double box, double *H, double *S)
{
    if (!finite_pos(alpha) || !finite_pos(box) || !H || !S) return RBE_ERR_INVALID;
    const double h = normaliser_H(alpha, box);
    *H = h;
    *S = h * h * h - 1.0;
    return RBE_OK;
}

const char *rbe_last_error(const rbe_ctx *ctx)
{
    if (!ctx) return g_create_error.c_str();
    return ctx->err.c_str();
}

int32_t rbe_num_systems(const rbe_ctx *ctx) { return ctx ? ctx->R : 0; }
int64_t rbe_num_particles(const rbe_ctx *ctx) { return ctx ? ctx->ntot : 0; }
int32_t rbe_num_modes(const rbe_ctx *ctx) { return ctx ? ctx->mtot : 0; }

rbe_status rbe_batch_create(const rbe_params *params, int32_t R, void *stream, rbe_ctx **out)
{
    if (out) *out = nullptr;
    if (!params || !out || R < 1) {
        g_create_error = "params and out must be non-NULL and R >= 1";
        return RBE_ERR_INVALID;
    }
    int64_t ntot = 0;
    for (int r = 0; r < R; ++r) {
        std::string e;
        rbe_status st = validate(params[r], e);
        if (st != RBE_OK) {
            g_create_error = fmt("system %d: %s", r, e.c_str());
            return st;
        }
        if (params[r].precision != params[0].precision) {
            g_create_error = "all systems of a batch must share one precision";
            return RBE_ERR_INVALID;
        }
        ntot += params[r].n;
    }
    if (ntot >= (int64_t)1 << 31) {
        g_create_error = "total particle count must be below 2^31";
        return RBE_ERR_INVALID;
    }
    int ndev = 0;
    if (hipGetDeviceCount(&ndev) != hipSuccess || ndev < 1) {
        (void)hipGetLastError();
        g_create_error = "no HIP device available";
        return RBE_ERR_NO_DEVICE;
    }
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        g_create_error = "hipGetDevice failed";
        return RBE_ERR_NO_DEVICE;
    }
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess || std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) {
        g_create_error = fmt("device %d is not gfx950 (%s)", dev, prop.gcnArchName);
        return RBE_ERR_NO_DEVICE;
    }

    rbe_ctx *c = new rbe_ctx();
    c->R = R;
    c->prec = params[0].precision;
    c->device = dev;
    c->stream = (hipStream_t)stream;
    c->prm.assign(params, params + R);
    c->ntot = ntot;

    // ---- per-system constants ----
    std::vector<double> cdf;
    int64_t off = 0;
    int moff = 0, cell_off = 0, max_table = 0;
    bool edge = false;
    // the neighbour list is used only when every system of the batch asks for it
    bool all_skin = true;
    for (int r = 0; r < R; ++r) all_skin = all_skin && params[r].skin > 0.0;
    int kmax = 0;
    bool any_diam = false;
    for (int r = 0; r < R; ++r) {
        const rbe_params &p = params[r];
        SysDev s{};
        fourier_constants(p, s);
        s.off = (int32_t)off;
        s.moff = moff;
        s.cdf_off = (int32_t)cdf.size();
        build_cdf(p.alpha, p.box, cdf);
        const double rmax = std::max(p.r_cut, p.lj_eps > 0.0 ? lj_reach(p) : 0.0);
        const double rlist = rmax + p.skin;
        int nc = (int)std::floor(p.box / rlist);
        s.nh = 1;
        if (nc < 3) {
            nc = 1;   // fewer than 3 cells along the box: one cell, all pairs
        } else {
            // Cells of side radius / nh.  Where a cell of one radius would hold
            // many particles, finer ones keep the candidates of the cell pass
            // close to the search sphere (27 radius^3 against its 4.2 with
            // nh = 1, about 10 with nh = 3); where it holds few, a wave's sixteen
            // particles span several cells anyway and finer ones only add rows.
            const double occ = (double)p.n * std::pow(rlist / p.box, 3.0);
            s.nh = std::min(3, std::max(1, (int)std::cbrt(occ / 6.0)));
            // Pairs at exactly the radius: their r^2 may round to it from either side. The nh
            // finer cells on either side reach 1e-6 beyond it, so that such a pair is found
            // also where it straddles their faces.  Boxes of three radii (to 1e-5) would have
            // five cells with nh = 2, which reach half a box from their middle, where the sign
            // of an offset is a matter of its rounding (cell_pairs needs nc >= 2 nh + 2, or
            // three cells).  They take nh = 3, eight cells, or without a list three cells up
            // to 120 particles in each (real-space call with three and with eight: N = 420
            // 33 and 106 us, N = 2500 113 and 142, N = 4000 170 and 117; 16 systems of 2500 191
            // and 245, of 4000 376 and 325; double precision N = 420 45 and 143, N = 4000 292 and 198).
            const double reach = rlist * (1.0 + 1e-6);
            if (p.box < 3.0 * rlist * (1.0 + 1e-5)) {
                s.nh = occ < 120.0 && !all_skin ? 1 : 3;
                edge |= s.nh == 1;
            }
            nc = std::min((int)std::floor(s.nh * p.box / (s.nh == 1 ? rlist : reach)), 128);
            // a wave takes sixteen particles of one row of cells at a time: at
            // least about eight particles per row of a sparse system
            nc = std::min(nc, std::max(3 * s.nh, (int)std::sqrt(p.n / 8.0)));
        }
        s.nc = nc;
        s.ncell = nc * nc * nc;
        s.cell_off = cell_off;   // kept a multiple of 4 for vector loads of the counts
        s.lj_on = p.lj_eps > 0.0 ? 1 : 0;
        s.integrator = p.integrator;
        s.mh_state_off = 3 * r;
        s.rc2 = p.r_cut * p.r_cut;
        s.lj_eps = p.lj_eps;
        s.lj_sig2 = p.lj_sigma * p.lj_sigma;
        s.lj_rc2 = p.lj_rcut * p.lj_rcut;
        s.lj_sig = p.lj_sigma;
        s.lj_rc = p.lj_rcut;
        s.rsearch2 = rmax * rmax;
        s.n_fixed = p.n_fixed;
        s.diam_on = (p.diameter && s.lj_on) ? 1 : 0;
        any_diam = any_diam || s.diam_on;
        if (s.lj_on) {
            const double sr6 = std::pow(p.lj_sigma / p.lj_rcut, 6.0);
            s.lj_shift = -4.0 * p.lj_eps * (sr6 * sr6 - sr6);
        }
        s.kT = p.kT;
        s.gamma = p.gamma;
        s.dt = p.dt;
        s.mass = p.mass;
        s.c1 = std::exp(-p.gamma * p.dt / p.mass);
        s.c2 = std::sqrt((1.0 - s.c1 * s.c1) * p.kT / p.mass);
        s.nu_dt = p.nu * p.dt;
        s.h_m = 0.5 * p.dt / p.mass;
        s.sv = std::sqrt(p.kT / p.mass);
        s.nu = p.nu;
        s.anneal = 0.0;
        s.seed = p.seed;
        s.use_list = (all_skin && nc >= 3) ? 1 : 0;
        s.rlist2 = rlist * rlist;
        s.half_skin2 = 0.25 * p.skin * p.skin;
        pair_constants(s);
        if (s.use_list) {
            const double dens = (double)p.n / (p.box * p.box * p.box);
            const double mean = dens * 4.0 / 3.0 * kPi * rlist * rlist * rlist;
            kmax = std::max(kmax, (int)std::ceil(1.5 * mean + 32.0));
            c->mean_list = std::max(c->mean_list, (int)mean);
        }
        c->sysh.push_back(s);
        if (p.sampler == RBE_SAMPLER_MH) c->any_mh = true;
        if (p.sampler == RBE_SAMPLER_FIXED) c->fixed = true;
        off += p.n;
        moff += p.p;
        cell_off += (s.ncell + 3) & ~3;
        max_table = std::max(max_table, 2 * s.M + 1);
    }
    set_polar(c);
    if (c->fixed && R != 1) {
        g_create_error = "the fixed sampler needs a single-system context";
        delete c;
        return RBE_ERR_INVALID;
    }
    c->mcap = moff;
    refresh_cfg_modes(c);

    // ---- launch configuration ----
    LaunchCfg &g = c->cfg;
    g.stream = c->stream;
    g.R = R;
    g.prec = c->prec;
    g.ntot = ntot;
    g.mcap = c->mcap;
    g.force_split = default_force_split(ntot);
    g.real_split = 4;
    g.kmax = std::min((kmax + 7) & ~7, 1024);
    g.list_on = 0;
    g.all_pairs = 1;
    for (int r = 0; r < R; ++r) {
        g.list_on |= c->sysh[r].use_list;
        g.all_pairs &= c->sysh[r].nc == 1 ? 1 : 0;
    }
    default_rho_shape(ntot, c->max_p, c->prec, g.all_pairs, &g.rho_chunk, &g.rho_block, &g.call_block);
    g.ncell_tot = cell_off;
    g.max_p = c->max_p;
    g.max_n = 0;
    for (int r = 0; r < R; ++r) g.max_n = std::max(g.max_n, c->sysh[r].n);
    g.cell_edge = edge ? 1 : 0;
    g.max_table = max_table;
    g.wait_limit = kWaitLimit;

    std::vector<Tile> ftiles, ptiles;
    for (int r = 0; r < R; ++r) {
        const int n = c->sysh[r].n;
        for (int k = 0; k < n; k += 64) ftiles.push_back(Tile{r, k, std::min(64, n - k), 0});
        for (int k = 0; k < n; k += 256) ptiles.push_back(Tile{r, k, std::min(256, n - k), 0});
    }
    g.n_force_tiles = (int)ftiles.size();
    g.n_part_tiles = (int)ptiles.size();
    std::vector<Tile> rtiles;
    build_real_tiles(c, rtiles);
    g.n_real_tiles = (int)rtiles.size();

    // wave tiles of force, energy and adjoint calls: eight particles per wave
    // while sixteen would leave most of the chip's 1024 SIMDs with fewer than
    // four waves; the entries of all-pairs systems are fixed, the others are
    // written with each cell list
    g.cell_ppw = ntot < 65536 ? 8 : 16;
    std::vector<Tile> ctiles, rowtiles;
    bool any_pairs = false;
    for (int r = 0; r < R; ++r) any_pairs = any_pairs || c->sysh[r].nc == 1;
    int64_t nct = 0;
    for (int r = 0; r < R; ++r) {
        SysDev &s = c->sysh[r];
        s.ctile_off = (int32_t)nct;
        if (s.nc == 1) {
            for (int k = 0; k < s.n; ++k) ctiles.push_back(Tile{r, k, 1, 1});
            nct += s.n;
        } else {
            const int rows = s.nc * s.nc;
            nct += s.n / g.cell_ppw + rows;
            for (int k = 0; k < rows; k += 256) rowtiles.push_back(Tile{r, k, std::min(256, rows - k), 0});
        }
        // the four waves of a block share one system (and one use of the LDS)
        nct = (nct + 3) & ~(int64_t)3;
        if (any_pairs) ctiles.resize(nct, Tile{r, 0, 0, 0});
    }
    // a context of sparse systems has fixed wave tiles for its force and energy calls
    std::vector<Tile> sptiles;
    if (sparse_pass(c)) {
        for (int r = 0; r < R; ++r) {
            SysDev &s = c->sysh[r];
            s.stile_off = (int32_t)sptiles.size();
            const int step = s.nc == 1 ? 1 : sparse_per_tile();
            for (int k = 0; k < s.n; k += step)
                sptiles.push_back(Tile{r, k, std::min(step, s.n - k), s.nc == 1 ? 1 : 0});
            sptiles.resize((sptiles.size() + 3) & ~(size_t)3, Tile{r, 0, 0, 0});
        }
    }
    g.n_sparse_tiles = (int)sptiles.size();
    g.n_cell_tiles = (int)nct;
    g.n_row_tiles = (int)rowtiles.size();

    // ---- device memory ----
    const size_t esz = c->prec == RBE_FP64 ? 8 : 4;
    const size_t pack_sz = c->prec == RBE_FP64 ? 32 : 16;
    const size_t km_sz = c->prec == RBE_FP64 ? sizeof(KModeD) : sizeof(KModeF);
    const size_t kv_sz = c->prec == RBE_FP64 ? sizeof(KVjpD) : sizeof(KVjpF);
    // the largest rho tile list is the one for the smallest chunk (64)
    const int64_t max_rho_tiles = tiles64(c);
    c->partial_cap = partial_room(partial_need(c, 64) / 2, max_rho_tiles, partial_twice(R, ntot));
    Workspace &w = c->w;
    rbe_status st = RBE_OK;
#define ALLOC(ptr, bytes)                                   \
    do {                                                    \
        if ((st = dalloc(c, &(ptr), (bytes))) != RBE_OK) {  \
            g_create_error = c->err;                        \
            free_all(c);                                    \
            delete c;                                       \
            return st;                                      \
        }                                                   \
    } while (0)
    ALLOC(w.sys, sizeof(SysDev) * R);
    ALLOC(w.rho_tiles, sizeof(Tile) * max_rho_tiles);
    // the tile lists that never change shape: one allocation, one upload
    std::vector<Tile> tiles;
    // (the wave tiles start as zeros, but for the entries of all-pairs systems)
    Tile **const lists[] = {&w.force_tiles, &w.part_tiles, &w.real_tiles, &w.row_tiles, &w.sparse_tiles};
    size_t at[5], nt = 0;
    for (const std::vector<Tile> *v : {&ftiles, &ptiles, &rtiles, &rowtiles, &sptiles}) {
        at[nt++] = tiles.size();
        tiles.insert(tiles.end(), v->begin(), v->end());
    }
    const size_t n_up = tiles.size();
    if (any_pairs) tiles.insert(tiles.end(), ctiles.begin(), ctiles.end());
    Tile *tile_base = nullptr;
    ALLOC(tile_base, sizeof(Tile) * (n_up + (size_t)g.n_cell_tiles));
    for (int k = 0; k < 5; ++k) *lists[k] = tile_base + at[k];
    w.cell_tiles = tile_base + n_up;
    ALLOC(w.modes, sizeof(int32_t) * 3 * c->mcap);
    ALLOC(w.mode_w, sizeof(double) * c->mcap);
    ALLOC(w.partial, sizeof(double) * c->partial_cap);
    ALLOC(w.partial_off, sizeof(int32_t) * 2 * R);
    ALLOC(w.rho, sizeof(double) * 2 * c->mcap);
    ALLOC(w.ab, sizeof(double) * 2 * c->mcap);
    ALLOC(w.kmode, km_sz * c->mcap);
    ALLOC(w.kvjp, kv_sz * c->mcap);
    ALLOC(w.cdf, sizeof(double) * cdf.size());
    ALLOC(w.mh_state, sizeof(int32_t) * 3 * R);
    ALLOC(w.cell_count, sizeof(int32_t) * cell_off);
    ALLOC(w.cell_start, sizeof(int32_t) * (cell_off + R));
    ALLOC(w.cellid, sizeof(int32_t) * ntot);
    ALLOC(w.rank, sizeof(int32_t) * ntot);
    ALLOC(w.sorted_idx, sizeof(int32_t) * ntot);
    ALLOC(w.packed, pack_sz * ntot);
    ALLOC(w.sorted, pack_sz * ntot);
    ALLOC(w.gsorted, 4 * esz * ntot);
    ALLOC(w.modes_alt, sizeof(int32_t) * 3 * c->mcap);
    ALLOC(w.mode_w_alt, sizeof(double) * c->mcap);
    ALLOC(w.energy_part, sizeof(double) * 8 * (size_t)std::max(g.n_cell_tiles, g.n_sparse_tiles));
    ALLOC(w.flag, sizeof(int32_t) * 4);
    ALLOC(w.lflag, sizeof(int32_t) * 8);
    ALLOC(w.step_base, sizeof(uint64_t));
    if (any_diam) {
        ALLOC(w.diam, sizeof(double) * ntot);
        ALLOC(w.dsorted, sizeof(double) * ntot);
    }
    {
        const int64_t nlist = g.list_on ? ntot : 1;
        ALLOC(w.list_tiles, sizeof(Tile) * (g.list_on ? list_tile_room(c) : 1));
        ALLOC(w.slot_of, sizeof(int32_t) * nlist);
        ALLOC(w.ref, pack_sz * nlist);
        ALLOC(w.nbr, sizeof(int32_t) * (g.list_on ? (int64_t)g.kmax * ntot : 1));
        ALLOC(w.nnb, sizeof(int32_t) * nlist);
    }
#undef ALLOC

    auto up = [&](void *dst, const void *src, size_t bytes) -> bool {
        return hipMemcpy(dst, src, bytes, hipMemcpyHostToDevice) == hipSuccess;
    };
    bool ok = up(w.sys, c->sysh.data(), sizeof(SysDev) * R) &&
              up(tile_base, tiles.data(), sizeof(Tile) * tiles.size()) &&
              (any_pairs || hipMemset(w.cell_tiles, 0, sizeof(Tile) * (size_t)g.n_cell_tiles) == hipSuccess) &&
              up(w.cdf, cdf.data(), sizeof(double) * cdf.size()) &&
              hipMemset(w.mh_state, 0, sizeof(int32_t) * 3 * R) == hipSuccess &&
              hipMemset(w.cell_count, 0, sizeof(int32_t) * cell_off) == hipSuccess &&
              hipMemset(w.flag, 0, sizeof(int32_t) * 4) == hipSuccess &&
              hipMemset(w.lflag, 0, sizeof(int32_t) * 8) == hipSuccess &&
              hipMemset(w.cell_start, 0, sizeof(int32_t) * (cell_off + R)) == hipSuccess &&
              hipMemset(w.modes, 0, sizeof(int32_t) * 3 * c->mcap) == hipSuccess;
    if (ok) {
        // every slot names a particle of its own system until the first scatter
        std::vector<int32_t> iota(ntot);
        for (int64_t i = 0; i < ntot; ++i) iota[i] = (int32_t)i;
        ok = up(w.sorted_idx, iota.data(), sizeof(int32_t) * ntot);
    }
    if (ok && any_diam) {
        std::vector<double> d(ntot);
        for (int r = 0; r < R; ++r) {
            const rbe_params &p = params[r];
            for (int i = 0; i < p.n; ++i) d[c->sysh[r].off + i] = p.diameter ? p.diameter[i] : p.lj_sigma;
        }
        ok = up(w.diam, d.data(), sizeof(double) * ntot);
    }
    {
        // shapes from the tile cache, when it holds this configuration
        rbe_tiles t;
        c->arch = prop.gcnArchName;
        if (tune_lookup(tune_key(prop.gcnArchName, c->prec, ntot, c->max_p, R), &t) && tiles_fit(t)) {
            g.rho_chunk = t.rho_chunk;
            g.rho_block = g.call_block = t.rho_block;
            g.force_split = t.force_split;
            g.real_split = t.real_split;
            c->tiles_from_cache = c->shape_set = true;
        }
    }
    if (ok) ok = upload_rho_tiles(c) == RBE_OK;
    if (ok) ok = upload_list_tiles(c) == RBE_OK;
    if (ok && g.list_on) {
        // in-bounds slots and zeroed records until the first build replaces them
        std::vector<int32_t> iota(ntot);
        for (int64_t i = 0; i < ntot; ++i) iota[i] = (int32_t)i;
        ok = up(w.slot_of, iota.data(), sizeof(int32_t) * ntot) &&
             hipMemset(w.ref, 0, pack_sz * ntot) == hipSuccess &&
             hipMemset(w.nnb, 0, sizeof(int32_t) * ntot) == hipSuccess;
    }
    if (ok) ok = hipDeviceSynchronize() == hipSuccess;
    if (!ok) {
        g_create_error = "uploading the context constants failed";
        free_all(c);
        delete c;
        return RBE_ERR_HIP;
    }
    *out = c;
    return RBE_OK;
}

rbe_status rbe_create(const rbe_params *params, void *stream, rbe_ctx **out)
{
    return rbe_batch_create(params, 1, stream, out);
}

void rbe_destroy(rbe_ctx *ctx)
{
    if (!ctx) return;
    (void)hipStreamSynchronize(ctx->stream);
    for (auto &p : ctx->pend) {
        (void)hipEventDestroy(p.a);
        (void)hipEventDestroy(p.b);
    }
    for (auto e : ctx->pool) (void)hipEventDestroy(e);
    free_all(ctx);
    delete ctx;
}

rbe_status rbe_reserve_modes(rbe_ctx *c, int32_t cap)
{
    if (!c) return RBE_ERR_INVALID;
    if (c->R != 1) return set_err(c, RBE_ERR_STATE, "rbe_reserve_modes needs a single-system context");
    if (cap < 1 || cap > (1 << 24)) return set_err(c, RBE_ERR_INVALID, "capacity must be in [1, 2^24]");
    if (cap <= c->mcap) return RBE_OK;
    HIPCHK(c, hipStreamSynchronize(c->stream));
    const size_t km_sz = c->prec == RBE_FP64 ? sizeof(KModeD) : sizeof(KModeF);
    const size_t kv_sz = c->prec == RBE_FP64 ? sizeof(KVjpD) : sizeof(KVjpF);
    // replace the mode-sized buffers
    auto swap_alloc = [&](void **slot, size_t bytes) -> rbe_status {
        void *old = *slot;
        void *nw = nullptr;
        rbe_status s = dalloc(c, &nw, bytes);
        if (s != RBE_OK) return s;
        auto it = std::find(c->allocs.begin(), c->allocs.end(), old);
        if (it != c->allocs.end()) c->allocs.erase(it);
        (void)hipFree(old);
        *slot = nw;
        return RBE_OK;
    };
    drop_graphs(c);
    c->sample_pending = false;
    c->cfg.cols = ColumnSet{};
    c->cur_drawn = c->next_ready = false;
    const int old_cap = c->mcap;
    c->mcap = cap;
    rbe_status s;
    if ((s = swap_alloc((void **)&c->w.modes, sizeof(int32_t) * 3 * cap)) != RBE_OK ||
        (s = swap_alloc((void **)&c->w.mode_w, sizeof(double) * cap)) != RBE_OK ||
        (s = swap_alloc((void **)&c->w.modes_alt, sizeof(int32_t) * 3 * cap)) != RBE_OK ||
        (s = swap_alloc((void **)&c->w.mode_w_alt, sizeof(double) * cap)) != RBE_OK ||
        (s = swap_alloc((void **)&c->w.rho, sizeof(double) * 2 * cap)) != RBE_OK ||
        (s = swap_alloc((void **)&c->w.ab, sizeof(double) * 2 * cap)) != RBE_OK ||
        (s = swap_alloc(&c->w.kmode, km_sz * cap)) != RBE_OK || (s = swap_alloc(&c->w.kvjp, kv_sz * cap)) != RBE_OK) {
        c->mcap = old_cap;
        c->modes_valid = false;
        return s;
    }
    // sized for the smallest of the current chunk, the defaults of short and long lists
    // and that of a block per compute unit (a long list at a smaller one would need
    // tiles x cap partials); rbe_set_tiles refuses smaller chunks afterwards
    int chunk = std::min(c->cfg.rho_chunk, default_rho_chunk(c->ntot));
    for (int p : {1, cap}) {
        int ch, block, call;
        default_rho_shape(c->ntot, p, c->prec, c->cfg.all_pairs, &ch, &block, &call);
        chunk = std::min(chunk, ch);
    }
    c->partial_cap = partial_room(partial_need(c, chunk) / 2, tiles64(c), false);
    if ((s = swap_alloc((void **)&c->w.partial, sizeof(double) * c->partial_cap)) != RBE_OK) return s;
    if (cap > 1024) {
        // partial forces of mode-split force passes
        const size_t esz = c->prec == RBE_FP64 ? sizeof(double) : sizeof(float);
        if ((s = swap_alloc(&c->w.fpart, esz * 3 * (size_t)kMaxModeSplit * c->ntot)) != RBE_OK) return s;
    }
    c->modes_valid = false;
    refresh_cfg_modes(c);
    return upload_rho_tiles(c);
}

rbe_status rbe_sample_k(rbe_ctx *c, uint64_t step, int32_t *modes_out)
{
    if (!c) return RBE_ERR_INVALID;
    bool dirty = false;
    for (int r = 0; r < c->R; ++r)
        if (c->sysh[r].p != c->prm[r].p) {
            c->sysh[r].p = c->prm[r].p;
            dirty = true;
        }
    if (dirty) {
        c->next_ready = false;
        rbe_status s = upload_sys(c);
        if (s != RBE_OK) return s;
        refresh_cfg_modes(c);
        if ((s = upload_rho_tiles(c)) != RBE_OK) return s;
    }
    c->modes_valid = true;
    c->cfg.cols = ColumnSet{};
    c->cur_drawn = !c->any_mh;
    c->cur_step = step;
    if (!c->any_mh && c->next_ready && c->next_step == step) {
        // drawn already by the totals launch of the last force call
        std::swap(c->w.modes, c->w.modes_alt);
        std::swap(c->w.mode_w, c->w.mode_w_alt);
        c->next_ready = false;
        c->sample_pending = false;
    } else if (!c->any_mh && !modes_out) {
        c->sample_pending = true;
        c->sample_step = step;
        return RBE_OK;
    } else {
        c->sample_pending = false;
        RUN(c, K_SAMPLE, launch_sample(c->cfg, c->w, step, c->any_mh ? 1 : 0));
    }
    if (modes_out) {
        for (int d = 0; d < 3; ++d)
            HIPCHK(c, hipMemcpyAsync(modes_out + (size_t)d * c->mtot, c->w.modes + (size_t)d * c->mcap,
                                     sizeof(int32_t) * c->mtot, hipMemcpyDeviceToDevice, c->stream));
    }
    return RBE_OK;
}

// Lays the list out as columns when it is dense.  Their buffers grow with the
// longest such list; where they do not fit in memory the sums by mode stay.
static rbe_status use_columns(rbe_ctx *c, const int32_t *modes, int nm)
{
    ColumnLists cl;
    // the partial sums share the buffer of the sums by mode
    build_columns(modes, nm, c->ntot, c->prec, c->partial_cap, cl);
    if (cl.set.ncols == 0) return RBE_OK;
    auto pad = [](size_t b) { return (b + 255) & ~(size_t)255; };
    const size_t b0 = pad(cl.cols.size() * sizeof(ColumnDev)), b1 = pad(cl.slot_col.size() * 4),
                 b2 = pad(cl.slot_mode.size() * 4), b3 = pad(cl.tiles.size() * 4), b4 = pad(cl.coef * 8);
    const size_t need = b0 + b1 + b2 + b3 + b4;
    if (need > c->col_bytes) {
        void *nw = nullptr;
        const hipError_t e = hipMalloc(&nw, need);
        if (e != hipSuccess) {
            (void)hipGetLastError();
            return RBE_OK;
        }
        auto it = std::find(c->allocs.begin(), c->allocs.end(), c->col_mem);
        if (it != c->allocs.end()) c->allocs.erase(it);
        if (c->col_mem) (void)hipFree(c->col_mem);
        c->col_mem = nw;
        c->col_bytes = need;
        c->allocs.push_back(nw);
    }
    char *base = (char *)c->col_mem;
    std::vector<char> h(b0 + b1 + b2 + b3, 0);
    std::memcpy(h.data(), cl.cols.data(), cl.cols.size() * sizeof(ColumnDev));
    std::memcpy(h.data() + b0, cl.slot_col.data(), cl.slot_col.size() * 4);
    std::memcpy(h.data() + b0 + b1, cl.slot_mode.data(), cl.slot_mode.size() * 4);
    std::memcpy(h.data() + b0 + b1 + b2, cl.tiles.data(), cl.tiles.size() * 4);
    c->w.cols = (ColumnDev *)base;
    c->w.col_slot = (int32_t *)(base + b0);
    c->w.col_mode = (int32_t *)(base + b0 + b1);
    c->w.col_tile = (int32_t *)(base + b0 + b1 + b2);
    c->w.col_coef = (double *)(base + b0 + b1 + b2 + b3);
    HIPCHK(c, hipMemcpy(base, h.data(), h.size(), hipMemcpyHostToDevice));
    HIPCHK(c, hipMemset(c->w.col_coef, 0, cl.coef * 8));   // rows past a column's end stay zero
    HIPCHK(c, hipStreamSynchronize(nullptr));
    c->cfg.cols = cl.set;
    return RBE_OK;
}

rbe_status rbe_set_k(rbe_ctx *c, const int32_t *modes, int32_t nm, const double *weights)
{
    if (!c) return RBE_ERR_INVALID;
    if (c->R != 1) return set_err(c, RBE_ERR_STATE, "rbe_set_k needs a single-system context");
    if (!modes || nm < 1) return set_err(c, RBE_ERR_INVALID, "modes must be non-NULL and nm >= 1");
    if (nm > c->mcap)
        return set_err(c, RBE_ERR_INVALID, fmt("nm = %d exceeds the mode capacity %d (rbe_reserve_modes)", nm, c->mcap));
    std::vector<int32_t> m(3 * (size_t)c->mcap, 0);
    std::vector<double> wv(nm);
    const double S = c->sysh[0].S;
    for (int l = 0; l < nm; ++l) {
        const int32_t a = modes[l], b = modes[nm + l], d = modes[2 * nm + l];
        if (a == 0 && b == 0 && d == 0) return set_err(c, RBE_ERR_INVALID, fmt("mode %d is the zero vector", l));
        m[l] = a;
        m[c->mcap + l] = b;
        m[2 * (size_t)c->mcap + l] = d;
        wv[l] = weights ? weights[l] : S / (double)nm;
        if (!std::isfinite(wv[l])) return set_err(c, RBE_ERR_INVALID, "non-finite weight");
    }
    c->sample_pending = false;
    c->cur_drawn = c->next_ready = false;
    HIPCHK(c, hipStreamSynchronize(c->stream));
    HIPCHK(c, hipMemcpy(c->w.modes, m.data(), sizeof(int32_t) * m.size(), hipMemcpyHostToDevice));
    HIPCHK(c, hipMemcpy(c->w.mode_w, wv.data(), sizeof(double) * nm, hipMemcpyHostToDevice));
    c->cfg.cols = ColumnSet{};
    if (c->sysh[0].p != nm) {
        c->sysh[0].p = nm;
        rbe_status s = upload_sys(c);
        if (s != RBE_OK) return s;
        refresh_cfg_modes(c);
        if ((s = upload_rho_tiles(c)) != RBE_OK) return s;
    }
    c->modes_valid = true;
    return use_columns(c, modes, nm);
}

// ---- classical Ewald mode lists (eq. 2.9, second term, truncated) ----

rbe_status rbe_ewald_radius2(double alpha, double box, double tol, int32_t *mmax2)
{
    if (!finite_pos(alpha) || !finite_pos(box) || !(tol > 0.0 && tol < 1.0) || !mmax2) {
        null_errf("alpha and box must be positive, tol in (0, 1), mmax2 non-NULL");
        return RBE_ERR_INVALID;
    }
    // exp(-pi^2 |m|^2 / (alpha L^2)) >= tol  <=>  |m|^2 <= ln(1/tol) alpha L^2 / pi^2
    const double v = std::log(1.0 / tol) * alpha * box * box / (M_PI * M_PI);
    if (!(v < 2.0e9)) {
        null_errf("the mode radius for alpha = %g, L = %g, tol = %g is beyond 32 bits", alpha, box, tol);
        return RBE_ERR_INVALID;
    }
    *mmax2 = (int32_t)std::floor(v);
    return RBE_OK;
}

rbe_status rbe_ewald_modes(double alpha, double box, int32_t mmax2, int32_t *modes, double *weights, int32_t cap,
                           int32_t *nm)
{
    if (!finite_pos(alpha) || !finite_pos(box) || mmax2 < 1 || !nm) {
        null_errf("alpha and box must be positive, mmax2 >= 1, nm non-NULL");
        return RBE_ERR_INVALID;
    }
    int R = 0;
    while ((int64_t)(R + 1) * (R + 1) <= mmax2) ++R;
    int64_t count = 0;
    for (int64_t a = -R; a <= R; ++a)
        for (int64_t b = -R; b <= R; ++b)
            for (int64_t d = -R; d <= R; ++d) {
                const int64_t m2 = a * a + b * b + d * d;
                count += m2 > 0 && m2 <= mmax2;
            }
    if (count > INT32_MAX) {
        null_errf("%lld modes do not fit 32-bit counts", (long long)count);
        return RBE_ERR_INVALID;
    }
    *nm = (int32_t)count;
    if (!modes && !weights) return RBE_OK;
    if (!modes || !weights || cap < count) {
        null_errf("modes and weights need room for %lld modes (cap = %d)", (long long)count, cap);
        return RBE_ERR_INVALID;
    }
    // Ewald weight of mode m: exp(-k^2 / (4 alpha)) with k = 2 pi |m| / L
    const double g = M_PI * M_PI / (alpha * box * box);
    int64_t l = 0;
    for (int64_t a = -R; a <= R; ++a)
        for (int64_t b = -R; b <= R; ++b)
            for (int64_t d = -R; d <= R; ++d) {
                const int64_t m2 = a * a + b * b + d * d;
                if (m2 == 0 || m2 > mmax2) continue;
                modes[l] = (int32_t)a;
                modes[(int64_t)cap + l] = (int32_t)b;
                modes[2 * (int64_t)cap + l] = (int32_t)d;
                weights[l] = std::exp(-g * (double)m2);
                ++l;
            }
    return RBE_OK;
}

rbe_status rbe_set_k_ewald(rbe_ctx *c, int32_t mmax2, int32_t *nm_out)
{
    if (!c) return RBE_ERR_INVALID;
    if (c->R != 1) return set_err(c, RBE_ERR_STATE, "rbe_set_k_ewald needs a single-system context");
    const double alpha = c->sysh[0].alpha, L = c->sysh[0].L;
    int32_t nm = 0;
    if (rbe_ewald_modes(alpha, L, mmax2, nullptr, nullptr, 0, &nm) != RBE_OK || nm < 1)
        return set_err(c, RBE_ERR_INVALID, fmt("no Ewald modes with 0 < |m|^2 <= %d", mmax2));
    std::vector<int32_t> m(3 * (size_t)nm);
    std::vector<double> w(nm);
    if (rbe_ewald_modes(alpha, L, mmax2, m.data(), w.data(), nm, &nm) != RBE_OK)
        return set_err(c, RBE_ERR_INVALID, g_create_error.c_str());
    if (nm > c->mcap) {
        rbe_status s = rbe_reserve_modes(c, nm);
        if (s != RBE_OK) return s;
    }
    rbe_status s = rbe_set_k(c, m.data(), nm, w.data());
    if (s == RBE_OK && nm_out) *nm_out = nm;
    return s;
}

// Structure factors of pos with the active modes (one staging launch and
// the reduction), then the force pass when force is given.
// Long mode lists (classical Ewald) are split over blocks so that a launch
// holds a few blocks per compute unit even for small N.
static int mode_split(int blocks, int modes, int modes_per_part)
{
    if (blocks >= 512) return 1;
    const int want = (512 + blocks - 1) / blocks;
    const int most = (modes + modes_per_part - 1) / modes_per_part;
    return std::max(1, std::min(std::min(want, most), kMaxModeSplit));
}

// Draw a recorded sample now, with its own launch.
static rbe_status materialize_sample(rbe_ctx *c)
{
    if (!c->sample_pending) return RBE_OK;
    c->sample_pending = false;
    RUN(c, K_SAMPLE, launch_sample(c->cfg, c->w, c->sample_step, 0));
    return RBE_OK;
}

static rbe_status kspace_impl(rbe_ctx *c, const void *pos, const void *q, void *force, int accumulate,
                              bool *cells = nullptr)
{
    if (c->cfg.cols.ncols) {
        RUN(c, K_STAGE, launch_col_rho(c->cfg, c->w, pos, q));
        RUN(c, K_MID, launch_col_final(c->cfg, c->w));
        if (force) RUN(c, K_KFORCE, launch_col_force(c->cfg, c->w, pos, q, force, accumulate));
        return RBE_OK;
    }
    LaunchCfg cfg = c->cfg;
    cfg.rho_block = c->cfg.call_block;
    StageRequest rq{const_cast<void *>(pos), nullptr, nullptr, q, 0, 0, 0, 0, 0, 1};
    rq.mode_split = mode_split(c->cfg.n_rho_tiles, c->max_p, 256);
    if (c->sample_pending) {
        int table_lds = 0, tab_max = 0;
        // fused when the launch has at most two blocks per CU: every block
        // draws the modes it needs, which costs more than one sampling
        // launch once there are many blocks
        if (c->cfg.n_rho_tiles <= 512 && stage_lds_bytes(cfg, 1, &table_lds, &tab_max) <= 64 * 1024) {
            // the staging launch draws the recorded sample (every block the
            // modes it needs; the first tile of each system stores them)
            rq.sample = 1;
            rq.sample_step = c->sample_step;
            rq.mode_split = 1;
            c->sample_pending = false;
        } else {
            rbe_status st = materialize_sample(c);
            if (st != RBE_OK) return st;
        }
    }
    // an energy call's cell list: binned and scanned by the same two launches when no
    // mode split makes several blocks stage a chunk
    const bool bin = cells && rq.mode_split == 1;
    if (cells) *cells = bin;
    rq.bin = bin ? 1 : 0;
    RUN(c, K_STAGE, launch_stage(cfg, c->w, rq));
    // the totals launch also draws the sample of the next step into the
    // alternate mode arrays (one block per system, beside the totals blocks)
    const bool predict = c->cur_drawn && !c->any_mh && !c->fixed &&
                         !(c->next_ready && c->next_step == c->cur_step + 1);
    RUN(c, K_MID, launch_mid(c->cfg, c->w, 1, bin ? 1 : 0, nullptr, nullptr, nullptr, predict ? 1 : 0,
                             c->cur_step + 1));
    if (predict) {
        c->next_ready = true;
        c->next_step = c->cur_step + 1;
    }
    const int fblocks = (c->cfg.n_force_tiles * c->cfg.force_split + 3) / 4;
    const int fs = c->w.fpart ? mode_split(fblocks, c->max_p, 1024) : 1;
    if (force) RUN(c, K_KFORCE, launch_kforce(c->cfg, c->w, pos, q, force, accumulate, 0, fs));
    return RBE_OK;
}

// Cell list of pos: bin (staging launch without the structure factor),
// scan, scatter into cell order.
static rbe_status cells_impl(rbe_ctx *c, const void *pos, const void *q, const void *gF = nullptr)
{
    c->list_valid = false;   // the cell order changes under the list
    StageRequest rq{const_cast<void *>(pos), nullptr, nullptr, q, 0, 0, 0, 1, 0, 0};
    RUN(c, K_STAGE, launch_stage(c->cfg, c->w, rq));
    RUN(c, K_MID, launch_mid(c->cfg, c->w, 0, 1));
    RUN(c, K_SCATTER, launch_scatter(c->cfg, c->w, gF));
    return RBE_OK;
}

rbe_status rbe_kspace_forces(rbe_ctx *c, const void *pos, const void *q, void *force, int32_t accumulate)
{
    if (!c) return RBE_ERR_INVALID;
    if (!pos || !q || !force) return set_err(c, RBE_ERR_INVALID, "pos, q and force must be non-NULL");
    if (!c->modes_valid) return set_err(c, RBE_ERR_STATE, "no active modes: call rbe_sample_k or rbe_set_k first");
    return kspace_impl(c, pos, q, force, accumulate);
}

rbe_status rbe_real_forces(rbe_ctx *c, const void *pos, const void *q, void *force, int32_t accumulate)
{
    if (!c) return RBE_ERR_INVALID;
    if (!pos || !q || !force) return set_err(c, RBE_ERR_INVALID, "pos, q and force must be non-NULL");
    rbe_status s = cells_impl(c, pos, q);
    if (s != RBE_OK) return s;
    RUN(c, K_REAL, launch_real(c->cfg, c->w, force, accumulate, nullptr));
    return RBE_OK;
}

// The three launches of one list-mode or all-pairs step (plus the sampling launch of a
// call's first step when it is not fused).  With base set (graph capture),
// s and ks are offsets from the device step number *base, and the force
// launch advances it by bump.
static rbe_status list_step(rbe_ctx *c, void *pos, void *vel, const void *q, void *force, uint64_t s, uint64_t ks,
                            bool first, bool last, bool fuse_sample, bool andersen, uint64_t *base, uint32_t bump)
{
    const int par = (int)(c->list_gen & 1);
    ListStep ls{c->w.lflag + par, c->w.lflag + (1 - par), c->w.lflag + 2, c->w.lflag + 3, c->w.lflag + 4,
                c->w.lflag + 5, c->w.lflag + 6, c->list_valid ? 0 : 1};
    ls.step_base = base;
    ls.step_bump = bump ? base : nullptr;
    ls.bump = bump;
    // the staging launch integrates (in particle order); the modes of every
    // step after the first of a call were drawn by the totals launch of the
    // step before (exact sampler)
    const bool drawn = c->fixed || (!first && !c->any_mh);
    if (!drawn && !fuse_sample) RUN(c, K_SAMPLE, launch_sample(c->cfg, c->w, ks, c->any_mh ? 1 : 0));
    StageRequest rq{pos, vel, force, q, s, ks, 1, 0, (!drawn && fuse_sample) ? 1 : 0, 1, &ls};
    // BAOAB: the closing half kick of a step is applied by the next step's
    // integrator (the force pass would touch the velocities in scattered
    // original order); only the last step of a call kicks in the force pass
    rq.kick = !first && !andersen;
    RUN(c, K_STAGE, launch_stage(c->cfg, c->w, rq));
    const bool draw_next = !c->any_mh && !c->fixed && !last;
    // an all-pairs context has nothing to rebuild, and a small one no totals launch
    const PairsStep ps{totals_in_force(c->cfg), draw_next ? 1 : 0, ks + 1};
    if (!ps.totals)
        RUN(c, K_MID, launch_mid(c->cfg, c->w, 1, 0, nullptr, c->cfg.list_on ? ls.rebuild : nullptr, ls.rebuild_next,
                             draw_next ? 1 : 0, ks + 1, &ls, pos, q));
    RUN(c, K_REAL, launch_real_step(c->cfg, c->w, ls, ps, force, (andersen || !last) ? nullptr : vel, s));
    c->list_valid = true;
    ++c->list_gen;
    if (draw_next) {
        std::swap(c->w.modes, c->w.modes_alt);
        std::swap(c->w.mode_w, c->w.mode_w_alt);
    }
    return RBE_OK;
}

static bool same_bytes(const void *a, const void *b, size_t n) { return std::memcmp(a, b, n) == 0; }

// Step pairs per captured graph (a replay covers 2 * kGraphPairs steps).
constexpr int kGraphPairs = 8;

// Graph of 2 * kGraphPairs steady-state list steps (neither the first nor the last of a
// call, modes drawn by the step before, list valid) for the current buffers
// and parity; captured on first use.
static rbe_status step_graph(rbe_ctx *c, void *pos, void *vel, const void *q, void *force, bool andersen,
                             hipGraphExec_t *out)
{
    const int par = (int)(c->list_gen & 1);
    LaunchCfg cfg = c->cfg;
    for (auto &g : c->step_graphs)
        if (g.pos == pos && g.vel == vel && g.q == q && g.force == force && g.par == par && g.andersen == andersen &&
            same_bytes(&g.w, &c->w, sizeof(Workspace)) && same_bytes(&g.cfg, &cfg, sizeof(LaunchCfg))) {
            g.used = ++c->graph_clock;
            *out = g.exec;
            return RBE_OK;
        }
    if (!c->cap_stream) HIPCHK(c, hipStreamCreateWithFlags(&c->cap_stream, hipStreamNonBlocking));
    rbe_ctx::StepGraph g;
    g.cfg = c->cfg;
    g.w = c->w;
    g.pos = pos;
    g.vel = vel;
    g.q = q;
    g.force = force;
    g.par = par;
    g.andersen = andersen;
    // capture on the context's own stream, leaving the state as it was
    const uint64_t gen = c->list_gen;
    const Workspace w0 = c->w;
    c->cfg.stream = c->cap_stream;
    hipGraph_t graph = nullptr;
    hipError_t e = hipStreamBeginCapture(c->cap_stream, hipStreamCaptureModeThreadLocal);
    rbe_status st = RBE_OK;
    if (e == hipSuccess) {
        // kGraphPairs copies of the two steps; each pair's second force
        // launch advances the device step number by 2
        const uint64_t k0 = andersen ? 1 : 0;
        for (int k = 0; k < kGraphPairs && st == RBE_OK; ++k) {
            st = list_step(c, pos, vel, q, force, 0, k0, false, false, false, andersen, c->w.step_base, 0);
            if (st == RBE_OK)
                st = list_step(c, pos, vel, q, force, 1, k0 + 1, false, false, false, andersen, c->w.step_base, 2);
        }
        e = hipStreamEndCapture(c->cap_stream, &graph);
    }
    c->cfg.stream = cfg.stream;
    c->list_gen = gen;
    c->w = w0;
    if (st != RBE_OK) {
        if (graph) (void)hipGraphDestroy(graph);
        return st;
    }
    if (e == hipSuccess) e = hipGraphInstantiate(&g.exec, graph, nullptr, nullptr, 0);
    if (graph) (void)hipGraphDestroy(graph);
    if (e != hipSuccess) return hip_fail(c, e, "capturing the step graph");
    if (c->step_graphs.size() >= 4) {
        auto lru = std::min_element(c->step_graphs.begin(), c->step_graphs.end(),
                                    [](const auto &a, const auto &b) { return a.used < b.used; });
        (void)hipGraphExecDestroy(lru->exec);
        c->step_graphs.erase(lru);
    }
    g.used = ++c->graph_clock;
    c->step_graphs.push_back(g);
    *out = g.exec;
    return RBE_OK;
}

rbe_status rbe_step(rbe_ctx *c, void *pos, void *vel, const void *q, void *force, uint64_t first_step,
                    int32_t nsteps)
{
    if (!c) return RBE_ERR_INVALID;
    if (!pos || !vel || !q || !force) return set_err(c, RBE_ERR_INVALID, "pos, vel, q and force must be non-NULL");
    if (nsteps < 0) return set_err(c, RBE_ERR_INVALID, "nsteps must be >= 0");
    const bool andersen = c->prm[0].integrator == RBE_LEAPFROG_ANDERSEN;
    for (int r = 1; r < c->R; ++r)
        if ((c->prm[r].integrator == RBE_LEAPFROG_ANDERSEN) != andersen)
            return set_err(c, RBE_ERR_INVALID, "all systems of a batch must use one integrator");
    if (c->fixed && !c->modes_valid)
        return set_err(c, RBE_ERR_STATE, "fixed sampler: set the modes with rbe_set_k or rbe_sample_k first");
    if (c->fixed) {
        rbe_status st = materialize_sample(c);
        if (st != RBE_OK) return st;
    } else if (nsteps > 0) {
        c->sample_pending = false;   // the first step draws its own modes
        c->cfg.cols = ColumnSet{};
        c->cur_drawn = false;
    }
    // time steps draw the next step's modes into the alternate arrays
    if (nsteps > 0) c->next_ready = false;
    for (int r = 0; r < c->R && !c->fixed; ++r)
        if (c->sysh[r].p != c->prm[r].p) {
            // explicit modes were set: stepping resamples, so restore p
            c->sysh[r].p = c->prm[r].p;
            rbe_status s = upload_sys(c);
            if (s != RBE_OK) return s;
            refresh_cfg_modes(c);
            if ((s = upload_rho_tiles(c)) != RBE_OK) return s;
        }
    // one step on the cell list = four launches: [closing kick of the step
    // before + integrate + bin + draw modes + structure-factor partials] ->
    // [totals + cell scan] -> [Fourier force + scatter] -> [real space + LJ
    // (+ the closing half kick on the last step of the call)].  In list mode, three: [closing
    // kick + integrate + list bookkeeping + partials] -> [totals + next
    // step's modes + binning, cell scan and scatter] -> [Fourier + real space
    // + LJ (+ closing kick on the last step)], where binning, scan and
    // scatter do work only on rebuild steps (decided on the device).  A context
    // of one-cell systems takes the same three launches without any cell work
    // (50 steps + energy of the 300-ion electrolyte: 1503 -> 1034 us against the four
    // launches, whose first one also draws the modes).  With graphs on, the
    // steady-state steps of a call (after the first, before the last) are
    // replayed from a captured graph.
    int table_lds = 0, tab_max = 0;
    const size_t lds = stage_lds_bytes(c->cfg, 1, &table_lds, &tab_max);
    const bool fuse_sample = !c->any_mh && lds <= 64 * 1024;
    const bool list = c->cfg.list_on != 0;
    const bool fused = list || c->cfg.all_pairs;
    const bool graphs = list && c->graphs && !c->any_mh && !c->prof;
    for (int32_t t = 0; t < nsteps;) {
        const uint64_t s = first_step + (uint64_t)t;
        const uint64_t ks = andersen ? s + 1 : s;
        if (fused) {
            const int32_t reps = (nsteps - 1 - t) / (2 * kGraphPairs);
            if (graphs && t > 0 && c->list_valid && reps > 0) {
                hipGraphExec_t exec;
                rbe_status st = step_graph(c, pos, vel, q, force, andersen, &exec);
                if (st != RBE_OK) return st;
                RUN(c, K_MISC, launch_set_step(c->cfg, c->w, s));
                for (int32_t k = 0; k < reps; ++k) HIPCHK(c, hipGraphLaunch(exec, c->stream));
                c->list_gen += 2 * (uint64_t)kGraphPairs * reps;
                t += 2 * kGraphPairs * reps;
                continue;
            }
            rbe_status st = list_step(c, pos, vel, q, force, s, ks, t == 0, t == nsteps - 1, fuse_sample, andersen,
                                      nullptr, 0);
            if (st != RBE_OK) return st;
        } else {
            if (!c->fixed && !fuse_sample) RUN(c, K_SAMPLE, launch_sample(c->cfg, c->w, ks, c->any_mh ? 1 : 0));
            StageRequest rq{pos, vel, force, q, s, ks, 1, 1, (!c->fixed && fuse_sample) ? 1 : 0, 1};
            rq.kick = t > 0 && !andersen;
            RUN(c, K_STAGE, launch_stage(c->cfg, c->w, rq));
            RUN(c, K_MID, launch_mid(c->cfg, c->w, 1, 1));
            RUN(c, K_KFORCE, launch_kforce(c->cfg, c->w, pos, q, force, 0, 1));
            const bool last = t == nsteps - 1;
            RUN(c, K_REAL, launch_real(c->cfg, c->w, force, 1, (andersen || !last) ? nullptr : vel, s));
        }
        ++t;
    }
    if (nsteps > 0) c->modes_valid = true;
    return RBE_OK;
}

rbe_status rbe_pair_histogram(rbe_ctx *c, const void *pos, const void *q, double r_max, int32_t nbins,
                              int64_t *counts)
{
    if (!c) return RBE_ERR_INVALID;
    if (!pos || !q || !counts) return set_err(c, RBE_ERR_INVALID, "pos, q and counts must be non-NULL");
    if (nbins < 1 || nbins > 4096) return set_err(c, RBE_ERR_INVALID, "nbins must be in [1, 4096]");
    if (!std::isfinite(r_max) || r_max <= 0.0) return set_err(c, RBE_ERR_INVALID, "r_max must be > 0");
    for (int r = 0; r < c->R; ++r)
        if (r_max > 0.5 * c->sysh[r].L)
            return set_err(c, RBE_ERR_INVALID, fmt("r_max %.6g exceeds half the box of system %d", r_max, r));
    RUN(c, K_MISC, launch_pair_hist(c->cfg, c->w, pos, q, r_max, nbins, counts));
    return RBE_OK;
}

rbe_status rbe_set_dt(rbe_ctx *c, double dt, double anneal)
{
    if (!c) return RBE_ERR_INVALID;
    if (!std::isfinite(dt) || dt < 0.0) return set_err(c, RBE_ERR_INVALID, "dt must be finite and >= 0");
    if (!std::isfinite(anneal) || anneal < 0.0) return set_err(c, RBE_ERR_INVALID, "anneal must be finite and >= 0");
    for (int r = 0; r < c->R; ++r) {
        rbe_params &p = c->prm[r];
        SysDev &s = c->sysh[r];
        p.dt = dt;
        s.dt = dt;
        s.c1 = std::exp(-p.gamma * dt / p.mass);
        s.c2 = std::sqrt((1.0 - s.c1 * s.c1) * p.kT / p.mass);
        s.nu_dt = p.nu * dt;
        s.h_m = 0.5 * dt / s.mass;
        s.anneal = anneal;
    }
    return upload_sys(c);
}

rbe_status rbe_use_graphs(rbe_ctx *c, int32_t enable)
{
    if (!c) return RBE_ERR_INVALID;
    HIPCHK(c, hipStreamSynchronize(c->stream));
    c->graphs = enable != 0;
    if (!c->graphs) drop_graphs(c);
    return RBE_OK;
}

rbe_status rbe_batch_step(rbe_ctx *c, void *pos, void *vel, const void *q, void *force, uint64_t first_step,
                          int32_t nsteps)
{
    return rbe_step(c, pos, vel, q, force, first_step, nsteps);
}

// Reads the device error word and clears the bits in `mask` (synchronises).
// After a timeout the neighbour list is marked stale so that the next step
// rebuilds from the cell counts, which the force launch of the failed step
// cleared.
static rbe_status take_device_errors(rbe_ctx *c, int32_t *bits, int32_t mask = -1)
{
    int32_t flag = 0;
    HIPCHK(c, hipMemcpyAsync(&flag, c->w.flag, sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    if (flag & mask) {
        const int32_t keep = flag & ~mask;
        HIPCHK(c, hipMemcpy(c->w.flag, &keep, sizeof(int32_t), hipMemcpyHostToDevice));
    }
    if (flag & mask & (kFlagTimeout | kFlagBounds)) c->list_valid = false;
    *bits = flag & mask;
    return RBE_OK;
}

static rbe_status device_error_status(rbe_ctx *c, int32_t bits)
{
    if (bits & kFlagTimeout)
        return set_err(c, RBE_ERR_TIMEOUT, "a bounded wait of a neighbour-list rebuild gave up; the forces of the "
                                           "steps since the last check are not valid");
    if (bits & kFlagBounds)
        return set_err(c, RBE_ERR_TIMEOUT, "a neighbour-list rebuild met stale cell counts; the forces of the "
                                           "steps since the last check are not valid");
    if (bits & kFlagNonFinite) return set_err(c, RBE_ERR_NONFINITE, "a kernel met a non-finite force");
    if (bits & kFlagRange)
        return set_err(c, RBE_ERR_NONFINITE, "a real-space force reached 2^20 (overlapping particles): single-precision "
                                             "pair sums are no longer exact and the forces are not valid");
    return RBE_OK;
}

rbe_status rbe_check(rbe_ctx *c)
{
    if (!c) return RBE_ERR_INVALID;
    int32_t bits = 0;
    rbe_status s = take_device_errors(c, &bits);
    if (s != RBE_OK) return s;
    return device_error_status(c, bits);
}

rbe_status rbe_set_wait_limit(rbe_ctx *c, int32_t limit)
{
    if (!c) return RBE_ERR_INVALID;
    if (limit < 0) return set_err(c, RBE_ERR_INVALID, "the wait limit must be >= 0");
    HIPCHK(c, hipStreamSynchronize(c->stream));
    c->cfg.wait_limit = limit;
    return RBE_OK;
}

rbe_status rbe_energy(rbe_ctx *c, const void *pos, const void *q, const void *vel, rbe_energy_t *out)
{
    if (!c) return RBE_ERR_INVALID;
    if (!pos || !q || !out) return set_err(c, RBE_ERR_INVALID, "pos, q and out must be non-NULL");
    if (!c->modes_valid) return set_err(c, RBE_ERR_STATE, "no active modes: call rbe_sample_k or rbe_set_k first");
    const size_t nout = (size_t)kEnergyOut * c->R + 1;
    if (!c->energy_h) HIPCHK(c, hipHostMalloc((void **)&c->energy_h, sizeof(double) * nout, hipHostMallocMapped));
    void *dev = nullptr;
    HIPCHK(c, hipHostGetDevicePointer(&dev, c->energy_h, 0));
    bool cells = false;
    rbe_status s = kspace_impl(c, pos, q, nullptr, 0, &cells);
    if (s != RBE_OK) return s;
    if (cells) {
        c->list_valid = false;   // the cell order changes under the list
        RUN(c, K_SCATTER, launch_scatter(c->cfg, c->w));
    } else if ((s = cells_impl(c, pos, q)) != RBE_OK) {
        return s;
    }
    RUN(c, K_ENERGY, launch_energy(c->cfg, c->w, q, vel));
    RUN(c, K_ENERGY, launch_energy_sum(c->cfg, c->w, (double *)dev));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    int32_t flag = (int32_t)c->energy_h[nout - 1];
    if (flag) {
        rbe_status es = take_device_errors(c, &flag);
        if (es != RBE_OK) return es;
    }
    rbe_status ret = RBE_OK;
    for (int r = 0; r < c->R; ++r) {
        const SysDev &S = c->sysh[r];
        const double *acc = c->energy_h + kEnergyOut * (size_t)r;
        rbe_energy_t &e = out[r];
        e.e_kspace = acc[8];
        e.virial_kspace = acc[9];
        e.e_self = -S.coulomb * std::sqrt(S.alpha / kPi) * acc[4];
        e.e_real = acc[0];
        e.e_lj = acc[1];
        e.virial = acc[2];
        e.e_kin = vel ? acc[3] : 0.0;
        e.charge_sum = acc[5];
        e.nonfinite = (flag & (kFlagNonFinite | kFlagRange)) ? 1 : 0;
        e.timeout = (flag & (kFlagTimeout | kFlagBounds)) ? 1 : 0;
        if (std::fabs(acc[5]) > 1e-6 * acc[6] && ret == RBE_OK) {
            ret = set_err(c, RBE_ERR_NOT_NEUTRAL,
                          fmt("system %d is not neutral: sum q = %.6g, sum |q| = %.6g", r, acc[5],
                              acc[6]));
        }
    }
    if (flag) ret = device_error_status(c, flag);
    return ret;
}

rbe_status rbe_get_rho(rbe_ctx *c, double *rho)
{
    if (!c || !rho) return c ? set_err(c, RBE_ERR_INVALID, "rho must be non-NULL") : RBE_ERR_INVALID;
    HIPCHK(c, hipMemcpyAsync(rho, c->w.rho, sizeof(double) * 2 * c->mtot, hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    return RBE_OK;
}

rbe_status rbe_forces_vjp(rbe_ctx *c, const void *pos, const void *q, const void *grad_force, void *grad_pos,
                          void *grad_q, int32_t parts)
{
    if (!c) return RBE_ERR_INVALID;
    if (!pos || !q || !grad_force || !grad_pos || !grad_q)
        return set_err(c, RBE_ERR_INVALID, "pointers must be non-NULL");
    if (parts < 1 || parts > 3) return set_err(c, RBE_ERR_INVALID, "parts must be RBE_PART_KSPACE, _REAL or _ALL");
    if ((parts & RBE_PART_KSPACE) && !c->modes_valid)
        return set_err(c, RBE_ERR_STATE, "no active modes: call rbe_sample_k or rbe_set_k first");
    if (parts & RBE_PART_REAL)
        for (int r = 0; r < c->R; ++r)
            if (c->sysh[r].diam_on)
                return set_err(c, RBE_ERR_STATE, "the real-space adjoint does not cover per-particle diameters");
    const bool kspace = parts & RBE_PART_KSPACE, real = parts & RBE_PART_REAL;
    if (kspace) {
        rbe_status s = materialize_sample(c);
        if (s != RBE_OK) return s;
        if (real) c->list_valid = false;   // the cell order changes under the list
        // a pass over the modes needs four sums per tile and mode: all modes
        // at once where the partials have room (as allocated at creation), else a
        // single system's long list in slices
        const int slices = c->R == 1 ? vjp_slices(c->cfg.n_rho_tiles, c->max_p, c->partial_cap) : 1;
        if (slices < 1) return set_err(c, RBE_ERR_STATE, "no room for the partial sums of one mode");
        for (int k = 0; k < slices; ++k) {
            const int l0 = slices == 1 ? 0 : (int)((int64_t)c->max_p * k / slices);
            const int l1 = slices == 1 ? 0 : (int)((int64_t)c->max_p * (k + 1) / slices);
            const int first = real && k == 0 ? 1 : 0;
            RUN(c, K_VJP_REDUCE, launch_vjp_stage(c->cfg, c->w, pos, q, grad_force, l0, l1, first,
                                                  mode_split(c->cfg.n_rho_tiles, (l1 ? l1 - l0 : c->max_p), 256)));
            RUN(c, K_VJP_REDUCE, launch_vjp_final(c->cfg, c->w, l0, l1, first));
        }
        RUN(c, K_VJP_GATHER, launch_vjp_gather(c->cfg, c->w, pos, q, grad_force, grad_pos, grad_q, real ? 1 : 0));
    } else {
        rbe_status s = cells_impl(c, pos, q, grad_force);
        if (s != RBE_OK) return s;
    }
    if (real) RUN(c, K_VJP_REAL, launch_vjp_real(c->cfg, c->w, grad_force, grad_pos, grad_q, kspace ? 1 : 0));
    return RBE_OK;
}

rbe_status rbe_list_builds(rbe_ctx *c, int64_t *builds)
{
    if (!c || !builds) return RBE_ERR_INVALID;
    int32_t v = 0;
    HIPCHK(c, hipMemcpyAsync(&v, c->w.lflag + 3, sizeof(int32_t), hipMemcpyDeviceToHost, c->stream));
    HIPCHK(c, hipStreamSynchronize(c->stream));
    *builds = c->cfg.list_on ? (int64_t)v : -1;
    // a non-finite force is left for rbe_energy / rbe_check to report
    int32_t bits = 0;
    rbe_status s = take_device_errors(c, &bits, kFlagTimeout | kFlagBounds);
    if (s != RBE_OK) return s;
    return device_error_status(c, bits);
}

rbe_status rbe_get_tiles(const rbe_ctx *c, rbe_tiles *t)
{
    if (!c || !t) return RBE_ERR_INVALID;
    t->rho_chunk = c->cfg.rho_chunk;
    t->rho_block = c->cfg.rho_block;
    t->force_split = c->cfg.force_split;
    t->real_split = c->cfg.real_split;
    return RBE_OK;
}

rbe_status rbe_set_tiles(rbe_ctx *c, const rbe_tiles *t)
{
    if (!c || !t) return RBE_ERR_INVALID;
    rbe_tiles n{c->cfg.rho_chunk, c->cfg.rho_block, c->cfg.force_split, c->cfg.real_split};
    if (t->rho_chunk) n.rho_chunk = t->rho_chunk;
    if (t->rho_block) n.rho_block = t->rho_block;
    if (t->force_split) n.force_split = t->force_split;
    if (t->real_split) n.real_split = t->real_split;
    if (n.rho_chunk < 64 || n.rho_chunk > 2048 || (n.rho_chunk % 8))
        return set_err(c, RBE_ERR_INVALID, "rho_chunk must be a multiple of 8 in [64, 2048]");
    if (n.rho_block != 256 && n.rho_block != 512 && n.rho_block != 1024)
        return set_err(c, RBE_ERR_INVALID, "rho_block must be 256, 512 or 1024");
    if (n.force_split != 1 && n.force_split != 2 && n.force_split != 4)
        return set_err(c, RBE_ERR_INVALID, "force_split must be 1, 2 or 4");
    if (n.real_split != 1 && n.real_split != 2 && n.real_split != 4 && n.real_split != 8)
        return set_err(c, RBE_ERR_INVALID, "real_split must be 1, 2, 4 or 8");
    if (!tiles_fit(n)) return set_err(c, RBE_ERR_INVALID, "rho_chunk and rho_block need more than 64 KB of LDS");
    if (partial_need(c, n.rho_chunk) > c->partial_cap)
        return set_err(c, RBE_ERR_INVALID, "rho_chunk too small for the structure-factor partials of the reserved "
                                           "mode capacity");
    HIPCHK(c, hipStreamSynchronize(c->stream));
    c->cfg.rho_chunk = n.rho_chunk;
    c->cfg.rho_block = n.rho_block;
    c->cfg.force_split = n.force_split;
    c->cfg.real_split = n.real_split;
    if (t->real_split) c->lanes_set = true;
    if (t->rho_chunk || t->rho_block) c->shape_set = true;
    if (c->shape_set) c->cfg.call_block = n.rho_block;
    rbe_status st = upload_rho_tiles(c);
    if (st != RBE_OK) return st;
    return upload_list_tiles(c);
}

rbe_status rbe_tune_lookup(const char *arch, int32_t precision, int64_t ntot, int32_t max_p, int32_t R,
                           rbe_tiles *out)
{
    if (!arch || !out || ntot < 1 || max_p < 1 || R < 1) return RBE_ERR_INVALID;
    return tune_lookup(tune_key(arch, precision, ntot, max_p, R), out) ? RBE_OK : RBE_ERR_STATE;
}

rbe_status rbe_autotune(rbe_ctx *c, const void *pos, const void *q, int32_t reps, rbe_tiles *best)
{
    if (!c) return RBE_ERR_INVALID;
    if (!pos || !q) return set_err(c, RBE_ERR_INVALID, "pos and q must be non-NULL");
    if (!c->modes_valid) return set_err(c, RBE_ERR_STATE, "no active modes: call rbe_sample_k or rbe_set_k first");
    if (reps < 1) reps = 10;
    {
        rbe_status st = materialize_sample(c);
        if (st != RBE_OK) return st;
    }
    const bool prof = c->prof;
    c->prof = false;
    hipEvent_t a, b;
    HIPCHK(c, hipEventCreate(&a));
    HIPCHK(c, hipEventCreate(&b));
    auto timeit = [&](auto &&body, float *ms) -> rbe_status {
        rbe_status s = body();  // warm-up
        if (s != RBE_OK) return s;
        HIPCHK(c, hipEventRecord(a, c->stream));
        for (int k = 0; k < reps; ++k)
            if ((s = body()) != RBE_OK) return s;
        HIPCHK(c, hipEventRecord(b, c->stream));
        HIPCHK(c, hipEventSynchronize(b));
        HIPCHK(c, hipEventElapsedTime(ms, a, b));
        return RBE_OK;
    };
    rbe_tiles cur;
    rbe_get_tiles(c, &cur);
    rbe_tiles win = cur;
    float best_rho = 1e30f, best_f = 1e30f;
    const int fill = (int)std::min<int64_t>(2048, std::max<int64_t>(64, ((c->ntot + 255) / 256 + 7) / 8 * 8));
    const int chunks[] = {128, 256, 512, 1024, fill};
    const int blocks[] = {256, 512, 1024};
    rbe_status s = RBE_OK;
    for (int ch : chunks)
        for (int bl : blocks) {
            rbe_tiles t{ch, bl, cur.force_split, 0};
            if (rbe_set_tiles(c, &t) != RBE_OK) continue;   // shape does not fit
            float ms = 0.f;
            s = timeit(
                [&]() -> rbe_status {
                    StageRequest rq{const_cast<void *>(pos), nullptr, nullptr, q, 0, 0, 0, 0, 0, 1};
                    RUN(c, K_STAGE, launch_stage(c->cfg, c->w, rq));
                    RUN(c, K_MID, launch_mid(c->cfg, c->w, 1, 0));
                    return RBE_OK;
                },
                &ms);
            if (s != RBE_OK) break;
            if (ms < best_rho) {
                best_rho = ms;
                win.rho_chunk = ch;
                win.rho_block = bl;
            }
        }
    if (s == RBE_OK) {
        rbe_tiles t{win.rho_chunk, win.rho_block, 0, 0};
        s = rbe_set_tiles(c, &t);
    }
    void *fbuf = nullptr;
    if (s == RBE_OK) {
        const size_t esz = c->prec == RBE_FP64 ? 8 : 4;
        // the force pass needs an output: borrow the sorted workspace, which
        // is large enough (16 or 32 bytes per particle >= 3 elements); the
        // neighbour list reads that workspace, so it must be rebuilt
        fbuf = c->w.sorted;
        c->list_valid = false;
        (void)esz;
        for (int sp : {1, 2, 4}) {
            rbe_tiles t{0, 0, sp, 0};
            if ((s = rbe_set_tiles(c, &t)) != RBE_OK) break;
            float ms = 0.f;
            s = timeit(
                [&]() -> rbe_status {
                    RUN(c, K_KFORCE, launch_kforce(c->cfg, c->w, pos, q, fbuf, 0, 0));
                    return RBE_OK;
                },
                &ms);
            if (s != RBE_OK) break;
            if (ms < best_f) {
                best_f = ms;
                win.force_split = sp;
            }
        }
    }
    (void)hipEventDestroy(a);
    (void)hipEventDestroy(b);
    c->prof = prof;
    if (s != RBE_OK) return s;
    const bool lanes_set = c->lanes_set;   // the lanes are not tuned
    if ((s = rbe_set_tiles(c, &win)) != RBE_OK) return s;
    if (c->lanes_set != lanes_set) {
        c->lanes_set = lanes_set;
        if ((s = upload_list_tiles(c)) != RBE_OK) return s;
    }
    tune_store(tune_key(c->arch.c_str(), c->prec, c->ntot, c->max_p, c->R), win);
    if (best) *best = win;
    return RBE_OK;
}

}  // extern "C"

// ---------------------------------------------------------------------------
// Fourier force without allocation.  Its workspace (system constants, tiles,
// structure-factor partials and totals, per-mode constants) is one
// file-scope device array of fixed size: each GPU the library runs on holds
// its own copy until the process ends.  Host code never uses the array's
// name as an address; each device's address is taken once, with that device
// current, by hipGetSymbolAddress, and only that pointer reaches kernels.
// ---------------------------------------------------------------------------
namespace {
constexpr int64_t kStaticMaxN = 1 << 20;     // particles
constexpr int kStaticMaxP = 512;             // modes
constexpr int kStaticMaxRhoTiles = 2048;     // structure-factor tiles of default_rho_chunk up to kStaticMaxN
constexpr size_t align256(size_t x) { return (x + 255) & ~size_t(255); }
constexpr size_t kOffSys = 0;
constexpr size_t kOffPartOff = kOffSys + align256(sizeof(SysDev));
constexpr size_t kOffFlag = kOffPartOff + 256;
constexpr size_t kOffRhoTiles = kOffFlag + 256;
constexpr size_t kOffForceTiles = kOffRhoTiles + align256(sizeof(Tile) * kStaticMaxRhoTiles);
constexpr size_t kOffModeW = kOffForceTiles + align256(sizeof(Tile) * (kStaticMaxN / 64));
constexpr size_t kOffRho = kOffModeW + align256(sizeof(double) * kStaticMaxP);
constexpr size_t kOffKmode = kOffRho + align256(sizeof(double) * 2 * kStaticMaxP);
constexpr size_t kOffPartial = kOffKmode + align256(sizeof(KModeD) * kStaticMaxP);
constexpr size_t kStaticBytes = kOffPartial + sizeof(double) * 2 * (size_t)kStaticMaxRhoTiles * kStaticMaxP;
}  // namespace

static __device__ __align__(256) unsigned char scratch[kStaticBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
unsigned char *g_scratch_ptr[kMaxDevices] = {};

// This device's copy of `scratch` (the device must be current).  The first
// call on a device checks that it is a gfx950 and takes the address.
rbe_status scratch_of_device(int dev, unsigned char **out)
{
    if (dev < 0 || dev >= kMaxDevices) {
        null_errf("device %d is beyond the %d devices this entry point tracks", dev, kMaxDevices);
        return RBE_ERR_NO_DEVICE;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        hipDeviceProp_t prop;
        if (hipGetDeviceProperties(&prop, dev) != hipSuccess || std::strncmp(prop.gcnArchName, "gfx950", 6) != 0) {
            (void)hipGetLastError();
            null_errf("device %d is not gfx950", dev);
            return RBE_ERR_NO_DEVICE;
        }
        unsigned char *ptr = nullptr;
        const hipError_t e = hipGetSymbolAddress((void **)&ptr, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !ptr) {
            null_errf("hipGetSymbolAddress of the static workspace failed on device %d: %s", dev,
                      hipGetErrorString(e));
            return RBE_ERR_HIP;
        }
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return RBE_OK;
}
}  // namespace

extern "C" {

rbe_status rbe_kspace_forces_noalloc(const rbe_params *params, const int32_t *modes, const void *pos,
                                     const void *q, void *force, int32_t accumulate, void *stream)
{
    if (!params || !modes || !pos || !q || !force) {
        g_create_error = "params, modes, pos, q and force must be non-NULL";
        return RBE_ERR_INVALID;
    }
    const rbe_params &p = *params;
    if (p.n < 1 || p.n > kStaticMaxN) {
        null_errf("n = %d is outside [1, %lld], the size of this entry point's fixed workspace", p.n,
                  (long long)kStaticMaxN);
        return RBE_ERR_INVALID;
    }
    if (p.p < 1 || p.p > kStaticMaxP) {
        null_errf("p = %d is outside [1, %d], the size of this entry point's fixed workspace", p.p, kStaticMaxP);
        return RBE_ERR_INVALID;
    }
    if (!finite_pos(p.box) || !finite_pos(p.alpha) || !std::isfinite(p.coulomb)) {
        null_errf("box and alpha must be finite and > 0, coulomb finite");
        return RBE_ERR_INVALID;
    }
    if (p.precision != RBE_FP32 && p.precision != RBE_FP64) {
        null_errf("unknown precision %d", p.precision);
        return RBE_ERR_INVALID;
    }
    const double H = normaliser_H(p.alpha, p.box);
    if (1.0 / (H * H * H) > 0.5 || (p.precision == RBE_FP32 && table_half_width(p.alpha, p.box) > 4095)) {
        null_errf("alpha L^2 = %.3g is outside the range of the mode table", p.alpha * p.box * p.box);
        return RBE_ERR_INVALID;
    }
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess) {
        (void)hipGetLastError();
        null_errf("no HIP device available");
        return RBE_ERR_NO_DEVICE;
    }
    unsigned char *base = nullptr;
    rbe_status st = scratch_of_device(dev, &base);
    if (st != RBE_OK) return st;

    SysDev sys{};
    fourier_constants(p, sys);
    sys.polar = polar_form((int64_t)p.n * p.p, p.precision);
    LaunchCfg c{};
    c.stream = (hipStream_t)stream;
    c.R = 1;
    c.prec = p.precision;
    c.ntot = p.n;
    c.mcap = p.p;
    c.max_p = p.p;
    c.rho_chunk = default_rho_chunk(p.n);
    c.rho_block = 1024;
    c.force_split = default_force_split(p.n);
    c.n_rho_tiles = (p.n + c.rho_chunk - 1) / c.rho_chunk;
    c.max_sys_rho_tiles = c.n_rho_tiles;
    c.n_force_tiles = (p.n + 63) / 64;
    if (c.n_rho_tiles > kStaticMaxRhoTiles) {
        null_errf("internal: %d structure-factor tiles exceed the fixed workspace", c.n_rho_tiles);
        return RBE_ERR_INVALID;
    }
    Workspace w{};
    w.sys = reinterpret_cast<SysDev *>(base + kOffSys);
    w.partial_off = reinterpret_cast<int32_t *>(base + kOffPartOff);
    w.flag = reinterpret_cast<int32_t *>(base + kOffFlag);
    w.rho_tiles = reinterpret_cast<Tile *>(base + kOffRhoTiles);
    w.force_tiles = reinterpret_cast<Tile *>(base + kOffForceTiles);
    w.mode_w = reinterpret_cast<double *>(base + kOffModeW);
    w.rho = reinterpret_cast<double *>(base + kOffRho);
    w.kmode = base + kOffKmode;
    w.partial = reinterpret_cast<double *>(base + kOffPartial);
    w.modes = const_cast<int32_t *>(modes);

    auto hip_err = [](hipError_t e, const char *what) {
        null_errf("%s: %s", what, hipGetErrorString(e));
        return RBE_ERR_HIP;
    };
    hipError_t e = launch_static_setup(c, w, sys);
    if (e != hipSuccess) return hip_err(e, "static workspace set-up");
    StageRequest rq{const_cast<void *>(pos), nullptr, nullptr, q, 0, 0, 0, 0, 0, 1};
    rq.mode_split = mode_split(c.n_rho_tiles, p.p, 256);
    if ((e = launch_stage(c, w, rq)) != hipSuccess) return hip_err(e, "structure-factor launch");
    if ((e = launch_mid(c, w, 1, 0)) != hipSuccess) return hip_err(e, "totals launch");
    if ((e = launch_kforce(c, w, pos, q, force, accumulate, 0, 1)) != hipSuccess) return hip_err(e, "force launch");
    return RBE_OK;
}

rbe_status rbe_profile_enable(rbe_ctx *c, int32_t enable)
{
    if (!c) return RBE_ERR_INVALID;
    HIPCHK(c, hipStreamSynchronize(c->stream));
    for (auto &p : c->pend) {
        c->pool.push_back(p.a);
        c->pool.push_back(p.b);
    }
    c->pend.clear();
    for (int k = 0; k < K_COUNT; ++k) {
        c->prof_ms[k] = 0.0;
        c->prof_n[k] = 0;
    }
    c->prof = enable != 0;
    return RBE_OK;
}

rbe_status rbe_profile_read(rbe_ctx *c, int32_t id, double *total_ms, int64_t *launches)
{
    if (!c) return RBE_ERR_INVALID;
    if (id < 0 || id >= K_COUNT) return set_err(c, RBE_ERR_INVALID, "unknown kernel id");
    HIPCHK(c, hipStreamSynchronize(c->stream));
    for (auto &p : c->pend) {
        float ms = 0.f;
        HIPCHK(c, hipEventElapsedTime(&ms, p.a, p.b));
        c->prof_ms[p.id] += ms;
        c->prof_n[p.id] += 1;
        c->pool.push_back(p.a);
        c->pool.push_back(p.b);
    }
    c->pend.clear();
    if (total_ms) *total_ms = c->prof_ms[id];
    if (launches) *launches = c->prof_n[id];
    return RBE_OK;
}

const char *rbe_profile_name(int32_t id)
{
    if (id < 0 || id >= K_COUNT) return nullptr;
    return kKernelNames[id];
}

int32_t rbe_profile_count(void) { return K_COUNT; }

}  // extern "C"

// ---------------------------------------------------------------------------
// Sizes and shapes as host arithmetic, for tests of their bounds without a device.  Not
// part of the interface.
// ---------------------------------------------------------------------------
extern "C" {
void rbe_plan_pair_hist(int64_t max_n, int32_t R, int32_t *tile, int32_t *jw, int32_t *blocks, int32_t *flush)
{
    const PairHistPlan p = pair_hist_plan(max_n, R);
    *tile = kPairHistTile;
    *jw = p.jw;
    *blocks = p.blocks;
    *flush = p.flush;
}

// Single system of n particles and p modes created at any chunk: doubles of its partials, and the
// adjoint's slices of `modes` modes at `chunk`.
void rbe_plan_adjoint(int32_t n, int32_t p, int32_t chunk, int32_t modes, int64_t *room, int32_t *slices)
{
    const int64_t t64 = ((int64_t)n + 63) / 64;
    *room = (int64_t)partial_room(t64 * p, t64, partial_twice(1, n));
    *slices = vjp_slices(((int64_t)n + chunk - 1) / chunk, modes, (size_t)*room);
}

// Columns of a list of nm modes for n particles in the given precision, with room for `room` doubles of partial sums: number (0: summed
// by mode) and trigonometric slots, particles per block of the two passes, particle groups.
void rbe_plan_columns(const int32_t *modes, int32_t nm, int64_t n, int32_t prec, int64_t room, int32_t *out)
{
    ColumnLists cl;
    build_columns(modes, nm, n, prec, (size_t)room, cl);
    const ColumnSet &s = cl.set;
    const int32_t v[5] = {s.ncols, s.D, s.rho_nb, s.force_nb, s.groups};
    std::copy(v, v + 5, out);
}

// What a context runs: lanes per particle of the list pass, its tiles and the room for them; columns of the
// active list (0: sums by mode) and the particles per block of their two passes.
void rbe_plan_of_context(const rbe_ctx *c, int32_t *out)
{
    const int32_t v[6] = {c->cfg.list_lanes, c->cfg.n_list_tiles, (int32_t)list_tile_room(c), c->cfg.cols.ncols, c->cfg.cols.rho_nb,
                          c->cfg.cols.force_nb};
    std::copy(v, v + 6, out);
}

// Wave tiles of the sparse cell pass (0: the context does not take it).
int32_t rbe_plan_sparse(const rbe_ctx *c) { return c->cfg.n_sparse_tiles; }
}  // extern "C"

// sc_compact_host.cpp -- sizes of the compacted sum (see sc_compact.h): how many rows and columns
// interpolate the kernel to rounding, and whether the compacted sum is the faster one.
#include "sc_compact.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace sc {

namespace {

// Interpolation error aimed at, relative to the largest kernel value, as the estimates below state it.
// Over 140 random problems the largest errors met were 0.3 of it and the median 0.02: 2e-9 in the FP32
// form, whose own rounding is 1e-7, and 1e-16 in FP64.
constexpr double EPS_FP32 = 1e-7, EPS_FP64 = 1e-14;

constexpr int N_ETA = 80;             // widths of the strip of analyticity tried: 0.05 ... 4
constexpr double ETA_STEP = 0.05;
constexpr int N_ALPHA = 8, N_S = 16, N_TAU = 8;
constexpr double ALPHAS[N_ALPHA] = {0.3, 0.7, 0.8, 0.85, 0.9, 0.93, 0.95, 0.97};

// What the plans share: strips in phi, and the ellipses of every alpha in theta / theta_max.
struct Tables {
    double sinh_[N_ETA], lead[N_ETA];   // sinh(eta), log(4 / (1 - e^-eta)) + eta
    struct Ellipse {
        double s, lead;                 // parameter; log(4 / (1 - e^-s))
        double re[N_TAU], im[N_TAU];    // asin(alpha cosh(s + i tau)) / beta, tau over a quarter
    } ell[N_ALPHA][N_S];
    double beta[N_ALPHA], node[N_ALPHA][8];   // asin(alpha); theta / theta_max of 8 rows
    Tables()
    {
        for (int i = 0; i < N_ETA; ++i) {
            const double e = ETA_STEP * (i + 1);
            sinh_[i] = std::sinh(e);
            lead[i] = std::log(4.0 / (1.0 - std::exp(-e))) + e;
        }
        for (int a = 0; a < N_ALPHA; ++a) {
            beta[a] = std::asin(ALPHAS[a]);
            const double s_max = std::min(2.5, std::acosh(1.0 / ALPHAS[a]));
            for (int i = 0; i < N_S; ++i) {
                Ellipse &e = ell[a][i];
                e.s = s_max * (i + 1) / N_S;
                e.lead = std::log(4.0 / (1.0 - std::exp(-e.s)));
                for (int t = 0; t < N_TAU; ++t) {
                    const double tau = (t + 0.5) * M_PI / (2 * N_TAU);
                    const double x = ALPHAS[a] * std::cosh(e.s) * std::cos(tau), y = ALPHAS[a] * std::sinh(e.s) * std::sin(tau);
                    const double p = std::hypot(x + 1.0, y), m = std::hypot(x - 1.0, y);   // asin(x + iy)
                    e.re[t] = std::asin(0.5 * (p - m)) / beta[a];
                    e.im[t] = std::acosh(std::max(1.0, 0.5 * (p + m))) / beta[a];
                }
            }
            for (int m = 0; m < 8; ++m)
                node[a][m] = std::asin(ALPHAS[a] * std::cos((2 * m + 1) * M_PI / 32.0)) / beta[a];
        }
    }
};

}  // namespace

bool compact_plan(const CompactInput &in, CompactPlan &plan)
{
    static const Tables T;
    std::memset(&plan, 0, sizeof plan);   // plans are compared as bytes
    if (!(in.obs_r2max >= 0.0) || !(in.f > 0.0) || !(in.r_max > 0.0)) return false;
    const double rp = std::sqrt(in.obs_r2max), rho = std::sqrt(std::max(in.obs_rho2max, 0.0));
    const double q = rp / in.f;   // |r_s| >= f on the paraboloid
    // farther out the singularity R = 0 comes near the strip (and few nodes would be saved)
    if (!(q <= 0.25) || !std::isfinite(in.k_max * rp)) return false;
    // Very deep mirrors: |r_s| at the rim is many f, where the kernel is that much smaller than at the vertex while
    // its nodes stand for larger areas, so an error relative to the largest kernel value is not small there, and the
    // FP32 form's second FP16 parts reach their smallest number.  With the rim lit alone the FP32 error was 1.0 times
    // the direct sum's at a rim of 8 f (aperture radius 5.3 f), 1.1 to 1.3 times at 17 f, twice at 37 f and 150 times
    // at 401 f; in FP64 the difference to the direct sum grew from 4e-15 at 8 f to 6e-15 and 4e-14.
    if (in.r_max * in.r_max > 28.0 * in.f * in.f) return false;   // |r_s| = f + r^2 / 4f
    // Wavelengths beyond the mirror's size: 1 / kR in the FP32 form's H leaves the range of FP16.
    if (!in.fp64 && !(in.k_min * in.f >= 1.0 / 32.0)) return false;
    // Which sum is faster, in us of 1024 SIMDs' cycles (measured: 1.5 cycles per direct FP32 evaluation on the
    // tied tables and 4.4 in FP64, 1.2 and 5.3 per compacted one, a quarter more for the last round of
    // tiles; the matrix instructions of the two interpolations at 32 FP64 flops per cycle) and, for small
    // problems, the serial chain of a wave (0.3 us per node of a direct chunk) and the reduction of the chunks,
    // against the launches that build the tables (32 us at 64 x 64 nodes, 52 at 256 x 256).  The tables
    // serve every evaluation until the field changes, so they count for 0.7 of one.  That is where a first pass
    // breaks even: 36 random problems that are compacted at 0.7 and would not be at 1 took, over the direct sum's
    // time, 1.00 with a new built-in beam (0.77 to 1.21), 0.87 with a new field of the caller's (slower in 6), 0.79
    // without allocation, where the tables are built on each call (slower in 2), and 0.21 with the tables there.
    const int64_t n_tot = (int64_t)(in.n_r + 1) * in.n_phi;
    const double pts = (double)in.n_k * in.n_obs_pad, cyc = 1024.0 * 2.2e3;   // cycles per us
    const double launches = 20.0 + 0.065 * ((double)in.n_r + in.n_phi);
    const int64_t chunk = std::min<int64_t>(2048, direct_chunk_nodes(n_tot, in.n_obs_pad, in.n_k, in.fp64));
    const double direct = std::max(0.3 * chunk, 1.25 * pts * (double)n_tot * (in.fp64 ? 4.4 : 1.5) / cyc) + 5.0 +
                          (in.fp64 ? 0.05 : 0.035) * (double)((n_tot + chunk - 1) / chunk);
    if (direct < 0.7 * launches) return false;
    const double theta_max = 2.0 * std::atan(in.r_max / (2.0 * in.f));
    const double logeps = std::log(in.fp64 ? EPS_FP64 : EPS_FP32);

    // Columns of a row.  On Im phi = eta the phase's imaginary part is at most X cos(phi), X = x sinh(eta),
    // x = k rho' sin(theta), so |K| is about e^{X cos(phi)}, whose mean is I_0(X) < e^X / (1 + X)^1/2; P
    // equispaced points (P odd) alias the harmonics beyond (P - 1) / 2, which sum to at most
    // 4 I_0(X) e^{-eta (P + 1) / 2} / (1 - e^-eta): (P + 1) / 2 is the least over eta of
    // (X - log(1 + X) / 2 + amp) / eta, which has one minimum, at a smaller eta for a larger x.
    double amp[N_ETA];
    int n_eta = 0;
    for (; n_eta < N_ETA; ++n_eta) {
        const double near = q * std::exp(ETA_STEP * (n_eta + 1));
        if (near > 0.7) break;
        amp[n_eta] = T.lead[n_eta] - 3.0 * std::log1p(-near) - logeps;
    }
    auto columns = [&](double theta, int &at) {
        const double x = in.k_max * rho * std::sin(theta);
        auto half = [&](int i) {
            const double X = x * T.sinh_[i];
            return (X - 0.5 * std::log1p(X) + amp[i]) / (ETA_STEP * (i + 1));
        };
        double best = half(at);
        while (at > 0) {
            const double h = half(at - 1);
            if (h > best) break;
            best = h;
            --at;
        }
        while (at + 1 < n_eta) {
            const double h = half(at + 1);
            if (h >= best) break;
            best = h;
            ++at;
        }
        return best;
    };
    const double top = std::min(theta_max, 0.5 * M_PI);
    int eta0 = n_eta / 2, eta1 = eta0;
    const double half0 = columns(0.0, eta0), half1 = (columns(top, eta1) - half0) / std::sin(top);

    // Rows.  At theta = a + ih the phase k delta, delta = |r_s - r'| - |r_s|, has an imaginary part of at
    // most k |rho' cos(a) + z' sin(a)| sinh(h) (1 + q cosh h), and R stays away from 0 while
    // q cosh^2(h / 2) e^h < 1.  theta = theta_max asin(alpha y) / beta maps the ellipse of parameter s
    // about y in [-1, 1], which ends before the branch points while alpha cosh(s) <= 1, and interpolation
    // at N Chebyshev points y errs by at most 4 M e^{-(N - 1) s} / (e^s - 1), M the mean of |K| over the
    // ellipse (half of it has h < 0, where |K| is below 1): N >= (log M + log(4 / (1 - e^-s)) - log eps) / s
    // for the best s.  Half of the N points are rows; of the alphas the one with the least nodes is taken
    // (their columns estimated as linear in sin(theta), at 8 rows).
    const double zp = std::sqrt(std::max(rp * rp - rho * rho, 0.0));
    auto points = [&](const Tables::Ellipse &e) {   // N of this ellipse
        double ex[N_TAU], most = 0.0;
        for (int t = 0; t < N_TAU; ++t) {
            const double a = theta_max * e.re[t], h = theta_max * e.im[t], eh = std::exp(h);
            const double sh = 0.5 * (eh - 1.0 / eh), ch = 0.5 * (eh + 1.0 / eh), ch2 = 0.5 * (ch + 1.0);   // cosh^2(h / 2)
            const double near = q * ch2 * eh;
            if (!(near <= 0.7)) return 1e300;
            const double ca = std::fabs(std::cos(a)), sa = std::fabs(std::sin(a));
            const double reach = rp * ca <= rho ? rp : rho * ca + zp * sa;   // of the points of the sphere and the cylinder
            ex[t] = in.k_max * reach * sh * (1.0 + q * ch) + 2.0 * std::log(ch2 / ((1.0 - near) * (1.0 - near)));
            most = std::max(most, ex[t]);
        }
        double mean = 0.0;
        for (int t = 0; t < N_TAU; ++t) mean += std::exp(ex[t] - most) / (2 * N_TAU);
        return (std::log(mean) + most + e.lead - logeps) / e.s;
    };
    int rows = 0;
    double least = 1e300;
    auto try_alpha = [&](int a) {   // whether it is the best so far
        double n_rows = 1e300;
        int at = N_S - 1;
        for (int i = N_S - 1; i >= 0; i -= 3) {   // one minimum: in steps of 3, then its neighbours
            const double n = points(T.ell[a][i]);
            if (n > n_rows) break;
            n_rows = n;
            at = i;
        }
        for (int i = std::max(0, at - 2); i <= std::min(N_S - 1, at + 2); ++i)
            if (i != at) n_rows = std::min(n_rows, points(T.ell[a][i]));
        if (!(0.5 * n_rows < COMPACT_MAX_ROWS)) return false;
        const int n = std::max(2, (int)std::ceil(0.5 * n_rows));
        double nodes = 0.0;
        for (int m = 0; m < 8; ++m) nodes += (half0 + half1 * std::sin(theta_max * T.node[a][m])) * n;
        if (nodes >= least) return false;
        least = nodes;
        rows = n;
        plan.alpha = ALPHAS[a];
        plan.beta = T.beta[a];
        return true;
    };
    // one minimum over the alphas too
    try_alpha(2);
    int a = 3;
    for (; a < N_ALPHA && try_alpha(a); ++a) {}
    if (a == 3)
        for (a = 1; a >= 0 && try_alpha(a); --a) {}
    if (rows == 0 || rows > in.n_r) return false;

    const int own = in.n_phi % 2 ? 2 * in.n_phi : in.n_phi;   // the grid's phi, and those + pi
    int64_t n_c = 0, n_pad = 0, n_w = 0;
    for (int m = 0; m < rows; ++m) {
        const double half = columns(theta_max / plan.beta * std::asin(plan.alpha * std::cos((2 * m + 1) * M_PI / (4.0 * rows))), eta1);
        int p = half < 30000.0 ? 2 * std::max(1, (int)std::ceil(half)) - 1 : own;
        if (p >= own) p = own;
        if (p > 65535) return false;
        plan.cols[m] = (uint16_t)p;
        plan.off[m] = (int32_t)n_c;
        plan.poff[m] = (int32_t)n_pad;
        plan.woff[m] = (int32_t)n_w;
        n_c += p;
        n_pad += (p + 15) / 16 * 16;
        n_w += angular_kept(p);
    }
    if (n_c > 65536 || 2 * n_c > n_tot) return false;
    plan.off[rows] = (int32_t)n_c;
    plan.poff[rows] = (int32_t)n_pad;
    plan.woff[rows] = (int32_t)n_w;
    plan.rows = rows;
    plan.fold = in.n_phi % 2 == 0;
    plan.n_c = (int)n_c;
    plan.theta_max = theta_max;

    // The quadrature's chunk, at least 64 nodes.  FP64 (tiles of 64 points x 2 frequencies per wave): about
    // four rounds of tiles over the resident waves, so that the last round's empty slots stay below a
    // quarter of the time and the partials below 252 MB (20480 tiles of 64 x 2 x 12 x 8 bytes) plus one chunk's.  FP32 (128 points x 4
    // frequencies per workgroup): about four rounds of workgroups, and no more than 256 nodes, because a
    // chunk is one FP32 sum.
    if (in.fp64) {
        const int64_t units = (int64_t)(in.n_obs_pad / 64) * ((in.n_k + 1) / 2), chunks = (20480 + units - 1) / units;
        plan.chunk = (int)std::max<int64_t>(64, ((n_c + chunks - 1) / chunks + 31) / 32 * 32);
    } else {
        const int64_t units = (int64_t)(in.n_obs_pad / 128) * ((in.n_k + 3) / 4), chunks = (4096 + units - 1) / units;
        plan.chunk = (int)std::min<int64_t>(MM_CHUNK_MAX, std::max<int64_t>(64, ((n_c + chunks - 1) / chunks + 31) / 32 * 32));
    }
    // Near the focus H = (ik - 1/R) G / R is G / R times (ik - 1/|r_s|) to q / (k f) and J~ G is G / R times
    // J~ |r_s| (1 + delta / |r_s|).  The columns that r' multiplies need one part of two below q = 1/1000, where
    // their 11 bits are 23 of the sum's.  (With one part up to 1/100 a beam's B at q = 0.0099 and k r' = 6 erred by
    // 5.2e-7 against the direct sum's 1.3e-7, random tables at k r' = 19 by 1.3e-6 against 7.5e-7.)
    plan.form = q <= 1e-3 ? (q <= 1e-9 * in.k_min * in.f ? FORM_NEAR : FORM_GH) : FORM_GH_FAR;
    plan.scale = std::ldexp(1.0, std::ilogb(in.f));
    // The radii's sum: cut until there are about 1024 waves of it, at least 32 radii each, at most 8 parts.
    const int tiles = plan.fold ? (in.n_phi / 2 + 15) / 16 * ((rows + 15) / 16) : (in.n_phi + 15) / 16 * ((2 * rows + 15) / 16);
    const int64_t waves = (int64_t)in.n_k * tiles;
    plan.split = (int)std::max<int64_t>(
        1, std::min<int64_t>({(1024 + waves - 1) / waves, (in.n_r + 1) / 32, (int64_t)COMPACT_MAX_SPLIT}));
    if ((double)n_w * own > 8e6 || (double)rows * in.n_r > 4e6 ||
        (double)plan.split * rows * in.n_phi > 1e6)   // far outside: keep the sizes below in range
        return false;
    const int64_t fixed = 8 * (compact_radial_doubles(plan, in.n_r) + compact_angular_doubles(plan, in.n_phi));
    const int64_t row_bytes = 8 * compact_rows_doubles(plan, in.n_phi);
    // of a frequency: records, packed rows of the FP32 sum, and per 64 points the partials
    const int64_t tab_bytes = in.fp64 ? 64 * n_c : 32 * n_c + (form_rows(plan.form) * 1024 / form_nodes(plan.form)) * (n_c + 7) + 4096;
    const int64_t part_bytes = 64 * 12 * (in.fp64 ? 8 : 4) * ((n_c + plan.chunk - 1) / plan.chunk);
    const int64_t room = COMPACT_SCRATCH - 64 * (n_c + 7) - fixed;   // (less the node records)
    if (fixed + row_bytes > COMPACT_WORK_MAX || row_bytes + tab_bytes + 2 * part_bytes > room) return false;
    // Weights that fill the scratch leave an evaluation without allocation slabs of a few frequencies,
    // each with launches of its own.
    const int64_t per_k = std::max<int64_t>(1, room / (row_bytes + tab_bytes + in.n_obs_pad / 64 * part_bytes));
    const double slabs = fixed > 24 << 20 ? (double)((in.n_k + per_k - 1) / per_k) : 1.0;

    const double compact = std::max((in.fp64 ? 0.3 : 0.15) * plan.chunk, pts * (double)n_c * (in.fp64 ? 5.3 : 1.2) / cyc);
    const double build = (double)in.n_k * 0.5 * ((in.n_r + 1.0) * 256.0 * tiles * (plan.fold ? 2 : 1) + (double)n_c * own);
    return compact + 0.7 * (launches * slabs + 1.5 * build / cyc) < direct;
}

}  // namespace sc

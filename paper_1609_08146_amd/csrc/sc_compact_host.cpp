// sc_compact_host.cpp -- sizes of the compacted sum (see sc_compact.h): how many rows and columns
// interpolate the kernel to rounding, and whether the compacted sum is the faster one.
#include "sc_compact.h"

#include <algorithm>
#include <cmath>
#include <cstring>

namespace sc {

namespace {

// Interpolation error aimed at, relative to the largest kernel value, as the bounds below state it.
// The bounds are pessimistic: the errors met are 50 to 1000 times smaller, so 1e-8 gives about
// 1e-10 in the FP32 form (whose own rounding is 1e-7) and 1e-14 about 1e-16 in FP64.
constexpr double EPS_FP32 = 1e-8, EPS_FP64 = 1e-14;

constexpr int N_ETA = 80;             // widths of the strip of analyticity tried: 0.05 ... 4
constexpr double ETA_STEP = 0.05;

struct EtaTable {
    double sinh_[N_ETA], lead[N_ETA];   // sinh(eta), log(4 / (1 - e^-eta)) + eta
    EtaTable()
    {
        for (int i = 0; i < N_ETA; ++i) {
            const double e = ETA_STEP * (i + 1);
            sinh_[i] = std::sinh(e);
            lead[i] = std::log(4.0 / (1.0 - std::exp(-e))) + e;
        }
    }
};

}  // namespace

bool compact_plan(const CompactInput &in, CompactPlan &plan)
{
    static const EtaTable T;
    std::memset(&plan, 0, sizeof plan);   // plans are compared as bytes
    if (!(in.obs_r2max >= 0.0) || !(in.f > 0.0) || !(in.r_max > 0.0)) return false;
    const double rp = std::sqrt(in.obs_r2max), rho = std::sqrt(std::max(in.obs_rho2max, 0.0));
    const double q = rp / in.f;   // |r_s| >= f on the paraboloid
    // farther out the singularity R = 0 comes near the strip (and few nodes would be saved)
    if (!(q <= 0.25) || !std::isfinite(in.k_max * rp)) return false;
    const double theta_max = 2.0 * std::atan(in.r_max / (2.0 * in.f));
    const double logeps = std::log(in.fp64 ? EPS_FP64 : EPS_FP32);

    // Rows.  On the complex theta with |Im theta| <= h the phase k delta, delta = |r_s - r'| - |r_s|,
    // has an imaginary part of at most k |r'| sinh(h) (1 + q cosh h) and R stays away from 0 while
    // q cosh^2(h / 2) e^h < 1.  [0, theta_max] mapped to [-1, 1]: the ellipse with parameter
    // s = asinh(2 h / theta_max) lies in that strip, and interpolation at N Chebyshev points errs by
    // at most 4 M e^{-N s} / (e^s - 1), M the largest |K| on the ellipse: N >= (log M + log(4 / (e^s
    // - 1)) - log eps) / s for the best s.
    double n_rows = 1e300;
    for (int i = 0; i < 60; ++i) {
        const double h = ETA_STEP * (i + 1), ch2 = std::cosh(0.5 * h);
        const double near = q * ch2 * ch2 * std::exp(h);
        if (near > 0.7) break;
        const double s = std::asinh(2.0 * h / theta_max);
        const double logm = in.k_max * rp * T.sinh_[i] * (1.0 + q * std::cosh(h)) - 4.0 * std::log1p(-near) +
                            4.0 * std::log(ch2) + std::log(4.0 / std::expm1(s));
        n_rows = std::min(n_rows, (logm - logeps) / s);
    }
    if (!(n_rows < COMPACT_MAX_ROWS)) return false;
    const int rows = std::max(3, (int)std::ceil(n_rows));
    if (rows > in.n_r) return false;

    // Columns of each row.  On |Im phi| <= eta the phase's imaginary part is at most
    // k rho' sin(theta) sinh(eta); P equispaced points (P odd) alias the harmonics beyond (P - 1) / 2,
    // which sum to at most 4 M e^{-eta (P + 1) / 2} / (1 - e^-eta).
    double amp[N_ETA];
    int n_eta = 0;
    for (; n_eta < N_ETA; ++n_eta) {
        const double near = q * std::exp(ETA_STEP * (n_eta + 1));
        if (near > 0.7) break;
        amp[n_eta] = T.lead[n_eta] - 3.0 * std::log1p(-near) - logeps;
    }
    int64_t n_c = 0, n_pad = 0;
    for (int m = 0; m < rows; ++m) {
        const double theta = 0.5 * theta_max * (1.0 + std::cos((2 * m + 1) * M_PI / (2.0 * rows)));
        const double x = in.k_max * rho * std::sin(theta);
        double half = 1e300;
        for (int i = 0; i < n_eta; ++i) half = std::min(half, (x * T.sinh_[i] + amp[i]) / (ETA_STEP * (i + 1)));
        int p = half < 30000.0 ? 2 * std::max(1, (int)std::ceil(half)) - 1 : in.n_phi;
        if (p >= in.n_phi) p = in.n_phi;
        if (p > 65535) return false;
        plan.cols[m] = (uint16_t)p;
        plan.off[m] = (int32_t)n_c;
        plan.poff[m] = (int32_t)n_pad;
        n_c += p;
        n_pad += (p + 15) / 16 * 16;
    }
    const int64_t n_tot = (int64_t)(in.n_r + 1) * in.n_phi;
    if (n_c > 65536 || 2 * n_c > n_tot) return false;
    plan.off[rows] = (int32_t)n_c;
    plan.poff[rows] = (int32_t)n_pad;
    plan.rows = rows;
    plan.n_c = (int)n_c;
    plan.theta_max = theta_max;

    // The quadrature's chunk, at least 64 nodes.  FP64 (tiles of 64 points x 2 frequencies per wave): about
    // four rounds of tiles over the resident waves, so that the last round's empty slots stay below a
    // quarter of the time and the partials below 125 MB plus one chunk's.  FP32 (128 points x 4
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
    // J~ |r_s| (1 + delta / |r_s|); the columns that r' multiplies need one part of two below q = 1/100.
    plan.form = q <= 1e-3 && q <= 1e-9 * in.k_min * in.f ? FORM_NEAR : q <= 0.01 ? FORM_GH : FORM_GH_FAR;
    plan.scale = std::ldexp(1.0, std::ilogb(in.f));
    // The radii's sum: cut until there are about 1024 waves of it, at least 32 radii each.
    const int64_t waves = (int64_t)in.n_k * ((in.n_phi + 15) / 16) * ((rows + 15) / 16);
    plan.split = (int)std::max<int64_t>(1, std::min<int64_t>((1024 + waves - 1) / waves, (in.n_r + 1) / 32));
    if ((double)n_pad * in.n_phi > 4e6 || (double)rows * in.n_r > 4e6 ||
        (double)plan.split * rows * in.n_phi > 1e6)   // far outside: keep the sizes below in range
        return false;
    if (8 * (compact_radial_doubles(plan, in.n_r) + compact_angular_doubles(plan, in.n_phi) +
             compact_rows_doubles(plan, in.n_phi)) > COMPACT_WORK_MAX)
        return false;

    // Which sum is faster, in SIMD cycles over the chip's 1024 SIMDs (measured rates: 1.5 cycles per
    // direct FP32 evaluation on the tied tables and 4.4 in FP64, 1.2 and 5.3 per compacted one; the
    // matrix instructions of the two interpolations at 32 FP64 flops per cycle), and for small
    // problems the serial chain of a wave (0.11 us per node of a 2048-node chunk against chunk nodes
    // and three more launches).
    const double pts = (double)in.n_k * in.n_obs_pad, cyc = 1024.0 * 2.2e3;   // cycles per us
    const double direct = std::max(0.11 * (double)std::min<int64_t>(n_tot, 2048),
                                   pts * (double)n_tot * (in.fp64 ? 4.4 : 1.5) / cyc);
    const double build = (double)in.n_k * 0.5 * ((double)n_tot * ((rows + 15) / 16 * 16) + (double)n_c * in.n_phi);
    const double compact = std::max(0.15 * std::min(plan.chunk, 512), pts * (double)n_c * (in.fp64 ? 5.3 : 1.2) / cyc) + build / cyc +
                           25.0;
    return compact < 0.8 * direct;
}

}  // namespace sc

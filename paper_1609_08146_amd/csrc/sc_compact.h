// sc_compact.h -- the compacted form of a mirror's sum, shared by the planner (host), the kernels
// that build the compacted tables and the host runtime.  Not part of the public ABI.
//
// The sum over the mirror is E(o) = sum_n K(o, n) c_n: c the table records (any incident field), K
// the kernel values e^{ik delta} / R and (ik - 1/R) e^{ik delta} R / R^2 of node n and point o.  As
// a function of the node's direction (theta, phi) seen from the focus, K is analytic and oscillates
// no faster than the phase k r'.(direction), so K(o, n) = sum_m L_m(n) K(o, m) over a few nodes m of
// an interpolation rule, to rounding, and
//   E(o) = sum_m K(o, m) c~_m,   c~_m = sum_n L_m(n) c_n:
// the same sum over every record, with the points' part taken over far fewer nodes.  On the
// paraboloid r = 2 f tan(theta / 2), |r_s| = f / cos^2(theta / 2), the nodes are a tensor grid in
// (r, phi) with equispaced phi, so L is a product: Chebyshev interpolation in theta to the n_r + 1 radii
// (the rim is one of them), and on each row trigonometric interpolation from cols[m] equispaced phi to
// the n_phi.  A meridian goes on through the vertex, K(-theta, phi) = K(theta, phi + pi), so theta is
// interpolated from 2 x `rows` points of [-theta_max, theta_max], of which half are the other half turned
// by pi.  They are Chebyshev points y of theta = theta_max asin(alpha y) / asin(alpha), and the
// interpolation is polynomial in y: Chebyshev points of theta itself crowd at both ends, where
// the kernel oscillates no faster than elsewhere and a row at the rim has the most columns; alpha spreads
// them, at the price of branch points at y = +-1 / alpha.  On a mirror of theta_max 41 degrees and points
// within 5.7 wavelengths of 800 nm +-16 %, for the FP32 form: 25 rows and 1799 nodes, 2066 with alpha near 0; in
// FP64 34 rows and 3168 nodes, 3422.
#pragma once

#include <stdint.h>

namespace sc {

constexpr int COMPACT_MAX_ROWS = 192;

// How the FP32 sum forms its kernel values (sc_quad_mm.hip): G and H of every node; the same with
// the columns that r' multiplies in two parts; or G / R alone, near the focus.
enum CompactForm { FORM_GH = 0, FORM_GH_FAR = 1, FORM_NEAR = 2 };
// Nodes per step and 16-byte rows per lane and step of the packed tables.
constexpr int form_nodes(int form) { return form == FORM_NEAR ? 8 : 4; }
constexpr int form_rows(int form) { return form == FORM_GH ? 1 : 2; }

constexpr int MM_CHUNK_MAX = 256;   // nodes per chunk of the FP32 sum

constexpr int COMPACT_MAX_SPLIT = 8;

struct CompactPlan {
    int rows;                               // interpolation rows in theta > 0
    int fold;                               // n_phi is even: phi + pi is a grid point too
    int n_c;                                // compacted nodes in all (sum of cols)
    int split;                              // parts the sum over the radii is cut into (partial rows)
    int chunk;                              // compacted nodes per split-K chunk of the quadrature
    int form;                               // CompactForm of the FP32 sum
    double scale;                           // power of two near f
    double theta_max;                       // 2 atan(r_max / 2f)
    double alpha, beta;                     // of the rows' spread; beta = asin(alpha)
    uint16_t cols[COMPACT_MAX_ROWS];        // phi per row: odd, or the grid's own and those + pi
    int32_t off[COMPACT_MAX_ROWS + 1];      // first compacted node of each row
    int32_t poff[COMPACT_MAX_ROWS + 1];     // the same with every row's columns rounded up to 16
    int32_t woff[COMPACT_MAX_ROWS + 1];     // and with the columns whose weights are kept (angular_kept)
};

// Working memory of the two interpolations (doubles): the radial weights [n_r + 1 rounded up to
// 4][compact_radial_stride], the angular weights of every row [n_phi][angular_kept], and
// the partial rows of one frequency [split][rows][n_phi][8]; with an odd n_phi, where theta < 0 needs
// weights and partial rows of its own, [2 n_phi] and [2 rows].  The planner keeps their sum below
// COMPACT_WORK_MAX bytes, and with a frequency's tables and its partials of OBS_PAD points below
// COMPACT_SCRATCH bytes, what an evaluation without allocation has.
constexpr int64_t COMPACT_WORK_MAX = 56 << 20, COMPACT_SCRATCH = 63 << 20;
// The weights of column p > P / 2 at phi are those of column P - p at -phi, another point of the grid, so
// half the columns are kept, rounded up to 16.  (All of them were more than the scratch holds for an odd
// n_phi of 500 and more with 5 000 nodes, which were then summed directly.)
constexpr int angular_kept(int cols) { return (cols / 2 + 16) / 16 * 16; }
// Even and odd part of L_m in theta, each rounded up to 16 rows; with an odd n_phi L_m and L_-m, together.
constexpr int compact_radial_stride(const CompactPlan &p)
{
    return p.fold ? 2 * ((p.rows + 15) / 16 * 16) : (2 * p.rows + 15) / 16 * 16;
}
inline int64_t compact_radial_doubles(const CompactPlan &p, int n_r)
{
    return (int64_t)((n_r + 4) / 4 * 4) * compact_radial_stride(p);
}
inline int64_t compact_angular_doubles(const CompactPlan &p, int n_phi)
{
    return (int64_t)p.woff[p.rows] * n_phi * (p.fold ? 1 : 2);
}
inline int64_t compact_rows_doubles(const CompactPlan &p, int n_phi)
{
    return (int64_t)p.split * p.rows * (p.fold ? 1 : 2) * n_phi * 8;
}

// Nodes per chunk that the direct sum would take for itself: as many tiles (64 points, the usual 4
// frequencies or 2 in FP64) as waves are resident, and at least 64 nodes.
inline int64_t direct_chunk_nodes(int64_t n_tot, int n_obs_pad, int n_k, bool fp64)
{
    const int f = fp64 ? 2 : 4, waves = fp64 ? 4096 : 5120;
    const int64_t units = (int64_t)(n_obs_pad / 64) * ((n_k + f - 1) / f);
    const int64_t want = (n_tot * units + waves - 1) / waves;
    return want < 64 ? 64 : (want + 31) / 32 * 32;
}

// What the plan depends on.
struct CompactInput {
    double f, r_max;       // paraboloid
    int n_r, n_phi;
    double k_max, k_min;
    int n_k, n_obs_pad;
    double obs_r2max;      // max |r'|^2 over the points
    double obs_rho2max;    // max x'^2 + y'^2
    bool fp64;
};

// Plans the compacted sum of a problem; false where it does not apply or does not pay, and the sum
// is then taken directly.  Depends on nothing but its input (no launch shape, no history).
bool compact_plan(const CompactInput &in, CompactPlan &plan);

}  // namespace sc

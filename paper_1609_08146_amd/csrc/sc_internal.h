// sc_internal.h -- host-side declarations shared by the C ABI (sc_api.cpp) and
// the kernel translation unit (sc_kernels.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sc_compact.h"
#include "sc_quadjob.h"

namespace sc {

// ---- launchers (all asynchronous on `stream`; return hipError_t)
// (hinv64[q], hinv32[q] = 1 / (2 |r_s|), 0 where |r_s| = 0)
hipError_t launch_node_tables(hipStream_t st, int n_r, int n_phi, double f, const double *r,
                              const double *wr, const double *cphi, const double *sphi, double dphi,
                              double *pos64, float *pos32, double *nrm, double *wgt, double *tan,
                              double *hinv64, float *hinv32);
// General surface: node records from surface nodes + n dS and boundary nodes + normal + dl.
hipError_t launch_surface_records(hipStream_t st, int n_surf, int n_rim, const double *xyz, const double *ndS,
                                  const double *rim_xyz, const double *rim_n, const double *rim_dl, double *pos64,
                                  float *pos32, double *nrm, double *wgt, double *tan,
                              double *hinv64, float *hinv32);
hipError_t launch_obs_prep(hipStream_t st, const double *xyz, int n_obs, int n_obs_pad, double *obs64,
                           float *obs32);
hipError_t launch_tables_from_fields(hipStream_t st, int n_k, int n_surf, int n_tot, const double *k,
                                     const double *pos64, const double *nrm, const double *wgt,
                                     const double *tan, const double *E, const double *B, double *tab64);
// beam: 0 linear Gaussian, 1 radially, 2 azimuthally polarised, 3 Laguerre-Gauss mode set
// (modes: device [n_modes][SC_LG_RECORD] = p, l, ex re, ex im, ey re, ey im, the normalisation
// C_{p,l} (including 1 / w0), unused; unused for the other beams)
constexpr int SC_LG_RECORD = 8;
// With `out` the factored tables and their test in the same pass (see FactorOut); kb: the frequency where
// |Jt| is expected largest, k |amplitude|.  With `out`, tab64 may be NULL; part and P (the power) may be.
struct FactorOut;
hipError_t launch_tables_beam(hipStream_t st, int n_k, int n_surf, int n_tot, const double *k, const double *pos64,
                              const double *nrm, const double *wgt, const double *tan, int beam, double w0, double pol,
                              const double *spectrum, int consistent, const double *modes, int n_modes, double *tab64,
                              int kb, const FactorOut *out, double *part, double *P);
// FP32 tables from the FP64 ones (tab64), or from FP32 split tables (src32, when tab64 is null)
hipError_t launch_tables_cast(hipStream_t st, int n_k, int n_tot, const double *k, const double *pos64,
                              const double *tab64, const float *src32, float *tab32, int naive);
// Incident power per frequency through the aperture, P[k] = 4 pi sum_surface W Re(E x B^*).(-z):
// from field tables E, B [n_k][n_tot][3] complex (launch_tables_beam does it for its own fields).
// `part` holds power_partial_count(n_k, n_tot) doubles of scratch; P is [n_k] (device).
hipError_t launch_power_fields(hipStream_t st, int n_k, int n_surf, int n_tot, const double *nrm, const double *wgt,
                               const double *E, const double *B, double *part, double *P);
int64_t power_partial_count(int n_k, int n_tot);
// tab[k][node] *= fac[k] (complex128 [n_k]) for the n_cplx complex numbers of each record (4 general,
// 2 factored); exactly one of tab64, tab32 non-null
hipError_t launch_tables_scale(hipStream_t st, int n_k, int n_tot, int n_cplx, const double *fac, double *tab64,
                               float *tab32);
// Factored tables (Jt = u s per node): tabf [n_k][n_tot][4] = (s, rho_t), posf [n_tot][8] =
// (x, y, z, |r_s|, u, 1 / (2|r_s|)) in FP32, tabf64 / posf64 the same in FP64 (each output may be
// NULL);
// the flags get bit 0 when some node's current has no single real direction
// within tol32 (relative to its largest |Jt| over k), bit 1 for tol64; bits 2 and 3 when some
// node's charge is not tied to its current (rho_t = -i beta s / k, beta real) within tol32, tol64
// (relative to its largest (|rho_t|^2 + |Jt / k|^2)^1/2).
struct FactorOut {
    const float *pos32;
    const double *pos64;
    double tol32, tol64;
    float *tabf, *posf, *betaf, *tabp;
    double *tabf64, *posf64, *betaf64;
    unsigned int *bad;     // [4]: word b is set to `epoch` for bit b
    unsigned int epoch;
};
hipError_t launch_tables_factor(hipStream_t st, int n_k, int n_tot, const double *k, const double *tab64,
                                const FactorOut &out);
// tabp[r] = (|s|, arg(s) / 2 pi) from the FP32 factored records tabf[r] = (s, rho_t), r < n_rec.
hipError_t launch_tables_polar(hipStream_t st, int64_t n_rec, const float *tabf, float *tabp);
// Maxwell-residual diagnostics (sc_diag.hip).  Stencil results [rows][13 n_pts][3] complex (double
// if is_f64, else float); work holds diag_slots() doubles per (row, point), mx 4 per row, out 1 per
// (row, point).  The time form reads [n_t * 5][13 n_pts][3] (times t_m + (j - 2) dt).
hipError_t launch_maxwell_freq(hipStream_t st, int is_f64, int n_k, int n_pts, double h, const double *k,
                               const void *E, const void *B, double *work, double *mx, double *out);
hipError_t launch_maxwell_time(hipStream_t st, int is_f64, int n_t, int n_pts, double h, double dt, const void *E,
                               const void *B, double *work, double *mx, double *out);
int diag_slots();
// Energy 1/2 dV sum (|2 Re E|^2 + |2 Re B|^2) per time row of [n_t][n_obs][3]; part: energy_partial_count(n_t).
int energy_partial_count(int n_t);
hipError_t launch_energy(hipStream_t st, int is_f64, int n_t, int n_obs, const void *E, const void *B, double half_dv,
                         double *part, double *W);
// The direct sums over all tiles of n_jobs jobs in device memory, or of the job `one` (jobs NULL, n_jobs 1);
// counter: QUAD_SEGMENTS * QUAD_COUNTER_STRIDE words, cleared here where the launch uses them.
hipError_t launch_quad(hipStream_t st, int mode, int obs_per_lane, int freq_per_lane, int waves_per_block,
                       int grid, const QuadJob &one, const QuadJob *jobs, int n_jobs, int64_t n_tiles,
                       unsigned int *counter);
// E, B [n_k][n_obs][3] at the points o0 ... o0 + n_o - 1 from partials of those points (n_o_pad padded).
// The compacted FP32 sums (sc_quad_mm.hip): packed rows of the compacted tables [n_k][n_c][8] for the matrix
// instructions (mtab: mm_table_bytes, mscale: [n_k][16]), and the quadrature over the tiles of one
// job or of several on the device, fpb (1, 2 or 4) frequencies per tile.
inline size_t mm_table_bytes(int n_k, int n_c, int form)
{
    return (size_t)n_k * ((n_c + form_nodes(form) - 1) / form_nodes(form)) * 1024 * form_rows(form);
}
size_t mm_scale_bytes(int n_k);   // of mscale: the scales, and the maxima they come from
hipError_t launch_mm_tables(hipStream_t st, int n_k, int n_c, int form, const double *k, double scale, const float *ctab,
                            const float *pos, float *mscale, void *mtab);
// (jobs whose tile0 counts the tiles that each XCD has before them; `per`: what it has in all)
inline int64_t mm_tiles_per_xcd(const QuadJob &j) { return (j.n_tiles + QUAD_SEGMENTS - 1) / QUAD_SEGMENTS; }
hipError_t launch_quad_mm_one(hipStream_t st, int fpb, const QuadJob &job);
hipError_t launch_quad_mm(hipStream_t st, int fpb, const QuadJob *jobs, int n_jobs, int64_t per);
// (E or B may be NULL; and in E2, B2 where given)
hipError_t launch_reduce(hipStream_t st, int mode, const void *partial, int n_chunks, int n_k, int n_o, int n_o_pad,
                         const double *k, int b_scale, int n_obs, int o0, void *E, void *B, void *E2, void *B2);
// Compacted tables (sc_compact.h): weights and node records, then the tables of frequencies k0 ...
// k0 + n_k - 1 (T: n_k x compact_rows_doubles) into out [n_k][n_c][8] of the precision.
hipError_t launch_compact_geometry(hipStream_t st, const CompactPlan &plan, int n_r, int n_phi, double f,
                                   const double *r, double *wrad, double *wang, int is_f64, void *pos, void *hinv);
hipError_t launch_compact_tables(hipStream_t st, const CompactPlan &plan, int n_r, int n_phi, int k0, int n_k,
                                 int is_f64, int fact, const void *tab, const void *pos, const double *wrad,
                                 const double *wang, double *T, void *out);
// Twiddles of the transform to time (twiddle_bytes), and E, B [n_k][n_x] complex -> Et, Bt [n_t][n_x].
size_t twiddle_bytes(int n_k, int n_t);
hipError_t launch_twiddles(hipStream_t st, int n_k, const double *k, int n_t, const double *t, double dk,
                           double *tw);
hipError_t launch_time(hipStream_t st, int is_f64, int n_k, int n_t, int64_t n_x, const double *tw, const void *E,
                       const void *B, void *Et, void *Bt);
hipError_t launch_fill_u32(hipStream_t st, unsigned int *p, unsigned int v, int n);

// Occupancy helper: max resident workgroups per CU for a quadrature variant.
int quad_max_blocks_per_cu(int mode, int obs_per_lane, int freq_per_lane, int waves_per_block);

}  // namespace sc

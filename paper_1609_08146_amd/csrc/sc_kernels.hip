// sc_kernels.hip -- gfx950 kernels of the Stratton-Chu mirror-focusing path.
//
//  k_node_tables         mirror nodes, normals, weights            (Sec. III-C)
//  k_obs_prep            observation records
//  k_tables_from_fields  POA current / charge tables from given E_inc, B_inc
//  k_tables_beam         same for the built-in collimated beams: linearly, radially or azimuthally
//                        polarised Gaussian, Laguerre-Gauss modes (Sec. III-A, IV-A); with the
//                        factored tables in the same pass
//  k_tables_cast         FP64 tables -> FP32 (split: as is; naive: node phase removed)
//  k_tables_factor       FP64 tables -> factored FP32 / FP64 tables J~ = u s, when the current
//                        of every node keeps one real direction over the frequencies, and
//                        the real beta of the charge tied to it, rho_t = -i beta s / k
//  k_power_*             incident power per frequency through the aperture (Sec. III-B)
//  k_tables_scale        spectral amplitude / phase applied to the tables (Sec. III-B)
//  k_reduce<MODE>        deterministic split-K reduction into E, B
//  (the quadrature kernel itself is in sc_quad.hip)
//  k_twiddles, k_time    semi-discrete transform to time (Sec. III-B)
//
// All floating-point expressions are written with explicit fma/mul/add and
// the file is compiled with -ffp-contract=off, so the rounding sequence of
// every observation point is fixed by the source: results do not depend on
// the launch shape, only on the chunking.
#include "sc_device.h"
#include "sc_internal.h"

#include <algorithm>

namespace sc {

// ======================================================================= prep

// 1 / (2|r_s|) of a node in FP64 and FP32, for the series forms of delta and 1/|R| in the split quadrature (0
// for a node at the origin, where the series is never used).
__device__ __forceinline__ void store_half_inverse(double rs, int q, double *__restrict__ hinv64,
                                                   float *__restrict__ hinv32)
{
    const double h = rs > 0.0 ? 0.5 / rs : 0.0;
    hinv64[q] = h;
    hinv32[q] = (float)h;
}

__global__ void k_node_tables(int n_r, int n_phi, double f, const double *__restrict__ r,
                              const double *__restrict__ wr, const double *__restrict__ cphi,
                              const double *__restrict__ sphi, double dphi, double *__restrict__ pos64,
                              float *__restrict__ pos32, double *__restrict__ nrm, double *__restrict__ wgt,
                              double *__restrict__ tan, double *__restrict__ hinv64, float *__restrict__ hinv32)
{
    const int n_tot = (n_r + 1) * n_phi;
    const int64_t gq = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gq >= n_tot) return;
    const int q = (int)gq;
    const int i = q / n_phi;
    const int j = q - i * n_phi;
    const bool rim = (i == n_r);
    const double ri = r[i];            // r has n_r + 1 entries; r[n_r] = r_max
    const double c = cphi[j], s = sphi[j];
    const double x = ri * c;
    const double y = ri * s;
    const double z = ri * ri / (4.0 * f) - f;
    const dd rs = dd_norm3(x, y, z);
    pos64[4 * q + 0] = x;
    pos64[4 * q + 1] = y;
    pos64[4 * q + 2] = z;
    pos64[4 * q + 3] = rs.hi;
    pos32[4 * q + 0] = (float)x;
    pos32[4 * q + 1] = (float)y;
    pos32[4 * q + 2] = (float)z;
    pos32[4 * q + 3] = (float)rs.hi;
    store_half_inverse(rs.hi, q, hinv64, hinv32);
    // d r_s/dr x d r_s/dphi = r (-F'(r) cos, -F'(r) sin, 1), F'(r) = r / 2f
    const double dFdr = ri / (2.0 * f);
    nrm[3 * q + 0] = -dFdr * c;
    nrm[3 * q + 1] = -dFdr * s;
    nrm[3 * q + 2] = 1.0;
    wgt[q] = rim ? dphi : wr[i] * ri * dphi;
    if (rim) {
        tan[3 * j + 0] = -ri * s;
        tan[3 * j + 1] = ri * c;
        tan[3 * j + 2] = 0.0;
    }
}

// Node records of a general surface given by its quadrature: surface nodes with
// their area-weighted normals n dS (weight 1), then the boundary nodes with the
// surface normal there (direction only), weight 1 and the oriented line
// element dl in `tan`.
__global__ void k_surface_records(int n_surf, int n_rim, const double *__restrict__ xyz,
                                  const double *__restrict__ ndS, const double *__restrict__ rim_xyz,
                                  const double *__restrict__ rim_n, const double *__restrict__ rim_dl,
                                  double *__restrict__ pos64, float *__restrict__ pos32, double *__restrict__ nrm,
                                  double *__restrict__ wgt, double *__restrict__ tan, double *__restrict__ hinv64,
                                  float *__restrict__ hinv32)
{
    const int64_t gq = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gq >= (int64_t)n_surf + n_rim) return;
    const int q = (int)gq;
    const bool rim = q >= n_surf;
    const int j = q - n_surf;
    const double *src = rim ? rim_xyz + 3 * j : xyz + 3 * q;
    const double *nv = rim ? rim_n + 3 * j : ndS + 3 * q;
    const double x = src[0], y = src[1], z = src[2];
    const dd rs = dd_norm3(x, y, z);
    pos64[4 * q + 0] = x;
    pos64[4 * q + 1] = y;
    pos64[4 * q + 2] = z;
    pos64[4 * q + 3] = rs.hi;
    pos32[4 * q + 0] = (float)x;
    pos32[4 * q + 1] = (float)y;
    pos32[4 * q + 2] = (float)z;
    pos32[4 * q + 3] = (float)rs.hi;
    store_half_inverse(rs.hi, q, hinv64, hinv32);
    for (int c = 0; c < 3; ++c) nrm[3 * q + c] = nv[c];
    wgt[q] = 1.0;
    if (rim)
        for (int c = 0; c < 3; ++c) tan[3 * j + c] = rim_dl[3 * j + c];
}

__global__ void k_obs_prep(const double *__restrict__ xyz, int n_obs, int n_obs_pad, double *__restrict__ obs64,
                           float *__restrict__ obs32)
{
    const int64_t go = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (go >= n_obs_pad) return;
    const int o = (int)go;
    const int src = (o < n_obs) ? o : 0;   // padding repeats a valid point; its result is discarded
    const double x = xyz[3 * src], y = xyz[3 * src + 1], z = xyz[3 * src + 2];
    const double r2 = __fma_rn(x, x, __fma_rn(y, y, z * z));
    obs64[4 * o + 0] = x;
    obs64[4 * o + 1] = y;
    obs64[4 * o + 2] = z;
    obs64[4 * o + 3] = r2;
    obs32[4 * o + 0] = (float)x;
    obs32[4 * o + 1] = (float)y;
    obs32[4 * o + 2] = (float)z;
    obs32[4 * o + 3] = (float)r2;
}

// complex helpers (FP64)
struct c64 {
    double re, im;
};
__device__ __forceinline__ c64 cmul(c64 a, c64 b)
{
    return {__fma_rn(a.re, b.re, -(a.im * b.im)), __fma_rn(a.re, b.im, a.im * b.re)};
}

// Write one table record from the fields at node q (without/with phase folded by caller).
// P is the node phase factor; for surface nodes uses E, B; for rim nodes B only.
__device__ __forceinline__ void write_record(double *__restrict__ rec, bool rim, double k, double W,
                                             const double *n, const double *t, const c64 *E, const c64 *B,
                                             c64 P)
{
    if (!rim) {
        // J = n~ x B_inc, rho = n~ . E_inc
        c64 J[3], rho;
        J[0] = {n[1] * B[2].re - n[2] * B[1].re, n[1] * B[2].im - n[2] * B[1].im};
        J[1] = {n[2] * B[0].re - n[0] * B[2].re, n[2] * B[0].im - n[0] * B[2].im};
        J[2] = {n[0] * B[1].re - n[1] * B[0].re, n[0] * B[1].im - n[1] * B[0].im};
        rho = {n[0] * E[0].re + n[1] * E[1].re + n[2] * E[2].re, n[0] * E[0].im + n[1] * E[1].im + n[2] * E[2].im};
        const double cR = 2.0 * W / FOUR_PI;   // rho_t = cR rho P
        const double cJ = k * cR;              // Jt = i cJ J P
        for (int c = 0; c < 3; ++c) {
            c64 v = cmul(J[c], P);
            rec[2 * c + 0] = -cJ * v.im;
            rec[2 * c + 1] = cJ * v.re;
        }
        c64 v = cmul(rho, P);
        rec[6] = cR * v.re;
        rec[7] = cR * v.im;
    } else {
        // b = [n^ x (n^ x B)] . t = (n^ (n^ . B) - B) . t,   n^ = n~ / |n~|
        const double nn = n[0] * n[0] + n[1] * n[1] + n[2] * n[2];
        c64 nB = {n[0] * B[0].re + n[1] * B[1].re + n[2] * B[2].re, n[0] * B[0].im + n[1] * B[1].im + n[2] * B[2].im};
        c64 b = {0.0, 0.0};
        for (int c = 0; c < 3; ++c) {
            b.re += (n[c] * nB.re / nn - B[c].re) * t[c];
            b.im += (n[c] * nB.im / nn - B[c].im) * t[c];
        }
        // line term -(2/ik) sum W grad g b  ->  rho_t = i (2 W / (4 pi k)) b P
        const double cL = 2.0 * W / (FOUR_PI * k);
        c64 v = cmul(b, P);
        for (int c = 0; c < 6; ++c) rec[c] = 0.0;
        rec[6] = -cL * v.im;
        rec[7] = cL * v.re;
    }
}

__global__ void k_tables_from_fields(int n_k, int n_surf, int n_tot, const double *__restrict__ kv,
                                     const double *__restrict__ pos64, const double *__restrict__ nrm,
                                     const double *__restrict__ wgt, const double *__restrict__ tan,
                                     const double *__restrict__ Ein, const double *__restrict__ Bin,
                                     double *__restrict__ tab64)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n_k * n_tot) return;
    const int kk = (int)(idx / n_tot);
    const int q = (int)(idx - (int64_t)kk * n_tot);
    const double k = kv[kk];
    const double *p = pos64 + 4 * q;
    const dd rs = dd_norm3(p[0], p[1], p[2]);
    double sp, cp;
    sincos(phase_mod_2pi(k, rs), &sp, &cp);   // P = e^{ik|r_s|}
    c64 E[3], B[3];
    const double *e = Ein + idx * 6, *b = Bin + idx * 6;
    for (int c = 0; c < 3; ++c) {
        E[c] = {e[2 * c], e[2 * c + 1]};
        B[c] = {b[2 * c], b[2 * c + 1]};
    }
    const bool rim = q >= n_surf;
    write_record(tab64 + idx * 8, rim, k, wgt[q], nrm + 3 * q, rim ? tan + 3 * (q - n_surf) : nullptr, E, B,
                 {cp, sp});
}

// Incident collimated beams travelling along -z at node (X, Y), without their
// propagation phase e^{-ikz} (the table kernel fuses that with the node phase;
// the power kernel does not need it).  Sec. III-A.
//   beam 0, linearly polarised Gaussian, psi = amp exp(-(x^2+y^2)/w0^2) in the
//     frame where the polarisation is along x (`pol` rotates it about z):
//     literal E = x psi, B = -y psi; curl-consistent B = psi (0, -1, -2iy/(k w0^2)),
//     E = (i/k) curl B;
//   beam 1, radially polarised, g = amp exp(-r^2/w0^2) / w0:
//     E = (x, y, c) g, B = (y, -x, 0) g;
//   beam 2, azimuthally polarised: E = (-y, x, 0) g, B = (x, y, c) g;
//   with c = (2i/k)(r^2/w0^2 - 1) for the curl-consistent variants (E = (i/k) curl B,
//   resp. B = (-i/k) curl E) and c = 0 for the literal ones (B = -z x E).  The
//   cylindrical beams are axisymmetric, so `pol` does not enter;
//   beam 3, a Laguerre-Gauss mode set (lg_shape), literal.
// Laguerre-Gauss mode set (Sec. III-A: the Laguerre-Gauss modes of the paraxial wave equation are
// the expansion basis of the incident beams), each mode in its waist cross-section carried along -z:
//   u_{p,l} = C_{p,l} ((X + i sgn(l) Y) sqrt(2) / w0)^|l| L_p^|l|(2 r^2 / w0^2) exp(-r^2 / w0^2),
//   C_{p,l} = sqrt(2 p! / (pi (p + |l|)!)) / w0   (unit power over the plane),
// that is (sqrt(2) r / w0)^|l| e^{i l phi} times the radial factor, with L_p^a by its three-term
// recurrence.  modes: [n_modes][SC_LG_RECORD] = (p, l, ex re, ex im, ey re, ey im, C_{p,l}, unused),
// C from the host (it does not depend on the position; a device lgamma here cost the table
// kernels 72 VGPRs and 380 bytes of scratch per lane);
//   E = sum_m (ex_m x + ey_m y) u_m amp,   B = (-z) x E = sum_m (ey_m x - ex_m y) u_m amp.
//
// What does not depend on the frequency is a node's BeamShape, formed once per thread (the exponential,
// the sine of the polarisation angle, the mode sum); beam_at adds the frequency's amplitude.
struct BeamShape {
    double x, y, G;   // beam 0: position in the frame of the polarisation, else (X, Y); amplitude at it
    double cl, sl;    // beam 0: cosine and sine of the polarisation angle
    c64 ex, ey;       // beam 3: the mode sum
};

__device__ __forceinline__ void lg_shape(const double *__restrict__ modes, int n_modes, double X, double Y,
                                         double w0, BeamShape &b)
{
    const double s2w = 1.4142135623730951 / w0;
    const double t = 2.0 * (X * X + Y * Y) / (w0 * w0);
    const double gauss = exp(-0.5 * t);
    c64 ex = {0.0, 0.0}, ey = {0.0, 0.0};
    for (int m = 0; m < n_modes; ++m) {
        const double *md = modes + SC_LG_RECORD * m;
        const int p = (int)md[0], l = (int)md[1], al = l < 0 ? -l : l;
        // L_p^al(t): L_0 = 1, L_1 = 1 + al - t, (n + 1) L_{n+1} = (2n + 1 + al - t) L_n - (n + al) L_{n-1}
        double l0 = 1.0, l1 = 1.0 + al - t;
        const double lag = p == 0 ? 1.0 : l1;
        for (int n = 1; n < p; ++n) {
            const double l2 = ((2.0 * n + 1.0 + al - t) * l1 - (n + al) * l0) / (n + 1.0);
            l0 = l1;
            l1 = l2;
        }
        const double L = p <= 1 ? lag : l1;
        // ((X +- iY) sqrt(2) / w0)^|l|
        const c64 z1 = {X * s2w, (l < 0 ? -Y : Y) * s2w};
        c64 zp = {1.0, 0.0};
        for (int j = 0; j < al; ++j) zp = cmul(zp, z1);
        const double radial = md[6] * L * gauss;   // md[6]: the mode's normalisation C_{p,l}
        const c64 u = {radial * zp.re, radial * zp.im};
        const c64 cx = cmul(u, {md[2], md[3]}), cy = cmul(u, {md[4], md[5]});
        ex = {ex.re + cx.re, ex.im + cx.im};
        ey = {ey.re + cy.re, ey.im + cy.im};
    }
    b.ex = ex;
    b.ey = ey;
}

__device__ __forceinline__ BeamShape beam_shape(int beam, double X, double Y, double w0, double pol,
                                                const double *__restrict__ modes, int n_modes)
{
    BeamShape b = {};
    if (beam == 3) {
        lg_shape(modes, n_modes, X, Y, w0, b);
    } else if (beam != 0) {
        b.x = X;
        b.y = Y;
        b.G = exp(-(X * X + Y * Y) / (w0 * w0)) / w0;
    } else {
        sincos(pol, &b.sl, &b.cl);
        // frame where the polarisation is along x
        b.x = b.cl * X + b.sl * Y;
        b.y = -b.sl * X + b.cl * Y;
        b.G = exp(-(b.x * b.x + b.y * b.y) / (w0 * w0));
    }
    return b;
}

__device__ __forceinline__ void beam_at(int beam, const BeamShape &b, double k, double w0, c64 amp, int consistent,
                                        c64 *E, c64 *B)
{
    const c64 zero = {0.0, 0.0};
    if (beam == 3) {
        const c64 ex = cmul(b.ex, amp), ey = cmul(b.ey, amp);
        E[0] = ex;
        E[1] = ey;
        E[2] = zero;
        B[0] = ey;
        B[1] = {-ex.re, -ex.im};
        B[2] = zero;
        return;
    }
    const double x = b.x, y = b.y;
    if (beam != 0) {
        const c64 g = {b.G * amp.re, b.G * amp.im};
        const double r2 = x * x + y * y;
        const double c = consistent ? 2.0 / k * (r2 / (w0 * w0) - 1.0) : 0.0;   // longitudinal: i c g
        const c64 lg = {-c * g.im, c * g.re};
        const c64 rx = {x * g.re, x * g.im}, ry = {y * g.re, y * g.im};
        if (beam == 1) {
            E[0] = rx;
            E[1] = ry;
            E[2] = lg;
            B[0] = ry;
            B[1] = {-rx.re, -rx.im};
            B[2] = zero;
        } else {
            E[0] = {-ry.re, -ry.im};
            E[1] = rx;
            E[2] = zero;
            B[0] = rx;
            B[1] = ry;
            B[2] = lg;
        }
        return;
    }
    const c64 psi = {b.G * amp.re, b.G * amp.im};
    c64 e[3], bb[3];
    if (consistent) {
        const double kw2 = k * w0 * w0;
        const double c1 = 1.0 + 2.0 / (k * kw2) - 4.0 * y * y / (kw2 * kw2);
        const double c2 = 4.0 * x * y / (kw2 * kw2);
        const double c3 = 2.0 * x / kw2;    // E_z = i c3 psi
        const double c4 = -2.0 * y / kw2;   // B_z = i c4 psi
        e[0] = {c1 * psi.re, c1 * psi.im};
        e[1] = {c2 * psi.re, c2 * psi.im};
        e[2] = {-c3 * psi.im, c3 * psi.re};
        bb[0] = zero;
        bb[1] = {-psi.re, -psi.im};
        bb[2] = {-c4 * psi.im, c4 * psi.re};
    } else {
        e[0] = psi;
        e[1] = zero;
        e[2] = zero;
        bb[0] = zero;
        bb[1] = {-psi.re, -psi.im};
        bb[2] = zero;
    }
    E[0] = {b.cl * e[0].re - b.sl * e[1].re, b.cl * e[0].im - b.sl * e[1].im};
    E[1] = {b.sl * e[0].re + b.cl * e[1].re, b.sl * e[0].im + b.cl * e[1].im};
    E[2] = e[2];
    B[0] = {b.cl * bb[0].re - b.sl * bb[1].re, b.cl * bb[0].im - b.sl * bb[1].im};
    B[1] = {b.sl * bb[0].re + b.cl * bb[1].re, b.sl * bb[0].im + b.cl * bb[1].im};
    B[2] = bb[2];
}

// ------------------------------------------------------------ incident power
// Power of one frequency component of the incident beam through the mirror
// aperture (Sec. III-B, the Poynting integral that fixes each component's
// energy):  P_n = 4 pi SS Re(E_n x B_n^*) . dA  with dA = -z dx dy, since the
// beam travels along -z.  The surface weights W = w_r r dphi integrate over the
// aperture disk in the (x, y) plane, so P_n = 4 pi sum_q W_q Re(E x B^*) . (-z)
// over the surface nodes; for a general surface the aperture element of a node
// is the z component of its n dS, (n~ W).z (n~.z = 1 on the paraboloid).
// Deterministic: each part (64 nodes in k_tables_beam, one of POWER_BLOCKS ranges in
// k_power_fields) is summed in a fixed order, and so are the parts in k_power_finish.
constexpr int POWER_BLOCKS = 64;

__device__ __forceinline__ double flux_minus_z(const c64 *E, const c64 *B)
{
    // Re(E x B^*)_z = Re(E_x B_y^*) - Re(E_y B_x^*)
    return -((E[0].re * B[1].re + E[0].im * B[1].im) - (E[1].re * B[0].re + E[1].im * B[0].im));
}

__device__ __forceinline__ void block_sum_256(double v, double *out)
{
    __shared__ double red[256];
    red[threadIdx.x] = v;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) red[threadIdx.x] += red[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0) *out = red[0];
}

// grid (POWER_BLOCKS, n_k), 256 threads; E, B: [n_k][n_tot][3] complex
__global__ void __launch_bounds__(256) k_power_fields(int n_surf, int n_tot, const double *__restrict__ nrm,
                                                      const double *__restrict__ wgt,
                                                      const double *__restrict__ Ein,
                                                      const double *__restrict__ Bin, double *__restrict__ part)
{
    const int kk = blockIdx.y;
    const int span = (n_surf + POWER_BLOCKS - 1) / POWER_BLOCKS;
    const int q0 = blockIdx.x * span, q1 = min(q0 + span, n_surf);
    double acc = 0.0;
    for (int q = q0 + (int)threadIdx.x; q < q1; q += 256) {
        const double *e = Ein + ((size_t)kk * n_tot + q) * 6, *b = Bin + ((size_t)kk * n_tot + q) * 6;
        c64 E[3], B[3];
        for (int c = 0; c < 3; ++c) {
            E[c] = {e[2 * c], e[2 * c + 1]};
            B[c] = {b[2 * c], b[2 * c + 1]};
        }
        acc += (nrm[3 * q + 2] * wgt[q]) * flux_minus_z(E, B);
    }
    block_sum_256(acc, part + (size_t)kk * POWER_BLOCKS + blockIdx.x);
}

// One workgroup per frequency.
__global__ void __launch_bounds__(256) k_power_finish(int n_part, const double *__restrict__ part, double *__restrict__ P)
{
    double s = 0.0;
    for (int b = threadIdx.x; b < n_part; b += 256) s += part[(size_t)blockIdx.x * n_part + b];
    __shared__ double sum;
    block_sum_256(s, &sum);
    if (threadIdx.x == 0) P[blockIdx.x] = FOUR_PI * sum;
}

// Multiply every record of frequency k by the complex factor fac[k] (spectral
// amplitude and phase, Sec. III-B); tab64 in FP64, or tab32 (FP32 storage).
// n_cplx complex numbers per (k, node) record: 4 for the general tables, 2 for the factored ones (s, rho_t).
__global__ void k_tables_scale(int n_k, int n_tot, int n_cplx, const double *__restrict__ fac,
                               double *__restrict__ tab64, float *__restrict__ tab32)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n_k * n_tot) return;
    const int kk = (int)(idx / n_tot);
    const c64 f = {fac[2 * kk], fac[2 * kk + 1]};
    const int64_t base = idx * 2 * n_cplx;
    for (int c = 0; c < n_cplx; ++c) {
        if (tab64) {
            const c64 v = cmul({tab64[base + 2 * c], tab64[base + 2 * c + 1]}, f);
            tab64[base + 2 * c] = v.re;
            tab64[base + 2 * c + 1] = v.im;
        } else {
            const c64 v = cmul({(double)tab32[base + 2 * c], (double)tab32[base + 2 * c + 1]}, f);
            tab32[base + 2 * c] = (float)v.re;
            tab32[base + 2 * c + 1] = (float)v.im;
        }
    }
}

__global__ void k_tables_cast(int n_k, int n_tot, const double *__restrict__ kv, const double *__restrict__ pos64,
                              const double *__restrict__ tab64, const float *__restrict__ src32,
                              float *__restrict__ tab32, int naive)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (int64_t)n_k * n_tot) return;
    double v[8];
    for (int c = 0; c < 8; ++c) v[c] = tab64 ? tab64[idx * 8 + c] : (double)src32[idx * 8 + c];
    float *dst = tab32 + idx * 8;
    if (!naive) {
        for (int c = 0; c < 8; ++c) dst[c] = (float)v[c];
        return;
    }
    // remove the folded node phase: multiply by e^{-ik|r_s|}
    const int kk = (int)(idx / n_tot);
    const int q = (int)(idx - (int64_t)kk * n_tot);
    const double *p = pos64 + 4 * q;
    const dd rs = dd_norm3(p[0], p[1], p[2]);
    double sp, cp;
    sincos(phase_mod_2pi(kv[kk], rs), &sp, &cp);
    const c64 P = {cp, -sp};
    for (int c = 0; c < 4; ++c) {
        c64 w = cmul({v[2 * c], v[2 * c + 1]}, P);
        dst[2 * c] = (float)w.re;
        dst[2 * c + 1] = (float)w.im;
    }
}

// Factored tables.  The surface current of the integrand (Sec. II: J = n x B,
// folded into Jt with the weights and the node phase) often keeps one real
// direction at every frequency (e.g. a linearly polarised Gaussian with any
// spectrum, or a radially or azimuthally polarised beam): then
// Jt[k][q] = u_q s[k][q] and the quadrature can use u_q and s.  One thread per
// node q: u_q is the unit vector along the longer of Re Jt, Im Jt at the
// frequency kb where |Jt[k][q]| is largest (u_q = 0 if Jt vanishes), s = u_q . Jt.
// Often the charge is tied to that current as well: when E and B of the beam
// share one complex amplitude, n . E and n x B carry the same s, and with
// rho_t = (2W / 4 pi) (n . E) P against Jt = i k (2W / 4 pi) (n x B) P,
//   rho_t[k][q] = -i beta_q s[k][q] / k   with beta_q real,
// beta_q = k (Re rho_t Im s - Im rho_t Re s) / |s|^2 at kb.  A node without current
// (the rim, whose line term is a charge only) takes u_q = 0, beta_q = 1 and
// s = i k rho_t, which ties its charge exactly and leaves Jt = u s = 0.
// Bit 0 of the flags is set if |Jt[k][q] - u_q s[k][q]| > tol32 max_k |Jt[k][q]| for any
// node and k, bit 1 if it exceeds tol64; bits 2 and 3 the same for
// |rho_t[k][q] + i beta_q s[k][q] / k| against max_k (|rho_t[k][q]|^2 + |Jt[k][q] / k|^2)^1/2,
// the node's scale of the charge term (a charge that vanishes but for rounding, as
// n . E of the azimuthally polarised beam does, is tied with beta = 0).  The tables of a
// precision must not be used when its bit is set.  Outputs, each optional (NULL
// skips it): FP32 tabf[k][q] = (s, rho_t), posf[q] = (x, y, z, |r_s|, u_q, 1 / (2|r_s|)),
// betaf[q] = beta_q and tabp[k][q] = (|s|, arg(s) / 2 pi), s in polar form for the tied
// charge (the turn in (-1/2, 1/2]); FP64 tabf64, posf64 and betaf64, the same in double.
struct FactorDir {
    double u[3], beta;
    bool current;   // whether the node carries any
};

// From the node's record v (|Jt|^2 = m) at wavenumber k.
__device__ __forceinline__ FactorDir factor_dir(const double *v, double m, double k)
{
    FactorDir d = {{0.0, 0.0, 0.0}, 1.0, m > 0.0};
    if (!d.current) return d;
    const double re2 = v[0] * v[0] + v[2] * v[2] + v[4] * v[4];
    const double im2 = v[1] * v[1] + v[3] * v[3] + v[5] * v[5];
    const int part = re2 >= im2 ? 0 : 1;
    const double inv = 1.0 / sqrt(part ? im2 : re2);
    for (int c = 0; c < 3; ++c) d.u[c] = (part ? v[2 * c + 1] : v[2 * c]) * inv;
    const double sr = d.u[0] * v[0] + d.u[1] * v[2] + d.u[2] * v[4];
    const double si = d.u[0] * v[1] + d.u[1] * v[3] + d.u[2] * v[5];
    const double s2 = sr * sr + si * si;
    d.beta = s2 > 0.0 ? k * (v[6] * si - v[7] * sr) / s2 : 0.0;
    return d;
}

// s of the record v, and the squared residuals of the current (r2) and of the tied charge (t2).
// (ik = 1 / k)
__device__ __forceinline__ c64 factor_record(const double *v, double k, double ik, const FactorDir &d, double &r2,
                                             double &t2)
{
    c64 s;
    if (d.current) s = {d.u[0] * v[0] + d.u[1] * v[2] + d.u[2] * v[4], d.u[0] * v[1] + d.u[1] * v[3] + d.u[2] * v[5]};
    else s = {-k * v[7], k * v[6]};   // s = i k rho_t
    r2 = 0.0;
    for (int c = 0; c < 3; ++c) {
        const double dr = v[2 * c] - d.u[c] * s.re, di = v[2 * c + 1] - d.u[c] * s.im;
        r2 += dr * dr + di * di;
    }
    // rho_t + i beta s / k
    const double bk = d.beta * ik, tr = v[6] - bk * s.im, ti = v[7] + bk * s.re;
    t2 = tr * tr + ti * ti;
    return s;
}

__device__ __forceinline__ void factor_store(const FactorOut &o, int64_t rec, const double *v, c64 s)
{
    typedef float f4 __attribute__((ext_vector_type(4)));
    typedef float f2 __attribute__((ext_vector_type(2)));
    typedef double d2 __attribute__((ext_vector_type(2)));
    if (o.tabf) {
        *(f4 *)(o.tabf + rec * 4) = f4{(float)s.re, (float)s.im, (float)v[6], (float)v[7]};
        *(f2 *)(o.tabp + rec * 2) =
            f2{(float)sqrt(s.re * s.re + s.im * s.im), (float)(atan2(s.im, s.re) * INV_TWO_PI)};
    }
    if (o.tabf64) {
        d2 *t = (d2 *)(o.tabf64 + rec * 4);
        t[0] = d2{s.re, s.im};
        t[1] = d2{v[6], v[7]};
    }
}

__device__ __forceinline__ void factor_store_node(const FactorOut &o, int64_t q, const FactorDir &d)
{
    const double rs = o.pos64[q * 4 + 3], hinv = rs > 0.0 ? 0.5 / rs : 0.0;   // 1 / (2 |r_s|)
    if (o.posf) {
        float *pr = o.posf + q * 8;
        for (int c = 0; c < 4; ++c) pr[c] = o.pos32[q * 4 + c];
        for (int c = 0; c < 3; ++c) pr[4 + c] = (float)d.u[c];
        pr[7] = (float)hinv;
        o.betaf[q] = (float)d.beta;
    }
    if (o.posf64) {
        double *pr = o.posf64 + q * 8;
        for (int c = 0; c < 4; ++c) pr[c] = o.pos64[q * 4 + c];
        for (int c = 0; c < 3; ++c) pr[4 + c] = d.u[c];
        pr[7] = hinv;
        o.betaf64[q] = d.beta;
    }
}

// The bits of `flags` in FactorOut::bad, which needs no clearing between tests: each holds the last one it was set in.
__device__ __forceinline__ void factor_flags(const FactorOut &o, unsigned int flags)
{
    for (int b = 0; b < 4; ++b)
        if (flags >> b & 1u) o.bad[b] = o.epoch;
}

__device__ __forceinline__ double current2(const double *v)
{
    double m = 0.0;
    for (int c = 0; c < 6; ++c) m += v[c] * v[c];
    return m;
}

__global__ void k_tables_factor(int n_k, int n_tot, const double *__restrict__ kv, const double *__restrict__ tab64,
                                FactorOut o)
{
    const int64_t gq = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gq >= n_tot) return;
    double best = 0.0, bestr = 0.0;
    int kb = 0;
    for (int kk = 0; kk < n_k; ++kk) {
        const double *v = tab64 + ((int64_t)kk * n_tot + gq) * 8;
        const double m = current2(v), ik = 1.0 / kv[kk];
        if (m > best) {
            best = m;
            kb = kk;
        }
        bestr = fmax(bestr, v[6] * v[6] + v[7] * v[7] + m * (ik * ik));
    }
    const FactorDir dir = factor_dir(tab64 + ((int64_t)kb * n_tot + gq) * 8, best, kv[kb]);
    const double lim32 = o.tol32 * o.tol32 * best, lim64 = o.tol64 * o.tol64 * best;
    const double rlim32 = o.tol32 * o.tol32 * bestr, rlim64 = o.tol64 * o.tol64 * bestr;
    unsigned int flags = 0;
    for (int kk = 0; kk < n_k; ++kk) {
        const int64_t rec = (int64_t)kk * n_tot + gq;
        const double *v = tab64 + rec * 8;
        double r2, t2;
        const c64 s = factor_record(v, kv[kk], 1.0 / kv[kk], dir, r2, t2);
        if (!(r2 <= lim32)) flags |= 1u;
        if (!(r2 <= lim64)) flags |= 2u;
        if (!(t2 <= rlim32)) flags |= 4u;
        if (!(t2 <= rlim64)) flags |= 8u;
        factor_store(o, rec, v, s);
    }
    factor_store_node(o, gq, dir);
    factor_flags(o, flags);
}

// Four lanes' records of 8 doubles, written so that each store instruction writes whole records: the 4 x 4
// pieces of 16 bytes are transposed within the four lanes.
__device__ __forceinline__ double quad_xor(double x, int ctrl_xor2)
{
    const long long b = __double_as_longlong(x);
    int lo = (int)b, hi = (int)(b >> 32);
    if (ctrl_xor2) {
        lo = __builtin_amdgcn_mov_dpp(lo, 0x4E, 0xF, 0xF, true);   // quad_perm [2, 3, 0, 1]
        hi = __builtin_amdgcn_mov_dpp(hi, 0x4E, 0xF, 0xF, true);
    } else {
        lo = __builtin_amdgcn_mov_dpp(lo, 0xB1, 0xF, 0xF, true);   // quad_perm [1, 0, 3, 2]
        hi = __builtin_amdgcn_mov_dpp(hi, 0xB1, 0xF, 0xF, true);
    }
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
__device__ __forceinline__ void store_records(double *base, int count, const double *rec)
{
    typedef double d2 __attribute__((ext_vector_type(2)));
    const int j = threadIdx.x & 3;
    double v[8];
    for (int c = 0; c < 8; ++c) v[c] = rec[c];
    const bool b0 = j & 1, b1 = j & 2;
#pragma unroll
    for (int p = 0; p < 8; p += 4)
#pragma unroll
        for (int c = p; c < p + 2; ++c) {
            const double r = quad_xor(b0 ? v[c] : v[c + 2], 0);
            v[c] = b0 ? r : v[c];
            v[c + 2] = b0 ? v[c + 2] : r;
        }
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        const double r = quad_xor(b1 ? v[c] : v[c + 4], 1);
        v[c] = b1 ? r : v[c];
        v[c + 4] = b1 ? v[c + 4] : r;
    }
    for (int i = 0; i < 4; ++i)
        if (i < count) *(d2 *)(base + 8 * i + 2 * j) = d2{v[2 * i], v[2 * i + 1]};
}

template <int CTRL, int ROWS>
__device__ __forceinline__ double dpp_or_zero(double x)
{
    const long long b = __double_as_longlong(x);
    const int lo = __builtin_amdgcn_update_dpp(0, (int)b, CTRL, ROWS, 0xF, false);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(b >> 32), CTRL, ROWS, 0xF, false);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}
// The sum over a wave, in lane 63.
__device__ __forceinline__ double wave_sum_63(double x)
{
    x += dpp_or_zero<0x111, 0xF>(x);   // row_shr 1, 2, 4, 8: lane 15 of each row of 16 holds its sum
    x += dpp_or_zero<0x112, 0xF>(x);
    x += dpp_or_zero<0x114, 0xF>(x);
    x += dpp_or_zero<0x118, 0xF>(x);
    x += dpp_or_zero<0x142, 0xA>(x);   // row_bcast 15: rows 0, 2 into rows 1, 3
    x += dpp_or_zero<0x143, 0xC>(x);   // row_bcast 31: rows 0, 1 into rows 2, 3
    return x;
}

// The tables of a built-in beam, and with TEST their factored form and its test in the same pass (the two
// separate kernels wrote the FP64 tables once and read them twice: 0.51 + 0.67 ms at 128 frequencies and
// 160 400 nodes, 3.9 GB; now 0.41 ms with the FP64 tables, 1.8 GB, at the rate of a large copy, and 0.32
// without them, where the FP64 pipe bounds it).  Workgroups of 64 nodes x blockDim.y shares of the
// frequencies; what does not depend on the frequency is formed once per thread.  The node's direction is taken from its
// record at the host's guess of the largest, kb = argmax k |amplitude| (exact for a beam whose shape does
// not depend on the frequency), which is formed first; the largest |Jt| and the residuals are
// collected on the way and compared at the end.  Where the guess proves bad (less than half of the largest
// |Jt|), the pass is made again from the true one.  tab64 may be NULL (the FP64 tables not kept),
// and so may part and P.
constexpr int BEAM_PARTS = 8;
template <int beam, bool TEST>
__global__ void __launch_bounds__(64 * BEAM_PARTS) __attribute__((amdgpu_waves_per_eu(2)))
k_tables_beam(int n_k, int n_surf, int n_tot, const double *__restrict__ kv, const double *__restrict__ pos64,
              const double *__restrict__ nrm, const double *__restrict__ wgt, const double *__restrict__ tan, double w0, double pol, const double *__restrict__ spectrum, int consistent,
              const double *__restrict__ modes, int n_modes, double *__restrict__ tab64,
              double *__restrict__ power, int kb, FactorOut o)
{
    const int lane = threadIdx.x, part = __builtin_amdgcn_readfirstlane(threadIdx.y), parts = blockDim.y;
    const int64_t gq = (int64_t)blockIdx.x * 64 + lane;
    const bool valid = gq < n_tot;
    const int q = valid ? (int)gq : n_tot - 1;
    const int64_t q4 = gq & ~int64_t(3);   // the four lanes' first node, and how many of them there are
    const int n4 = (int)max(int64_t(0), min(int64_t(4), n_tot - q4));
    const double X = pos64[4 * (size_t)q], Y = pos64[4 * (size_t)q + 1], Z = pos64[4 * (size_t)q + 2];
    const BeamShape shape = beam_shape(beam, X, Y, w0, pol, modes, n_modes);
    // propagation phase e^{-ikz} fused with the node phase e^{ik|r_s|}: e^{ik(|r_s| - z)},
    // formed in double-double so that no ~1e6 rad phase is ever rounded to double
    const dd path = dd_sub_d(dd_norm3(X, Y, Z), Z);
    const bool rim = q >= n_surf;
    const double W = wgt[q];
    const double n[3] = {nrm[3 * (size_t)q], nrm[3 * (size_t)q + 1], nrm[3 * (size_t)q + 2]};
    double t[3] = {0.0, 0.0, 0.0};
    if (rim)
        for (int c = 0; c < 3; ++c) t[c] = tan[3 * (size_t)(q - n_surf) + c];
    const double flux_w = valid && !rim ? n[2] * W : 0.0;
    auto record = [&](int kk, double *v, bool store_power) {
        const double k = kv[kk];
        const c64 amp = spectrum ? c64{spectrum[2 * kk], spectrum[2 * kk + 1]} : c64{1.0, 0.0};
        c64 E[3], B[3];
        beam_at(beam, shape, k, w0, amp, consistent, E, B);
        double sp, cp;
        sincos(phase_mod_2pi(k, path), &sp, &cp);
        write_record(v, rim, k, W, n, t, E, B, {cp, sp});
        if (store_power && power) {
            const double sum = wave_sum_63(flux_w * flux_minus_z(E, B));
            if (lane == 63) power[(size_t)kk * gridDim.x + blockIdx.x] = sum;
        }
    };
    if constexpr (!TEST) {
        for (int kk = part; kk < n_k; kk += parts) {
            double v[8];
            record(kk, v, true);
            store_records(tab64 + ((int64_t)kk * n_tot + q4) * 8, n4, v);
        }
        return;
    } else {
        __shared__ double sh_best[BEAM_PARTS][64], sh_charge[BEAM_PARTS][64], sh_r2[BEAM_PARTS][64], sh_t2[BEAM_PARTS][64];
        __shared__ int sh_kb[BEAM_PARTS][64], sh_nan[BEAM_PARTS][64];
        for (int pass = 0;; ++pass) {
            double v[8];
            record(kb, v, false);
            const double mkb = current2(v);
            const FactorDir dir = factor_dir(v, mkb, kv[kb]);
            double best = 0.0, bestr = 0.0, r2max = 0.0, t2max = 0.0;
            int kbest = 0, nan = 0;
            for (int kk = part; kk < n_k; kk += parts) {
                record(kk, v, true);
                const int64_t rec = (int64_t)kk * n_tot + q;
                if (tab64) store_records(tab64 + ((int64_t)kk * n_tot + q4) * 8, n4, v);
                const double k = kv[kk], ik = 1.0 / k, m = current2(v);
                if (m > best) {
                    best = m;
                    kbest = kk;
                }
                bestr = fmax(bestr, v[6] * v[6] + v[7] * v[7] + m * (ik * ik));
                double r2, t2;
                const c64 s = factor_record(v, k, ik, dir, r2, t2);
                r2max = fmax(r2max, r2);
                t2max = fmax(t2max, t2);
                nan |= (r2 != r2 ? 3 : 0) | (t2 != t2 ? 12 : 0);
                if (valid) factor_store(o, rec, v, s);
            }
            sh_best[part][lane] = best;
            sh_charge[part][lane] = bestr;
            sh_r2[part][lane] = r2max;
            sh_t2[part][lane] = t2max;
            sh_kb[part][lane] = kbest;
            sh_nan[part][lane] = nan;
            __syncthreads();
            best = bestr = r2max = t2max = 0.0;
            kbest = nan = 0;
            for (int p = 0; p < parts; ++p) {
                if (sh_best[p][lane] > best) {
                    best = sh_best[p][lane];
                    kbest = sh_kb[p][lane];
                }
                bestr = fmax(bestr, sh_charge[p][lane]);
                r2max = fmax(r2max, sh_r2[p][lane]);
                t2max = fmax(t2max, sh_t2[p][lane]);
                nan |= sh_nan[p][lane];
            }
            const bool again = pass == 0 && mkb < 0.25 * best;
            if (__syncthreads_or(again)) {
                if (again) kb = kbest;
                continue;
            }
            if (part == 0 && valid) {
                unsigned int flags = (unsigned int)nan;
                if (r2max > o.tol32 * o.tol32 * best) flags |= 1u;
                if (r2max > o.tol64 * o.tol64 * best) flags |= 2u;
                if (t2max > o.tol32 * o.tol32 * bestr) flags |= 4u;
                if (t2max > o.tol64 * o.tol64 * bestr) flags |= 8u;
                factor_store_node(o, gq, dir);
                factor_flags(o, flags);
            }
            return;
        }
    }
}

// The polar records of the tied charge again from the FP32 factored records, after these were
// scaled in place (a spectral factor on FP32-only tables): tabp[r] = (|s|, arg(s) / 2 pi).
__global__ void k_tables_polar(int64_t n_rec, const float *__restrict__ tabf, float *__restrict__ tabp)
{
    const int64_t r = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (r >= n_rec) return;
    const double sr = tabf[r * 4], si = tabf[r * 4 + 1];
    tabp[r * 2] = (float)sqrt(sr * sr + si * si);
    tabp[r * 2 + 1] = (float)(atan2(si, sr) * INV_TWO_PI);
}

// Split-K reduction: E[k][o][c] = sum over chunks (in FP64, fixed order); B gets the 1/(ik) factor,
// less the part of 1/k that the quadrature's B sums carry already (b_scale).  Bound by the partials' read.
// One workgroup per frequency and 64 points, one wave per real of the record: a wave's loads are
// consecutive, and a small problem has 12 times the waves that one thread per point gave it; the
// records are put together in LDS and written as one run.
template <typename PT, typename OT>
__global__ void __launch_bounds__(768)
k_reduce(const PT *__restrict__ partial, int n_chunks, int n_k, int n_o, int n_obs_pad, const double *__restrict__ kv,
         int b_scale, int n_obs, int o0, OT *__restrict__ E, OT *__restrict__ B, OT *__restrict__ E2,
         OT *__restrict__ B2)
{
    const int groups = (n_o + 63) / 64, c = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int half = threadIdx.x < 384 ? 0 : 1, t = threadIdx.x - 384 * half;
    const size_t stride = (size_t)n_k * 12 * (size_t)n_obs_pad;
    __shared__ OT rec[2][384];
    for (int64_t b = blockIdx.x; b < (int64_t)n_k * groups; b += gridDim.x) {
        const int kk = (int)(b / groups), g = (int)(b - (int64_t)kk * groups);
        // partials [chunk][k][point / 64][12][64]
        const PT *p = partial + (size_t)kk * 12 * (size_t)n_obs_pad + (size_t)g * 768 + c * 64 + lane;
        double acc = 0.0;
#pragma unroll 8
        for (int ch = 0; ch < n_chunks; ++ch) acc += (double)p[ch * stride];
        const double k = kv[kk];   // 1/(ik) = -i/k
        const double ik_inv = b_scale == B_OVER_K ? 1.0 : (b_scale == B_OVER_K_POW2 ? ldexp(1.0, ilogb(k)) : 1.0) / k;
        // E: re, im of x, y, z; B: times -i / k, so the real part comes from the imaginary sum
        if (c < 6) rec[0][6 * lane + c] = (OT)acc;
        else if (c & 1) rec[1][6 * lane + c - 7] = (OT)(acc * ik_inv);
        else rec[1][6 * lane + c - 5] = (OT)(-acc * ik_inv);
        __syncthreads();
        if (64 * g + t / 6 < n_o) {
            const size_t at = ((size_t)kk * n_obs + o0 + 64 * g) * 6 + t;
            if (OT *first = half ? B : E) first[at] = rec[half][t];
            if (OT *second = half ? B2 : E2) second[at] = rec[half][t];
        }
        __syncthreads();
    }
}

// ================================================================ time transform

constexpr int TIME_MT = 8;   // time samples per thread (register tile)
__host__ __device__ constexpr int time_rows(int n_t) { return (n_t + TIME_MT - 1) / TIME_MT * TIME_MT; }

// tw[n][m] = dk * e^{-i k_n t_m}, m up to a multiple of TIME_MT (the last again); phase formed in
// double-double and reduced mod 2pi.
__global__ void k_twiddles(int n_k, const double *__restrict__ kv, int n_t, const double *__restrict__ t, double dk,
                           double *__restrict__ tw)
{
    const int64_t idx = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const int rows = time_rows(n_t);
    if (idx >= (int64_t)n_k * rows) return;
    const int n = (int)(idx / rows), m = min((int)(idx - (int64_t)n * rows), n_t - 1);
    double s, c;
    sincos(-phase_mod_2pi(kv[n], dd{t[m], 0.0}), &s, &c);
    tw[2 * idx] = dk * c;
    tw[2 * idx + 1] = dk * s;
}

// Constant-address-space view: wave-uniform loads through it become scalar loads.
typedef __attribute__((address_space(4))) const double cdouble;

// Ft[m][x] = sum_n F[n][x] tw[n][m] for E (blockIdx.z 0) and B, accumulated in FP64.  The twiddles are
// wave-uniform and read through scalar loads, the 8 of a frequency side by side: laid out [m][n] they were
// 8 lines per frequency, and two launches of half the waves took 187 us at 128 frequencies, 256 times and
// 4160 points, now 151 (3.3e9 FP64 multiply-adds, 84 us at the pipe's peak).
template <typename T>
__global__ void __launch_bounds__(256) k_time(int n_k, int n_t, int64_t n_x, const double *__restrict__ tw_,
                                              const T *__restrict__ E, const T *__restrict__ B, T *__restrict__ Et,
                                              T *__restrict__ Bt)
{
    typedef T t2 __attribute__((ext_vector_type(2)));
    const int m0 = blockIdx.y * TIME_MT, mt = min(TIME_MT, n_t - m0), rows = time_rows(n_t);
    cdouble *tw = (cdouble *)tw_ + 2 * m0;
    const t2 *F = (const t2 *)(blockIdx.z ? B : E);
    t2 *Ft = (t2 *)(blockIdx.z ? Bt : Et);
    const int64_t x = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (x >= n_x) return;
    double ar[TIME_MT], ai[TIME_MT];
#pragma unroll
    for (int mm = 0; mm < TIME_MT; ++mm) ar[mm] = ai[mm] = 0.0;
    for (int n = 0; n < n_k; ++n) {
        const t2 f = F[(size_t)n * n_x + x];
        const double fr = (double)f.x, fi = (double)f.y;
#pragma unroll
        for (int mm = 0; mm < TIME_MT; ++mm) {
            const double wr = tw[2 * ((size_t)n * rows + mm)], wi = tw[2 * ((size_t)n * rows + mm) + 1];
            ar[mm] = __fma_rn(fr, wr, __fma_rn(-fi, wi, ar[mm]));
            ai[mm] = __fma_rn(fr, wi, __fma_rn(fi, wr, ai[mm]));
        }
    }
    for (int mm = 0; mm < mt; ++mm) Ft[(size_t)(m0 + mm) * n_x + x] = t2{(T)ar[mm], (T)ai[mm]};
}

__global__ void k_fill_u32(unsigned int *p, unsigned int v, int n)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// ================================================================== launchers

static inline unsigned int nblocks(int64_t n, int bs) { return (unsigned int)((n + bs - 1) / bs); }

hipError_t launch_node_tables(hipStream_t st, int n_r, int n_phi, double f, const double *r, const double *wr,
                              const double *cphi, const double *sphi, double dphi, double *pos64, float *pos32,
                              double *nrm, double *wgt, double *tan, double *hinv64, float *hinv32)
{
    const int n = (n_r + 1) * n_phi;
    hipLaunchKernelGGL(k_node_tables, dim3(nblocks(n, 256)), dim3(256), 0, st, n_r, n_phi, f, r, wr, cphi, sphi,
                       dphi, pos64, pos32, nrm, wgt, tan, hinv64, hinv32);
    return hipGetLastError();
}

hipError_t launch_surface_records(hipStream_t st, int n_surf, int n_rim, const double *xyz, const double *ndS,
                                  const double *rim_xyz, const double *rim_n, const double *rim_dl, double *pos64,
                                  float *pos32, double *nrm, double *wgt, double *tan, double *hinv64, float *hinv32)
{
    hipLaunchKernelGGL(k_surface_records, dim3(nblocks((int64_t)n_surf + n_rim, 256)), dim3(256), 0, st, n_surf,
                       n_rim, xyz, ndS, rim_xyz, rim_n, rim_dl, pos64, pos32, nrm, wgt, tan, hinv64, hinv32);
    return hipGetLastError();
}

hipError_t launch_obs_prep(hipStream_t st, const double *xyz, int n_obs, int n_obs_pad, double *obs64, float *obs32)
{
    hipLaunchKernelGGL(k_obs_prep, dim3(nblocks(n_obs_pad, 256)), dim3(256), 0, st, xyz, n_obs, n_obs_pad, obs64,
                       obs32);
    return hipGetLastError();
}

hipError_t launch_tables_from_fields(hipStream_t st, int n_k, int n_surf, int n_tot, const double *k,
                                     const double *pos64, const double *nrm, const double *wgt, const double *tan,
                                     const double *E, const double *B, double *tab64)
{
    hipLaunchKernelGGL(k_tables_from_fields, dim3(nblocks((int64_t)n_k * n_tot, 256)), dim3(256), 0, st, n_k,
                       n_surf, n_tot, k, pos64, nrm, wgt, tan, E, B, tab64);
    return hipGetLastError();
}

hipError_t launch_tables_beam(hipStream_t st, int n_k, int n_surf, int n_tot, const double *k, const double *pos64,
                              const double *nrm, const double *wgt, const double *tan, int beam, double w0, double pol,
                              const double *spectrum, int consistent, const double *modes, int n_modes, double *tab64,
                              int kb, const FactorOut *out, double *part, double *P)
{
    // shares of the frequencies: until there are eight waves per SIMD
    const unsigned int nb = nblocks(n_tot, 64);
    int parts = 1;
    while (parts < BEAM_PARTS && 2 * parts <= n_k && (int64_t)nb * parts < 8192) parts *= 2;
#define SC_BEAM(BM, TEST)                                                                                          \
    hipLaunchKernelGGL((k_tables_beam<BM, TEST>), dim3(nb), dim3(64, parts), 0, st, n_k, n_surf, n_tot, k, pos64, nrm, \
                       wgt, tan, w0, pol, spectrum, consistent, modes, n_modes, tab64, part, kb,       \
                       out ? *out : FactorOut{})
    switch (beam + (out ? 4 : 0)) {
    case 0: SC_BEAM(0, false); break;
    case 1: SC_BEAM(1, false); break;
    case 2: SC_BEAM(2, false); break;
    case 3: SC_BEAM(3, false); break;
    case 4: SC_BEAM(0, true); break;
    case 5: SC_BEAM(1, true); break;
    case 6: SC_BEAM(2, true); break;
    default: SC_BEAM(3, true); break;
    }
#undef SC_BEAM
    if (part) hipLaunchKernelGGL(k_power_finish, dim3(n_k), dim3(256), 0, st, (int)nb, part, P);
    return hipGetLastError();
}

hipError_t launch_power_fields(hipStream_t st, int n_k, int n_surf, int n_tot, const double *nrm, const double *wgt,
                               const double *E, const double *B, double *part, double *P)
{
    hipLaunchKernelGGL(k_power_fields, dim3(POWER_BLOCKS, n_k), dim3(256), 0, st, n_surf, n_tot, nrm, wgt, E, B,
                       part);
    hipLaunchKernelGGL(k_power_finish, dim3(n_k), dim3(256), 0, st, POWER_BLOCKS, part, P);
    return hipGetLastError();
}

int64_t power_partial_count(int n_k, int n_tot) { return (int64_t)n_k * std::max<unsigned int>(POWER_BLOCKS, nblocks(n_tot, 64)); }

hipError_t launch_tables_scale(hipStream_t st, int n_k, int n_tot, int n_cplx, const double *fac, double *tab64,
                               float *tab32)
{
    hipLaunchKernelGGL(k_tables_scale, dim3(nblocks((int64_t)n_k * n_tot, 256)), dim3(256), 0, st, n_k, n_tot,
                       n_cplx, fac, tab64, tab32);
    return hipGetLastError();
}

hipError_t launch_tables_factor(hipStream_t st, int n_k, int n_tot, const double *k, const double *tab64,
                                const FactorOut &out)
{
    hipLaunchKernelGGL(k_tables_factor, dim3(nblocks(n_tot, 256)), dim3(256), 0, st, n_k, n_tot, k, tab64, out);
    return hipGetLastError();
}

hipError_t launch_tables_polar(hipStream_t st, int64_t n_rec, const float *tabf, float *tabp)
{
    hipLaunchKernelGGL(k_tables_polar, dim3(nblocks(n_rec, 256)), dim3(256), 0, st, n_rec, tabf, tabp);
    return hipGetLastError();
}

hipError_t launch_tables_cast(hipStream_t st, int n_k, int n_tot, const double *k, const double *pos64,
                              const double *tab64, const float *src32, float *tab32, int naive)
{
    hipLaunchKernelGGL(k_tables_cast, dim3(nblocks((int64_t)n_k * n_tot, 256)), dim3(256), 0, st, n_k, n_tot, k,
                       pos64, tab64, src32, tab32, naive);
    return hipGetLastError();
}

hipError_t launch_reduce(hipStream_t st, int mode, const void *partial, int n_chunks, int n_k, int n_o, int n_o_pad,
                         const double *k, int b_scale, int n_obs, int o0, void *E, void *B, void *E2, void *B2)
{
    const int64_t all = (int64_t)n_k * ((n_o + 63) / 64);
    const unsigned int nb = (unsigned int)(all < (1 << 20) ? all : (1 << 20));
    if (mode == MODE_FP64)
        hipLaunchKernelGGL((k_reduce<double, double>), dim3(nb), dim3(768), 0, st, (const double *)partial, n_chunks,
                           n_k, n_o, n_o_pad, k, b_scale, n_obs, o0, (double *)E, (double *)B, (double *)E2, (double *)B2);
    else
        hipLaunchKernelGGL((k_reduce<float, float>), dim3(nb), dim3(768), 0, st, (const float *)partial, n_chunks,
                           n_k, n_o, n_o_pad, k, b_scale, n_obs, o0, (float *)E, (float *)B, (float *)E2, (float *)B2);
    return hipGetLastError();
}

size_t twiddle_bytes(int n_k, int n_t) { return sizeof(double) * 2 * (size_t)n_k * time_rows(n_t); }

hipError_t launch_twiddles(hipStream_t st, int n_k, const double *k, int n_t, const double *t, double dk, double *tw)
{
    hipLaunchKernelGGL(k_twiddles, dim3(nblocks((int64_t)n_k * time_rows(n_t), 256)), dim3(256), 0, st, n_k, k, n_t, t,
                       dk, tw);
    return hipGetLastError();
}

hipError_t launch_time(hipStream_t st, int is_f64, int n_k, int n_t, int64_t n_x, const double *tw, const void *E,
                       const void *B, void *Et, void *Bt)
{
    dim3 g(nblocks(n_x, 256), time_rows(n_t) / TIME_MT, 2);
    if (is_f64)
        hipLaunchKernelGGL((k_time<double>), g, dim3(256), 0, st, n_k, n_t, n_x, tw, (const double *)E,
                           (const double *)B, (double *)Et, (double *)Bt);
    else
        hipLaunchKernelGGL((k_time<float>), g, dim3(256), 0, st, n_k, n_t, n_x, tw, (const float *)E, (const float *)B,
                           (float *)Et, (float *)Bt);
    return hipGetLastError();
}

hipError_t launch_fill_u32(hipStream_t st, unsigned int *p, unsigned int v, int n)
{
    hipLaunchKernelGGL(k_fill_u32, dim3(nblocks(n, 256)), dim3(256), 0, st, p, v, n);
    return hipGetLastError();
}

}  // namespace sc

// The kernels of the compacted sum belong to this translation unit, so that whoever compiles the library from the
// sources of build.py needs no longer a list for them.
#include "sc_compact.hip"
#include "sc_quad_mm.hip"

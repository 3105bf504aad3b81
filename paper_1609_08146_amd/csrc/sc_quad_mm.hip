// sc_quad_mm.hip -- the quadrature over compacted nodes in the FP32 split form, its contraction on the
// FP16 matrix instructions.
//
// With G = e^{ik delta} / R and H = (ik - 1/R) G / R of a node and a point, R_vec = r_s - r',
//   E  = sum G J~ + H rho~ r_s - r' sum H rho~
//   B' = sum H (J~ x r_s) - (sum H J~) x r'
// so the kernel values G and H (four reals per node, point and frequency) meet ten complex columns
// of table data that do not depend on the point: a matrix product.  The vector ALU forms G and H (one
// phase, one sine, one cosine, 7 more instructions) and v_mfma_f32_32x32x16_f16 sums them over the
// nodes, where the plain form spends 47 more FMAs per term on the vector ALU.
//
// Near the focus (|r'| <= |r_s| / 1000, and k |r_s| so large that 1/R in ik - 1/R may stand at |r_s|) one
// complex kernel value is enough: with V = e^{ik delta} / R^2, H = (ik - 1/|r_s|) V and
// G = R V = |r_s| V + delta V, so the columns meet V, and J~ |r_s| meets V delta / |r_s| besides.
//
// Precision.  Every kernel value and every table entry of E and B is the sum of two FP16 numbers,
// hi = fp16(x) and lo = fp16(x - hi): 22 bits, and all four products of the parts are summed in FP32
// (rows of A: hi and lo of the table; two products per step: hi and lo of the kernel values).  The
// columns that r' multiplies, and the term with delta / |r_s|, are hi alone where that factor is below
// 1/1000; FORM_GH_FAR gives those columns their lo part by a third product.  Table columns are scaled by
// powers of two to 2^12 at most, and the kernel values to about 2^6, so that no lo part falls below
// FP16's smallest number.  Near the focus the error against 64 bits is about half the plain FP32
// form's (0.1 m mirror, points within 4 wavelengths: 1.8e-7, plain 3.3e-7); elsewhere the same.
//
// One step is 4 nodes (near: 8): lane l holds point l % 32 and its half's nodes as B's 8 consecutive
// values (Gr, Gi, Hr, Hi of two nodes; near: Vr, Vi of four), and row l % 32 of A, 16 B loaded as they lie.
//
// Bound by the vector ALU's issue: instructions with the long encoding (cvt_pk, fma_mix) take 4.4 to 4.6
// SIMD cycles, sine and cosine 8.4, the short ones 2.4, and the matrix instructions (37 cycles each)
// overlap only in part: near the focus a kernel value and its products take 18 vector and 0.75 matrix
// instructions, 67 + 28 cycles per 64 terms, and the launch takes 93 (128 frequencies, 4160 points and 1799
// nodes, 9.7e8 terms with the padding, in 0.65 ms at 2.1 GHz; 126 with node records and rows loaded where
// they are used).  Two waves per SIMD with the compiler's free choice of registers beat three and four (at
// 2500 nodes 0.86, 1.04 and 1.20 ms).
#include "sc_device.h"
#include "sc_internal.h"

namespace sc {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v2f __attribute__((ext_vector_type(2)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef __attribute__((address_space(4))) const QuadJob cjob;
typedef __attribute__((address_space(4))) const double cdouble;
typedef __attribute__((address_space(4))) const float cfloat;

// Kernel values are formed as G s * 2^6 and H s^2 / k * 2^6 with s a power of two near the focal length.
// The near form's are V s^2 * 2^6 and V s^2 * 2^6 * delta / |r_s| * 2^10.
constexpr float KERNEL_SCALE = 64.0f, NEAR_SCALE = 1024.0f;

// v = hi + lo to 22 bits; m1 is -1 from memory, so that the difference is one mixed-precision FMA.
__device__ __forceinline__ void split2(float a, float b, float m1, h2 &hi, h2 &lo)
{
    const v2f v = {a, b};
    hi = __builtin_convertvector(v, h2);
    const v2f l = {__builtin_fmaf((float)hi.x, m1, a), __builtin_fmaf((float)hi.y, m1, b)};
    lo = __builtin_convertvector(l, h2);
}

// Sums of one lane into the partials.  Rows of a lane: lanes 0-31 E hi (6), E lo (6), sum H rho~ (2),
// (sum H J~).z (2); lanes 32-63 B hi, B lo, (sum H J~).x, .y.
template <int F>
__device__ __forceinline__ void store_mm(cjob *job, int chunk, int pt, int kb, const v4f o, const v16f *acc)
{
    const int half = (threadIdx.x >> 5) & 1, n_k = job->n_k;
    const float ox = o.x, oy = o.y, oz = o.z;
#pragma unroll
    for (int f = 0; f < F; ++f) {
        const int k = kb * F + f;
        float jzr = __shfl_xor(acc[f][14], 32), jzi = __shfl_xor(acc[f][15], 32);
        if (k >= n_k) continue;
        cfloat *sc = (cfloat *)job->mscale + 16 * (size_t)k;
        float v[6];
#pragma unroll
        for (int c = 0; c < 6; ++c) v[c] = (acc[f][c] + acc[f][6 + c]) * (half ? sc[4 + c / 2] : sc[c / 2]);
        if (half == 0) {
            const float sr = acc[f][12] * sc[3], si = acc[f][13] * sc[3];
            v[0] = __fmaf_rn(-sr, ox, v[0]);
            v[1] = __fmaf_rn(-si, ox, v[1]);
            v[2] = __fmaf_rn(-sr, oy, v[2]);
            v[3] = __fmaf_rn(-si, oy, v[3]);
            v[4] = __fmaf_rn(-sr, oz, v[4]);
            v[5] = __fmaf_rn(-si, oz, v[5]);
        } else {
            const float jxr = acc[f][12] * sc[7], jxi = acc[f][13] * sc[7];
            const float jyr = acc[f][14] * sc[8], jyi = acc[f][15] * sc[8];
            jzr *= sc[9];
            jzi *= sc[9];
            v[0] -= __fmaf_rn(jyr, oz, -(jzr * oy));
            v[1] -= __fmaf_rn(jyi, oz, -(jzi * oy));
            v[2] -= __fmaf_rn(jzr, ox, -(jxr * oz));
            v[3] -= __fmaf_rn(jzi, ox, -(jxi * oz));
            v[4] -= __fmaf_rn(jxr, oy, -(jyr * ox));
            v[5] -= __fmaf_rn(jxi, oy, -(jyi * ox));
        }
        // partials [chunk][k][point / 64][12][64]
        float *part = (float *)job->partial + ((size_t)chunk * n_k + k) * 12 * (size_t)job->n_obs_pad +
                      (size_t)(pt >> 6) * 768 + half * 384 + (pt & 63);
#pragma unroll
        for (int c = 0; c < 6; ++c) part[c * 64] = v[c];
    }
}

// delta = |R| - |r_s| and s / R, by series near the focus as in the plain form: p = (r_s / |r_s|, h),
// h = 1 / 2|r_s|, for the series, else (x, y, z, |r_s|).  (With the direction rounded once from FP64 the
// phase takes two roundings less than from r_s and h, of which h's is common to a row of nodes: error
// against 64 bits 1.8e-7 for 3.4e-7.)
template <bool SER>
__device__ __forceinline__ void geom_mm(const v4f p, const v4f o, float s, float &delta, float &ph)
{
    const float dot = __fmaf_rn(p.x, o.x, __fmaf_rn(p.y, o.y, p.z * o.z));
    if constexpr (SER) {
        const float h = p.w;
        const float d1 = __fmaf_rn(o.w, h, -dot), x = d1 * h;
        delta = __fmaf_rn(d1 * x, __fmaf_rn(2.0f, x, -1.0f), d1);
        const float h2 = h + h, y = delta * h2;
        ph = (h2 * s) * __fmaf_rn(y, y - 1.0f, 1.0f);
    } else {
        const float num = __fmaf_rn(-2.0f, dot, o.w);
        const float dx = p.x - o.x, dy = p.y - o.y, dz = p.z - o.z;
        const float R2 = __fmaf_rn(dx, dx, __fmaf_rn(dy, dy, dz * dz));
        const float rinv = __builtin_amdgcn_rsqf(R2);
        delta = num * __builtin_amdgcn_rcpf(__fmaf_rn(R2, rinv, p.w));
        ph = rinv * s;
    }
}

// Operands of one step and frequency: rows a (and b), kernel values hi, lo (and y, near).
struct Products {
    h8 a = {}, b = {}, hi = {}, lo = {}, y = {};
};
template <int FORM>
__device__ __forceinline__ void mm_products(const Products &w, v16f &acc)
{
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(w.a, w.hi, acc, 0, 0, 0);
    if constexpr (FORM == FORM_GH_FAR) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(w.b, w.hi, acc, 0, 0, 0);
    acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(w.a, w.lo, acc, 0, 0, 0);
    if constexpr (FORM == FORM_NEAR) acc = __builtin_amdgcn_mfma_f32_32x32x16_f16(w.b, w.y, acc, 0, 0, 0);
}

template <int F, bool RAW, bool SER, int FORM>
__device__ __forceinline__ void tile_mm(cjob *job, int chunk, int pg, int kb, float m1)
{
    constexpr int NODES = form_nodes(FORM), ROWS = form_rows(FORM), Q = NODES / 2;   // nodes per lane and step
    const int lane = threadIdx.x & 63, half = lane >> 5;
    const int n_k = job->n_k, steps = (job->n_tot + NODES - 1) / NODES;
    const int s0 = chunk * (job->chunk / NODES), s1 = min(s0 + job->chunk / NODES, steps);
    const int pt = pg * 128 + (threadIdx.x >> 6) * 32 + (lane & 31);
    const float s = job->scale;
    float kt[F], iks[F];
    const h8 *A[F];
    const size_t row = (size_t)steps * 64;
#pragma unroll
    for (int f = 0; f < F; ++f) {
        const int k = min(kb * F + f, n_k - 1);
        const double kv = ((cdouble *)job->k)[k];
        kt[f] = (float)(kv * INV_TWO_PI);
        iks[f] = (float)(1.0 / (kv * (double)s));
        A[f] = (const h8 *)job->mtab + (size_t)k * ROWS * row + lane;
    }
    const v4f o = ((const v4f *)job->obs)[pt];
    // the chunk's node records in LDS: every lane of a half reads the same one, which through L1 would
    // take as many cycles as 64 different ones
    __shared__ v4f node[MM_CHUNK_MAX];
    __syncthreads();
    for (int i = threadIdx.x; i < (s1 - s0) * NODES; i += 256) {
        node[i] = ((const v4f *)(SER ? job->hinv : job->pos))[s0 * NODES + i];
    }
    __syncthreads();
    v16f acc[F];
#pragma unroll
    for (int f = 0; f < F; ++f)
#pragma unroll
        for (int v = 0; v < 16; ++v) acc[f][v] = 0.0f;

    h8 a0[F], a1[F];   // this step's rows, loaded a step ahead
#pragma unroll
    for (int f = 0; f < F; ++f) {
        a0[f] = A[f][(size_t)s0 * 64];
        if constexpr (ROWS == 2) a1[f] = A[f][row + (size_t)s0 * 64];
    }
    Products w;   // none pending: zeros add nothing
    for (int st = s0; st < s1; ++st) {
        const size_t next = (size_t)min(st + 1, s1 - 1) * 64;
        const v4f *p = node + NODES * (st - s0) + Q * half;
        float ph[Q], delta[Q], yy[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            geom_mm<SER>(p[q], o, s, delta[q], ph[q]);
            if constexpr (FORM == FORM_NEAR) {
                // delta / |r_s|
                yy[q] = delta[q] * (SER ? p[q].w * (2.0f * NEAR_SCALE) : __builtin_amdgcn_rcpf(p[q].w) * NEAR_SCALE);
                ph[q] = (ph[q] * ph[q]) * KERNEL_SCALE;
            }
        }
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const h8 a = a0[f], b = ROWS == 2 ? a1[f] : a0[f];
            a0[f] = A[f][next];
            if constexpr (ROWS == 2) a1[f] = A[f][row + next];
            h2 hi[4], lo[4], yv[4];
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const float turn = kt[f] * delta[q];
                const float r = RAW ? turn : __builtin_amdgcn_fractf(turn);
                if constexpr (FORM == FORM_NEAR) {
                    const float vr = __builtin_amdgcn_cosf(r) * ph[q], vi = __builtin_amdgcn_sinf(r) * ph[q];
                    split2(vr, vi, m1, hi[q], lo[q]);
                    const v2f y = {vr * yy[q], vi * yy[q]};
                    yv[q] = __builtin_convertvector(y, h2);
                } else {
                    const float pa = ph[q] * KERNEL_SCALE, nph = -ph[q];
                    const float gr = __builtin_amdgcn_cosf(r) * pa, gi = __builtin_amdgcn_sinf(r) * pa;
                    const float nb = (nph * ph[q]) * iks[f];
                    // H s^2 / k = (i s / R - (s / R)^2 / (k s)) G s
                    const float hr = __fmaf_rn(gi, nph, gr * nb), him = __fmaf_rn(gr, ph[q], gi * nb);
                    split2(gr, gi, m1, hi[2 * q], lo[2 * q]);
                    split2(hr, him, m1, hi[2 * q + 1], lo[2 * q + 1]);
                }
            }
            // the products of the frequency before, so that they run beside this one's kernel values
            mm_products<FORM>(w, acc[(f + F - 1) % F]);
            w.a = a;
            w.b = b;
            w.hi = h8{hi[0].x, hi[0].y, hi[1].x, hi[1].y, hi[2].x, hi[2].y, hi[3].x, hi[3].y};
            w.lo = h8{lo[0].x, lo[0].y, lo[1].x, lo[1].y, lo[2].x, lo[2].y, lo[3].x, lo[3].y};
            if constexpr (FORM == FORM_NEAR)
                w.y = h8{yv[0].x, yv[0].y, yv[1].x, yv[1].y, yv[2].x, yv[2].y, yv[3].x, yv[3].y};
        }
    }
    mm_products<FORM>(w, acc[F - 1]);
    store_mm<F>(job, chunk, pt, kb, o, acc);
}

// One workgroup per tile: 128 points (32 per wave) x F frequencies x one chunk of nodes, the four waves
// reading the same table rows through L1.  Tiles run points fastest; workgroups go to the 8 XCDs in turn,
// and each XCD takes a contiguous eighth of every job's tiles, so that its L2 serves the rows that they
// share.  (An eighth of the tiles of all jobs together, whose tiles are of 64 to 256 nodes, left XCDs idle:
// eight problems 3.06 ms, now 2.41.)  job_tile: the XCD's i-th tile of the launch, which is one of this job's.
template <int F>
__device__ __forceinline__ void job_tile(cjob *job, int64_t i, float m1)
{
    const int64_t eighth = (job->n_tiles + QUAD_SEGMENTS - 1) / QUAD_SEGMENTS;
    const int64_t t = eighth * (blockIdx.x % QUAD_SEGMENTS) + i - job->tile0;
    if (t >= job->n_tiles) return;
    const int64_t local = t + job->tile_offset;
    const int pgs = job->n_obs_pad / 128;
    const int pg = (int)(local % pgs);
    const int64_t rest = local / pgs;
    const int chunk = (int)(rest % job->n_chunks), kb = (int)(rest / job->n_chunks);
    // (the series of delta hold to |r'| <= 4e-4 |r_s|, so they come with the near form alone)
    const bool raw = job->raw_phase != 0, ser = job->series_delta != 0;
    if (job->form == FORM_NEAR) {
        if (ser && raw) tile_mm<F, true, true, FORM_NEAR>(job, chunk, pg, kb, m1);
        else if (ser) tile_mm<F, false, true, FORM_NEAR>(job, chunk, pg, kb, m1);
        else tile_mm<F, false, false, FORM_NEAR>(job, chunk, pg, kb, m1);
    } else if (job->form == FORM_GH) {
        if (raw) tile_mm<F, true, false, FORM_GH>(job, chunk, pg, kb, m1);
        else tile_mm<F, false, false, FORM_GH>(job, chunk, pg, kb, m1);
    } else {
        if (raw) tile_mm<F, true, false, FORM_GH_FAR>(job, chunk, pg, kb, m1);
        else tile_mm<F, false, false, FORM_GH_FAR>(job, chunk, pg, kb, m1);
    }
}

// The tiles of this workgroup: its XCD's `per` from its own place on.
#define SC_MM_TILES(t) \
    for (int64_t t = blockIdx.x / QUAD_SEGMENTS; t < per; t += gridDim.x / QUAD_SEGMENTS)

// One job, which travels as the kernel's first argument and is read where it lies.
template <int F>
__global__ void __launch_bounds__(256) k_quad_mm_one(QuadJob, int64_t per, float m1)
{
    cjob *job = (cjob *)__builtin_amdgcn_kernarg_segment_ptr();
    SC_MM_TILES(t) job_tile<F>(job, t, m1);
}

// Tiles of several jobs.
template <int F>
__global__ void __launch_bounds__(256)
k_quad_mm(const QuadJob *__restrict__ jobs_, int n_jobs, int64_t per, float m1)
{
    cjob *jobs = (cjob *)jobs_;
    SC_MM_TILES(t) {
        int lo = 0, hi = n_jobs - 1;
        while (lo < hi) {
            const int mid = (lo + hi + 1) >> 1;
            if (jobs[mid].tile0 <= t) lo = mid;
            else hi = mid - 1;
        }
        job_tile<F>(jobs + lo, t, m1);
    }
}

// ------------------------------------------------------------------------------- packed tables

// The ten complex columns of a node at wavenumber k, in the order of the scales: E.x, E.y, E.z, the sum
// of rho~, (J~ x r_s).x, .y, .z, J~.x, .y, .z.  G and H forms: h the factors of H s^2 / k, and g those of
// G s in E (J~ / s).  Near form: h the factors of V s^2 = e^{ik delta} (s / R)^2, g those of V s^2 delta / |r_s|.
__device__ __forceinline__ void mm_columns(int form, const float *__restrict__ rec, const v4f p, double k, double s,
                                           double *g, double *h)
{
    const double r[3] = {p.x, p.y, p.z}, is2 = 1.0 / (s * s);
    double J[6], rho[2];
    if (form == FORM_NEAR) {
        // times (ik - 1/|r_s|) / s^2
        const double cr = -is2 / (double)p.w, ci = k * is2;
        for (int c = 0; c < 3; ++c) {
            J[2 * c] = cr * (double)rec[2 * c] - ci * (double)rec[2 * c + 1];
            J[2 * c + 1] = cr * (double)rec[2 * c + 1] + ci * (double)rec[2 * c];
        }
        rho[0] = cr * (double)rec[6] - ci * (double)rec[7];
        rho[1] = cr * (double)rec[7] + ci * (double)rec[6];
    } else {
        for (int c = 0; c < 6; ++c) J[c] = k * is2 * (double)rec[c];
        rho[0] = k * is2 * (double)rec[6];
        rho[1] = k * is2 * (double)rec[7];
    }
    const double gs = form == FORM_NEAR ? is2 * (double)p.w : 1.0 / s;
    for (int c = 0; c < 6; ++c) g[c] = gs * (double)rec[c];
    for (int z = 0; z < 2; ++z) {   // re, im
        for (int c = 0; c < 3; ++c) h[2 * c + z] = rho[z] * r[c] + (form == FORM_NEAR ? g[2 * c + z] : 0.0);
        h[6 + z] = rho[z];
        h[8 + z] = J[2 + z] * r[2] - J[4 + z] * r[1];
        h[10 + z] = J[4 + z] * r[0] - J[z] * r[2];
        h[12 + z] = J[z] * r[1] - J[2 + z] * r[0];
        for (int c = 0; c < 3; ++c) h[14 + 2 * c + z] = J[2 * c + z];
    }
}

// The largest entry of each column over a part of the nodes, SCALE_PARTS workgroups per frequency (one for
// all nodes took 11 us, now 6): mmax[k][part][10].
constexpr int SCALE_PARTS = 8;
__global__ void __launch_bounds__(256)
k_mm_max(int n_c, int form, const double *__restrict__ kv, double s, const float *__restrict__ ctab,
         const v4f *__restrict__ pos, double *__restrict__ mmax)
{
    const int kk = blockIdx.x;
    double mx[10] = {};
    for (int q = blockIdx.y * 256 + threadIdx.x; q < n_c; q += 256 * SCALE_PARTS) {
        double g[6], h[20];
        mm_columns(form, ctab + ((size_t)kk * n_c + q) * 8, pos[q], kv[kk], s, g, h);
        for (int c = 0; c < 10; ++c) {
            double m = fmax(fabs(h[2 * c]), fabs(h[2 * c + 1]));
            if (c < 3) m = fmax(m, fmax(fabs(g[2 * c]), fabs(g[2 * c + 1])));
            mx[c] = fmax(mx[c], m);
        }
    }
    __shared__ double red[4][10];
    for (int c = 0; c < 10; ++c) {
        double m = mx[c];
        for (int o = 32; o > 0; o >>= 1) m = fmax(m, __shfl_xor(m, o));
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6][c] = m;
    }
    __syncthreads();
    if (threadIdx.x < 10) {
        double m = 0.0;
        for (int w = 0; w < 4; ++w) m = fmax(m, red[w][threadIdx.x]);
        mmax[((size_t)kk * SCALE_PARTS + blockIdx.y) * 10 + threadIdx.x] = m;
    }
}

// mtab[k][row][step][lane][8] halves, row 0: lane's row l % 32 of the step's nodes of its half (l / 32), for each
// node the factors of the kernel values (Gr, Gi, Hr, Hi; near Vr, Vi).  Row 1, in FORM_GH_FAR: the lo
// parts of the columns that r' multiplies; in FORM_NEAR: the factors of V delta / |r_s|, those of E's G J~
// and, in E and B, i (k - k32) |r_s| times row 0's, the first order of the phase (k - k32) delta that
// the quadrature's FP32 wavenumber k32 leaves out.
// One workgroup per PACK_STEPS steps, their nodes' columns formed once each and kept in LDS
// (formed by every lane for its own row: 67 us at 128 frequencies and 4 000 nodes, now 19).
constexpr int PACK_STEPS = 16;
template <int FORM>
__global__ void __launch_bounds__(256)
k_mm_pack(int n_c, const double *__restrict__ kv, double s, const float *__restrict__ ctab,
          const v4f *__restrict__ pos, const double *__restrict__ mmax, float *__restrict__ mscale,
          h8 *__restrict__ mtab)
{
    constexpr int NODES = form_nodes(FORM), ROWS = form_rows(FORM), Q = NODES / 2, W = 8 / Q;   // values per node
    constexpr int ALL = PACK_STEPS * NODES;
    static_assert(ALL <= 256, "one thread per node");
    const int steps = (n_c + NODES - 1) / NODES, st0 = blockIdx.x * PACK_STEPS, kk = blockIdx.y;
    // per node and column: factors of H or V, then of G or V delta / |r_s|, scaled
    __shared__ float colh[20][ALL + 1], colg[12][ALL + 1];
    // powers of two that bring each column's largest entry to 2^11 ... 2^12; mscale[k][16] holds what the sums
    // are multiplied by (scale / KERNEL_SCALE, and for B over the power of two at or below k: the sums of B' = ik B
    // would leave FP32's range 2^23 earlier than B in metres), over the whole range of FP32
    __shared__ double inv[10];
    if (threadIdx.x < 16) {
        double m = 0.0;
        if (threadIdx.x < 10)
            for (int w = 0; w < SCALE_PARTS; ++w) m = fmax(m, mmax[((size_t)kk * SCALE_PARTS + w) * 10 + threadIdx.x]);
        // m = f 2^e with f in [0.5, 1): times 2^(12 - e)
        const int kb = threadIdx.x >= 4 ? ilogb(kv[kk]) : 0;
        const int e = m > 0.0 && m < 1e300 ? max(kb - 131, min(kb + 145, ilogb(m) + 1)) : 12;
        if (threadIdx.x < 10) inv[threadIdx.x] = ldexp(1.0, 12 - e);
        if (blockIdx.x == 0) mscale[16 * (size_t)kk + threadIdx.x] = (float)(ldexp(1.0, e - 12 - kb) / KERNEL_SCALE);
    }
    __syncthreads();
    if (threadIdx.x < ALL) {
        const int n = st0 * NODES + threadIdx.x;
        double g[12] = {}, h[20] = {};   // past the last node: zero
        if (n < n_c) {
            const v4f p = pos[n];
            const double k = kv[kk];
            mm_columns(FORM, ctab + ((size_t)kk * n_c + n) * 8, p, k, s, g, h);
            if (FORM == FORM_NEAR) {
                const double turns = k * INV_TWO_PI, x = (turns - (double)(float)turns) * TWO_PI_1 * (double)p.w;
                const double y = fabs(x) <= (double)NEAR_SCALE ? x : 0.0;   // (keeps to FP16's range)
                for (int c = 0; c < 6; ++c) {
                    const int hc = c < 3 ? c : c + 1;   // E, then B past the sum of rho~
                    g[2 * c] -= y * h[2 * hc + 1];
                    g[2 * c + 1] += y * h[2 * hc];
                }
            }
        }
        for (int c = 0; c < 10; ++c) {
            const int gc = c < 3 ? c : c - 1;
            for (int z = 0; z < 2; ++z) {
                colh[2 * c + z][threadIdx.x] = (float)(h[2 * c + z] * inv[c]);
                if (c != 3 && gc < 6) colg[2 * gc + z][threadIdx.x] = (float)(g[2 * gc + z] * inv[c]);
            }
        }
    }
    __syncthreads();
    const int lane = threadIdx.x & 63, r = lane & 31, rh = (r >> 2) & 1, v = (r & 3) + 4 * (r >> 3);
    // row r holds value v of half rh (see store_mm): its column, part (re, im) and whether it is the lo half
    int col, lo = 0;
    const int part = v & 1;
    if (v < 12) {
        lo = v >= 6;
        col = (rh ? 4 : 0) + (v % 6) / 2;
    } else if (rh == 0) {
        col = v < 14 ? 3 : 9;
    } else {
        col = v < 14 ? 7 : 8;
    }
    const int gcol = v < 12 ? 3 * rh + (v % 6) / 2 : -1;   // of E and B
    for (int j = threadIdx.x >> 6; j < PACK_STEPS && st0 + j < steps; j += 4) {
        h8 out = {}, out2 = {};
#pragma unroll
        for (int q = 0; q < Q; ++q) {
            const int i = NODES * j + Q * (lane >> 5) + q;
            const float hr = colh[2 * col][i], hi = colh[2 * col + 1][i];
            const float gr = gcol < 0 ? 0.0f : colg[2 * max(gcol, 0)][i];
            const float gi = gcol < 0 ? 0.0f : colg[2 * max(gcol, 0) + 1][i];
            // (a + ib)(Vr + iVi): re = a Vr - b Vi, im = b Vr + a Vi
            const float wg[2] = {part ? gi : gr, part ? gr : -gi};
            const float wh[2] = {part ? hi : hr, part ? hr : -hi};
#pragma unroll
            for (int e = 0; e < W; ++e) {
                const float w = W == 2 ? wh[e] : e < 2 ? wg[e] : wh[e - 2];
                const _Float16 a = (_Float16)w, b = (_Float16)(w - (float)a);
                out[W * q + e] = lo ? b : a;
                if (FORM == FORM_GH_FAR && v >= 12) out2[W * q + e] = b;
                if (FORM == FORM_NEAR && v < 6) out2[W * q + e] = (_Float16)(wg[e] / NEAR_SCALE);
            }
        }
        h8 *dst = mtab + ((size_t)kk * ROWS * steps + st0 + j) * 64 + lane;
        dst[0] = out;
        if (ROWS == 2) dst[(size_t)steps * 64] = out2;
    }
}

// ================================================================== launchers

size_t mm_scale_bytes(int n_k) { return (size_t)n_k * (sizeof(float) * 16 + sizeof(double) * 10 * SCALE_PARTS); }

hipError_t launch_mm_tables(hipStream_t st, int n_k, int n_c, int form, const double *k, double scale, const float *ctab,
                            const float *pos, float *mscale, void *mtab)
{
    const int steps = (n_c + form_nodes(form) - 1) / form_nodes(form);
    const dim3 g((steps + PACK_STEPS - 1) / PACK_STEPS, n_k), b(256);
    double *mmax = (double *)((char *)mscale + mm_scale_bytes(n_k)) - (size_t)n_k * SCALE_PARTS * 10;
    hipLaunchKernelGGL(k_mm_max, dim3(n_k, SCALE_PARTS), b, 0, st, n_c, form, k, scale, ctab, (const v4f *)pos, mmax);
#define SC_MM_PACK(FORM)                                                                              \
    hipLaunchKernelGGL((k_mm_pack<FORM>), g, b, 0, st, n_c, k, scale, ctab, (const v4f *)pos, mmax, mscale, \
                       (h8 *)mtab)
    if (form == FORM_NEAR) SC_MM_PACK(FORM_NEAR);
    else if (form == FORM_GH) SC_MM_PACK(FORM_GH);
    else SC_MM_PACK(FORM_GH_FAR);
#undef SC_MM_PACK
    return hipGetLastError();
}

static unsigned int mm_grid(int64_t per)
{
    const int64_t grid = per * QUAD_SEGMENTS;
    return (unsigned int)(grid < (1 << 20) ? grid : (1 << 20));
}

hipError_t launch_quad_mm_one(hipStream_t st, int fpb, const QuadJob &job)
{
    const int64_t per = mm_tiles_per_xcd(job);
    const dim3 g(mm_grid(per)), b(256);
    if (fpb == 4) hipLaunchKernelGGL((k_quad_mm_one<4>), g, b, 0, st, job, per, -1.0f);
    else if (fpb == 2) hipLaunchKernelGGL((k_quad_mm_one<2>), g, b, 0, st, job, per, -1.0f);
    else hipLaunchKernelGGL((k_quad_mm_one<1>), g, b, 0, st, job, per, -1.0f);
    return hipGetLastError();
}

hipError_t launch_quad_mm(hipStream_t st, int fpb, const QuadJob *jobs, int n_jobs, int64_t per)
{
    const dim3 g(mm_grid(per)), b(256);
    if (fpb == 4) hipLaunchKernelGGL((k_quad_mm<4>), g, b, 0, st, jobs, n_jobs, per, -1.0f);
    else if (fpb == 2) hipLaunchKernelGGL((k_quad_mm<2>), g, b, 0, st, jobs, n_jobs, per, -1.0f);
    else hipLaunchKernelGGL((k_quad_mm<1>), g, b, 0, st, jobs, n_jobs, per, -1.0f);
    return hipGetLastError();
}

}  // namespace sc

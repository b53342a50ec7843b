// Physically-based shading with image-based lighting, for gfx950: the
// irradiance and prefiltered environment maps built from the environment
// image, the BRDF integration table, and split-sum shading (the render
// graph of appendix B; appendix C optimises an environment map with it).
//
// The filters are dense sums over every environment texel, contracted on the
// matrix cores in double in a fixed order.  Their adjoint is the transposed
// sum, so the environment gradient is exact and needs no atomics.  Shading follows the
// split sum per fragment; its backward is analytic, with the material's
// scalar gradients reduced in a fixed order.
#include "texcore.h"

#include <algorithm>

#define PBS_BS 256

// ---------------------------------------------------------------------------
// cube texels: direction (the sampler's major-axis convention) and solid angle
// ---------------------------------------------------------------------------
__device__ __forceinline__ double3 cube_texel_dir(int S, int64_t idx) {
    const int f = (int)(idx / ((int64_t)S * S));
    const int rem = (int)(idx - (int64_t)f * S * S);
    const int j = rem / S, i = rem - j * S;
    const double a = 2.0 * (i + 0.5) / S - 1.0, b = 2.0 * (j + 0.5) / S - 1.0;
    double x, y, z;
    switch (f) {
    case 0: x = 1.0; y = -b; z = -a; break;
    case 1: x = -1.0; y = -b; z = a; break;
    case 2: x = a; y = 1.0; z = b; break;
    case 3: x = a; y = -1.0; z = -b; break;
    case 4: x = a; y = -b; z = 1.0; break;
    default: x = -a; y = -b; z = -1.0; break;
    }
    const double inv = 1.0 / sqrt(x * x + y * y + z * z);
    return make_double3(x * inv, y * inv, z * inv);
}

__device__ __forceinline__ double cube_texel_omega(int S, int64_t idx) {
    const int rem = (int)(idx % ((int64_t)S * S));
    const int j = rem / S, i = rem - j * S;
    const double a0 = 2.0 * i / S - 1.0, a1 = 2.0 * (i + 1) / S - 1.0;
    const double b0 = 2.0 * j / S - 1.0, b1 = 2.0 * (j + 1) / S - 1.0;
    auto F = [](double a, double b) { return atan2(a * b, sqrt(a * a + b * b + 1.0)); };
    return F(a1, b1) - F(a0, b1) - F(a1, b0) + F(a0, b0);
}

__device__ __forceinline__ double level_alpha(int l, int L) {
    const double r = (double)l / (double)(L - 1);
    return fmax(r * r, 1e-3);
}

// The filters' kernel between output q (direction) and environment texel e
// (direction w, solid angle O): max(0, q.w) O for the irradiance; for a
// prefiltered level max(0, R.w) D(h) O with (R.h)^2 = (1 + R.w) / 2 for unit
// vectors, D(h) = alpha^2 / (pi T^2), T = (R.h)^2 (alpha^2 - 1) + 1 =
// (1 - c) / 2 + (1 + c) alpha^2 / 2 (without cancellation: T is of order
// alpha^2 near the lobe's axis).  With A = (1 + alpha^2) / 2, T = A (1 + c) - c;
// A = 1 gives T = 1, the irradiance's kernel.  O and the output's factor
// (alpha^2 / pi, or 1) leave the sums: the pair's part is max(0, c) / T^2.
__device__ __forceinline__ double2 output_factor(const dressi_ibl_desc &g, int64_t o, double3 &d) {
    const int64_t ni = 6ll * g.Si * g.Si, np = 6ll * g.Sp * g.Sp;
    if (o < ni) {
        d = cube_texel_dir(g.Si, o);
        return make_double2(1.0, 1.0);
    }
    const int l = (int)((o - ni) / np);
    d = cube_texel_dir(g.Sp, (o - ni) - (int64_t)l * np);
    const double al = level_alpha(l, g.L), a2 = al * al;
    return make_double2(0.5 + 0.5 * a2, a2 / 3.14159265358979323846);
}

// Outputs o < 6 Si^2 are the irradiance's texels, the rest the prefiltered
// levels, level by level.  The tables of both sides: environment texels
// (direction, solid angle) and outputs (direction, A), and the rows of the
// contraction's right factor: for the filter O (env, 1) per texel, for the
// adjoint factor / norm (grad, 0) per output.
__global__ void k_ibl_tables(dressi_ibl_desc g, int64_t ne, int64_t no, const float *__restrict__ env,
                             const double *__restrict__ norm,
                             const float *__restrict__ g_irr, const float *__restrict__ g_pref,
                             double4 *__restrict__ tab, double4 *__restrict__ otab, double4 *__restrict__ rhs) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < ne) {
        const double3 d = cube_texel_dir(g.S, i);
        const double om = cube_texel_omega(g.S, i);
        tab[i] = make_double4(d.x, d.y, d.z, om);
        if (env) rhs[i] = make_double4(om * env[3 * i], om * env[3 * i + 1], om * env[3 * i + 2], om);
    }
    if (i < no) {
        double3 d;
        const double2 f = output_factor(g, i, d);
        otab[i] = make_double4(d.x, d.y, d.z, f.x);
        if (!env) {
            const int64_t ni = 6ll * g.Si * g.Si;
            const float *go = i < ni ? g_irr + 3 * i : g_pref + 3 * (i - ni);
            const double s = f.y / norm[i];
            rhs[i] = make_double4(go[0] * s, go[1] * s, go[2] * s, 0.0);
        }
    }
}

// D[row][n] = sum over columns of max(0, c) / T^2 rhs[column][n]: the filters
// (rows: outputs, columns: environment texels) and their adjoint (rows and
// columns exchanged), exact sums with no atomics, in a fixed order.
//
// It is bound by the pair's arithmetic: c and T in double (their cancellation
// is the lobe's shape), the quotient in float, the sums in double.  The
// contraction runs on the matrix cores: v_mfma_f64_4x4x4_4b takes one pair of
// each lane (lane = 16 (column mod 4) + row mod 16), so a lane feeds the
// kernel value that it computed and the four sums of a row cost one
// instruction, where the vector unit would convert, multiply and add each
// channel.  (The dot products on v_mfma_f64_16x16x4 measured no faster: 416 us
// against 380.)  A lane holds R rows' directions in
// registers; the eight wavefronts of a workgroup take every eighth group of
// 64 columns, each through its own LDS (the next group's loads in flight), and
// add their sums in wavefront order.  One workgroup per output summing 256 lanes in a tree,
// with every pair's tables loaded anew, took 1.45 ms (filter) and 1.50 ms
// (adjoint) at 6 x 64^2 -> 16^2 + 5 x 6 x 32^2 (0.79 G pairs); see the launches
// for this form's times.
//
// A column with a value that is not finite must not reach rows that it does
// not light (0 x inf): such a step multiplies on the vector unit and skips
// zero kernel values.
#define IBL_WAVES 8
#define IBL_COLS (64 * IBL_WAVES)   // columns of a workgroup's step
template <int R, bool ADJOINT>
__global__ void __launch_bounds__(64 * IBL_WAVES)
    k_ibl_contract(const double4 *__restrict__ rows, int64_t n_rows, const double4 *__restrict__ cols,
                   const double4 *__restrict__ rhs, int64_t n_cols, int64_t n_irr, dressi_ibl_desc g,
                   float *__restrict__ out, float *__restrict__ pref, double *__restrict__ norm) {
    __shared__ double4 scol[IBL_WAVES][64], srhs[IBL_WAVES][64];
    __shared__ double part[IBL_WAVES][R][64];
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    const int kk = lane >> 4, low = lane & 15;
    const int64_t row0 = (int64_t)blockIdx.x * (16 * R);
    double qx[R], qy[R], qz[R], qa[R], acc[R];
#pragma unroll
    for (int r = 0; r < R; r++) {
        const double4 q = rows[min(row0 + 16 * r + low, n_rows - 1)];
        qx[r] = q.x;
        qy[r] = q.y;
        qz[r] = q.z;
        qa[r] = q.w;
        acc[r] = 0.0;
    }
    // the pairs' kernel values of one column (this lane's) and the R rows
    const auto kernel = [&](const double4 &e, float *k) {
#pragma unroll
        for (int r = 0; r < R; r++) {
            const double c = fma(qz[r], e.z, fma(qy[r], e.y, qx[r] * e.x));
            const double A = ADJOINT ? e.w : qa[r];
            const float t = (float)(fma(A, c, A) - c);
            k[r] = fminf(fmaxf((float)c, 0.0f), 1.0f) * __builtin_amdgcn_rcpf(t * t);
        }
    };
    // 64 columns at a time, one a lane, through the wavefront's own LDS
    // (past the end: a direction that lights nothing)
    int64_t base = 64 * w;
    double4 e, v;
    const auto load = [&](int64_t i) {
        const int64_t at = min(i, n_cols - 1);
        const double in = i < n_cols ? 1.0 : 0.0;
        e = cols[at];
        v = rhs[at];
        e.x *= in;
        e.y *= in;
        e.z *= in;
        if (i >= n_cols) v.x = v.y = v.z = v.w = 0.0;
    };
    load(base + lane);
    for (; base < n_cols; base += IBL_COLS) {
        scol[w][lane] = e;
        srhs[w][lane] = v;
        const bool finite = !__ballot(!(isfinite(v.x) && isfinite(v.y) && isfinite(v.z) && isfinite(v.w)));
        load(base + IBL_COLS + lane);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        const int n = (int)min((int64_t)64, n_cols - base);
        const double *sr = reinterpret_cast<const double *>(srhs[w]);
        if (finite) {
            for (int c = kk; c - kk < n; c += 8) {   // two steps side by side
                float k0[R], k1[R];
                const double v0 = sr[4 * c + (lane & 3)], v1 = sr[4 * c + 16 + (lane & 3)];
                kernel(scol[w][c], k0);
                kernel(scol[w][c + 4], k1);
#pragma unroll
                for (int r = 0; r < R; r++) {
                    acc[r] = __builtin_amdgcn_mfma_f64_4x4x4f64((double)k0[r], v0, acc[r], 0, 0, 0);
                    acc[r] = __builtin_amdgcn_mfma_f64_4x4x4f64((double)k1[r], v1, acc[r], 0, 0, 0);
                }
            }
        } else {
            for (int c = kk; c - kk < n; c += 4) {
                float k[R];
                kernel(scol[w][c], k);
                // this lane's sums: row (lane >> 4) of its block, channel lane & 3
                for (int q = 0; q < 4; q++) {
                    const double vq = sr[4 * (c - kk + q) + (lane & 3)];
#pragma unroll
                    for (int r = 0; r < R; r++) {
                        const float kq = __shfl(k[r], 16 * q + (lane & 12) + (lane >> 4), 64);
                        if (kq != 0.0f) acc[r] += (double)kq * vq;
                    }
                }
            }
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    }
#pragma unroll
    for (int r = 0; r < R; r++) part[w][r][lane] = acc[r];
    __syncthreads();
    // the sums of row 16 r + 4 (block) + (lane >> 4), channel lane & 3
    for (int r = w; r < R; r += IBL_WAVES) {
        double d = 0.0;
#pragma unroll
        for (int k = 0; k < IBL_WAVES; k++) d += part[k][r][lane];
        const double sum = __shfl(d, lane | 3, 64);   // the row's fourth channel
        const int64_t row = row0 + 16 * r + (lane & 12) + (lane >> 4);
        const int n = lane & 3;
        if (row >= n_rows) continue;
        if (ADJOINT) {
            if (n < 3) out[3 * row + n] = (float)(d * rows[row].w);
        } else if (n < 3) {
            (row < n_irr ? out + 3 * row : pref + 3 * (row - n_irr))[n] = (float)(d * (1.0 / sum));
        } else {
            double3 dir;
            norm[row] = output_factor(g, row, dir).y * d;
        }
    }
}

static int check_ibl(dressi_ctx *ctx, const dressi_ibl_desc *d) {
    if (!ctx) return DRESSI_EINVAL;
    if (!d || d->S < 1 || d->Si < 1 || d->Sp < 1 || d->L < 2 || d->S > 1024 || d->Si > 1024 || d->Sp > 1024 ||
        d->L > 16)
        return dressi_fail(ctx, DRESSI_EINVAL, "ibl: bad descriptor (S, Si, Sp in 1..1024, L in 2..16)");
    return DRESSI_OK;
}

// The tables of k_ibl_tables in the context's scratch; env (the filter) or
// norm and the gradients (the adjoint).
struct IblTables {
    double4 *tab, *otab, *rhs;
    int64_t ne, no;
};
static size_t ibl_layout(const dressi_ibl_desc &d, IblTables &t, Carver &c, size_t *o) {
    t.ne = 6ll * d.S * d.S;
    t.no = 6ll * d.Si * d.Si + (int64_t)d.L * 6 * d.Sp * d.Sp;
    o[0] = c.take(sizeof(double4) * (size_t)t.ne);
    o[1] = c.take(sizeof(double4) * (size_t)t.no);
    o[2] = c.take(sizeof(double4) * (size_t)std::max(t.ne, t.no));
    return c.off;
}
static int ibl_tables(dressi_ctx *ctx, const dressi_ibl_desc *d, hipStream_t st, const float *env, const double *norm,
                      const float *g_irr, const float *g_pref, IblTables &t) {
    Carver c;
    size_t o[3];
    int rc = dressi_scratch(ctx, ibl_layout(*d, t, c, o), st);
    if (rc) return rc;
    t.tab = at<double4>(ctx->scratch, o[0]);
    t.otab = at<double4>(ctx->scratch, o[1]);
    t.rhs = at<double4>(ctx->scratch, o[2]);
    DR_LAUNCH("k_ibl_tables", (k_ibl_tables), (int)((std::max(t.ne, t.no) + 255) / 256), 256, 0, st, *d, t.ne,
              t.no, env, norm, g_irr, g_pref, t.tab, t.otab, t.rhs);
    return DRESSI_OK;
}

// Rows a lane: the more, the fewer LDS reads a pair, but the fewer workgroups.
// Below 4,096 rows (128 workgroups of two) one; else four where their last
// round over the 256 CUs is full enough, a round of four costing 1.7 of two.
// Measured with 1, 2 and 4 rows (us; rows x columns): 960 x 1,536 7.4, 10.4, 14.8;
// 8,064 x 6,144 36, 35, 51; 32,256 x 24,576 (504 workgroups of four) 487, 450, 380;
// 24,576 x 32,256 (384) 488, 431, 536; 57,888 x 38,400 1255, 1224, 1098.
template <bool ADJOINT>
static void ibl_contract(const char *name, const dressi_ibl_desc &d, const double4 *rows, int64_t n_rows,
                         const double4 *cols, const double4 *rhs, int64_t n_cols, float *out, float *pref,
                         double *norm, hipStream_t st) {
    const int64_t n_irr = 6ll * d.Si * d.Si;
    const auto grid = [&](int R) { return (int)((n_rows + 16 * R - 1) / (16 * R)); };
    const auto rounds = [&](int R) { return (grid(R) + 255) / 256; };
#define DR_IBL(RR)                                                                                               \
    DR_LAUNCH(name, (k_ibl_contract<RR, ADJOINT>), grid(RR), 64 * IBL_WAVES, 0, st, rows, n_rows, cols, rhs, n_cols, \
              n_irr, d, out, pref, norm)
    if (n_rows < 4096) DR_IBL(1);
    else if (17 * rounds(4) < 10 * rounds(2)) DR_IBL(4);
    else DR_IBL(2);
#undef DR_IBL
}

extern "C" size_t dressi_ibl_norm_bytes(const dressi_ibl_desc *d) {
    if (!d || d->Si < 1 || d->Sp < 1 || d->L < 2) return 0;
    return sizeof(double) * (6ull * d->Si * d->Si + (size_t)d->L * 6ull * d->Sp * d->Sp);
}

extern "C" int dressi_ibl_filter(dressi_ctx *ctx, const float *env, const dressi_ibl_desc *d, float *irr,
                                 float *pref, double *norm, void *stream) {
    int rc = check_ibl(ctx, d);
    if (rc) return rc;
    if (!env || !irr || !pref || !norm) return dressi_fail(ctx, DRESSI_EINVAL, "ibl_filter: null pointer");
    hipStream_t st = (hipStream_t)stream;
    IblTables t;
    if ((rc = ibl_tables(ctx, d, st, env, nullptr, nullptr, nullptr, t))) return rc;
    ibl_contract<false>("k_ibl_filter", *d, t.otab, t.no, t.tab, t.rhs, t.ne, irr, pref, norm, st);
    return dressi_launch_check(ctx, "ibl_filter");
}

extern "C" int dressi_ibl_filter_bwd(dressi_ctx *ctx, const dressi_ibl_desc *d, const double *norm,
                                     const float *grad_irr, const float *grad_pref, float *grad_env,
                                     void *stream) {
    int rc = check_ibl(ctx, d);
    if (rc) return rc;
    if (!norm || !grad_irr || !grad_pref || !grad_env)
        return dressi_fail(ctx, DRESSI_EINVAL, "ibl_filter_bwd: null pointer");
    hipStream_t st = (hipStream_t)stream;
    IblTables t;
    if ((rc = ibl_tables(ctx, d, st, nullptr, norm, grad_irr, grad_pref, t))) return rc;
    ibl_contract<true>("k_ibl_filter_bwd", *d, t.tab, t.ne, t.otab, t.rhs, t.no, grad_env, nullptr, nullptr, st);
    return dressi_launch_check(ctx, "ibl_filter_bwd");
}

// ---------------------------------------------------------------------------
// BRDF integration table
// ---------------------------------------------------------------------------
__global__ void k_brdf_lut(int N, int M, float2 *__restrict__ lut) {
    const int idx = blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= N * N) return;
    const int j = idx / N, i = idx - j * N;   // row: roughness, column: n.v
    const double r = (j + 0.5) / N, a = r * r, k = a / 2.0;
    const double c = (i + 0.5) / N;
    const double vx = sqrt(1.0 - c * c), vz = c;   // v in the xz plane, n = +z
    const double g1v = c / (c * (1.0 - k) + k);
    double A = 0.0, B = 0.0;
    for (int s = 0; s < M; s++) {
        const double x = (s + 0.5) / M;
        const double y = (double)__brev((unsigned)s) * (1.0 / 4294967296.0);   // radical inverse base 2
        const double ct = sqrt((1.0 - y) / (1.0 + (a * a - 1.0) * y));
        const double stt = sqrt(fmax(0.0, 1.0 - ct * ct));
        const double ph = 2.0 * 3.14159265358979323846 * x;
        const double hx = stt * cos(ph), hz = ct;
        const double vdh = vx * hx + vz * hz;
        const double ndl = 2.0 * vdh * hz - vz;
        if (!(ndl > 0.0)) continue;
        const double G = g1v * (ndl / (ndl * (1.0 - k) + k));
        const double gv = G * vdh / (hz * c);
        const double fc = pow(1.0 - vdh, 5.0);
        A += (1.0 - fc) * gv;
        B += fc * gv;
    }
    lut[idx] = make_float2((float)(A / M), (float)(B / M));
}

extern "C" int dressi_brdf_lut(dressi_ctx *ctx, int N, int M, float *lut, void *stream) {
    if (!ctx) return DRESSI_EINVAL;
    if (N < 1 || N > 1024 || M < 1 || !lut) return dressi_fail(ctx, DRESSI_EINVAL, "brdf_lut: bad arguments");
    DR_LAUNCH("k_brdf_lut", (k_brdf_lut), (N * N + 255) / 256, 256, 0, (hipStream_t)stream, N, M,
              reinterpret_cast<float2 *>(lut));
    return dressi_launch_check(ctx, "brdf_lut");
}

// ---------------------------------------------------------------------------
// split-sum shading
// ---------------------------------------------------------------------------
__device__ __forceinline__ double3 ld3f(const float *p) { return make_double3(p[0], p[1], p[2]); }

struct PbsFrag {
    double3 nn, v, R;   // shading normal, view direction, reflection
    double nlen, vlen, ndv, c;
    int l0;
    double f;
    bool rin;   // roughness inside [0, 1]: the level weight depends on it
};

// The lower level of the pair that a roughness samples, and the upper one's
// weight: the roughness clamped to [0, 1] (also keeping the level index in
// range for any roughness, NaN included)
__device__ __forceinline__ int pbs_level(double rough, int levels, double &f) {
    const double x = fmin(fmax(rough, 0.0), 1.0) * (levels - 1);
    const int l0 = min((int)floor(x), levels - 2);
    f = x - l0;
    return l0;
}

__device__ __forceinline__ PbsFrag pbs_geometry(const dressi_pbs_in &in, const float *eye, int64_t i,
                                                double rough) {
    PbsFrag q;
    const double3 n = ld3f(in.normal + i * in.normal_stride), p = ld3f(in.pos + i * in.pos_stride);
    q.nlen = sqrt(n.x * n.x + n.y * n.y + n.z * n.z);
    q.nn = make_double3(n.x / q.nlen, n.y / q.nlen, n.z / q.nlen);
    double3 v = make_double3(eye[0] - p.x, eye[1] - p.y, eye[2] - p.z);
    q.vlen = sqrt(v.x * v.x + v.y * v.y + v.z * v.z);
    q.v = make_double3(v.x / q.vlen, v.y / q.vlen, v.z / q.vlen);
    q.ndv = q.nn.x * q.v.x + q.nn.y * q.v.y + q.nn.z * q.v.z;
    q.c = fmax(q.ndv, 1e-4);
    q.R = make_double3(2.0 * q.ndv * q.nn.x - q.v.x, 2.0 * q.ndv * q.nn.y - q.v.y, 2.0 * q.ndv * q.nn.z - q.v.z);
    q.l0 = pbs_level(rough, in.levels, q.f);
    q.rin = rough >= 0.0 && rough <= 1.0;
    return q;
}

// bilinear lookup of the (A, B) table at (c, r), clamped, with its derivatives
struct LutS {
    double A, B, dAc, dBc, dAr, dBr;
};
__device__ __forceinline__ LutS lut_sample(const float *lut, int N, double c, double r) {
    const double s = c * N - 0.5, t = r * N - 0.5;
    const double x0 = floor(s), y0 = floor(t);
    const double fx = s - x0, fy = t - y0;
    auto cl = [N](double q) { return (int)fmin(fmax(q, 0.0), (double)(N - 1)); };
    const int X0 = cl(x0), X1 = cl(x0 + 1.0), Y0 = cl(y0), Y1 = cl(y0 + 1.0);
    const float *T00 = lut + 2 * (Y0 * N + X0), *T01 = lut + 2 * (Y0 * N + X1);
    const float *T10 = lut + 2 * (Y1 * N + X0), *T11 = lut + 2 * (Y1 * N + X1);
    LutS o;
    o.A = (1 - fx) * (1 - fy) * T00[0] + fx * (1 - fy) * T01[0] + (1 - fx) * fy * T10[0] + fx * fy * T11[0];
    o.B = (1 - fx) * (1 - fy) * T00[1] + fx * (1 - fy) * T01[1] + (1 - fx) * fy * T10[1] + fx * fy * T11[1];
    o.dAc = N * ((1 - fy) * ((double)T01[0] - T00[0]) + fy * ((double)T11[0] - T10[0]));
    o.dBc = N * ((1 - fy) * ((double)T01[1] - T00[1]) + fy * ((double)T11[1] - T10[1]));
    o.dAr = N * ((1 - fx) * ((double)T10[0] - T00[0]) + fx * ((double)T11[0] - T01[0]));
    o.dBr = N * ((1 - fx) * ((double)T10[1] - T00[1]) + fx * ((double)T11[1] - T01[1]));
    return o;
}

// directions for the lookups and the per-level fragment masks
__global__ void k_pbs_dirs(dressi_pbs_in in, const float *__restrict__ eye, const int32_t *__restrict__ tri_id,
                           int64_t Npv, int64_t n, float *__restrict__ dir_n, float *__restrict__ dir_r,
                           int32_t *__restrict__ level_tid) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const int t = tri_id[i];
    const double rough = in.material[1];
    int l0 = -1;
    if (t >= 0) {
        const PbsFrag q = pbs_geometry(in, eye + 3 * (i / Npv), i, rough);
        l0 = q.l0;
        if (dir_n) {
            dir_n[3 * i] = (float)q.nn.x;
            dir_n[3 * i + 1] = (float)q.nn.y;
            dir_n[3 * i + 2] = (float)q.nn.z;
        }
        if (dir_r) {
            dir_r[3 * i] = (float)q.R.x;
            dir_r[3 * i + 1] = (float)q.R.y;
            dir_r[3 * i + 2] = (float)q.R.z;
        }
    } else {
        for (int c = 0; c < 3; c++) {
            if (dir_n) dir_n[3 * i + c] = 0.0f;
            if (dir_r) dir_r[3 * i + c] = 0.0f;
        }
    }
    if (level_tid)
        for (int l = 0; l < in.levels; l++)
            level_tid[(int64_t)l * n + i] = (t >= 0 && (l == l0 || l == l0 + 1)) ? t : -1;
}

// x^5 and x^4 by squares
__device__ __forceinline__ double pow4(double x) { return (x * x) * (x * x); }
__device__ __forceinline__ double pow5(double x) { return pow4(x) * x; }

// a fragment's colour from its albedo, its irradiance sample and its samples
// of the level pair
__device__ __forceinline__ void pbs_color(const dressi_pbs_in &in, const PbsFrag &q, double m, double r,
                                          const float *a, const float *ir, const float *p0, const float *p1,
                                          float *o) {
    const LutS ab = lut_sample(in.lut, in.lut_n, q.c, r);
    const double w5 = pow5(1.0 - q.c);
#pragma unroll
    for (int ch = 0; ch < 3; ch++) {
        const double F0 = 0.04 * (1.0 - m) + a[ch] * m;
        const double F = F0 + (fmax(1.0 - r, F0) - F0) * w5;
        const double P = (1.0 - q.f) * p0[ch] + q.f * p1[ch];
        const double C = (1.0 - F) * (1.0 - m) * a[ch] * ir[ch] + P * (F0 * ab.A + ab.B);
        o[ch] = (float)(C / (1.0 + C));
    }
}

// its adjoint: the gradients of the albedo ga, the irradiance sample girr and
// the level pair's samples gp0, gp1 (stored as they are rounded), of n.v
// (returned) and, added, of the material
__device__ __forceinline__ double pbs_color_bwd(const dressi_pbs_in &in, const PbsFrag &q, double m, double r,
                                                const float *a, const float *ir, const float *p0, const float *p1,
                                                const float *go, float *oa, float *oirr, float *op0, float *op1,
                                                double &gm, double &gr) {
    const LutS ab = lut_sample(in.lut, in.lut_n, q.c, r);
    const double w5 = pow5(1.0 - q.c);
    double gA = 0.0, gB = 0.0, gw5 = 0.0, gf = 0.0;
#pragma unroll
    for (int ch = 0; ch < 3; ch++) {
        const double ac = a[ch];
        const double F0 = 0.04 * (1.0 - m) + ac * m;
        const bool fr_f0 = F0 > 1.0 - r;     // max(1 - r, F0) takes F0
        const double Fr = fr_f0 ? F0 : 1.0 - r;
        const double F = F0 + (Fr - F0) * w5;
        const double P = (1.0 - q.f) * p0[ch] + q.f * p1[ch];
        const double kd = (1.0 - F) * (1.0 - m);
        const double C = kd * ac * ir[ch] + P * (F0 * ab.A + ab.B);
        const double gC = go[ch] / ((1.0 + C) * (1.0 + C));
        // diffuse: kd a irr
        const double gkd = gC * ac * ir[ch];
        double ga = gC * kd * ir[ch];
        const double girr = gC * kd * ac;
        double gF = -gkd * (1.0 - m);
        gm += -gkd * (1.0 - F);
        // specular: P (F0 A + B)
        const double gP = gC * (F0 * ab.A + ab.B);
        double gF0 = gC * P * ab.A;
        gA += gC * P * F0;
        gB += gC * P;
        // F = F0 + (Fr - F0) w5
        gF0 += gF * (1.0 - w5);
        if (fr_f0) gF0 += gF * w5;
        else gr += -gF * w5;
        gw5 += gF * (Fr - F0);
        // F0 = 0.04 (1 - m) + a m
        gm += gF0 * (ac - 0.04);
        ga += gF0 * m;
        // P = (1 - f) p0 + f p1
        gf += gP * ((double)p1[ch] - p0[ch]);
        oa[ch] = (float)ga;
        oirr[ch] = (float)girr;
        op0[ch] = (float)(gP * (1.0 - q.f));
        op1[ch] = (float)(gP * q.f);
    }
    if (q.rin) gr += gf * (in.levels - 1);
    gr += gA * ab.dAr + gB * ab.dBr;
    return gw5 * (-5.0 * pow4(1.0 - q.c)) + gA * ab.dAc + gB * ab.dBc;
}

// the sum of a block's material gradients, one pair a block
__device__ __forceinline__ void pbs_material_part(double gm, double gr, double (*red)[PBS_BS],
                                                  double *__restrict__ part) {
    red[0][threadIdx.x] = gm;
    red[1][threadIdx.x] = gr;
    __syncthreads();
    for (int s = PBS_BS / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            red[0][threadIdx.x] += red[0][threadIdx.x + s];
            red[1][threadIdx.x] += red[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        part[2 * blockIdx.x] = red[0][0];
        part[2 * blockIdx.x + 1] = red[1][0];
    }
}

__global__ void k_pbs_shade(dressi_pbs_in in, const float *__restrict__ eye, const int32_t *__restrict__ tri_id,
                            int64_t Npv, int64_t n, float *__restrict__ color) {
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float *o = color + 3 * i;
    if (tri_id[i] < 0) {
        o[0] = o[1] = o[2] = 0.0f;
        return;
    }
    const double m = in.material[0], r = in.material[1];
    const PbsFrag q = pbs_geometry(in, eye + 3 * (i / Npv), i, r);
    const float *p0 = in.pref + (int64_t)q.l0 * in.pref_level_stride + i * in.pref_stride;
    pbs_color(in, q, m, r, in.albedo + i * in.albedo_stride, in.irr + i * in.irr_stride, p0,
              p0 + in.pref_level_stride, o);
}

// Backward per fragment.  Writes, when given: the albedo, irradiance-sample
// and prefiltered-sample gradients (every level, 0 off the two in use),
// normal and position gradients (with the lookups' direction gradients),
// and per-block partial sums of the material gradient.
__global__ void __launch_bounds__(PBS_BS)
    k_pbs_shade_bwd(dressi_pbs_in in, const float *__restrict__ eye, const int32_t *__restrict__ tri_id,
                    int64_t Npv, int64_t n, const float *__restrict__ grad_color,
                    const float *__restrict__ grad_dir_n, const float *__restrict__ grad_dir_r,
                    dressi_pbs_grad g, double *__restrict__ part) {
    __shared__ double red[2][PBS_BS];
    const int64_t i = (int64_t)blockIdx.x * PBS_BS + threadIdx.x;
    double gm = 0.0, gr = 0.0;
    if (i < n) {
        const bool cov = tri_id[i] >= 0;
        const int L = in.levels;
        if (!cov) {
            for (int ch = 0; ch < 3; ch++) {
                if (g.albedo) g.albedo[i * g.albedo_stride + ch] = 0.0f;
                if (g.irr) g.irr[3 * i + ch] = 0.0f;
                if (g.normal) g.normal[i * g.normal_stride + ch] = 0.0f;
                if (g.pos) g.pos[i * g.pos_stride + ch] = 0.0f;
                if (g.pref)
                    for (int l = 0; l < L; l++) g.pref[(int64_t)l * 3 * n + 3 * i + ch] = 0.0f;
            }
        } else {
            const double m = in.material[0], r = in.material[1];
            const float *e = eye + 3 * (i / Npv);
            const PbsFrag q = pbs_geometry(in, e, i, r);
            const float *p0 = in.pref + (int64_t)q.l0 * in.pref_level_stride + i * in.pref_stride;
            float oa[3], oirr[3], op0[3], op1[3];
            const double gc = pbs_color_bwd(in, q, m, r, in.albedo + i * in.albedo_stride,
                                            in.irr + i * in.irr_stride, p0, p0 + in.pref_level_stride,
                                            grad_color + 3 * i, oa, oirr, op0, op1, gm, gr);
#pragma unroll
            for (int ch = 0; ch < 3; ch++) {
                if (g.albedo) g.albedo[i * g.albedo_stride + ch] = oa[ch];
                if (g.irr) g.irr[3 * i + ch] = oirr[ch];
                if (g.pref)
                    for (int l = 0; l < L; l++)
                        g.pref[(int64_t)l * 3 * n + 3 * i + ch] =
                            l == q.l0 ? op0[ch] : (l == q.l0 + 1 ? op1[ch] : 0.0f);
            }
            if (g.normal || g.pos) {
                const double gndv = q.ndv >= 1e-4 ? gc : 0.0;
                double3 gnn = make_double3(gndv * q.v.x, gndv * q.v.y, gndv * q.v.z);
                double3 gv = make_double3(gndv * q.nn.x, gndv * q.nn.y, gndv * q.nn.z);
                if (grad_dir_n) {
                    gnn.x += grad_dir_n[3 * i];
                    gnn.y += grad_dir_n[3 * i + 1];
                    gnn.z += grad_dir_n[3 * i + 2];
                }
                if (grad_dir_r) {
                    double3 gR = make_double3(0.0, 0.0, 0.0);
                    for (int l = 0; l < L; l++) {
                        const float *gl = grad_dir_r + (int64_t)l * 3 * n + 3 * i;
                        gR.x += gl[0];
                        gR.y += gl[1];
                        gR.z += gl[2];
                    }
                    // R = 2 (n.v) n - v
                    const double gRn = gR.x * q.nn.x + gR.y * q.nn.y + gR.z * q.nn.z;
                    gnn.x += 2.0 * q.ndv * gR.x + 2.0 * gRn * q.v.x;
                    gnn.y += 2.0 * q.ndv * gR.y + 2.0 * gRn * q.v.y;
                    gnn.z += 2.0 * q.ndv * gR.z + 2.0 * gRn * q.v.z;
                    gv.x += 2.0 * gRn * q.nn.x - gR.x;
                    gv.y += 2.0 * gRn * q.nn.y - gR.y;
                    gv.z += 2.0 * gRn * q.nn.z - gR.z;
                }
                if (g.normal) {
                    const double d = gnn.x * q.nn.x + gnn.y * q.nn.y + gnn.z * q.nn.z;
                    float *gn = g.normal + i * g.normal_stride;
                    gn[0] = (float)((gnn.x - d * q.nn.x) / q.nlen);
                    gn[1] = (float)((gnn.y - d * q.nn.y) / q.nlen);
                    gn[2] = (float)((gnn.z - d * q.nn.z) / q.nlen);
                }
                if (g.pos) {
                    // v = (eye - p) / |eye - p|
                    const double d = gv.x * q.v.x + gv.y * q.v.y + gv.z * q.v.z;
                    float *gp = g.pos + i * g.pos_stride;
                    gp[0] = (float)(-(gv.x - d * q.v.x) / q.vlen);
                    gp[1] = (float)(-(gv.y - d * q.v.y) / q.vlen);
                    gp[2] = (float)(-(gv.z - d * q.v.z) / q.vlen);
                }
            }
        }
    }
    if (!g.material) return;   // uniform over the launch
    pbs_material_part(gm, gr, red, part);
}

__global__ void __launch_bounds__(PBS_BS) k_pbs_material_sum(const double *__restrict__ part, int nb,
                                                             float *__restrict__ out) {
    __shared__ double red[2][PBS_BS];
    double a = 0.0, b = 0.0;
    // eight pairs in flight, added in block order
    for (int k = threadIdx.x; k < nb; k += 8 * PBS_BS) {
        double2 v[8];
#pragma unroll
        for (int j = 0; j < 8; j++)
            v[j] = k + j * PBS_BS < nb ? reinterpret_cast<const double2 *>(part)[k + j * PBS_BS] : make_double2(0.0, 0.0);
#pragma unroll
        for (int j = 0; j < 8; j++) {
            if (k + j * PBS_BS >= nb) break;
            a += v[j].x;
            b += v[j].y;
        }
    }
    red[0][threadIdx.x] = a;
    red[1][threadIdx.x] = b;
    __syncthreads();
    for (int s = PBS_BS / 2; s > 0; s >>= 1) {
        if (threadIdx.x < s) {
            red[0][threadIdx.x] += red[0][threadIdx.x + s];
            red[1][threadIdx.x] += red[1][threadIdx.x + s];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        out[0] = (float)red[0][0];
        out[1] = (float)red[1][0];
    }
}

static int check_pbs(dressi_ctx *ctx, const dressi_pbs_in *in, const float *eye, const int32_t *tri_id, int B,
                     int64_t Npv) {
    if (!ctx) return DRESSI_EINVAL;
    if (!in || B < 0 || Npv < 0) return dressi_fail(ctx, DRESSI_EINVAL, "shade_pbs: bad arguments");
    if ((int64_t)B * Npv == 0) return DRESSI_OK;
    if (!in->normal || !in->pos || !in->material || !eye || !tri_id)
        return dressi_fail(ctx, DRESSI_EINVAL, "shade_pbs: null input");
    if (in->levels < 2 || in->levels > 16) return dressi_fail(ctx, DRESSI_EINVAL, "shade_pbs: levels in 2..16");
    if (in->normal_stride < 3 || in->pos_stride < 3)
        return dressi_fail(ctx, DRESSI_EINVAL, "shade_pbs: strides below 3");
    return DRESSI_OK;
}

extern "C" int dressi_shade_pbs(dressi_ctx *ctx, const dressi_pbs_in *in, const float *eye,
                                const int32_t *tri_id, int B, int64_t Npv, float *color, float *dir_n,
                                float *dir_r, int32_t *level_tri_id, void *stream) {
    int rc = check_pbs(ctx, in, eye, tri_id, B, Npv);
    if (rc) return rc;
    const int64_t n = (int64_t)B * Npv;
    if (n == 0) return DRESSI_OK;
    if (color && (!in->albedo || !in->irr || !in->pref || !in->lut || in->lut_n < 1 || in->albedo_stride < 3 ||
                  in->irr_stride < 3 || in->pref_stride < 3))
        return dressi_fail(ctx, DRESSI_EINVAL, "shade_pbs: colour needs albedo, samples and the table");
    hipStream_t st = (hipStream_t)stream;
    const int g = (int)((n + 255) / 256);
    if (dir_n || dir_r || level_tri_id)
        DR_LAUNCH("k_pbs_dirs", (k_pbs_dirs), g, 256, 0, st, *in, eye, tri_id, Npv, n, dir_n, dir_r, level_tri_id);
    if (color) DR_LAUNCH("k_pbs_shade", (k_pbs_shade), g, 256, 0, st, *in, eye, tri_id, Npv, n, color);
    return dressi_launch_check(ctx, "shade_pbs");
}

extern "C" int dressi_shade_pbs_bwd(dressi_ctx *ctx, const dressi_pbs_in *in, const float *eye,
                                    const int32_t *tri_id, int B, int64_t Npv, const float *grad_color,
                                    const float *grad_dir_n, const float *grad_dir_r, const dressi_pbs_grad *grad,
                                    void *stream) {
    int rc = check_pbs(ctx, in, eye, tri_id, B, Npv);
    if (rc) return rc;
    if (!grad) return dressi_fail(ctx, DRESSI_EINVAL, "shade_pbs_bwd: null grad");
    const int64_t n = (int64_t)B * Npv;
    hipStream_t st = (hipStream_t)stream;
    if (n == 0) {
        if (grad->material) dressi_fill_f32(grad->material, 0.0f, 2, st);
        return dressi_launch_check(ctx, "shade_pbs_bwd");
    }
    if (!grad_color || !in->albedo || !in->irr || !in->pref || !in->lut || in->lut_n < 1)
        return dressi_fail(ctx, DRESSI_EINVAL, "shade_pbs_bwd: null input");
    const int nb = (int)((n + PBS_BS - 1) / PBS_BS);
    double *part = nullptr;
    if (grad->material) {
        if ((rc = dressi_scratch(ctx, sizeof(double) * 2 * (size_t)nb, st))) return rc;
        part = at<double>(ctx->scratch, 0);
    }
    DR_LAUNCH("k_pbs_shade_bwd", (k_pbs_shade_bwd), nb, PBS_BS, 0, st, *in, eye, tri_id, Npv, n, grad_color,
              grad_dir_n, grad_dir_r, *grad, part);
    if (grad->material)
        DR_LAUNCH("k_pbs_material_sum", (k_pbs_material_sum), 1, PBS_BS, 0, st, part, nb, grad->material);
    return dressi_launch_check(ctx, "shade_pbs_bwd");
}

// ---------------------------------------------------------------------------
// packed PBS pass
// ---------------------------------------------------------------------------
// A step's fragments in one forward and one backward kernel in place of the
// directions, the albedo's, the irradiance's and every level's lookup, the
// shading, and their adjoints.  The roughness is one for all fragments, so all
// of them sample the same two levels (which two, only the device knows): the
// others need no lookup and their gradient is zero.  The irradiance map and
// the level pair keep one inverse-UV map each, registered by the forward; the
// backward stores sample gradients only for the pixels they kept, all that the
// texel gathers read.  20 views of 256^2 x 2 layers (8^2 and 16^2 faces, 5
// levels): 33 launches, 480 us, of which 152 the pixels' registration (many
// pixels a cell: now one atomic for a wavefront's run of them), in place of 8,
// 126 us; the two kernels here take 35 and 47, bound by the double-precision
// shading and, the backward, by 132 registers.
struct PbsMaps {
    int32_t *inv_irr, *inv_pref;   // [S, 6 Si Si], [S, 6 Sp Sp]
    float *dir_n, *dir_r;          // [N, 3] at kept pixels
    float *g_irr, *g_pref;         // [N, 3], [N, 8] (level l0, 0, level l0 + 1, 0) at kept pixels
    float *part_irr, *part_pref;   // the gathers' partial sums
};
static size_t pbs_maps(int Si, int Sp, int S, int64_t N, void *ws, PbsMaps &m) {
    const int64_t ci = (int64_t)6 * Si * Si, cp = (int64_t)6 * Sp * Sp;
    Carver c;
    char *b = static_cast<char *>(ws);
    m.inv_irr = reinterpret_cast<int32_t *>(b + c.take(sizeof(int32_t) * (size_t)(ci + cp) * S));
    m.inv_pref = m.inv_irr + ci * S;
    m.dir_n = reinterpret_cast<float *>(b + c.take(sizeof(float) * 3 * (size_t)N));
    m.dir_r = reinterpret_cast<float *>(b + c.take(sizeof(float) * 3 * (size_t)N));
    m.g_irr = reinterpret_cast<float *>(b + c.take(sizeof(float) * 3 * (size_t)N));
    m.g_pref = reinterpret_cast<float *>(b + c.take(sizeof(float) * 8 * (size_t)N));
    m.part_irr = reinterpret_cast<float *>(b + c.take(sizeof(float) * 3 * (size_t)ci * dressi_invuv_nsplit(ci, S)));
    m.part_pref = reinterpret_cast<float *>(b + c.take(sizeof(float) * 8 * (size_t)cp * dressi_invuv_nsplit(cp, S)));
    return c.off;
}
static dressi_tex_desc pbs_cube(int size, int Ct) {
    dressi_tex_desc d{};
    d.kind = DRESSI_TEX_CUBE;
    d.Ht = d.Wt = size;
    d.Ct = Ct;
    d.wrap_u = d.wrap_v = DRESSI_WRAP_CLAMP;
    return d;
}

__global__ void __launch_bounds__(256)
    k_pbs_layers_fwd(dressi_pbs_layers L, dressi_tex_desc ti, dressi_tex_desc tp, const float *__restrict__ eye,
                     const int32_t *__restrict__ tri_id, int K, uint32_t npix, int64_t n, float *__restrict__ samp,
                     float *__restrict__ irr_s, float *__restrict__ pref_s, float *__restrict__ color, PbsMaps mp,
                     int skip_empty) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i >= n) return;
    if (tri_id[i] < 0) {
        if (skip_empty) return;
        reinterpret_cast<float4 *>(samp)[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
        for (int c = 0; c < 3; c++)
            irr_s[3 * i + c] = pref_s[3 * i + c] = pref_s[3 * (n + i) + c] = color[3 * i + c] = 0.0f;
        return;
    }
    int sl, pix;
    slice_pixel(blockIdx.x, npix, sl, pix);
    const double m = L.in.material[0], r = L.in.material[1];
    const float q2[2] = {L.uv[2 * i], L.uv[2 * i + 1]};
    const PbsFrag q = pbs_geometry(L.in, eye + 3 * (sl / K), i, r);
    const float dn[3] = {(float)q.nn.x, (float)q.nn.y, (float)q.nn.z};
    const float dr[3] = {(float)q.R.x, (float)q.R.y, (float)q.R.z};
    const Taps ta = make_taps(L.td, q2, 0), tn = make_taps(ti, dn, 0), tr = make_taps(tp, dr, 0);
    float a[4] = {0.0f, 0.0f, 0.0f, 0.0f}, ir[3] = {0.0f, 0.0f, 0.0f}, p0[3] = {0.0f, 0.0f, 0.0f},
          p1[3] = {0.0f, 0.0f, 0.0f};
    if (ta.ok) tex_bilinear<4>(L.tex, L.td, ta, a, 4);
    if (tn.ok) tex_bilinear<3>(L.irr_map, ti, tn, ir, 3);
    const int64_t ci = (int64_t)6 * ti.Ht * ti.Wt, cp = (int64_t)6 * tp.Ht * tp.Wt;
    if (tr.ok) {
        const float *lv = L.pref_map + (int64_t)q.l0 * cp * 3;
        tex_bilinear<3>(lv, tp, tr, p0, 3);
        tex_bilinear<3>(lv + cp * 3, tp, tr, p1, 3);
    }
    tex_register(mp.inv_irr, tn.ok ? sl * ci + tex_cell(ti, tn, dn) : -1, pix);
    tex_register(mp.inv_pref, tr.ok ? sl * cp + tex_cell(tp, tr, dr) : -1, pix);
    float o[3];
    pbs_color(L.in, q, m, r, a, ir, p0, p1, o);
    reinterpret_cast<float4 *>(samp)[i] = make_float4(a[0], a[1], a[2], a[3]);
#pragma unroll
    for (int c = 0; c < 3; c++) {
        irr_s[3 * i + c] = ir[c];
        pref_s[3 * i + c] = p0[c];
        pref_s[3 * (n + i) + c] = p1[c];
        color[3 * i + c] = o[c];
    }
}

__global__ void __launch_bounds__(PBS_BS)
    k_pbs_layers_bwd(dressi_pbs_layers L, dressi_tex_desc ti, dressi_tex_desc tp, const float *__restrict__ eye,
                     const int32_t *__restrict__ tri_id, int K, uint32_t npix, int64_t n,
                     const float *__restrict__ samp, const float *__restrict__ irr_s,
                     const float *__restrict__ pref_s, const float *__restrict__ grad_color,
                     float *__restrict__ g_samp, PbsMaps mp, double *__restrict__ part, int skip_empty) {
    __shared__ double red[2][PBS_BS];
    const int64_t i = (int64_t)blockIdx.x * PBS_BS + threadIdx.x;
    double gm = 0.0, gr = 0.0;
    if (i < n) {
        if (tri_id[i] >= 0) {
            int sl, pix;
            slice_pixel(blockIdx.x, npix, sl, pix);
            const double m = L.in.material[0], r = L.in.material[1];
            float ir[3], p0[3], p1[3], go[3];
            const float4 a4 = reinterpret_cast<const float4 *>(samp)[i];
            const float a[3] = {a4.x, a4.y, a4.z};
#pragma unroll
            for (int c = 0; c < 3; c++) {
                ir[c] = irr_s[3 * i + c];
                p0[c] = pref_s[3 * i + c];
                p1[c] = pref_s[3 * (n + i) + c];
                go[c] = grad_color[3 * i + c];
            }
            const PbsFrag q = pbs_geometry(L.in, eye + 3 * (sl / K), i, r);
            const float dn[3] = {(float)q.nn.x, (float)q.nn.y, (float)q.nn.z};
            const float dr[3] = {(float)q.R.x, (float)q.R.y, (float)q.R.z};
            const Taps tn = make_taps(ti, dn, 0), tr = make_taps(tp, dr, 0);
            const int64_t ci = (int64_t)6 * ti.Ht * ti.Wt, cp = (int64_t)6 * tp.Ht * tp.Wt;
            const bool kn = tn.ok && mp.inv_irr[sl * ci + tex_cell(ti, tn, dn)] == pix;
            const bool kr = tr.ok && mp.inv_pref[sl * cp + tex_cell(tp, tr, dr)] == pix;
            float oa[3], oirr[3], op0[3], op1[3];
            pbs_color_bwd(L.in, q, m, r, a, ir, p0, p1, go, oa, oirr, op0, op1, gm, gr);
#pragma unroll
            for (int c = 0; c < 3; c++) g_samp[4 * i + c] = oa[c];
            if (kn) {
#pragma unroll
                for (int c = 0; c < 3; c++) {
                    mp.dir_n[3 * i + c] = dn[c];
                    mp.g_irr[3 * i + c] = oirr[c];
                }
            }
            if (kr) {
#pragma unroll
                for (int c = 0; c < 3; c++) mp.dir_r[3 * i + c] = dr[c];
                float4 *o = reinterpret_cast<float4 *>(mp.g_pref + 8 * i);
                o[0] = make_float4(op0[0], op0[1], op0[2], 0.0f);
                o[1] = make_float4(op1[0], op1[1], op1[2], 0.0f);
            }
        } else if (!skip_empty) {
            for (int c = 0; c < 3; c++) g_samp[4 * i + c] = 0.0f;
        }
    }
    pbs_material_part(gm, gr, red, part);
}

// The gathers' parts added in order: the irradiance map's gradient, the level
// pair's at its levels, zero at the others.
__global__ void k_pbs_map_grads(PbsMaps mp, int ns_irr, int64_t n_irr, int ns_pref, int64_t cells, int levels,
                                const float *__restrict__ material, float *__restrict__ g_irr,
                                float *__restrict__ g_pref) {
    int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_irr) {
        float a = mp.part_irr[i];
        for (int k = 1; k < ns_irr; k++) a += mp.part_irr[k * n_irr + i];
        g_irr[i] = a;
        return;
    }
    i -= n_irr;
    if (i >= levels * cells * 3) return;
    const int l = (int)(i / (cells * 3)), c = (int)(i % 3);
    const int64_t cell = i / 3 - l * cells;
    double f;
    const int l0 = pbs_level(material[1], levels, f);
    float a = 0.0f;
    if (l == l0 || l == l0 + 1) {
        const float *p = mp.part_pref + 8 * cell + 4 * (l - l0) + c;
        a = p[0];
        for (int k = 1; k < ns_pref; k++) a += p[(int64_t)k * cells * 8];
    }
    g_pref[i] = a;
}

extern "C" size_t dressi_pbs_layers_bytes(int Si, int Sp, int S, int H, int W) {
    if (Si < 1 || Sp < 1 || S < 0 || H < 0 || W < 0) return 0;
    PbsMaps m;
    return pbs_maps(Si, Sp, S, (int64_t)S * H * W, nullptr, m);
}

static int check_pbs_layers(dressi_ctx *ctx, const dressi_pbs_layers *L, const float *eye, const int32_t *tri_id,
                            int B, int K, int H, int W, const float *samp, const float *irr_s, const float *pref_s,
                            const void *ws) {
    if (!L || B < 0 || K < 1 || K > DRESSI_MAX_K || H < 0 || W < 0)
        return ctx ? dressi_fail(ctx, DRESSI_EINVAL, "pbs_layers: bad arguments") : DRESSI_EINVAL;
    int rc = check_pbs(ctx, &L->in, eye, tri_id, B, (int64_t)K * H * W);
    if (rc) return rc;
    const dressi_tex_desc ti = pbs_cube(L->Si, 3), tp = pbs_cube(L->Sp, 3);
    if (L->td.kind != DRESSI_TEX_2D || L->td.Ct != 4 || (((uintptr_t)L->tex | (uintptr_t)samp | (uintptr_t)ws) & 15u))
        return dressi_fail(ctx, DRESSI_EINVAL, "pbs_layers: the albedo is a 2-D RGBA texture, 16-byte aligned");
    if ((rc = dr_check_tex(ctx, L->tex, &L->td, L->uv, tri_id, B * K, H, W))) return rc;
    if ((rc = dr_check_tex(ctx, L->irr_map, &ti, L->uv, tri_id, B * K, H, W))) return rc;
    if ((rc = dr_check_tex(ctx, L->pref_map, &tp, L->uv, tri_id, B * K, H, W))) return rc;
    if ((int64_t)B * H * W > 0 && (!samp || !irr_s || !pref_s || !ws || !L->in.lut || L->in.lut_n < 1))
        return dressi_fail(ctx, DRESSI_EINVAL, "pbs_layers: null input or output");
    return DRESSI_OK;
}

extern "C" int dressi_pbs_layers_forward(dressi_ctx *ctx, const dressi_pbs_layers *L, const float *eye,
                                         const int32_t *tri_id, int B, int K, int H, int W, float *samp,
                                         float *irr_s, float *pref_s, float *color, void *ws, void *stream) {
    int rc = check_pbs_layers(ctx, L, eye, tri_id, B, K, H, W, samp, irr_s, pref_s, ws);
    if (rc) return rc;
    const int64_t npix = (int64_t)H * W, n = (int64_t)B * K * npix;
    if (n == 0) return DRESSI_OK;
    if (!color) return dressi_fail(ctx, DRESSI_EINVAL, "pbs_layers: null colour");
    hipStream_t st = (hipStream_t)stream;
    PbsMaps mp;
    pbs_maps(L->Si, L->Sp, B * K, n, ws, mp);
    dressi_fill_i32(mp.inv_irr, -1, (int64_t)6 * (L->Si * L->Si + L->Sp * L->Sp) * B * K, st);
    DR_LAUNCH("k_pbs_layers_fwd", (k_pbs_layers_fwd), (unsigned)((n + 255) / 256), 256, 0, st, *L,
              pbs_cube(L->Si, 3), pbs_cube(L->Sp, 3), eye, tri_id, K, (uint32_t)npix, n, samp, irr_s, pref_s, color,
              mp, ctx->skip_empty);
    return dressi_launch_check(ctx, "pbs_layers_forward");
}

extern "C" int dressi_pbs_layers_backward(dressi_ctx *ctx, const dressi_pbs_layers *L, const float *eye,
                                          const int32_t *tri_id, int B, int K, int H, int W, const float *samp,
                                          const float *irr_s, const float *pref_s, const float *grad_color,
                                          float *grad_samp, void *ws, float *grad_irr, float *grad_pref,
                                          float *grad_material, void *stream) {
    int rc = check_pbs_layers(ctx, L, eye, tri_id, B, K, H, W, samp, irr_s, pref_s, ws);
    if (rc) return rc;
    if (!grad_irr || !grad_pref || !grad_material)
        return dressi_fail(ctx, DRESSI_EINVAL, "pbs_layers: null gradient");
    const int S = B * K, levels = L->in.levels;
    const int64_t npix = (int64_t)H * W, n = S * npix;
    const int64_t ci = (int64_t)6 * L->Si * L->Si, cp = (int64_t)6 * L->Sp * L->Sp;
    hipStream_t st = (hipStream_t)stream;
    if (n == 0) {
        dressi_fill_f32(grad_irr, 0.0f, 3 * ci, st);
        dressi_fill_f32(grad_pref, 0.0f, 3 * cp * levels, st);
        dressi_fill_f32(grad_material, 0.0f, 2, st);
        return dressi_launch_check(ctx, "pbs_layers_backward");
    }
    if (!grad_color || !grad_samp) return dressi_fail(ctx, DRESSI_EINVAL, "pbs_layers: null gradient");
    const int nb = (int)((n + PBS_BS - 1) / PBS_BS);
    if ((rc = dressi_scratch(ctx, sizeof(double) * 2 * (size_t)nb, st))) return rc;
    double *part = at<double>(ctx->scratch, 0);
    PbsMaps mp;
    pbs_maps(L->Si, L->Sp, S, n, ws, mp);
    DR_LAUNCH("k_pbs_layers_bwd", (k_pbs_layers_bwd), nb, PBS_BS, 0, st, *L, pbs_cube(L->Si, 3), pbs_cube(L->Sp, 3),
              eye, tri_id, K, (uint32_t)npix, n, samp, irr_s, pref_s, grad_color, grad_samp, mp, part,
              ctx->skip_empty);
    DR_LAUNCH("k_pbs_material_sum", (k_pbs_material_sum), 1, PBS_BS, 0, st, part, nb, grad_material);
    const int nsi = dr_gather_parts(pbs_cube(L->Si, 3), mp.dir_n, tri_id, S, npix, mp.inv_irr, mp.g_irr, mp.part_irr,
                                    st, ctx->iv_rows);
    const int nsp = dr_gather_parts(pbs_cube(L->Sp, 8), mp.dir_r, tri_id, S, npix, mp.inv_pref, mp.g_pref,
                                    mp.part_pref, st, ctx->iv_rows);
    const int64_t no = 3 * (ci + cp * levels);
    DR_LAUNCH("k_pbs_map_grads", (k_pbs_map_grads), (int)((no + 255) / 256), 256, 0, st, mp, nsi, 3 * ci, nsp, cp,
              levels, L->in.material, grad_irr, grad_pref);
    return dressi_launch_check(ctx, "pbs_layers_backward");
}

// ibl_filter(_bwd) tables and shade_pbs_bwd's material partials
size_t dr_need_pbs(const dressi_limits &l) {
    size_t need = 0;
    if (l.ibl_S > 0) {
        IblTables t;
        Carver c;
        size_t o[3];
        ibl_layout(dressi_ibl_desc{l.ibl_S, l.ibl_Si, l.ibl_Sp, l.ibl_L}, t, c, o);
        need = c.off;
    }
    if (l.pbs_fragments > 0)
        need = std::max(need, sizeof(double) * 2 * (size_t)((l.pbs_fragments + PBS_BS - 1) / PBS_BS));
    return need;
}

// Interpolation kernels of the Chebyshev far field (Sec. III.A.1 Eq. p2m).
//
// Both kernels use the tensor-product structure of the interpolant,
// S(xbar_m, t) = S_x(i, t_x) S_y(j, t_y) S_z(k, t_z) for node m = (i n + j) n + k,
// with the 1D Lagrange polynomial of node i written as
// S(i, t) = sum_k coef[i][k] T_k(t) (T_k by the three-term recurrence, its
// derivative as k U_{k-1}). One wave handles one box.
//
// P2M: lane (j, k) owns the n nodes (0..n-1, j, k) and keeps their n sums in
// registers; each source is reduced once to the 3n values S_c(i, t_c) (and
// 3n derivatives for the double layer) when it is staged in LDS, so the
// inner loop costs 2 LDS reads and about 2n + 8 FMAs per (source, lane).
// The double layer uses
//   sum_j m . grad S = dS_x (m_x S_y S_z) + S_x (m_y dS_y S_z + m_z S_y dS_z).
//
// L2P: lane = target. The contraction over the n^3 node values (staged in
// LDS, read by broadcast) runs axis by axis: z inside, then y, then x.
#include "chebyshev.hpp"

namespace fmm {

namespace {

// T_k(t), k < N, and (if D) T_k'(t) = k U_{k-1}(t), into registers. The
// interpolation weights are formed in float64: a float32 weight is off by
// about 1e-7 absolute, and n^3 such errors against a smooth kernel do not
// cancel (they would cap the far field near 1e-6).
template <int N, bool D>
__device__ inline void cheb_basis(double t, double *tk, double *dtk) {
    tk[0] = 1.0;
    if (N > 1) tk[1] = t;
#pragma unroll
    for (int k = 2; k < N; ++k) tk[k] = 2.0 * t * tk[k - 1] - tk[k - 2];
    if (D) {
        double u0 = 1.0, u1 = 2.0 * t;  // U_0, U_1
        dtk[0] = 0.0;
        if (N > 1) dtk[1] = 1.0;
#pragma unroll
        for (int k = 2; k < N; ++k) {
            dtk[k] = k * u1;
            const double u2 = 2.0 * t * u1 - u0;
            u0 = u1;
            u1 = u2;
        }
    }
}

// S(i, t) and (if D) dS/dt for every node i of one axis; cf [N][N] float64.
template <int N, bool D, typename T>
__device__ inline void cheb_lagrange_1d(const double *cf, double t, T *s, T *ds) {
    double tk[N], dtk[N];
    cheb_basis<N, D>(t, tk, dtk);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        double v = 0.0, dv = 0.0;
#pragma unroll
        for (int k = 0; k < N; ++k) {
            v += cf[i * N + k] * tk[k];
            if (D) dv += cf[i * N + k] * dtk[k];
        }
        s[i] = (T)v;
        if (D) ds[i] = (T)dv;
    }
}

// acc[i][r] += the terms of two staged sources at nodes (i, jy, kz): their
// float32 terms are added, then one float64 add
template <int N, int NRHS, bool SL, bool DL, int W, int OS, int OD, int OQ, int OM>
__device__ inline void pair_to_nodes(const float *p0, int jy, int kz, double (&acc)[N][NRHS]) {
    // the weights of x-node i for one source: S_x(i) A + dS_x(i) B
    auto weights = [&](const float *p, float (&A)[NRHS], float (&B)[NRHS]) {
        const float sy = p[OS + N + jy], sz = p[OS + 2 * N + kz];
#pragma unroll
        for (int r = 0; r < NRHS; ++r) {
            A[r] = SL ? p[OQ + r] * (sy * sz) : 0.f;
            B[r] = 0.f;
        }
        if (DL) {
            const float dsy = p[OD + N + jy], dsz = p[OD + 2 * N + kz];
#pragma unroll
            for (int r = 0; r < NRHS; ++r) {
                A[r] += p[OM + 3 * r + 1] * (dsy * sz) + p[OM + 3 * r + 2] * (sy * dsz);
                B[r] = p[OM + 3 * r] * (sy * sz);
            }
        }
    };
    const float *p1 = p0 + W;
    float A0[NRHS], B0[NRHS], A1[NRHS], B1[NRHS];
    weights(p0, A0, B0);
    weights(p1, A1, B1);
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const float sx0 = p0[OS + i], sx1 = p1[OS + i];
        const float dsx0 = DL ? p0[OD + i] : 0.f, dsx1 = DL ? p1[OD + i] : 0.f;
#pragma unroll
        for (int r = 0; r < NRHS; ++r) {
            const float t0 = DL ? sx0 * A0[r] + dsx0 * B0[r] : sx0 * A0[r];
            const float t1 = DL ? sx1 * A1[r] + dsx1 * B1[r] : sx1 * A1[r];
            acc[i][r] += (double)(t0 + t1);
        }
    }
}

template <int N, int NRHS, bool SL, bool DL>
__global__ __launch_bounds__(64) void k_points_to_nodes(const double *coef, const int32_t *items, const int32_t *roff,
                                                       const int32_t *rng, SurfaceGeom g, PointSrc src, float *out) {
    // per staged source: S_c(i) for c = x, y, z; dS_c(i) (DL); then q, m / h
    constexpr int OS = 0, OD = 3 * N, OQ = DL ? 6 * N : 3 * N, OM = OQ + (SL ? NRHS : 0);
    constexpr int W = OM + (DL ? 3 * NRHS : 0);
    __shared__ float sh[64 * W];
    __shared__ double cf[N * N];
    const int lane = threadIdx.x;
    const int b = items[blockIdx.x];
    if (lane < N * N) cf[lane] = coef[lane];
    const double cx = g.centre[3 * b], cy = g.centre[3 * b + 1], cz = g.centre[3 * b + 2];
    const double ih = 1.0 / g.half[b];
    const bool act = lane < N * N;
    const int jy = act ? lane / N : 0, kz = act ? lane % N : 0;
    // float64 sums: the Lagrange weights take both signs and cancel
    double acc[N][NRHS];
#pragma unroll
    for (int i = 0; i < N; ++i)
        for (int r = 0; r < NRHS; ++r) acc[i][r] = 0.0;
    __syncthreads();
    for (int e = roff[blockIdx.x]; e < roff[blockIdx.x + 1]; ++e) {
        const int s0 = rng[2 * e], s1 = rng[2 * e + 1];
        for (int j0 = s0; j0 < s1; j0 += 64) {
            const int j = j0 + lane;
            const int cnt = min(64, s1 - j0);
            if (j >= s1 && lane < ((cnt + 1) & ~1)) {
                // the odd tail slot: a zero-strength record, so the loop below takes sources in pairs
                float *p = sh + lane * W;
                for (int k = 0; k < W; ++k) p[k] = 0.f;
            }
            if (j < s1) {
                float *p = sh + lane * W;
                const double t[3] = {((double)src.x[j] - cx) * ih, ((double)src.y[j] - cy) * ih,
                                     ((double)src.z[j] - cz) * ih};
#pragma unroll
                for (int c = 0; c < 3; ++c) cheb_lagrange_1d<N, DL>(cf, t[c], p + OS + c * N, p + OD + c * N);
                if (SL)
                    for (int r = 0; r < NRHS; ++r) p[OQ + r] = src.q[r * src.n + j];
                if (DL)
                    for (int r = 0; r < NRHS; ++r) {
                        p[OM + 3 * r] = (float)(src.mx[r * src.n + j] * ih);
                        p[OM + 3 * r + 1] = (float)(src.my[r * src.n + j] * ih);
                        p[OM + 3 * r + 2] = (float)(src.mz[r * src.n + j] * ih);
                    }
            }
            __syncthreads();
            for (int jj = 0; jj < cnt; jj += 2)
                pair_to_nodes<N, NRHS, SL, DL, W, OS, OD, OQ, OM>(sh + jj * W, jy, kz, acc);
            __syncthreads();
        }
    }
    if (!act) return;
#pragma unroll
    for (int i = 0; i < N; ++i)
        for (int r = 0; r < NRHS; ++r)
            out[((int64_t)b * NRHS + r) * g.n_pad + (i * N + jy) * N + kz] = (float)acc[i][r];
}

// P2M where there are fewer leaves than the chip has wave slots: four waves
// per leaf. Tiles of 64 sources are staged by all (wave c < 3 forms the
// weights of axis c, wave 3 copies the strengths) and their pairs of sources
// dealt to the waves, whose sums are added in LDS in a fixed order. Each pair's
// term and the float64 accumulation are those of the kernel above.
// Bound by latency there (one wave a leaf runs two tiles of staging and 64
// sources in sequence); with more leaves the staging's barriers and the final
// sums cost more than they save. Measured, one wave -> four: 224 leaves, double
// layer, n = 8 20 -> 11.5 us; 6953 leaves 28 -> 35 us; 77,834 leaves 502 -> 634
// us. About the line of 1024 leaves it depends on their points (n = 8, single
// layer; both layers and four densities): 512 leaves of 39 points 10.1 -> 9.8 and
// 23.8 -> 16.7 us, of 11 points 8.9 -> 8.1 and 14.6 -> 13.2; 1100 of 93 30.7 -> 17.3
// and 93 -> 51; 1480 of 8 9.3 -> 11.0 and 15.2 -> 22.2; 3800 of 26 16.8 -> 21.2 and
// 46.7 -> 54.5.
template <int N, int NRHS, bool SL, bool DL>
__global__ __launch_bounds__(256) void k_points_to_nodes4(const double *coef, const int32_t *items,
                                                         const int32_t *roff, const int32_t *rng, SurfaceGeom g,
                                                         PointSrc src, float *out) {
    constexpr int OS = 0, OD = 3 * N, OQ = DL ? 6 * N : 3 * N, OM = OQ + (SL ? NRHS : 0);
    constexpr int W = OM + (DL ? 3 * NRHS : 0), NW = 4;
    constexpr size_t NSH = sizeof(float) * 64 * W, NRED = sizeof(double) * NW * 64 * N;
    __shared__ __align__(16) unsigned char lds[NSH > NRED ? NSH : NRED];
    float *sh = (float *)lds;
    double *red = (double *)lds;  // the sums of the end reuse the records' space
    __shared__ double cf[N * N];
    const int lane = threadIdx.x & 63, w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int b = items[blockIdx.x];
    if (threadIdx.x < N * N) cf[threadIdx.x] = coef[threadIdx.x];
    const double ctr = g.centre[3 * b + min(w, 2)];
    const double ih = 1.0 / g.half[b];
    const bool act = lane < N * N;
    const int jy = act ? lane / N : 0, kz = act ? lane % N : 0;
    const float *xyz = w == 0 ? src.x : w == 1 ? src.y : src.z;
    double acc[N][NRHS];
#pragma unroll
    for (int i = 0; i < N; ++i)
        for (int r = 0; r < NRHS; ++r) acc[i][r] = 0.0;
    for (int e = roff[blockIdx.x]; e < roff[blockIdx.x + 1]; ++e) {
        const int s0 = rng[2 * e], s1 = rng[2 * e + 1];
        for (int j0 = s0; j0 < s1; j0 += 64) {
            const int j = j0 + lane;
            const int cnt = min(64, s1 - j0);
            __syncthreads();  // cf; every wave is done with the previous tile
            float *p = sh + lane * W;
            if (w < 3) {
                // past the range: zero weights (the odd tail slot of the pairs below)
                if (j < s1) {
                    const double t = ((double)xyz[j] - ctr) * ih;
                    cheb_lagrange_1d<N, DL>(cf, t, p + OS + w * N, p + OD + w * N);
                } else {
#pragma unroll
                    for (int k = 0; k < N; ++k) {
                        p[OS + w * N + k] = 0.f;
                        if (DL) p[OD + w * N + k] = 0.f;
                    }
                }
            } else {
                if (SL)
                    for (int r = 0; r < NRHS; ++r) p[OQ + r] = j < s1 ? src.q[r * src.n + j] : 0.f;
                if (DL)
                    for (int r = 0; r < NRHS; ++r) {
                        p[OM + 3 * r] = j < s1 ? (float)(src.mx[r * src.n + j] * ih) : 0.f;
                        p[OM + 3 * r + 1] = j < s1 ? (float)(src.my[r * src.n + j] * ih) : 0.f;
                        p[OM + 3 * r + 2] = j < s1 ? (float)(src.mz[r * src.n + j] * ih) : 0.f;
                    }
            }
            __syncthreads();
            for (int jj = 2 * w; jj < cnt; jj += 2 * NW)
                pair_to_nodes<N, NRHS, SL, DL, W, OS, OD, OQ, OM>(sh + jj * W, jy, kz, acc);
        }
    }
#pragma unroll
    for (int r = 0; r < NRHS; ++r) {  // static index keeps acc in registers
        __syncthreads();
#pragma unroll
        for (int i = 0; i < N; ++i) red[(w * N + i) * 64 + lane] = acc[i][r];
        __syncthreads();
        if (act)
            for (int i = w; i < N; i += NW) {
                double v = red[i * 64 + lane];
                for (int k = 1; k < NW; ++k) v += red[(k * N + i) * 64 + lane];
                out[((int64_t)b * NRHS + r) * g.n_pad + i * N * N + lane] = (float)v;
            }
    }
}

template <int N, int NRHS, bool FIELD>
__global__ __launch_bounds__(64) void k_nodes_to_points(const double *coef, EvalArgs a, SurfaceGeom g, const float *L) {
    constexpr int NN = N * N * N;
    // node values as stored (float32): every lane reads each of them, so LDS
    // return bandwidth, not arithmetic, bounds this kernel; float32 halves it
    // and the float64 arithmetic sees the same values
    __shared__ __align__(16) float sl[NRHS * NN];
    __shared__ double cf[N * N];
    const int lane = threadIdx.x;
    const int leaf = a.wleaf[blockIdx.x];
    const int64_t t_first = a.tbeg[leaf] + a.wt0[blockIdx.x];
    const int nt = (int)min((int64_t)64, a.tend[leaf] - t_first);
    if (lane < N * N) cf[lane] = coef[lane];
    {
        // all loads first, then the LDS writes (the loads overlap)
        constexpr int NV = (NN + 63) / 64;
        float lv[NRHS][NV];
#pragma unroll
        for (int r = 0; r < NRHS; ++r)
#pragma unroll
            for (int i = 0; i < NV; ++i)  // clamped index: no branch per load
                lv[r][i] = L[((int64_t)leaf * NRHS + r) * g.n_pad + min(lane + 64 * i, NN - 1)];
#pragma unroll
        for (int r = 0; r < NRHS; ++r)
#pragma unroll
            for (int i = 0; i < NV; ++i)
                if (lane + 64 * i < NN) sl[r * NN + lane + 64 * i] = lv[r][i];
    }
    __syncthreads();
    // SP lanes per target for short items (SP a power of two, nt SP <= 64):
    // lane part takes x-nodes i = part, part + SP, ..., and the SP partial
    // sums are added across the group's lanes at the end (a fixed order)
    int SP = 1;
    while (SP * 2 <= N && nt * SP * 2 <= 64) SP *= 2;
    const int part = lane & (SP - 1), tl = lane / SP;
    const bool valid = tl < nt;
    const int64_t k = t_first + (valid ? tl : 0);
    const double ih = 1.0 / g.half[leaf];
    const double tx = ((double)a.tx[k] - g.centre[3 * leaf]) * ih;
    const double ty = ((double)a.ty[k] - g.centre[3 * leaf + 1]) * ih;
    const double tz = ((double)a.tz[k] - g.centre[3 * leaf + 2]) * ih;
    double sy[N], sz[N], dsy[N], dsz[N], tk[N], dtk[N];
    cheb_lagrange_1d<N, FIELD>(cf, ty, sy, dsy);
    cheb_lagrange_1d<N, FIELD>(cf, tz, sz, dsz);
    cheb_basis<N, FIELD>(tx, tk, dtk);
    const int64_t dst = a.trg_perm ? a.trg_perm[k] : k;
#pragma unroll
    for (int r = 0; r < NRHS; ++r) {
        const float *lr = sl + r * NN;
        double pot = 0.0, gx = 0.0, gy = 0.0, gz = 0.0;
        // the x axis stays a loop (n^2 node values live at a time); S_x(i) is
        // formed from row i of the coefficients
#pragma unroll 1
        for (int i = part; i < N; i += SP) {
            double sxi = 0.0, dsxi = 0.0;
#pragma unroll
            for (int q = 0; q < N; ++q) {
                sxi += cf[i * N + q] * tk[q];
                if (FIELD) dsxi += cf[i * N + q] * dtk[q];
            }
            double bi = 0.0, biy = 0.0, biz = 0.0;
#pragma unroll
            for (int j = 0; j < N; ++j) {
                double az = 0.0, azd = 0.0;
#pragma unroll
                for (int kk = 0; kk < N; ++kk) {
                    const double l = (double)lr[(i * N + j) * N + kk];
                    az += sz[kk] * l;
                    if (FIELD) azd += dsz[kk] * l;
                }
                bi += sy[j] * az;
                if (FIELD) {
                    biy += dsy[j] * az;
                    biz += sy[j] * azd;
                }
            }
            pot += sxi * bi;
            if (FIELD) {
                gx += dsxi * bi;
                gy += sxi * biy;
                gz += sxi * biz;
            }
        }
        for (int o = 1; o < SP; o <<= 1) {
            pot += __shfl_xor(pot, o);
            if (FIELD) {
                gx += __shfl_xor(gx, o);
                gy += __shfl_xor(gy, o);
                gz += __shfl_xor(gz, o);
            }
        }
        if (!valid || part != 0) continue;
        if (a.pot) {
            float *pp = a.pot + r * a.n_trg + dst;
            *pp = a.accumulate ? (float)((double)*pp + pot) : (float)pot;
        }
        if (FIELD && a.field) {
            // field = -grad_x f = -(1/h) grad_t f
            float *f = a.field + ((int64_t)r * a.n_trg + dst) * 3;
            const double gr[3] = {-ih * gx, -ih * gy, -ih * gz};
            for (int c = 0; c < 3; ++c) f[c] = a.accumulate ? (float)((double)f[c] + gr[c]) : (float)gr[c];
        }
    }
}

// L2P with 8 nodes a side: one wave per item, 16 targets at a time. The z sum
// of every (i, j) is a matrix product, 64 (i, j) x 8 nodes by 8 x 16 targets, in
// v_mfma_f64_16x16x4_f64: the node values are held in registers, converted
// once per item, where one lane per target read all 512 from LDS and converted
// them in every lane. The rows are dealt so that lane group g = 2 ga + gb
// (lane = 16 g + target) gets the sums of half ga of the x nodes and half gb of
// the y nodes and needs 4 + 4 + 2 of the 24 one-dimensional weights, five
// mirrored pairs; the groups' shares of a target are added across lanes at the
// end. Bound by latency and the reads of the coefficients from LDS. Measured,
// one lane per target -> this: 99,230 items (4M points) 308 -> 210 us; 35,709
// items, three right-hand sides 178 -> 105; 8535 items with the field 64 -> 38.
typedef double f64x4 __attribute__((ext_vector_type(4)));

template <int NRHS, bool FIELD>
__global__ __launch_bounds__(64, NRHS > 2 ? 3 : 4) void k_nodes_to_points8(const double *coef, EvalArgs a, SurfaceGeom g, const float *L) {
    constexpr int N = 8;
    __shared__ __align__(16) double cf[N * N];
    const int lane = threadIdx.x, c16 = lane & 15, grp = lane >> 4, ga = grp >> 1, gb = grp & 1;
    const int leaf = a.wleaf[blockIdx.x];
    const int64_t t_first = a.tbeg[leaf] + a.wt0[blockIdx.x];
    const int nt = (int)min((int64_t)64, a.tend[leaf] - t_first);
    cf[lane] = coef[lane];
    // node v of the half h of an axis: the pairs n, 7 - n of n = 2 h, 2 h + 1
    auto node = [](int h, int v) { return v & 1 ? 7 - (2 * h + (v >> 1)) : 2 * h + (v >> 1); };
    // A fragments: row c16 of block ii is i = node(row >> 1 & 1, ii), j = node(row & 1, row >> 2);
    // the product of step s takes k = grp, then 7 - grp
    double av[NRHS][4][2];
#pragma unroll
    for (int r = 0; r < NRHS; ++r)
#pragma unroll
        for (int ii = 0; ii < 4; ++ii) {
            const int i = node(c16 >> 1 & 1, ii), j = node(c16 & 1, c16 >> 2);
            const float *v = L + ((int64_t)leaf * NRHS + r) * g.n_pad + (i * N + j) * N;
            av[r][ii][0] = (double)v[grp];
            av[r][ii][1] = (double)v[7 - grp];
        }
    const double ih = 1.0 / g.half[leaf];
    const double cx = g.centre[3 * leaf], cy = g.centre[3 * leaf + 1], cz = g.centre[3 * leaf + 2];
    __syncthreads();
#pragma unroll 1
    for (int t0 = 0; t0 < nt; t0 += 16) {
        asm volatile("" ::: "memory");  // the coefficients stay in LDS: 80 of them would take 160 registers
        const bool valid = t0 + c16 < nt;
        const int64_t k = t_first + (valid ? t0 + c16 : 0);
        const int64_t dst = a.trg_perm ? a.trg_perm[k] : k;
        double tk[N], dtk[N];
        // S and dS of nodes n and 7 - n, mirror images, for the basis values
        // in tk: the sums over even and odd degrees, added and subtracted
        auto lagrange = [&](int n, double *v, double *dv) {
            double e[2] = {0.0, 0.0}, de[2] = {0.0, 0.0};
#pragma unroll
            for (int q = 0; q < N; ++q) {
                const double c = cf[n * N + q];
                e[q & 1] += c * tk[q];
                if (FIELD) de[q & 1] += c * dtk[q];
            }
            v[0] = e[0] + e[1];
            v[1] = e[0] - e[1];
            if (FIELD) {
                dv[0] = de[0] + de[1];
                dv[1] = de[0] - de[1];
            }
        };
        double sx[4], sy[4], sz[2], dsx[4], dsy[4], dsz[2];
        cheb_basis<N, FIELD>(((double)a.tz[k] - cz) * ih, tk, dtk);
        lagrange(grp, sz, dsz);
        cheb_basis<N, FIELD>(((double)a.ty[k] - cy) * ih, tk, dtk);
        lagrange(2 * gb, sy, dsy);
        lagrange(2 * gb + 1, sy + 2, dsy + 2);
        cheb_basis<N, FIELD>(((double)a.tx[k] - cx) * ih, tk, dtk);
        lagrange(2 * ga, sx, dsx);
        lagrange(2 * ga + 1, sx + 2, dsx + 2);
#pragma unroll
        for (int r = 0; r < NRHS; ++r) {
            double o[4] = {0.0, 0.0, 0.0, 0.0};  // potential, then its gradient in t
#pragma unroll
            for (int ii = 0; ii < 4; ++ii) {
                f64x4 c = {0.0, 0.0, 0.0, 0.0}, cd = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < 2; ++s) {
                    c = __builtin_amdgcn_mfma_f64_16x16x4f64(av[r][ii][s], sz[s], c, 0, 0, 0);
                    if (FIELD) cd = __builtin_amdgcn_mfma_f64_16x16x4f64(av[r][ii][s], dsz[s], cd, 0, 0, 0);
                }
                double b = 0.0, by = 0.0, bz = 0.0;
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    b += sy[jj] * c[jj];
                    if (FIELD) {
                        by += dsy[jj] * c[jj];
                        bz += sy[jj] * cd[jj];
                    }
                }
                o[0] += sx[ii] * b;
                if (FIELD) {
                    o[1] += dsx[ii] * b;
                    o[2] += sx[ii] * by;
                    o[3] += sx[ii] * bz;
                }
            }
#pragma unroll
            for (int q = 0; q < (FIELD ? 4 : 1); ++q) {
                o[q] += __shfl_xor(o[q], 16);
                o[q] += __shfl_xor(o[q], 32);
            }
            if (!valid) continue;
            if (grp == 0) {
                if (a.pot) {
                    float *pp = a.pot + r * a.n_trg + dst;
                    *pp = a.accumulate ? (float)((double)*pp + o[0]) : (float)o[0];
                }
            } else if (FIELD && a.field) {
                // field = -grad_x f = -(1/h) grad_t f, one component from each group
                float *f = a.field + ((int64_t)r * a.n_trg + dst) * 3 + (grp - 1);
                const double gr = -ih * (grp == 1 ? o[1] : grp == 2 ? o[2] : o[3]);
                *f = a.accumulate ? (float)((double)*f + gr) : (float)gr;
            }
        }
    }
}

// out (+)= (A_x (x) A_y (x) A_z) in with A_c = S[side_c] (M2M) or its
// transpose (L2L). Lane (q, s) = (lane / N, lane % N): the z pass gives
// T1[p'][q][s] (to LDS), the y pass T2[p'] for the lane's (q, s) in
// registers, the x pass acc[p] for every p.
//
// M2M: one workgroup per (parent, right-hand side), one wave per child: a
// level's few parents are bound by latency, and eight children in sequence in
// one wave were eight times its chain of LDS passes. Waves share nothing until
// the end, where the children's results are added in child order through LDS.
// Measured, one wave per parent -> this: n = 8, 48 to 748 parents 14-19 -> 5-10
// us a level; n = 5, two right-hand sides, 48 to 587 parents 18-20 -> 5-8 us; n =
// 8, three right-hand sides, 8463 parents in three levels 230 -> 214 us.
template <int N, bool L2L>
__global__ __launch_bounds__(L2L ? 64 : 512) void k_cheb_tensor(const double *s1, const int32_t *dst,
                                                               const int32_t *src, const int8_t *oct, int nrhs,
                                                               const float *in, float *out, int n_pad) {
    constexpr int NN = N * N * N, NT = L2L ? 1 : 8;
    __shared__ double sm[2 * N * N];
    __shared__ __align__(16) float Xs[NT][NN];  // the child's values as stored; widened per use
    __shared__ double T1s[NT][NN];
    const int lane = threadIdx.x & 63, item = blockIdx.x, r = blockIdx.y;
    const int t = NT == 1 ? 0 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    float *X = Xs[t];
    double *T1 = T1s[t];
    for (int e = threadIdx.x; e < 2 * N * N; e += 64 * NT) sm[e] = s1[e];
    const bool act = lane < N * N;
    const int q = act ? lane / N : 0, sz = act ? lane % N : 0;
    // A_c[p][p'] from table side: S[side][p][p'] (M2M) or S[side][p'][p] (L2L)
    auto A = [&](int side, int p, int p2) { return L2L ? sm[(side * N + p2) * N + p] : sm[(side * N + p) * N + p2]; };
    const int64_t d = dst[item];
    const int64_t sb = src[(int64_t)item * NT + t];  // uniform across the wave
    const int o = L2L ? oct[item] : t;
    const int sx = (o >> 2) & 1, sy = (o >> 1) & 1, szd = o & 1;
    if (sb >= 0) {
        // all loads first, then the LDS writes, so the loads are in
        // flight together rather than one latency each
        constexpr int NV = (NN + 63) / 64;
        float xv[NV];
#pragma unroll
        for (int i = 0; i < NV; ++i)  // clamped index: no branch per load
            xv[i] = in[(sb * nrhs + r) * n_pad + min(lane + 64 * i, NN - 1)];
#pragma unroll
        for (int i = 0; i < NV; ++i)
            if (lane + 64 * i < NN) X[lane + 64 * i] = xv[i];
    }
    __syncthreads();
    if (act && sb >= 0) {
        // z pass: T1[p'][q][s] = sum_s' A_z[s][s'] X[p'][q][s']
        double az[N];
#pragma unroll
        for (int s2 = 0; s2 < N; ++s2) az[s2] = A(szd, sz, s2);
#pragma unroll
        for (int p2 = 0; p2 < N; ++p2) {
            double v = 0.0;
#pragma unroll
            for (int s2 = 0; s2 < N; ++s2) v += az[s2] * (double)X[(p2 * N + q) * N + s2];
            T1[(p2 * N + q) * N + sz] = v;
        }
    }
    __syncthreads();
    double acc[N];
#pragma unroll
    for (int p = 0; p < N; ++p) acc[p] = 0.0;
    if (act && sb >= 0) {
        // y pass: T2[p'] = sum_q' A_y[q][q'] T1[p'][q'][s]
        double ay[N], t2[N];
#pragma unroll
        for (int q2 = 0; q2 < N; ++q2) ay[q2] = A(sy, q, q2);
#pragma unroll
        for (int p2 = 0; p2 < N; ++p2) {
            double v = 0.0;
#pragma unroll
            for (int q2 = 0; q2 < N; ++q2) v += ay[q2] * T1[(p2 * N + q2) * N + sz];
            t2[p2] = v;
        }
        // x pass: acc[p] += sum_p' A_x[p][p'] T2[p']
#pragma unroll
        for (int p = 0; p < N; ++p) {
            double v = 0.0;
#pragma unroll
            for (int p2 = 0; p2 < N; ++p2) v += A(sx, p, p2) * t2[p2];
            acc[p] = v;
        }
    }
    float *op = out + (d * nrhs + r) * n_pad + lane;  // + p N^2
    if constexpr (L2L) {
        if (!act) return;
#pragma unroll
        for (int p = 0; p < N; ++p) op[p * N * N] = (float)((double)op[p * N * N] + acc[p]);
    } else {
        __syncthreads();  // every wave is done with its T1
        if (act)
#pragma unroll
            for (int p = 0; p < N; ++p) T1[p * N * N + lane] = acc[p];  // zeros for a missing child
        __syncthreads();
        if (act && t < N) {  // wave t adds plane p = t
            double v = 0.0;
#pragma unroll
            for (int c = 0; c < NT; ++c) v += T1s[c][t * N * N + lane];
            op[t * N * N] = (float)v;
        }
    }
}

#define FMM_CHEB_N_SWITCH(N_VAR, CALL)                                   \
    switch (N_VAR) {                                                     \
    case 2: { constexpr int N = 2; CALL; } break;                        \
    case 3: { constexpr int N = 3; CALL; } break;                        \
    case 4: { constexpr int N = 4; CALL; } break;                        \
    case 5: { constexpr int N = 5; CALL; } break;                        \
    case 6: { constexpr int N = 6; CALL; } break;                        \
    case 7: { constexpr int N = 7; CALL; } break;                        \
    case 8: { constexpr int N = 8; CALL; } break;                        \
    default: throw Error(FMM_ERR_ARG, "Chebyshev order must be 2..8");   \
    }

#define FMM_CHEB_SWITCH(N_VAR, NRHS_VAR, CALL)                                      \
    switch ((N_VAR) * 8 + (NRHS_VAR)) {                                             \
    case 2 * 8 + 1: { constexpr int N = 2, R = 1; CALL; } break;                    \
    case 2 * 8 + 2: { constexpr int N = 2, R = 2; CALL; } break;                    \
    case 2 * 8 + 3: { constexpr int N = 2, R = 3; CALL; } break;                    \
    case 2 * 8 + 4: { constexpr int N = 2, R = 4; CALL; } break;                    \
    case 3 * 8 + 1: { constexpr int N = 3, R = 1; CALL; } break;                    \
    case 3 * 8 + 2: { constexpr int N = 3, R = 2; CALL; } break;                    \
    case 3 * 8 + 3: { constexpr int N = 3, R = 3; CALL; } break;                    \
    case 3 * 8 + 4: { constexpr int N = 3, R = 4; CALL; } break;                    \
    case 4 * 8 + 1: { constexpr int N = 4, R = 1; CALL; } break;                    \
    case 4 * 8 + 2: { constexpr int N = 4, R = 2; CALL; } break;                    \
    case 4 * 8 + 3: { constexpr int N = 4, R = 3; CALL; } break;                    \
    case 4 * 8 + 4: { constexpr int N = 4, R = 4; CALL; } break;                    \
    case 5 * 8 + 1: { constexpr int N = 5, R = 1; CALL; } break;                    \
    case 5 * 8 + 2: { constexpr int N = 5, R = 2; CALL; } break;                    \
    case 5 * 8 + 3: { constexpr int N = 5, R = 3; CALL; } break;                    \
    case 5 * 8 + 4: { constexpr int N = 5, R = 4; CALL; } break;                    \
    case 6 * 8 + 1: { constexpr int N = 6, R = 1; CALL; } break;                    \
    case 6 * 8 + 2: { constexpr int N = 6, R = 2; CALL; } break;                    \
    case 6 * 8 + 3: { constexpr int N = 6, R = 3; CALL; } break;                    \
    case 6 * 8 + 4: { constexpr int N = 6, R = 4; CALL; } break;                    \
    case 7 * 8 + 1: { constexpr int N = 7, R = 1; CALL; } break;                    \
    case 7 * 8 + 2: { constexpr int N = 7, R = 2; CALL; } break;                    \
    case 7 * 8 + 3: { constexpr int N = 7, R = 3; CALL; } break;                    \
    case 7 * 8 + 4: { constexpr int N = 7, R = 4; CALL; } break;                    \
    case 8 * 8 + 1: { constexpr int N = 8, R = 1; CALL; } break;                    \
    case 8 * 8 + 2: { constexpr int N = 8, R = 2; CALL; } break;                    \
    case 8 * 8 + 3: { constexpr int N = 8, R = 3; CALL; } break;                    \
    case 8 * 8 + 4: { constexpr int N = 8, R = 4; CALL; } break;                    \
    default: throw Error(FMM_ERR_ARG, "Chebyshev order must be 2..8 and nrhs 1..4"); \
    }

}  // namespace

void points_to_nodes(int nrhs, bool sl, bool dl, int n, const double *coef, const int32_t *items, int nitems,
                     const int32_t *roff, const int32_t *rng, const SurfaceGeom &g, const PointSrc &src, float *out,
                     hipStream_t s) {
    if (nitems <= 0) return;
    FMM_REQUIRE(g.ns == n * n * n && g.n_pad >= g.ns, "points_to_nodes: node count does not match the order");
    const bool four = nitems < 1024;  // fewer leaves than SIMDs
    const dim3 gr(nitems), bl(four ? 256 : 64);
    auto go = [&](auto kern1, auto kern4) {
        hipLaunchKernelGGL((four ? kern4 : kern1), gr, bl, 0, s, coef, items, roff, rng, g, src, out);
    };
    if (sl && dl) {
        FMM_CHEB_SWITCH(n, nrhs, go(k_points_to_nodes<N, R, true, true>, k_points_to_nodes4<N, R, true, true>));
    } else if (dl) {
        FMM_CHEB_SWITCH(n, nrhs, go(k_points_to_nodes<N, R, false, true>, k_points_to_nodes4<N, R, false, true>));
    } else {
        FMM_CHEB_SWITCH(n, nrhs, go(k_points_to_nodes<N, R, true, false>, k_points_to_nodes4<N, R, true, false>));
    }
    FMM_HIP(hipGetLastError());
}

void cheb_tensor(int nrhs, int n, bool l2l, const double *s1, int nitems, const int32_t *dst, const int32_t *src,
                 const int8_t *oct, const float *in, float *out, int n_pad, hipStream_t s) {
    if (nitems <= 0) return;
    FMM_REQUIRE(n_pad >= n * n * n, "cheb_tensor: rows shorter than n^3");
    const dim3 gr(nitems, nrhs);
    if (l2l) {
        FMM_CHEB_N_SWITCH(n, hipLaunchKernelGGL((k_cheb_tensor<N, true>), gr, dim3(64), 0, s, s1, dst, src, oct, nrhs, in,
                                                out, n_pad));
    } else {
        FMM_CHEB_N_SWITCH(n, hipLaunchKernelGGL((k_cheb_tensor<N, false>), gr, dim3(512), 0, s, s1, dst, src, oct, nrhs,
                                                in, out, n_pad));
    }
    FMM_HIP(hipGetLastError());
}

// 8 nodes a side fill the matrix tiles (64 x 8); other orders pad rows or k
template <int N, int R, bool FIELD>
static void launch_nodes_to_points(dim3 gr, dim3 bl, hipStream_t s, const double *coef, const EvalArgs &a,
                                   const SurfaceGeom &g, const float *L) {
    if constexpr (N == 8)
        hipLaunchKernelGGL((k_nodes_to_points8<R, FIELD>), gr, bl, 0, s, coef, a, g, L);
    else
        hipLaunchKernelGGL((k_nodes_to_points<N, R, FIELD>), gr, bl, 0, s, coef, a, g, L);
}

void nodes_to_points(int nrhs, int n, const double *coef, const EvalArgs &a, const SurfaceGeom &g, const float *L,
                     hipStream_t s) {
    if (a.nwork <= 0) return;
    FMM_REQUIRE(g.ns == n * n * n && g.n_pad >= g.ns, "nodes_to_points: node count does not match the order");
    dim3 gr(a.nwork), bl(64);
    if (a.field) {
        FMM_CHEB_SWITCH(n, nrhs, (launch_nodes_to_points<N, R, true>(gr, bl, s, coef, a, g, L)));
    } else {
        FMM_CHEB_SWITCH(n, nrhs, (launch_nodes_to_points<N, R, false>(gr, bl, s, coef, a, g, L)));
    }
    FMM_HIP(hipGetLastError());
}

}  // namespace fmm

// Matrix-free restarted GMRES on the device (gmres_solve in include/fmm.h).
//
// The paper solves its dense boundary-integral systems with GMRES in
// matrix-free form: only the action of A is defined, and the boundary integral
// inside it is the dominant cost (Sec. III, electrostatic problem). Here every
// iteration is one FMM apply plus float64 vector work on the device:
// classical Gram-Schmidt applied twice (CGS2) for the Arnoldi step, the small
// Hessenberg least-squares problem kept triangular by Givens rotations on the
// host, and the true residual recomputed at every restart.
//
// The vector work of a step is four kernels, since on the bodies one solves for
// (10,000 to 100,000 points) it is bound by launches, not by the vectors:
//   k_operator    y = A v from the apply's output, and the block sums of V_k . y
//   k_orthogonal  (twice) h_k from those block sums, y -= sum_k h_k V_k, and the
//                 block sums of the next pass, or of y . y
//   k_normalise   |y|, v = y / |y|, the density of the next apply, and the
//                 step's coefficients to pinned host memory
// Every block adds the block sums itself, in a fixed order (deterministic).
// Against separate kernels for the density, the operator, the dot products,
// their reduction, the subtractions and the normalisation (eleven a step) and a
// copy of the coefficients: a solve of 5 steps on 14,700 points 1190 -> 930 us
// (seven applies of it about 800).
#include <cmath>

#include "plan.hpp"

namespace fmm {

namespace {

constexpr int kBlock = 256;
constexpr int kBigBlock = 1024;
constexpr int kDots = 4;         // dot products accumulated at once
constexpr int kCoefArg = 64;     // update coefficients passed as a kernel argument

// Blocks that share a vector, at most 512, as each of them reads all blocks'
// sums: of 256 threads while that is one element a thread, then of 1024, with
// which more of the vectors is in flight. Per step beyond the apply, blocks of
// 256 and 1024: 196,000 points, 60 vectors 134 and 107 us (separate kernels 128);
// 1M points, 30 vectors 178 and 151 (194), 60 vectors 318 and 255 (269).
int vec_threads(int64_t n) { return n <= 512 * kBlock ? kBlock : kBigBlock; }
int vec_blocks(int64_t n) {
    const int64_t t = vec_threads(n);
    return (int)std::max<int64_t>(1, std::min<int64_t>(n <= 65536 ? 256 : 512, (n + t - 1) / t));
}

__device__ inline double wave_sum(double v) {
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// partial[k * gridDim.x + block] = this block's share of V_k . y, k < nk
// (V NULL: y . y, nk = 1); each thread reads back only elements it wrote.
__device__ inline void block_dots(const double *V, int64_t ldv, int nk, const double *y, int64_t n, double *partial) {
    __shared__ double sh[kBigBlock / 64][kDots];
    const int waves = blockDim.x >> 6;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    for (int k0 = 0; k0 < nk; k0 += kDots) {
        double acc[kDots];
#pragma unroll
        for (int j = 0; j < kDots; ++j) acc[j] = 0.0;
        for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
            const double yi = y[i];
#pragma unroll
            for (int j = 0; j < kDots; ++j)
                acc[j] += (V ? V[(int64_t)min(k0 + j, nk - 1) * ldv + i] : yi) * yi;
        }
#pragma unroll
        for (int j = 0; j < kDots; ++j) acc[j] = wave_sum(acc[j]);
        __syncthreads();
        if (lane == 0)
#pragma unroll
            for (int j = 0; j < kDots; ++j) sh[w][j] = acc[j];
        __syncthreads();
        if (threadIdx.x < kDots && k0 + threadIdx.x < nk) {
            double v = sh[0][threadIdx.x];
            for (int q = 1; q < waves; ++q) v += sh[q][threadIdx.x];
            partial[(int64_t)(k0 + threadIdx.x) * gridDim.x + blockIdx.x] = v;
        }
    }
}

// h[k] (LDS) = sum over the blocks of partial[k], k < nk
__device__ inline void sum_partials(const double *partial, int nk, double *h) {
    const int lane = threadIdx.x & 63;
    for (int k = threadIdx.x >> 6; k < nk; k += (int)(blockDim.x >> 6)) {
        double v = 0.0;
        for (int b = lane; b < (int)gridDim.x; b += 64) v += partial[(int64_t)k * gridDim.x + b];
        v = wave_sum(v);
        if (lane == 0) h[k] = v;
    }
    __syncthreads();
}

__global__ void k_density(const double *x, const float *w, float *dens, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i < n) dens[i] = (float)(x[i] * (double)w[i]);
}

// y = a x + pot                      (FK)
// y = a x + c (field . n)            (dielectric)
// and, with b given, y = b - that (the residual). Block sums: V_k . y for k < nk,
// or (b given) y . y in partial[0] and b . b in partial[1].
__global__ __launch_bounds__(kBigBlock) void k_operator(int kind, const double *x, const float *a, const float *c,
                                                     const float *pot, const float *field, const float *nrm,
                                                     const double *b, double *y, int64_t n, const double *V,
                                                     int64_t ldv, int nk, double *partial) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double v = (double)a[i] * x[i];
        if (kind == FMM_OP_FK) {
            v += (double)pot[i];
        } else {
            double en = (double)field[3 * i] * nrm[3 * i] + (double)field[3 * i + 1] * nrm[3 * i + 1] +
                        (double)field[3 * i + 2] * nrm[3 * i + 2];
            v += (double)c[i] * en;
        }
        y[i] = b ? b[i] - v : v;
    }
    if (b) {
        block_dots(nullptr, 0, 1, y, n, partial);
        block_dots(nullptr, 0, 1, b, n, partial + gridDim.x);
    } else {
        block_dots(V, ldv, nk, y, n, partial);
    }
}

// One Gram-Schmidt pass: h_k = the block sums `in`, w -= sum_k h_k V_k, block
// sums of the new V_k . w (last = 0) or of w . w (last = 1) to `out`; block 0
// keeps the coefficients in hdev.
__global__ __launch_bounds__(kBigBlock) void k_orthogonal(const double *V, int64_t ldv, int nk, const double *in, double *w,
                                                       int64_t n, double *hdev, double *out, int last) {
    extern __shared__ double h[];
    sum_partials(in, nk, h);
    if (blockIdx.x == 0)
        for (int k = threadIdx.x; k < nk; k += blockDim.x) hdev[k] = h[k];
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        double acc = w[i];
        for (int k = 0; k < nk; ++k) acc -= h[k] * V[(int64_t)k * ldv + i];
        w[i] = acc;
    }
    block_dots(last ? nullptr : V, ldv, last ? 1 : nk, w, n, out);
}

// v = w / |w| with |w|^2 the block sums `in`, unless |w| <= floor (Arnoldi
// breakdown: v = w), and dens = v wgt. Block 0 hands the host the coefficients
// of both passes (nk each; h2 after stride doubles) and, from index 2 stride,
// the nsum sums of `in`. w and v may be the same.
__global__ __launch_bounds__(kBigBlock) void k_normalise(const double *w, double *v, const double *in, int nsum,
                                                      double floor, const float *wgt, float *dens, int64_t n,
                                                      const double *hdev, int nk, int stride, double *host) {
    __shared__ double sum[2];
    sum_partials(in, nsum, sum);
    const double nrm = sqrt(sum[0]);
    const bool keep = nrm <= floor;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const double x = keep ? w[i] : w[i] / nrm;
        v[i] = x;
        dens[i] = (float)(x * (double)wgt[i]);
    }
    if (blockIdx.x == 0) {
        for (int k = threadIdx.x; k < nk; k += blockDim.x) {
            host[k] = hdev[k];
            host[stride + k] = hdev[stride + k];
        }
        if (threadIdx.x < (unsigned)nsum) host[2 * stride + threadIdx.x] = sum[threadIdx.x];
    }
}

// x += sum_k y[k] V[k], and dens = x wgt; y by value or (many) from memory
struct Coefs {
    double v[kCoefArg];
};
__global__ __launch_bounds__(kBlock) void k_update(const double *V, int64_t ldv, int nk, Coefs c, const double *y,
                                                   double *x, const float *wgt, float *dens, int64_t n) {
    int64_t i = (int64_t)blockIdx.x * kBlock + threadIdx.x;
    if (i >= n) return;
    double acc = x[i];
    for (int k = 0; k < nk; ++k) acc += (y ? y[k] : c.v[k]) * V[(int64_t)k * ldv + i];
    x[i] = acc;
    dens[i] = (float)(acc * (double)wgt[i]);
}

struct Gmres {
    Plan &P;
    const fmm_operator &op;
    hipStream_t s;
    int64_t n;
    int nb;                          // blocks of the vector kernels
    int kmax;                        // most vectors a Gram-Schmidt pass works on (restart + 1)
    DBuf<float> dens, pot, field;
    DBuf<double> pa, pb;             // [kmax][nb] block sums (two, used in turn)
    DBuf<double> hdev;               // [2 kmax] coefficients of both passes
    double *host;                    // pinned [2 kmax + 2]: the same, and the squared norms

    Gmres(Plan &p, const fmm_operator &o, int restart, hipStream_t st)
        : P(p), op(o), s(st), n(p.t.n_src), nb(vec_blocks(n)), kmax(restart + 1) {
        dens.alloc(n);
        if (op.kind == FMM_OP_FK) pot.alloc(n);
        else field.alloc(3 * n);
        pa.alloc((size_t)nb * std::max(kmax, 2));
        pb.alloc((size_t)nb * std::max(kmax, 2));
        hdev.alloc(2 * (size_t)kmax);
        host = P.solve_host.get(2 * (size_t)kmax + 2);
    }

    // the operator's FMM evaluation of the density in dens
    void apply() {
        // the same buffers every iteration: with graph replay on, one capture per solve
        const float *q = op.kind == FMM_OP_FK ? nullptr : dens.p;
        const float *mu = op.kind == FMM_OP_FK ? dens.p : nullptr;
        float *pt = op.kind == FMM_OP_FK ? pot.p : nullptr;
        float *fd = op.kind == FMM_OP_FK ? nullptr : field.p;
        if (P.graph.enabled && !P.timing)
            plan_apply_graph(P, q, mu, pt, fd, s);
        else
            plan_apply(P, q, mu, pt, fd, s);
    }
    void oper(const double *x, const double *b, double *y, const double *V, int64_t ldv, int nk) {
        apply();
        hipLaunchKernelGGL(k_operator, dim3(nb), dim3(vec_threads(n)), 0, s, op.kind, x, op.a, op.c, pot.p, field.p,
                           P.trg_nrm_user.p, b, y, n, V, ldv, nk, pa.p);
        FMM_HIP(hipGetLastError());
    }
    void normalise(const double *w, double *v, const double *sums, int nsum, double floor, int nk) {
        hipLaunchKernelGGL(k_normalise, dim3(nb), dim3(vec_threads(n)), 0, s, w, v, sums, nsum, floor, op.w, dens.p, n, hdev.p,
                           nk, kmax, host);
        FMM_HIP(hipGetLastError());
        FMM_HIP(hipStreamSynchronize(s));  // the host reads the coefficients
    }

    // r = b - A x (dens holds x w), v = r / |r|, dens = v w; returns |r| and |b|
    void residual(const double *x, const double *b, double *r, double *v, double &rn, double &bn) {
        oper(x, b, r, nullptr, 0, 0);
        normalise(r, v, pa.p, 2, 0.0, 0);
        rn = std::sqrt(host[2 * kmax]);
        bn = std::sqrt(host[2 * kmax + 1]);
    }

    // One Arnoldi step: w = A V[nk - 1] (dens holds its density) orthogonalised
    // against V[0..nk) twice and normalised unless its norm is at most `floor`;
    // one wait brings back both passes' coefficients (summed into h[0..nk)) and
    // the norm.
    double step(const double *V, int64_t ldv, int nk, double *w, double floor, double *h) {
        if (nk > kmax) throw Error(FMM_ERR_ARG, "gmres: more Krylov vectors than the restart length");
        oper(V + (int64_t)(nk - 1) * ldv, nullptr, w, V, ldv, nk);
        const size_t sh = (size_t)nk * sizeof(double);
        hipLaunchKernelGGL(k_orthogonal, dim3(nb), dim3(vec_threads(n)), sh, s, V, ldv, nk, pa.p, w, n, hdev.p, pb.p, 0);
        FMM_HIP(hipGetLastError());
        hipLaunchKernelGGL(k_orthogonal, dim3(nb), dim3(vec_threads(n)), sh, s, V, ldv, nk, pb.p, w, n, hdev.p + kmax, pa.p, 1);
        FMM_HIP(hipGetLastError());
        normalise(w, w, pa.p, 1, floor, nk);
        for (int i = 0; i < nk; ++i) h[i] = host[i] + host[kmax + i];
        return std::sqrt(host[2 * kmax]);
    }
};

}  // namespace

double *PinnedBuf::get(size_t count) {
    if (count > n) {
        release();
        FMM_HIP(hipHostMalloc((void **)&p, count * sizeof(double), hipHostMallocDefault));
        n = count;
    }
    return p;
}
void PinnedBuf::release() {
    if (p) (void)hipHostFree(p);
    p = nullptr;
    n = 0;
}

void plan_gmres(Plan &P, const fmm_operator &op, const double *b, double *x, double rtol, int restart, int max_iter,
                int *iters_out, double *rel_out, int *status, hipStream_t s) {
    Arena mem;  // the call's buffers
    ArenaScope scope(&mem, &mem);
    Gmres G(P, op, restart, s);
    const int64_t n = G.n;
    const int m = restart;
    DBuf<double> V((size_t)(m + 1) * n), r(n), dy(m);
    std::vector<double> H((size_t)(m + 1) * m), cs(m), sn(m), g(m + 1), y(m), h(m + 1);
    int iters = 0;
    *status = FMM_OK;
    hipLaunchKernelGGL(k_density, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, x, op.w, G.dens.p, n);
    FMM_HIP(hipGetLastError());
    double rel = 0.0;
    while (true) {
        double beta, bnorm;
        G.residual(x, b, r.p, V.p, beta, bnorm);
        // (known only after an apply: a wait for |b| before it makes a zero right-hand side
        // cheaper, 14,700 points 157 -> 33 us, and every other solve dearer, 884 -> 945 us)
        if (bnorm == 0.0) {
            FMM_HIP(hipMemsetAsync(x, 0, n * sizeof(double), s));
            break;
        }
        rel = beta / bnorm;
        if (rel <= rtol) break;
        if (iters >= max_iter) {
            *status = FMM_ERR_NOT_CONVERGED;
            break;
        }
        std::fill(g.begin(), g.end(), 0.0);
        g[0] = beta;
        int k = 0;
        const int mm = std::min(m, max_iter - iters);
        const double floor = 1e-14 * beta;
        for (int j = 0; j < mm; ++j) {
            double *vj1 = V.p + (int64_t)(j + 1) * n;
            const double hn = G.step(V.p, n, j + 1, vj1, floor, h.data());
            const bool breakdown = hn <= floor;
            for (int i = 0; i <= j; ++i) H[(size_t)i * m + j] = h[i];
            H[(size_t)(j + 1) * m + j] = hn;
            for (int i = 0; i < j; ++i) {
                double a = H[(size_t)i * m + j], c = H[(size_t)(i + 1) * m + j];
                H[(size_t)i * m + j] = cs[i] * a + sn[i] * c;
                H[(size_t)(i + 1) * m + j] = -sn[i] * a + cs[i] * c;
            }
            double den = std::hypot(H[(size_t)j * m + j], H[(size_t)(j + 1) * m + j]);
            cs[j] = H[(size_t)j * m + j] / den;
            sn[j] = H[(size_t)(j + 1) * m + j] / den;
            H[(size_t)j * m + j] = den;
            H[(size_t)(j + 1) * m + j] = 0.0;
            g[j + 1] = -sn[j] * g[j];
            g[j] = cs[j] * g[j];
            ++iters;
            k = j + 1;
            if (std::fabs(g[j + 1]) / bnorm <= rtol || breakdown) break;
        }
        for (int i = k - 1; i >= 0; --i) {
            double acc = g[i];
            for (int l = i + 1; l < k; ++l) acc -= H[(size_t)i * m + l] * y[l];
            y[i] = acc / H[(size_t)i * m + i];
        }
        Coefs c;
        const bool by_value = k <= kCoefArg;
        if (by_value)
            std::copy(y.begin(), y.begin() + k, c.v);
        else
            h2d(dy.p, y.data(), k, s);
        hipLaunchKernelGGL(k_update, dim3(grid_for(n, kBlock)), dim3(kBlock), 0, s, V.p, n, k, c, by_value ? nullptr : dy.p,
                           x, op.w, G.dens.p, n);
        FMM_HIP(hipGetLastError());
    }
    FMM_HIP(hipStreamSynchronize(s));
    *iters_out = iters;
    *rel_out = rel;
}

}  // namespace fmm

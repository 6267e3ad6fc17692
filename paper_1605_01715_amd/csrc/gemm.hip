// Batched box GEMMs in float64 on the CDNA4 matrix cores, a float32 MFMA GEMM
// for the Chebyshev basis changes (below, k_gemm_f32), and float64 helpers
// for the operator precompute.
//
// The upward and downward passes apply small dense matrices to per-box
// vectors: M2M (8 octant matrices), L2L (8 octant matrices), the projections
// of point-generated check potentials onto the compressed basis and the
// check-to-equivalent expansions. They are cheap next to M2L and they feed
// every M2L, so they run in float64 (v_mfma_f64_16x16x4_f64) on float32 data.
// The kernel is target-stationary: 1, 2, 4 or 8 waves own 16 rows of a tile of
// 32 output vectors, keep their accumulators in registers across all terms
// and write each output once.
//
// Bound: at the sizes of one tree level, latency. Most levels have fewer
// tiles than the chip has CUs, and a parent's eight child terms are one chain
// of 8 K / 16 steps of eight float64 MFMAs (64 cycles each). So the (term, k)
// steps of an output block are shared by `split` waves, whose partial sums are
// added in LDS in a fixed order; with eight, an M2M wave runs one child.
// Matrices are stored in fragment order and both operands go straight from
// global memory to registers (lane group g of a fragment holds k = 4 g + s for
// MFMA s, the same on both sides, so that a lane's four k of a vector are one
// 16-byte load), the next step's loads under the current step's MFMAs: no
// barrier before the final sum. Against staging the vectors in LDS for four
// row blocks and running the terms in sequence: M2M of 200 to 600 boxes at K =
// 224 87-104 -> 13-23 us, L2L of the same 15-19 -> 8 us, projections of 4274
// boxes 28 -> 22 us; the surface form's apply on eight spheres (196,000 points)
// 1092 -> 754 us and on a 4M cloud (order 8) 9.07 -> 8.80 ms.
#include "gemm.hpp"

#include "bf16.hpp"

#include <algorithm>

namespace fmm {

namespace {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kMaxK = 512;
constexpr int kGemmWaves = 8;  // per workgroup: 8 / split row blocks of one tile

// D: steps whose loads are in flight
template <int D>
__global__ __launch_bounds__(64 * kGemmWaves) void k_gemm_f64(GemmLaunch a, int split) {
    __shared__ double red[kGemmWaves][8][64];  // partial sums: [wave][column block, element][lane]
    const int lane = threadIdx.x & 63, c16 = lane & 15, g = lane >> 4;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int part = w % split;
    const int nrb = a.m_pad / 16, nkc = a.k_pad / 16;
    const int rb = (int)blockIdx.y * (kGemmWaves / split) + w / split;  // wave-uniform
    const bool live = rb < nrb;
    const int64_t tile = blockIdx.x;
    f64x4 acc[2];
    acc[0] = acc[1] = f64x4{0.0, 0.0, 0.0, 0.0};
    if (live) {
        // this wave's steps [s0, s1) of the tile's nterm * nkc, term by term
        const int total = a.nterm * nkc;
        const int s0 = total * part / split, s1 = total * (part + 1) / split;
        const int32_t *ts = a.term_src + (size_t)tile * a.nterm * kGemmCols + c16;
        struct Frag {
            double a[4];
            float4 b[2];
        };
        Frag f[D];
        int term = s0 / nkc;
        int32_t n0 = 0, n1 = 0;  // the next term's sources of the lane's two columns
        if (s0 < s1) {
            n0 = ts[term * kGemmCols];
            n1 = ts[term * kGemmCols + 16];
        }
        for (int at = s0; at < s1; ++term) {
            const int k0 = at - term * nkc, k1 = min(nkc, s1 - term * nkc);
            at += k1 - k0;
            const int32_t v0 = n0, v1 = n1;
            if (at < s1) {
                n0 = ts[(term + 1) * kGemmCols];
                n1 = ts[(term + 1) * kGemmCols + 16];
            }
            if (__ballot(v0 >= 0 || v1 >= 0) == 0) continue;  // no column has a source
            const int mat = a.term_mat ? a.term_mat[(size_t)tile * a.nterm + term] : term;
            const double *ap = a.mats + (size_t)mat * a.mat_elems + ((size_t)rb * nkc * 64 + lane) * 4;
            const float4 *b0 = (const float4 *)(a.in + (size_t)max(v0, 0) * a.k_pad) + g;
            const float4 *b1 = (const float4 *)(a.in + (size_t)max(v1, 0) * a.k_pad) + g;
            auto load = [&](Frag &x, int kc) {
                kc = min(kc, k1 - 1);  // past the term's end its last step again: no branch around the loads
                const double *q = ap + (size_t)kc * 256;
#pragma unroll
                for (int s = 0; s < 4; ++s) x.a[s] = q[s];
                x.b[0] = b0[4 * kc];
                x.b[1] = b1[4 * kc];
            };
            auto mma = [&](const Frag &x) {
#pragma unroll
                for (int s = 0; s < 4; ++s)
#pragma unroll
                    for (int cb = 0; cb < 2; ++cb) {
                        const float4 v = x.b[cb];
                        const float e = s == 0 ? v.x : s == 1 ? v.y : s == 2 ? v.z : v.w;
                        const double bv = (double)((cb ? v1 : v0) < 0 ? 0.f : e);
                        acc[cb] = __builtin_amdgcn_mfma_f64_16x16x4f64(x.a[s], bv, acc[cb], 0, 0, 0);
                    }
            };
#pragma unroll
            for (int d = 0; d < D - 1; ++d) load(f[d], k0 + d);
            for (int kc = k0; kc < k1; kc += D) {
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    load(f[(d + D - 1) % D], kc + d + D - 1);
                    if (kc + d < k1) mma(f[d]);
                }
            }
        }
    }
    const int j0 = part * (8 / split);  // of the block's 8 elements per lane, this wave writes 8 / split
    if (split > 1) {
#pragma unroll
        for (int j = 0; j < 8; ++j) red[w][j][lane] = acc[j >> 2][j & 3];
        __syncthreads();
    }
    if (!live) return;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if (j < j0 || j >= j0 + 8 / split) continue;
        const int o = a.tile_cols[tile * kGemmCols + 16 * (j >> 2) + c16];
        if (o < 0) continue;
        double sum = split > 1 ? red[w - part][j][lane] : acc[j >> 2][j & 3];
        for (int p = 1; p < split; ++p) sum += red[w - part + p][j][lane];
        const double sc = a.col_scale ? a.col_scale[o] : 1.0;
        // f64 16x16 accumulator: element v of lane l is row l / 16 + 4 v
        float *op = a.out + (size_t)o * a.m_pad + rb * 16 + g + 4 * (j & 3);
        const float r = (float)(sum * sc);
        *op = a.accumulate ? *op + r : r;
    }
}

__global__ void k_frag_f64(const double *M, int rows, int cols, int m_pad, int k_pad, double *out) {
    int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)m_pad * k_pad) return;
    const int nkc = k_pad / 16;
    int s = (int)(idx % 4);
    int64_t r = idx / 4;
    int lane = (int)(r % 64);
    r /= 64;
    int kc = (int)(r % nkc);
    int rb = (int)(r / nkc);
    int row = rb * 16 + (lane & 15), k = kc * 16 + 4 * (lane >> 4) + s;
    out[idx] = (row < rows && k < cols) ? M[(int64_t)row * cols + k] : 0.0;
}

__global__ void k_padded_f32(const double *M, int rows, int cols, int m_pad, int k_pad, float *out) {
    int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)m_pad * k_pad) return;
    int row = (int)(idx / k_pad), k = (int)(idx % k_pad);
    out[idx] = (row < rows && k < cols) ? (float)M[(int64_t)row * cols + k] : 0.f;
}

__global__ void k_laplace_mats(const double *Y, int n, int nb, const double *prm, double *G) {
    int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    int64_t per = (int64_t)n * n;
    if (idx >= per * nb) return;
    int b = (int)(idx / per);
    int i = (int)((idx % per) / n), j = (int)(idx % n);
    const double *p = prm + 9 * b;
    double d2 = 0.0;
    for (int c = 0; c < 3; ++c) {
        double x = p[c] + p[3] * Y[3 * i + c];
        double y = p[4 + c] + p[7] * Y[3 * j + c];
        d2 += (x - y) * (x - y);
    }
    G[idx] = p[8] / (kFourPi * sqrt(d2));
}

__global__ __launch_bounds__(256) void k_dgemm(const double *A, size_t sa, const double *B, size_t sb, double *C,
                                              size_t sc, int M, int N, int K) {
    __shared__ double As[16][17], Bsh[16][17];
    const int b = blockIdx.z;
    const int tx = threadIdx.x & 15, ty = threadIdx.x >> 4;
    const int row = blockIdx.y * 16 + ty, col = blockIdx.x * 16 + tx;
    const double *Ab = A + (size_t)b * sa;
    const double *Bb = B + (size_t)b * sb;
    double acc = 0.0;
    for (int k0 = 0; k0 < K; k0 += 16) {
        As[ty][tx] = (row < M && k0 + tx < K) ? Ab[(size_t)row * K + k0 + tx] : 0.0;
        Bsh[ty][tx] = (k0 + ty < K && col < N) ? Bb[(size_t)(k0 + ty) * N + col] : 0.0;
        __syncthreads();
        for (int k = 0; k < 16; ++k) acc += As[ty][k] * Bsh[k][tx];
        __syncthreads();
    }
    if (row < M && col < N) C[(size_t)b * sc + (size_t)row * N + col] = acc;
}

// One matrix for every column, float32 on the matrix cores
// (v_mfma_f32_32x32x2f32, float32 accumulation): the Chebyshev form's
// compression into the M2L basis and expansion out of it, the two largest
// box GEMMs (every box, 512 x r). One workgroup per tile of 32 columns, so
// the tile's source vectors are read from memory once: they are staged in
// LDS 128 k at a time with coalesced loads (rows of k_pad floats) and shared
// by the waves. Wave w owns the 32-row blocks w, w + NW (MAXRB of them) and
// reads its matrix fragments from global memory in fragment order (every
// load instruction reads 1 KB contiguous), the next chunk's while the
// current chunk's MFMAs run. Lane l supplies row (or column) l % 32 at
// k = 16 (l / 32) + q for MFMA q, so MFMA q contracts k = q and 16 + q of a
// 32-k chunk (a permutation of the k order, the same on both operands).
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kF32Slice = 128;            // k staged per slice
constexpr int kF32BStr = kF32Slice + 4;   // floats per column in LDS

// The four rows k = row .. row + 3 (a multiple of 4) of vector o, split into
// np parts: the M2L's input straight from the basis change, without a float32
// copy of it in between.
__device__ inline void store_split(uint16_t *out_bf, int np, int m_pad, int o, int row, float4 r) {
    typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
    const float v[4] = {r.x, r.y, r.z, r.w};
    u16x4 h, m, l;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        uint16_t a, b, c;
        split3(v[e], a, b, c);
        h[e] = a;
        m[e] = b;
        l[e] = c;
    }
    uint16_t *p = out_bf + o * vec_bf_stride(m_pad, np) + (row / 32) * np * 32 + row % 32;
    *(u16x4 *)p = h;
    *(u16x4 *)(p + 32) = m;
    if (np == 3) *(u16x4 *)(p + 64) = l;
}

template <int MAXRB>
__global__ __launch_bounds__(512) void k_gemm_f32(int m_pad, int k_pad, const int32_t *tile_cols, const float *Mf,
                                                  const float *in, float *out, const double *col_scale,
                                                  int accumulate, const int8_t *add_col, uint16_t *out_bf, int np) {
    __shared__ __align__(16) float Bs[kGemmCols * kF32BStr];
    __shared__ int32_t cols[kGemmCols];
    const int t = threadIdx.x, lane = t & 63, c = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int nt = blockDim.x, nw = nt >> 6, nrb = m_pad / 32, nkc = k_pad / 32;
    const int64_t tile = blockIdx.x;
    if (t < kGemmCols) cols[t] = tile_cols[tile * kGemmCols + t];
    const float4 *ap[MAXRB];
    bool live[MAXRB];
#pragma unroll
    for (int i = 0; i < MAXRB; ++i) {
        const int rb = w + nw * i;
        live[i] = rb < nrb;  // wave-uniform
        ap[i] = (const float4 *)Mf + (size_t)min(rb, nrb - 1) * nkc * 256 + lane;
    }
    float4 a[2][MAXRB][4];
    auto load_a = [&](int buf, int kc) {
#pragma unroll
        for (int i = 0; i < MAXRB; ++i)
            if (live[i])
#pragma unroll
                for (int f = 0; f < 4; ++f) a[buf][i][f] = ap[i][(size_t)kc * 256 + 64 * f];
    };
    f32x16 acc[MAXRB];
#pragma unroll
    for (int i = 0; i < MAXRB; ++i)
        for (int v = 0; v < 16; ++v) acc[i][v] = 0.f;
    auto mma = [&](int buf, int kl) {  // kl: chunk offset inside the staged slice
        float4 b[4];
#pragma unroll
        for (int f = 0; f < 4; ++f) b[f] = *(const float4 *)&Bs[c * kF32BStr + kl + 16 * h + 4 * f];
#pragma unroll
        for (int i = 0; i < MAXRB; ++i) {
            if (!live[i]) continue;
#pragma unroll
            for (int f = 0; f < 4; ++f) {
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[buf][i][f].x, b[f].x, acc[i], 0, 0, 0);
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[buf][i][f].y, b[f].y, acc[i], 0, 0, 0);
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[buf][i][f].z, b[f].z, acc[i], 0, 0, 0);
                acc[i] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[buf][i][f].w, b[f].w, acc[i], 0, 0, 0);
            }
        }
    };
    load_a(0, 0);
    for (int k0 = 0; k0 < k_pad; k0 += kF32Slice) {
        const int kn = min(kF32Slice, k_pad - k0), kq = kn / 4;  // kn: a multiple of 32
        __syncthreads();  // cols; every wave is done with the previous slice
        for (int idx = t; idx < kGemmCols * kq; idx += nt) {
            const int col = idx / kq, k4 = (idx % kq) * 4;
            const int o = cols[col];
            *(float4 *)&Bs[col * kF32BStr + k4] =
                o >= 0 ? *(const float4 *)(in + (size_t)o * k_pad + k0 + k4) : make_float4(0.f, 0.f, 0.f, 0.f);
        }
        __syncthreads();
        const int c0 = k0 / 32, c1 = c0 + kn / 32;
        for (int kc = c0; kc < c1; kc += 2) {
            if (kc + 1 < nkc) load_a(1, kc + 1);
            mma(0, (kc - c0) * 32);
            if (kc + 1 < c1) {
                if (kc + 2 < nkc) load_a(0, kc + 2);
                mma(1, (kc + 1 - c0) * 32);
            }
        }
    }
    const int o = cols[c];
    if (o < 0) return;
    const float sc = col_scale ? (float)col_scale[o] : 1.f;
    const bool add = accumulate || (add_col && add_col[o]);
#pragma unroll
    for (int i = 0; i < MAXRB; ++i) {
        if (!live[i]) continue;
        // 32x32 accumulator: element v of lane l is row 8 (v / 4) + 4 (l / 32) + v % 4, column l % 32
        float *op = out + (size_t)o * m_pad + (w + nw * i) * 32 + 4 * h;
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
            float4 r = make_float4(acc[i][4 * v4] * sc, acc[i][4 * v4 + 1] * sc, acc[i][4 * v4 + 2] * sc,
                                   acc[i][4 * v4 + 3] * sc);
            if (out_bf) {
                store_split(out_bf, np, m_pad, o, (w + nw * i) * 32 + 4 * h + 8 * v4, r);
                continue;
            }
            float4 *dst = (float4 *)(op + 8 * v4);
            if (add) {
                const float4 old = *dst;
                r.x += old.x;
                r.y += old.y;
                r.z += old.z;
                r.w += old.w;
            }
            *dst = r;
        }
    }
}

// The same product where there are too few tiles to fill the chip (a body of
// 14,700 points has nine): the workgroups above are then bound by the latency
// of one chain of k chunks, staging and barriers. Here a workgroup of eight
// waves computes 8 / split blocks of 32 rows by 32 columns, the `split` waves
// of a block share its k chunks, read both operands in fragment order straight
// from global memory and add their partial sums in LDS in a fixed order.
// Measured (tiles, rows x K), against one workgroup per tile: 9, 192 x 512 26 ->
// 6 us; 9, 512 x 192 20 -> 5.5 us; 261, 192 x 512 38 -> 25 us; 382, 160 x 512 37 ->
// 31 us.
constexpr int kF32Waves = 8;
__global__ __launch_bounds__(64 * kF32Waves) void k_gemm_f32_split(int m_pad, int k_pad, const int32_t *tile_cols,
                                                                  const float *Mf, const float *in, float *out,
                                                                  const double *col_scale, int accumulate,
                                                                  const int8_t *add_col, uint16_t *out_bf, int np,
                                                                  int split) {
    __shared__ __align__(16) float4 red[kF32Waves][4][64];  // [wave][4 accumulator values][lane]
    const int lane = threadIdx.x & 63, c = lane & 31, h = lane >> 5;
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), part = w % split;
    const int nrb = m_pad / 32, nkc = k_pad / 32;
    const int rb = (int)blockIdx.y * (kF32Waves / split) + w / split;  // wave-uniform
    const int o = tile_cols[(size_t)blockIdx.x * kGemmCols + c];
    f32x16 acc;
#pragma unroll
    for (int v = 0; v < 16; ++v) acc[v] = 0.f;
    if (rb < nrb) {
        const int k0 = nkc * part / split, k1 = nkc * (part + 1) / split;
        const float4 *ap = (const float4 *)Mf + (size_t)rb * nkc * 256 + lane;
        const float4 *bp = (const float4 *)(in + (size_t)max(o, 0) * k_pad + 16 * h);
        struct Frag {
            float4 a[4], b[4];
        } f[2];
        auto load = [&](Frag &x, int kc) {
            kc = min(kc, k1 - 1);  // past the end the last chunk again: no branch around the loads
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                x.a[i] = ap[(size_t)kc * 256 + 64 * i];
                x.b[i] = bp[8 * kc + i];
            }
        };
        auto mma = [&](const Frag &x) {
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                float4 b = x.b[i];
                if (o < 0) b = make_float4(0.f, 0.f, 0.f, 0.f);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.a[i].x, b.x, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.a[i].y, b.y, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.a[i].z, b.z, acc, 0, 0, 0);
                acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x.a[i].w, b.w, acc, 0, 0, 0);
            }
        };
        if (k0 < k1) {
            load(f[0], k0);
            for (int kc = k0; kc < k1; kc += 2) {
                load(f[1], kc + 1);
                mma(f[0]);
                load(f[0], kc + 2);
                if (kc + 1 < k1) mma(f[1]);
            }
        }
    }
    if (split > 1) {
#pragma unroll
        for (int j = 0; j < 4; ++j)
            red[w][j][lane] = make_float4(acc[4 * j], acc[4 * j + 1], acc[4 * j + 2], acc[4 * j + 3]);
        __syncthreads();
    }
    if (rb >= nrb || o < 0) return;
    const float sc = col_scale ? (float)col_scale[o] : 1.f;
    const bool add = accumulate || (add_col && add_col[o]);
    // element 4 j + e of lane l is row 8 j + 4 (l / 32) + e; the waves of a block write its j in turn
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        if (j % split != part % 4 || (split == 8 && part >= 4)) continue;
        float4 r = split > 1 ? red[w - part][j][lane] : make_float4(acc[4 * j], acc[4 * j + 1], acc[4 * j + 2], acc[4 * j + 3]);
        for (int p = 1; p < split; ++p) {
            const float4 x = red[w - part + p][j][lane];
            r.x += x.x;
            r.y += x.y;
            r.z += x.z;
            r.w += x.w;
        }
        float4 *dst = (float4 *)(out + (size_t)o * m_pad + 32 * rb + 8 * j + 4 * h);
        r.x *= sc;
        r.y *= sc;
        r.z *= sc;
        r.w *= sc;
        if (out_bf) {
            store_split(out_bf, np, m_pad, o, 32 * rb + 8 * j + 4 * h, r);
            continue;
        }
        if (add) {
            const float4 old = *dst;
            r.x += old.x;
            r.y += old.y;
            r.z += old.z;
            r.w += old.w;
        }
        *dst = r;
    }
}

// float64 row-major [rows][cols] -> the float32 fragment order of k_gemm_f32:
// out[((rb * nkc + kc) * 4 + f) * 256 + 4 lane + e] = M[32 rb + lane % 32][32 kc + 16 (lane / 32) + 4 f + e]
__global__ void k_frag_f32(const double *M, int rows, int cols, int m_pad, int k_pad, float *out) {
    int64_t idx = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (idx >= (int64_t)m_pad * k_pad) return;
    const int nkc = k_pad / 32;
    const int e = (int)(idx % 4), lane = (int)((idx / 4) % 64), f = (int)((idx / 256) % 4);
    const int64_t q = idx / 1024;
    const int kc = (int)(q % nkc), rb = (int)(q / nkc);
    const int row = rb * 32 + (lane & 31), k = kc * 32 + 16 * (lane >> 5) + 4 * f + e;
    out[idx] = (row < rows && k < cols) ? (float)M[(int64_t)row * cols + k] : 0.f;
}

}  // namespace

void box_gemm_f64(const GemmLaunch &a, hipStream_t s) {
    if (a.ntile <= 0 || a.nterm <= 0) return;
    FMM_REQUIRE(a.m_pad % 16 == 0 && a.k_pad % 16 == 0 && a.m_pad <= 512 && a.k_pad <= kMaxK,
                "box_gemm: unsupported size");
    // waves per output block: enough for two on each of the 1024 SIMDs
    const int nrb = a.m_pad / 16;
    int split = 1;
    while (split < kGemmWaves && (int64_t)a.ntile * nrb * split < 2048) split *= 2;
    const int per = kGemmWaves / split;  // row blocks per workgroup
    const dim3 g((unsigned)a.ntile, (unsigned)((nrb + per - 1) / per)), b(64 * kGemmWaves);
    // A child term of 12 steps or more (K >= 192) hides more of its loads'
    // latency with four steps in flight (K = 224, few tiles: 21 -> 14 us);
    // shorter runs only load what they do not use (K = 224 in two steps a
    // wave: 7.7 -> 9.1 us)
    if (a.nterm > 1 && a.k_pad >= 192)
        hipLaunchKernelGGL(k_gemm_f64<4>, g, b, 0, s, a, split);
    else
        hipLaunchKernelGGL(k_gemm_f64<2>, g, b, 0, s, a, split);
    FMM_HIP(hipGetLastError());
}

void dense_gemm_f32(int m_pad, int k_pad, int ntile, const int32_t *tile_cols, const float *M, const float *in,
                    float *out, const double *col_scale, int accumulate, hipStream_t s, const int8_t *add_col,
                    uint16_t *out_bf, int np) {
    if (ntile <= 0) return;
    FMM_REQUIRE(m_pad > 0 && k_pad > 0 && m_pad % 32 == 0 && k_pad % 32 == 0 && m_pad <= 512,
                "dense_gemm_f32: unsupported size");
    FMM_REQUIRE(!out_bf || np == 2 || np == 3, "dense_gemm_f32: 2 or 3 bfloat16 parts");
    const int nrb = m_pad / 32, nw = std::min(nrb, 8);  // waves per workgroup; each owns ceil(nrb / nw) row blocks
    // Few tiles: k chunks shared by enough waves for two on each SIMD. Short
    // products (fewer than 8 chunks) gain only with very few tiles (257 tiles,
    // 96 x 128: 7.0 us in one workgroup a tile, 9.1-11 us split).
    int split = 1;
    if (k_pad >= 256 || ntile <= 64)
        while (split < kF32Waves && (int64_t)ntile * nrb * split < 2048) split *= 2;
    if (split > 1) {
        const int per = kF32Waves / split;
        hipLaunchKernelGGL(k_gemm_f32_split, dim3((unsigned)ntile, (unsigned)((nrb + per - 1) / per)),
                           dim3(64 * kF32Waves), 0, s, m_pad, k_pad, tile_cols, M, in, out, col_scale, accumulate, add_col,
                           out_bf, np, split);
        FMM_HIP(hipGetLastError());
        return;
    }
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, dim3((unsigned)ntile), dim3(64 * nw), 0, s, m_pad, k_pad, tile_cols, M, in, out,
                           col_scale, accumulate, add_col, out_bf, np);
    };
    if (nrb <= 8)
        go(k_gemm_f32<1>);
    else
        go(k_gemm_f32<2>);
    FMM_HIP(hipGetLastError());
}

void to_frag_f32(const double *M, int rows, int cols, int m_pad, int k_pad, float *out, hipStream_t s) {
    FMM_REQUIRE(m_pad % 32 == 0 && k_pad % 32 == 0, "to_frag_f32: sizes must be multiples of 32");
    int64_t total = (int64_t)m_pad * k_pad;
    hipLaunchKernelGGL(k_frag_f32, dim3(grid_for(total, 256)), dim3(256), 0, s, M, rows, cols, m_pad, k_pad, out);
    FMM_HIP(hipGetLastError());
}

void to_frag_f64(const double *M, int rows, int cols, int m_pad, int k_pad, double *out, hipStream_t s) {
    int64_t total = (int64_t)m_pad * k_pad;
    hipLaunchKernelGGL(k_frag_f64, dim3(grid_for(total, 256)), dim3(256), 0, s, M, rows, cols, m_pad, k_pad, out);
    FMM_HIP(hipGetLastError());
}

void to_padded_f32(const double *M, int rows, int cols, int m_pad, int k_pad, float *out, hipStream_t s) {
    int64_t total = (int64_t)m_pad * k_pad;
    hipLaunchKernelGGL(k_padded_f32, dim3(grid_for(total, 256)), dim3(256), 0, s, M, rows, cols, m_pad, k_pad,
                       out);
    FMM_HIP(hipGetLastError());
}

void build_laplace_mats(const double *Y, int n, int nb, const double *params, double *G, hipStream_t s) {
    int64_t total = (int64_t)n * n * nb;
    hipLaunchKernelGGL(k_laplace_mats, dim3(grid_for(total, 256)), dim3(256), 0, s, Y, n, nb, params, G);
    FMM_HIP(hipGetLastError());
}

void dgemm_batched(const double *A, size_t sa, const double *B, size_t sb, double *C, size_t sc, int M, int N,
                   int K, int nb, hipStream_t s) {
    dim3 g((N + 15) / 16, (M + 15) / 16, nb);
    hipLaunchKernelGGL(k_dgemm, g, dim3(256), 0, s, A, sa, B, sb, C, sc, M, N, K);
    FMM_HIP(hipGetLastError());
}

}  // namespace fmm

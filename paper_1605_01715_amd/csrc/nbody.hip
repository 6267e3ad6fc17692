// n-body shaped kernels of the FMM: P2M, P2L, L2P, M2P, P2P and the
// all-pairs direct sum.
//
// The kernels are the Laplace single layer q / (4 pi r), the double layer
// m . (x - y) / (4 pi r^3) with m = mu n_y (the normal derivative applied at
// the source side, Sec. III.A.1 Eq. p2m), and the field q (x - y) / (4 pi r^3)
// (Sec. III.A.2 Eq. kernel_pol). Pairs closer than the tolerance radius are
// excluded in the near field (Sec. III.A.1).
//
// One wave (64 lanes) handles one box. Sources are staged in LDS, 64 at a
// time, and every lane reads them by broadcast. Surface points and the
// sources seen from a box surface are expressed relative to the box centre in
// float64 before rounding to float32, so the rounding error of a coordinate
// is relative to the box size, not to the distance from the origin. The
// near field uses the float32 input coordinates directly (x - y of two close
// float32 values is exact). Per-target sums are accumulated per LDS tile in
// float32 and folded into a (hi, lo) pair with Knuth's TwoSum.
#include <algorithm>
#include <limits>
#include <type_traits>

#include "nbody.hpp"

namespace fmm {

namespace {

constexpr float kInv4Pi = 0.079577471545947667884f;

__device__ inline float rsq(float x) { return __builtin_amdgcn_rsqf(x); }

__device__ inline void two_sum_into(float &hi, float &lo, float p) {
    float s = hi + p;
    float bb = s - hi;
    float err = (hi - (s - bb)) + (p - bb);
    hi = s;
    lo += err;
}

// ------------------------------------------------------------ P2M / P2L

// q / r + (m . d) / r^3 = (q + (m . d) / r^2) / r for one (surface point,
// source) pair; v holds the source's offset from the box centre, then its
// strengths. Check points lie outside every box that feeds them (P2M: radius
// 2.95 around the sources' own box; P2L: X-list boxes are a box width away),
// so r > 0; the floor only keeps a degenerate input finite.
template <int NRHS, bool SL, bool DL>
__device__ inline void pair_terms(float x, float y, float z, const float *v, float *t) {
    const float dx = x - v[0], dy = y - v[1], dz = z - v[2];
    const float r2 = dx * dx + dy * dy + dz * dz;
    const float inv = rsq(fmaxf(r2, 1e-30f));
    const float inv2 = inv * inv;
#pragma unroll
    for (int r = 0; r < NRHS; ++r) {
        float u = SL ? v[3 + r] : 0.f;
        if (DL) {
            const int o = 3 + (SL ? NRHS : 0) + 3 * r;
            u += (v[o] * dx + v[o + 1] * dy + v[o + 2] * dz) * inv2;
        }
        t[r] = u * inv;
    }
}

template <int NRHS, bool SL, bool DL>
__global__ __launch_bounds__(64) void k_points_to_surface(const int32_t *items, const int32_t *roff,
                                                         const int32_t *rng, double rfac, SurfaceGeom g,
                                                         PointSrc src, float *out, int accumulate) {
    constexpr int TPL = 8;        // surface points per lane (n_s <= 512)
    constexpr int W = 3 + (SL ? NRHS : 0) + (DL ? 3 * NRHS : 0);
    __shared__ float sh[64 * W];
    const int lane = threadIdx.x;
    const int b = items[blockIdx.x];
    const double cx = g.centre[3 * b], cy = g.centre[3 * b + 1], cz = g.centre[3 * b + 2];
    const double rr = rfac * g.half[b];
    float xm[TPL], ym[TPL], zm[TPL];
    // float64 sums (of float32 sums of two pairs): check potentials feed every translation
    double acc[TPL][NRHS];
    for (int i = 0; i < TPL; ++i) {
        int m = lane + 64 * i;
        bool ok = m < g.ns;
        xm[i] = ok ? (float)(rr * g.Y[3 * m]) : 0.f;
        ym[i] = ok ? (float)(rr * g.Y[3 * m + 1]) : 0.f;
        zm[i] = ok ? (float)(rr * g.Y[3 * m + 2]) : 0.f;
        for (int r = 0; r < NRHS; ++r) acc[i][r] = 0.0;
    }
    const int ntpl = (g.ns + 63) / 64;
    for (int e = roff[blockIdx.x]; e < roff[blockIdx.x + 1]; ++e) {
        const int s0 = rng[2 * e], s1 = rng[2 * e + 1];
        for (int j0 = s0; j0 < s1; j0 += 64) {
            const int j = j0 + lane;
            const int cnt = min(64, s1 - j0);
            {
                // lanes past the range stage a zero-strength source at the box centre (r > 0 from
                // every check point), so the pair loop below can run over an even count
                float *p = sh + lane * W;
#pragma unroll
                for (int k = 0; k < W; ++k) p[k] = 0.f;
                if (j < s1) {
                    p[0] = (float)((double)src.x[j] - cx);
                    p[1] = (float)((double)src.y[j] - cy);
                    p[2] = (float)((double)src.z[j] - cz);
                    int o = 3;
                    if (SL)
                        for (int r = 0; r < NRHS; ++r) p[o++] = src.q[r * src.n + j];
                    if (DL)
                        for (int r = 0; r < NRHS; ++r) {
                            p[o++] = src.mx[r * src.n + j];
                            p[o++] = src.my[r * src.n + j];
                            p[o++] = src.mz[r * src.n + j];
                        }
                }
            }
            __syncthreads();
            for (int jj = 0; jj < cnt; jj += 2) {
                // two sources per step, read into registers once for all surface points
                float v0[W], v1[W];
#pragma unroll
                for (int k = 0; k < W; ++k) {
                    v0[k] = sh[jj * W + k];
                    v1[k] = sh[(jj + 1) * W + k];
                }
#pragma unroll
                for (int i = 0; i < TPL; ++i) {
                    if (i >= ntpl) continue;  // static index keeps acc in registers
                    float t0[NRHS], t1[NRHS];
                    pair_terms<NRHS, SL, DL>(xm[i], ym[i], zm[i], v0, t0);
                    pair_terms<NRHS, SL, DL>(xm[i], ym[i], zm[i], v1, t1);
#pragma unroll
                    for (int r = 0; r < NRHS; ++r) acc[i][r] += (double)(t0[r] + t1[r]);
                }
            }
            __syncthreads();
        }
    }
    // The padding is written too (zero): the projection reads whole rows, and the
    // surface form's downward expansion writes the same rows' padding, which is
    // NaN after an apply of densities that are not finite.
#pragma unroll
    for (int i = 0; i < TPL; ++i) {
        int m = lane + 64 * i;
        if (m >= (accumulate ? g.ns : g.n_pad)) continue;
        for (int r = 0; r < NRHS; ++r) {
            float *op = out + ((int64_t)b * NRHS + r) * g.n_pad + m;
            double v = m < g.ns ? acc[i][r] * (1.0 / kFourPi) : 0.0;
            *op = accumulate ? (float)((double)*op + v) : (float)v;
        }
    }
}

// ------------------------------------------------------------ leaf evaluation
//
// One workgroup per work item (up to 64 targets of a leaf), of one wave or
// of 2, 4 or 8 that share the item's sources (EvalArgs.waves). In a wave,
// lanes are laid out as S source slices x L lane-targets, each lane holding
// TPL targets (1 to 4 with one output and one right-hand side, else 1 or 2),
// chosen per item to keep most lane-slots busy: a 45-target item runs as 15
// lanes x 3 targets x 4 slices (94% of the slots) instead of 45 of 64 lanes,
// or 23 x 2 x 2 (70%). More targets per lane also read each staged source once
// for more pairs. Sources are staged in the wave's own part of LDS 64 at a
// time (records padded to 16 bytes, the tail of a tile filled with
// zero-density sources far away), so the loop over a tile has the same trip
// count in every lane, no per-pair validity test and no barrier. Slices, then
// waves, are summed through LDS at the end, in a fixed order.
constexpr int kFar = 1000000000;  // far-away coordinate of padding records (1e9)

template <int NRHS, bool SL, bool DL, bool FIELD>
struct EvalShape {
    static constexpr int NOUT = FIELD ? 4 : 1;
    static constexpr int WP = 3 + (SL ? NRHS : 0) + (DL ? 3 * NRHS : 0);  // point source record
    static constexpr int WS = 3 + NRHS;                                   // surface source record
    static constexpr int W = ((WP > WS ? WP : WS) + 3) / 4 * 4;           // floats, 16-byte aligned
    static constexpr int NREC = 128;                                      // 64 + room for slice overrun
};

// Orders this wave's LDS writes before its later LDS reads (and the reverse):
// one wave's LDS operations complete in order, so only the compiler must not
// move them.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// The wave's share of an item; sh_all: the workgroup's LDS, NSH floats for
// each wave. MW: the workgroup has several waves (a kernel of its own: the
// share's bookkeeping spills scalar registers, 1.4% of a 300,000-point apply).
template <int TPL, int NRHS, bool SL, bool DL, bool FIELD, bool MW, int NSH, bool L2P = false>
__device__ void eval_item(const EvalArgs &a, const SurfaceGeom &g, const PointSrc &src, int leaf, int64_t t_first,
                          int nt, float *sh_all) {
    const int w = MW ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) : 0, nw = MW ? blockDim.x >> 6 : 1;
    using E = EvalShape<NRHS, SL, DL, FIELD>;
    constexpr int NOUT = E::NOUT, W = E::W;
    const int lane = threadIdx.x & 63;
    float *sh = sh_all + (size_t)w * NSH;
    const int L = (nt + TPL - 1) / TPL;      // lanes per slice
    const int S = 64 / L;                    // slices
    const int slice = lane / L, tl = lane % L;
    const int niter = (64 + S - 1) / S;      // uniform trip count over a tile
    const bool active = slice < S;

    float xg[TPL], yg[TPL], zg[TPL], xl[TPL], yl[TPL], zl[TPL];
    const double cx = g.centre[3 * leaf], cy = g.centre[3 * leaf + 1], cz = g.centre[3 * leaf + 2];
#pragma unroll
    for (int u = 0; u < TPL; ++u) {
        const int t = tl + u * L;
        const int64_t k = t_first + (t < nt ? t : 0);
        xg[u] = a.tx[k];
        yg[u] = a.ty[k];
        zg[u] = a.tz[k];
        xl[u] = (float)((double)xg[u] - cx);
        yl[u] = (float)((double)yg[u] - cy);
        zl[u] = (float)((double)zg[u] - cz);
    }
    float hi[TPL][NRHS][NOUT], lo[TPL][NRHS][NOUT];
#pragma unroll
    for (int u = 0; u < TPL; ++u)
        for (int r = 0; r < NRHS; ++r)
            for (int o = 0; o < NOUT; ++o) hi[u][r][o] = lo[u][r][o] = 0.f;

    // padding records: slots 64..127 once (every tile's overrun), slots
    // [cnt, 64) per tile
    auto pad = [&](int slot) {
        float *p = sh + slot * W;
        p[0] = p[1] = p[2] = (float)kFar;
        for (int c = 3; c < W; ++c) p[c] = 0.f;
    };
    if constexpr (!L2P) pad(64 + lane);

    // one staged tile of 64 surface points added to the targets' sums; surface
    // points never coincide with targets (they lie outside the box)
    auto surface_tile = [&](const float *tile) {
        float part[TPL][NRHS][NOUT];
#pragma unroll
        for (int u = 0; u < TPL; ++u)
            for (int r = 0; r < NRHS; ++r)
                for (int o = 0; o < NOUT; ++o) part[u][r][o] = 0.f;
        for (int i = 0; i < niter; ++i) {
            const int rec = slice + i * S;
            const float4 *p4 = (const float4 *)(tile + (L2P ? min(rec, 64) : rec) * W);
            const float4 r0 = p4[0];
            float ph[NRHS];
            ph[0] = r0.w;
            if (NRHS > 1) {
                const float4 r1 = p4[1];
                const float rest[3] = {r1.x, r1.y, r1.z};
                for (int r = 1; r < NRHS; ++r) ph[r] = rest[r - 1];
            }
#pragma unroll
            for (int u = 0; u < TPL; ++u) {
                const float dx = xl[u] - r0.x, dy = yl[u] - r0.y, dz = zl[u] - r0.z;
                const float r2 = dx * dx + dy * dy + dz * dz;
                const float inv = rsq(r2);
                if constexpr (FIELD) {
                    const float inv3 = inv * inv * inv;
                    for (int r = 0; r < NRHS; ++r) {
                        part[u][r][0] += ph[r] * inv;
                        const float di3 = ph[r] * inv3;
                        part[u][r][1] += di3 * dx;
                        part[u][r][2] += di3 * dy;
                        part[u][r][3] += di3 * dz;
                    }
                } else {
                    for (int r = 0; r < NRHS; ++r) part[u][r][0] += ph[r] * inv;
                }
            }
        }
#pragma unroll
        for (int u = 0; u < TPL; ++u)
            for (int r = 0; r < NRHS; ++r)
                for (int o = 0; o < NOUT; ++o) two_sum_into(hi[u][r][o], lo[u][r][o], part[u][r][o]);
    };
    if constexpr (L2P) {
        // L2P: the leaf's own downward surface, every tile staged at once
        // (65 records a tile: the last serves the slices' overrun), so that
        // an item waits for its density and the surface's points once
        const float *phi = a.phi_d + (int64_t)leaf * NRHS * g.n_pad;
        const double rr = a.rad_down * g.half[leaf];
        const int ntile = (g.ns + 63) / 64;
        constexpr int UN = 4;
        for (int t0 = 0; t0 < ntile; t0 += UN) {
            double y[UN][3];
            float ph[UN][NRHS];
#pragma unroll
            for (int u = 0; u < UN; ++u) {  // clamped: no branch around the loads
                const int m = min(64 * (t0 + u) + lane, g.ns - 1);
#pragma unroll
                for (int c = 0; c < 3; ++c) y[u][c] = g.Y[3 * m + c];
                for (int r = 0; r < NRHS; ++r) ph[u][r] = phi[r * g.n_pad + m];
            }
#pragma unroll
            for (int u = 0; u < UN; ++u) {
                if (t0 + u >= ntile) break;
                const bool ok = 64 * (t0 + u) + lane < g.ns;
                float *p = sh + ((t0 + u) * 65 + lane) * W;
#pragma unroll
                for (int c = 0; c < 3; ++c) p[c] = ok ? (float)(rr * y[u][c]) : (float)kFar;
                for (int r = 0; r < NRHS; ++r) p[3 + r] = ok ? ph[u][r] : 0.f;
                if (lane == 0) pad((t0 + u) * 65 + 64);
            }
        }
        wave_sync();
        for (int t = 0; t < ntile; ++t) surface_tile(sh + t * 65 * W);
        wave_sync();
    } else {
        int turn = 0;
        // surfaces: M2P (W-list boxes)
        for (int e = a.soff[leaf]; e < a.soff[leaf + 1]; ++e) {
            const int box = a.sbox[e];
            const double rr = a.rad_up * g.half[box];
            const double ox = g.centre[3 * box] - cx, oy = g.centre[3 * box + 1] - cy, oz = g.centre[3 * box + 2] - cz;
            const float *phi = a.phi_u + (int64_t)box * NRHS * g.n_pad;
            for (int m0 = 0; m0 < g.ns; m0 += 64) {
                if (MW && turn++ % nw != w) continue;  // the item's surface tiles in turn
                const int m = m0 + lane;
                if (m < g.ns) {
                    float *p = sh + lane * W;
                    p[0] = (float)(ox + rr * g.Y[3 * m]);
                    p[1] = (float)(oy + rr * g.Y[3 * m + 1]);
                    p[2] = (float)(oz + rr * g.Y[3 * m + 2]);
                    for (int r = 0; r < NRHS; ++r) p[3 + r] = phi[r * g.n_pad + m];
                } else {
                    pad(lane);
                }
                wave_sync();
                surface_tile(sh);
                wave_sync();
            }
        }

        // points: P2P (U list) and the direct W / X pairs; r < delta excluded
        // (delta2 > 0 also excludes r = 0). Ranges [poff, pmid) may hold a pair
        // closer than delta and are tested pair by pair; for ranges [pmid,
        // poff + 1) the setup has shown that the points' bounding boxes are
        // farther apart than delta, and the test is skipped.
        const float delta2 = a.delta2;
        // The ranges e0 .. e1 - 1 as one sequence of sources, staged 64 at a
        // time: a tile runs across range boundaries, so only the sequence's last
        // tile is padded (per-range tiles left a quarter of the slots padding on
        // the clustered cloud, whose leaves have about ten merged ranges each).
        // (e, off) is the wave-uniform position of the tile's first source.
        // Range bounds are wave-uniform: read through the constant address space
        // they become scalar loads, and the four bounds pairs a tile looks at
        // first are read together (the array is padded by 8 entries, so reads
        // past the last range stay inside it).
        const int32_t __attribute__((address_space(4))) *rng =
            (const int32_t __attribute__((address_space(4))) *)a.prng;
        auto stream = [&](auto test_tag, int e0, int e1, int rank) {
            constexpr bool TEST = decltype(test_tag)::value;
            int e = e0, off = 0, left = 0x7fffffff;  // tiles left for this wave
            if (MW && e0 < e1) {
                // a contiguous share of the sequence's tiles for each wave (whole
                // tiles apart from the sequence's last), found from the running
                // counts, 64 ranges at a time
                const int c0 = a.pcum[e0];
                const int ntile = (a.pcum[e1 - 1] - c0 + rng[2 * e1 - 1] - rng[2 * e1 - 2] + 63) / 64;
                const int at = ntile * rank / nw;
                left = ntile * (rank + 1) / nw - at;
                for (int k = e0; k < e1; k += 64) {
                    const bool below = k + lane < e1 && a.pcum[min(k + lane, e1 - 1)] - c0 <= 64 * at;
                    const int nbelow = __popcll(__ballot(below));
                    if (nbelow == 0) break;
                    e = k + nbelow - 1;
                }
                e = __builtin_amdgcn_readfirstlane(e);
                off = 64 * at - (a.pcum[e] - c0);
            }
            while (e < e1) {
                if (MW && left-- <= 0) break;
                // this lane's source: the tile covers the rest of range e and,
                // past its end, the next ranges (a tile rarely spans more than four)
                int j = -1;
                {
                    int bnd[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) bnd[u] = rng[2 * e + u];
                    int base = 0, k = e;  // base: tile position where range k starts
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int r0 = bnd[2 * u] + (u == 0 ? off : 0);
                        const int len = (k < e1) ? bnd[2 * u + 1] - r0 : 0;
                        if (lane >= base && lane < base + len) j = r0 + (lane - base);
                        base += len;
                        k += k < e1 ? 1 : 0;
                    }
                    while (k < e1 && base < 64) {
                        const int r0 = rng[2 * k], len = rng[2 * k + 1] - r0;
                        if (lane >= base && lane < base + len) j = r0 + (lane - base);
                        base += len;
                        ++k;
                    }
                }
                if (j >= 0) {
                    float *p = sh + lane * W;
                    p[0] = src.x[j];
                    p[1] = src.y[j];
                    p[2] = src.z[j];
                    int o = 3;
                    if (SL)
                        for (int r = 0; r < NRHS; ++r) p[o++] = src.q[r * src.n + j];
                    if (DL)
                        for (int r = 0; r < NRHS; ++r) {
                            p[o++] = src.mx[r * src.n + j];
                            p[o++] = src.my[r * src.n + j];
                            p[o++] = src.mz[r * src.n + j];
                        }
                } else {
                    pad(lane);
                }
                wave_sync();
                float part[TPL][NRHS][NOUT];
#pragma unroll
                for (int u = 0; u < TPL; ++u)
                    for (int r = 0; r < NRHS; ++r)
                        for (int o = 0; o < NOUT; ++o) part[u][r][o] = 0.f;
                for (int i = 0; i < niter; ++i) {
                    const float *p = sh + (slice + i * S) * W;
                    float rec[W];
#pragma unroll
                    for (int c = 0; c < W; c += 4) {
                        const float4 v = *(const float4 *)(p + c);
                        rec[c] = v.x;
                        rec[c + 1] = v.y;
                        rec[c + 2] = v.z;
                        rec[c + 3] = v.w;
                    }
#pragma unroll
                    for (int u = 0; u < TPL; ++u) {
                        const float dx = xg[u] - rec[0], dy = yg[u] - rec[1], dz = zg[u] - rec[2];
                        const float r2 = dx * dx + dy * dy + dz * dz;
                        const float inv = TEST ? (r2 >= delta2 ? rsq(r2) : 0.f) : rsq(r2);
                        const float inv2 = inv * inv;
                        int o = 3;
                        float sl[NRHS];
                        for (int r = 0; r < NRHS; ++r) sl[r] = SL ? rec[o + r] : 0.f;
                        if (SL) o += NRHS;
                        if constexpr (FIELD) {
                            const float inv3 = inv2 * inv;
                            for (int r = 0; r < NRHS; ++r) {
                                part[u][r][0] += sl[r] * inv;
                                const float di3 = sl[r] * inv3;
                                part[u][r][1] += di3 * dx;
                                part[u][r][2] += di3 * dy;
                                part[u][r][3] += di3 * dz;
                            }
                        } else {
                            for (int r = 0; r < NRHS; ++r) {
                                // q / r + (m . d) / r^3 = (q + (m . d) / r^2) / r
                                float t = sl[r];
                                if (DL) {
                                    const float md = rec[o + 3 * r] * dx + rec[o + 3 * r + 1] * dy + rec[o + 3 * r + 2] * dz;
                                    t += md * inv2;
                                }
                                part[u][r][0] += t * inv;
                            }
                        }
                    }
                }
#pragma unroll
                for (int u = 0; u < TPL; ++u)
                    for (int r = 0; r < NRHS; ++r)
                        for (int o = 0; o < NOUT; ++o) two_sum_into(hi[u][r][o], lo[u][r][o], part[u][r][o]);
                wave_sync();
                // advance the position by 64 sources
                int adv = 64;
                while (e < e1) {
                    const int rest = rng[2 * e + 1] - rng[2 * e] - off;
                    if (adv < rest) {
                        off += adv;
                        break;
                    }
                    adv -= rest;
                    ++e;
                    off = 0;
                }
            }
        };
        const int pmid = a.pmid ? a.pmid[leaf] : a.poff[leaf + 1];
        stream(std::true_type{}, a.poff[leaf], pmid, w);
        stream(std::false_type{}, pmid, a.poff[leaf + 1], nw - 1 - w);
    }

    // sum the slices of each target through the wave's LDS
    constexpr int NV = TPL * NRHS * NOUT;
    auto put = [&](float *q) {
        int v = 0;
#pragma unroll
        for (int u = 0; u < TPL; ++u)
            for (int r = 0; r < NRHS; ++r)
                for (int o = 0; o < NOUT; ++o, ++v) {
                    q[2 * v] = hi[u][r][o];
                    q[2 * v + 1] = lo[u][r][o];
                }
    };
    auto add = [&](const float *q) {
        int v = 0;
#pragma unroll
        for (int u = 0; u < TPL; ++u)
            for (int r = 0; r < NRHS; ++r)
                for (int o = 0; o < NOUT; ++o, ++v) {
                    two_sum_into(hi[u][r][o], lo[u][r][o], q[2 * v]);
                    lo[u][r][o] += q[2 * v + 1];
                }
    };
    if (active && slice > 0) put(sh + (size_t)lane * NV * 2);
    wave_sync();
    if (active && slice == 0)
        for (int sl2 = 1; sl2 < S; ++sl2) add(sh + (size_t)(sl2 * L + tl) * NV * 2);
    if constexpr (MW) {
        // the other waves' sums, added by wave 0 in their order
        wave_sync();
        if (w > 0 && lane < L) put(sh + (size_t)lane * NV * 2);
        __syncthreads();
        if (w > 0) return;
        if (lane < L)
            for (int w2 = 1; w2 < nw; ++w2) add(sh_all + (size_t)w2 * NSH + (size_t)lane * NV * 2);
    }
    if (active && slice == 0) {
#pragma unroll
        for (int u = 0; u < TPL; ++u) {
            const int t = tl + u * L;
            if (t >= nt) continue;
            const int64_t k = t_first + t;
            const int64_t dst = a.trg_perm ? a.trg_perm[k] : k;
            for (int r = 0; r < NRHS; ++r) {
                if (a.pot) {
                    float *pp = a.pot + r * a.n_trg + dst;
                    const float v = (hi[u][r][0] + lo[u][r][0]) * kInv4Pi;
                    *pp = a.accumulate ? *pp + v : v;
                }
                if (FIELD && a.field) {
                    float *f = a.field + ((int64_t)r * a.n_trg + dst) * 3;
                    for (int c = 0; c < 3; ++c) {
                        const float v = (hi[u][r][1 + c] + lo[u][r][1 + c]) * kInv4Pi;
                        f[c] = a.accumulate ? f[c] + v : v;
                    }
                }
            }
        }
    }
}

template <int NRHS, bool SL, bool DL, bool FIELD>
struct EvalLds {
    using E = EvalShape<NRHS, SL, DL, FIELD>;
    // up to 4 targets per lane where one output and one right-hand side
    // keep the accumulators few; 2 otherwise
    static constexpr int MAXTPL = (E::NOUT == 1 && NRHS == 1) ? 4 : 2;
    // floats per wave; the sums of the end reuse the source records' space
    static constexpr int NSH = E::NREC * E::W, NRED = 64 * MAXTPL * NRHS * E::NOUT * 2;
    static constexpr int N = NSH > NRED ? NSH : NRED;
};

// targets per lane of an item of nt targets
template <int MAXTPL>
__device__ inline int targets_per_lane(int nt) {
    // targets per lane (TPL): the count that keeps the most lane-slots busy,
    // nt * S / (64 TPL) with S = 64 / ceil(nt / TPL) slices; ties to the larger
    // (fewer LDS reads per pair)
    int best = 1, bnum = nt * (64 / nt), bden = 64;
#pragma unroll
    for (int tpl = 2; tpl <= MAXTPL; ++tpl) {
        const int num = nt * (64 / ((nt + tpl - 1) / tpl)), den = 64 * tpl;
        if (num * bden >= bnum * den) {
            best = tpl;
            bnum = num;
            bden = den;
        }
    }
    return best;
}

template <int NRHS, bool SL, bool DL, bool FIELD, bool MW, bool L2P>
__device__ inline void eval_items(const EvalArgs &a, const SurfaceGeom &g, const PointSrc &src, float *sh) {
    using M = EvalLds<NRHS, SL, DL, FIELD>;
    constexpr int MAXTPL = M::MAXTPL;
    const int leaf = a.wleaf[blockIdx.x];
    if constexpr (L2P)
        if (a.level[leaf] < 2) return;
    const int64_t t_first = a.tbeg[leaf] + a.wt0[blockIdx.x];
    const int nt = (int)min((int64_t)64, a.tend[leaf] - t_first);
    const int best = targets_per_lane<MAXTPL>(nt);
    if constexpr (MAXTPL == 4) {
        if (best == 4) return eval_item<4, NRHS, SL, DL, FIELD, MW, M::N, L2P>(a, g, src, leaf, t_first, nt, sh);
        if (best == 3) return eval_item<3, NRHS, SL, DL, FIELD, MW, M::N, L2P>(a, g, src, leaf, t_first, nt, sh);
    }
    if (best >= 2)
        eval_item<2, NRHS, SL, DL, FIELD, MW, M::N, L2P>(a, g, src, leaf, t_first, nt, sh);
    else
        eval_item<1, NRHS, SL, DL, FIELD, MW, M::N, L2P>(a, g, src, leaf, t_first, nt, sh);
}

template <int NRHS, bool SL, bool DL, bool FIELD, bool MW>
__global__ __launch_bounds__(MW ? 64 * kEvalMaxWaves : 64) void k_eval(EvalArgs a, SurfaceGeom g, PointSrc src) {
    extern __shared__ __align__(16) float sh[];
    eval_items<NRHS, SL, DL, FIELD, MW, false>(a, g, src, sh);
}

// L2P of the surface form: bound by latency (three to eight tiles of 64 surface
// points for an item). With every tile staged before the first is summed,
// against the evaluation kernel's tile by tile (the sums and their order are
// the same): 512 items of 152 points 14.7 -> 13.2 us, 16,726 45.5 -> 40.6, 5333
// items of 296 points 38.3 -> 37.0.
template <int NRHS, bool FIELD>
__global__ __launch_bounds__(64) void k_surface_to_points(EvalArgs a, SurfaceGeom g) {
    extern __shared__ __align__(16) float sh[];
    eval_items<NRHS, true, false, FIELD, false, true>(a, g, PointSrc{}, sh);
}

// ------------------------------------------------------------ all pairs
//
// Bound: VALU issue, 15-16 instructions a pair (3 subtractions, 3 for r^2,
// v_rsq, the exclusion's compare and select, 1/r^2, 3 + 2 for the double
// layer), as long as the chip is full. A workgroup of 16 waves owns
// T = TPL << lgL targets and runs all sources: thread (s, tl) holds the TPL
// targets tl + u L (L = 1 << lgL <= 64 lanes) and takes the staged sources
// s, s + S, ... of every tile (S = 1024 / L slices), so that a few thousand
// targets, or a few hundred, still fill 256 CUs; the slices are summed across
// lanes, then across waves through LDS, in a fixed order and without scratch
// memory. The next tile's values load while the current one is used. Tiles
// are 1024 sources in two buffers (one barrier a tile), or with one target
// per lane 4096 in one: the few pairs of a 1024-tile then end before the next
// one's loads do (300 targets, 300,000 sources: 237 -> 126 us). Records are one
// (single layer) or two float4 in separate arrays, so that lanes of different
// slices read consecutive 16-byte slots. Kernels for the potential of the
// single layer, of the double layer (with or without the single) and for the
// field (with the potential) leave out the other's arithmetic.
// Float32 sums of at most 64 sources are folded into (hi, lo) pairs.
// Measured against one thread per target, workgroups of 256 and every output
// computed: 801 x 801 52 -> 8.5 us (a launch), 300 x 300,000 single layer
// 18,990 -> 126 us, 4000 x 1M both layers 64,440 -> 1,980 us (2.0e12 pairs/s,
// 0.82 of 3.93e13 lane-instructions/s at 16 a pair), 60,000 x 60,000 single
// layer 3,720 -> 1,020 us.
constexpr int kDirThreads = 1024;

// one pair, as in k_direct below: v the source and its charge, m its dipole
template <bool DL, bool FIELD, int NOUT>
__device__ inline void direct_pair(float x, float y, float z, const float4 &v, const float4 &m, float delta2,
                                   float (&part)[NOUT]) {
    const float dx = x - v.x, dy = y - v.y, dz = z - v.z;
    const float r2 = dx * dx + dy * dy + dz * dz;
    float inv = rsq(r2);
    inv = r2 < delta2 ? 0.f : inv;
    const float inv2 = inv * inv;
    if constexpr (FIELD) {
        const float qi = v.w * inv, di3 = qi * inv2;
        part[0] += qi;
        part[1] += di3 * dx;
        part[2] += di3 * dy;
        part[3] += di3 * dz;
    } else {
        float w = v.w;
        if (DL) w += (m.x * dx + m.y * dy + m.z * dz) * inv2;
        part[0] += w * inv;
    }
}

// Few sources: one thread per target, workgroups of 256, the sources staged 256
// at a time. The slices of the kernel below cost a workgroup of 1024 threads and
// two sums across it, which many targets with a few sources each do not repay.
// 1M targets, 16 sources, single layer 44 -> 8 us (a launch), field 68 -> 11;
// 10,000 targets, 64 sources, field 22 -> 8.
template <bool DL, bool FIELD>
__global__ __launch_bounds__(256) void k_direct_few(const float *trg, int64_t n_trg, const float *src,
                                                   const float *nrm, int64_t n_src, const float *q, const float *mu,
                                                   float delta2, float *pot, float *field) {
    constexpr int NOUT = FIELD ? 4 : 1, TILE = 256;
    __shared__ float4 a[TILE], b[DL ? TILE : 1];
    const int t = threadIdx.x;
    const int64_t i = (int64_t)blockIdx.x * TILE + t, ic = min(i, n_trg - 1);
    const float x = trg[3 * ic], y = trg[3 * ic + 1], z = trg[3 * ic + 2];
    float hi[NOUT], lo[NOUT], part[NOUT];
#pragma unroll
    for (int o = 0; o < NOUT; ++o) hi[o] = lo[o] = 0.f;
    for (int64_t j0 = 0; j0 < n_src; j0 += TILE) {
        if (j0) __syncthreads();  // every wave is done with the tile before
        const int cnt = (int)min((int64_t)TILE, n_src - j0);
        if (t < cnt) {
            const int64_t j = j0 + t;
            float4 v = make_float4(src[3 * j], src[3 * j + 1], src[3 * j + 2], q ? q[j] : 0.f);
            // a coordinate that is not finite makes every sum NaN, also where 1/r alone would give 0
            v.w += 0.f * v.x + 0.f * v.y + 0.f * v.z;
            a[t] = v;
            if (DL) b[t] = make_float4(mu[j] * nrm[3 * j], mu[j] * nrm[3 * j + 1], mu[j] * nrm[3 * j + 2], 0.f);
        }
        __syncthreads();
        for (int k0 = 0; k0 < cnt; k0 += 64) {  // float32 sums of at most 64 sources
            const int k1 = min(cnt, k0 + 64);
#pragma unroll
            for (int o = 0; o < NOUT; ++o) part[o] = 0.f;
#pragma unroll 4
            for (int k = k0; k < k1; ++k) direct_pair<DL, FIELD>(x, y, z, a[k], DL ? b[k] : a[k], delta2, part);
#pragma unroll
            for (int o = 0; o < NOUT; ++o) two_sum_into(hi[o], lo[o], part[o]);
        }
    }
    if (i >= n_trg) return;
    const float nf = n_src > 0 ? 0.f * x + 0.f * y + 0.f * z : 0.f;  // as for the sources
    if (pot) pot[i] = (hi[0] + lo[0]) * kInv4Pi + nf;
    if (FIELD && field)
#pragma unroll
        for (int c = 0; c < 3; ++c) field[3 * i + c] = (hi[NOUT - 3 + c] + lo[NOUT - 3 + c]) * kInv4Pi + nf;
}

template <bool DL, bool FIELD, int TPL, int KS>
__global__ __launch_bounds__(kDirThreads) void k_direct(const float *trg, int64_t n_trg, const float *src,
                                                       const float *nrm, int64_t n_src, const float *q,
                                                       const float *mu, float delta2, int lgL, float *pot,
                                                       float *field) {
    constexpr int NOUT = FIELD ? 4 : 1, NREC = DL ? 2 : 1, NW = kDirThreads / 64;
    constexpr int TILE = KS * kDirThreads, NBUF = KS == 1 ? 2 : 1;
    constexpr int NTILE = NBUF * NREC * TILE * 4, NRED = NW * 64 * TPL * NOUT * 2;
    __shared__ __align__(16) float sh[NTILE > NRED ? NTILE : NRED];
    float4 *rec = (float4 *)sh;  // [buffer][record part][source of the tile]
    const int t = threadIdx.x, lane = t & 63, wave = t >> 6;
    const int L = 1 << lgL, S = kDirThreads >> lgL, s = t >> lgL, tl = t & (L - 1);
    const int64_t t0 = (int64_t)blockIdx.x * (TPL * L);
    float x[TPL], y[TPL], z[TPL], hi[TPL][NOUT], lo[TPL][NOUT], part[TPL][NOUT];
#pragma unroll
    for (int u = 0; u < TPL; ++u) {
        const int64_t i = min(t0 + tl + u * L, n_trg - 1);
        x[u] = trg[3 * i];
        y[u] = trg[3 * i + 1];
        z[u] = trg[3 * i + 2];
#pragma unroll
        for (int o = 0; o < NOUT; ++o) hi[u][o] = lo[u][o] = part[u][o] = 0.f;
    }
    float4 r0[KS], r1[KS];
    auto load = [&](int64_t j0) {
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            const int64_t j = j0 + k * kDirThreads + t;
            r0[k] = make_float4((float)kFar, (float)kFar, (float)kFar, 0.f);  // past the end: no strength, far away
            r1[k] = make_float4(0.f, 0.f, 0.f, 0.f);
            if (j < n_src) {
                r0[k].x = src[3 * j];
                r0[k].y = src[3 * j + 1];
                r0[k].z = src[3 * j + 2];
                r0[k].w = q ? q[j] : 0.f;
                if (DL) {
                    r1[k].x = nrm[3 * j];
                    r1[k].y = nrm[3 * j + 1];
                    r1[k].z = nrm[3 * j + 2];
                    r1[k].w = mu[j];
                }
            }
        }
    };
    auto stage = [&](float4 *a, float4 *b) {
#pragma unroll
        for (int k = 0; k < KS; ++k) {
            // a coordinate that is not finite makes every sum NaN, also where 1/r alone would give 0
            r0[k].w += 0.f * r0[k].x + 0.f * r0[k].y + 0.f * r0[k].z;
            a[k * kDirThreads + t] = r0[k];
            if (DL) b[k * kDirThreads + t] = make_float4(r1[k].w * r1[k].x, r1[k].w * r1[k].y, r1[k].w * r1[k].z, 0.f);
        }
    };
    auto fold = [&] {
#pragma unroll
        for (int u = 0; u < TPL; ++u)
#pragma unroll
            for (int o = 0; o < NOUT; ++o) {
                two_sum_into(hi[u][o], lo[u][o], part[u][o]);
                part[u][o] = 0.f;
            }
    };
    load(0);
    int buf = 0, held = 0;
    for (int64_t j0 = 0; j0 < n_src; j0 += TILE, buf ^= NBUF - 1) {
        float4 *a = rec + buf * NREC * TILE, *b = a + TILE;
        if (NBUF == 1) __syncthreads();  // every wave is done with the tile before
        stage(a, b);
        __syncthreads();  // the tile is staged (with two buffers: and the one before no longer read)
        if (j0 + TILE < n_src) load(j0 + TILE);
        const int cnt = (int)min((int64_t)TILE, n_src - j0);
        const int niter = (cnt + S - 1) >> (10 - lgL);  // sources per slice, at most KS L
        for (int i = 0; i < niter; ++i) {
            const float4 v = a[s + i * S];
            float4 m;
            if (DL) m = b[s + i * S];
#pragma unroll
            for (int u = 0; u < TPL; ++u) {
                const float dx = x[u] - v.x, dy = y[u] - v.y, dz = z[u] - v.z;
                const float r2 = dx * dx + dy * dy + dz * dz;
                float inv = rsq(r2);
                inv = r2 < delta2 ? 0.f : inv;
                const float inv2 = inv * inv;
                if constexpr (FIELD) {
                    const float qi = v.w * inv, di3 = qi * inv2;
                    part[u][0] += qi;
                    part[u][1] += di3 * dx;
                    part[u][2] += di3 * dy;
                    part[u][3] += di3 * dz;
                } else {
                    float w = v.w;
                    if (DL) w += (m.x * dx + m.y * dy + m.z * dz) * inv2;
                    part[u][0] += w * inv;
                }
            }
        }
        held += niter;
        if (held + KS * L > 64) {
            fold();
            held = 0;
        }
    }
    fold();
    // slices of one wave: lanes that differ in the bits above L
    for (int o = L; o < 64; o <<= 1)
#pragma unroll
        for (int u = 0; u < TPL; ++u)
#pragma unroll
            for (int c = 0; c < NOUT; ++c) {
                const float h = __shfl_xor(hi[u][c], o), l = __shfl_xor(lo[u][c], o);
                two_sum_into(hi[u][c], lo[u][c], h);
                lo[u][c] += l;
            }
    __syncthreads();  // the tiles are no longer read
    const int nt = TPL * L;
    if (lane < L)
#pragma unroll
        for (int u = 0; u < TPL; ++u)
#pragma unroll
            for (int c = 0; c < NOUT; ++c) {
                float *p = sh + 2 * ((wave * NOUT + c) * nt + u * L + lane);
                p[0] = hi[u][c];
                p[1] = lo[u][c];
            }
    __syncthreads();
    const int64_t i = t0 + t;
    if (t >= nt || i >= n_trg) return;
    // as for the sources: 0, or NaN for a target that is not finite
    const float nf = n_src > 0 ? 0.f * trg[3 * i] + 0.f * trg[3 * i + 1] + 0.f * trg[3 * i + 2] : 0.f;
#pragma unroll
    for (int c = 0; c < NOUT; ++c) {
        float h = 0.f, l = 0.f;
        for (int w = 0; w < NW; ++w) {
            const float *p = sh + 2 * ((w * NOUT + c) * nt + t);
            two_sum_into(h, l, p[0]);
            l += p[1];
        }
        const float v = (h + l) * kInv4Pi + nf;
        if (c == 0) {
            if (pot) pot[i] = v;
        } else if (field) {
            field[3 * i + c - 1] = v;
        }
    }
}

template <bool DL, bool FIELD>
void launch_direct(const float *trg, int64_t n_trg, const float *src, const float *nrm, int64_t n_src, const float *q,
                   const float *mu, float delta2, float *pot, float *field, hipStream_t s) {
    const auto few = [&] {
        hipLaunchKernelGGL((k_direct_few<DL, FIELD>), dim3((unsigned)((n_trg + 255) / 256)), dim3(256), 0, s, trg, n_trg,
                           src, nrm, n_src, q, mu, delta2, pot, field);
    };
    // up to here a pass of k_direct_few ends within the launch's own 8 us
    // (192 sources, field: 10.2 us, sliced 8.4)
    if (n_src <= 128 && n_trg <= 65536) return few();
    // Targets per workgroup T = TPL << lg by a fit of the measured times: a
    // round of 256 workgroups (one per CU) costs T plus about 5.6 for staging
    // and latency, which two resident workgroups share. (300,000 sources,
    // single layer, one round: T = 4 169 us, 8 232, 16 385.) More targets per
    // lane read each staged record from LDS fewer times, hence the weights,
    // which only decide between splits of the same T; ties go to the larger T.
    constexpr int kTplMax = FIELD ? 2 : 4;
    int tpl = 1, lg = 0;
    double best = 1e300, rounds_best = 0;
    for (int c = kTplMax, lc = FIELD ? 1 : 2; c >= 1; c >>= 1, --lc)
        for (int l = 6; l >= 0; --l) {
            if (c > 1 && l < 2) continue;  // fewer than four lanes a slice: one target per lane instead
            const int64_t T = (int64_t)c << l, wg = (n_trg + T - 1) >> (lc + l);
            const int64_t rounds = (wg + 255) >> 8;
            const double cost = (double)rounds * (double)T * (c >= 4 ? 1.0 : c == 2 ? 1.02 : 1.05) +
                                5.6 * (double)((rounds + 1) / 2);
            if (cost < best) {
                best = cost;
                rounds_best = (double)rounds;
                tpl = c;
                lg = l;
            }
        }
    // One thread per target instead where that ends sooner. Sliced, a source
    // costs 0.0587 ns per unit of the cost above (single layer), and each round
    // its start and final sums; one thread per target, a source takes the chain
    // of its pair, or, from three waves a SIMD, its issue. Microseconds, sliced
    // and this: 1M targets and 64 sources 47 and 18 (field 81 and 27), 512
    // sources 132 and 122, 100,000 targets and 256 sources 25 and 11 (field 42
    // and 16), 1536 54 and 56. Each is off by up to 15% (200,000 targets, 1024
    // sources: 61 and 70), hence the margin; with more than one of the sliced
    // kernel's tiles its rounds overlap, and it is never far behind (1M targets,
    // 2048 sources: 496 and 468; 100,000, field: 101 and 112).
    constexpr double kPair = FIELD ? 1.43 : DL ? 1.4 : 1.0, kRound = FIELD ? 2.7 : DL ? 1.9 : 1.6;
    constexpr double kChain = FIELD || DL ? 0.043 : 0.033, kIssue = FIELD ? 0.0235 : DL ? 0.022 : 0.0155;
    const double waves = (double)((n_trg + 65535) / 65536);  // per SIMD
    if (n_src <= 1024 && 1.15 * ((double)n_src * std::max(kChain, waves * kIssue) + 0.1 * waves) <=
                             (double)n_src * 5.87e-5 * kPair * best + kRound * rounds_best)
        return few();
    const int64_t T = (int64_t)tpl << lg;
    const dim3 g((unsigned)((n_trg + T - 1) / T)), b(kDirThreads);
    auto go = [&](auto kern) {
        hipLaunchKernelGGL(kern, g, b, 0, s, trg, n_trg, src, nrm, n_src, q, mu, delta2, lg, pot, field);
    };
    if constexpr (kTplMax == 4)
        if (tpl == 4) return go(k_direct<DL, FIELD, 4, 1>);
    if (tpl == 2)
        go(k_direct<DL, FIELD, 2, 1>);
    else if (lg <= 4 && n_src > kDirThreads)
        go(k_direct<DL, FIELD, 1, 4>);
    else
        go(k_direct<DL, FIELD, 1, 1>);
}

}  // namespace

#define FMM_NRHS_SWITCH(NRHS_VAR, CALL)                                                        \
    switch (NRHS_VAR) {                                                                        \
    case 1: { constexpr int R = 1; CALL; } break;                                              \
    case 2: { constexpr int R = 2; CALL; } break;                                              \
    case 3: { constexpr int R = 3; CALL; } break;                                              \
    case 4: { constexpr int R = 4; CALL; } break;                                              \
    default: throw Error(FMM_ERR_ARG, "nrhs must be 1..4");                                    \
    }

void points_to_surface(int nrhs, bool sl, bool dl, const int32_t *items, int nitems, const int32_t *roff,
                       const int32_t *rng, double rfac, const SurfaceGeom &g, const PointSrc &src, float *out,
                       bool accumulate, hipStream_t s) {
    if (nitems <= 0) return;
    FMM_REQUIRE(g.ns <= g.n_pad && g.n_pad <= 512, "points_to_surface: surface too large");
    dim3 gr(nitems), bl(64);
    int acc = accumulate ? 1 : 0;
    if (sl && dl) {
        FMM_NRHS_SWITCH(nrhs, hipLaunchKernelGGL((k_points_to_surface<R, true, true>), gr, bl, 0, s, items, roff, rng,
                                                 rfac, g, src, out, acc));
    } else if (dl) {
        FMM_NRHS_SWITCH(nrhs, hipLaunchKernelGGL((k_points_to_surface<R, false, true>), gr, bl, 0, s, items, roff,
                                                 rng, rfac, g, src, out, acc));
    } else {
        FMM_NRHS_SWITCH(nrhs, hipLaunchKernelGGL((k_points_to_surface<R, true, false>), gr, bl, 0, s, items, roff,
                                                 rng, rfac, g, src, out, acc));
    }
    FMM_HIP(hipGetLastError());
}

void surface_to_points(int nrhs, const EvalArgs &a, const SurfaceGeom &g, hipStream_t s) {
    if (a.nwork <= 0) return;
    FMM_REQUIRE(g.ns > 0 && g.ns <= 512 && g.n_pad >= g.ns, "surface_to_points: surface points");
    FMM_REQUIRE(a.level, "surface_to_points: box levels");
    const int rec = (g.ns + 63) / 64 * 65;  // staged records
    const dim3 gr(a.nwork), bl(64);
#define FMM_L2P_GO(FIELD)                                                                                        \
    FMM_NRHS_SWITCH(nrhs, hipLaunchKernelGGL((k_surface_to_points<R, FIELD>), gr, bl,                            \
                                             sizeof(float) * std::max(rec * EvalShape<R, true, false, FIELD>::W, \
                                                                      EvalLds<R, true, false, FIELD>::NRED),     \
                                             s, a, g))
    if (a.field) {
        FMM_L2P_GO(true);
    } else {
        FMM_L2P_GO(false);
    }
#undef FMM_L2P_GO
    FMM_HIP(hipGetLastError());
}

size_t eval_wave_lds(int nrhs, bool sl, bool dl, bool field) {
    size_t floats = 0;
    if (field) {
        FMM_NRHS_SWITCH(nrhs, (floats = EvalLds<R, true, false, true>::N));
    } else if (sl && dl) {
        FMM_NRHS_SWITCH(nrhs, (floats = EvalLds<R, true, true, false>::N));
    } else if (dl) {
        FMM_NRHS_SWITCH(nrhs, (floats = EvalLds<R, false, true, false>::N));
    } else {
        FMM_NRHS_SWITCH(nrhs, (floats = EvalLds<R, true, false, false>::N));
    }
    return floats * sizeof(float);
}

void eval_leaves(int nrhs, bool sl, bool dl, const EvalArgs &a, const SurfaceGeom &g, const PointSrc &src,
                 hipStream_t s) {
    if (a.nwork <= 0) return;
    const int nw = a.waves;
    FMM_REQUIRE(nw >= 1 && nw <= kEvalMaxWaves && (nw == 1 || a.pcum), "eval_leaves: waves per item");
    const bool field = a.field != nullptr;
    auto go = [&](auto kern1, auto kern, int floats) {
        hipLaunchKernelGGL((nw == 1 ? kern1 : kern), dim3(a.nwork), dim3(64 * nw), (size_t)nw * floats * sizeof(float), s,
                           a, g, src);
    };
#define FMM_EVAL_GO(SL, DL, FIELD) \
    FMM_NRHS_SWITCH(nrhs, go(k_eval<R, SL, DL, FIELD, false>, k_eval<R, SL, DL, FIELD, true>, EvalLds<R, SL, DL, FIELD>::N))
    if (field) {
        FMM_REQUIRE(sl && !dl, "field output is defined for the single layer only");
        FMM_EVAL_GO(true, false, true);
    } else if (sl && dl) {
        FMM_EVAL_GO(true, true, false);
    } else if (dl) {
        FMM_EVAL_GO(false, true, false);
    } else {
        FMM_EVAL_GO(true, false, false);
    }
#undef FMM_EVAL_GO
    FMM_HIP(hipGetLastError());
}

void direct_all_pairs(const float *trg, int64_t n_trg, const float *src, const float *nrm, int64_t n_src,
                      const float *q, const float *mu, float delta, float *pot, float *field, hipStream_t s) {
    if (n_trg <= 0 || (!pot && !field)) return;
    // pairs with r^2 < delta^2 and pairs at r = 0 are left out: one test against the larger bound
    const float delta2 = std::max(delta * delta, std::numeric_limits<float>::denorm_min());
    if (field)
        launch_direct<false, true>(trg, n_trg, src, nrm, n_src, q, nullptr, delta2, pot, field, s);
    else if (mu)
        launch_direct<true, false>(trg, n_trg, src, nrm, n_src, q, mu, delta2, pot, nullptr, s);
    else
        launch_direct<false, false>(trg, n_trg, src, nrm, n_src, q, nullptr, delta2, pot, nullptr, s);
    FMM_HIP(hipGetLastError());
}

}  // namespace fmm

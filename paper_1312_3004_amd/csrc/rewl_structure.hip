// rewl_structure.hip -- structural observables of lipid configurations
// (Sec. 3.2, Eqs. 6-8): the bond order parameter S_mol of the head bonds, the
// clusters of lipids whose tails touch, and the gyration tensor and
// prolateness of the largest cluster in unfolded coordinates.
//
// One workgroup of four wavefronts per configuration.  The lipid beads go to
// LDS; the contact graph is held as one bit row per lipid, built 64 partners
// at a time with a ballot, each pair tested once (the rows are shared among
// the four wavefronts, the blocks left of the diagonal filled by transposing
// bits).  Then wavefront 1 takes S_mol, and wavefront 0 finds the clusters
// (free set, frontier and finds as bit masks, the contact rows in registers up
// to 256 lipids), takes the largest one again with its tree, unfolds it level
// by level and reduces it.
// 125 lipids, 4,096 configurations: 299 -> 121 us; 64 configurations, one a CU,
// 108 -> 43 us, bound by the chain of levels on wavefront 0.
// Sums across lanes are taken in butterfly order, so the floating-point outputs
// agree with a plain evaluation to rounding, while every integer output
// (cluster count and sizes, the tree that unfolds a cluster) is decided as in
// the definition (binary32 minimum images, binary64 squared distances, a
// screen on 16-bit places, or in binary32 for places outside [0, box),
// settling only the pairs it provably can) and is exact.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "rewl_host.h"
#include "rewl_moves.h"

namespace rewl_gpu {

namespace {

constexpr int kStructMaxLipids = 512;
constexpr int kStructWords = kStructMaxLipids / 64;
constexpr double kTailContact2 = 1.96;   // (1.4 sigma)^2
constexpr int kStructWaves = 4;          // wavefronts per configuration for the contact rows

// Orders a wavefront's own LDS writes before its later reads by other lanes.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// b - a moved once by -+box when beyond +-box/2 (selects, no branches).
__device__ __forceinline__ double st_min_image(float a, float b, float box, float half) {
    const float x = b - a;
    const float lo = x - box, hi = x + box;
    return (double)(x > half ? lo : (x < -half ? hi : x));
}

__device__ __forceinline__ void st_diff(const float *a, const float *b, float box, float half, double d[3]) {
    d[0] = st_min_image(a[0], b[0], box, half);
    d[1] = st_min_image(a[1], b[1], box, half);
    d[2] = st_min_image(a[2], b[2], box, half);
}

__device__ __forceinline__ double st_r2(const double d[3]) { return (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2]; }

// Sum over the 64 lanes (all active), in the order of a butterfly over lane
// distances 32, 16, 8, 4, 2, 1; every lane returns it.  Without LDS: the
// halves and the rows of 16 swapped (v_permlane32_swap, v_permlane16_swap),
// rows rotated by 8, then by 4 (equal to distance 4 where lanes 8 apart agree),
// quads permuted.
template <int CTRL>
__device__ __forceinline__ double dpp_d(double v) {
    return __longlong_as_double(dpp64<CTRL, 0xF>(__double_as_longlong(v)));
}
template <int ROWS>
__device__ __forceinline__ double swap_sum(double v) {
    const uint64_t b = (uint64_t)__double_as_longlong(v);
    const uint32_t lo = (uint32_t)b, hi = (uint32_t)(b >> 32);
    const auto l = ROWS == 32 ? __builtin_amdgcn_permlane32_swap(lo, lo, false, false)
                              : __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto h = ROWS == 32 ? __builtin_amdgcn_permlane32_swap(hi, hi, false, false)
                              : __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __longlong_as_double((long long)(((uint64_t)h[0] << 32) | l[0])) +
           __longlong_as_double((long long)(((uint64_t)h[1] << 32) | l[1]));
}
__device__ __forceinline__ double wave_sum(double v) {
    v = swap_sum<32>(v);
    v = swap_sum<16>(v);
    v += dpp_d<0x128>(v);   // row_ror:8
    v += dpp_d<0x124>(v);   // row_ror:4
    v += dpp_d<0x4E>(v);    // quad_perm [2, 3, 0, 1]
    v += dpp_d<0xB1>(v);    // quad_perm [1, 0, 3, 2]
    return v;
}

__device__ __forceinline__ bool tails_touch(const float *xi, const float *xj, float box, float half) {
    // xi, xj: the lipid's three beads (head, centre, end) as 9 floats.
    double d[3];
    int hit = 0;
#pragma unroll
    for (int a = 1; a < 3; ++a)
#pragma unroll
        for (int b = 1; b < 3; ++b) {
            st_diff(xi + 3 * a, xj + 3 * b, box, half, d);
            hit |= (int)(st_r2(d) < kTailContact2);
        }
    return hit != 0;
}

// The same decision from binary32 squared distances where they settle it:
// fl32((dx^2 + dy^2) + dz^2) of the binary32 differences is within 3 ulp
// (1.8e-7 relative) of the exact sum, and the binary64 sum within 2.3e-16, so
// a value below 1.959997 (1.96 (1 - 1.5e-6)) is a contact and one above
// 1.960003 is not.  *unsure is set when a pair falls between (NaN never
// does); the caller then takes tails_touch.
__device__ __forceinline__ bool tails_touch_fast(const float *xi, const float *xj, float box, float half,
                                                 bool *unsure) {
    int hit = 0, amb = 0;
#pragma unroll
    for (int a = 1; a < 3; ++a)
#pragma unroll
        for (int b = 1; b < 3; ++b) {
            float d[3];
#pragma unroll
            for (int c = 0; c < 3; ++c) {
                const float x = xj[3 * b + c] - xi[3 * a + c];
                const float lo = x - box, hi = x + box;
                d[c] = x > half ? lo : (x < -half ? hi : x);
            }
            const float r2 = (d[0] * d[0] + d[1] * d[1]) + d[2] * d[2];
            hit |= (int)(r2 < 1.959997f);
            amb |= (int)(r2 >= 1.959997f && r2 <= 1.960003f);
        }
    *unsure = amb != 0;
    return hit != 0;
}

// The same decision from places rounded down to box / 65536 (16 bits an axis,
// rewl_moves.h): differences wrap by themselves and the squared distance takes
// 4 operations where the binary32 minimum image takes 26.  The rounding moves
// a distance by less than 1.8 units, so below 1.4 by 2 units is a contact and
// above it by 2 is none; the squares of the two limits are lim.x and lim.y.
// t: (xy, z) of the centre and end bead.
__device__ __forceinline__ bool tails_touch_grid(uint4 ti, uint4 tj, uint2 lim, bool *unsure) {
    const MoveGrid a0{ti.x, ti.y}, a1{ti.z, ti.w}, b0{tj.x, tj.y}, b1{tj.z, tj.w};
    const uint32_t d0 = move_grid2(a0, b0), d1 = move_grid2(a0, b1), d2 = move_grid2(a1, b0), d3 = move_grid2(a1, b1);
    const uint32_t e0 = d0 < d1 ? d0 : d1, e1 = d2 < d3 ? d2 : d3, d = e0 < e1 ? e0 : e1;
    *unsure = d >= lim.x && d <= lim.y;
    return d < lim.x;
}

// LDS layout for M lipids (W = ceil(M / 64) mask words):
//   gt  uint4 [M]         tail beads on the 16-bit grid
//   xs  float [M][9]      bead coordinates (head, centre, end)
//   adj u64   [M][W]      contact rows
//   u   double[M][9]      unfolded beads of the largest cluster
// NW >= W mask words are unrolled; up to four, a lane keeps the contact rows of
// its lipids (64 w + lane) in registers, else it reads them from LDS.
template <int NW>
__global__ __launch_bounds__(256) void k_lipid_structure(const unsigned char *xbase, size_t xstride,
                                                       const unsigned char *lbase, size_t lstride, int np, int M,
                                                       float box, double *out) {
    extern __shared__ __align__(16) unsigned char st_lds[];
    const int W = (M + 63) >> 6;
    uint4 *gt = (uint4 *)st_lds;
    uint64_t *adj = (uint64_t *)(gt + M);
    double *u = (double *)(adj + (size_t)M * W);
    float *xs = (float *)(u + (size_t)M * 9);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int c = blockIdx.x;
    const float half = 0.5f * box;
    const float *x = (const float *)(xbase + (size_t)c * xstride);
    const int32_t *lp = (const int32_t *)(lbase + (size_t)c * lstride);
    double *rec = out + (size_t)c * 8;

    // Beads to LDS; an index outside [0, np) turns the record into NaN.
    bool bad = false, outside = false;
    const float scale = 65536.0f / box;
    for (int l = tid; l < M; l += 64 * kStructWaves) {
        for (int b = 0; b < 3; ++b) {
            const int p = lp[3 * l + b];
            const bool ok = p >= 0 && p < np;
            bad = bad || !ok;
            const int q = ok ? p : 0;
            for (int a = 0; a < 3; ++a) xs[9 * l + 3 * b + a] = x[3 * (size_t)q + a];
        }
        const float *tail = xs + 9 * l + 3;
        for (int a = 0; a < 6; ++a) outside = outside || !(tail[a] >= 0.0f && tail[a] < box);
        const MoveGrid g0 = move_grid(tail, scale), g1 = move_grid(tail + 3, scale);
        gt[l] = make_uint4(g0.xy, g0.z, g1.xy, g1.z);
    }
    // the grid knows places in [0, box) only
    const bool on_grid = __syncthreads_or(outside) == 0;
    if (__syncthreads_or(bad)) {
        if (tid < 8) rec[tid] = __builtin_nan("");
        return;
    }

    // Contact rows: row i, word w holds partners j = 64 w + lane; wavefront v
    // builds rows i = v mod 4, words from the one holding i onwards (the test
    // is symmetric in i and j).  Each lane keeps its own lipid's beads in
    // registers (NaN past the end, which never touches) and reads lipid i's,
    // the same address for all lanes.
    const float r = 1.4f * scale;
    const float in = fminf(fmaxf(r - 2.0f, 0.0f), 65535.0f), out_ = fminf(r + 2.0f, 65535.0f);
    const uint2 lim = make_uint2((uint32_t)(in * in), (uint32_t)(out_ * out_) + 1u);
    for (int w = 0; w < W; ++w) {
        const int j = 64 * w + lane;
        float tj[9];
        for (int a = 0; a < 9; ++a) tj[a] = j < M ? xs[9 * j + a] : __builtin_nanf("");
        const uint4 gj = gt[j < M ? j : 0];
        const uint64_t real = M - 64 * w >= 64 ? ~0ull : (1ull << (M - 64 * w)) - 1ull;
        for (int i = wave; i < M && (i >> 6) <= w; i += kStructWaves) {
            bool unsure;
            uint64_t m;
            if (on_grid) {
                const bool hit = tails_touch_grid(gt[i], gj, lim, &unsure);
                m = __ballot(hit) & real;
                if (__ballot(unsure) & real) m = __ballot(tails_touch(xs + 9 * i, tj, box, half));
            } else {
                const bool hit = tails_touch_fast(xs + 9 * i, tj, box, half, &unsure);
                m = __any(unsure) ? __ballot(tails_touch(xs + 9 * i, tj, box, half)) : __ballot(hit);
            }
            if ((i >> 6) == w) m &= ~(1ull << (i & 63));
            if (lane == 0) adj[(size_t)i * W + w] = m;
        }
    }
    __syncthreads();
    // Words left of row i's own block, by transposing: bit j of row i is bit
    // i of row j, a word already built above.
    for (int i = 64 + wave; i < M; i += kStructWaves) {
        for (int w = 0; w < (i >> 6); ++w) {
            const int j = 64 * w + lane;
            const bool hit = (adj[(size_t)j * W + (i >> 6)] >> (i & 63)) & 1ull;
            const uint64_t m = __ballot(hit);
            if (lane == 0) adj[(size_t)i * W + w] = m;
        }
    }
    __syncthreads();
    // Wavefront 1 takes Eq. 6 while wavefront 0 takes the clusters; all meet
    // once more at the end.
    __shared__ double s_cos[3];
    if (wave > 1) {
        __syncthreads();
        return;
    }
    if (wave == 1) {
        // Eq. 6: <cos^2> of the head-to-centre bonds along each axis.
        double cx = 0.0, cy = 0.0, cz = 0.0;
        for (int l = lane; l < M; l += 64) {
            double d[3];
            st_diff(xs + 9 * l, xs + 9 * l + 3, box, half, d);
            const double r2 = st_r2(d);
            cx += d[0] * d[0] / r2;
            cy += d[1] * d[1] / r2;
            cz += d[2] * d[2] / r2;
        }
        cx = wave_sum(cx);
        cy = wave_sum(cy);
        cz = wave_sum(cz);
        if (lane == 0) {
            s_cos[0] = cx;
            s_cos[1] = cy;
            s_cos[2] = cz;
        }
        __syncthreads();
        return;
    }

    // Clusters.  Visited set, frontier and finds are bit masks held by the whole
    // wavefront.  Lipids without contacts are clusters of one, all at once; the
    // others are grown breadth first from their lowest free lipid, only to know
    // their size.
    constexpr bool kRegs = NW <= 4;
    uint64_t rows[kRegs ? NW : 1][kRegs ? NW : 1];
    auto row = [&](int w, int v) -> uint64_t {
        if constexpr (kRegs) return rows[w][v];
        else return v < W && 64 * w + lane < M ? adj[(size_t)(64 * w + lane) * W + v] : 0ull;
    };
    if constexpr (kRegs) {
#pragma unroll
        for (int w = 0; w < NW; ++w)
#pragma unroll
            for (int v = 0; v < NW; ++v)
                rows[w][v] = v < W && 64 * w + lane < M ? adj[(size_t)(64 * w + lane) * W + v] : 0ull;
    }
    uint64_t free_[NW], front[NW];
    int ncl = 0, best_root = 0, best_size = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int left = M - 64 * w;   // lipids in word w
        free_[w] = left >= 64 ? ~0ull : (left <= 0 ? 0ull : (1ull << left) - 1ull);
        uint64_t any = 0ull;
#pragma unroll
        for (int v = 0; v < NW; ++v) any |= row(w, v);
        const uint64_t alone = __ballot(any == 0ull) & free_[w];
        if (alone && best_size == 0) {
            best_size = 1;
            best_root = 64 * w + (int)__builtin_ctzll(alone);
        }
        ncl += __builtin_popcountll(alone);
        free_[w] &= ~alone;
    }
    // one level: the free lipids that touch the frontier
    auto grow = [&](uint64_t *found) -> int {
        int n = 0;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            uint64_t t = 0ull;
#pragma unroll
            for (int v = 0; v < NW; ++v) t |= row(w, v) & front[v];
            found[w] = __ballot(t != 0ull) & free_[w];
            n += __builtin_popcountll(found[w]);
        }
        return n;
    };
    auto start_at = [&](int r) {
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            front[w] = w == (r >> 6) ? 1ull << (r & 63) : 0ull;
            free_[w] &= ~front[w];
        }
    };
    for (;;) {
        int r = -1;
#pragma unroll
        for (int w = NW - 1; w >= 0; --w)
            if (free_[w]) r = 64 * w + (int)__builtin_ctzll(free_[w]);
        if (r < 0) break;
        ++ncl;
        start_at(r);
        int size = 1;
        for (;;) {
            uint64_t found[NW];
            const int n = grow(found);
            if (n == 0) break;
            size += n;
#pragma unroll
            for (int w = 0; w < NW; ++w) {
                front[w] = found[w];
                free_[w] &= ~found[w];
            }
        }
        if (size > best_size) {
            best_size = size;
            best_root = r;
        }
    }

    // The largest cluster again, with the tree that unfolds it: level and the
    // lowest touching lipid of the level before.
    int level[NW], parent[NW], depth = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int left = M - 64 * w;
        free_[w] = left >= 64 ? ~0ull : (left <= 0 ? 0ull : (1ull << left) - 1ull);
        level[w] = 64 * w + lane == best_root ? 0 : -1;
        parent[w] = -1;
    }
    start_at(best_root);
    for (;;) {
        uint64_t found[NW];
        if (grow(found) == 0) break;
        ++depth;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            if ((found[w] >> lane) & 1ull) {
                level[w] = depth;
#pragma unroll
                for (int v = NW - 1; v >= 0; --v) {
                    const uint64_t t = row(w, v) & front[v];
                    if (t) parent[w] = 64 * v + (int)__builtin_ctzll(t);
                }
            }
        }
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            front[w] = found[w];
            free_[w] &= ~found[w];
        }
    }

    // Unfolding.  First, for all lipids at once, the bead a lipid is placed by
    // (through its first touching tail pair; the root by its stored head), its
    // difference from the parent's bead, and its bonds: to u, from which a lipid
    // is then placed, level after level, by additions alone.
    int hang[NW];   // 4 parent bead + own bead
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        hang[w] = 0;
        const int j = 64 * w + lane;
        if (level[w] < 0) continue;
        const float *xj = xs + 9 * j;
        double *uj = u + 9 * j;
        double d[3], to_head[3], to_end[3];   // from the centre bead
        st_diff(xj + 3, xj, box, half, to_head);
        st_diff(xj + 3, xj + 6, box, half, to_end);
        int bb = 0;
        if (level[w] == 0) {
            for (int a = 0; a < 3; ++a) d[a] = (double)xj[a];
        } else {
            const float *xi = xs + 9 * parent[w];
            for (int pr = 3; pr >= 0; --pr) {   // the first that touches is written last
                double e[3];
                const int ba = 1 + (pr >> 1), b2 = 1 + (pr & 1);
                st_diff(xi + 3 * ba, xj + 3 * b2, box, half, e);
                if (st_r2(e) < kTailContact2) {
                    bb = b2;
                    hang[w] = 4 * ba + b2;
                    for (int a = 0; a < 3; ++a) d[a] = e[a];
                }
            }
        }
        for (int a = 0; a < 3; ++a) {
            // bead bb: its difference; the beads along the chain from it: the bond
            uj[a] = bb == 0 ? d[a] : to_head[a];
            uj[3 + a] = bb == 1 ? d[a] : (bb == 0 ? -to_head[a] : -to_end[a]);
            uj[6 + a] = bb == 2 ? d[a] : to_end[a];
        }
    }
    wave_sync();
    for (int k = 0; k <= depth; ++k) {
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            if (level[w] != k) continue;
            double *uj = u + 9 * (64 * w + lane);
            const int bb = hang[w] & 3;
            const double *ui = u + 9 * (k == 0 ? 0 : parent[w]) + 3 * (hang[w] >> 2);
            for (int a = 0; a < 3; ++a) {
                double h = uj[a], c0 = uj[3 + a], t = uj[6 + a];
                const double at = k == 0 ? 0.0 : ui[a];
                if (bb == 0) {
                    h = k == 0 ? h : at + h;
                    c0 = h + c0;
                    t = c0 + t;
                } else if (bb == 1) {
                    c0 = at + c0;
                    h = c0 + h;
                    t = c0 + t;
                } else {
                    t = at + t;
                    c0 = t + c0;
                    h = c0 + h;
                }
                uj[a] = h;
                uj[3 + a] = c0;
                uj[6 + a] = t;
            }
        }
        wave_sync();
    }

    // Eq. 7 over the 3 x best_size beads, then Eq. 8.
    double s[3] = {0.0, 0.0, 0.0};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        if (level[w] < 0) continue;
        for (int b = 0; b < 3; ++b)
            for (int a = 0; a < 3; ++a) s[a] += u[9 * (64 * w + lane) + 3 * b + a];
    }
    const double n = 3.0 * (double)best_size;
    double com[3], q[3];
    for (int a = 0; a < 3; ++a) com[a] = wave_sum(s[a]) / n;
    for (int a = 0; a < 3; ++a) s[a] = 0.0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        if (level[w] < 0) continue;
        for (int b = 0; b < 3; ++b)
            for (int a = 0; a < 3; ++a) {
                const double e = u[9 * (64 * w + lane) + 3 * b + a] - com[a];
                s[a] += e * e;
            }
    }
    for (int a = 0; a < 3; ++a) q[a] = wave_sum(s[a]) / n;
    __syncthreads();
    const double cx = s_cos[0], cy = s_cos[1], cz = s_cos[2];

    if (lane == 0) {
        const double sx = 1.5 * (cx / (double)M) - 0.5;
        const double sy = 1.5 * (cy / (double)M) - 0.5;
        const double sz = 1.5 * (cz / (double)M) - 0.5;
        double smax = sx;
        int axis = 0;
        if (sy > smax) { smax = sy; axis = 1; }
        if (sz > smax) { smax = sz; axis = 2; }
        const double tr = q[0] + q[1] + q[2];
        const double lam = tr / 3.0;
        const double e0 = q[0] - lam, e1 = q[1] - lam, e2 = q[2] - lam;
        const double num = e0 * e0 * e0 + e1 * e1 * e1 + e2 * e2 * e2;
        rec[0] = smax;
        rec[1] = (double)axis;
        rec[2] = (double)ncl;
        rec[3] = (double)best_size;
        rec[4] = q[0];
        rec[5] = q[1];
        rec[6] = q[2];
        rec[7] = 9.0 * num / (tr * tr * tr);
    }
}

// H(E, O) of the lipid model at a sync point (Sec. 3.2), one thread per
// walker, from the record just computed: O = lipids in the largest cluster
// (field 3), O bin O obs_bins / (nlip + 1); or, for a floating-point field v,
// O = its bin floor((v - lo) / (hi - lo) * obs_bins) held to [0, obs_bins).
// The sample goes to the walker's energy bin within its window (each walker
// owns its cells: no atomics).
__global__ __launch_bounds__(64) void k_measure_lipid(DevState st) {
    const int w = blockIdx.x * blockDim.x + threadIdx.x;
    if (w >= st.nw || *st.converged) return;
    const int b = st.E[w] - st.start[w / st.m];
    if (b < 0 || b >= st.W) return;
    int O, ob;
    if (st.obs_field == 3) {
        const double v = st.obs_rec[(size_t)w * 8 + 3];
        if (!(v >= 1.0 && v <= (double)st.nmol)) return;   // only a NaN record (never in a run)
        O = (int)v;
        ob = (int)(((long long)O * st.obs_bins) / (st.nmol + 1));
    } else {
        const double v = st.obs_rec[(size_t)w * 8 + st.obs_field];
        const double t = (v - st.obs_lo) / (st.obs_hi - st.obs_lo) * (double)st.obs_bins;
        O = t >= 0.0 ? (t < (double)st.obs_bins ? (int)t : st.obs_bins - 1) : 0;
        ob = O;
    }
    const size_t cell = (size_t)w * st.Wpad + b;
    st.obs_hist[cell * st.obs_bins + ob] += 1u;
    st.obs_sum[cell] += (unsigned long long)O;
    st.obs_cnt[cell] += 1u;
}

}  // namespace

size_t lipid_structure_lds_bytes(int M) {
    const size_t W = (size_t)(M + 63) / 64;
    return (size_t)M * 16 + (size_t)M * W * 8 + (size_t)M * 72 + (size_t)M * 36;
}

hipError_t launch_lipid_structure(const void *coords, size_t xstride, const void *lipids, size_t lstride, int nconf,
                                  int np, int M, float box, double *out, hipStream_t s) {
    const size_t lds = lipid_structure_lds_bytes(M);
    auto go = [&](auto kernel) -> hipError_t {
        if (lds > 48 * 1024) {   // with margin for the kernel's own static LDS
            const hipError_t e = hipFuncSetAttribute((const void *)kernel,
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
            if (e != hipSuccess) return e;
        }
        hipLaunchKernelGGL(kernel, dim3(nconf), dim3(64 * kStructWaves), lds, s, (const unsigned char *)coords,
                           xstride, (const unsigned char *)lipids, lstride, np, M, box, out);
        return hipGetLastError();
    };
    if (M <= 64) return go(k_lipid_structure<1>);
    if (M <= 128) return go(k_lipid_structure<2>);
    if (M <= 256) return go(k_lipid_structure<4>);
    return go(k_lipid_structure<8>);
}

hipError_t launch_lipid_measure(const DevState &st, hipStream_t s) {
    const unsigned char *rows = (const unsigned char *)st.spins;
    hipError_t e = launch_lipid_structure(rows, (size_t)st.Npad, rows + st.lip_off_lip, (size_t)st.Npad, st.nw, st.nb,
                                          st.nmol, st.box, st.obs_rec, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_measure_lipid, dim3((unsigned)((st.nw + 63) / 64)), dim3(64), 0, s, st);
    return hipGetLastError();
}

}  // namespace rewl_gpu

using rewl_host::fail;

static int check_structure_args(int nconf, int np, int nlip, float box) {
    if (nconf < 0) return fail(REWL_EINVAL, "nconf must be >= 0");
    if (nlip < 1 || nlip > rewl_gpu::kStructMaxLipids) return fail(REWL_EINVAL, "nlip must be in [1, 512]");
    if (np < 3 * nlip) return fail(REWL_EINVAL, "np must be >= 3 nlip");
    if (!(box > 0.0f) || !(box < 1e30f)) return fail(REWL_EINVAL, "box must be positive and finite");
    return REWL_OK;
}

extern "C" int rewl_lipid_structure(const float *coords, size_t coord_stride, const int32_t *lipids,
                                    size_t lipid_stride, int nconf, int np, int nlip, float box, double *out,
                                    void *hip_stream) {
    int st = check_structure_args(nconf, np, nlip, box);
    if (st != REWL_OK) return st;
    if (nconf == 0) return REWL_OK;
    if (!coords || !lipids || !out) return fail(REWL_EINVAL, "null pointer");
    if (((uintptr_t)coords & 3) || ((uintptr_t)lipids & 3) || ((uintptr_t)out & 7) || (coord_stride & 3) ||
        (lipid_stride & 3))
        return fail(REWL_EINVAL, "coords and lipids must be 4-byte aligned (strides too), out 8-byte aligned");
    if (nconf > 1 && (coord_stride < (size_t)12 * np || lipid_stride < (size_t)12 * nlip))
        return fail(REWL_EINVAL, "strides smaller than one configuration");
    HIP_TRY(rewl_gpu::launch_lipid_structure(coords, coord_stride, lipids, lipid_stride, nconf, np, nlip, box, out,
                                             (hipStream_t)hip_stream));
    return REWL_OK;
}

extern "C" int rewl_lipid_obs_field(rewl_t *r, int field, double lo, double hi) {
    if (!r) return fail(REWL_EINVAL, "null handle");
    rewl_gpu::DevState &d = r->st;
    if (d.model != rewl_gpu::kModelLipid3D) return fail(REWL_EINVAL, "not a run of the lipid model");
    if (d.obs_bins <= 0) return fail(REWL_EINVAL, "the run samples no observable (opts.obs_bins = 0)");
    if (field == 3) {
        d.obs_field = 3;
        d.obs_lo = d.obs_hi = 0.0;
        return REWL_OK;
    }
    if (field != 0 && (field < 4 || field > 7)) return fail(REWL_EINVAL, "field must be 0, 3, 4, 5, 6 or 7");
    if (!(lo > -1e300 && hi < 1e300 && hi > lo)) return fail(REWL_EINVAL, "need finite lo < hi");
    d.obs_field = field;
    d.obs_lo = lo;
    d.obs_hi = hi;
    return REWL_OK;
}

// Record buffer of rewl_structure_noalloc: a file-scope device array (one
// copy on every GPU the library runs on, held until the process ends) for
// callers that cannot allocate device memory.  Host code never passes the
// array's name to a kernel: it takes the device address of each GPU's copy
// once, with that GPU current, and passes that address.
constexpr int kNoallocMaxWalkers = 4096;
static __device__ __align__(256) double scratch[kNoallocMaxWalkers * 8];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
double *g_scratch_ptr[kMaxDevices] = {};

// Device address of GPU `dev`'s copy of `scratch`.
int scratch_on(int dev, double **out) {
    if (dev < 0 || dev >= kMaxDevices) return fail(REWL_EDEVICE, "device index beyond the record buffers kept");
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        int cur = 0;
        HIP_TRY(hipGetDevice(&cur));
        if (cur != dev) HIP_TRY(hipSetDevice(dev));
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (cur != dev) HIP_TRY(hipSetDevice(cur));
        if (e != hipSuccess || !p)
            return fail(REWL_EDEVICE, std::string("hipGetSymbolAddress(scratch): ") + hipGetErrorString(e));
        g_scratch_ptr[dev] = (double *)p;
    }
    *out = g_scratch_ptr[dev];
    return REWL_OK;
}
}  // namespace

extern "C" int rewl_structure_noalloc(rewl_t *r, double *out) {
    if (!r || !out) return fail(REWL_EINVAL, "null argument");
    const rewl_gpu::DevState &d = r->st;
    if (d.model != rewl_gpu::kModelLipid3D) return fail(REWL_EINVAL, "not a run of the lipid model");
    int st = check_structure_args(d.nw, d.nb, d.nmol, d.box);
    if (st != REWL_OK) return st;
    if (d.nw > kNoallocMaxWalkers)
        return fail(REWL_EINVAL, "more than 4096 walkers: the static record buffer holds 4096 records");
    int dev = 0;
    HIP_TRY(hipStreamGetDevice(r->stream, &dev));
    double *buf = nullptr;
    st = scratch_on(dev, &buf);
    if (st != REWL_OK) return st;
    const size_t bytes = (size_t)d.nw * 8 * sizeof(double);
    HIP_TRY(rewl_gpu::launch_lipid_structure(d.spins, (size_t)d.Npad, (const unsigned char *)d.spins + d.lip_off_lip,
                                             (size_t)d.Npad, d.nw, d.nb, d.nmol, d.box, buf, r->stream));
    HIP_TRY(hipMemcpyAsync(out, buf, bytes, hipMemcpyDeviceToHost, r->stream));
    HIP_TRY(hipStreamSynchronize(r->stream));
    return REWL_OK;
}

extern "C" int rewl_structure(rewl_t *r, double *out) {
    if (!r || !out) return fail(REWL_EINVAL, "null argument");
    const rewl_gpu::DevState &d = r->st;
    if (d.model != rewl_gpu::kModelLipid3D) return fail(REWL_EINVAL, "not a run of the lipid model");
    int st = check_structure_args(d.nw, d.nb, d.nmol, d.box);
    if (st != REWL_OK) return st;
    double *dev = nullptr;
    const size_t bytes = (size_t)d.nw * 8 * sizeof(double);
    HIP_TRY(hipMalloc((void **)&dev, bytes));
    hipError_t e = rewl_gpu::launch_lipid_structure(d.spins, (size_t)d.Npad, (const unsigned char *)d.spins + d.lip_off_lip,
                                                    (size_t)d.Npad, d.nw, d.nb, d.nmol, d.box, dev, r->stream);
    if (e == hipSuccess) e = hipMemcpyAsync(out, dev, bytes, hipMemcpyDeviceToHost, r->stream);
    if (e == hipSuccess) e = hipStreamSynchronize(r->stream);
    (void)hipFree(dev);
    if (e != hipSuccess) return fail(REWL_EDEVICE, std::string("structure kernel: ") + hipGetErrorString(e));
    return REWL_OK;
}

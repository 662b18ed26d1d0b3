// rewl_moves.h -- main-phase attempts of the continuous models (trimer,
// lipid): blocks of consecutive displacement attempts evaluated side by side.
//
// The attempts of a walker are a strict sequence, but the energy change of an
// attempt depends on the attempts before it only through the particles they
// moved.  Energies are exact integer sums of pair terms, so that dependence
// can be added afterwards: one wavefront per attempt evaluates its change
// against the configuration at the start of the block, together with the
// correction c[l][i] the change of attempt l takes if attempt i < l is
// accepted,
//   c = V(n_l, n_i) - V(o_l, n_i) - V(n_l, o_i) + V(o_l, o_i)
// (o, n: old and new place of the moved particle).  Wavefront 0 then decides
// the attempts in order.  An attempt on a particle that an earlier attempt of
// the block has moved ends the block before it: its proposal starts from
// another place.
//
// Hard overlaps (terms outside the fixed-point range) count as 0 in the sums
// and are counted on the side: an attempt is refused if one is left among its
// new pairs, the corrections of the count being one bit per earlier attempt
// each for (n_l, n_i) and (n_l, o_i).  V(o, .) terms of the configuration
// itself are never hard overlaps, and V(o_l, n_i) can be one only if attempt
// i is refused.
//
// A wavefront screens its partners 64 at a time on places rounded down to box
// / 65536 and held as 16-bit integers: the differences wrap at the periodic
// boundary by themselves and two 16-bit dot products give the squared distance,
// 5 operations where the binary32 minimum image takes 13; the next 64 places
// are on their way meanwhile.  Partners within the cut-off plus the length of
// the move of the old place go to a list in LDS, and the pair energies
// (binary64 divisions and roots) are evaluated for the list alone, 32 partners
// x 2 places per pass.  In the N = 1000 lipid system 6% of the partners pass
// the screen.
//
// Decisions go from one accepted attempt to the next, all lanes at once, the
// corrections in registers (a lane's 16, the column by a uniform index).
//
// Measured on 64 walkers (one workgroup each), us per attempt of a walker:
// 64 trimers 1.45 -> 0.49 (six wavefronts sharing the partners of one attempt
// before), N = 1000 lipids 4.06 -> 1.18 (sixteen).  A block of 14.5 trimer
// attempts takes 1,350 cycles of proposals, 7,100 of evaluation (VALU issue,
// four wavefronts per SIMD, 76% busy) and 5,050 of decisions (one wavefront,
// 6.7 accepted attempts; 8,000 with a read of the correction table and the
// bin paid in the chain of each); one of 11.9 lipid attempts 2,650, 13,700
// (14,300 with the partners that a bond or the bead itself rules out tested in
// the screen) and 6,750, and every second block a reptation, 17,100.
#pragma once

#include "rewl_device.h"

namespace rewl_gpu {

constexpr int kMoveMaxWaves = 16;
constexpr int kMoveList = 96;    // list entries of a wavefront: at most 31 left over plus 64 of a chunk

// Row of one attempt of a block, written by its wavefront.
struct MoveRow {
    int64_t de;        // energy change against the block-start configuration
    uint32_t bad;      // bits 0-15: (n_l, n_i) is a hard overlap; bits 16-31: (n_l, o_i) is one
    uint32_t same;     // earlier attempts on the same particle
    int32_t nbad;      // hard overlaps against the block-start configuration
    int32_t pad;
};
// Proposal of one attempt of a block, written by wavefront 0.
struct MoveProp {
    float n[3], reach;   // new place; length of the move plus rounding slack
    float o[3];
    int b;
};

// A place on the 16-bit grid of the periodic box, x and y in one word, z in
// the other.  scale = 65536 / box; a coordinate at the upper edge wraps to 0.
struct MoveGrid {
    uint32_t xy, z;
};
typedef short move_s2 __attribute__((ext_vector_type(2)));
__host__ __device__ __forceinline__ MoveGrid move_grid(const float *x, float scale) {
    MoveGrid g;
    g.xy = ((uint32_t)(x[0] * scale) & 0xffffu) | ((uint32_t)(x[1] * scale) << 16);
    g.z = (uint32_t)(x[2] * scale) & 0xffffu;
    return g;
}
// Squared distance in grid units (below 2^32: each axis is at most 32768).
__device__ __forceinline__ uint32_t move_grid2(MoveGrid a, MoveGrid b) {
    const move_s2 dxy = __builtin_bit_cast(move_s2, a.xy) - __builtin_bit_cast(move_s2, b.xy);
    const move_s2 dz = __builtin_bit_cast(move_s2, a.z) - __builtin_bit_cast(move_s2, b.z);
    return (uint32_t)__builtin_amdgcn_sdot2(dz, dz, __builtin_amdgcn_sdot2(dxy, dxy, 0, false), false);
}
// Square of a radius in grid units that no pair within the radius exceeds: the
// places are rounded down, which moves a difference by less than a unit an axis
// and a distance by less than sqrt(3) = 1.732; the binary32 products add less
// than 0.02, and the conversion drops less than 1.
__host__ __device__ __forceinline__ uint32_t move_grid_limit(float r, float scale) {
    const float u = r * scale + 3.0f;
    const uint32_t v = u < 65535.0f ? (uint32_t)u : 65535u;
    return v * v;
}

// b - a moved by -+box when beyond +-box/2, in binary32.
__host__ __device__ __forceinline__ double move_image(float a, float b, float box, float half) {
#pragma clang fp contract(off)
    const float x = b - a;
    const float y = x - __builtin_copysignf(box, x);
    return (double)(fabsf(x) > half ? y : x);
}
__host__ __device__ __forceinline__ double move_r2(const float *a, const float *b, float box, float half) {
#pragma clang fp contract(off)
    const double dx = move_image(a[0], b[0], box, half);
    const double dy = move_image(a[1], b[1], box, half);
    const double dz = move_image(a[2], b[2], box, half);
    return (dx * dx + dy * dy) + dz * dz;
}

// Binary32 rounding of places and distances, a few units of box 2^-24, and more.
__host__ __device__ __forceinline__ float move_slack(float box) { return 1e-3f + box * 1e-6f; }
// Distance between the old and the new place of a displacement, with slack.
__host__ __device__ __forceinline__ float move_reach(float d0, float d1, float d2, float box) {
    return __builtin_sqrtf(d0 * d0 + d1 * d1 + d2 * d2) + move_slack(box);
}

// Entries of the correction table of `waves` wavefronts: their rows, and room
// for the entries read behind the last one.
__host__ __device__ inline int move_table(int waves) { return waves * waves + kMoveMaxWaves; }
// LDS behind the walker's state, ln g and H: block header, rows, proposals,
// correction table and lists of `waves` wavefronts.
__host__ __device__ inline size_t move_lds_bytes(int waves) {
    return (size_t)waves * (sizeof(MoveRow) + sizeof(MoveProp) + kMoveList * 2) + (size_t)move_table(waves) * 8 + 64;
}
// Workgroup of a walker beside `used` bytes of LDS (state, ln g, H, the model's
// own) and `per_wave` more of the model for each wavefront.
//
// Sixteen wavefronts are fastest for one walker a CU of 64 particles or more
// and fill the CU's registers.  Fewer where they would do less or wait longer:
// * blocks of few particles end early, on a particle that has moved;
// * several walkers a CU run side by side, and one decides while another
//   evaluates, if they have 16 wavefronts between them and the LDS holds them.
// us per 1,000 attempts of every walker (300 for the lipids) with 16, 8, 4, 2
// wavefronts, and with 6 (lipids 16) sharing the partners of one attempt:
//   16 trimers,    64 walkers    708   661   857  1291   1247
//   32 trimers,    64            597   624   850  1317   1339
//   64 trimers,   512            909   716   934  1467   1772
//   64 trimers, 1,024           1778  1352  1193  1583   3143
//   64 trimers, 2,048           3347  2471  2122  2020   6210
//    4 trimers, 1,024           4636  2340  1437  1637   1984
//   N = 1000 lipids,   512       798   608   767  1239   2311
//   N = 1000 lipids, 1,024      1494  1117   974  1300   4547
// The 16-bit places (8 bytes a particle) are kept where they fit, else taken
// from the coordinates each time (three conversions more per partner); then
// the wavefronts are halved until the LDS holds them.
struct MovePlan {
    int waves, grid;
    size_t lds;
};
inline MovePlan move_plan(size_t used, size_t per_wave, int particles, int walkers) {
    constexpr int kCUs = 256;
    auto bytes = [&](int k, int grid) {
        return used + k * per_wave + move_lds_bytes(k) + (grid ? (size_t)particles * sizeof(MoveGrid) : 0);
    };
    const int per_cu = (walkers + kCUs - 1) / kCUs;
    int most = kMoveMaxWaves;
    while (most > 2 && kMoveMaxWaves / most < per_cu && kLdsBytes / bytes(most, 1) > (size_t)(kMoveMaxWaves / most)) most /= 2;
    const int few = particles < 64 ? 8 : kMoveMaxWaves;
    const int first = few < most ? few : most;
    for (int k = first; k >= 1; k /= 2)
        for (int grid = k == first ? 1 : 0; grid >= 0; --grid)
            if (bytes(k, grid) <= kLdsBytes || (k == 1 && !grid)) return MovePlan{k, grid, bytes(k, grid)};
    return MovePlan{1, 0, 0};
}

// Energy bin as fx_bin gives it: the binary64 quotient's floor is exact
// unless its fraction lies within 2^-20 of an integer (the estimate is off by
// less than 2^-50 |q|, 2^-30 of a bin for |q| < 2^20); a lane in that case, or
// beyond 2^20 bins, sends the wavefront through fx_bin.
__device__ __forceinline__ int move_bin(const DevState &st, int64_t e) {
#pragma clang fp contract(off)
    const double qd = (double)(e - st.emin_fx) * st.binw_inv;
    const double fl = __builtin_floor(qd);
    const double fr = qd - fl;
    int bin = (int)fl;
    if (__ballot(!(fabs(qd) < 0x1p20 && fr > 0x1p-20 && fr < 1.0 - 0x1p-20)))
        bin = fx_bin(st.emin_fx, st.binw_fx, st.binw_inv, e);
    return bin;
}

__device__ __forceinline__ int move_mbcnt(unsigned long long m) {
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}
// Orders this wavefront's LDS writes before its later LDS reads by other lanes.
__device__ __forceinline__ void move_wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}
__device__ __forceinline__ int64_t move_readlane64(int64_t v, int l) {
    const uint32_t lo = __builtin_amdgcn_readlane((uint32_t)v, l);
    const uint32_t hi = __builtin_amdgcn_readlane((uint32_t)((uint64_t)v >> 32), l);
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int64_t move_uniform64(int64_t v) {
    const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v);
    const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)((uint64_t)v >> 32));
    return (int64_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ double move_readlane_d(double v, int l) {
    return __longlong_as_double(move_readlane64(__double_as_longlong(v), l));
}
__device__ __forceinline__ float move_readlane_f(float v, int l) {
    return __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(v), l));
}
__device__ __forceinline__ uint32_t move_perm(uint32_t v, int l) {
    return (uint32_t)__builtin_amdgcn_ds_bpermute(l << 2, (int)v);
}

// Displacement of one axis: 0.1 (2u - 1), u a 23-bit uniform; periodic wrap.
__host__ __device__ __forceinline__ float move_disp(uint32_t r) {
#pragma clang fp contract(off)
    return 0.1f * ((float)(r >> 9) * 0x1p-22f - 1.0f);
}
__host__ __device__ __forceinline__ float move_wrap(float v, float box) {
#pragma clang fp contract(off)
    if (v < 0.0f) v = v + box;
    if (v >= box) v = v - box;
    return v;
}

// Wavefront l's share of a block: the energy change of attempt l against the
// block-start configuration and its corrections for the attempts before it.
template <class Model>
__device__ __forceinline__ void move_evaluate(const DevState &st, const Model &md, const MoveProp *props, int l,
                                              int waves, MoveRow *rows, int64_t *tab, uint16_t *list, int lane) {
#pragma clang fp contract(off)
    const float box = st.box;
    const MoveProp p = props[l];
    const int b = __builtin_amdgcn_readfirstlane(p.b);
    int64_t acc = 0;
    int nbad = 0;
    int p0 = -1, p1 = -1;
    int cnt = md.bonds(b, p0, p1);
    if (lane == 0) {
        list[0] = (uint16_t)(p0 | 0x8000);
        list[1] = (uint16_t)(p1 | 0x8000);
    }
    // one pass over the last n <= 32 list entries: lane = 2 entry + place
    auto pass = [&](int n) {
        move_wave_sync();
        if ((lane >> 1) < n) {
            const uint32_t ent = list[cnt - n + (lane >> 1)];
            const int j = (int)(ent & 0x7fffu);
            const bool old = lane & 1, bond = (ent & 0x8000u) != 0;
            const float q[3] = {old ? p.o[0] : p.n[0], old ? p.o[1] : p.n[1], old ? p.o[2] : p.n[2]};
            int64_t t = 0;
            const bool ok = fx_term(md.pair(b, j, q, md.x + 3 * j, bond), t);
            // the screen lets the bead itself and its bonded partners through
            const bool skip = !bond && (j == b || j == p0 || j == p1);
            nbad += (int)(!ok && !skip);
            acc += skip ? 0 : (old ? -t : t);
        }
        cnt -= n;
        move_wave_sync();
    };
    // screen: partners near the old place
    const float scale = md.scale;
    const MoveGrid go = move_grid(p.o, scale);
    const uint32_t far2 = move_grid_limit(2.5f + p.reach, scale);
    const uint32_t near2 = Model::kHeads ? move_grid_limit(1.1225f + p.reach, scale) : 0u;
    int r3 = lane % 3;                      // j mod 3
    const bool tail = b % 3 != 0;
    auto place = [&](int j) -> MoveGrid { return Model::kGrid ? md.grid[j] : move_grid(md.x + 3 * j, scale); };
    bool real = lane < st.nb;
    MoveGrid ahead = place(real ? lane : 0);
    for (int c = 0; c < st.nb; c += 64) {
        const MoveGrid gj = ahead;          // the next chunk's places are read while this one is screened
        uint32_t lim = far2;
        if constexpr (Model::kHeads) {
            lim = tail && r3 != 0 ? far2 : near2;
            r3 = r3 == 2 ? 0 : r3 + 1;      // 64 mod 3 = 1
        }
        const unsigned long long m = __ballot(move_grid2(gj, go) <= lim) & __ballot(real);
        const int jn = c + 64 + lane;
        real = jn < st.nb;
        ahead = place(real ? jn : 0);
        if (__builtin_amdgcn_inverse_ballot_w64(m)) list[cnt + move_mbcnt(m)] = (uint16_t)(c + lane);
        cnt += __builtin_popcountll(m);
        while (cnt >= 32) pass(32);
    }
    if (cnt) pass(cnt);
    // corrections: lane = 16 role + i, roles (n_l, n_i), (o_l, n_i), (n_l, o_i), (o_l, o_i)
    const int i = lane & 15, role = lane >> 4;
    int64_t c = 0;
    bool same = false, bad = false, close = false;
    MoveProp pi{};
    if (i < l) {
        pi = props[i];
        same = pi.b == b;
        // reach of both moves, or a bond, which may be longer than any cut-off
        close = !same && (move_grid2(move_grid(pi.o, scale), go) <= move_grid_limit(2.5f + p.reach + pi.reach, scale) ||
                          pi.b == p0 || pi.b == p1);
    }
    const unsigned long long samem = __ballot(same);
    if (__ballot(close)) {
        if (close) {
            const bool oldl = role & 1, oldi = role & 2;
            const float q[3] = {oldl ? p.o[0] : p.n[0], oldl ? p.o[1] : p.n[1], oldl ? p.o[2] : p.n[2]};
            const float qi[3] = {oldi ? pi.o[0] : pi.n[0], oldi ? pi.o[1] : pi.n[1], oldi ? pi.o[2] : pi.n[2]};
            int64_t t = 0;
            bad = !fx_term(md.pair(b, pi.b, q, qi, pi.b == p0 || pi.b == p1), t);
            c = (role == 0 || role == 3) ? t : -t;
        }
        c += __shfl_xor(c, 16, 64);
        c += __shfl_xor(c, 32, 64);
    }
    if (lane < l) tab[l * waves + lane] = c;
    const unsigned long long badm = __ballot(bad);
    const int64_t de = wave_sum64(acc);
    // the lanes' overlap counts (new places only can have one)
    int over = 0;
    if (__ballot(nbad != 0)) over = (int)wave_sum64((int64_t)nbad);
    if (lane == 0) {
        MoveRow r;
        r.de = de;
        r.bad = (uint32_t)(badm & 0xffffull) | ((uint32_t)(badm >> 32) << 16);
        r.same = (uint32_t)(samem & 0xffffull);
        r.nbad = over;
        r.pad = 0;
        rows[l] = r;
    }
}

// Lane `lane`'s corrections for attempts 0 .. 15 of a block (those for itself
// and later ones, and of lanes past the block, are never looked at).
typedef long long move_l16 __attribute__((ext_vector_type(16)));
template <class Table>
__host__ __device__ __forceinline__ move_l16 move_corrections(Table tab, int lane, int waves) {
    const int row = (lane < waves ? lane : waves - 1) * waves;
    move_l16 corr;
#pragma unroll
    for (int r = 0; r < kMoveMaxWaves; ++r) corr[r] = tab[row + r];
    return corr;
}

// Attempts s0 .. s0+n-1 of walker w (Sec. 2): propose, reject a new bin
// outside the window, else accept with min[1, g(old)/g(new)]; then
// ln g += ln f and H += 1 at the bin after the decision.  `waves` wavefronts
// (a power of two, at most 16) of one workgroup; mv: move_lds_bytes(waves)
// of LDS; words of attempt t: Philox blocks (t, w, MOVE) and (t, w, MOVE_U).
template <class Model, int PREC>
__device__ __forceinline__ void move_sweep(const DevState &st, Model &md, int w, int64_t s0, int64_t n, double *g,
                                           float *gh, float *gl, uint32_t *H, unsigned char *mv) {
#pragma clang fp contract(off)
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int waves = (int)(blockDim.x >> 6);
    MoveRow *rows = (MoveRow *)mv;
    MoveProp *props = (MoveProp *)(rows + waves);
    int64_t *tab = (int64_t *)(props + waves);
    uint32_t *head = (uint32_t *)(tab + move_table(waves));   // [16]: attempts of the block, kind, words
    uint16_t *list = (uint16_t *)(head + 16) + wave * kMoveList;

    const int k = w / st.m;
    const int lo = st.start[k], W = st.W;
    const double lnf = st.lnf[k];
    const float lnf32 = (float)lnf;
    const float box = st.box;
    int E = __builtin_amdgcn_readfirstlane(st.E[w]);
    int64_t Ef = move_uniform64(st.Efx[w]);
    // wavefront 0: words of attempts base .. base+63, one per lane, and ln u
    U4 la{}, lu{};
    double lnu_b = 0.0;
    int64_t t = 0;         // attempts done
    int64_t base = 0;      // attempt of lane 0's words
    bool drawn = false;
    int nblk = 0;
    float nx = 0.0f, ny = 0.0f, nz = 0.0f;
    int bead = 0;
    uint32_t uw = 0;
    double lnu = 0.0;
    if constexpr (Model::kGrid) {
        for (int j = threadIdx.x; j < st.nb; j += blockDim.x) md.grid[j] = move_grid(md.x + 3 * j, md.scale);
    }
    for (;;) {
        if (wave == 0) {
            // ---- proposals of the next block, attempt t + lane on lane `lane`
            if (!drawn || (t - base > 64 - waves && base + 64 < n)) {
                base = t;
                drawn = true;
                const uint64_t a = (uint64_t)(s0 + base + lane);
                la = philox10((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)w, st.ctr3 | (kDomMove << 24), st.key0, st.key1);
                lu = philox10((uint32_t)a, (uint32_t)(a >> 32), (uint32_t)w, st.ctr3 | (kDomMoveU << 24), st.key0, st.key1);
                if (PREC == 0) lnu_b = lu.x == 0u ? -64.0 : log((double)lu.x * 0x1p-32);
                else lnu_b = (lu.x >> 8) == 0u ? -64.0 : log((double)(lu.x >> 8) * 0x1p-24);
            }
            const int off = (int)(t - base);
            const int left = (int)((n - t) < (int64_t)(64 - off) ? (n - t) : (int64_t)(64 - off));
            nblk = __builtin_amdgcn_readfirstlane(left < waves ? left : waves);
            uint32_t kind = 0;
            if constexpr (Model::kReptation) {
                const unsigned long long rep = __ballot(lu.y < st.lip_rep_thr) >> off;
                if (nblk > 0 && (rep & 1ull)) {
                    kind = 1;
                    nblk = 1;
                    if (lane == off) {
                        head[4] = la.x;
                        head[5] = lu.x;
                        head[6] = lu.z;
                        head[7] = lu.w;
                    }
                } else if (rep) {
                    const int first = (int)__builtin_ctzll(rep);
                    nblk = first < nblk ? first : nblk;
                }
            }
            if (kind == 0) {
                const int src = (off + lane) & 63;
                bead = (int)mul_shift(move_perm(la.x, src), (uint32_t)st.nb);
                const float d0 = move_disp(move_perm(la.y, src)), d1 = move_disp(move_perm(la.z, src)),
                            d2 = move_disp(move_perm(la.w, src));
                uw = move_perm(lu.x, src);
                const uint64_t lb = (uint64_t)__double_as_longlong(lnu_b);
                lnu = __longlong_as_double((long long)(((uint64_t)move_perm((uint32_t)(lb >> 32), src) << 32) |
                                                       move_perm((uint32_t)lb, src)));
                const float *xo = md.x + 3 * bead;
                const float o0 = xo[0], o1 = xo[1], o2 = xo[2];
                nx = move_wrap(o0 + d0, box);
                ny = move_wrap(o1 + d1, box);
                nz = move_wrap(o2 + d2, box);
                if (lane < nblk) {
                    MoveProp p;
                    p.n[0] = nx; p.n[1] = ny; p.n[2] = nz;
                    p.o[0] = o0; p.o[1] = o1; p.o[2] = o2;
                    p.reach = move_reach(d0, d1, d2, box);
                    p.b = bead;
                    props[lane] = p;
                }
            }
            if (lane == 0) {
                head[0] = (uint32_t)nblk;
                head[1] = kind;
            }
        }
        __syncthreads();
        const int cur = __builtin_amdgcn_readfirstlane((int)head[0]);
        if (cur == 0) break;
        if (Model::kReptation && __builtin_amdgcn_readfirstlane(head[1]) == 1u) {
            // ---- a reptation, by the whole workgroup
            if constexpr (Model::kReptation) md.reptation(st, head[4], head[5], head[6], head[7], g, H, list, lo, lnf, E, Ef);
            t += 1;
            continue;
        }
        if (wave < cur) move_evaluate(st, md, props, wave, waves, rows, tab, list, lane);
        __syncthreads();
        if (wave != 0) {
            continue;
        }
        // ---- decisions, lane l attempt l of the block.  The lanes from the
        // next attempt on decide at once as if all attempts before them were
        // refused; the first one that is not is taken, the energies of the
        // later ones corrected for it, and so on.
        int64_t tot = 0;
        uint32_t bad = 0, prior = 0;         // prior: earlier attempts on the same particle
        int over = 0;
        const bool mine = lane < nblk;
        if (mine) {
            const MoveRow r = rows[lane];
            tot = r.de;
            bad = r.bad;
            prior = r.same;
            over = r.nbad;
        }
        const uint32_t blkm = (1u << nblk) - 1u;
        uint32_t accm = 0;
        int i = 0, bE = E - lo;              // next attempt; the walker's bin in its window
        int hist = bE;                       // bin after the lane's attempt
        double gE = 0.0;
        float gEh = 0.0f, gEl = 0.0f;
        if (PREC == 0) gE = g[bE];
        else { gEh = gh[bE]; gEl = gl[bE]; }
        auto add_lnf = [&](int times) {
            for (int r = 0; r < times; ++r) {
                if (PREC == 0) gE = gE + lnf;
                else two_sum_add(gEh, gEl, lnf32);
            }
        };
        auto flush = [&]() {
            if (lane == 0) {
                if (PREC == 0) g[bE] = gE;
                else { gh[bE] = gEh; gl[bE] = gEl; }
            }
        };
        // The common case in a loop of its own: no overlaps, energies of the
        // window inside the fixed-point range (B < 2^16 bins: the walk-in's
        // counts are in LDS).  It is bound by the chain from one accepted
        // attempt to the next, so the corrections are in registers, what an
        // event does not change is kept (A = (lane) ln f - ln u), and the lanes'
        // next ln g is read while the walker's bin is paid; lanes that go back
        // to it take the paid value.
        const bool plain = st.binw_fx <= ((int64_t)1 << 44) && !__ballot(over != 0 || bad != 0u);
        if (plain) {
            const move_l16 corr = move_corrections((const int64_t *)tab, lane, waves);
            const double slope = PREC == 0 ? lnf : (double)lnf32;
            const double ls = (double)lane * slope, A = ls - lnu;
            // t is off by at most 64 roundings of values up to |ln g| + 64 ln f + |ln u|
            const double Mc = PREC == 0 ? 1e-10 + (64.0 * slope + 1024.0) * 0x1p-46 : 1e-5 + (64.0 * slope + 1024.0) * 0x1p-18;
            int64_t e_new = 0;
            int bn = 0, from = -1;            // the lanes' new bins; the bin left last
            double gN = 0.0, paid = 0.0;      // ln g of the new bin
            float gNh = 0.0f, gNl = 0.0f, paidh = 0.0f, paidl = 0.0f;
            bool in = false;
            auto look = [&]() {
                e_new = Ef + tot;
                const double qd = (double)(e_new - st.emin_fx) * st.binw_inv;
                const double fl = __builtin_floor(qd), fr = qd - fl;
                bn = (int)fl - lo;
                if (__ballot(!(fabs(fr - 0.5) < 0.5 - 0x1p-20))) bn = fx_bin(st.emin_fx, st.binw_fx, st.binw_inv, e_new) - lo;
                in = (unsigned)bn < (unsigned)W;
                const int bi = in ? bn : 0;
                if (PREC == 0) gN = g[bi];
                else { gNh = gh[bi]; gNl = gl[bi]; }
            };
            uint32_t S = 0u, first = 0u;      // may be the event; the event, if accepted for sure
            auto weigh = [&]() {
                const double base = PREC == 0 ? gE : (double)gEh + (double)gEl;
                const double gb = base - move_readlane_d(ls, i);
                const double M = PREC == 0 ? __builtin_fma(fabs(base), 0x1p-46, Mc)
                                           : __builtin_fma(fabs(base) * 0x1p-24 + (double)fabsf(gEl), 0x1p-18, Mc);
                const uint32_t C = (uint32_t)__ballot((prior & accm) != 0u), rem = blkm & (~0u << i);
                double v;
                if (PREC == 0) {
                    gN = bn == from ? paid : gN;
                    v = gN;
                } else {
                    gNh = bn == from ? paidh : gNh;
                    gNl = bn == from ? paidl : gNl;
                    v = (double)gNh + (double)gNl;
                }
                // the walker's own bin: accepted; outside the window: refused (both
                // while ln g(E) is finite; else all lanes are left to the exact round)
                const uint64_t vb = (uint64_t)__double_as_longlong(v);
                uint32_t hi = (uint32_t)(vb >> 32);
                hi = bn == bE ? 0xffe00000u : hi;
                hi = in ? hi : 0x7fe00000u;
                v = __longlong_as_double((long long)(((uint64_t)hi << 32) | (uint32_t)vb));
                const double d = gb - v, t = d + A;
                const double Mt = PREC == 0 ? M : M + (fabs(d) + (double)fabsf(gNl)) * 0x1p-18;
                S = ((uint32_t)__ballot(!(t < -Mt)) | C) & rem;
                first = (uint32_t)__ballot(t > Mt) & ~C & S & (0u - S);
            };
            look();
            weigh();
            while (first != 0u) {
                const int j = (int)__builtin_ctz(first);
                const int bj = __builtin_amdgcn_readlane(bn, j);
                Ef = move_readlane64(e_new, j);
                const double gj = PREC == 0 ? move_readlane_d(gN, j) : 0.0;
                const float hj = PREC == 0 ? 0.0f : move_readlane_f(gNh, j), lj = PREC == 0 ? 0.0f : move_readlane_f(gNl, j);
                tot += corr[j];
                accm |= first;
                look();
                add_lnf(j - i);
                i = j + 1;
                from = bE;
                paid = gE;
                paidh = gEh;
                paidl = gEl;
                if (bj != bE) {
                    flush();
                    bE = bj;
                    if (PREC == 0) gE = gj;
                    else { gEh = hj; gEl = lj; }
                    hist = lane >= j ? bj : hist;
                }
                add_lnf(1);
                weigh();
            }
            if (S == 0u) {
                add_lnf(nblk - i);
                i = nblk;
            }
        }
        while (i < nblk) {
            int64_t e_new = 0;
            const bool none = over - __builtin_popcount((bad >> 16) & accm) + __builtin_popcount(bad & accm) == 0;
            const bool ok = none && fx_add(Ef, tot, e_new);
            const int bn = move_bin(st, ok ? e_new : Ef) - lo;   // bin within the window
            const bool in = ok && bn >= 0 && bn < W;
            const int bi = in ? bn : 0;
            const double nadd = (double)(lane - i);
            // same bin: ln g cancels, always accepted (infinite ln g: NaN, settled below)
            const bool stay = bn == bE && (PREC == 0 ? __builtin_isfinite(gE) : __builtin_isfinite(gEh + gEl));
            bool yes, no;
            double gN = 0.0;
            float gNh = 0.0f, gNl = 0.0f;
            if (PREC == 0) {
                gN = g[bi];
                const double d = (gE + nadd * lnf) - gN;
                const double tt = d - lnu;
                const double M = 1e-10 + (fabs(gE) + 64.0 * lnf + fabs(gN) + 1.0) * 0x1p-46;
                yes = d > M || tt > M;
                no = tt < -M;
            } else {
                gNh = gh[bi];
                gNl = gl[bi];
                const double d = (((double)gEh + (double)gEl) + nadd * (double)lnf32) - ((double)gNh + (double)gNl);
                const double tt = d - lnu;
                const double M = 1e-5 + (fabs(d) + (double)fabsf(gEl) + (double)fabsf(gNl) + 64.0 * (double)lnf32 + 1.0) * 0x1p-18;
                yes = d > M || tt > M;
                no = tt < -M;
            }
            const uint32_t Y = (uint32_t)__ballot(in && (yes || stay)), C = (uint32_t)__ballot((prior & accm) != 0u);
            const uint32_t S = ((uint32_t)__ballot(in && (!no || stay)) | C) & blkm & (~0u << i);
            const int j = S ? (int)__builtin_ctz(S) : nblk;
            add_lnf(j - i);
            i = j;
            if (j >= nblk || ((C >> j) & 1u)) break;
            bool acc = (Y >> j) & 1u;
            const int bj = __builtin_amdgcn_readlane(bi, j);
            if (PREC == 0) {
                const double gj = move_readlane_d(gN, j);
                if (!acc) acc = __ballot(accept64(gE - (bj == bE ? gE : gj), __builtin_amdgcn_readlane(uw, j))) != 0ull;
                if (acc && bj != bE) { flush(); gE = gj; }
            } else {
                const float hj = move_readlane_f(gNh, j), lj = move_readlane_f(gNl, j);
                if (!acc) {
                    const bool st_ = bj == bE;
                    acc = __ballot(accept32((gEh - (st_ ? gEh : hj)) + (gEl - (st_ ? gEl : lj)),
                                            __builtin_amdgcn_readlane(uw, j))) != 0ull;
                }
                if (acc && bj != bE) { flush(); gEh = hj; gEl = lj; }
            }
            if (acc) {
                Ef = move_readlane64(e_new, j);
                bE = bj;
                hist = lane >= j ? bj : hist;
                accm |= 1u << j;
                if (mine && lane > j) tot += tab[lane * waves + j];   // the correction for attempt j
            }
            add_lnf(1);
            i = j + 1;
        }
        flush();
        if (lane < i) atomicAdd(&H[hist], 1u);
        E = bE + lo;
        if ((accm >> (lane & 31)) & 1u & (uint32_t)(lane < nblk)) {
            float *xo = md.x + 3 * bead;
            xo[0] = nx;
            xo[1] = ny;
            xo[2] = nz;
            if constexpr (Model::kGrid) md.grid[bead] = move_grid(xo, md.scale);
        }
        t += i;
        move_wave_sync();
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        st.E[w] = E;
        st.Efx[w] = Ef;
    }
}

}  // namespace rewl_gpu

// rewl_trimer.hip -- the continuous-move model of the library: amphiphilic
// head-tail-tail trimers in a periodic cube, sampled by single-bead
// displacements with the Wang-Landau rule on energy bins (Vogel, Li, Wuest,
// Landau, J. Phys.: Conf. Ser. (2014): Sec. 2 for the method, Sec. 3.2 for a
// bead-spring amphiphile sampled with local displacement moves).
//
// Force field: bonds head-tail1 and tail1-tail2 are harmonic, k (r - r0)^2
// with k = 100, r0 = 1; every other pair interacts by 4 (r^-12 - r^-6):
// tail-tail pairs cut at r = 2.5 without shift, pairs involving a head cut at
// r = 2^(1/6) and shifted by +1 (Weeks-Chandler-Andersen).  Coordinates are
// binary32 in [0, box); the minimum-image difference per axis is binary32;
// pair energies are binary64 from those differences, the bond length by the
// correctly rounded binary64 square root.
//
// Energies are fixed point (units of 2^-32): every pair term is rounded once
// and totals and changes are exact integer sums, so the lanes may add the
// partner terms in any order and every implementation agrees to the bit.
//
// Mapping: one walker per workgroup.  Its coordinates, ln g and H live in
// LDS.  Attempts are sequential; the main phase evaluates blocks of them side
// by side, a wavefront each (rewl_moves.h), walk-in one after the other on one
// wavefront.
#include "rewl_moves.h"

namespace rewl_gpu {

namespace {

constexpr double kBondK = 100.0;
constexpr double kBondR0 = 1.0;
constexpr double kTailCut2 = 6.25;                    // 2.5^2
constexpr double kWcaCut2 = 0x1.428a2f98d728bp+0;     // RN(2^(1/3)) = RN((2^(1/6))^2)

// Energy of two beads at squared distance r2: bonded, both tails, or one of
// them a head.  No branch on the kind: a wavefront nearly always holds
// several, and the division is the cost.
__device__ __forceinline__ double pair_terms(bool tails, bool bond, double r2) {
#pragma clang fp contract(off)
    const double s2 = 1.0 / r2;
    const double s6 = (s2 * s2) * s2;
    double v = 4.0 * ((s6 * s6) - s6);
    v = tails ? v : v + 1.0;
    v = r2 >= (tails ? kTailCut2 : kWcaCut2) ? 0.0 : v;
    if (bond) {
        const double x = __builtin_sqrt(r2) - kBondR0;
        v = kBondK * (x * x);
    }
    return v;
}

// Energy of beads i (at p) and j (at r).
__device__ __forceinline__ double pair_energy(int i, int j, const float *p, const float *r, float box, float half) {
    const int ti = i % 3, tj = j % 3;
    return pair_terms(ti > 0 && tj > 0, i / 3 == j / 3 && (ti - tj == 1 || tj - ti == 1), move_r2(p, r, box, half));
}

// Energy change of moving bead b (coordinates in LDS x) to n: the sum over
// partners j of fx(V(b at n, j)) - fx(V(b, j)); false for a hard overlap.
// Every lane returns the same result.
__device__ __forceinline__ bool delta_e(const DevState &st, const float *x, int b, float n0, float n1, float n2,
                                        int lane, int64_t &de) {
#pragma clang fp contract(off)
    const float box = st.box, half = 0.5f * st.box;
    const float nw[3] = {n0, n1, n2};
    int64_t acc = 0;
    bool bad = false;
    for (int c = 0; c < st.nb; c += 64) {
        const int j = c + lane;
        if (j < st.nb && j != b) {
            int64_t tn = 0, to = 0;
            bad |= !fx_term(pair_energy(b, j, nw, x + 3 * j, box, half), tn);
            bad |= !fx_term(pair_energy(b, j, x + 3 * b, x + 3 * j, box, half), to);
            acc += tn - to;
        }
    }
    de = wave_sum64(acc);
    return __ballot(bad) == 0ull;
}

// Bin of a fixed-point energy (also outside [0, B), bounded to +-2^30).
__device__ __forceinline__ int energy_bin(const DevState &st, int64_t e) { return fx_bin(st.emin_fx, st.binw_fx, st.binw_inv, e); }

// ---------------------------------------------------------------------------
// Energy of every walker's starting configuration: the exact sum of the
// pair terms over i < j, rows i dealt to the lanes.  Each term is split into
// its high and low 32 bits, summed separately (neither sum can overflow), and
// the total is checked against the energy range; a start with a hard
// overlap or out of range gets the bin INT32_MIN, which the host refuses.
__global__ __launch_bounds__(64) void k_trimer_init(DevState st) {
#pragma clang fp contract(off)
    const int w = blockIdx.x;
    const int lane = threadIdx.x;
    const float *x = (const float *)(st.spins + (size_t)w * st.Npad);
    const float box = st.box, half = 0.5f * st.box;
    int64_t shi = 0, slo = 0;
    bool bad = false;
    for (int i = lane; i < st.nb; i += 64) {
        for (int j = i + 1; j < st.nb; ++j) {
            int64_t t = 0;
            bad |= !fx_term(pair_energy(i, j, x + 3 * i, x + 3 * j, box, half), t);
            shi += t >> 32;
            slo += t & 0xffffffffll;
        }
    }
    shi = wave_sum64(shi);
    slo = wave_sum64(slo);
    bad = __ballot(bad) != 0ull;
    if (lane == 0) {
        int64_t e = 0;
        const bool ok = !bad && shi > -(1ll << 30) && shi < (1ll << 30) && fx_add(shi * 4294967296ll, slo, e);
        st.Efx[w] = ok ? e : 0;
        st.E[w] = ok ? energy_bin(st, e) : INT32_MIN;
    }
}

// Random words of 64 attempts, one attempt per lane: bead, displacement,
// uniform word (Philox blocks (t, walker, dom) and (t, walker, dom_u)).
struct Draw {
    int bead;
    float d0, d1, d2;
    uint32_t u;
};

__device__ __forceinline__ Draw draw(const DevState &st, uint32_t dom, uint32_t dom_u, uint64_t t, uint32_t w) {
    const U4 r = philox10((uint32_t)t, (uint32_t)(t >> 32), w, st.ctr3 | (dom << 24), st.key0, st.key1);
    const U4 ru = philox10((uint32_t)t, (uint32_t)(t >> 32), w, st.ctr3 | (dom_u << 24), st.key0, st.key1);
    Draw d;
    d.bead = (int)mul_shift(r.x, (uint32_t)st.nb);
    d.d0 = move_disp(r.y);
    d.d1 = move_disp(r.z);
    d.d2 = move_disp(r.w);
    d.u = ru.x;
    return d;
}

// ---------------------------------------------------------------------------
// Walk-in (the Potts walk-in rule on energy bins): Wang-Landau with ln f = 1
// as uint32 visit counts over the B bins (an energy outside the range counts
// at the nearest end bin), under the lid, until the bin lies in the window.
__global__ __launch_bounds__(64) void k_trimer_walkin(DevState st, int64_t chunk, int64_t budget) {
#pragma clang fp contract(off)
    const int w = blockIdx.x;
    const int lane = threadIdx.x;
    if (st.walkin_done[w]) return;
    extern __shared__ __align__(16) unsigned char smem[];
    float *x = (float *)smem;
    uint32_t *cnt = (uint32_t *)(smem + st.Npad);
    const uint32_t *gx = (const uint32_t *)(st.spins + (size_t)w * st.Npad);
    for (int i = lane; i < st.Npad / 4; i += 64) ((uint32_t *)x)[i] = gx[i];
    const uint32_t *gcnt = st.walkin_cnt + (size_t)w * st.Bpad;
    for (int b = lane; b < st.B; b += 64) cnt[b] = gcnt[b];
    __syncthreads();

    const int k = w / st.m;
    const int lo = st.start[k], hi = lo + st.W - 1;
    const int B = st.B;
    int E = st.E[w];
    int64_t Ef = st.Efx[w];
    int64_t t = st.walkin_att[w];
    const int slack = st.walkin_slack;
    const bool down = E > hi;
    int bound = t == 0 ? (down ? E + slack : E - slack) : st.walkin_bound[w];
    const int64_t end = (t + chunk < budget) ? t + chunk : budget;
    bool done = (E >= lo && E <= hi);
    while (!done && t < end) {
        const Draw dr = draw(st, kDomWalkin, kDomWalkinU, (uint64_t)(t + lane), (uint32_t)w);
        const int todo = (int)((end - t) < 64 ? (end - t) : 64);
        for (int j = 0; j < todo; ++j) {
            const int b = __builtin_amdgcn_readlane(dr.bead, j);
            const float d0 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(dr.d0), j));
            const float d1 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(dr.d1), j));
            const float d2 = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(dr.d2), j));
            const uint32_t u = __builtin_amdgcn_readlane(dr.u, j);
            const float n0 = move_wrap(x[3 * b] + d0, st.box);
            const float n1 = move_wrap(x[3 * b + 1] + d1, st.box);
            const float n2 = move_wrap(x[3 * b + 2] + d2, st.box);
            int64_t de = 0, e_new = 0;
            const bool ok = delta_e(st, x, b, n0, n1, n2, lane, de) && fx_add(Ef, de, e_new);
            const int bn = ok ? energy_bin(st, e_new) : 0;
            const int co = E < 0 ? 0 : (E >= B ? B - 1 : E);
            const int cn = bn < 0 ? 0 : (bn >= B ? B - 1 : bn);
            const double d = (double)((int64_t)cnt[co] - (int64_t)cnt[cn]);
            const bool inside = slack == 0 || (down ? bn <= bound : bn >= bound);
            if (ok && inside && accept64(d, u)) {
                if (lane == 0) {
                    x[3 * b] = n0;
                    x[3 * b + 1] = n1;
                    x[3 * b + 2] = n2;
                }
                Ef = e_new;
                E = bn;
                if (slack && down && E + slack < bound) bound = E + slack;
                if (slack && !down && E - slack > bound) bound = E - slack;
            }
            if (lane == 0) cnt[E < 0 ? 0 : (E >= B ? B - 1 : E)] += 1u;
            __syncthreads();
            ++t;
            if (E >= lo && E <= hi) { done = true; break; }
        }
    }
    __syncthreads();
    uint32_t *ox = (uint32_t *)(st.spins + (size_t)w * st.Npad);
    for (int i = lane; i < st.Npad / 4; i += 64) ox[i] = ((uint32_t *)x)[i];
    uint32_t *ocnt = st.walkin_cnt + (size_t)w * st.Bpad;
    for (int b = lane; b < B; b += 64) ocnt[b] = cnt[b];
    if (lane == 0) {
        st.E[w] = E;
        st.Efx[w] = Ef;
        st.walkin_att[w] = t;
        st.walkin_done[w] = done ? 1 : 0;
        st.walkin_bound[w] = bound;
    }
}

// ---------------------------------------------------------------------------
// Main-phase attempts s0 .. s0+n-1 of every walker (Sec. 2): propose a bead
// displacement, reject it if the new energy bin leaves the window, else
// accept with min[1, g(bin_old)/g(bin_new)]; then ln g += ln f and H += 1 at
// the bin after the decision.
//
// One workgroup per walker, an attempt per wavefront: blocks of consecutive
// attempts evaluated side by side and decided in order (rewl_moves.h, with the
// choice of the workgroup); up to eight beads on one wavefront (trimer_few).
template <bool GRID>
struct TrimerMoves {
    static constexpr bool kGrid = GRID;    // 16-bit places in LDS
    static constexpr bool kReptation = false;
    static constexpr bool kHeads = true;   // pairs with a head reach 2^(1/6) only
    float *x;
    MoveGrid *grid;
    float box, half, scale;
    __device__ __forceinline__ int bonds(int b, int &p0, int &p1) const {
        const int t = b % 3;
        p0 = t == 0 ? b + 1 : b - 1;
        p1 = t == 1 ? b + 1 : -1;
        return t == 1 ? 2 : 1;
    }
    __device__ __forceinline__ double pair(int b, int j, const float *p, const float *r, bool bond) const {
        return pair_terms(b % 3 > 0 && j % 3 > 0, bond, move_r2(p, r, box, half));
    }
};

// Attempts of a walker of at most eight beads, one after the other on one
// wavefront: a block of them would end on a bead that has moved after two or
// three.  Lane j holds bead j and evaluates it against the moved bead's new
// place, lane 8 + j against the old one.  Bound by the chain of one attempt
// (minimum image, division, sum, bin, ln g): us per 1,000 attempts of 64 and of
// 1,024 walkers, one trimer 821 and 904, in blocks 1666 and 2310, with two
// wavefronts sharing an attempt 1253 and 1646; two trimers 820 and 905, 1230 and
// 1753, 1286 and 1675.
constexpr int kFewBeads = 8;
template <int PREC>
__device__ __forceinline__ void trimer_few(const DevState &st, float *x, int w, int64_t s0, int64_t n, double *g,
                                           float *gh, float *gl, uint32_t *H) {
#pragma clang fp contract(off)
    const int lane = threadIdx.x;
    const int j = lane & (kFewBeads - 1);
    const bool old = lane >= kFewBeads, live = lane < 2 * kFewBeads && j < st.nb;
    const int k = w / st.m;
    const int lo = st.start[k], W = st.W;
    const double lnf = st.lnf[k];
    const float lnf32 = (float)lnf;
    const float box = st.box, half = 0.5f * st.box;
    float own[3] = {0.0f, 0.0f, 0.0f};
    if (live)
        for (int c = 0; c < 3; ++c) own[c] = x[3 * j + c];
    int E = __builtin_amdgcn_readfirstlane(st.E[w]) - lo;   // bin in the window
    int64_t Ef = move_uniform64(st.Efx[w]);
    for (int64_t base = 0; base < n; base += 64) {
        const int todo = (int)((n - base) < 64 ? (n - base) : 64);
        const Draw dr = draw(st, kDomMove, kDomMoveU, (uint64_t)(s0 + base + lane), (uint32_t)w);
        double lnu;
        if (PREC == 0) lnu = dr.u == 0u ? -64.0 : log((double)dr.u * 0x1p-32);
        else lnu = (dr.u >> 8) == 0u ? -64.0 : log((double)(dr.u >> 8) * 0x1p-24);
        for (int a = 0; a < todo; ++a) {
            const int b = __builtin_amdgcn_readlane(dr.bead, a);
            const float o[3] = {move_readlane_f(own[0], b), move_readlane_f(own[1], b), move_readlane_f(own[2], b)};
            const float nw[3] = {move_wrap(o[0] + move_readlane_f(dr.d0, a), box),
                                 move_wrap(o[1] + move_readlane_f(dr.d1, a), box),
                                 move_wrap(o[2] + move_readlane_f(dr.d2, a), box)};
            const float q[3] = {old ? o[0] : nw[0], old ? o[1] : nw[1], old ? o[2] : nw[2]};
            int64_t t = 0;
            const bool with = live && j != b;
            const bool bad = !fx_term(pair_energy(b, j, q, own, box, half), t) && with;
            const int64_t de = wave_sum64(with ? (old ? -t : t) : 0);
            int64_t e_new = 0;
            const bool ok = __ballot(bad) == 0ull && fx_add(Ef, de, e_new);
            const int bn = (ok ? energy_bin(st, e_new) : st.B) - lo;
            bool acc = false;
            if (ok && bn >= 0 && bn < W) {
                const double luj = move_readlane_d(lnu, a);
                const uint32_t u = __builtin_amdgcn_readlane(dr.u, a);
                if (PREC == 0) {
                    const double d = g[E] - g[bn], v = d - luj;
                    acc = fabs(v) > 1e-10 ? v > 0.0 : accept64(d, u);
                } else {
                    const float d = (gh[E] - gh[bn]) + (gl[E] - gl[bn]);
                    const double v = (double)d - luj;
                    acc = fabs(v) > 1e-5 ? v > 0.0 : accept32(d, u);
                }
            }
            if (__ballot(acc) != 0ull) {
                Ef = e_new;
                E = bn;
                if (j == b)
                    for (int c = 0; c < 3; ++c) own[c] = nw[c];
            }
            if (lane == 0) {
                if (PREC == 0) {
                    g[E] = g[E] + lnf;
                } else {
                    float h = gh[E], l = gl[E];
                    two_sum_add(h, l, lnf32);
                    gh[E] = h;
                    gl[E] = l;
                }
                atomicAdd(&H[E], 1u);
            }
            move_wave_sync();
        }
    }
    if (live && !old)
        for (int c = 0; c < 3; ++c) x[3 * j + c] = own[c];
    if (lane == 0) {
        st.E[w] = E + lo;
        st.Efx[w] = Ef;
    }
    __syncthreads();
}

// FORM: attempts one after the other (at most kFewBeads beads), blocks without
// or with the 16-bit places.
enum { kFormFew = 0, kFormBlocks = 1, kFormGrid = 2 };
template <int PREC, int FORM>
__global__ __launch_bounds__(FORM == kFormFew ? 64 : 1024) void k_trimer_sweep(DevState st, int64_t s0, int64_t n) {
    if (*st.converged) return;
    const int w = blockIdx.x;
    const int k = w / st.m;
    extern __shared__ __align__(16) unsigned char smem[];
    const int W = st.W, Wpad = st.Wpad;
    double *g = (double *)(smem + st.Npad);
    float *gh = (float *)(smem + st.Npad);
    float *gl = gh + Wpad;
    uint32_t *H = (uint32_t *)(smem + st.Npad + (size_t)Wpad * 8);
    const int E = st.E[w];
    if (E < st.start[k] || E >= st.start[k] + W) return;   // not walked in: leave the walker untouched
    const uint32_t *gx = (const uint32_t *)(st.spins + (size_t)w * st.Npad);
    for (int i = threadIdx.x; i < st.Npad / 4; i += blockDim.x) ((uint32_t *)smem)[i] = gx[i];
    const size_t row = (size_t)w * Wpad;
    for (int b = threadIdx.x; b < W; b += blockDim.x) {
        if (PREC == 0) {
            g[b] = st.lng[row + b];
        } else {
            gh[b] = st.lng_hi[row + b];
            gl[b] = st.lng_lo[row + b];
        }
        H[b] = st.H[row + b];
    }
    __syncthreads();
    if constexpr (FORM == kFormFew) {
        trimer_few<PREC>(st, (float *)smem, w, s0, n, g, gh, gl, H);
    } else {
        constexpr bool kGrid = FORM == kFormGrid;
        unsigned char *mv = smem + st.Npad + (size_t)Wpad * 12;
        MoveGrid *grid = kGrid ? (MoveGrid *)(mv + move_lds_bytes((int)(blockDim.x >> 6))) : nullptr;
        TrimerMoves<kGrid> md{(float *)smem, grid, st.box, 0.5f * st.box, 65536.0f / st.box};
        move_sweep<TrimerMoves<kGrid>, PREC>(st, md, w, s0, n, g, gh, gl, H, mv);
    }
    uint32_t *ox = (uint32_t *)(st.spins + (size_t)w * st.Npad);
    for (int i = threadIdx.x; i < st.Npad / 4; i += blockDim.x) ox[i] = ((uint32_t *)smem)[i];
    for (int b = threadIdx.x; b < W; b += blockDim.x) {
        if (PREC == 0) {
            st.lng[row + b] = g[b];
        } else {
            st.lng_hi[row + b] = gh[b];
            st.lng_lo[row + b] = gl[b];
        }
        st.H[row + b] = H[b];
    }
}

hipError_t allow(const void *fn, size_t bytes) {
    if (bytes <= 65536) return hipSuccess;
    return hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

}  // namespace

static MovePlan trimer_plan(const DevState &st) {
    const size_t rows = (size_t)st.Npad + (size_t)st.Wpad * 12;
    if (st.nb <= kFewBeads) return MovePlan{1, 0, rows};
    return move_plan(rows, 0, st.nb, st.nw);
}
size_t trimer_sweep_lds_bytes(const DevState &st) { return trimer_plan(st).lds; }
size_t trimer_walkin_lds_bytes(const DevState &st) { return (size_t)st.Npad + (size_t)st.Bpad * 4; }

hipError_t launch_trimer_init(const DevState &st, hipStream_t s) {
    hipLaunchKernelGGL(k_trimer_init, dim3(st.nw), dim3(64), 0, s, st);
    return hipGetLastError();
}

hipError_t launch_trimer_walkin(const DevState &st, int64_t chunk, int64_t budget, hipStream_t s) {
    const size_t lds = trimer_walkin_lds_bytes(st);
    hipError_t e = allow((const void *)k_trimer_walkin, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_trimer_walkin, dim3(st.nw), dim3(64), lds, s, st, chunk, budget);
    return hipGetLastError();
}

hipError_t launch_trimer_sweep(const DevState &st, int64_t s0, int64_t n, hipStream_t s) {
    const MovePlan p = trimer_plan(st);
    auto go = [&](auto kernel) -> hipError_t {
        const hipError_t e = allow((const void *)kernel, p.lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(kernel, dim3(st.nw), dim3(64 * p.waves), p.lds, s, st, s0, n);
        return hipGetLastError();
    };
    if (st.nb <= kFewBeads) return st.precision == 0 ? go(k_trimer_sweep<0, kFormFew>) : go(k_trimer_sweep<1, kFormFew>);
    if (p.grid) return st.precision == 0 ? go(k_trimer_sweep<0, kFormGrid>) : go(k_trimer_sweep<1, kFormGrid>);
    return st.precision == 0 ? go(k_trimer_sweep<0, kFormBlocks>) : go(k_trimer_sweep<1, kFormBlocks>);
}

}  // namespace rewl_gpu

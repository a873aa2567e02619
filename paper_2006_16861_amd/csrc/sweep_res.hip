// Resident-tile 2-D recurrence sweep: the Table 1 loop on a real field
// (integrator I_acd of Def. 2) for tables without corner mass terms, with
// every tile held on chip for a whole run of steps.
//
// The blocked kernels of sweep_tb.hip reload their tile and refold its
// coefficients for every k steps, and a launch of them is bound by that
// prologue and by the scheduling of a few thousand workgroups.  Here one
// workgroup owns one tile for up to TDP_RES_MAXSTEPS steps:
// - at the start it loads the extended tile (exact region plus a k-wide halo)
//   once and folds the cell slowness into per-node coefficients; F is kept in
//   LDS;
// - it then advances k steps at a time in registers, exactly as the blocked
//   tile does (rows per lane, DPP x-neighbours, edge rows through LDS, one
//   barrier per step);
// - after each block of k steps it publishes the border of its exact region
//   (u_j and u_{j-1}) to its slot of a global exchange buffer and reads its
//   halo from its neighbours' slots.
//
// Two workgroups share a compute unit (at most 80 KB of LDS and 256 VGPRs on 4
// waves each), so that one computes while the other waits for its halo: a
// block's exchange is a chain of memory round trips through the fabric, about
// as long as four steps, and nothing inside one tile can hide it.  Measured at
// 1024^2 in FP64 (494 tiles of 48 x 64, k = 4): 1.55 us a step, against 2.21
// with one 88 x 64 tile per compute unit, flags and acknowledged bands, and 3.0
// for the blocked sweep; in FP32 (441 tiles of 64 x 64, k = 8) 1.12 against 1.63
// (112 x 64 tiles) and 1.93.  Of a 4-step block's 14.1 k cycles (mean over
// tiles) 6.3 k are steps (5.4 k where a tile has the vector units to itself,
// 8.1 k in the younger of two that run together), 1.6 k stage and publish,
// 2.5-5 k wait for the neighbours' words, the rest is barriers, the landing
// and the emptied slot.  Bound by the vector units while the two compute
// together (a step issues 930 of its 1375 cycles) and by the round trip between.
//
// Exchange without flags.  A slot holds a reserved signalling-NaN pattern
// until its tile publishes; a reader loads the halo values themselves and
// loads again while any of them is that pattern.  The arithmetic never makes
// it (results that are NaN are quiet), so a value that is not the pattern is
// the published one.  This saves the two round trips of a flag protocol (the
// band stores acknowledged before the flag store, the flag seen before the
// band loads).  Slots are used in turn, three per tile:
//   exchange e publishes in slot e mod 3, reads the neighbours' slots e mod
//   3, and then, with every neighbour's exchange-e data in hand, so that all of
//   them have read this tile's exchange e-1, returns slot (e-1) mod 3 to the
//   pattern.  Those stores are complete (s_waitcnt, barrier) before exchange
//   e+1 publishes, so a neighbour that polls for exchange e+2 in that slot,
//   which it does only after it has read exchange e+1, finds the pattern or
//   new values, never old ones.
// Values travel whole: 64- or 32-bit agent-scope relaxed atomics, which the
// compiler emits with the coherent cache policy (sc1): they bypass the
// per-XCD L2 state that is not kept coherent between XCDs.
//
// Tile geometry: tile (ty, tx) extends over rows ty OY .. ty OY + EY - 1 and
// columns tx OX .. tx OX + 63, OX = 64 - 2k, OY = EY - 2k; the k outermost
// rows and columns are halo where a neighbour exists, while at the domain's
// edge the exact region reaches it (nothing is lost to a halo there: a
// Dirichlet wall needs none).  A grid of one tile needs no exchange at all.
// A slot holds, per level, the k rows above and below the halo rows over all
// 64 columns and the k columns beside the halo columns over all EY rows.
//
// Every tile must be resident at once: the host launches no more workgroups
// than the device holds, over all such launches that may overlap.  A wait that exceeds
// its poll limit, or sees another tile's abort, raises the abort word and the
// whole grid leaves early; the host, or k_res_recover behind it on the
// stream, then redoes the application.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "tdp_internal.h"
#include "lanes.h"

namespace tdp {

namespace {

constexpr int kResX = 64;           // columns of an extended tile (one wave)
constexpr int kRecRows = 32;        // rows of a block of the recovery (64 columns)

template <typename T>
__device__ __forceinline__ void st_coh(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T ld_coh(const T *p)
{
    return __hip_atomic_load(const_cast<T *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The exchange moves field values as words: a comparison of floating-point
// values cannot tell one NaN from another.
template <typename T>
struct Word;
template <>
struct Word<double> {
    using type = unsigned long long;
    static constexpr type empty = 0x7FF4A11FEE11C0DEull;      // quiet bit clear
    static __device__ __forceinline__ type of(double v) { return (type)__double_as_longlong(v); }
    static __device__ __forceinline__ double value(type w) { return __longlong_as_double((long long)w); }
};
template <>
struct Word<float> {
    using type = unsigned;
    static constexpr type empty = 0x7FA1C0DEu;
    static __device__ __forceinline__ type of(float v) { return __float_as_uint(v); }
    static __device__ __forceinline__ float value(type w) { return __uint_as_float(w); }
};

// words per level of a tile's slot
constexpr int res_band(int EY, int K) { return 2 * K * kResX + 2 * K * EY; }

// Per-node coefficients of a wave's R rows and the update of one row.
// FP64: the stencil weights without the damping factor d, which is applied
// once per update,
//   u_{j+1} = d (sum_q w_q u_j(q) + fa Re F + fb Im F - 2 u_{j-1}) + u_{j-1}:
// the weight of the edge between rows i and i+1 serves both (R + 1 per lane)
// and the corner weight is uniform, so a node holds 7 words with its two
// levels instead of 8, which is what lets 12 rows fit 256 VGPRs.
// FP32: the coefficients premultiplied by d, as in the blocked tile's second
// form and in its order of operations (the results are the same, bit for
// bit); registers are not short there.
template <typename T, int SC, int R>
struct Rows;

template <int SC, int R>
struct Rows<double, SC, R> {
    double wc[R], ww[R], we[R], wy[R + 1], d[R];
    double s2;
    __device__ __forceinline__ void fold(const Stencil<double> &st, const double (&ca)[R + 1],
                                         const double (&cb)[R + 1], const double (&dd)[R])
    {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            wc[i] = st.c0 + st.m[0] * ((ca[i] + cb[i]) + (ca[i + 1] + cb[i + 1]));
            ww[i] = st.s[1] + st.m[1] * (ca[i] + ca[i + 1]);
            we[i] = st.s[1] + st.m[1] * (cb[i] + cb[i + 1]);
            d[i] = dd[i];
        }
#pragma unroll
        for (int i = 0; i <= R; ++i) wy[i] = st.s[1] + st.m[1] * (ca[i] + cb[i]);
        s2 = st.s[2];
    }
    __device__ __forceinline__ double2 forcing(int, double2 f) const { return f; }
    __device__ __forceinline__ double update(int i, double cc, double cw, double ce, double pc,
                                             double xc, double corners, double2 f, double fas,
                                             double fbs, double prev) const
    {
        double acc = wc[i] * cc;
        acc += ww[i] * cw;
        acc += we[i] * ce;
        acc += wy[i] * pc;
        acc += wy[i + 1] * xc;
        if (SC > 2) acc += s2 * corners;
        acc += fas * f.x;
        acc += fbs * f.y;
        acc += -2.0 * prev;
        return d[i] * acc + prev;
    }
};

template <int SC, int R>
struct Rows<float, SC, R> {
    float co[R][5], d[R];
    float s2;
    __device__ __forceinline__ void fold(const Stencil<float> &st, const float (&ca)[R + 1],
                                         const float (&cb)[R + 1], const float (&dd)[R])
    {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            fold_node<float, 2, 2, 5>(st, dd[i], ca[i], cb[i], ca[i + 1], cb[i + 1], co[i]);
            d[i] = dd[i];
        }
        s2 = st.s[2];
    }
    __device__ __forceinline__ float2 forcing(int i, float2 f) const
    {
        f.x *= d[i];
        f.y *= d[i];
        return f;
    }
    __device__ __forceinline__ float update(int i, float cc, float cw, float ce, float pc, float xc,
                                            float corners, float2 f, float fas, float fbs,
                                            float prev) const
    {
        float acc = co[i][0] * cc;
        acc += co[i][1] * cw;
        acc += co[i][2] * ce;
        acc += co[i][3] * pc;
        acc += co[i][4] * xc;
        if (SC > 2) acc += (d[i] * s2) * corners;
        acc += fas * f.x;
        acc += fbs * f.y;
        return acc + (1.0f - 2.0f * d[i]) * prev;
    }
};

// x-1, x, x+1 of one row, and the sum of the outer two (shared by the corner
// terms of the rows above and below)
template <typename T>
struct Row3 {
    T w, c, e, s;
};
template <typename T>
__device__ __forceinline__ Row3<T> row_of(T c)
{
    Row3<T> r;
    r.c = c;
    r.w = lane_west(c);
    r.e = lane_east(c);
    r.s = r.w + r.e;
    return r;
}
template <typename T>
__device__ __forceinline__ Row3<T> row_at(const T *p)
{
    Row3<T> r;
    r.w = p[-1];
    r.c = p[0];
    r.e = p[1];
    r.s = r.w + r.e;
    return r;
}

// One step of the wave's R rows: the halo rows south and north come from the
// edge-row slots around cur[rs] and cur[rn]; the new first and last rows go to
// nxt[wf] and nxt[wl].  b holds u_{j-1} on entry and u_{j+1} on exit.
// With one or two waves per SIMD the step is bound by latency.  An update is
// one chain of dependent operations, so two rows are updated at a time, and
// the next two rows' F is read from LDS meanwhile.  The pairs go down from
// the second to the first and then from the last to the third: the halo rows
// are needed only after the first pair, and the new edge rows are in LDS
// while the inner pairs are still to do, so that neither LDS latency stands
// beside the barrier.
template <typename T, int SC, int R>
__device__ __forceinline__ void res_step(const T *__restrict__ cur, T *__restrict__ nxt, int rs,
                                         int rn, int wf, int wl,
                                         const typename V2t<T>::type *__restrict__ fl,
                                         const Rows<T, SC, R> &co, const T (&a)[R], T (&b)[R],
                                         T fas, T fbs)
{
    static_assert(R % 2 == 0 && R >= 6, "rows go in pairs");
    constexpr int NP = R / 2;
    auto f0 = fl[2 * kResX], f1 = fl[3 * kResX];
    const Row3<T> south = row_at(cur + rs), north = row_at(cur + rn);
    Row3<T> x = row_of(a[3]), y = row_of(a[4]);
#pragma unroll
    for (int q = 0; q < NP; ++q) {
        // pair i: rows 2i-1 (p), 2i (c), 2i+1 (x), 2i+2 (y)
        const int i = q < 2 ? 1 - q : NP + 1 - q, n = q < 1 ? 0 : NP - q;
        if (q == 2) {
            x = row_of(a[R - 1]);
            y = north;
        }
        const Row3<T> c = row_of(a[2 * i]);
        const Row3<T> p = i > 0 ? row_of(a[2 * (i > 0 ? i : 1) - 1]) : south;
        auto g0 = f0, g1 = f1;
        if (q + 1 < NP) {                // pair n is next
            g0 = fl[2 * n * kResX];
            g1 = fl[(2 * n + 1) * kResX];
        }
        b[2 * i] = co.update(2 * i, c.c, c.w, c.e, p.c, x.c, p.s + x.s, f0, fas, fbs, b[2 * i]);
        b[2 * i + 1] = co.update(2 * i + 1, x.c, x.w, x.e, c.c, y.c, c.s + y.s, f1, fas, fbs,
                                 b[2 * i + 1]);
        if (i == 0) nxt[wf] = b[0];
        if (i == NP - 1) nxt[wl] = b[R - 1];
        x = p;
        y = c;
        f0 = g0;
        f1 = g1;
        // keep the window a window: hoisting later rows' shifts would make
        // every row's neighbours live at once
        __builtin_amdgcn_sched_barrier(0);
    }
}

// A zero the optimiser cannot see through.  Added to a wave's first row where
// samples are written, and to the lane in the exchange, it keeps the
// addresses and conditions of that code there: hoisted out of the block
// loop, the rows' worth of them would take the registers the tile needs.
__device__ __forceinline__ int opaque_zero()
{
    int z;
    asm volatile("s_mov_b32 %0, 0" : "=s"(z));
    return z;
}

// LDS of one tile: the packed edge-row slots (two copies), F, and the staging
// of the exchange: the border columns being published, later each wave's
// incoming halo columns.
template <typename T, int R, int W, int K, bool MULTI>
struct ResLds {
    static constexpr int EY = R * W;
    static constexpr int CB = (2 * W + 2) * (kResX + 2);
    static constexpr int BAND = res_band(EY, K);
    static constexpr int LAND = 4 * R * K;                     // words per wave
    static constexpr int STAGE = MULTI ? 4 * K * EY : 1;       // = W * LAND
};

template <typename T, int SC, int R, int W, int K, bool MULTI>
__global__ __launch_bounds__(64 * W) __attribute__((amdgpu_waves_per_eu(2)))
void k_sweep2d_res(ResArgs a, Stencil<T> st)
{
    using V2 = typename V2t<T>::type;
    using Wd = Word<T>;
    using word = typename Wd::type;
    using L = ResLds<T, R, W, K, MULTI>;
    constexpr int EX = kResX, EY = L::EY, US = EX + 2, CB = L::CB, BAND = L::BAND;
    constexpr int OX = EX - 2 * K, OY = EY - 2 * K;
    __shared__ T xl[2 * CB];
    __shared__ V2 fl_all[EY * EX];
    __shared__ word stage[L::STAGE];
    __shared__ double2 fab[64];
    __shared__ int s_abort;

    const int ny = a.ny, nx = a.nx, nsteps = a.nsteps;
    const int ntl = a.tiles_x * a.tiles_y;
    const int part = (int)blockIdx.x >= ntl ? 1 : 0;
    const int tile = blockIdx.x - part * ntl;
    const int ty = tile / a.tiles_x, tx = tile - ty * a.tiles_x;
    const int lane = threadIdx.x & 63, lane_ = lane;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r0 = wv * R;
    const int gy0 = ty * OY, gx = tx * OX + lane;
    const bool xin = gx < nx;
    // which sides of the tile have a neighbour (elsewhere: the domain's edge)
    const bool nbW = MULTI && tx > 0, nbE = MULTI && tx + 1 < a.tiles_x;
    const bool nbS = MULTI && ty > 0, nbN = MULTI && ty + 1 < a.tiles_y;
    const bool xexact = xin && (!nbW || lane >= K) && (!nbE || lane < EX - K);
    // forcing scalars, a ring of 64 steps in LDS refilled 32 at a time: read
    // from memory as they are used, by vector or by scalar loads (whose wait
    // is shared with the LDS reads'), they cost a round trip per step
    const double *const tab = a.tab[part];
    double *const out0 = a.out[part][0], *const out1 = a.out[part][1];
    int *const abort_word = a.abort_word;
    if (MULTI && threadIdx.x == 0) s_abort = 0;
    if (threadIdx.x < 128) ((double *)fab)[threadIdx.x] = tab[threadIdx.x];
    for (int t = threadIdx.x; t < 2 * CB; t += 64 * W) xl[t] = T(0);

    // the extended tile: cells, d, F and, for a run that continues another
    // launch, u_j and u_{j-1} (else they start from zero); every load is
    // issued before the first use
    Rows<T, SC, R> co;
    T u0[R], u1[R];
    {
        const T *m = (const T *)a.m, *dn = (const T *)a.dn;
        const double2 *F = (const double2 *)a.F;
        const T *u_in = (const T *)a.u_in, *up_in = (const T *)a.up_in;
        T ca[R + 1], cb[R + 1], d[R];
        double2 f[R];
#pragma unroll
        for (int i = 0; i <= R; ++i) {
            const int sy = gy0 + r0 + i;
            const T *mrow = m + (int64_t)sy * (nx + 1);
            ca[i] = (sy <= ny && gx <= nx) ? mrow[gx] : T(0);
            cb[i] = (sy <= ny && gx + 1 <= nx) ? mrow[gx + 1] : T(0);
        }
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int gy = gy0 + r0 + i;
            const int64_t row = (int64_t)gy * nx;
            u0[i] = u1[i] = d[i] = T(0);
            f[i].x = f[i].y = 0.0;
            if (xin && gy < ny) {
                d[i] = (dn + row)[gx];
                f[i] = (F + row)[gx];
                if (u_in) {
                    u0[i] = (u_in + row)[gx];
                    u1[i] = (up_in + row)[gx];
                }
            }
        }
        co.fold(st, ca, cb, d);
#pragma unroll
        for (int i = 0; i < R; ++i) {
            V2 v;
            v.x = (T)f[i].x;
            v.y = (T)f[i].y;
            fl_all[(r0 + i) * EX + lane] = co.forcing(i, v);
        }
    }
    const int rs = 2 * wv * US + lane + 1, rn = (2 * wv + 3) * US + lane + 1;
    const int wf = (2 * wv + 1) * US + lane + 1, wl = (2 * wv + 2) * US + lane + 1;
    T *const c0 = xl, *const c1 = xl + CB;
    const V2 *fl = fl_all + r0 * EX + lane;

    // the exchange: words of the halo columns this lane fetches (per level,
    // side, row and column of the wave's rows), as offsets into the exchange
    // slots of one parity.  A halo row's columns belong to a diagonal
    // neighbour, whose rows are OY further on (south) or back (north)
    constexpr int NQ = MULTI ? (L::LAND + 63) / 64 : 1;
    int off[NQ];
    word *const slots = (word *)a.slots;
    const int64_t slot_words = (int64_t)2 * BAND;
    const int64_t par_words = slot_words * gridDim.x;
    word *const mine = slots + blockIdx.x * slot_words;
    const int lo_row = nbS ? K : 0, hi_row = nbN ? EY - K : EY;   // rows that are not halo
    if constexpr (MULTI) {
#pragma unroll
        for (int q = 0; q < NQ; ++q) {
            const int e = q * 64 + lane;
            const int lev = e / (2 * R * K), side = e / (R * K) & 1;
            const int i = e / K % R, c = e % K, r = r0 + i;
            const bool south = r < lo_row, north = r >= hi_row;
            const int nb = (side ? 1 : -1) + (south ? -a.tiles_x : (north ? a.tiles_x : 0));
            const int ro = south ? r + OY : (north ? r - OY : r);
            off[q] = e < L::LAND && (side ? nbE : nbW)
                         ? nb * (int)slot_words + lev * BAND + 2 * K * EX + (side ? 0 : K * EY) +
                               ro * K + c
                         : INT32_MIN;
        }
    }
    __syncthreads();
    c0[wf] = u0[0];
    c0[wl] = u0[R - 1];
    __syncthreads();

    auto snapshot = [&](int step, const T(&v)[R]) __attribute__((always_inline)) {   // step: 1-based within the launch
        if (step == a.out_step[0] || step == a.out_step[1]) {
            double *o = step == a.out_step[0] ? out0 : out1;
            const int rb = r0 + opaque_zero();
            const int re = min(hi_row, ny - gy0);
            double *p = o + 2 * ((int64_t)(gy0 + rb) * nx + gx);
            if (xexact) {
#pragma unroll
                for (int i = 0; i < R; ++i) {
                    if (rb + i >= lo_row && rb + i < re) *p = (double)v[i];
                    p += 2 * (int64_t)nx;
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        }
    };

    // publish levels j and j-1 in slot `par`, read the halo from the
    // neighbours' slots `par`, return slot `prev` to the empty pattern;
    // false: a wait gave up
    auto exchange = [&](int par, int prev) __attribute__((always_inline)) -> bool {
        static_assert(2 * K <= 2 * R && K <= R, "halo rows lie in the first and last wave");
        const int lane = lane_ + opaque_zero(), tid = wv * 64 + lane;
        word *const out = mine + par * par_words;
        // the border columns go through LDS, so that they leave in whole
        // lines; the border rows, a line or more each, from registers
        const bool side_l = lane >= K && lane < 2 * K, side_r = lane >= OX && lane < EX - K;
        if (side_l || side_r) {
            word *sb = stage + r0 * K + (side_l ? lane - K : K * EY + lane - OX);
#pragma unroll
            for (int i = 0; i < R; ++i) {
                sb[i * K] = Wd::of(u0[i]);
                sb[2 * K * EY + i * K] = Wd::of(u1[i]);
            }
        }
        // stores of the last exchange's emptied slot are complete before this
        // exchange publishes
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
        auto put_row = [&](int i, int at) __attribute__((always_inline)) {
            st_coh(out + at * EX + lane, Wd::of(u0[i]));
            st_coh(out + BAND + at * EX + lane, Wd::of(u1[i]));
        };
        // rows K .. 2K-1 and EY-2K .. EY-K-1 of the tile, in the first and
        // last wave (and, where 2K > R, the ones beside them)
        if (wv == 0) {
#pragma unroll
            for (int i = K; i < (2 * K < R ? 2 * K : R); ++i) put_row(i, i - K);
        }
        if (2 * K > R && wv == 1) {
#pragma unroll
            for (int i = 0; i < 2 * K - R; ++i) put_row(i, R + i - K);
        }
        if (wv == W - 1) {
#pragma unroll
            for (int i = (R > 2 * K ? R - 2 * K : 0); i < R - K; ++i) put_row(i, i - R + 3 * K);
        }
        if (2 * K > R && wv == W - 2) {
#pragma unroll
            for (int i = 2 * R - 2 * K; i < R; ++i) put_row(i, i - 2 * R + 3 * K);
        }
        {
            constexpr int NS = 2 * K * EY, NT = 64 * W;           // words per level
            word v[(2 * NS + NT - 1) / NT];
#pragma unroll
            for (int q = 0; q * NT < 2 * NS; ++q)
                if (2 * NS % NT == 0 || q * NT + tid < 2 * NS) v[q] = stage[q * NT + tid];
#pragma unroll
            for (int q = 0; q * NT < 2 * NS; ++q) {
                const int t = q * NT + tid;
                if (2 * NS % NT == 0 || t < 2 * NS)
                    st_coh(out + 2 * K * EX + t + (t >= NS ? BAND - NS : 0), v[q]);
            }
        }
        __syncthreads();                                         // the staging is free

        const word *const in = mine + par * par_words;
        // whole halo rows: the south neighbour's last rows before its halo,
        // the north one's first (their halo columns are replaced below)
        const bool south = wv == 0 && nbS, north = wv == W - 1 && nbN;
        const int64_t vstep = slot_words * a.tiles_x;
        const word *const rowsrc = in + (south ? K * EX - vstep : vstep) + lane;
        word t0[NQ], h0[K], h1[K];
#pragma unroll
        for (int i = 0; i < K; ++i) h0[i] = h1[i] = word(0);
        // what has arrived is not read again; the abort word is looked at
        // now and then (a read of it would double the time of a poll)
        bool cols = false, rows = !(south || north);
        for (int polls = 0;;) {
            if (!cols) {
#pragma unroll
                for (int q = 0; q < NQ; ++q)
                    t0[q] = off[q] != INT32_MIN ? ld_coh(in + off[q]) : word(0);
            }
            if (!rows) {
#pragma unroll
                for (int i = 0; i < K; ++i) {
                    h0[i] = ld_coh(rowsrc + i * EX);
                    h1[i] = ld_coh(rowsrc + BAND + i * EX);
                }
            }
            bool miss = a.wait_bias != 0;
#pragma unroll
            for (int q = 0; q < NQ; ++q) miss |= t0[q] == Wd::empty;
            cols = !__any(miss);
            miss = a.wait_bias != 0;
#pragma unroll
            for (int i = 0; i < K; ++i) miss |= h0[i] == Wd::empty || h1[i] == Wd::empty;
            rows = !__any(miss);
            if (cols && rows) break;
            ++polls;
            if (polls >= a.poll_limit ||
                (polls % 16 == 0 && __builtin_amdgcn_readfirstlane(ld_coh(abort_word)) != 0)) {
                st_coh(abort_word, 1);
                s_abort = 1;
                break;
            }
        }
        if (south) {
#pragma unroll
            for (int i = 0; i < K; ++i) {
                u0[i] = Wd::value(h0[i]);
                u1[i] = Wd::value(h1[i]);
            }
        }
        if (north) {
#pragma unroll
            for (int i = 0; i < K; ++i) {
                u0[R - K + i] = Wd::value(h0[i]);
                u1[R - K + i] = Wd::value(h1[i]);
            }
        }
        // halo columns to their lanes, through the wave's part of the staging
        word *const land = stage + wv * L::LAND;
#pragma unroll
        for (int q = 0; q < NQ; ++q)
            if (L::LAND % 64 == 0 || q * 64 + lane < L::LAND) land[q * 64 + lane] = t0[q];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        if ((nbW && lane < K) || (nbE && lane >= EX - K)) {
            const word *la = land + (lane < K ? lane : R * K + lane - (EX - K));
#pragma unroll
            for (int i = 0; i < R; ++i) {
                u0[i] = Wd::value(la[i * K]);
                u1[i] = Wd::value(la[2 * R * K + i * K]);
            }
        }
        c0[wf] = u0[0];
        c0[wl] = u0[R - 1];
        __syncthreads();
        if (s_abort) return false;               // halo values may be missing
        if (prev >= 0) {
#pragma unroll
            for (int q = 0; q * 64 * W < 2 * BAND; ++q) {
                const int t = q * 64 * W + tid;
                if (2 * BAND % (64 * W) == 0 || t < 2 * BAND)
                    st_coh(mine + prev * par_words + t, word(Wd::empty));
            }
        }
        return true;
    };

    // A run of steps ends at every sample step, so that samples are written
    // outside the step loop; a run starts with an exchange (the first has its
    // halo from the load) and has one every K steps.  Two steps a turn (the
    // level arrays swap roles); after a run of odd length the newest level is
    // in u1 and the two arrays swap back.
    double ring = 0.0;
    int par = 0, prev = -1;          // exchange slot (1, 2, 0, 1, ...) and the one before
    for (int done = 0; done < nsteps;) {
        int end = nsteps;
#pragma unroll
        for (int q = 0; q < 2; ++q)
            if (a.out_step[q] > done && a.out_step[q] < end) end = a.out_step[q];
        int left = done > 0 ? 0 : K;
#pragma unroll 1
        for (int j = done; j < end; j += 2, left -= 2) {
            // the ring's other half: fetched half a round ahead, in place a turn ahead
            if ((j >> 1 & 15) == 8 && threadIdx.x < 64) ring = tab[2 * ((j & ~31) + 32) + threadIdx.x];
            if ((j >> 1 & 15) == 15 && threadIdx.x < 64)
                ((double *)fab)[((j & 32) ^ 32) * 2 + threadIdx.x] = ring;
            if (MULTI && left == 0) {
                const int next = par == 2 ? 0 : par + 1;
                if (!exchange(next, prev)) return;
                prev = par = next;
                left = K;
            }
            const double2 f0 = fab[j & 63];
            res_step<T, SC, R>(c0, c1, rs, rn, wf, wl, fl, co, u0, u1, (T)f0.x, (T)f0.y);
            __syncthreads();
            if (j + 1 == end) break;
            const double2 f1 = fab[j + 1 & 63];
            res_step<T, SC, R>(c1, c0, rs, rn, wf, wl, fl, co, u1, u0, (T)f1.x, (T)f1.y);
            __syncthreads();
        }
        if ((end - done) & 1) {
#pragma unroll
            for (int i = 0; i < R; ++i) {
                const T t = u0[i];
                u0[i] = u1[i];
                u1[i] = t;
            }
            if (!MULTI) {            // no exchange refreshes the edge rows
                c0[wf] = u0[0];
                c0[wl] = u0[R - 1];
                __syncthreads();
            }
        }
        done = end;
        snapshot(done, u0);
    }
    T *u_out = (T *)a.u_out, *up_out = (T *)a.up_out;
    if (u_out) {
#pragma unroll
        for (int i = 0; i < R; ++i) {
            const int r = r0 + i, gy = gy0 + r;
            if (xexact && r >= lo_row && r < hi_row && gy < ny) {
                const int64_t row = (int64_t)gy * nx;
                (u_out + row)[gx] = u0[i];
                (up_out + row)[gx] = u1[i];
            }
        }
    }
}

// Before a launch: every slot empty; at an application's first, the abort word
// lowered and the recovery's counters (`words` ints from the abort word on) at 0.
template <typename T>
__global__ __launch_bounds__(256) void k_res_init(typename Word<T>::type *slots, int64_t n,
                                                  int *abort_word, int words)
{
    const int64_t t = (int64_t)blockIdx.x * 256 + threadIdx.x, nt = (int64_t)gridDim.x * 256;
    for (int64_t i = t; i < words; i += nt) abort_word[i] = 0;
    for (int64_t i = t; i < n; i += nt) slots[i] = Word<T>::empty;
}

// Behind a resident run on its stream, where the host does not wait for it:
// returns at once unless the run gave up, else redoes the whole application
// from zero fields, one step after the other on fields in global memory, and
// tells the host (host_word).
// A counter hands out the tasks, (part, step, block of 32 x 64 nodes) in this
// order.  A block's step needs the step before on the block and its eight
// neighbours: tasks of lower tickets, which workgroups that already run have
// taken.  So every wait ends, whatever share of the workgroups is resident, and
// one step's distance between neighbours is all that two field copies need.
// Field values travel as in the exchange (sc1, complete before the flag);
// aborted run and recovery of 48 steps of 700 x 640 in FP64 take 0.98 ms (the
// blocked sweep 0.16), with plain accesses and fences, which write an XCD's L2
// back for every task, 5.2 ms, and in one workgroup 36 ms.
template <typename T>
__global__ __launch_bounds__(1024) void k_res_recover(ResRecover a, Stencil<T> st)
{
    if (*a.abort_word == 0) return;
    __shared__ unsigned s_task[2];
    const int nx = a.nx, ny = a.ny;
    const int bx = (nx + 63) / 64, by = (ny + kRecRows - 1) / kRecRows, nb = bx * by;
    const unsigned long long total = (unsigned long long)a.parts * a.nsteps * nb;
    const T *m = (const T *)a.m, *dn = (const T *)a.dn;
    const double2 *F = (const double2 *)a.F;
    const int lane = threadIdx.x & 63, wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (blockIdx.x == 0 && threadIdx.x == 0) {
        const int n = *a.count + 1;
        *a.count = n;
        __hip_atomic_store(a.host_word, n, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
    // What one wave does for all stands behind branches on scalars: with
    // branches on a lane at the loop's end and start, the compiler sends the
    // other lanes round the loop, through its barriers, while that lane waits
    // for them to leave it.
    for (;;) {
        if (wv == 0) {
            unsigned long long t = 0;
            if (lane == 0)
                t = __hip_atomic_fetch_add(a.ticket, 1ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            s_task[0] = __builtin_amdgcn_readfirstlane((unsigned)t);
            s_task[1] = __builtin_amdgcn_readfirstlane((unsigned)(t >> 32));
        }
        __syncthreads();
        const unsigned lo = __builtin_amdgcn_readfirstlane(s_task[0]);
        const unsigned hi = __builtin_amdgcn_readfirstlane(s_task[1]);
        const unsigned long long task = (unsigned long long)hi << 32 | lo;
        if (task >= total) return;
        const int g = (int)(task / nb), b = (int)(task - (unsigned long long)g * nb);
        const int part = g >= a.nsteps ? 1 : 0, cy = b / bx, cx = b - cy * bx;
        const int64_t j = g - part * a.nsteps;
        if (wv == 0) {
            const int yy = cy + lane / 3 - 1, xx = cx + lane % 3 - 1;
            const bool in = lane < 9 && (unsigned)yy < (unsigned)by && (unsigned)xx < (unsigned)bx;
            const int *flag = a.done + (in ? yy * bx + xx : b);
            while (__any(ld_coh(flag) < g)) __builtin_amdgcn_s_sleep(1);
        }
        __syncthreads();
        // u_j in copy j mod 2, u_{j+1} into the other in place of u_{j-1}; u_0 =
        // u_{-1} = 0 are not read
        const T *u = (const T *)(j & 1 ? a.u1 : a.u0);
        T *un = (T *)(j & 1 ? a.u0 : a.u1);
        const T fa = (T)a.tab[part][2 * j], fb = (T)a.tab[part][2 * j + 1];
        double *o = j + 1 == a.out_step[0] ? a.out[part][0]
                  : j + 1 == a.out_step[1] ? a.out[part][1] : nullptr;
        const int x = cx * 64 + lane;
#pragma unroll
        for (int r = 0; r < kRecRows; r += 16) {
            const int y = cy * kRecRows + r + wv;
            if (y < ny && x < nx) {
                const int64_t i = (int64_t)y * nx + x;
                auto U = [&](int oy, int ox) -> T {
                    return j > 0 && (unsigned)(y + oy) < (unsigned)ny && (unsigned)(x + ox) < (unsigned)nx
                               ? ld_coh(u + i + (int64_t)oy * nx + ox) : T(0);
                };
                const T *c = m + (int64_t)y * (nx + 1) + x;
                T co[6];
                fold_node<T, 3, 2, 6>(st, dn[i], c[0], c[1], c[nx + 1], c[nx + 2], co);
                T acc = co[0] * U(0, 0);
                acc += co[1] * U(0, -1);
                acc += co[2] * U(0, 1);
                acc += co[3] * U(-1, 0);
                acc += co[4] * U(1, 0);
                acc += co[5] * ((U(-1, -1) + U(-1, 1)) + (U(1, -1) + U(1, 1)));
                acc += fa * (dn[i] * (T)F[i].x);
                acc += fb * (dn[i] * (T)F[i].y);
                const T v = acc + (T(1) - T(2) * dn[i]) * (j > 1 ? ld_coh(un + i) : T(0));
                st_coh(un + i, v);
                if (o) o[2 * i] = (double)v;
            }
        }
        __builtin_amdgcn_s_waitcnt(0);         // the block's stores are complete
        __syncthreads();
        if (wv == 0) st_coh(a.done + b, g + 1);
    }
}

}  // namespace

// tile shapes: rows per lane x waves (64 columns), FP64 / FP32
//   0: 12 x 4 / 16 x 4, two workgroups per compute unit; where there is one (and
//      k is at most the rows of a wave), 6 x 8 / 8 x 8 on the same rows: two
//      waves per SIMD hide each other's latency.  512 x 512, k = 6: 0.945
//      against 1.14 us a step in FP64, 0.818 against 0.93 in FP32
//   1:  8 x 8 / 8 x 8, for grids of one tile (up to 48 rows in FP64: 6 x 8)
//   2:  8 x 4 / 8 x 4, 32 rows, for grids of at most one such tile per compute
//      unit: a step takes as long as a compute unit's rows are many.  300 x 300,
//      k = 8: 0.745 against 1.01 us a step in FP64 (on 48 rows; k = 6 and 6 x 8
//      waves: 0.94), 0.604 against 0.75 in FP32; the blocked sweep 0.99 and 1.7
template <typename T>
struct ResShape0;
template <>
struct ResShape0<double> {
    static constexpr int R = 12, W = 4;
};
template <>
struct ResShape0<float> {
    static constexpr int R = 16, W = 4;
};

int res_tile_rows(bool f64, int shape)
{
    if (shape == 2) return 32;
    return shape == 1 ? 64 : (f64 ? ResShape0<double>::R * ResShape0<double>::W
                                  : ResShape0<float>::R * ResShape0<float>::W);
}

size_t res_slot_bytes(bool f64, int k, int shape)
{
    return 3 * 2 * (size_t)res_band(res_tile_rows(f64, shape), k) * (f64 ? sizeof(double) : sizeof(float));
}

int res_tiles(int ny, int nx, int k, bool f64, int shape, int *tiles_x, int *tiles_y)
{
    if (k < 2 || k > 8 || (k & 1)) return 0;
    if (ny <= res_tile_rows(f64, 1) && nx <= kResX) {      // one tile
        if (tiles_x) *tiles_x = 1;
        if (tiles_y) *tiles_y = 1;
        return 1;
    }
    const int rows = res_tile_rows(f64, shape), ox = kResX - 2 * k, oy = rows - 2 * k;
    // tile t covers 64 + t ox columns with the ones before it
    const int tx = nx <= kResX ? 1 : 1 + (nx - kResX + ox - 1) / ox;
    const int tyc = ny <= rows ? 1 : 1 + (ny - rows + oy - 1) / oy;
    if (tiles_x) *tiles_x = tx;
    if (tiles_y) *tiles_y = tyc;
    return (int64_t)tx * tyc > (1 << 20) ? (1 << 20) : tx * tyc;
}

template <typename T, int SC, int R, int W, int K, bool MULTI>
static int res_per_cu()
{
    static const int v = [] {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_sweep2d_res<T, SC, R, W, K, MULTI>,
                                                         64 * W, 0) != hipSuccess)
            nb = 0;
        return nb;
    }();
    return v;
}

template <typename T, int SC>
static int res_slots_sc(int k)
{
    constexpr int R = ResShape0<T>::R, W = ResShape0<T>::W;
    switch (k) {
    case 2: return res_per_cu<T, SC, R, W, 2, true>();
    case 4: return res_per_cu<T, SC, R, W, 4, true>();
    case 6: return res_per_cu<T, SC, R, W, 6, true>();
    default: return res_per_cu<T, SC, R, W, 8, true>();
    }
}

int res_workgroups_per_cu(int k, int sc, bool f64)
{
    if (f64) return sc > 2 ? res_slots_sc<double, 3>(k) : res_slots_sc<double, 2>(k);
    return sc > 2 ? res_slots_sc<float, 3>(k) : res_slots_sc<float, 2>(k);
}

template <typename T, int SC>
static hipError_t launch_res_sc(const ResArgs &a, const Stencil<T> &st, hipStream_t s)
{
    constexpr int R = ResShape0<T>::R, W = ResShape0<T>::W, RH = R / 2, WH = 2 * W;
    const int nt = a.tiles_x * a.tiles_y * a.parts;
#define TDP_RES(R, W, K, MULTI) \
    hipLaunchKernelGGL((k_sweep2d_res<T, SC, R, W, K, MULTI>), dim3(nt), dim3(64 * W), 0, s, a, st)
    if (a.tiles_x * a.tiles_y == 1) {
        if (a.ny <= R * W) TDP_RES(RH, WH, 2, false);
        else TDP_RES(8, 8, 2, false);
    } else if (a.shape == 2) {
        switch (a.k) {
        case 2: TDP_RES(8, 4, 2, true); break;
        case 4: TDP_RES(8, 4, 4, true); break;
        case 6: TDP_RES(8, 4, 6, true); break;
        default: TDP_RES(8, 4, 8, true); break;
        }
    } else if (nt <= a.ncu && a.k <= RH) {
        switch (a.k) {
        case 2: TDP_RES(RH, WH, 2, true); break;
        case 4: TDP_RES(RH, WH, 4, true); break;
        case 6: TDP_RES(RH, WH, 6, true); break;
        default: if constexpr (RH >= 8) TDP_RES(RH, WH, 8, true);
        }
    } else {
        switch (a.k) {
        case 2: TDP_RES(R, W, 2, true); break;
        case 4: TDP_RES(R, W, 4, true); break;
        case 6: TDP_RES(R, W, 6, true); break;
        default: TDP_RES(R, W, 8, true); break;
        }
    }
#undef TDP_RES
    return hipGetLastError();
}

hipError_t launch_sweep2d_res_f64(const ResArgs &a, const Stencil<double> &st, hipStream_t s)
{
    return a.sc > 2 ? launch_res_sc<double, 3>(a, st, s) : launch_res_sc<double, 2>(a, st, s);
}

hipError_t launch_sweep2d_res_f32(const ResArgs &a, const Stencil<float> &st, hipStream_t s)
{
    return a.sc > 2 ? launch_res_sc<float, 3>(a, st, s) : launch_res_sc<float, 2>(a, st, s);
}

int res_recover_blocks(int ny, int nx)
{
    return (ny + kRecRows - 1) / kRecRows * ((nx + 63) / 64);
}

hipError_t launch_res_recover(const ResRecover &a, const Stencil<double> &st,
                              const Stencil<float> &st32, bool f64, hipStream_t s)
{
    const int grid = std::max(1, std::min(a.workgroups, res_recover_blocks(a.ny, a.nx)));
    if (f64)
        hipLaunchKernelGGL(k_res_recover<double>, dim3(grid), dim3(1024), 0, s, a, st);
    else
        hipLaunchKernelGGL(k_res_recover<float>, dim3(grid), dim3(1024), 0, s, a, st32);
    return hipGetLastError();
}

hipError_t launch_res_init(void *slots, size_t bytes, int *abort_word, int words, bool f64,
                           hipStream_t s)
{
    const int64_t n = bytes / (f64 ? 8 : 4);
    const int grid = (int)std::min<int64_t>((n + 1023) / 1024, 2048);
    if (f64)
        hipLaunchKernelGGL(k_res_init<double>, dim3(grid), dim3(256), 0, s,
                           (unsigned long long *)slots, n, abort_word, words);
    else
        hipLaunchKernelGGL(k_res_init<float>, dim3(grid), dim3(256), 0, s, (unsigned *)slots, n,
                           abort_word, words);
    return hipGetLastError();
}

}  // namespace tdp

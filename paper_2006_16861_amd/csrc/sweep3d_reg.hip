// 3-D recurrence sweep, two steps per launch, streamed along axis 0 with the
// rows in registers (tables with centre and face mass entries only: at most
// three stiffness and two mass classes; Table 1 loop, integrator I_acd).
//
// Here a wave owns R rows of 64 nodes along axis 2, one node per lane, and
// walks the planes:
// - x-neighbours come from the adjacent lanes (DPP), y-neighbours from the
//   lane's own rows, z-neighbours from the planes it has passed;
// - of level 0 (u_j) a wave loads its rows and the one above and below straight
//   from memory, so forming level 1 (u_{j+1}) needs no other wave; only the
//   first and last level-1 row of each wave go through LDS, where the waves
//   beside it read them for level 2 (u_{j+2}): one barrier per plane, four LDS
//   accesses per lane;
// - what a plane contributes to its neighbours is summed once: per node the
//   cross (N + S) + (W + E) serves the planes before and after, the pair W + E
//   the rows above and below, the cells' row, column and plane sums the next
//   plane's coefficients.
// In iteration a (a = zb-1 ..) a wave forms level 1 on plane a and level 2 on
// plane a-1, for which the folded coefficients of that plane are carried over
// (two register sets, the loop unrolled by two).  Loads for the next iteration
// are issued as soon as the registers they fill are free.  They are buffer
// loads: rows, columns and planes outside the grid lie outside the buffer's
// range and read as 0, so there is not a branch around any of them; stores
// outside the tile's own nodes are dropped the same way.
//
// It took the place of a form that read every stencil point of both steps
// from LDS (about 47 words per node and plane) and spent 2.3 to 3 us on a plane
// whatever the grid.  Per step, that form and this one: FP64 14.1 and 6.7 us at
// 64^3, 20.7 and 17.4 at 128^3, 146 and 118 at 256^3; FP32 11.4 and 5.2, 16.0 and
// 12.0, 96 and 72 (short applications; in long ones 107 and 61 at 256^3).  There
// it is held by HBM: 1250 MB a launch at 5.8 TB/s in FP64, 689 MB at 5.6 in FP32.
// Two nodes per lane (half a wave to a row, 16-byte loads) halve the memory
// instructions and measured the same: 125.8 and 72.5 us.
//
// A tile is 64 columns x EY = R W rows (columns x0 .. x0+63, x0 = ox bx; rows
// y0 .. y0+EY-1, y0 = (EY-2) by).  Each level costs a column on either side,
// level 2 a row (level 1 has the loaded row beyond the tile): up to 60 columns
// and EY-2 rows are the tile's own, and more where the grid's edge, which
// costs nothing, takes the place of a neighbour: 64 columns are one tile.
// ox is 48 or 56 where that needs no more tiles than 60 does: 64 lanes then
// start on a line (or half or quarter line) of memory, while at 60 every part
// of a store touches a sector more.
// Column blocks are split along axis 0 into runs at the same planes, so that
// neighbours walk together and their halo loads hit L2.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>

#include "tdp_internal.h"
#include "buffer.h"
#include "lanes.h"

namespace tdp {

namespace {

// offset of a lane or row outside the grid: past every buffer's end, doubled too
constexpr unsigned kOutside = 0x7ffffff0u;
constexpr int kAuxNt = 2;            // non-temporal (cache policy bits of buffer accesses)

// the value of the lane to the right; lane 63 gets `last`, which is uniform
__device__ __forceinline__ float east_or(float v, float last)
{
    return __int_as_float(__builtin_amdgcn_update_dpp(__float_as_int(last), __float_as_int(v),
                                                      0x130 /* wave_shl:1 */, 0xF, 0xF, false));
}
__device__ __forceinline__ double east_or(double v, double last)
{
    const long long b = __double_as_longlong(v), l = __double_as_longlong(last);
    const unsigned lo = (unsigned)__builtin_amdgcn_update_dpp((int)l, (int)b, 0x130, 0xF, 0xF, false);
    const unsigned hi = (unsigned)__builtin_amdgcn_update_dpp((int)(l >> 32), (int)(b >> 32), 0x130,
                                                              0xF, 0xF, false);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}
__device__ __forceinline__ float from_lane(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double from_lane(double v, int l)
{
    const long long b = __double_as_longlong(v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)b, l);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(b >> 32), l);
    return __longlong_as_double((long long)(((unsigned long long)hi << 32) | lo));
}

// A field's planes around the one being updated: plane a with the rows beyond
// the wave's own (a[0], a[R+1]), the centres of the plane before (m), and the
// crosses of the plane before and of a.  x-neighbours are shifted out again
// where they are used: kept, they would not fit the registers, and a spilled
// register costs more than its reload, which waits behind every load in flight.
template <typename T, int R>
struct Planes {
    T a[R + 2], m[R], cm[R], ca[R];
};

// crosses of a plane's own rows
template <typename T, int R>
__device__ __forceinline__ void crosses(const T (&b)[R + 2], T (&c)[R])
{
#pragma unroll
    for (int r = 0; r < R; ++r)
        c[r] = (b[r] + b[r + 2]) + (lane_west(b[r + 1]) + lane_east(b[r + 1]));
}

// Fused multiply-adds are written out here (and not left to the compiler), so
// that every instantiation rounds alike and FP32 results are those of the LDS
// form, bit for bit.
#pragma clang fp contract(off)

__device__ __forceinline__ double fma_(double a, double b, double c) { return __builtin_fma(a, b, c); }
__device__ __forceinline__ float fma_(float a, float b, float c) { return __builtin_fmaf(a, b, c); }

// coefficients of a node carried from level 1 to level 2 (see Fold3c in
// sweep3d.hip: opposite faces sum to cx) with d F
template <typename T>
struct Fold {
    T c0, cx, cw, cs, cd, d, fr, fi;
};
// the faces opposite to the west, south and lower one
template <typename T>
struct Opposite {
    T e, n, u;
};

// plane a's rows one step on, the plane after having rows b and crosses cb
template <typename T, int R>
__device__ __forceinline__ void plane_update(const Planes<T, R> &p, const T (&b)[R + 2],
                                             const T (&cb)[R], const Fold<T> (&f)[R],
                                             const Opposite<T> (&o)[R], T s2, T fa, T fb,
                                             const T (&uprev)[R], T (&v)[R])
{
    T w[R + 2], e[R + 2], pr[R + 2];
#pragma unroll
    for (int r = 0; r < R + 2; ++r) {
        w[r] = lane_west(p.a[r]);
        e[r] = lane_east(p.a[r]);
        pr[r] = w[r] + e[r];
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const T edges = (p.cm[r] + cb[r]) + (pr[r] + pr[r + 2]);
        T acc = f[r].cw * w[r + 1];
        acc = fma_(f[r].c0, p.a[r + 1], acc);
        acc = fma_(o[r].e, e[r + 1], acc);
        acc = fma_(f[r].cs, p.a[r], acc);
        acc = fma_(o[r].n, p.a[r + 2], acc);
        acc = fma_(f[r].cd, p.m[r], acc);
        acc = fma_(o[r].u, b[r + 1], acc);
        acc = fma_(f[r].d * s2, edges, acc);
        acc = fma_(fa, f[r].fr, acc);
        acc = fma_(fb, f[r].fi, acc);
        v[r] = fma_(fma_(T(-2), f[r].d, T(1)), uprev[r], acc);
    }
}

template <typename T, int R>
__device__ __forceinline__ void next_plane(Planes<T, R> &p, const T (&b)[R + 2], const T (&c)[R])
{
#pragma unroll
    for (int r = 0; r < R; ++r) {
        p.m[r] = p.a[r + 1];
        p.cm[r] = p.ca[r];
        p.ca[r] = c[r];
    }
#pragma unroll
    for (int r = 0; r < R + 2; ++r) p.a[r] = b[r];
}

template <typename T, int R, int W, int OCC, bool NTS, bool OUT>
__global__ __launch_bounds__(64 * W, OCC) void k_sweep3d_reg2(
    const T *__restrict__ u, const T *__restrict__ um, T *__restrict__ u2o, T *__restrict__ u1o,
    const T *__restrict__ m, const T *__restrict__ dn, const typename V2t<T>::type *__restrict__ F,
    int nz, int ny, int nx, Stencil<T> st, T fa1, T fb1, T fa2, T fb2, double *__restrict__ out1,
    double *__restrict__ out2, int tiles_x, int tiles_y, int ox, int nrun, int per_xcd)
{
    using V2 = typename V2t<T>::type;
    constexpr int EY = R * W, OY = EY - 2, NT = NTS ? kAuxNt : 0;
    // FP64 stores too: their rows are whole lines; FP32 ones are left to L2 to complete
    constexpr int NTW = sizeof(T) == 8 ? NT : 0;
    __shared__ T edge[2][2 * W + 2][64];     // level-1 rows: wave w's first and last at 2w+1, 2w+2

    const int id = blockIdx.x;
    const int wg = (id % 8) * per_xcd + id / 8;
    const int ncb = tiles_x * tiles_y;
    if (wg >= ncb * nrun) return;
    const int run = wg / ncb, cblk = wg - run * ncb;
    const int bx = cblk % tiles_x, by = cblk / tiles_x;
    const int zb = (int)((int64_t)run * nz / nrun), ze = (int)((int64_t)(run + 1) * nz / nrun);
    const int lane = threadIdx.x & 63;
    const int wv = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int r0 = wv * R, x0 = bx * ox, y0 = by * OY;
    const int gx = x0 + lane;
    const int64_t plane = (int64_t)ny * nx, cplane = (int64_t)(ny + 1) * (nx + 1);

    // byte offsets from the tile's first row (the one before y0, if any; cells:
    // y0): rows r0-1 .. r0+R of the fields, the wave's R+1 cell rows, and (lane
    // i: row i) the cell beyond lane 63.  Buffers end with the tile's last row.
    const int yb = y0 > 0 ? y0 - 1 : 0;
    const int64_t base = (int64_t)yb * nx, cbase = (int64_t)y0 * (nx + 1);
    const unsigned pbytes = (unsigned)(min(EY + 2, ny - yb) * nx) * (unsigned)sizeof(T);
    const unsigned cbytes = (unsigned)(min(EY + 1, ny + 1 - y0) * (nx + 1)) * (unsigned)sizeof(T);
    unsigned fo[R + 2], co[R + 1], cxo, so[R];
    const int hx = (64 - ox) / 2;
    const bool xown = gx < nx && (lane >= hx || bx == 0) && (lane < 64 - hx || bx == tiles_x - 1);
#pragma unroll
    for (int i = 0; i < R + 2; ++i) {
        const int gy = y0 + r0 + i - 1;
        fo[i] = (unsigned)gy < (unsigned)ny && gx < nx ? (unsigned)((gy - yb) * nx + gx) * (unsigned)sizeof(T)
                                                       : kOutside;
    }
#pragma unroll
    for (int i = 0; i <= R; ++i) {
        const int sy = r0 + i;
        co[i] = y0 + sy <= ny && gx <= nx ? (unsigned)(sy * (nx + 1) + gx) * (unsigned)sizeof(T)
                                          : kOutside;
    }
    {
        const int sy = r0 + lane;
        cxo = lane <= R && y0 + sy <= ny && x0 + 64 <= nx
                  ? (unsigned)(sy * (nx + 1) + x0 + 64) * (unsigned)sizeof(T) : kOutside;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int t = r0 + r;       // own rows: not the tile's first and last beside a neighbour
        so[r] = xown && (t >= 1 || by == 0) && (t < EY - 1 || by == tiles_y - 1) ? fo[r + 1] : kOutside;
    }

    // the cells beyond lane 63 matter where its column is a node of the last tile
    const bool need63 = bx == tiles_x - 1 && x0 + 64 <= nx;

    T nu[R + 2], nc[R + 1], nx_ = T(0), nup[R], nd[R];
    V2 nf[R];
    // (lim: planes from there on are not fetched)
    auto fetch_u = [&](int p, int lim) __attribute__((always_inline)) {
        const Rsrc b = rsrc_of(u + (int64_t)p * plane + base,
                               (unsigned)p < (unsigned)nz && p < lim ? pbytes : 0);
#pragma unroll
        for (int i = 0; i < R + 2; ++i) bload<0>(nu[i], b, fo[i]);
    };
    auto fetch_c = [&](int p, int lim) __attribute__((always_inline)) {
        const Rsrc b = rsrc_of(m + (int64_t)p * cplane + cbase,
                               (unsigned)p <= (unsigned)nz && p < lim ? cbytes : 0);
#pragma unroll
        for (int i = 0; i <= R; ++i) bload<0>(nc[i], b, co[i]);
        if (need63) bload<0>(nx_, b, cxo);
    };
    auto fetch_node = [&](int p, int lim) __attribute__((always_inline)) {
        const bool in = (unsigned)p < (unsigned)nz && p < lim;
        const Rsrc b0 = rsrc_of(um + (int64_t)p * plane + base, in ? pbytes : 0);
        const Rsrc b1 = rsrc_of(dn + (int64_t)p * plane + base, in ? pbytes : 0);
        const Rsrc b2 = rsrc_of(F + (int64_t)p * plane + base, in ? 2 * pbytes : 0);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            bload<NT>(nup[r], b0, fo[r + 1]);
            bload<NT>(nd[r], b1, fo[r + 1]);
            bload<NT>(nf[r], b2, 2 * fo[r + 1]);
        }
    };

    // cells: of the plane below the current nodes, row pairs q, plane sums s
    // (four cells around a node) and column pairs h (x only)
    T q[R + 1], s4[R], h[R];
    auto cells = [&](T (&q1)[R + 1], T (&s1)[R], T (&h1)[R]) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i <= R; ++i) q1[i] = nc[i] + east_or(nc[i], from_lane(nx_, i));
#pragma unroll
        for (int r = 0; r < R; ++r) {
            s1[r] = q1[r] + q1[r + 1];
            h1[r] = nc[r] + nc[r + 1];
        }
    };

    Planes<T, R> p0, p1;              // levels 0 and 1
    T c[R];
#pragma unroll
    for (int r = 0; r < R + 2; ++r) p0.a[r] = p1.a[r] = T(0);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        p0.m[r] = p0.cm[r] = p0.ca[r] = T(0);
        p1.m[r] = p1.cm[r] = p1.ca[r] = T(0);
    }
    for (int t = threadIdx.x; t < 2 * (2 * W + 2) * 64; t += 64 * W) (&edge[0][0][0])[t] = T(0);
    // planes zb-2 and zb-1 of level 0, the cells below plane zb-1
    fetch_u(zb - 2, nz);
    fetch_c(zb - 1, nz);
    crosses<T, R>(nu, c);
    next_plane<T, R>(p0, nu, c);
    cells(q, s4, h);
    fetch_u(zb - 1, nz);
    crosses<T, R>(nu, c);
    next_plane<T, R>(p0, nu, c);
    fetch_u(zb, nz);
    fetch_c(zb, nz + 1);
    fetch_node(zb - 1, nz);
    __syncthreads();

    Fold<T> kA[R], kB[R];
#pragma unroll
    for (int r = 0; r < R; ++r) kA[r] = kB[r] = Fold<T>{};
    const T s2 = st.s[2];

    auto step = [&](int a, Fold<T> (&k0)[R], const Fold<T> (&k1)[R]) __attribute__((always_inline)) {
        T up[R], u1[R], x[R];
        Opposite<T> opp[R];
        // coefficients of plane a's nodes
        {
            T cq[R + 1], cs[R], ch[R];
            cells(cq, cs, ch);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const T d = nd[r], wd = s4[r], wu = cs[r], w0 = wd + wu;
                const T ws = q[r] + cq[r], ww = h[r] + ch[r];
                const T fw = fma_(st.m[1], ww, st.s[1]), fs = fma_(st.m[1], ws, st.s[1]);
                const T fd = fma_(st.m[1], wd, st.s[1]);
                k0[r].c0 = d * fma_(st.m[0], w0, st.c0);
                k0[r].cx = d * fma_(st.m[1], w0, T(2) * st.s[1]);
                k0[r].cw = d * fw;
                k0[r].cs = d * fs;
                k0[r].cd = d * fd;
                opp[r].e = fma_(-d, fw, k0[r].cx);
                opp[r].n = fma_(-d, fs, k0[r].cx);
                opp[r].u = fma_(-d, fd, k0[r].cx);
                k0[r].d = d;
                k0[r].fr = d * nf[r].x;
                k0[r].fi = d * nf[r].y;
                up[r] = nup[r];
                s4[r] = cs[r];
                h[r] = ch[r];
            }
#pragma unroll
            for (int i = 0; i <= R; ++i) q[i] = cq[i];
        }
        fetch_c(a + 2, ze + 2);
        fetch_node(a + 1, ze + 1);
        __builtin_amdgcn_sched_barrier(0);
        // level 1 on plane a
        crosses<T, R>(nu, c);
        plane_update<T, R>(p0, nu, c, k0, opp, s2, fa1, fb1, up, x);
        const bool zin = (unsigned)a < (unsigned)nz, own = a >= zb && a < ze;
        T vb[R + 2];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            vb[r + 1] = fo[r + 1] != kOutside && zin ? x[r] : T(0);
            u1[r] = p0.m[r];
        }
        edge[a & 1][2 * wv + 1][lane] = vb[1];
        edge[a & 1][2 * wv + 2][lane] = vb[R];
        next_plane<T, R>(p0, nu, c);
        fetch_u(a + 2, ze + 2);
        {
            const Rsrc o = rsrc_of(u1o + (int64_t)a * plane + base, own ? pbytes : 0);
#pragma unroll
            for (int r = 0; r < R; ++r) bstore<NTW>(vb[r + 1], o, so[r]);
        }
        if (OUT && out1 && own) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (so[r] != kOutside)
                    out1[2 * ((int64_t)a * plane + base + so[r] / sizeof(T))] = (double)vb[r + 1];
        }
        // the rows beside the wave's own; two copies, so one barrier orders them
        __syncthreads();
        vb[0] = edge[a & 1][2 * wv][lane];
        vb[R + 1] = edge[a & 1][2 * wv + 3][lane];
        // level 2 on plane a-1 (stored from plane zb on)
        crosses<T, R>(vb, c);
#pragma unroll
        for (int r = 0; r < R; ++r) {
            opp[r].e = k1[r].cx - k1[r].cw;
            opp[r].n = k1[r].cx - k1[r].cs;
            opp[r].u = k1[r].cx - k1[r].cd;
        }
        plane_update<T, R>(p1, vb, c, k1, opp, s2, fa2, fb2, u1, x);
        {
            const Rsrc o = rsrc_of(u2o + (int64_t)(a - 1) * plane + base, a > zb ? pbytes : 0);
#pragma unroll
            for (int r = 0; r < R; ++r) bstore<NTW>(x[r], o, so[r]);
        }
        if (OUT && out2 && a > zb) {
#pragma unroll
            for (int r = 0; r < R; ++r)
                if (so[r] != kOutside)
                    out2[2 * ((int64_t)(a - 1) * plane + base + so[r] / sizeof(T))] = (double)x[r];
        }
        next_plane<T, R>(p1, vb, c);
    };
    // level 1 on planes zb-1 .. ze, level 2 on zb .. ze-1, a plane behind
#pragma unroll 1
    for (int a = zb - 1; a <= ze; a += 2) {
        step(a, kA, kB);
        __builtin_amdgcn_sched_barrier(0);
        if (a + 1 <= ze) step(a + 1, kB, kA);
        __builtin_amdgcn_sched_barrier(0);
    }
}

// workgroups of one instantiation resident per compute unit, queried once
// (sweep3d_stream2_prepare runs the query before any stream capture)
template <typename T, int R, int W, int OCC, bool NTS>
int reg2_per_cu()       // (the form without samples)
{
    static const int v = [] {
        int nb = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&nb, k_sweep3d_reg2<T, R, W, OCC, NTS, false>,
                                                         64 * W, 0) != hipSuccess || nb < 1)
            nb = 1;
        return nb;
    }();
    return v;
}

template <typename T, int R, int W, int OCC>
hipError_t launch_reg2(const Stream2Args &a, const Stencil<T> &st, hipStream_t s)
{
    const int nz = a.n[0], ny = a.n[1], nx = a.n[2];
    constexpr int EY = R * W;
    auto tiles_at = [&](int ox) { return nx <= 64 ? 1 : 1 + (nx - 64 + ox - 1) / ox; };
    const int tiles_x = tiles_at(60);
    const int ox = tiles_at(48) == tiles_x ? 48 : (tiles_at(56) == tiles_x ? 56 : 60);
    const int tiles_y = ny <= EY ? 1 : 1 + (ny - EY + EY - 3) / (EY - 2);
    const int64_t ncb = (int64_t)tiles_x * tiles_y;
    if (!sweep3d_reg2_applies(a.n, a.sc, a.mc) || ncb * nz > ((int64_t)1 << 31) - 1)
        return hipErrorInvalidValue;
    const bool nt = stream_nt((int64_t)7 * sizeof(T) * nz * ny * nx);
    const int64_t slots = (int64_t)(nt ? reg2_per_cu<T, R, W, OCC, true>()
                                       : reg2_per_cu<T, R, W, OCC, false>()) * a.ncu;
    const int nrun = stream2_runs(ncb, nz, a.zc, std::max<int64_t>(slots, 1));
    const int per_xcd = (int)((ncb * nrun + 7) / 8);
#define TDP_REG2(NTS, OUT)                                                                              \
    hipLaunchKernelGGL((k_sweep3d_reg2<T, R, W, OCC, NTS, OUT>), dim3(8 * per_xcd), dim3(64 * W), 0, s, \
                       (const T *)a.u, (const T *)a.up, (T *)a.u2out, (T *)a.u1out,                \
                       (const T *)a.m, (const T *)a.dn, (const typename V2t<T>::type *)a.F, nz,    \
                       ny, nx, st, (T)a.fa[0], (T)a.fb[0], (T)a.fa[1], (T)a.fb[1], a.out1, a.out2, \
                       tiles_x, tiles_y, ox, nrun, per_xcd)
    const bool out = a.out1 || a.out2;
    if (nt) {
        if (out) TDP_REG2(true, true);
        else TDP_REG2(true, false);
    } else {
        if (out) TDP_REG2(false, true);
        else TDP_REG2(false, false);
    }
#undef TDP_REG2
    return hipGetLastError();
}

}  // namespace

// The offsets within a tile (at most 34 rows, with cells one column more; F is
// complex) have to stay below 2^32 bytes.
bool sweep3d_reg2_applies(const int *n, int sc, int mc)
{
    return sc <= 3 && mc <= 2 && (int64_t)34 * (n[2] + 1) * 8 < (int64_t)kOutside;
}

hipError_t launch_sweep3d_reg2_f64(const Stream2Args &a, const Stencil<double> &st, hipStream_t s)
{
    return launch_reg2<double, 2, 8, 2>(a, st, s);
}

// Shape 0: tiles of 16 rows, two rows and four waves per SIMD; else 32 rows, four
// rows and two waves.  Per step 5.2 against 6.5 us at 64^3 (fewer workgroups
// than compute units either way), 12.2 and 12.5 at 128^3, 77 and 72 at 256^3
// (two of 32 rows are halo, not two of 16).
hipError_t launch_sweep3d_reg2_f32(const Stream2Args &a, const Stencil<float> &st, int shape,
                                   hipStream_t s)
{
    return shape == 0 ? launch_reg2<float, 2, 8, 4>(a, st, s) : launch_reg2<float, 4, 8, 2>(a, st, s);
}

void sweep3d_reg2_prepare(bool f64)
{
    if (f64) {
        reg2_per_cu<double, 2, 8, 2, true>();
        reg2_per_cu<double, 2, 8, 2, false>();
    } else {
        reg2_per_cu<float, 2, 8, 4, true>();
        reg2_per_cu<float, 2, 8, 4, false>();
        reg2_per_cu<float, 4, 8, 2, true>();
        reg2_per_cu<float, 4, 8, 2, false>();
    }
}

}  // namespace tdp

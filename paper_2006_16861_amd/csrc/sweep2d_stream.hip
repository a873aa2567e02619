// 2-D recurrence sweep, K steps per launch, streamed along axis 0 (tables
// without corner mass terms; Table 1 loop, integrator I_acd of Def. 2).
//
// A tile of the blocked sweep (sweep_tb.hip) loses k rows and k columns on every
// side to its halo: 32 x 64 nodes at depth 8 keep 16 x 48, so 2.7 updates are
// made for one that counts, and at large grids that, not HBM, sets its pace.
// Here one wave owns a strip of 64 columns, one column per lane, and walks
// down the rows with all K levels in flight: in iteration a it reads row a of
// level 0 (u_j) and forms row a-l of level l (u_{j+l}) for l = 1 .. K, each from
// the three newest rows of the level before.  Only columns are lost, and the
// 2K-2 rows a run starts and ends with: 64 against 64-2K, about 1.6 updates for one
// with K = 8 and runs of 77 rows.  Everything is the wave's own: x-neighbours by
// DPP, rows in registers, no barrier.
//
// Per level a lane keeps the newest two rows and the older one's pair sum; per
// row in flight the folded weights.  These are a ring of K rows and the loop is
// unrolled by K, so they stay in place; F (and d, in FP64) is a ring of rows in
// LDS (a lane reads only what it wrote).  A level's row is finished while the
// next level's is begun.  A row's loads are issued two iterations ahead; the
// loop has no exit inside a turn, since behind one the compiler moves them
// down to their use: runs are K t + 2 rows long, whole turns.  They are buffer
// loads: rows and columns outside the grid lie outside the buffer's range and
// read as 0, where the damping factor 0 keeps every level at 0 (Dirichlet);
// stores of what is not the wave's own are dropped the same way.
//
// us per step, the blocked sweep (32 x 64 tiles in FP64, 128 x 64 in FP32, depth
// 8) and this one: FP64 23.6 and 15.8 at 2999 x 2503, 12.5 and 8.4 to 9.2 at 2000
// x 2000, 7.9 and 6.8 at 1500 x 1600; FP32 13.2 and 9.5, 7.1 and 6.0, 4.6 and 4.35
// at 1500 x 1500.  At 2999 x 2503 it is held by HBM: a launch moves 561 MB (436
// read, 125 written; it cannot do with less than 480) at 4.4 TB/s.  Smaller
// grids are held by the length of a run against the 14 rows it forms beside
// its own, and by latency with two waves per SIMD.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdint>

#include "tdp_internal.h"
#include "buffer.h"
#include "lanes.h"

namespace tdp {

namespace {

// steps per launch and waves per SIMD (183 registers in FP64, 170 in FP32, no
// spills).  At 2999 x 2503 and 2000 x 2000 in FP64 8 steps take 16.7 and 8.4 us
// each, 10 take 16.3 and 9.6 (fewer own columns a strip), 6 take 20.5 and 9.6; in
// FP32 8 take 9.5 and 6.0, 10 take 10.3 and 6.7
constexpr int kSteps = 8, kWaves = 2;
constexpr unsigned kDropped = 0x7ffffff0u;      // offset of a store outside any buffer

// Folded weights of the rows in flight and the update of one node; the two
// forms of sweep_res.hip.  FP64: weights without the damping factor, which is
// applied once; the weight of the edge to the row before serves that row too.
// FP32: premultiplied by d, in the blocked tile's order of operations (its
// results, bit for bit).
template <typename T, int SC, int K>
struct Ring;

template <int SC, int K>
struct Ring<double, SC, K> {
    double wc[K], ww[K], we[K], wy[K], wlast, s2;
    __device__ __forceinline__ void fold(int s, const Stencil<double> &st, double a0, double b0,
                                         double a1, double b1, double dd)
    {
        wlast = wy[s];                       // of the row K before, for its last update
        wc[s] = st.c0 + st.m[0] * ((a0 + b0) + (a1 + b1));
        ww[s] = st.s[1] + st.m[1] * (a0 + a1);
        we[s] = st.s[1] + st.m[1] * (b0 + b1);
        wy[s] = st.s[1] + st.m[1] * (a1 + b1);    // to the row after
        (void)dd;
    }
    __device__ __forceinline__ double2 forcing(int, double2 f) const { return f; }
    // the part of row s's update that needs no row after it, and the rest
    __device__ __forceinline__ double part(int s, double before, double c, double w, double e,
                                           double south, double2 f, double fa, double fb,
                                           double prev) const
    {
        double acc = wc[s] * c;
        acc += ww[s] * w;
        acc += we[s] * e;
        acc += before * south;
        acc += fa * f.x;
        acc += fb * f.y;
        acc += -2.0 * prev;
        return acc;
    }
    __device__ __forceinline__ double rest(int s, double acc, double north, double corners, double2,
                                           double d, double, double, double prev) const
    {
        acc += wy[s] * north;
        if (SC > 2) acc += s2 * corners;
        return d * acc + prev;
    }
    __device__ __forceinline__ double before(int s, bool last) const
    {
        return last ? wlast : wy[(s + K - 1) % K];
    }
};

template <int SC, int K>
struct Ring<float, SC, K> {
    float co[K][5], d[K], s2;
    __device__ __forceinline__ void fold(int s, const Stencil<float> &st, float a0, float b0,
                                         float a1, float b1, float dd)
    {
        fold_node<float, 2, 2, 5>(st, dd, a0, b0, a1, b1, co[s]);
        d[s] = dd;
    }
    __device__ __forceinline__ float2 forcing(int s, float2 f) const
    {
        f.x *= d[s];
        f.y *= d[s];
        return f;
    }
    __device__ __forceinline__ float part(int s, float, float c, float w, float e, float south,
                                          float2, float, float, float) const
    {
        float acc = __builtin_fmaf(co[s][0], c, co[s][1] * w);
        acc = __builtin_fmaf(co[s][2], e, acc);
        return __builtin_fmaf(co[s][3], south, acc);
    }
    __device__ __forceinline__ float rest(int s, float acc, float north, float corners, float2 f,
                                          float, float fa, float fb, float prev) const
    {
        acc = __builtin_fmaf(co[s][4], north, acc);
        if (SC > 2) acc = __builtin_fmaf(d[s] * s2, corners, acc);
        acc = __builtin_fmaf(fa, f.x, acc);
        acc = __builtin_fmaf(fb, f.y, acc);
        return __builtin_fmaf(__builtin_fmaf(-2.0f, d[s], 1.0f), prev, acc);
    }
    __device__ __forceinline__ float before(int, bool) const { return 0.0f; }
};

template <typename T, int SC, int K, int OCC, bool NTS, bool OUT>
__global__ __launch_bounds__(64) __attribute__((amdgpu_waves_per_eu(OCC)))
void k_sweep2d_stream(const T *__restrict__ u, const T *__restrict__ um, T *__restrict__ uo,
                      T *__restrict__ upo, const T *__restrict__ m, const T *__restrict__ dn,
                      const typename V2t<T>::type *__restrict__ F, int ny, int nx, Stencil<T> st,
                      TBCoef cf, int strips, int nrun, int len, int per_xcd)
{
    using V2 = typename V2t<T>::type;
    constexpr int OX = 64 - 2 * K;
    constexpr bool KEEP = sizeof(T) == 4;      // C's x-neighbours too, where registers allow
    // u_{j-1}, d and F are read once: non-temporal where the launch's working
    // set exceeds the 256 MB MALL (2999 x 2503 FP64: 15.8 against 16.7 us a step;
    // in FP32, where it fits, 10.1 against 9.6)
    constexpr int NT = NTS ? 2 : 0;
    // F and, in FP64, d of the rows in flight
    constexpr int KD = sizeof(T) == 8 ? K : 1;
    __shared__ V2 fl[K][64];
    __shared__ T dl[KD][64];

    const int id = blockIdx.x;
    const int wg = (id % 8) * per_xcd + id / 8;
    if (wg >= strips * nrun) return;
    const int run = wg / strips, bx = wg - run * strips;
    const int zb = run * len, ze = min(ny, zb + len);
    const int lane = threadIdx.x;
    const int x0 = bx * OX, gx = x0 + lane;
    const bool xown = gx < nx && (lane >= K || bx == 0) && (lane < 64 - K || bx == strips - 1);
    const unsigned so = xown ? lane * (unsigned)sizeof(T) : kDropped;
    const unsigned rbytes = (unsigned)min(64, nx - x0) * (unsigned)sizeof(T);
    const unsigned cbytes = (unsigned)min(64, nx + 1 - x0) * (unsigned)sizeof(T);

    const int a0 = zb - K + 2, aend = ze + K;
    // rows on their way: iteration a needs row a of level 0 and of the cells,
    // row a-1 of u_{j-1}, d and F
    struct Pre {
        T u, c, um, d;
        V2 f;
    } pre[2];
    auto fetch = [&](Pre &p, int a) __attribute__((always_inline)) {
        const bool in0 = (unsigned)a < (unsigned)ny && a < aend;
        const bool in1 = (unsigned)(a - 1) < (unsigned)ny && a < aend;
        const int64_t r0 = (int64_t)a * nx + x0, r1 = r0 - nx;
        bload<0>(p.u, rsrc_of(u + r0, in0 ? rbytes : 0), lane * (unsigned)sizeof(T));
        bload<0>(p.c, rsrc_of(m + r0 + a, (unsigned)a <= (unsigned)ny && a < aend ? cbytes : 0),
                 lane * (unsigned)sizeof(T));
        bload<NT>(p.um, rsrc_of(um + r1, in1 ? rbytes : 0), lane * (unsigned)sizeof(T));
        bload<NT>(p.d, rsrc_of(dn + r1, in1 ? rbytes : 0), lane * (unsigned)sizeof(T));
        bload<NT>(p.f, rsrc_of(F + r1, in1 ? 2 * rbytes : 0), lane * (unsigned)sizeof(V2));
    };

    Ring<T, SC, K> co;
    co.s2 = st.s[2];
    // level q's newest two rows C and S, C's x-neighbours, S's pair sum
    T S[K], C[K], wC[KEEP ? K : 1], eC[KEEP ? K : 1], pS[K];
    T ca, cb;                      // the cells of the last cell row
    {
        Pre p0, p1;
        fetch(p0, a0 - 2);
        fetch(p1, a0 - 1);
        fetch(pre[0], a0);
        fetch(pre[1], a0 + 1);
#pragma unroll
        for (int q = 0; q < K; ++q) {
            S[q] = C[q] = pS[q] = T(0);
            if (KEEP) wC[q] = eC[q] = T(0);
            // (levels below the first rows start from zeros: these rows lie
            // outside what reaches the run's own)
            co.fold(q, st, T(0), T(0), T(0), T(0), T(0));
            fl[q][lane].x = fl[q][lane].y = T(0);
            if (KD > 1) dl[q % KD][lane] = T(0);
        }
        S[0] = p0.u;
        pS[0] = lane_west(p0.u) + lane_east(p0.u);
        C[0] = p1.u;
        if (KEEP) {
            wC[0] = lane_west(p1.u);
            eC[0] = lane_east(p1.u);
        }
        ca = p1.c;
        cb = lane_east(p1.c);
        co.fold(K - 1, st, T(0), T(0), ca, cb, T(0));   // the edge weight to the first row
    }
    auto sample = [&](int l, int row, T v) __attribute__((always_inline)) {
        if (row < zb || row >= ze) return;
#pragma unroll
        for (int i = 0; i < 2; ++i)
            if (cf.out_step[i] == l && xown) cf.out[i][2 * ((int64_t)row * nx + gx)] = (double)v;
    };
    auto iter = [&](int a, int i) __attribute__((always_inline)) {
        Pre &p = pre[i & 1];
        T N = p.u, prev = p.um;
        {
            const T a1 = p.c, b1 = lane_east(p.c);
            co.fold(i, st, ca, cb, a1, b1, p.d);
            ca = a1;
            cb = b1;
        }
        V2 f = co.forcing(i, p.f), fn = fl[(i + K - 1) % K][lane];
        T d = p.d, dn1 = KD > 1 ? dl[(i + K - 1) % KD][lane] : T(0);
        fl[i][lane] = f;
        if (KD > 1) dl[i % KD][lane] = d;
        fetch(p, a + 2);
        T cw = KEEP ? wC[0] : lane_west(C[0]), ce = KEEP ? eC[0] : lane_east(C[0]);
        T acc = co.part(i, co.before(i, false), C[0], cw, ce, S[0], f, (T)cf.fa[0], (T)cf.fb[0], prev);
#pragma unroll
        for (int l = 1; l <= K; ++l) {
            // level l's row is finished while the next level's is begun: the
            // first is a chain of dependent operations
            const int q = l - 1, s = (i + K - q) % K, sn = (s + K - 1) % K, n = l < K ? l : q;
            const T Nw = lane_west(N), Ne = lane_east(N);
            const T v = co.rest(s, acc, N, pS[q] + (Nw + Ne), f, d, (T)cf.fa[q], (T)cf.fb[q], prev);
            prev = S[q];
            pS[q] = cw + ce;
            S[q] = C[q];
            C[q] = N;
            if (!KEEP) asm volatile("" : "+v"(C[q]));     // shifted again when it is used
            if (KEEP) {
                wC[q] = Nw;
                eC[q] = Ne;
            }
            N = v;
            if (l < K) {
                f = fn;
                d = dn1;
                if (l + 1 < K) {
                    fn = fl[(sn + K - 1) % K][lane];
                    if (KD > 1) dn1 = dl[(sn + K - 1) % KD][lane];
                }
                cw = KEEP ? wC[n] : lane_west(C[n]);
                ce = KEEP ? eC[n] : lane_east(C[n]);
                acc = co.part(sn, co.before(sn, l + 1 == K), C[n], cw, ce, S[n], f, (T)cf.fa[n],
                              (T)cf.fb[n], prev);
            }
            if (l >= K - 1) {
                const int row = a - l;
                const Rsrc b = rsrc_of((l == K ? uo : upo) + (int64_t)row * nx + x0,
                                       row >= zb && row < ze ? rbytes : 0);
                bstore<0>(v, b, so);
            }
            if (OUT) sample(l, a - l, v);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
#pragma unroll 1
    for (int a = a0; a < aend; a += K) {
#pragma unroll
        for (int i = 0; i < K; ++i) {
            iter(a + i, i);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
}

// Strips of 64 columns (the last one's lane 63 has no cell beyond it: 63 nodes)
// and the rows of a run, such that the rounds that the runs take on the
// resident waves, times a run's turns of the loop, are fewest: runs of K t + 2
// rows take K (t + 2) iterations, whole turns.  Returns that number.
int stream_split(int ny, int nx, int ncu, int *strips, int *len)
{
    constexpr int K = kSteps, OX = 64 - 2 * K;
    *strips = nx <= 63 ? 1 : 1 + (nx - 63 + OX - 1) / OX;
    const int64_t slots = (int64_t)ncu * 4 * kWaves;
    int64_t best = INT64_MAX;
    for (int t = 0; t < 4096; ++t) {
        const int64_t wgs = (int64_t)*strips * ((ny + K * t + 1) / (K * t + 2));
        const int64_t turns = (wgs + slots - 1) / slots * (t + 2);
        if (turns < best) {
            best = turns;
            *len = K * t + 2;
        }
        if (K * t + 2 >= ny) break;
    }
    return (int)std::min<int64_t>(best, INT32_MAX);
}

template <typename T, int SC, int K, int OCC>
hipError_t launch_stream(const TBArgs &a, const Stencil<T> &st, int ncu, hipStream_t s)
{
    static_assert(K == kSteps && OCC == kWaves, "the split is theirs");
    int strips, len = 2;
    stream_split(a.ny, a.nx, ncu, &strips, &len);
    const int nrun = (a.ny + len - 1) / len;
    const int per_xcd = (strips * nrun + 7) / 8;
#define TDP_STREAM(NTS, OUT)                                                                                 \
    hipLaunchKernelGGL((k_sweep2d_stream<T, SC, K, OCC, NTS, OUT>), dim3(8 * per_xcd), dim3(64), 0, s,       \
                       (const T *)a.u_in, (const T *)a.up_in, (T *)a.u_out, (T *)a.up_out,              \
                       (const T *)a.m, (const T *)a.dn, (const typename V2t<T>::type *)a.F, a.ny, a.nx, \
                       st, a.cf, strips, nrun, len, per_xcd)
    const bool out = a.cf.out_step[0] || a.cf.out_step[1];
    if ((int64_t)8 * sizeof(T) * a.ny * a.nx > ((int64_t)256 << 20)) {
        if (out) TDP_STREAM(true, true);
        else TDP_STREAM(true, false);
    } else {
        if (out) TDP_STREAM(false, true);
        else TDP_STREAM(false, false);
    }
#undef TDP_STREAM
    return hipGetLastError();
}

}  // namespace

int sweep2d_stream_depth() { return kSteps; }
int sweep2d_stream_turns(int ny, int nx, int ncu)
{
    int strips, len;
    return stream_split(ny, nx, ncu, &strips, &len);
}
hipError_t launch_sweep2d_stream_f64(const TBArgs &a, const Stencil<double> &st, int ncu, hipStream_t s)
{
    return a.sc > 2 ? launch_stream<double, 3, kSteps, kWaves>(a, st, ncu, s) : launch_stream<double, 2, kSteps, kWaves>(a, st, ncu, s);
}
hipError_t launch_sweep2d_stream_f32(const TBArgs &a, const Stencil<float> &st, int ncu, hipStream_t s)
{
    return a.sc > 2 ? launch_stream<float, 3, kSteps, kWaves>(a, st, ncu, s) : launch_stream<float, 2, kSteps, kWaves>(a, st, ncu, s);
}

}  // namespace tdp

// flb_step.hip -- the fused noisy D2Q9 step and the state utility kernels.
//
// One thread updates one site per row it owns: it gathers the nine
// post-collision values of the previous step from the neighbours x - v_i
// (streaming, Eq. 1, in pull form), forms the moments of Eq. (3), relaxes the
// non-conserved ones towards Eq. (10) by their own 1/tau^a (Eq. 5), adds the
// noise of Eq. (8) on moments 3..8, transforms back with n_i^a = w_i m_i^a
// and stores the nine new values at x.  Population planes are SoA, so every
// wave's loads and stores are contiguous 64-site runs of one plane.  There is
// no dense contraction here: the 9x9 transforms are written out using the
// sign structure of Eq. (9), about forty adds each way.
#include <type_traits>

#include "flb_collide.h"

namespace flbdev {

struct StepArgs {
    const void *src;
    void *dst;
    const LatticeParams *params;
    const StepItem *items;
    const uint32_t *step;  // step counter of the state in src
    uint32_t *step_next;   // ... and of the one in dst
    uint32_t key0, key1;
};

// Every step kernel calls this first: the launch's one writer of the new
// state's counter.  (The counter belongs to the population buffer, so a launch
// never writes the one its other blocks read, and none is needed to advance
// it: 256^2, 100 periods of ten steps and a sample, 3.95 ms with such a launch
// after each period's steps, 3.70 without.)
__device__ __forceinline__ void advance_counter(const StepArgs &g, int steps)
{
    if (blockIdx.x == 0 && threadIdx.x == 0) *g.step_next = *g.step + (uint32_t)steps;
}

static StepArgs step_args(const DeviceView &v, const StepItem *items)
{
    StepArgs a;
    a.src = v.pops[v.cur];
    a.dst = v.pops[v.cur ^ 1];
    a.params = v.params;
    a.items = items;
    a.step = v.step + v.cur;
    a.step_next = v.step + (v.cur ^ 1);
    a.key0 = (uint32_t)(v.seed & 0xFFFFFFFFu);
    a.key1 = (uint32_t)(v.seed >> 32);
    return a;
}

// V consecutive values of one storage row, as one vector access.
template <typename T, int V> struct Vec {
    typedef T type __attribute__((ext_vector_type(V)));
};
template <typename T> struct Vec<T, 1> {
    typedef T type;
};
template <typename T, int V>
__device__ __forceinline__ T lane(const typename Vec<T, V>::type &v, int k)
{
    if constexpr (V == 1) return v;
    else return v[k];
}

// A block covers a tile of TX threads along x by kThreads/TX rows; a thread
// updates V consecutive sites x0 .. x0+V-1 of its row.  Storage rows have a
// pitch px (a multiple of 4), so the V values of one population are one
// aligned vector access.  A population streaming along +x needs the value
// left of the group (x0 - 1, periodic) and one streaming along -x the value
// right of it (x0 + V): one extra scalar load each.  A group reaching past
// the last site of a row (nx not a multiple of V) takes the site-by-site path.
// Element `off` of a lattice's buffer through a 32-bit byte offset (a
// lattice's populations are limited to 4 GiB), so that the address is a
// scalar base plus a 32-bit vector offset.
template <typename U, typename T> __device__ __forceinline__ const U *at(const T *base, uint32_t off)
{
    return reinterpret_cast<const U *>(reinterpret_cast<const char *>(base) + off * (uint32_t)sizeof(T));
}
template <typename U, typename T> __device__ __forceinline__ U *at(T *base, uint32_t off)
{
    return reinterpret_cast<U *>(reinterpret_cast<char *>(base) + off * (uint32_t)sizeof(T));
}

template <int S, bool NT, bool NOISE, int TX, int V>
__global__ __launch_bounds__(kThreads) void step_kernel(StepArgs g)
{
    using T = typename Codec<S>::T;
    using VT = typename Vec<T, V>::type;
    constexpr int TH = kThreads / TX;
    advance_counter(g, 1);
    const StepItem it = g.items[blockIdx.x];
    if (it.lattice < 0) return;
    const LatticeParams &P = g.params[it.lattice];
    const int nx = P.nx, ny = P.ny;
    const uint32_t px = (uint32_t)P.px;
    const int tx = it.tile % P.tiles_x, ty = it.tile / P.tiles_x;
    const int x0 = (tx * TX + (int)(threadIdx.x % TX)) * V;
    const int y = ty * TH + (int)(threadIdx.x / TX);
    if (x0 >= nx || y >= ny) return;  // no barriers below: a thread may leave early
    // wave-uniform bases and unsigned 32-bit offsets: addresses are a scalar
    // base plus a vector offset, no 64-bit arithmetic per access
    const T *__restrict__ src = (const T *)g.src + P.base;
    T *__restrict__ dst = (T *)g.dst + P.base;
    const uint32_t plane = (uint32_t)P.plane;
    const uint32_t t = *g.step;
    const uint32_t ym = (y == 0) ? ny - 1 : y - 1;
    const uint32_t yp = (y == ny - 1) ? 0 : y + 1;
    const uint32_t rc = (uint32_t)y * px, rm = ym * px, rp = yp * px;
    const uint32_t ux0 = (uint32_t)x0;
    const uint32_t xm = (x0 == 0) ? nx - 1 : x0 - 1;  // left of the group
    const uint32_t site0 = (uint32_t)(y * nx + x0);   // noise counter of site x0

    if (x0 + V <= nx) {
        const uint32_t xr = (x0 + V == nx) ? 0u : (uint32_t)(x0 + V);  // right of the group
        // pull: population i arrives from x - v_i.  With streaming stores the
        // group's own values are read with the non-temporal hint too; the
        // edge values stay ordinary loads, as their lines are shared with the
        // neighbouring groups.
        const VT a0 = gload<NT>(at<VT>(src, rc + ux0));
        const VT a1 = gload<NT>(at<VT>(src, 1 * plane + rc + ux0));
        const VT a2 = gload<NT>(at<VT>(src, 2 * plane + rm + ux0));
        const VT a3 = gload<NT>(at<VT>(src, 3 * plane + rc + ux0));
        const VT a4 = gload<NT>(at<VT>(src, 4 * plane + rp + ux0));
        const VT a5 = gload<NT>(at<VT>(src, 5 * plane + rm + ux0));
        const VT a6 = gload<NT>(at<VT>(src, 6 * plane + rm + ux0));
        const VT a7 = gload<NT>(at<VT>(src, 7 * plane + rp + ux0));
        const VT a8 = gload<NT>(at<VT>(src, 8 * plane + rp + ux0));
        const T e1 = *at<T>(src, 1 * plane + rc + xm), e5 = *at<T>(src, 5 * plane + rm + xm);
        const T e8 = *at<T>(src, 8 * plane + rp + xm);
        const T e3 = *at<T>(src, 3 * plane + rc + xr), e6 = *at<T>(src, 6 * plane + rm + xr);
        const T e7 = *at<T>(src, 7 * plane + rp + xr);
        T o[9][V];
#pragma unroll
        for (int k = 0; k < V; ++k) {
            float d[9];
            d[0] = Work<S>::in(lane<T, V>(a0, k));
            d[2] = Work<S>::in(lane<T, V>(a2, k));
            d[4] = Work<S>::in(lane<T, V>(a4, k));
            d[1] = Work<S>::in(k > 0 ? lane<T, V>(a1, k - 1) : e1);
            d[5] = Work<S>::in(k > 0 ? lane<T, V>(a5, k - 1) : e5);
            d[8] = Work<S>::in(k > 0 ? lane<T, V>(a8, k - 1) : e8);
            d[3] = Work<S>::in(k < V - 1 ? lane<T, V>(a3, k + 1) : e3);
            d[6] = Work<S>::in(k < V - 1 ? lane<T, V>(a6, k + 1) : e6);
            d[7] = Work<S>::in(k < V - 1 ? lane<T, V>(a7, k + 1) : e7);
            update_site<NOISE, S>(d, P, site0 + (uint32_t)k, t, g.key0, g.key1);
#pragma unroll
            for (int i = 0; i < 9; ++i) o[i][k] = Work<S>::out(d[i]);
        }
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            VT v;
            if constexpr (V == 1) {
                v = o[i][0];
            } else {
#pragma unroll
                for (int k = 0; k < V; ++k) v[k] = o[i][k];
            }
            gstore<NT>(at<VT>(dst, i * plane + rc + ux0), v);
        }
    } else {
        for (int x = x0; x < nx; ++x) {
            const uint32_t ux = (uint32_t)x;
            const uint32_t xl = (x == 0) ? nx - 1 : x - 1, xr = (x == nx - 1) ? 0 : x + 1;
            float d[9];
            d[0] = Work<S>::in(*at<T>(src, rc + ux));
            d[1] = Work<S>::in(*at<T>(src, 1 * plane + rc + xl));
            d[2] = Work<S>::in(*at<T>(src, 2 * plane + rm + ux));
            d[3] = Work<S>::in(*at<T>(src, 3 * plane + rc + xr));
            d[4] = Work<S>::in(*at<T>(src, 4 * plane + rp + ux));
            d[5] = Work<S>::in(*at<T>(src, 5 * plane + rm + xl));
            d[6] = Work<S>::in(*at<T>(src, 6 * plane + rm + xr));
            d[7] = Work<S>::in(*at<T>(src, 7 * plane + rp + xr));
            d[8] = Work<S>::in(*at<T>(src, 8 * plane + rp + xl));
            update_site<NOISE, S>(d, P, (uint32_t)(y * nx + x), t, g.key0, g.key1);
#pragma unroll
            for (int i = 0; i < 9; ++i) gstore<NT>(at<T>(dst, i * plane + rc + ux), Work<S>::out(d[i]));
        }
    }
}

template <int S, bool NT, bool NOISE>
static hipError_t launch_step_tiles(const StepArgs &a, int nitems, int tx, int v, hipStream_t s)
{
    const dim3 grid(nitems), block(kThreads);
#define FLB_TILE(TX_, V_)                                                                     \
    if (tx == TX_ && v == V_) {                                                               \
        hipLaunchKernelGGL((step_kernel<S, NT, NOISE, TX_, V_>), grid, block, 0, s, a);       \
        return hipGetLastError();                                                             \
    }
    FLB_TILE(64, 1)
    FLB_TILE(128, 1)
    FLB_TILE(256, 1)
    FLB_TILE(64, 2)
    FLB_TILE(128, 2)
    FLB_TILE(256, 2)
    FLB_TILE(64, 4)
    FLB_TILE(128, 4)
    FLB_TILE(256, 4)
#undef FLB_TILE
    return hipErrorInvalidValue;
}

bool step_tile_supported(int tx, int v)
{
    return (tx == 64 || tx == 128 || tx == 256) && (v == 1 || v == 2 || v == 4);
}

hipError_t launch_step(const DeviceView &v, const StepItem *items, int nitems, int tile_w,
                       int sites, bool nontemporal, bool noise, hipStream_t s)
{
    const StepArgs a = step_args(v, items);
#define FLB_SEL(S_)                                                                              \
    if (v.storage == S_) {                                                                       \
        if (nontemporal)                                                                         \
            return noise ? launch_step_tiles<S_, true, true>(a, nitems, tile_w, sites, s)        \
                         : launch_step_tiles<S_, true, false>(a, nitems, tile_w, sites, s);      \
        return noise ? launch_step_tiles<S_, false, true>(a, nitems, tile_w, sites, s)           \
                     : launch_step_tiles<S_, false, false>(a, nitems, tile_w, sites, s);         \
    }
    FLB_SEL(kF32)
    FLB_SEL(kBF16)
    FLB_SEL(kF16)
#undef FLB_SEL
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------
// Two steps per launch (time blocking).  A block owns a tile of TW x TH
// sites.  Phase 1 collides the tile and the one-site ring around it at time
// t (each site pulled from HBM as in the one-step kernel, the ring
// recomputed by the neighbouring blocks too) and keeps the post-collision
// values in LDS in the storage format; phase 2 pulls the tile's values from
// LDS, collides them at t + 1 and stores them.  Every site goes through the
// same update function, noise counters and storage rounding as in two
// one-step launches, so the results are the same; the populations cross HBM
// once per two steps.
//
// Each thread collides the same tile sites in both phases (and one ring
// site in phase 1), so the rest population, which streams from the site
// itself, stays in a register: LDS holds planes 1..8 only (38 KB for a
// 64 x 16 tile in FP32).  All of a thread's phase-1 loads are
// issued before its first collision.
// ---------------------------------------------------------------------
constexpr int kStep2Threads = 512;

// Tile shapes of the two-step kernel: TW x TH = 1024 sites, TW a power of
// two.  Fixed carries the shape at compile time; Dyn at run time, so that
// one kernel body serves tiles of several shapes (the kernel's registers
// stay those of one shape).
template <int TW_, int TH_> struct Fixed {
    static_assert(TW_ * TH_ == 1024 && (TW_ & (TW_ - 1)) == 0, "tile shape");
    static constexpr int tw = TW_, th = TH_, rw = TW_ + 2, rn = (TW_ + 2) * (TH_ + 2);
    static constexpr int lg = TW_ == 32 ? 5 : TW_ == 64 ? 6 : TW_ == 128 ? 7 : 8;
};
struct Dyn {
    int tw, th, rw, rn, lg;
    __device__ explicit Dyn(int lg_) : tw(1 << lg_), th(1024 >> lg_), rw(tw + 2),
                                       rn((tw + 2) * (th + 2)), lg(lg_) {}
};

// region coordinates of the h-th site of the one-site ring around a tile
template <class SH>
__device__ __forceinline__ void ring_site(const SH &sh, int h, int &rx, int &ry)
{
    const int RW = sh.rw, TH = sh.th;
    if (h < RW) {
        ry = 0;
        rx = h;
    } else if (h < 2 * RW) {
        ry = TH + 1;
        rx = h - RW;
    } else if (h < 2 * RW + TH) {
        ry = h - 2 * RW + 1;
        rx = 0;
    } else {
        ry = h - 2 * RW - TH + 1;
        rx = RW - 1;
    }
}

// One tile's two steps; mid holds 8 x sh.rn values of LDS (planes 1..8
// after phase 1, plane-major).
template <int S, bool NT, bool NOISE, class SH>
__device__ __forceinline__ void step2_tile(const StepArgs &g, StepItem it, const SH sh,
                                           typename Codec<S>::T *__restrict__ mid)
{
    using T = typename Codec<S>::T;
    const int TW = sh.tw, TH = sh.th, RW = sh.rw, RN = sh.rn;
    constexpr int NTILE = 1024;
    const int NRING = RN - NTILE;              // at most 276 (128 x 8), below the thread count
    constexpr int KT = NTILE / kStep2Threads;  // tile sites per thread
    constexpr int K = KT + 1;                  // phase-1 sites per thread: tile sites, then a ring site
    static_assert(NTILE % kStep2Threads == 0, "tile shape");
    const LatticeParams &P = g.params[it.lattice];
    const int nx = P.nx, ny = P.ny;
    const int tiles_x = (nx + TW - 1) >> sh.lg;
    const int x0 = (it.tile % tiles_x) * TW, y0 = (it.tile / tiles_x) * TH;
    const T *__restrict__ src = (const T *)g.src + P.base;
    T *__restrict__ dst = (T *)g.dst + P.base;
    const uint32_t plane = (uint32_t)P.plane, px = (uint32_t)P.px;
    const uint32_t t = *g.step;
    const int tid = threadIdx.x;

    // An interior tile: the region and every site it pulls from lie inside
    // the lattice, so no coordinate wraps and each plane's pull is one
    // fixed shift of the site's own offset (block-uniform test).
    const bool interior = x0 >= 2 && y0 >= 2 && x0 + TW + 2 <= nx && y0 + TH + 2 <= ny;

    // phase-1 sites: region index and (wrapped) lattice coordinates
    int xs[K], ys[K], rs[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int rx, ry;
        if (k < KT) {
            const int o = tid + k * kStep2Threads;
            ry = (o >> sh.lg) + 1;
            rx = (o & (TW - 1)) + 1;
        } else {
            ring_site(sh, tid < NRING ? tid : 0, rx, ry);
        }
        rs[k] = ry * RW + rx;
        xs[k] = x0 - 1 + rx;
        ys[k] = y0 - 1 + ry;
    }
    if (!interior) {
        // wrap (x >= -1): at most one subtraction unless the lattice is
        // smaller than a tile
#pragma unroll
        for (int k = 0; k < K; ++k) {
            int x = xs[k], y = ys[k];
            x = x < 0 ? x + nx : x;
            y = y < 0 ? y + ny : y;
            while (x >= nx) x -= nx;
            while (y >= ny) y -= ny;
            xs[k] = x;
            ys[k] = y;
        }
    }
    // per-plane bases (wave-uniform) and byte offsets within a plane
    const char *sp[9];
    char *dp[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        sp[i] = reinterpret_cast<const char *>(src) + (size_t)i * plane * sizeof(T);
        dp[i] = reinterpret_cast<char *>(dst) + (size_t)i * plane * sizeof(T);
    }
    constexpr uint32_t E = sizeof(T);
    T raw[K][9];
    if (interior) {
        // plane i pulls from x - v_i: its base shifted by -(v_iy px + v_ix)
        // values, so one vector offset serves all nine loads of a site
        const int64_t row = (int64_t)px * E;
        const char *const sh0 = sp[0];
        const char *const sh1 = sp[1] - (int64_t)E;
        const char *const sh2 = sp[2] - row;
        const char *const sh3 = sp[3] + (int64_t)E;
        const char *const sh4 = sp[4] + row;
        const char *const sh5 = sp[5] - row - (int64_t)E;
        const char *const sh6 = sp[6] - row + (int64_t)E;
        const char *const sh7 = sp[7] + row + (int64_t)E;
        const char *const sh8 = sp[8] + row - (int64_t)E;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (k == KT && tid >= NRING) break;
            const uint32_t o = ((uint32_t)ys[k] * px + (uint32_t)xs[k]) * E;
            raw[k][0] = *reinterpret_cast<const T *>(sh0 + o);
            raw[k][1] = *reinterpret_cast<const T *>(sh1 + o);
            raw[k][2] = *reinterpret_cast<const T *>(sh2 + o);
            raw[k][3] = *reinterpret_cast<const T *>(sh3 + o);
            raw[k][4] = *reinterpret_cast<const T *>(sh4 + o);
            raw[k][5] = *reinterpret_cast<const T *>(sh5 + o);
            raw[k][6] = *reinterpret_cast<const T *>(sh6 + o);
            raw[k][7] = *reinterpret_cast<const T *>(sh7 + o);
            raw[k][8] = *reinterpret_cast<const T *>(sh8 + o);
        }
    } else {
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (k == KT && tid >= NRING) break;
        const int x = xs[k], y = ys[k];
        const uint32_t ux = (uint32_t)x * E;
        const uint32_t xm = (uint32_t)(x == 0 ? nx - 1 : x - 1) * E;
        const uint32_t xr = (uint32_t)(x == nx - 1 ? 0 : x + 1) * E;
        const uint32_t rc = (uint32_t)y * px * E, rm = (uint32_t)(y == 0 ? ny - 1 : y - 1) * px * E;
        const uint32_t rp = (uint32_t)(y == ny - 1 ? 0 : y + 1) * px * E;
        raw[k][0] = *reinterpret_cast<const T *>(sp[0] + (rc + ux));
        raw[k][1] = *reinterpret_cast<const T *>(sp[1] + (rc + xm));
        raw[k][2] = *reinterpret_cast<const T *>(sp[2] + (rm + ux));
        raw[k][3] = *reinterpret_cast<const T *>(sp[3] + (rc + xr));
        raw[k][4] = *reinterpret_cast<const T *>(sp[4] + (rp + ux));
        raw[k][5] = *reinterpret_cast<const T *>(sp[5] + (rm + xm));
        raw[k][6] = *reinterpret_cast<const T *>(sp[6] + (rm + xr));
        raw[k][7] = *reinterpret_cast<const T *>(sp[7] + (rp + xr));
        raw[k][8] = *reinterpret_cast<const T *>(sp[8] + (rp + xm));
    }
    }
    T own[KT];  // plane 0 of the tile sites after phase 1, in the storage format
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (k == KT && tid >= NRING) break;
        float d[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) d[i] = Work<S>::in(raw[k][i]);
        update_site<NOISE, S>(d, P, (uint32_t)(ys[k] * nx + xs[k]), t, g.key0, g.key1);
        if (k < KT) own[k] = Work<S>::out(d[0]);
#pragma unroll
        for (int i = 1; i < 9; ++i) mid[(i - 1) * RN + rs[k]] = Work<S>::out(d[i]);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        const int o = tid + k * kStep2Threads;
        const int oy = o >> sh.lg, ox = o & (TW - 1);
        const int x = x0 + ox, y = y0 + oy;
        if (x >= nx || y >= ny) continue;
        const int c = rs[k];
        float d[9];
        d[0] = Work<S>::in(own[k]);
        d[1] = Work<S>::in(mid[0 * RN + c - 1]);
        d[2] = Work<S>::in(mid[1 * RN + c - RW]);
        d[3] = Work<S>::in(mid[2 * RN + c + 1]);
        d[4] = Work<S>::in(mid[3 * RN + c + RW]);
        d[5] = Work<S>::in(mid[4 * RN + c - RW - 1]);
        d[6] = Work<S>::in(mid[5 * RN + c - RW + 1]);
        d[7] = Work<S>::in(mid[6 * RN + c + RW + 1]);
        d[8] = Work<S>::in(mid[7 * RN + c + RW - 1]);
        update_site<NOISE, S>(d, P, (uint32_t)(y * nx + x), t + 1, g.key0, g.key1);
        const uint32_t off = ((uint32_t)y * px + (uint32_t)x) * E;
#pragma unroll
        for (int i = 0; i < 9; ++i)
            gstore<NT>(reinterpret_cast<T *>(dp[i] + off), Work<S>::out(d[i]));
    }
}

// Every tile of the launch has the shape TW x TH.  (A CU holds three
// blocks: 65-71 registers a thread; a budget of 64 for four blocks of the
// 38 KB FP32 tiles made the compiler spill, and the spills cost 5 % more
// HBM bytes than the fourth block gained.)
template <int S, bool NT, bool NOISE, int TW, int TH>
__global__ __launch_bounds__(kStep2Threads) void step2_kernel(StepArgs g)
{
    using T = typename Codec<S>::T;
    using SH = Fixed<TW, TH>;
    __shared__ T mid[8 * SH::rn];
    advance_counter(g, 2);
    const StepItem it = g.items[blockIdx.x];
    if (it.lattice < 0) return;
    step2_tile<S, NT, NOISE>(g, it, SH{}, mid);
}

// Each work item has its own tile shape: 32 x 32 when the tile index
// carries kStep2Square, else 64 x 16 (a lattice's items all have the same
// shape).  The two shapes need about the same LDS (37 and 38 KB in FP32),
// so a batch can give each lattice the shape that fits its sides in one
// launch.
template <int S, bool NT, bool NOISE>
__global__ __launch_bounds__(kStep2Threads) void step2_mixed_kernel(StepArgs g)
{
    using T = typename Codec<S>::T;
    constexpr int RN = Fixed<32, 32>::rn > Fixed<64, 16>::rn ? Fixed<32, 32>::rn : Fixed<64, 16>::rn;
    __shared__ T mid[8 * RN];
    advance_counter(g, 2);
    StepItem it = g.items[blockIdx.x];
    if (it.lattice < 0) return;
    const bool square = (it.tile & kStep2Square) != 0;
    it.tile &= ~kStep2Square;
    step2_tile<S, NT, NOISE>(g, it, Dyn(square ? 5 : 6), mid);
}

template <int S, bool NT, bool NOISE>
static hipError_t launch_step2_tiles(const StepArgs &a, int nitems, int tw, hipStream_t s)
{
    const dim3 grid(nitems), block(kStep2Threads);
    if (tw == 64)
        hipLaunchKernelGGL((step2_kernel<S, NT, NOISE, 64, 16>), grid, block, 0, s, a);
    else if (tw == 128)
        hipLaunchKernelGGL((step2_kernel<S, NT, NOISE, 128, 8>), grid, block, 0, s, a);
    else if (tw == 32)
        hipLaunchKernelGGL((step2_kernel<S, NT, NOISE, 32, 32>), grid, block, 0, s, a);
    else if (tw == 0)
        hipLaunchKernelGGL((step2_mixed_kernel<S, NT, NOISE>), grid, block, 0, s, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

bool step2_tile_supported(int tw) { return tw == 32 || tw == 64 || tw == 128; }

hipError_t launch_step2(const DeviceView &v, const StepItem *items, int nitems, int tile_w,
                        bool nontemporal, bool noise, hipStream_t s)
{
    const StepArgs a = step_args(v, items);
#define FLB_SEL(S_)                                                                              \
    if (v.storage == S_) {                                                                       \
        if (nontemporal)                                                                         \
            return noise ? launch_step2_tiles<S_, true, true>(a, nitems, tile_w, s)              \
                         : launch_step2_tiles<S_, true, false>(a, nitems, tile_w, s);            \
        return noise ? launch_step2_tiles<S_, false, true>(a, nitems, tile_w, s)                 \
                     : launch_step2_tiles<S_, false, false>(a, nitems, tile_w, s);               \
    }
    FLB_SEL(kF32)
    FLB_SEL(kBF16)
    FLB_SEL(kF16)
#undef FLB_SEL
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------
// Three steps per launch.  A block owns a TW x TH tile; its region adds two
// rings of sites.  Phase 1 collides the whole region at t (each site pulled
// from HBM), phase 2 the tile and the inner ring at t + 1 (pulled from
// phase 1's values in LDS), phase 3 the tile at t + 2, which it stores.
// Every intermediate value is rounded to the storage format, so the
// results are the bits of three one-step launches; the populations cross
// HBM once per three steps.  A thread keeps its sites across the phases
// (its two tile sites in all three, its inner-ring site in the first two,
// its outer-ring site in the first), so a site's rest population stays in a
// register and LDS holds planes 1..8 of the region.  Phase 2 reads all its
// inputs before a barrier and then overwrites them in place.
// ---------------------------------------------------------------------

// region coordinates of the h-th site of the one-site ring around a w x hh
// box whose top-left site is at region (1, 1); the ring spans [0, w + 2) x
// [0, hh + 2)
__device__ __forceinline__ void ring_box(int w, int hh, int h, int &rx, int &ry)
{
    const int RW = w + 2;
    if (h < RW) {
        ry = 0;
        rx = h;
    } else if (h < 2 * RW) {
        ry = hh + 1;
        rx = h - RW;
    } else if (h < 2 * RW + hh) {
        ry = h - 2 * RW + 1;
        rx = 0;
    } else {
        ry = h - 2 * RW - hh + 1;
        rx = RW - 1;
    }
}

// (FP32: the register budget of six waves per SIMD, three blocks per CU as
// the 51 KB of LDS of a 128 x 8 region allow.)
template <int S, bool NT, bool NOISE, int TW, int TH>
__global__ __launch_bounds__(kStep2Threads)
__attribute__((amdgpu_waves_per_eu(S == kF32 ? 6 : 4))) void step3_kernel(StepArgs g)
{
    using T = typename Codec<S>::T;
    static_assert(TW * TH == 1024 && (TW & (TW - 1)) == 0, "tile shape");
    constexpr int RW = TW + 4, RN = RW * (TH + 4);
    constexpr int N1 = 2 * (TW + 2) + 2 * TH;        // inner ring
    constexpr int N2 = 2 * (TW + 4) + 2 * (TH + 2);  // outer ring
    constexpr int KT = 1024 / kStep2Threads;        // tile sites per thread
    constexpr int K = KT + 2;                       // phase-1 slots: tile, inner, outer
    static_assert(N1 <= kStep2Threads && N2 <= kStep2Threads, "tile shape");
    constexpr int LG = TW == 32 ? 5 : TW == 64 ? 6 : 7;
    __shared__ T mid[8 * RN];  // planes 1..8 of the region
    advance_counter(g, 3);
    const StepItem it = g.items[blockIdx.x];
    if (it.lattice < 0) return;
    const LatticeParams &P = g.params[it.lattice];
    const int nx = P.nx, ny = P.ny;
    const int tiles_x = (nx + TW - 1) >> LG;
    const int x0 = (it.tile % tiles_x) * TW, y0 = (it.tile / tiles_x) * TH;
    const T *__restrict__ src = (const T *)g.src + P.base;
    T *__restrict__ dst = (T *)g.dst + P.base;
    const uint32_t plane = (uint32_t)P.plane, px = (uint32_t)P.px;
    const uint32_t t = *g.step;
    const int tid = threadIdx.x;
    const bool has1 = tid < N1, has2 = tid >= kStep2Threads - N2;
    const bool interior = x0 >= 3 && y0 >= 3 && x0 + TW + 3 <= nx && y0 + TH + 3 <= ny;

    // slots: 0 .. KT-1 tile sites, KT the inner-ring site, KT+1 the outer
    int xs[K], ys[K], rs[K];
#pragma unroll
    for (int k = 0; k < K; ++k) {
        int rx, ry;
        if (k < KT) {
            const int o = tid + k * kStep2Threads;
            ry = (o >> LG) + 2;
            rx = (o & (TW - 1)) + 2;
        } else if (k == KT) {
            ring_box(TW, TH, has1 ? tid : 0, rx, ry);
            rx += 1;
            ry += 1;
        } else {
            ring_box(TW + 2, TH + 2, has2 ? tid - (kStep2Threads - N2) : 0, rx, ry);
        }
        rs[k] = ry * RW + rx;
        xs[k] = x0 - 2 + rx;
        ys[k] = y0 - 2 + ry;
    }
    if (!interior) {
        // wrap (x >= -2, nx >= 2): at most one subtraction unless the
        // lattice is smaller than a tile
#pragma unroll
        for (int k = 0; k < K; ++k) {
            int x = xs[k], y = ys[k];
            x = x < 0 ? x + nx : x;
            y = y < 0 ? y + ny : y;
            while (x >= nx) x -= nx;
            while (y >= ny) y -= ny;
            xs[k] = x;
            ys[k] = y;
        }
    }
    const char *sp[9];
    char *dp[9];
#pragma unroll
    for (int i = 0; i < 9; ++i) {
        sp[i] = reinterpret_cast<const char *>(src) + (size_t)i * plane * sizeof(T);
        dp[i] = reinterpret_cast<char *>(dst) + (size_t)i * plane * sizeof(T);
    }
    constexpr uint32_t E = sizeof(T);
    auto active = [&](int k) { return k < KT || (k == KT ? has1 : has2); };

    // phase 1 (t): every region site, pulled from HBM
    T raw[K][9];
    if (interior) {
        const int64_t row = (int64_t)px * E;
        const char *const sh0 = sp[0];
        const char *const sh1 = sp[1] - (int64_t)E;
        const char *const sh2 = sp[2] - row;
        const char *const sh3 = sp[3] + (int64_t)E;
        const char *const sh4 = sp[4] + row;
        const char *const sh5 = sp[5] - row - (int64_t)E;
        const char *const sh6 = sp[6] - row + (int64_t)E;
        const char *const sh7 = sp[7] + row + (int64_t)E;
        const char *const sh8 = sp[8] + row - (int64_t)E;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (!active(k)) continue;
            const uint32_t o = ((uint32_t)ys[k] * px + (uint32_t)xs[k]) * E;
            raw[k][0] = *reinterpret_cast<const T *>(sh0 + o);
            raw[k][1] = *reinterpret_cast<const T *>(sh1 + o);
            raw[k][2] = *reinterpret_cast<const T *>(sh2 + o);
            raw[k][3] = *reinterpret_cast<const T *>(sh3 + o);
            raw[k][4] = *reinterpret_cast<const T *>(sh4 + o);
            raw[k][5] = *reinterpret_cast<const T *>(sh5 + o);
            raw[k][6] = *reinterpret_cast<const T *>(sh6 + o);
            raw[k][7] = *reinterpret_cast<const T *>(sh7 + o);
            raw[k][8] = *reinterpret_cast<const T *>(sh8 + o);
        }
    } else {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            if (!active(k)) continue;
            const int x = xs[k], y = ys[k];
            const uint32_t ux = (uint32_t)x * E;
            const uint32_t xm = (uint32_t)(x == 0 ? nx - 1 : x - 1) * E;
            const uint32_t xr = (uint32_t)(x == nx - 1 ? 0 : x + 1) * E;
            const uint32_t rc = (uint32_t)y * px * E;
            const uint32_t rm = (uint32_t)(y == 0 ? ny - 1 : y - 1) * px * E;
            const uint32_t rp = (uint32_t)(y == ny - 1 ? 0 : y + 1) * px * E;
            raw[k][0] = *reinterpret_cast<const T *>(sp[0] + (rc + ux));
            raw[k][1] = *reinterpret_cast<const T *>(sp[1] + (rc + xm));
            raw[k][2] = *reinterpret_cast<const T *>(sp[2] + (rm + ux));
            raw[k][3] = *reinterpret_cast<const T *>(sp[3] + (rc + xr));
            raw[k][4] = *reinterpret_cast<const T *>(sp[4] + (rp + ux));
            raw[k][5] = *reinterpret_cast<const T *>(sp[5] + (rm + xm));
            raw[k][6] = *reinterpret_cast<const T *>(sp[6] + (rm + xr));
            raw[k][7] = *reinterpret_cast<const T *>(sp[7] + (rp + xr));
            raw[k][8] = *reinterpret_cast<const T *>(sp[8] + (rp + xm));
        }
    }
    T own[KT + 1];  // plane 0 of the tile and inner-ring sites, storage format
#pragma unroll
    for (int k = 0; k < K; ++k) {
        if (!active(k)) continue;
        float d[9];
#pragma unroll
        for (int i = 0; i < 9; ++i) d[i] = Work<S>::in(raw[k][i]);
        update_site<NOISE, S>(d, P, (uint32_t)(ys[k] * nx + xs[k]), t, g.key0, g.key1);
        if (k <= KT) own[k] = Work<S>::out(d[0]);
#pragma unroll
        for (int i = 1; i < 9; ++i) mid[(i - 1) * RN + rs[k]] = Work<S>::out(d[i]);
    }
    __syncthreads();

    // phase 2 (t + 1): tile and inner ring, pulled from LDS; every read
    // before the barrier, every write after it
    T nxt[KT + 1][8];
#pragma unroll
    for (int k = 0; k <= KT; ++k) {
        if (!active(k)) continue;
        const int c = rs[k];
        float d[9];
        d[0] = Work<S>::in(own[k]);
        d[1] = Work<S>::in(mid[0 * RN + c - 1]);
        d[2] = Work<S>::in(mid[1 * RN + c - RW]);
        d[3] = Work<S>::in(mid[2 * RN + c + 1]);
        d[4] = Work<S>::in(mid[3 * RN + c + RW]);
        d[5] = Work<S>::in(mid[4 * RN + c - RW - 1]);
        d[6] = Work<S>::in(mid[5 * RN + c - RW + 1]);
        d[7] = Work<S>::in(mid[6 * RN + c + RW + 1]);
        d[8] = Work<S>::in(mid[7 * RN + c + RW - 1]);
        update_site<NOISE, S>(d, P, (uint32_t)(ys[k] * nx + xs[k]), t + 1, g.key0, g.key1);
        own[k] = Work<S>::out(d[0]);
#pragma unroll
        for (int i = 1; i < 9; ++i) nxt[k][i - 1] = Work<S>::out(d[i]);
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k <= KT; ++k) {
        if (!active(k)) continue;
#pragma unroll
        for (int i = 1; i < 9; ++i) mid[(i - 1) * RN + rs[k]] = nxt[k][i - 1];
    }
    __syncthreads();

    // phase 3 (t + 2): the tile, stored
#pragma unroll
    for (int k = 0; k < KT; ++k) {
        const int o = tid + k * kStep2Threads;
        const int x = x0 + (o & (TW - 1)), y = y0 + (o >> LG);
        if (x >= nx || y >= ny) continue;
        const int c = rs[k];
        float d[9];
        d[0] = Work<S>::in(own[k]);
        d[1] = Work<S>::in(mid[0 * RN + c - 1]);
        d[2] = Work<S>::in(mid[1 * RN + c - RW]);
        d[3] = Work<S>::in(mid[2 * RN + c + 1]);
        d[4] = Work<S>::in(mid[3 * RN + c + RW]);
        d[5] = Work<S>::in(mid[4 * RN + c - RW - 1]);
        d[6] = Work<S>::in(mid[5 * RN + c - RW + 1]);
        d[7] = Work<S>::in(mid[6 * RN + c + RW + 1]);
        d[8] = Work<S>::in(mid[7 * RN + c + RW - 1]);
        update_site<NOISE, S>(d, P, (uint32_t)(y * nx + x), t + 2, g.key0, g.key1);
        const uint32_t off = ((uint32_t)y * px + (uint32_t)x) * E;
#pragma unroll
        for (int i = 0; i < 9; ++i)
            gstore<NT>(reinterpret_cast<T *>(dp[i] + off), Work<S>::out(d[i]));
    }
}

template <int S, bool NT, bool NOISE>
static hipError_t launch_step3_tiles(const StepArgs &a, int nitems, int tw, hipStream_t s)
{
    const dim3 grid(nitems), block(kStep2Threads);
    if (tw == 64)
        hipLaunchKernelGGL((step3_kernel<S, NT, NOISE, 64, 16>), grid, block, 0, s, a);
    else if (tw == 128)
        hipLaunchKernelGGL((step3_kernel<S, NT, NOISE, 128, 8>), grid, block, 0, s, a);
    else if (tw == 32)
        hipLaunchKernelGGL((step3_kernel<S, NT, NOISE, 32, 32>), grid, block, 0, s, a);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_step3(const DeviceView &v, const StepItem *items, int nitems, int tile_w,
                        bool nontemporal, bool noise, hipStream_t s)
{
    const StepArgs a = step_args(v, items);
#define FLB_SEL(S_)                                                                              \
    if (v.storage == S_) {                                                                       \
        if (nontemporal)                                                                         \
            return noise ? launch_step3_tiles<S_, true, true>(a, nitems, tile_w, s)              \
                         : launch_step3_tiles<S_, true, false>(a, nitems, tile_w, s);            \
        return noise ? launch_step3_tiles<S_, false, true>(a, nitems, tile_w, s)                 \
                     : launch_step3_tiles<S_, false, false>(a, nitems, tile_w, s);               \
    }
    FLB_SEL(kF32)
    FLB_SEL(kBF16)
    FLB_SEL(kF16)
#undef FLB_SEL
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------
// T = 4 or 5 steps per launch, marching along y without LDS or barriers.
// A wave owns a strip of W = 64 - 2 (T - 1) columns and `rows` rows; its
// lanes are the strip and T - 1 halo columns on either side.  It walks down
// the strip one row at a time and holds T time levels at once: while level
// 1 (t) collides row y, pulled from HBM, level k + 1 (t + k) collides row
// y - k from what level k left in registers.  A population moving along y
// reaches its next row in the same lane; one moving along x comes from the
// neighbour lane (wave shift).  So a level keeps nine values per lane
// (planes 0, 1, 3 of its last row, planes 2, 5, 6 of its last two), the
// other populations of a row are used at once, and nothing else is kept.
// The outermost columns of a wave go stale by one a level; they are the
// halo, which the neighbouring strips compute again.  Values pass from one
// level to the next rounded to the storage format, so the results are the
// bits of T one-step launches.
//
// What bounds it: VALU issue (160 instructions per collision, of which the
// noise is half).  Collisions per update: 64 / W for the halo columns times
// 1 + (T - 1) / rows for the halo rows, 1.20 at 4096^2 with T = 5 (75 rows
// a wave), against 1.16 of the three-step tiles (two barriers a step, 204
// instructions per update); HBM moves 72 / T bytes per update.  At 4096^2
// FP32: 166-174 GLUPS with T = 5, 166-173 with T = 4, tiles of three steps
// 148-153, of two 125-130 (T = 2 and 3 of this form 106 and 146).  BF16:
// T = 4 157, T = 5 149, two-step tiles 153.  Stores are ordinary: with the
// streaming hint a wave's 240-byte rows, whose ends share lines with the
// next strip, cost T = 4 12 %.
//
// The loop takes two rows a turn, so that the two rows kept of planes 2, 5,
// 6 swap names instead of registers, and its first rows run through the same
// code with the levels not yet fed skipped: peeled rows in front of the
// loop (25 KB more code, fetched cold by every launch) cost a quarter.
// ---------------------------------------------------------------------

// `base` plus a byte offset
template <typename U> __device__ __forceinline__ const U *bytes_at(const U *base, uint32_t off)
{
    return reinterpret_cast<const U *>(reinterpret_cast<const char *>(base) + off);
}
template <typename U> __device__ __forceinline__ U *bytes_at(U *base, uint32_t off)
{
    return reinterpret_cast<U *>(reinterpret_cast<char *>(base) + off);
}

// item: lattice and strip + segment * strips of the lattice; a block's waves
// take consecutive items (neighbouring strips, which share lines)
template <int S, bool NOISE, int T>
__global__ __launch_bounds__(64 * kMarchWaves)
__attribute__((amdgpu_waves_per_eu(4))) void march_kernel(StepArgs g, int rows)
{
    using E = typename Codec<S>::T;
    constexpr int W = march_cols(T);
    const int wv = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    advance_counter(g, T);
    const StepItem it = g.items[blockIdx.x * kMarchWaves + wv];
    if (it.lattice < 0) return;
    const LatticeParams &P = g.params[it.lattice];
    const int nx = P.nx, ny = P.ny;
    const int64_t px = P.px, plane = P.plane;
    const int nstrips = (nx + W - 1) / W;
    const int seg = it.tile / nstrips, strip = it.tile - seg * nstrips;
    const int y0 = seg * rows, h = min(rows, ny - y0);
    const int lane = (int)threadIdx.x & 63;
    const uint32_t t = *g.step;

    int x = strip * W - (T - 1) + lane;
    const bool own = lane >= T - 1 && lane < 64 - (T - 1) && x < nx;
    while (x < 0) x += nx;
    while (x >= nx) x -= nx;
    const uint32_t sx = (uint32_t)x;
    // byte offsets of the columns x, x - 1, x + 1
    uint32_t o0 = sx * sizeof(E), om = (uint32_t)(x == 0 ? nx - 1 : x - 1) * sizeof(E);
    uint32_t op = (uint32_t)(x == nx - 1 ? 0 : x + 1) * sizeof(E);
    const E *__restrict__ src = (const E *)g.src + P.base;
    E *__restrict__ dst = (E *)g.dst + P.base;

    int y = y0 - (T - 1);  // level 1's next row
    while (y < 0) y += ny;
    E nxt[9];
    auto load = [&]() {
        const int ym = y == 0 ? ny - 1 : y - 1, yp = y == ny - 1 ? 0 : y + 1;
        const E *rc = src + y * px, *rm = src + ym * px, *rp = src + yp * px;
        // (opaque here, so that each access is a scalar base and a 32-bit
        // offset: widened outside the loop they become 64-bit adds)
        asm("" : "+v"(o0), "+v"(om), "+v"(op));
        nxt[0] = *bytes_at(rc, o0);
        nxt[1] = *bytes_at(rc + plane, om);
        nxt[2] = *bytes_at(rm + 2 * plane, o0);
        nxt[3] = *bytes_at(rc + 3 * plane, op);
        nxt[4] = *bytes_at(rp + 4 * plane, o0);
        nxt[5] = *bytes_at(rm + 5 * plane, om);
        nxt[6] = *bytes_at(rm + 6 * plane, op);
        nxt[7] = *bytes_at(rp + 7 * plane, op);
        nxt[8] = *bytes_at(rp + 8 * plane, om);
    };
    load();
    // A[k]: planes 0, 1, 3 of level k's last row; B[k][i & 1]: planes 2, 5, 6
    // of the row before it, B[k][~i & 1] of the last row; all as level k + 1
    // reads them, at the sites they stream to
    float A[T][3] = {}, B[T][2][3] = {};
    int yk[T] = {};  // each level's row
    // row i: level k + 1 joins in with row 2 k, when its first row's
    // neighbours are there
    auto row = [&](int i, auto parity) {
        constexpr int p = decltype(parity)::value;
        float d[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) d[q] = Work<S>::in(nxt[q]);
#pragma unroll
        for (int k = T - 1; k > 0; --k) yk[k] = yk[k - 1];
        yk[0] = y;
        y = y == ny - 1 ? 0 : y + 1;
        load();  // the next row's, under this row's collisions
        update_site<NOISE, S>(d, P, (uint32_t)(yk[0] * nx) + sx, t, g.key0, g.key1);
#pragma unroll
        for (int k = 1; k < T; ++k) {
            if (i < 2 * k - 2) break;
            float e[9];
            e[0] = A[k][0];
            e[1] = A[k][1];
            e[3] = A[k][2];
            e[2] = B[k][p][0];
            e[5] = B[k][p][1];
            e[6] = B[k][p][2];
            e[4] = stored<S>(d[4]);
            e[7] = wave_from_right(stored<S>(d[7]));
            e[8] = wave_from_left(stored<S>(d[8]));
            A[k][0] = stored<S>(d[0]);
            A[k][1] = wave_from_left(stored<S>(d[1]));
            A[k][2] = wave_from_right(stored<S>(d[3]));
            B[k][p][0] = stored<S>(d[2]);
            B[k][p][1] = wave_from_left(stored<S>(d[5]));
            B[k][p][2] = wave_from_right(stored<S>(d[6]));
            if (i < 2 * k) break;
            update_site<NOISE, S>(e, P, (uint32_t)(yk[k] * nx) + sx, t + k, g.key0, g.key1);
#pragma unroll
            for (int q = 0; q < 9; ++q) d[q] = e[q];
            if (k == T - 1 && own) {
                asm("" : "+v"(o0));
                E *out = dst + yk[k] * px;
#pragma unroll
                for (int q = 0; q < 9; ++q) *bytes_at(out + q * plane, o0) = Work<S>::out(d[q]);
            }
        }
    };
    const int n = h + 2 * (T - 1);
    for (int i = 0; i < n; i += 2) {
        row(i, std::integral_constant<int, 0>());
        if (i + 1 >= n) break;
        row(i + 1, std::integral_constant<int, 1>());
    }
}

template <int S>
static hipError_t launch_march_s(const StepArgs &a, int nblocks, int steps, int rows, bool noise,
                                 hipStream_t s)
{
    const dim3 grid(nblocks), block(64 * kMarchWaves);
    if constexpr (S == kF32) {  // (16-bit storage: four steps are the faster)
        if (steps == 5 && noise) {
            hipLaunchKernelGGL((march_kernel<S, true, 5>), grid, block, 0, s, a, rows);
            return hipGetLastError();
        }
        if (steps == 5) {
            hipLaunchKernelGGL((march_kernel<S, false, 5>), grid, block, 0, s, a, rows);
            return hipGetLastError();
        }
    }
    if (steps != 4) return hipErrorInvalidValue;
    if (noise)
        hipLaunchKernelGGL((march_kernel<S, true, 4>), grid, block, 0, s, a, rows);
    else
        hipLaunchKernelGGL((march_kernel<S, false, 4>), grid, block, 0, s, a, rows);
    return hipGetLastError();
}

hipError_t launch_march(const DeviceView &v, const StepItem *items, int nitems, int steps,
                        int rows, bool noise, hipStream_t s)
{
    if (rows < 1 || nitems % kMarchWaves) return hipErrorInvalidValue;
    const StepArgs a = step_args(v, items);
    const int nb = nitems / kMarchWaves;
    if (v.storage == kF32) return launch_march_s<kF32>(a, nb, steps, rows, noise, s);
    if (v.storage == kBF16) return launch_march_s<kBF16>(a, nb, steps, rows, noise, s);
    if (v.storage == kF16) return launch_march_s<kF16>(a, nb, steps, rows, noise, s);
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------
// Any number of steps per launch on small tiles, for lattices that leave
// most of the device idle.  A block owns a tw x th tile; the region it
// starts from adds steps - 1 rings.  Each step collides the box of sites
// whose neighbours the step before left in LDS, one ring less every time,
// from one LDS buffer into another (one barrier a step); the first step
// reads HBM, the last writes it.  The threads share out each step's box
// anew, so no wave is left with a ring's idle lanes.
//
// What bounds it: a launch (about 4 us with its first loads) and then the
// VALU of the compute units that have a block, 0.28 us for every four waves
// of a step.  So the tile is small enough to give every compute unit one,
// and the rings, which grow with steps squared, are cheaper than another
// launch: 256^2, up to nine steps in one launch of 16 x 16 tiles (ten are two
// launches of five, 18.7 us; 30 in tiles of three and two steps).
// ---------------------------------------------------------------------
template <int S, bool NOISE>
__global__ __launch_bounds__(kPatchThreads) void patch_kernel(StepArgs g, int tw, int th, int steps)
{
    using E = typename Codec<S>::T;
    extern __shared__ float buf[];  // two buffers of nine planes of the region
    advance_counter(g, steps);
    const StepItem it = g.items[blockIdx.x];
    if (it.lattice < 0) return;
    const LatticeParams &P = g.params[it.lattice];
    const int nx = P.nx, ny = P.ny, px = P.px, plane = (int)P.plane;
    const int tiles_x = (nx + tw - 1) / tw;
    const int x0 = (it.tile % tiles_x) * tw, y0 = (it.tile / tiles_x) * th;
    const int halo = steps - 1, w0 = tw + 2 * halo, h0 = th + 2 * halo, RN = w0 * h0;
    const E *__restrict__ src = (const E *)g.src + P.base;
    E *__restrict__ dst = (E *)g.dst + P.base;
    const uint32_t t = *g.step;
    for (int s = 0; s < steps; ++s) {
        const int w = w0 - 2 * s, n = w * (h0 - 2 * s);
        const float rw = 1.0f / (float)w;
        const float *from = buf + ((s + 1) & 1) * 9 * RN;
        float *to = buf + (s & 1) * 9 * RN;
        for (int e = (int)threadIdx.x; e < n; e += kPatchThreads) {
            // row of the box by a float reciprocal: (e + 1/2) / w is 1/(2 w)
            // away from an integer (e < 2^13)
            const int by = (int)(((float)e + 0.5f) * rw), bx = e - by * w;
            int x = x0 - halo + s + bx, y = y0 - halo + s + by;
            float d[9];
            if (s == 0) {
                while (x < 0) x += nx;
                while (x >= nx) x -= nx;
                while (y < 0) y += ny;
                while (y >= ny) y -= ny;
                const int xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1;
                const int rc = y * px, rm = (y == 0 ? ny - 1 : y - 1) * px;
                const int rp = (y == ny - 1 ? 0 : y + 1) * px;
                d[0] = Work<S>::in(src[rc + x]);
                d[1] = Work<S>::in(src[1 * plane + rc + xm]);
                d[2] = Work<S>::in(src[2 * plane + rm + x]);
                d[3] = Work<S>::in(src[3 * plane + rc + xp]);
                d[4] = Work<S>::in(src[4 * plane + rp + x]);
                d[5] = Work<S>::in(src[5 * plane + rm + xm]);
                d[6] = Work<S>::in(src[6 * plane + rm + xp]);
                d[7] = Work<S>::in(src[7 * plane + rp + xp]);
                d[8] = Work<S>::in(src[8 * plane + rp + xm]);
            } else {
                const int c = (by + s) * w0 + bx + s;
                d[0] = from[c];
                d[1] = from[1 * RN + c - 1];
                d[2] = from[2 * RN + c - w0];
                d[3] = from[3 * RN + c + 1];
                d[4] = from[4 * RN + c + w0];
                d[5] = from[5 * RN + c - w0 - 1];
                d[6] = from[6 * RN + c - w0 + 1];
                d[7] = from[7 * RN + c + w0 + 1];
                d[8] = from[8 * RN + c + w0 - 1];
                while (x < 0) x += nx;
                while (x >= nx) x -= nx;
                while (y < 0) y += ny;
                while (y >= ny) y -= ny;
            }
            update_site<NOISE, S>(d, P, (uint32_t)(y * nx + x), t + s, g.key0, g.key1);
            if (s < halo) {
                const int c = (by + s) * w0 + bx + s;
#pragma unroll
                for (int i = 0; i < 9; ++i) to[i * RN + c] = stored<S>(d[i]);
            } else if (x0 + bx < nx && y0 + by < ny) {
                E *o = dst + y * px + x;
#pragma unroll
                for (int i = 0; i < 9; ++i) o[i * plane] = Work<S>::out(d[i]);
            }
        }
        __syncthreads();
    }
}

int patch_lds_bytes(int tw, int th, int steps)
{
    return steps < 2 ? 0 : 2 * 9 * (tw + 2 * steps - 2) * (th + 2 * steps - 2) * (int)sizeof(float);
}

hipError_t launch_patch(const DeviceView &v, const StepItem *items, int nitems, int tw, int th,
                        int steps, bool noise, hipStream_t s)
{
    const StepArgs a = step_args(v, items);
    const dim3 grid(nitems), block(kPatchThreads);
    const int lds = patch_lds_bytes(tw, th, steps);
    if (steps < 1 || (tw + 2 * steps) * (th + 2 * steps) > 8192) return hipErrorInvalidValue;
#define FLB_SEL(S_)                                                                              \
    if (v.storage == S_) {                                                                       \
        if (noise)                                                                               \
            hipLaunchKernelGGL((patch_kernel<S_, true>), grid, block, lds, s, a, tw, th, steps); \
        else                                                                                     \
            hipLaunchKernelGGL((patch_kernel<S_, false>), grid, block, lds, s, a, tw, th, steps); \
        return hipGetLastError();                                                                \
    }
    FLB_SEL(kF32)
    FLB_SEL(kBF16)
    FLB_SEL(kF16)
#undef FLB_SEL
    return hipErrorInvalidValue;
}

// ---------------------------------------------------------------------
// Step counter, after the kernels that step in place
// ---------------------------------------------------------------------
__global__ void advance_step_kernel(uint32_t *step, uint32_t n)
{
    if (threadIdx.x == 0 && blockIdx.x == 0) *step += n;
}

hipError_t launch_advance_step(uint32_t *step, uint32_t n, hipStream_t s)
{
    hipLaunchKernelGGL(advance_step_kernel, dim3(1), dim3(64), 0, s, step, n);
    return hipGetLastError();
}

// ---------------------------------------------------------------------
// Uniform equilibrium start, Eq. (2): every stored value is feq_i.
// ---------------------------------------------------------------------
template <int S>
__global__ __launch_bounds__(kThreads) void init_kernel(void *pops, const LatticeParams *params,
                                                        int lattice)
{
    using T = typename Codec<S>::T;
    const LatticeParams &P = params[lattice];
    const int64_t n = 9 * P.plane;
    T *p = (T *)pops + P.base;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(k / P.plane);
        p[k] = Codec<S>::encode(P.feq[i], P, i);
    }
}

static int grid_for(int64_t n)
{
    int64_t b = (n + kThreads - 1) / kThreads;
    return (int)(b < 4096 ? (b < 1 ? 1 : b) : 4096);
}

hipError_t launch_init(const DeviceView &v, int lattice, int64_t plane, hipStream_t s)
{
    const dim3 grid(grid_for(9 * plane)), block(kThreads);
    void *p = v.pops[v.cur];
    if (v.storage == kF32)
        hipLaunchKernelGGL(init_kernel<kF32>, grid, block, 0, s, p, v.params, lattice);
    else if (v.storage == kBF16)
        hipLaunchKernelGGL(init_kernel<kBF16>, grid, block, 0, s, p, v.params, lattice);
    else
        hipLaunchKernelGGL(init_kernel<kF16>, grid, block, 0, s, p, v.params, lattice);
    return hipGetLastError();
}

// ---------------------------------------------------------------------
// State export / import as full FP64 populations f_i(x) = w_i rho0 + d_i,
// with d_i(x) = stored_i(x - v_i): values first .. first + n - 1 of the
// lattice's [9][ny][nx] array, out[0] / in[0] being value `first`.
// ---------------------------------------------------------------------
__device__ constexpr double kWd[9] = {4.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9, 1.0 / 9,
                                      1.0 / 36, 1.0 / 36, 1.0 / 36, 1.0 / 36};

template <int S>
__global__ __launch_bounds__(kThreads) void get_kernel(const void *pops,
                                                       const LatticeParams *params, int lattice,
                                                       int64_t first, int64_t n, double *out,
                                                       StageDone done)
{
    using T = typename Codec<S>::T;
    const LatticeParams &P = params[lattice];
    const int nx = P.nx, ny = P.ny, px = P.px;
    const int64_t V = (int64_t)nx * ny, plane = P.plane;
    const T *p = (const T *)pops + P.base;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = first + j;
        const int i = (int)(k / V);
        const int s = (int)(k - (int64_t)i * V);
        const int y = s / nx, x = s - y * nx;
        const int xs = wrap_add(x, -kVX[i], nx), ys = wrap_add(y, -kVY[i], ny);
        const float d = Codec<S>::decode(p[(int64_t)i * plane + ys * px + xs], P, i);
        out[j] = kWd[i] * (double)P.rho0 + (double)d;
    }
    stage_signal(done);
}

template <int S>
__global__ __launch_bounds__(kThreads) void set_kernel(void *pops, const LatticeParams *params,
                                                       int lattice, int64_t first, int64_t n,
                                                       const double *in)
{
    using T = typename Codec<S>::T;
    const LatticeParams &P = params[lattice];
    const int nx = P.nx, ny = P.ny, px = P.px;
    const int64_t V = (int64_t)nx * ny, plane = P.plane;
    T *p = (T *)pops + P.base;
    for (int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; j < n;
         j += (int64_t)gridDim.x * blockDim.x) {
        const int64_t k = first + j;
        const int i = (int)(k / V);
        const int s = (int)(k - (int64_t)i * V);
        const int y = s / nx, x = s - y * nx;
        // f_i(x) is stored at x - v_i
        const int xs = wrap_add(x, -kVX[i], nx), ys = wrap_add(y, -kVY[i], ny);
        const double f = in[j];
        p[(int64_t)i * plane + ys * px + xs] = Codec<S>::encode((float)(f - kWd[i] * (double)P.rho0), P, i);
    }
}

hipError_t launch_get(const DeviceView &v, int lattice, int64_t first, int64_t n, double *out,
                      StageDone done, hipStream_t s)
{
    const dim3 grid(grid_for(n)), block(kThreads);
    const void *p = v.pops[v.cur];
    if (v.storage == kF32)
        hipLaunchKernelGGL(get_kernel<kF32>, grid, block, 0, s, p, v.params, lattice, first, n, out,
                           done);
    else if (v.storage == kBF16)
        hipLaunchKernelGGL(get_kernel<kBF16>, grid, block, 0, s, p, v.params, lattice, first, n, out,
                           done);
    else
        hipLaunchKernelGGL(get_kernel<kF16>, grid, block, 0, s, p, v.params, lattice, first, n, out,
                           done);
    return hipGetLastError();
}

hipError_t launch_set(const DeviceView &v, int lattice, int64_t first, int64_t n, const double *in,
                      hipStream_t s)
{
    const dim3 grid(grid_for(n)), block(kThreads);
    void *p = v.pops[v.cur];
    if (v.storage == kF32)
        hipLaunchKernelGGL(set_kernel<kF32>, grid, block, 0, s, p, v.params, lattice, first, n, in);
    else if (v.storage == kBF16)
        hipLaunchKernelGGL(set_kernel<kBF16>, grid, block, 0, s, p, v.params, lattice, first, n, in);
    else
        hipLaunchKernelGGL(set_kernel<kF16>, grid, block, 0, s, p, v.params, lattice, first, n, in);
    return hipGetLastError();
}

// ---------------------------------------------------------------------
// FP64 sums: mass, momentum and the staggered momenta.  Deterministic:
// fixed per-block partials, then one block adds them in a fixed order.
// ---------------------------------------------------------------------
template <int NV>
__device__ __forceinline__ void block_sum(double (&v)[NV], double *out)
{
    __shared__ double red[NV][kThreads / 64];
    const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < NV; ++q) {
        double x = v[q];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) x += __shfl_down(x, o, 64);
        if (lane == 0) red[q][wv] = x;
    }
    __syncthreads();
    if (threadIdx.x < NV) {
        double x = 0;
        for (int w2 = 0; w2 < kThreads / 64; ++w2) x += red[threadIdx.x][w2];
        out[threadIdx.x] = x;
    }
}

template <int S>
__global__ __launch_bounds__(kThreads) void conservation_kernel(const void *pops,
                                                                const LatticeParams *params,
                                                                int lattice, double *part)
{
    using T = typename Codec<S>::T;
    const LatticeParams &P = params[lattice];
    const int nx = P.nx, ny = P.ny, px = P.px;
    const int64_t V = (int64_t)nx * ny, plane = P.plane;
    const T *p = (const T *)pops + P.base;
    double acc[5] = {0, 0, 0, 0, 0};
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < V;
         s += (int64_t)gridDim.x * blockDim.x) {
        const int y = (int)(s / nx), x = (int)(s - (int64_t)y * nx);
        double r = 0, jx = 0, jy = 0;
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const int xs = wrap_add(x, -kVX[i], nx), ys = wrap_add(y, -kVY[i], ny);
            const double d = (double)Codec<S>::decode(p[(int64_t)i * plane + ys * px + xs], P, i);
            r += d;
            jx += kVX[i] * d;
            jy += kVY[i] * d;
        }
        acc[0] += r;
        acc[1] += jx;
        acc[2] += jy;
        acc[3] += (x & 1) ? -jx : jx;
        acc[4] += (y & 1) ? -jy : jy;
    }
    block_sum<5>(acc, part + 5 * blockIdx.x);
}

template <int NV>
__global__ __launch_bounds__(kThreads) void reduce_parts_kernel(const double *part, int nparts,
                                                                double *out)
{
    double acc[NV];
#pragma unroll
    for (int q = 0; q < NV; ++q) acc[q] = 0;
    for (int b = threadIdx.x; b < nparts; b += blockDim.x)
#pragma unroll
        for (int q = 0; q < NV; ++q) acc[q] += part[NV * b + q];
    block_sum<NV>(acc, out);
}

hipError_t launch_conservation(const DeviceView &v, int lattice, int nx, int ny, double *part,
                               int nblocks, double *out_dev, hipStream_t s)
{
    (void)nx;
    (void)ny;
    const dim3 grid(nblocks), block(kThreads);
    const void *p = v.pops[v.cur];
    if (v.storage == kF32)
        hipLaunchKernelGGL(conservation_kernel<kF32>, grid, block, 0, s, p, v.params, lattice, part);
    else if (v.storage == kBF16)
        hipLaunchKernelGGL(conservation_kernel<kBF16>, grid, block, 0, s, p, v.params, lattice,
                           part);
    else
        hipLaunchKernelGGL(conservation_kernel<kF16>, grid, block, 0, s, p, v.params, lattice, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_parts_kernel<5>, dim3(1), block, 0, s, part, nblocks, out_dev);
    return hipGetLastError();
}

// ---------------------------------------------------------------------
// Thermal start: add sqrt(mu rho0 w_i) z_i(x) to f_i(x) (stored at x - v_i),
// then subtract each population's spatial mean of what was added.
// ---------------------------------------------------------------------
template <int S>
__global__ __launch_bounds__(kThreads) void thermal_add_kernel(void *pops,
                                                               const LatticeParams *params,
                                                               int lattice, uint32_t key0,
                                                               uint32_t key1, double *part)
{
    using T = typename Codec<S>::T;
    const LatticeParams &P = params[lattice];
    const int nx = P.nx, ny = P.ny, px = P.px;
    const int64_t V = (int64_t)nx * ny, plane = P.plane;
    T *p = (T *)pops + P.base;
    double acc[9] = {0, 0, 0, 0, 0, 0, 0, 0, 0};
    for (int64_t s = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; s < V;
         s += (int64_t)gridDim.x * blockDim.x) {
        const int y = (int)(s / nx), x = (int)(s - (int64_t)y * nx);
        float z[12];
        normals6(philox4x32_10(make_uint4((uint32_t)s, 0xFFFFFFFFu, P.stream_id, 0u), key0, key1),
                 z);
        normals6(philox4x32_10(make_uint4((uint32_t)s, 0xFFFFFFFFu, P.stream_id, 1u), key0, key1),
                 z + 6);
#pragma unroll
        for (int i = 0; i < 9; ++i) {
            const float add = P.therm_amp[i] * z[i];
            const int xs = wrap_add(x, -kVX[i], nx), ys = wrap_add(y, -kVY[i], ny);
            T *q = p + (int64_t)i * plane + ys * px + xs;
            *q = Codec<S>::encode(Codec<S>::decode(*q, P, i) + add, P, i);
            acc[i] += (double)add;
        }
    }
    block_sum<9>(acc, part + 9 * blockIdx.x);
}

template <int S>
__global__ __launch_bounds__(kThreads) void thermal_sub_kernel(void *pops,
                                                               const LatticeParams *params,
                                                               int lattice, const double *sums)
{
    using T = typename Codec<S>::T;
    const LatticeParams &P = params[lattice];
    const int nx = P.nx, px = P.px;
    const int64_t V = (int64_t)nx * P.ny, plane = P.plane;
    T *p = (T *)pops + P.base;
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < 9 * V;
         k += (int64_t)gridDim.x * blockDim.x) {
        const int i = (int)(k / V);
        const int s = (int)(k - (int64_t)i * V);
        const int y = s / nx, x = s - y * nx;
        const float mean = (float)(sums[i] / (double)V);
        T *q = p + (int64_t)i * plane + y * px + x;
        *q = Codec<S>::encode(Codec<S>::decode(*q, P, i) - mean, P, i);
    }
}

hipError_t launch_thermalize(const DeviceView &v, int lattice, int nx, int ny, double *part,
                             int nblocks, double *sums_dev, hipStream_t s)
{
    const uint32_t k0 = (uint32_t)(v.seed & 0xFFFFFFFFu), k1 = (uint32_t)(v.seed >> 32);
    void *p = v.pops[v.cur];
    const dim3 block(kThreads);
    if (v.storage == kF32)
        hipLaunchKernelGGL(thermal_add_kernel<kF32>, dim3(nblocks), block, 0, s, p, v.params,
                           lattice, k0, k1, part);
    else if (v.storage == kBF16)
        hipLaunchKernelGGL(thermal_add_kernel<kBF16>, dim3(nblocks), block, 0, s, p, v.params,
                           lattice, k0, k1, part);
    else
        hipLaunchKernelGGL(thermal_add_kernel<kF16>, dim3(nblocks), block, 0, s, p, v.params,
                           lattice, k0, k1, part);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(reduce_parts_kernel<9>, dim3(1), block, 0, s, part, nblocks, sums_dev);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    const dim3 grid(grid_for(9LL * nx * ny));
    if (v.storage == kF32)
        hipLaunchKernelGGL(thermal_sub_kernel<kF32>, grid, block, 0, s, p, v.params, lattice,
                           sums_dev);
    else if (v.storage == kBF16)
        hipLaunchKernelGGL(thermal_sub_kernel<kBF16>, grid, block, 0, s, p, v.params, lattice,
                           sums_dev);
    else
        hipLaunchKernelGGL(thermal_sub_kernel<kF16>, grid, block, 0, s, p, v.params, lattice,
                           sums_dev);
    return hipGetLastError();
}

// ---------------------------------------------------------------------
// Noise words and normals as the step kernel computes them (testing).
// ---------------------------------------------------------------------
__global__ __launch_bounds__(kThreads) void debug_noise_kernel(uint32_t key0, uint32_t key1,
                                                               uint32_t stream_id, uint32_t t,
                                                               int64_t site0, int64_t n,
                                                               uint32_t *words, float *zout)
{
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * blockDim.x) {
        const uint4 w = philox4x32_10(make_uint4((uint32_t)(site0 + k), t, stream_id, 0u), key0,
                                      key1);
        float z[6];
        normals6(w, z);
        if (words) {
            words[4 * k + 0] = w.x;
            words[4 * k + 1] = w.y;
            words[4 * k + 2] = w.z;
            words[4 * k + 3] = w.w;
        }
        if (zout)
            for (int q = 0; q < 6; ++q) zout[6 * k + q] = z[q];
    }
}

hipError_t launch_debug_noise(uint64_t seed, uint32_t stream_id, uint32_t t, int64_t site0,
                              int64_t n, uint32_t *words_dev, float *z_dev, hipStream_t s)
{
    hipLaunchKernelGGL(debug_noise_kernel, dim3(grid_for(n)), dim3(kThreads), 0, s,
                       (uint32_t)(seed & 0xFFFFFFFFu), (uint32_t)(seed >> 32), stream_id, t,
                       site0, n, words_dev, z_dev);
    return hipGetLastError();
}

// Zero-fill without hipMemset (safe inside captured graphs).
__global__ __launch_bounds__(kThreads) void fill_kernel(double *p, int64_t n)
{
    for (int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; k < n;
         k += (int64_t)gridDim.x * blockDim.x)
        p[k] = 0.0;
}

hipError_t launch_fill(double *p, size_t n, hipStream_t s)
{
    hipLaunchKernelGGL(fill_kernel, dim3(grid_for((int64_t)n)), dim3(kThreads), 0, s, p,
                       (int64_t)n);
    return hipGetLastError();
}

}  // namespace flbdev

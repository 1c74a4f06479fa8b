// flb_small.hip -- lattices of at most kSmallSites sites, each resident in
// one block: the state is read into LDS once, stepped and sampled there any
// number of times, and written back.
//
// A thread owns one site.  A step reads the site's nine populations from
// the neighbours' LDS (pull, Eq. 1), waits until every site has, collides
// (update_site: the bits of every other step kernel) and writes the site's
// own nine.  A sample takes the fluctuation fields of the same gather,
// transforms them in LDS by direct sums over a row and then a column, and
// adds the products to the FP64 sums in memory (which the L2 holds).
//
// Why direct sums: the lines are a few dozen points of any length, where
// Bluestein's convolution works on lines of up to four times the length
// (20 points: 64) and every pass is a barrier (flb_direct.h).
//
// What bounds it: VALU issue and LDS of the compute units that hold a
// lattice; a step waits for nothing but its two barriers.
#include "flb_collide.h"
#include "flb_direct.h"
#include "flb_small.h"
#include "flb_sums.h"

namespace flbdev {

namespace {

struct SmallArgs {
    void *pops;
    const LatticeParams *params;
    const float2 *tables;
    const int32_t *lattices;
    const uint32_t *step;
    double *acc;
    double *csum_part;
    uint32_t nsteps, every;
    int sample_first, keep_sums;
    uint32_t key0, key1;
};

// Division of a task's index x by a count d of the lattice, by a multiply
// whose factor is made once (the compiler's division is some 25 instructions
// a task, of about 350; a sample with moments of 512 lattices of 20^2 9.9 and
// 8.9 us).  Exact where x d < 2^16: a lattice of V <= 1024 sites
// and sides n <= 64 has at most 6 (V / 4 + n) tasks of d <= n / 2 + 1, and
// 1024 sites of d <= 64.
struct SmallDiv {
    uint32_t d, m;
    __device__ __forceinline__ explicit SmallDiv(int n)
        : d((uint32_t)n), m((65535u + (uint32_t)n) / (uint32_t)n)
    {
    }
    __device__ __forceinline__ int div(int x, int &rem) const
    {
        const uint32_t q = __umul24((uint32_t)x, m) >> 16;
        rem = (int)((uint32_t)x - __umul24(q, d));
        return (int)q;
    }
};
struct SmallDivs {
    SmallDiv nx, ny, nkx, px, py;  // px, py: tasks per row and per column
    __device__ __forceinline__ SmallDivs(int x, int y, int k)
        : nx(x), ny(y), nkx(k), px(direct_tasks(x)), py(direct_tasks(y))
    {
    }
};

// Places from one row of a field to the next: odd, as a wave's tasks read
// several rows at the same column (32 columns: rows two apart would share
// their banks; a sample at 32^2 8.5 us without the odd place, 6.7 with it).
__host__ __device__ inline int small_row(int nx) { return nx | 1; }

// Half spectra of NF real fields [f][ny][small_row(nx)] along their rows:
// out[(f ny + y) nkx + k], k = 0 .. nx/2; roots[m] = exp(-2 pi i m / nx).
// A task is a pass over one row of two fields, which share the roots.
template <int NF>
__device__ __forceinline__ void small_rows(const float *fld, float2 *out, const float2 *roots,
                                           int nx, int ny, int nkx, const SmallDivs &by)
{
    constexpr int G = 2, NG = (NF + G - 1) / G;
    const int px = small_row(nx), V = px * ny;
    const int nt = NG * direct_tasks(nx) * ny;
    for (int task = (int)threadIdx.x; task < nt; task += (int)blockDim.x) {
        int y, k;
        const int grp = by.ny.div(by.px.div(task, k), y);
        const int f0 = grp * G, f1 = min(f0 + 1, NF - 1);  // (the last field again, not stored)
        const float *row[G] = {fld + f0 * V + y * px, fld + f1 * V + y * px};
        float c[G][2], s[G][2];
        direct_sums<G>(nx, k, roots, [&](int f, int j) { return row[f][j]; }, c, s);
#pragma unroll
        for (int f = 0; f < G; ++f) {
            if (f0 + f >= NF) break;
            float2 *o = out + ((f0 + f) * ny + y) * nkx;
            o[k] = make_float2(c[f][0] + c[f][1], s[f][0] + s[f][1]);
            if ((nx & 1) == 0 && 4 * k != nx)
                o[nx / 2 - k] = make_float2(c[f][0] - c[f][1], s[f][1] - s[f][0]);
        }
    }
}

// Column transforms of NF row spectra, [f][ny][nkx] to the same order: a
// task is a pass over one column of one field.
template <int NF>
__device__ __forceinline__ void small_cols(const float2 *in, float2 *out, const float2 *roots,
                                           int ny, int nkx, const SmallDivs &by)
{
    const int nt = NF * direct_tasks(ny) * nkx;
    for (int task = (int)threadIdx.x; task < nt; task += (int)blockDim.x) {
        int kx, ky;
        const int f = by.py.div(by.nkx.div(task, kx), ky);
        const float2 *col = in + f * ny * nkx + kx;
        float2 *o = out + f * ny * nkx + kx;
        float2 c[1][2], s[1][2];
        direct_sums<1>(ny, ky, roots, [&](int, int j) { return col[j * nkx]; }, c, s);
        direct_outputs<1>(ny, ky, c, s, [&](int k, const float2(&X)[1]) { o[k * nkx] = X[0]; });
    }
}

// The products of the spectra z[f][ny][nkx] added to the sums: held in LDS
// (lacc: [kind][ny nkx]) or in memory.
template <int NF>
__device__ __forceinline__ void small_add(const float2 *z, int ny, int nkx, double *lacc,
                                          double *acc, int64_t kstride)
{
    constexpr int NK = NF == kFields ? kKinds : NF, K0 = NF == kFields ? 0 : kKinds;
    const int np = ny * nkx;
    for (int p = (int)threadIdx.x; p < np; p += (int)blockDim.x) {
        if (p == 0) continue;  // k = 0 carries no fluctuation
        float2 X[NF];
#pragma unroll
        for (int f = 0; f < NF; ++f) X[f] = z[f * np + p];
        double u[NK];
        if constexpr (NF == kFields) products_k(u, X);
        else moment_products_k(u, X);
        if (lacc) {
            double *a = lacc + K0 * np + p;
#pragma unroll
            for (int q = 0; q < NK; ++q) a[q * np] += u[q];
        } else {
            const int y = p / nkx;
            add_to_sums(acc + K0 * kstride + spec_offset(y, p - y * nkx, ny), kstride, u);
        }
    }
}

// The sums between memory and LDS (store: back to memory).
__device__ __forceinline__ void small_move_sums(double *lacc, double *acc, int nk, int ny, int nkx,
                                                int64_t kstride, bool store)
{
    const int np = ny * nkx;
    for (int j = (int)threadIdx.x; j < nk * np; j += (int)blockDim.x) {
        const int q = j / np, p = j - q * np, y = p / nkx;
        double *a = acc + q * kstride + spec_offset(y, p - y * nkx, ny);
        if (store) *a = lacc[j];
        else lacc[j] = *a;
    }
}

// Block sum of five doubles into out[0 .. 4], in a fixed order.
__device__ __forceinline__ void small_sum5(double (&v)[5], double (*red)[16], double *out)
{
    const int lane = (int)threadIdx.x & 63, wv = (int)threadIdx.x >> 6;
#pragma unroll
    for (int q = 0; q < 5; ++q) {
        double x = v[q];
#pragma unroll
        for (int o = 32; o > 0; o >>= 1) x += __shfl_down(x, o, 64);
        if (lane == 0) red[q][wv] = x;
    }
    __syncthreads();
    if (threadIdx.x < 5) {
        double x = 0;
        for (int w = 0; w < (int)blockDim.x / 64; ++w) x += red[threadIdx.x][w];
        out[threadIdx.x] = x;
    }
}

// Site `e` of a small lattice: its coordinates and the LDS places its nine
// populations come from.
struct SmallSite {
    int x, y, src[9];
    __device__ __forceinline__ SmallSite(int e, int nx, int ny, const SmallDivs &by)
    {
        const int V = nx * ny;
        y = by.nx.div(e, x);
        const int xm = x == 0 ? nx - 1 : x - 1, xp = x == nx - 1 ? 0 : x + 1, rc = y * nx;
        const int rm = (y == 0 ? ny - 1 : y - 1) * nx, rp = (y == ny - 1 ? 0 : y + 1) * nx;
        src[0] = e;
        src[1] = 1 * V + rc + xm;
        src[2] = 2 * V + rm + x;
        src[3] = 3 * V + rc + xp;
        src[4] = 4 * V + rp + x;
        src[5] = 5 * V + rm + xm;
        src[6] = 6 * V + rm + xp;
        src[7] = 7 * V + rp + xp;
        src[8] = 8 * V + rp + xm;
    }
};

// A thread index the compiler knows nothing about: what is derived from it
// is computed where it is used, not kept in registers across the kernel's
// other phases (a sample fills them, and the step loop then spilled).
__device__ __forceinline__ int fresh_thread()
{
    int e = (int)threadIdx.x;
    asm volatile("" : "+v"(e));
    return e;
}

// A block's LDS: the post-collision values as stored, [9][V]; with samples
// also the fields of each set (later its spectra), the row spectra of one
// set, the roots of unity, and the sums if they are kept here.
struct SmallLds {
    float *st, *fld, *mom;
    float2 *spec, *rx, *ry;
    double *acc;
};
// Floats from one part to the next.
__host__ __device__ inline int small_even(int floats) { return (floats + 1) / 2 * 2; }
__host__ __device__ inline int small_set(int nf, int nx, int ny)
{
    const int a = nf * small_row(nx) * ny, b = 2 * nf * ny * (nx / 2 + 1);
    return small_even(a > b ? a : b);
}
// (the conservation sums' reduction uses the row spectra's place: 80 doubles)
__host__ __device__ inline int small_spec(int nf, int nx, int ny)
{
    const int a = 2 * nf * ny * (nx / 2 + 1);
    return a > 160 ? a : 160;
}

// A sample of the state in L.st: its products added to the lattice's sums;
// cons: also its conservation sums.
template <int S, bool MOM>
__device__ __forceinline__ void small_sample(const SmallArgs &g, const LatticeParams &P,
                                             const SmallLds &L, const SmallDivs &by, bool cons)
{
    using T = typename Codec<S>::T;
    const int nx = P.nx, ny = P.ny, nkx = P.nkx, V = nx * ny, e = fresh_thread();
    float *fld = L.fld, *mom = L.mom;
    double sums[5] = {0, 0, 0, 0, 0};
    if (e < V) {
        const SmallSite at(e, nx, ny, by);
        float d[9];
#pragma unroll
        for (int q = 0; q < 9; ++q) d[q] = Codec<S>::decode((T)L.st[at.src[q]], P, q);
        const float r = d[0] + (d[1] + d[3]) + (d[2] + d[4]) + (d[5] + d[7]) + (d[6] + d[8]);
        const float jx = (d[1] - d[3]) + (d[5] - d[7]) - (d[6] - d[8]);
        const float jy = (d[2] - d[4]) + (d[5] - d[7]) + (d[6] - d[8]);
        const float ir = __builtin_amdgcn_rcpf(P.rho0 + r);
        const int pad = small_row(nx) - nx, F = V + ny * pad, o = e + at.y * pad;
        fld[o] = r;
        fld[F + o] = jx - P.rho0 * P.u0x;
        fld[2 * F + o] = jy - P.rho0 * P.u0y;
        fld[3 * F + o] = fmaf(jx, ir, -P.u0x);
        fld[4 * F + o] = fmaf(jy, ir, -P.u0y);
        if constexpr (MOM) {
            float M[6];
            moments_of(d, M);
#pragma unroll
            for (int q = 0; q < 6; ++q) mom[q * F + o] = M[q];
        }
        const double Jx = jx, Jy = jy;
        sums[0] = r;
        sums[1] = Jx;
        sums[2] = Jy;
        sums[3] = (at.x & 1) ? -Jx : Jx;
        sums[4] = (at.y & 1) ? -Jy : Jy;
    }
    if (cons) {
        small_sum5(sums, reinterpret_cast<double(*)[16]>(L.spec),
                   g.csum_part + 5 * (int64_t)P.fld_part0);
    }
    __syncthreads();
    double *acc = g.acc + P.acc_base;
    const int64_t kstride = (int64_t)ny * P.kxp;
    // the spectra of a set take the place of its fields
    float2 *z = reinterpret_cast<float2 *>(fld);
    small_rows<kFields>(fld, L.spec, L.rx, nx, ny, nkx, by);
    __syncthreads();
    small_cols<kFields>(L.spec, z, L.ry, ny, nkx, by);
    __syncthreads();
    small_add<kFields>(z, ny, nkx, L.acc, acc, kstride);
    if constexpr (MOM) {
        z = reinterpret_cast<float2 *>(mom);
        small_rows<kMomentFields>(mom, L.spec, L.rx, nx, ny, nkx, by);
        __syncthreads();
        small_cols<kMomentFields>(L.spec, z, L.ry, ny, nkx, by);
        __syncthreads();
        small_add<kMomentFields>(z, ny, nkx, L.acc, acc, kstride);
    }
}

// One block per lattice of the list.  nsteps steps; a sample of the state
// before them (sample_first) and, with every > 0, after each step that
// reaches a time divisible by it.
template <int S, bool NOISE, bool MOM>
__global__ __launch_bounds__(kSmallSites) void small_kernel(SmallArgs g)
{
    using T = typename Codec<S>::T;
    extern __shared__ double lds[];
    const LatticeParams &P = g.params[g.lattices[blockIdx.x]];
    const int nx = P.nx, ny = P.ny, V = nx * ny;
    constexpr int NF = MOM ? kMomentFields : kFields, NK = kKinds + (MOM ? kMomentFields : 0);
    SmallLds L;
    L.st = reinterpret_cast<float *>(lds);
    L.fld = L.st + small_even(9 * V);
    L.mom = L.fld + small_set(kFields, nx, ny);
    L.spec = reinterpret_cast<float2 *>(MOM ? L.mom + small_set(kMomentFields, nx, ny) : L.mom);
    L.rx = L.spec + small_spec(NF, nx, ny) / 2;
    L.ry = nx == ny ? L.rx : L.rx + nx;
    L.acc = g.keep_sums ? reinterpret_cast<double *>(L.ry + ny) : nullptr;
    float *st = L.st;
    const SmallDivs by(nx, ny, P.nkx);
    const int64_t kstride = (int64_t)ny * P.kxp;
    const bool sampled = g.sample_first || g.every;
    {
        const int e = fresh_thread(), y = e / nx, x = e - y * nx;
        const T *pops = (const T *)g.pops + P.base + (int64_t)y * P.px + x;
        if (e < V)
#pragma unroll
            for (int i = 0; i < 9; ++i) st[i * V + e] = Work<S>::in(pops[i * P.plane]);
        if (sampled) {
            for (int j = e; j < nx; j += (int)blockDim.x) L.rx[j] = g.tables[P.roots_x + j];
            if (nx != ny)
                for (int j = e; j < ny; j += (int)blockDim.x) L.ry[j] = g.tables[P.roots_y + j];
            if (L.acc)
                small_move_sums(L.acc, g.acc + P.acc_base, NK, ny, P.nkx, kstride, false);
        }
    }
    __syncthreads();
    uint32_t t = *g.step, left = g.nsteps;
    bool due = g.sample_first != 0;
    for (;;) {
        // steps to the next sample after this one
        const uint32_t next = g.every ? g.every - t % g.every : 0xFFFFFFFFu;
        if (sampled && due)
            small_sample<S, MOM>(g, P, L, by, left < next);
        if (!left) break;
        const uint32_t n = min(left, next);
        const int e = fresh_thread();
        const SmallSite at(e, nx, ny, by);
        for (uint32_t k = 0; k < n; ++k) {
            float d[9];
            if (e < V)
#pragma unroll
                for (int q = 0; q < 9; ++q) d[q] = st[at.src[q]];
            __syncthreads();
            if (e < V) {
                update_site<NOISE, S>(d, P, (uint32_t)e, t + k, g.key0, g.key1);
#pragma unroll
                for (int q = 0; q < 9; ++q) st[q * V + e] = stored<S>(d[q]);
            }
            __syncthreads();
        }
        t += n;
        left -= n;
        due = n == next;
    }
    if (g.nsteps) {
        const int e = fresh_thread(), y = e / nx, x = e - y * nx;
        T *pops = (T *)g.pops + P.base + (int64_t)y * P.px + x;
        if (e < V)
#pragma unroll
            for (int i = 0; i < 9; ++i) pops[i * P.plane] = (T)st[i * V + e];
    }
    if (L.acc) {
        __syncthreads();
        small_move_sums(L.acc, g.acc + P.acc_base, NK, ny, P.nkx, kstride, true);
    }
}

template <int S, bool NOISE>
hipError_t launch_small_m(const SmallArgs &a, int nlat, int threads, int lds, bool moments,
                          hipStream_t s)
{
    if (moments)
        hipLaunchKernelGGL((small_kernel<S, NOISE, true>), dim3(nlat), dim3(threads), lds, s, a);
    else
        hipLaunchKernelGGL((small_kernel<S, NOISE, false>), dim3(nlat), dim3(threads), lds, s, a);
    return hipGetLastError();
}

}  // namespace

int small_lds_bytes(int nx, int ny, bool sampled, bool moments, bool keep_sums)
{
    const int V = nx * ny, nf = moments ? kMomentFields : kFields;
    int floats = small_even(9 * V);
    if (sampled)
        floats += small_set(kFields, nx, ny) + (moments ? small_set(kMomentFields, nx, ny) : 0) +
                  small_spec(nf, nx, ny) + 2 * (nx == ny ? nx : nx + ny);
    if (sampled && keep_sums)
        floats += 2 * (kKinds + (moments ? kMomentFields : 0)) * ny * (nx / 2 + 1);
    return floats * (int)sizeof(float);
}

hipError_t launch_small(const DeviceView &v, const int32_t *lattices, int nlat, int threads,
                        int lds_bytes, uint32_t nsteps, uint32_t every,
                        bool sample_first, bool keep_sums, bool noise, bool moments,
                        hipStream_t s)
{
    SmallArgs a;
    a.pops = v.pops[v.cur];
    a.params = v.params;
    a.tables = v.tables;
    a.lattices = lattices;
    a.step = v.step + v.cur;
    a.acc = v.acc;
    a.csum_part = v.csum_part;
    a.nsteps = nsteps;
    a.every = every;
    a.sample_first = sample_first;
    a.keep_sums = keep_sums;
    a.key0 = (uint32_t)(v.seed & 0xFFFFFFFFu);
    a.key1 = (uint32_t)(v.seed >> 32);
    if (threads < 64 || threads > kSmallSites || threads % 64) return hipErrorInvalidValue;
#define FLB_SEL(S_)                                                                          \
    if (v.storage == S_)                                                                     \
        return noise ? launch_small_m<S_, true>(a, nlat, threads, lds_bytes, moments, s)     \
                     : launch_small_m<S_, false>(a, nlat, threads, lds_bytes, moments, s);
    FLB_SEL(kF32)
    FLB_SEL(kBF16)
    FLB_SEL(kF16)
#undef FLB_SEL
    return hipErrorInvalidValue;
}

}  // namespace flbdev

// rt_kernels.hip -- gfx950 kernels of the explicit M1 RT step.
//
//   k_inject     point-source injection (Sec. 3.1)
//   k_transport  unsplit GLF/HLL update of (N, F), all groups (Sec. 3.2)
//   the dispatch of the thermochemistry kernels (rt_chem.hip)
//   k_reduce_*   photon budget and diagnostics (fixed-order tree sums)
//
// Radiation arrays are structure-of-arrays, x fastest, one plane of ncell
// values per group and component, so a wavefront reads 64 consecutive cells
// of one component with one coalesced access.
#include "rt_chem.h"

namespace rtm1 {

// ------------------------------------------------------------------ inject
// The source cells are distinct (sources sharing a cell are merged on the
// host), so each thread owns its cell.  prev, when given, receives the
// photon density before the injection (smoothed RT).
template <typename R>
__global__ void k_inject(R *__restrict__ N, size_t ncell, int M, int nsrc, const int32_t *__restrict__ cell,
                         const double *__restrict__ rate, double dtV, double *__restrict__ prev)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= nsrc) return;
    const size_t i = (size_t)cell[s];
    for (int g = 0; g < M; ++g) {
        R *p = N + (size_t)g * ncell + i;
        const double n0 = (double)*p;
        if (prev) prev[(size_t)s * M + g] = n0;
        *p = R(n0 + rate[(size_t)s * M + g] * dtV);
    }
}

hipError_t launch_inject(bool fp32, void *N, size_t ncell, int M, int nsrc, const int32_t *cell,
                         const double *rate, double dt_over_V, double *prev, hipStream_t s)
{
    if (nsrc <= 0) return hipSuccess;
    dim3 b(64), gr((nsrc + 63) / 64);
    if (fp32)
        hipLaunchKernelGGL(k_inject<float>, gr, b, 0, s, (float *)N, ncell, M, nsrc, cell, rate, dt_over_V, prev);
    else
        hipLaunchKernelGGL(k_inject<double>, gr, b, 0, s, (double *)N, ncell, M, nsrc, cell, rate, dt_over_V, prev);
    return hipGetLastError();
}

__global__ void k_fill_i32(int32_t *p, size_t n, int32_t v)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

__global__ void k_fill_u8(uint8_t *p, size_t n, uint8_t v)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

hipError_t launch_fill_u8(uint8_t *p, size_t n, uint8_t v, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    hipLaunchKernelGGL(k_fill_u8, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
    return hipGetLastError();
}

__global__ void k_source_map(int32_t *map, const int32_t *__restrict__ cell, int nsrc)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s < nsrc) map[cell[s]] = s;
}

hipError_t launch_source_map(int32_t *map, size_t ncell, const int32_t *cell, int nsrc, hipStream_t s)
{
    hipLaunchKernelGGL(k_fill_i32, dim3((unsigned)((ncell + 255) / 256)), dim3(256), 0, s, map, ncell, -1);
    if (nsrc > 0) hipLaunchKernelGGL(k_source_map, dim3((nsrc + 63) / 64), dim3(64), 0, s, map, cell, nsrc);
    return hipGetLastError();
}

// ---------------------------------------------------------- accounting
unsigned acct_blocks(size_t ncell) { return (unsigned)((ncell + ACCT_THREADS - 1) / ACCT_THREADS); }
size_t acct_bytes(size_t ncell) { return ((size_t)acct_blocks(ncell) * 6 * sizeof(double) + 255) & ~(size_t)255; }

// --------------------------------------------------------------- transport
template <typename R, int FLUX>
__global__ __launch_bounds__(256) void k_transport(KGrid g, int M, R c, R kdx, const R *__restrict__ Nin,
                                                   const R *__restrict__ Fin, R *__restrict__ Nout,
                                                   R *__restrict__ Fout, const R *__restrict__ tab, int nf,
                                                   int nth, double *__restrict__ acct)
{
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const size_t nc = g.ncell;
    double av[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (i < (uint32_t)nc) {
        int ix, iy, iz;
        cell_coords(g, i, ix, iy, iz);
        const Nbr nb = neighbours(g, i, ix, iy, iz);
        for (int grp = 0; grp < M; ++grp) {
            double bout = 0.0;
            const U4<R> o = transport_cell<R, FLUX>(nb, i, nc, Nin + (size_t)grp * nc, Fin + (size_t)3 * grp * nc,
                                                    c, kdx, tab, nf, nth, bout, g, grp);
            Nout[(size_t)grp * nc + i] = o.n;
            R *Fo = Fout + (size_t)3 * grp * nc;
            Fo[i] = o.fx;
            Fo[nc + i] = o.fy;
            Fo[2 * nc + i] = o.fz;
            if (grp < 3) {
                av[grp] = (double)o.n;
                av[3 + grp] = bout;
            }
        }
    }
    if (acct) block_acct(acct, av);
}

hipError_t launch_transport(bool fp32, int flux, const KGrid &g, int M, double c, double dt, const void *Nin,
                            const void *Fin, void *Nout, void *Fout, const void *hll, int nf, int nth,
                            double *acct, hipStream_t s)
{
    dim3 b(256), gr((unsigned)((g.ncell + 255) / 256));
    const double k = dt / g.dx;
    if (fp32) {
        auto kern = flux ? k_transport<float, 1> : k_transport<float, 0>;
        hipLaunchKernelGGL(kern, gr, b, 0, s, g, M, (float)c, (float)k, (const float *)Nin, (const float *)Fin,
                           (float *)Nout, (float *)Fout, (const float *)hll, nf, nth, acct);
    } else {
        auto kern = flux ? k_transport<double, 1> : k_transport<double, 0>;
        hipLaunchKernelGGL(kern, gr, b, 0, s, g, M, c, k, (const double *)Nin, (const double *)Fin,
                           (double *)Nout, (double *)Fout, (const double *)hll, nf, nth, acct);
    }
    return hipGetLastError();
}

// --------------------------------------------------------- thermochemistry
template <typename R>
static void launch_chem_pass(ChemPass pass, const KChem &kc, const ChemCall<R> &a, hipStream_t s)
{
    const int v = (a.io.sm.N ? V_SMOOTH : 0) | (kc.otsa ? 0 : V_CASE_A);
    if (v == 0) launch_chem_variant<R, 0>(pass, kc.M, a, s);
    else if (v == 1) launch_chem_variant<R, 1>(pass, kc.M, a, s);
    else if (v == 2) launch_chem_variant<R, 2>(pass, kc.M, a, s);
    else launch_chem_variant<R, 3>(pass, kc.M, a, s);
}

template <typename R>
static ChemIO<R> make_io(size_t ncell, void *N, void *F, double *xHII, double *xHeII, double *xHeIII, double *T,
                         const double *nH, int32_t *nacc, int32_t *natt, double *acct, unsigned long long *hist,
                         const SmoothArgs *sm, double dt, double a, uint8_t *prev_att)
{
    ChemIO<R> io;
    io.prev_att = prev_att;
    io.a3 = a * a * a;
    io.ia3 = 1.0 / io.a3;
    io.acct = acct;
    io.hist = hist;
    if (sm) {
        io.sm.N = (const R *)sm->N;
        io.sm.F = (const R *)sm->F;
        io.sm.map = sm->map;
        io.sm.prev = sm->prev;
        io.sm.dt = dt;
    }
    io.ncell = ncell;
    io.N = (R *)N;
    io.F = (R *)F;
    io.xHII = xHII;
    io.xHeII = xHeII;
    io.xHeIII = xHeIII;
    io.T = T;
    io.nH = nH;
    io.nacc = nacc;
    io.natt = natt;
    return io;
}

hipError_t launch_chem(int part, bool fp32, const KGrid &g, const KChem &kc, const KChem *dk, double dt, void *N, void *F, double *xHII,
                       double *xHeII, double *xHeIII, double *T, const double *nH, int32_t *nacc, int32_t *natt,
                       const QueueView &q, int K, unsigned long long *hist, const SmoothArgs *sm, double a,
                       uint8_t *prev_att, DevStats *stats, hipStream_t s)
{
    const ChemPass pass = part == 1 ? CHEM_HEAD : CHEM_TAIL;
    if (fp32)
        launch_chem_pass<float>(pass, kc,
                                {g, dk, dt, 0.f, 0.f, nullptr, nullptr,
                                 make_io<float>(g.ncell, N, F, xHII, xHeII, xHeIII, T, nH, nacc, natt, nullptr, hist, sm,
                                                dt, a, prev_att),
                                 nullptr, 0, 0, q, K, stats, kc.isothermal != 0},
                                s);
    else
        launch_chem_pass<double>(pass, kc,
                                 {g, dk, dt, 0.0, 0.0, nullptr, nullptr,
                                  make_io<double>(g.ncell, N, F, xHII, xHeII, xHeIII, T, nH, nacc, natt, nullptr, hist,
                                                  sm, dt, a, prev_att),
                                  nullptr, 0, 0, q, K, stats, kc.isothermal != 0},
                                 s);
    return hipGetLastError();
}

hipError_t launch_chem_all(bool fp32, const KGrid &g, const KChem &kc, const KChem *dk, double dt, void *N, void *F,
                           double *xHII, double *xHeII, double *xHeIII, double *T, const double *nH, int32_t *nacc,
                           int32_t *natt, const QueueView &q, unsigned long long *hist, const SmoothArgs *sm, double a,
                           uint8_t *prev_att, DevStats *stats, hipStream_t s)
{
    if (fp32)
        launch_chem_pass<float>(CHEM_ALL, kc,
                                {g, dk, dt, 0.f, 0.f, nullptr, nullptr,
                                 make_io<float>(g.ncell, N, F, xHII, xHeII, xHeIII, T, nH, nacc, natt, nullptr, hist, sm,
                                                dt, a, prev_att),
                                 nullptr, 0, 0, q, 0, stats, kc.isothermal != 0},
                                s);
    else
        launch_chem_pass<double>(CHEM_ALL, kc,
                                 {g, dk, dt, 0.0, 0.0, nullptr, nullptr,
                                  make_io<double>(g.ncell, N, F, xHII, xHeII, xHeIII, T, nH, nacc, natt, nullptr, hist,
                                                  sm, dt, a, prev_att),
                                  nullptr, 0, 0, q, 0, stats, kc.isothermal != 0},
                                 s);
    return hipGetLastError();
}

hipError_t launch_step_fused(int part, bool fp32, int flux, const KGrid &g, const KChem &kc, const KChem *dk, double dt, const void *Nin,
                             const void *Fin, void *Nout, void *Fout, double *xHII, double *xHeII, double *xHeIII,
                             double *T, const double *nH, int32_t *nacc, int32_t *natt, const void *hll, int nf,
                             int nth, const QueueView &q, int K, double *acct, unsigned long long *hist,
                             const SmoothArgs *sm, double a, uint8_t *prev_att, DevStats *stats, hipStream_t s)
{
    // super-comoving transport: light speed a c_r over dt / a^2
    const double kdx = dt / (a * a) / g.dx;
    const double ctr = a * kc.cr;
    const ChemPass pass = part == 2 ? CHEM_TAIL : (flux ? CHEM_FUSED_HLL : CHEM_FUSED_GLF);
    if (fp32)
        launch_chem_pass<float>(pass, kc,
                                {g, dk, dt, (float)ctr, (float)kdx, (const float *)Nin, (const float *)Fin,
                                 make_io<float>(g.ncell, Nout, Fout, xHII, xHeII, xHeIII, T, nH, nacc, natt, acct, hist,
                                                sm, dt, a, prev_att),
                                 (const float *)hll, nf, nth, q, K, stats, kc.isothermal != 0},
                                s);
    else
        launch_chem_pass<double>(pass, kc,
                                 {g, dk, dt, ctr, kdx, (const double *)Nin, (const double *)Fin,
                                  make_io<double>(g.ncell, Nout, Fout, xHII, xHeII, xHeIII, T, nH, nacc, natt, acct,
                                                  hist, sm, dt, a, prev_att),
                                  (const double *)hll, nf, nth, q, K, stats, kc.isothermal != 0},
                                 s);
    return hipGetLastError();
}

// -------------------------------------------------------------- reductions
size_t reduction_scratch_bytes() { return (size_t)RED_BLOCKS * sizeof(RedOut); }

// scratch layout: [reduction partials][queue counters, 512 B]
//                 [cell, acc, att: 3 x cap int32][QV_GRID (or QV_SMOOTH) x cap doubles]
// (the one-pass chemistry holds its order in the int32 planes and its slab
// counters behind them; order_only lays out nothing else)
static size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

size_t queue_bytes(unsigned cap, bool smooth, bool order_only)
{
    return 512 + align256((size_t)cap * 3 * sizeof(int32_t)) +
           (order_only ? CHEM_XCDS * QUEUE_SLAB_STRIDE * sizeof(unsigned)
                       : (size_t)(smooth ? QV_SMOOTH : QV_GRID) * cap * sizeof(double));
}

size_t queue_cell_bytes(bool smooth) { return 3 * sizeof(int32_t) + (size_t)(smooth ? QV_SMOOTH : QV_GRID) * sizeof(double); }

QueueView queue_view(void *scratch, unsigned cap, unsigned layout_cap)
{
    char *b = (char *)scratch + align256(reduction_scratch_bytes());
    QueueView q;
    q.count = (unsigned *)b;
    q.head = q.count + 1;
    q.cnt[0] = q.count + 64;
    q.cnt[1] = q.count + 32;
    q.cnt[2] = q.count;
    b += 512;
    q.cell = (int32_t *)b;
    q.acc = q.cell + layout_cap;
    q.att = q.acc + layout_cap;
    b += align256((size_t)layout_cap * 3 * sizeof(int32_t));
    q.v = (double *)b;
    q.slab = (unsigned *)b;
    q.cap = cap;
    q.rbeg[0] = 0;
    q.rlen[0] = cap / 16;
    q.rbeg[1] = q.rlen[0];
    q.rlen[1] = cap / 4;
    q.rbeg[2] = q.rbeg[1] + q.rlen[1];
    q.rlen[2] = cap - q.rbeg[2];
    q.stride = layout_cap;
    return q;
}

// Sum over the 64 lanes of a wavefront by butterfly exchanges: every lane
// ends with the same total, combined in the same order on every run.
__device__ __forceinline__ double wave_sum(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}
__device__ __forceinline__ double wave_max(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double w = __shfl_xor(v, o, 64);
        v = w > v ? w : v;
    }
    return v;
}
__device__ __forceinline__ double wave_min(double v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        const double w = __shfl_xor(v, o, 64);
        v = w < v ? w : v;
    }
    return v;
}

// Diagnostics of a state (rt_get_stats): per block, grid-stride over the
// cells in a fixed order, then wave butterflies and the block's four waves
// in order.
template <typename R>
__global__ __launch_bounds__(RED_THREADS) void k_reduce_partial(size_t nc, int M, double c, double V,
                                                                const R *__restrict__ N, const R *__restrict__ F,
                                                                const double *__restrict__ xHII,
                                                                const double *__restrict__ nH,
                                                                RedOut *__restrict__ part)
{
    double ph[3] = {0, 0, 0}, ion = 0, mf = 0, mn = 1e300;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < nc; i += (size_t)gridDim.x * blockDim.x) {
        for (int g = 0; g < M; ++g) {
            const double n = (double)N[(size_t)g * nc + i];
            const double fx = (double)F[(size_t)(3 * g) * nc + i];
            const double fy = (double)F[(size_t)(3 * g + 1) * nc + i];
            const double fz = (double)F[(size_t)(3 * g + 2) * nc + i];
            ph[g] += n;
            mn = n < mn ? n : mn;
            if (n > 0) {
                const double f = sqrt(fx * fx + fy * fy + fz * fz) / (c * n);
                mf = f > mf ? f : mf;
            }
        }
        ion += xHII[i] * nH[i];
    }
    __shared__ double s[RED_THREADS / 64][6];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const double v[6] = {wave_sum(ph[0]), wave_sum(ph[1]), wave_sum(ph[2]), wave_sum(ion), wave_max(mf),
                         wave_min(mn)};
    if (lane == 0)
#pragma unroll
        for (int q = 0; q < 6; ++q) s[w][q] = v[q];
    __syncthreads();
    if (threadIdx.x == 0) {
        double a[6];
#pragma unroll
        for (int q = 0; q < 6; ++q) a[q] = s[0][q];
        for (int k = 1; k < RED_THREADS / 64; ++k) {
            for (int q = 0; q < 4; ++q) a[q] += s[k][q];
            a[4] = s[k][4] > a[4] ? s[k][4] : a[4];
            a[5] = s[k][5] < a[5] ? s[k][5] : a[5];
        }
        RedOut r;
        for (int g = 0; g < 3; ++g) r.photons[g] = a[g] * V;
        r.ionised = a[3] * V;
        r.maxf = a[4];
        r.minN = a[5];
        part[blockIdx.x] = r;
    }
}

// The block partials in a fixed order: each of 256 threads combines the
// partials t, t + 256, ... in turn, then a tree over the threads.
__global__ __launch_bounds__(256) void k_reduce_final(const RedOut *__restrict__ part, int np, RedOut *__restrict__ out)
{
    __shared__ double s[6][256];
    const int t = threadIdx.x;
    double a[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 1e300};
    for (int b = t; b < np; b += 256) {
        const RedOut &r = part[b];
        for (int g = 0; g < 3; ++g) a[g] += r.photons[g];
        a[3] += r.ionised;
        a[4] = r.maxf > a[4] ? r.maxf : a[4];
        a[5] = r.minN < a[5] ? r.minN : a[5];
    }
#pragma unroll
    for (int q = 0; q < 6; ++q) s[q][t] = a[q];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (t < o) {
            for (int q = 0; q < 4; ++q) s[q][t] += s[q][t + o];
            s[4][t] = s[4][t + o] > s[4][t] ? s[4][t + o] : s[4][t];
            s[5][t] = s[5][t + o] < s[5][t] ? s[5][t + o] : s[5][t];
        }
        __syncthreads();
    }
    if (t == 0) {
        RedOut r;
        for (int g = 0; g < 3; ++g) r.photons[g] = s[g][0];
        r.ionised = s[3][0];
        r.maxf = s[4][0];
        r.minN = s[5][0];
        *out = r;
    }
}

// Four consecutive values of a group plane (16-byte aligned): one 16-byte
// load for FP32, two for FP64.
__device__ __forceinline__ void load4(const float *p, double v[4])
{
    const float4 a = *reinterpret_cast<const float4 *>(p);
    v[0] = a.x;
    v[1] = a.y;
    v[2] = a.z;
    v[3] = a.w;
}
__device__ __forceinline__ void load4(const double *p, double v[4])
{
    const double2 a = reinterpret_cast<const double2 *>(p)[0], b = reinterpret_cast<const double2 *>(p)[1];
    v[0] = a.x;
    v[1] = a.y;
    v[2] = b.x;
    v[3] = b.y;
}

// Photons per group of one radiation set, for the step's ledger: per block
// the sum of N of each group (grid-stride in a fixed order, wave
// butterflies, the four waves in order) at part[3 b + g].  When every group
// plane starts 16-byte aligned a thread takes four consecutive cells per
// round, two rounds' loads in flight before their sums.
template <typename R>
__global__ __launch_bounds__(RED_THREADS) void k_sum_n(size_t nc, int M, const R *__restrict__ N,
                                                       double *__restrict__ part)
{
    double sg[3] = {0.0, 0.0, 0.0};
    const size_t T = (size_t)gridDim.x * blockDim.x, t0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    size_t i0 = 0;
    if (((uintptr_t)N & 15) == 0 && ((nc * sizeof(R)) & 15) == 0) {
        const size_t n4 = nc / 4;
        size_t q = t0;
        for (; q + T < n4; q += 2 * T) {
            double v[3][2][4];
#pragma unroll
            for (int g = 0; g < 3; ++g)
                if (g < M) {
                    load4(N + (size_t)g * nc + 4 * q, v[g][0]);
                    load4(N + (size_t)g * nc + 4 * (q + T), v[g][1]);
                }
#pragma unroll
            for (int g = 0; g < 3; ++g)
                if (g < M)
#pragma unroll
                    for (int r = 0; r < 2; ++r)
#pragma unroll
                        for (int j = 0; j < 4; ++j) sg[g] += v[g][r][j];
        }
        for (; q < n4; q += T) {
#pragma unroll
            for (int g = 0; g < 3; ++g)
                if (g < M) {
                    double v[4];
                    load4(N + (size_t)g * nc + 4 * q, v);
#pragma unroll
                    for (int j = 0; j < 4; ++j) sg[g] += v[j];
                }
        }
        i0 = 4 * n4;
    }
    for (size_t i = i0 + t0; i < nc; i += T)
        for (int g = 0; g < M; ++g) sg[g] += (double)N[(size_t)g * nc + i];
    __shared__ double s[RED_THREADS / 64][3];
    const int w = threadIdx.x >> 6, lane = threadIdx.x & 63;
#pragma unroll
    for (int g = 0; g < 3; ++g) {
        const double v = wave_sum(sg[g]);
        if (lane == 0) s[w][g] = v;
    }
    __syncthreads();
    if (threadIdx.x < 3) {
        double a = s[0][threadIdx.x];
        for (int k = 1; k < RED_THREADS / 64; ++k) a += s[k][threadIdx.x];
        part[(size_t)3 * blockIdx.x + threadIdx.x] = a;
    }
}

hipError_t launch_sum_n(bool fp32, size_t ncell, int M, const void *N, double *part, hipStream_t s)
{
    if (fp32)
        hipLaunchKernelGGL(k_sum_n<float>, dim3(RED_BLOCKS), dim3(RED_THREADS), 0, s, ncell, M, (const float *)N, part);
    else
        hipLaunchKernelGGL(k_sum_n<double>, dim3(RED_BLOCKS), dim3(RED_THREADS), 0, s, ncell, M, (const double *)N,
                           part);
    return hipGetLastError();
}

// Photon ledger of one step (fixed-order sums; see launch_ledger): the
// photons of the current set from the k_sum_n partials, and with mode 2 the
// transported photons and the boundary outflow from the transport partials.
__global__ __launch_bounds__(256) void k_ledger(int mode, const double *__restrict__ acct, unsigned nblk,
                                                const double *__restrict__ npart, int M, double V, double dtdx2,
                                                DevStats *__restrict__ st)
{
    __shared__ double sh[9][256];
    const int t = threadIdx.x;
    double v[9] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    if (mode == 2)
        for (unsigned b = t; b < nblk; b += 256)
#pragma unroll
            for (int q = 0; q < 6; ++q) v[q] += acct[(size_t)6 * b + q];
    for (unsigned b = t; b < (unsigned)RED_BLOCKS; b += 256)
#pragma unroll
        for (int g = 0; g < 3; ++g) v[6 + g] += npart[(size_t)3 * b + g];
#pragma unroll
    for (int q = 0; q < 9; ++q) sh[q][t] = v[q];
    __syncthreads();
    for (int o = 128; o > 0; o >>= 1) {
        if (t < o)
#pragma unroll
            for (int q = 0; q < 9; ++q) sh[q][t] += sh[q][t + o];
        __syncthreads();
    }
    if (t != 0) return;
    for (int g = 0; g < M; ++g) {
        const double now = sh[6 + g][0] * V;
        if (mode == 0) {
            st->Tpre[g] = now;
            continue;
        }
        const double T0 = mode == 2 ? sh[g][0] * V : st->Tpre[g];
        st->absorbed[g] += T0 - now;
        if (mode == 2) st->outflow[g] += sh[3 + g][0] * dtdx2;
    }
}

hipError_t launch_ledger(int mode, const double *acct, unsigned nblk, const double *npart, int M, double V,
                         double dtdx2, DevStats *st, hipStream_t s)
{
    hipLaunchKernelGGL(k_ledger, dim3(1), dim3(256), 0, s, mode, acct, nblk, npart, M, V, dtdx2, st);
    return hipGetLastError();
}

hipError_t launch_reduce(bool fp32, size_t ncell, int M, double c, double V, const void *N, const void *F,
                         const double *xHII, const double *nH, void *scratch, RedOut *dev_out, hipStream_t s)
{
    RedOut *part = (RedOut *)scratch;
    if (fp32)
        hipLaunchKernelGGL(k_reduce_partial<float>, dim3(RED_BLOCKS), dim3(RED_THREADS), 0, s, ncell, M, c, V,
                           (const float *)N, (const float *)F, xHII, nH, part);
    else
        hipLaunchKernelGGL(k_reduce_partial<double>, dim3(RED_BLOCKS), dim3(RED_THREADS), 0, s, ncell, M, c, V,
                           (const double *)N, (const double *)F, xHII, nH, part);
    hipLaunchKernelGGL(k_reduce_final, dim3(1), dim3(256), 0, s, part, RED_BLOCKS, dev_out);
    return hipGetLastError();
}

}  // namespace rtm1

// rt_chem.hip -- the thermochemistry kernels of the grid (App. A): the
// persistent one-pass kernel, and the head and tail passes.  Compiled once
// per radiation type RT_CHEM_R (float, double) and method variant RT_CHEM_V
// (0..3: V_SMOOTH, V_CASE_A), which build in parallel.
#include "rt_chem.h"

namespace rtm1 {

// Reduction of the chemistry counters: butterflies in each wave, then the
// block's waves in LDS; one set of atomics per block.
__device__ __forceinline__ void block_stats(DevStats *st, unsigned long long acc, unsigned long long att,
                                            unsigned long long mx, unsigned fl)
{
    __shared__ unsigned long long s_st[16][3];
    __shared__ unsigned s_fl[16];
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) {
        acc += __shfl_xor(acc, o, 64);
        att += __shfl_xor(att, o, 64);
        const unsigned long long m = __shfl_xor(mx, o, 64);
        mx = m > mx ? m : mx;
        fl |= __shfl_xor(fl, o, 64);
    }
    const unsigned w = threadIdx.x >> 6;
    if ((threadIdx.x & 63u) == 0) {
        s_st[w][0] = acc;
        s_st[w][1] = att;
        s_st[w][2] = mx;
        s_fl[w] = fl;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (unsigned j = 1; j < (blockDim.x + 63u) >> 6; ++j) {
            acc += s_st[j][0];
            att += s_st[j][1];
            mx = s_st[j][2] > mx ? s_st[j][2] : mx;
            fl |= s_fl[j];
        }
        if (att) {
            atomicAdd(&st->acc_total, acc);
            atomicAdd(&st->att_total, att);
            atomicMax(&st->att_max, mx);
        }
        if (fl) atomicOr(&st->flags, fl);
    }
}

__device__ __forceinline__ int lane_id() { return (int)(threadIdx.x & 63u); }

// Histogram of accepted substeps per cell (bin 63: 63 or more), counted in
// LDS per block and added to the device statistics at the end of the block.
__device__ __forceinline__ void hist_init(unsigned *sh)
{
    if (threadIdx.x < 64) sh[threadIdx.x] = 0u;
    __syncthreads();
}
__device__ __forceinline__ void hist_add(unsigned *sh, int acc) { atomicAdd(&sh[acc < 63 ? acc : 63], 1u); }
__device__ __forceinline__ void hist_flush(const unsigned *sh, unsigned long long *hist)
{
    __syncthreads();
    if (threadIdx.x < 64 && sh[threadIdx.x]) atomicAdd(&hist[threadIdx.x], (unsigned long long)sh[threadIdx.x]);
}

// Head pass: one thread per cell.  With FUSE the cell is first transported
// (all groups, source set -> registers); then up to K chemistry attempts.
// Cells that finish are written to the destination arrays; the rest go to
// the queue (or, when it is full, finish in place).
// Waves per SIMD the head kernel is compiled for: three (168 VGPRs, a few
// bytes of spill) measured faster than two without spills, also for the
// FP64 three-group variant (191 VGPRs at two waves: 8.7 -> 7.9 ms per head
// launch at 256^3 x 3 once multiply-adds fuse per expression) and for the
// smoothed one (140 bytes of spill at three: 6.9 against 7.5 ms at two).
template <typename R, int M>
constexpr int head_waves() { return 3; }

// V selects the method variant of the chemistry (V_SMOOTH: it starts from
// the radiation before injection and transport, io.sm, and takes their
// change as a rate; V_CASE_A: no on-the-spot approximation).
template <typename R, int M, int FUSE, int FLUX, int V>
__global__ __launch_bounds__(256, (head_waves<R, M>())) void k_head(KGrid g, const KChem *__restrict__ kp, double dt, R c, R kdx, const R *__restrict__ Nin,
                                              const R *__restrict__ Fin, ChemIO<R> io, const R *__restrict__ tab,
                                              int nf, int nth, QueueView q, int K, DevStats *__restrict__ st)
{
    const KChem &k = *kp;
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    const bool valid = i < (uint32_t)g.ncell;
    const size_t nc = g.ncell;
    constexpr bool SM = (V & V_SMOOTH) != 0;
    ChemState<V> s;
    CC cc{1.0, 0.0, 0.0, 0.0};
    bool done = true;
    unsigned fl = 0;
    double av[6] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    __shared__ unsigned s_hist[64];
    if (io.hist) hist_init(s_hist);
#pragma unroll
    for (int grp = 0; grp < CM; ++grp) {
        s.N[grp] = 0.0;
        s.fs[grp] = 1.0;
        if constexpr (SM) s.Nr[grp] = 0.0;
    }
    if (valid) {
        bool fin = true;
        if (FUSE) {
            // transport of every group; the flux goes straight to the
            // destination, where the chemistry rescales it at the end
            int ix, iy, iz;
            cell_coords(g, i, ix, iy, iz);
            const Nbr nb = neighbours(g, i, ix, iy, iz);
#pragma unroll
            for (int grp = 0; grp < M; ++grp) {
                double bout = 0.0;
                const U4<R> o = transport_cell<R, FLUX>(nb, i, nc, Nin + (size_t)grp * nc,
                                                        Fin + (size_t)3 * grp * nc, c, kdx, tab, nf, nth, bout, g,
                                                        grp);
                s.N[grp] = (double)o.n * io.ia3;
                av[grp] = (double)o.n;
                av[3 + grp] = bout;
                io.F[(size_t)(3 * grp) * nc + i] = o.fx;
                io.F[(size_t)(3 * grp + 1) * nc + i] = o.fy;
                io.F[(size_t)(3 * grp + 2) * nc + i] = o.fz;
                fin = fin && isfinite(o.fx) && isfinite(o.fy) && isfinite(o.fz);
            }
        } else {
#pragma unroll
            for (int grp = 0; grp < M; ++grp) {
                s.N[grp] = (double)io.N[(size_t)grp * nc + i] * io.ia3;
#pragma unroll
                for (int d = 0; d < 3; ++d) fin = fin && isfinite(io.F[(size_t)(3 * grp + d) * nc + i]);
            }
        }
        if constexpr (SM) {
            // N^t from the pre-step set, or for a source cell its value
            // before the injection; rate (N' - N^t)/dt (eq. smoothrate1)
            const int si = io.sm.map ? io.sm.map[i] : -1;
#pragma unroll
            for (int grp = 0; grp < M; ++grp) {
                const double nt = (si >= 0 ? io.sm.prev[(size_t)si * M + grp] : (double)io.sm.N[(size_t)grp * nc + i]) *
                                  io.ia3;
                s.Nr[grp] = (s.N[grp] - nt) / dt;
                s.N[grp] = nt;
#pragma unroll
                for (int d = 0; d < 3; ++d) fin = fin && isfinite(io.sm.F[(size_t)(3 * grp + d) * nc + i]);
            }
        }
        s.x = io.xHII[i];
        s.y2 = io.xHeII[i];
        s.y3 = io.xHeIII[i];
        cc = make_cc(k, io.nH[i] * io.ia3, io.T[i]);
        if (chem_init<CM, V>(k, dt, cc.Tiso, fin, s)) {
            done = false;
            for (int a = 0; a < K && !done; ++a) done = chem_attempt<CM, V, false, false>(k, k.rates, nullptr, cc, s, fl);
        } else {
            fl |= 2u;
        }
    }
    if (FUSE && io.acct) block_acct(io.acct, av);
    // wave-aggregated enqueue of the unfinished cells, by expected length of
    // their chain of substeps: cells that took many attempts in the previous
    // pass (the fronts move little in a step), then cells that accepted no
    // substep in their K attempts here (a state that changes fast), then the
    // rest.  The tail works the regions off in this order, so that the
    // longest chains start first instead of draining the tail at its end.
    const bool want = !done;
    const int cls = !want ? 3
                          : (io.prev_att && (io.prev_att[i] & ATT_MASK) >= TAIL_LONG_ATTEMPTS) ? 0
                                                                                                 : (s.acc == 0 ? 1 : 2);
    unsigned p = ~0u;
#pragma unroll
    for (int r = 0; r < 3; ++r) {
        const bool cand = want && p == ~0u && cls <= r;  // a full region passes its cells on
        const unsigned long long m = __ballot(cand);
        if (m) {
            const int leader = __ffsll((long long)m) - 1;
            unsigned base = 0;
            if (lane_id() == leader) base = atomicAdd(q.cnt[r], (unsigned)__popcll(m));
            base = __shfl(base, leader);
            if (cand) {
                const unsigned k = base + (unsigned)__popcll(m & ((1ull << lane_id()) - 1ull));
                if (k < q.rlen[r]) p = q.rbeg[r] + k;
            }
        }
    }
    bool queued = false;
    if (p != ~0u) {
        q_store(q, p, i, s, cc);
        queued = true;
    }
    if (want && !queued) {
        while (!done) done = chem_attempt<CM, V, true, false>(k, k.rates, nullptr, cc, s, fl);
    }
    unsigned long long a_acc = 0, a_att = 0;
    if (valid && !queued) {
        const double T = chem_finish<CM>(k, cc, s, fl);
        store_cell<R, M>(io, i, s, T);
        a_acc = (unsigned long long)s.acc;
        a_att = (unsigned long long)s.att;
        if (io.hist) hist_add(s_hist, s.acc);
    }
    if (io.hist) hist_flush(s_hist, io.hist);
    block_stats(st, a_acc, a_att, a_att, fl);
}

// Tail pass over the queue: persistent waves whose lanes each take a queued
// cell, run one attempt per loop trip (an attempt that fails the photon
// check repeats at once with the halved substep), and refill from the
// wave's reservation of queue positions as soon as their cell has filled
// dt_RT, so that a few slow cells do not hold whole waves of finished
// lanes.  Compiled for three waves per SIMD: the smoothed
// variants would otherwise take 176-178 VGPRs and run two (a few bytes of
// spill at three: 4.6 -> 4.0 ms per tail at 256^3 x 3).
template <typename R, int M, int V>
__global__ __launch_bounds__(CHEM_THREADS, CHEM_WAVES) void k_tail(const KChem *__restrict__ kp, ChemIO<R> io, QueueView q, DevStats *__restrict__ st)
{
    const KChem &k = *kp;
    __shared__ double rt[rate_table_len<V>()];
    rate_table_to_lds<V>(k.rates, rt);
    // the regions in order: longest expected chains first
    const unsigned n0 = min(*q.cnt[0], q.rlen[0]);
    const unsigned n1 = min(*q.cnt[1], q.rlen[1]);
    const unsigned n = n0 + n1 + min(*q.cnt[2], q.rlen[2]);
    ChemState<V> s;
    // the cell's destination fluxes, loaded with the cell (as in k_chem_all)
    constexpr bool PRE = (V & V_SMOOTH) == 0;
    R fpre[PRE ? 3 * M : 1];
    uint32_t cell = 0;
    CC cc{1.0, 0.0, 0.0, 0.0};
    bool active = false, exhausted = false;
    bool raised = false;
    unsigned rbase = 0, ravail = 0;  // positions this wave has reserved and not yet handed out
    unsigned fl = 0;
    unsigned a_acc = 0, a_att = 0, a_max = 0;  // of this lane's cells (32 bits outlast a lane's work)
    __shared__ unsigned s_hist[64];
    if (io.hist) hist_init(s_hist);
    while (true) {
        if (!exhausted) {
            bool first = false;
            const bool need = !active;
            const unsigned long long m = __ballot(need);
            if (m) {
                const unsigned nneed = (unsigned)__popcll(m);
                const unsigned r = (unsigned)__popcll(m & ((1ull << lane_id()) - 1ull));
                unsigned t;
                if (ravail >= nneed) {
                    t = rbase + r;
                    rbase += nneed;
                    ravail -= nneed;
                } else {
                    // what is left of the reservation goes first; a new one
                    // of at least TAIL_CHUNK positions covers the rest
                    const unsigned more = nneed - ravail;
                    const unsigned take = more > TAIL_CHUNK ? more : TAIL_CHUNK;
                    const int leader = __ffsll((long long)m) - 1;
                    unsigned base = 0;
                    if (lane_id() == leader) base = atomicAdd(q.head, take);
                    base = __shfl(base, leader);
                    t = r < ravail ? rbase + r : base + (r - ravail);
                    rbase = base + more;
                    ravail = take - more;
                }
                // positions only grow: past n there is nothing left for this wave
                if (rbase >= n) exhausted = true;
                if (need && t < n) {
                    const unsigned pos = t < n0 ? t : (t < n0 + n1 ? q.rbeg[1] + (t - n0) : q.rbeg[2] + (t - n0 - n1));
                    cell = q_load(k, q, pos, s, cc);
                    if constexpr (PRE) {
#pragma unroll
                        for (int j = 0; j < 3 * M; ++j) fpre[j] = io.F[(size_t)j * io.ncell + cell];
                    }
                    active = true;
                    first = t < n0;
                }
            }
            // a wave holding cells of the first region (the longest chains)
            // issues ahead of the others for the rest of its life
            if (!raised && __any(first)) {
                __builtin_amdgcn_s_setprio(3);
                raised = true;
            }
        }
        if (!__any(active)) break;
        if (active) {
            if (chem_attempt<CM, V>(k, k.rates, rt, cc, s, fl)) {
                const double T = chem_finish<CM>(k, cc, s, fl);
                if constexpr (PRE) store_cell_with<R, M>(io, cell, s, T, fpre);
                else store_cell<R, M>(io, cell, s, T);
                if (io.hist) hist_add(s_hist, s.acc);
                a_acc += (unsigned)s.acc;
                a_att += (unsigned)s.att;
                a_max = a_max > (unsigned)s.att ? a_max : (unsigned)s.att;
                active = false;
            }
        }
    }
    if (io.hist) hist_flush(s_hist, io.hist);
    block_stats(st, a_acc, a_att, a_max, fl);
}

static __global__ void k_zero_u32(unsigned *p, int n)
{
    for (int k = threadIdx.x; k < n; k += blockDim.x) p[k] = 0u;
}

// Before the one-pass chemistry, cells go to three lists (regions of the
// queue's cell array) that the pass takes before it sweeps over the rest:
//   0  the previous pass took at least TAIL_LONG_ATTEMPTS attempts, cold gas
//   1  the same, warm gas
//   2  the other cells of warm gas (above T_COLD_COOL)
// Long chains first, so that they do not start late and drain the chip at
// the end; warm and cold gas apart, so that the waves of cold gas skip the
// Boltzmann factors, which take more than half of an attempt's instructions
// and which one warm lane makes its whole wave execute (256^3 x 3 groups with
// 200 bubbles, every wave mixed: 650 VALU instructions per trip and wave
// where cold gas needs 300).  T null: the gas is one class (isothermal).
// Listed cells are marked ATT_LISTED; what a region has no room for stays in
// the sweep.  A block takes 4,096 cells, four consecutive ones per thread
// (one 4-byte word of counts; the array is padded to 256 bytes), and adds to
// each counter once.
constexpr int ORDER_THREADS = 1024;
static __global__ __launch_bounds__(ORDER_THREADS) void k_order(uint8_t *__restrict__ prev, const double *__restrict__ T,
                                                                size_t nc, QueueView q)
{
    const size_t w = (size_t)blockIdx.x * ORDER_THREADS + threadIdx.x;  // word index
    const size_t i0 = 4 * w;
    uint32_t o = 0;
    double Tc[4] = {0.0, 0.0, 0.0, 0.0};
    if (i0 < nc) {
        o = reinterpret_cast<const uint32_t *>(prev)[w];
        if (T) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                if (i0 + j < nc) Tc[j] = T[i0 + j];
        }
    }
    int cls[4];  // 0..2: the list, 3: none
    unsigned long long c = 0;  // the thread's cells per list, 20 bits each
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const bool lng = ((o >> (8 * j)) & ATT_MASK) >= (unsigned)TAIL_LONG_ATTEMPTS;
        const bool warm = Tc[j] > T_COLD_COOL;
        cls[j] = i0 + j >= nc ? 3 : (lng ? (warm ? 1 : 0) : (warm ? 2 : 3));
        if (cls[j] < 3) c += 1ull << (20 * cls[j]);
    }
    // exclusive sums over the wave, then over the block's waves
    unsigned long long ex = c;
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
        const unsigned long long u = __shfl_up(ex, d, 64);
        if (lane_id() >= d) ex += u;
    }
    __shared__ unsigned long long wsum[ORDER_THREADS / 64];
    __shared__ unsigned base[3];
    if (lane_id() == 63) wsum[threadIdx.x >> 6] = ex;
    __syncthreads();
    unsigned long long before = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < ORDER_THREADS / 64; ++k) {
        if (k < (int)(threadIdx.x >> 6)) before += wsum[k];
        tot += wsum[k];
    }
    if (threadIdx.x < 3) {
        const unsigned n = (unsigned)(tot >> (20 * threadIdx.x)) & 0xFFFFFu;
        if (n) base[threadIdx.x] = atomicAdd(q.cnt[threadIdx.x], n);
    }
    __syncthreads();
    ex = before + ex - c;
    uint32_t nw = 0;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        uint32_t b = (o >> (8 * j)) & ATT_MASK;
        if (cls[j] < 3) {
            const unsigned k = base[cls[j]] + ((unsigned)(ex >> (20 * cls[j])) & 0xFFFFFu);
            ex += 1ull << (20 * cls[j]);
            if (k < q.rlen[cls[j]]) {
                q.cell[q.rbeg[cls[j]] + k] = (int32_t)(i0 + j);
                b |= ATT_LISTED;
            }
        }
        nw |= b << (8 * j);
    }
    if (i0 < nc && nw != o) reinterpret_cast<uint32_t *>(prev)[w] = nw;
}

// The chemistry of every cell in one persistent launch (the pass after a
// separate transport): each lane takes a cell, runs its attempts one per
// loop trip (an attempt that fails the photon check repeats at once with the
// halved substep), writes it when it has filled dt_RT and takes the next,
// from its wave's reservation of positions.  Positions run over the lists of
// k_order (the waves of long chains issue ahead of the others), then over all
// cells in grid order, passing over the listed ones.  Every cell goes
// through the same attempt code as in the head and tail passes, so results
// are those of the two-pass chemistry bit for bit; what changes is that a
// lane whose cell is done no longer idles until its wave's other lanes are.
template <typename R, int M, int V>
__global__ __launch_bounds__(CHEM_THREADS, CHEM_WAVES) void k_chem_all(const KChem *__restrict__ kp, double dt,
                                                                            ChemIO<R> io, QueueView q,
                                                                            unsigned sweep_chunk,
                                                                            DevStats *__restrict__ st)
{
    const KChem &k = *kp;
    __shared__ double rt[rate_table_len<V>()];
    rate_table_to_lds<V>(k.rates, rt);
    constexpr bool SM = (V & V_SMOOTH) != 0;
    const size_t nc = io.ncell;
    // the lists of k_order: positions below n0 and n1 are long chains, below nl listed
    const unsigned n0 = io.prev_att ? min(*q.cnt[0], q.rlen[0]) : 0u;
    const unsigned n1 = n0 + (io.prev_att ? min(*q.cnt[1], q.rlen[1]) : 0u);
    const unsigned nl = n1 + (io.prev_att ? min(*q.cnt[2], q.rlen[2]) : 0u);
    const unsigned n = nl + (unsigned)nc;
    ChemState<V> s;
    // the cell's destination fluxes, loaded with the cell (not with smoothed
    // RT, which has two sets of them)
    constexpr bool PRE = !SM;
    R fpre[PRE ? 3 * M : 1];
    uint32_t cell = 0;
    CC cc{1.0, 0.0, 0.0, 0.0};
    bool active = false, exhausted = false, raised = false;
    uint8_t mark = 0;
    // positions this wave has reserved and not yet handed out: the first
    // wave's width without an atomic, dealt out block by block so that a small
    // grid's waves spread over all CUs; the shared counter starts after those
    const unsigned first0 = gridDim.x * (blockDim.x >> 6) * 64u;
    unsigned rbase = ((threadIdx.x >> 6) * gridDim.x + blockIdx.x) * 64u, ravail = 64u;
    unsigned fl = 0, cfl = 0;        // flags of the lane, flags of its current cell
    unsigned a_acc = 0, a_att = 0, a_max = 0;  // of this lane's cells (32 bits outlast a lane's work)
    __shared__ unsigned s_hist[64];
    if (io.hist) hist_init(s_hist);
    // the cell's state as the head pass loads it, without the check of its
    // fluxes; returns chem_init's verdict
    auto load = [&](uint32_t c, bool fin) -> bool {
        const size_t i = c;
#pragma unroll
        for (int grp = 0; grp < CM; ++grp) {
            s.N[grp] = 0.0;
            s.fs[grp] = 1.0;
            if constexpr (SM) s.Nr[grp] = 0.0;
        }
#pragma unroll
        for (int grp = 0; grp < M; ++grp) s.N[grp] = (double)io.N[(size_t)grp * nc + i] * io.ia3;
        if constexpr (SM) {
            const int si = io.sm.map ? io.sm.map[i] : -1;
#pragma unroll
            for (int grp = 0; grp < M; ++grp) {
                const double nt =
                    (si >= 0 ? io.sm.prev[(size_t)si * M + grp] : (double)io.sm.N[(size_t)grp * nc + i]) * io.ia3;
                s.Nr[grp] = (s.N[grp] - nt) / dt;
                s.N[grp] = nt;
#pragma unroll
                for (int d = 0; d < 3; ++d) fin = fin && isfinite(io.sm.F[(size_t)(3 * grp + d) * nc + i]);
            }
        }
        s.x = io.xHII[i];
        s.y2 = io.xHeII[i];
        s.y3 = io.xHeIII[i];
        cc = make_cc(k, io.nH[i] * io.ia3, io.T[i]);
        // the fluxes are needed only when the cell is written: loaded now,
        // they arrive while the attempts run instead of stalling the wave
        // at the write
        if constexpr (PRE) {
#pragma unroll
            for (int j = 0; j < 3 * M; ++j) fpre[j] = io.F[(size_t)j * nc + i];
        }
        return chem_init<CM, V>(k, dt, cc.Tiso, fin, s);
    };
    // write a cell whose chemistry has ended.  Its fluxes are checked here,
    // where they are used: a non-finite one means the cell is written back
    // as loaded (what the head pass does when it finds one before the
    // chemistry), and the flags of the discarded attempts are dropped
    auto finish = [&]() {
        bool fin = true;
#pragma unroll
        for (int j = 0; j < 3 * M; ++j) fin = fin && isfinite(PRE ? fpre[j] : io.F[(size_t)j * nc + cell]);
        if (!fin) {
            load(cell, false);
            cfl = 2u;
        }
        fl |= cfl;
        const double T = chem_finish<CM>(k, cc, s, fl);
        if constexpr (PRE) store_cell_with<R, M>(io, cell, s, T, fpre, mark);
        else store_cell<R, M>(io, cell, s, T, mark);
        if (io.hist) hist_add(s_hist, s.acc);
        a_acc += (unsigned)s.acc;
        a_att += (unsigned)s.att;
        a_max = a_max > (unsigned)s.att ? a_max : (unsigned)s.att;
    };
    while (true) {
        if (!exhausted) {
            bool first = false;
            const bool need = !active;
            const unsigned long long m = __ballot(need);
            if (m) {
                const unsigned nneed = (unsigned)__popcll(m);
                const unsigned r = (unsigned)__popcll(m & ((1ull << lane_id()) - 1ull));
                unsigned t;
                if (ravail >= nneed) {
                    t = rbase + r;
                    rbase += nneed;
                    ravail -= nneed;
                } else {
                    // one wave's width at a time among the long chains, so
                    // that a wave does not hold a second set of them; more
                    // in the sweep (sweep_chunk), where each reservation is
                    // an atomic on the one counter every wave shares
                    const unsigned more = nneed - ravail;
                    const unsigned chunk = rbase < n1 ? TAIL_CHUNK : sweep_chunk;
                    const unsigned take = more > chunk ? more : chunk;
                    const int leader = __ffsll((long long)m) - 1;
                    unsigned base = 0;
                    if (lane_id() == leader) base = first0 + atomicAdd(q.head, take);
                    base = __shfl(base, leader);
                    t = r < ravail ? rbase + r : base + (r - ravail);
                    rbase = base + more;
                    ravail = take - more;
                }
                if (rbase >= n) exhausted = true;
                if (need && t < n) {
                    bool take = true;
                    if (t < nl) {
                        cell = (uint32_t)q.cell[t < n0 ? t : (t < n1 ? q.rbeg[1] + (t - n0) : q.rbeg[2] + (t - n1))];
                        mark = ATT_LISTED;
                        first = t < n1;
                    } else {
                        cell = t - nl;
                        mark = 0;
                        take = !io.prev_att || !(io.prev_att[cell] & ATT_LISTED);
                    }
                    if (take) {
                        cfl = 0;
                        if (load(cell, true)) {
                            active = true;
                        } else {
                            // a non-finite input: the cell is written back as loaded
                            cfl = 2u;
                            finish();
                        }
                    }
                }
            }
            if (!raised && __any(first)) {
                __builtin_amdgcn_s_setprio(3);
                raised = true;
            }
        }
        if (!__any(active)) {
            if (exhausted) break;
            continue;
        }
        if (active && chem_attempt<CM, V>(k, k.rates, rt, cc, s, cfl)) {
            finish();
            active = false;
        }
    }
    if (io.hist) hist_flush(s_hist, io.hist);
    block_stats(st, a_acc, a_att, a_max, fl);
}


// Positions a wave reserves at a time in the sweep: a quarter of a wave's
// share of the grid, between one wave's width and CHEM_SWEEP_CHUNK (on a
// small grid large reservations would leave the work to a few waves).
static unsigned chem_sweep_chunk(size_t ncell, unsigned waves)
{
    const size_t share = ncell / waves / 4;
    const size_t c = share < TAIL_CHUNK ? TAIL_CHUNK : (share > CHEM_SWEEP_CHUNK ? CHEM_SWEEP_CHUNK : share);
    return (unsigned)c;
}

// workgroups of a persistent chemistry kernel: one per CU, and no more than
// there are wave's widths of cells
static unsigned chem_blocks(size_t ncell)
{
    const size_t w = (ncell + 63) / 64;
    return (unsigned)(w < (size_t)CHEM_BLOCKS ? (w ? w : 1) : CHEM_BLOCKS);
}

template <typename R, int M, int V>
static void launch_M(ChemPass pass, const ChemCall<R> &a, hipStream_t s)
{
    const dim3 hb((unsigned)((a.g.ncell + 255) / 256)), pb(chem_blocks(a.g.ncell));
    if (pass != CHEM_TAIL) hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, s, a.q.count, 65);
    switch (pass) {
    case CHEM_HEAD:
        hipLaunchKernelGGL((k_head<R, M, 0, 0, V>), hb, dim3(256), 0, s, a.g, a.dk, a.dt, R(0), R(0), (const R *)nullptr,
                           (const R *)nullptr, a.io, (const R *)nullptr, 0, 0, a.q, a.K, a.st);
        break;
    case CHEM_FUSED_GLF:
        hipLaunchKernelGGL((k_head<R, M, 1, 0, V>), hb, dim3(256), 0, s, a.g, a.dk, a.dt, a.c, a.kdx, a.Nin, a.Fin, a.io,
                           a.tab, a.nf, a.nth, a.q, a.K, a.st);
        break;
    case CHEM_FUSED_HLL:
        hipLaunchKernelGGL((k_head<R, M, 1, 1, V>), hb, dim3(256), 0, s, a.g, a.dk, a.dt, a.c, a.kdx, a.Nin, a.Fin, a.io,
                           a.tab, a.nf, a.nth, a.q, a.K, a.st);
        break;
    case CHEM_TAIL:
        hipLaunchKernelGGL((k_tail<R, M, V>), pb, dim3(CHEM_THREADS), 0, s, a.dk, a.io, a.q, a.st);
        break;
    case CHEM_ALL:
        // queue counters reset, the lists, then the persistent kernel
        if (a.io.prev_att && a.io.ncell > 0)
            hipLaunchKernelGGL(k_order, dim3((unsigned)((a.io.ncell + 4 * ORDER_THREADS - 1) / (4 * ORDER_THREADS))),
                               dim3(ORDER_THREADS), 0, s, a.io.prev_att, a.isothermal ? nullptr : a.io.T, a.io.ncell,
                               a.q);
        hipLaunchKernelGGL((k_chem_all<R, M, V>), pb, dim3(CHEM_THREADS), 0, s, a.dk, a.dt, a.io, a.q,
                           chem_sweep_chunk(a.io.ncell, pb.x * (CHEM_THREADS / 64)), a.st);
        break;
    }
}

template <typename R, int V>
void launch_chem_variant(ChemPass pass, int M, const ChemCall<R> &a, hipStream_t s)
{
    if (M == 1) launch_M<R, 1, V>(pass, a, s);
    else if (M == 2) launch_M<R, 2, V>(pass, a, s);
    else launch_M<R, 3, V>(pass, a, s);
}
template void launch_chem_variant<RT_CHEM_R, RT_CHEM_V>(ChemPass, int, const ChemCall<RT_CHEM_R> &, hipStream_t);

}  // namespace rtm1

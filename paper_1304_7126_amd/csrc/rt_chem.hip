// rt_chem.hip -- the thermochemistry kernels of the grid (App. A): the
// persistent one-pass kernel, and the head and tail passes.  Compiled once
// per radiation type RT_CHEM_R (float, double) and method variant RT_CHEM_V
// (0..3: V_SMOOTH, V_CASE_A), which build in parallel.
#include "rt_chem.h"

namespace rtm1 {

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
// Waves per SIMD the head kernel is compiled for: three (168 VGPRs, of which
// 20 to 30 spill, with the transport fused in FP64 x 3 groups 85, smoothed 120)
// are faster than two without spills (185 to 210 VGPRs).  us per step with the
// fused transport, three / two waves: 96^3 x 3 490 / 540, FP64 612 / 634,
// smoothed 550 / 571, without OTSA 560 / 600; 160^3 1,305 / 1,525, FP64 1,880 /
// 1,948; 900 x 128 x 64 1,830 / 2,240.  With two passes after a separate
// transport both take the same time.
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
            fl |= chem_refused(k, s);
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
                          : (io.prev_att && io.prev_att[i] >= TAIL_LONG_ATTEMPTS) ? 0
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
// lanes.
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
    unsigned long long a_acc = 0, a_att = 0;  // of this lane's cells (INT_MAX attempts each at most, any number of cells)
    unsigned a_max = 0;
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
                a_acc += (unsigned long long)s.acc;
                a_att += (unsigned long long)s.att;
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

// The order in which the one-pass chemistry takes the cells.  Each block
// sorts the ORDER_CELLS cells of its piece of the grid by what their attempts
// will cost and how many they will be,
//   the temperature, by the thresholds above which an attempt evaluates
//   Boltzmann factors (a lane above one makes its whole wave execute them:
//   650 VALU instructions per trip where cold gas needs 300),
//   then the attempts of the previous pass (the state moves little in a step),
// so that the lanes of a wave run the same code and end together, and their
// next cells are neighbours again: the loads and stores of 64 cells then
// take one set of memory instructions instead of three or four.  Sorted
// pieces, not a sorted grid: one pass over T, and neighbours stay together.
// Measured with the slabs of k_chem_all, against three lists over the whole
// grid (us per step): 97 x 61 x 45 273 -> 222, 64^3 355 -> 304, shadowed 128^3
// 810 -> 750, smoothed 128^3 558 -> 520, 256^3 x 3 3,980 -> 3,765; pieces of
// 2,048 and 8,192 cells and half the keys are within 2% of that.  Sorted
// pieces without the slabs: 256^3 x 3 4,015 and 3 times the bytes fetched.
// Cells that took at least TAIL_LONG_ATTEMPTS go to two lists (cold gas in
// q.acc, warm gas in q.att) that the pass takes first, so that the longest
// chains do not start late and drain the chip at the end; -1 fills their
// places.  T null: the gas is one class (isothermal).
// Of a state without counts the warm cells go to the lists where they are few
// in their piece: next to sources they have the long chains (smoothed dense
// 128^3, first pass 5.2 ms, 8.0 with none listed).  A piece that is mostly warm
// is ionised gas at rest; taken through the lists, all its cells pass one
// counter 64 at a time (first step of a 256^3 x 3 state warm throughout 4,715 us
// with all listed, 2,290 without; 20% of the cells warm at random 29.5 ms
// with a bound of 1/2, 1/4 or 1/16, ionised bubbles 3.35 / 3.35 / 3.25).
constexpr int ORDER_THREADS = 512, ORDER_CELLS = 4096, ORDER_PER = ORDER_CELLS / ORDER_THREADS;
constexpr int ORDER_KEYS = 32;
constexpr unsigned ORDER_FEW = 4;  // few: at most a quarter of the piece
static __device__ __forceinline__ int order_bin(unsigned att)
{
    return att <= 4u ? (att ? (int)att - 1 : 0) : att <= 6u ? 4 : att <= 8u ? 5 : att <= 12u ? 6 : 7;
}
static __global__ __launch_bounds__(ORDER_THREADS) void k_order(const uint8_t *__restrict__ prev,
                                                                const double *__restrict__ T, size_t nc, QueueView q)
{
    // per key: its cells, then where its run starts; the last two: the lists
    __shared__ unsigned cnt[ORDER_KEYS + 2], beg[ORDER_KEYS + 2];
    __shared__ unsigned nwarm[ORDER_THREADS / 64];  // per wave: warm cells without a count
    __shared__ uint16_t place[ORDER_CELLS];
    const size_t c0 = (size_t)blockIdx.x * ORDER_CELLS;
    const unsigned nhere = nc - c0 < (size_t)ORDER_CELLS ? (unsigned)(nc - c0) : (unsigned)ORDER_CELLS;
    if (threadIdx.x < ORDER_KEYS + 2) cnt[threadIdx.x] = 0u;
    if (blockIdx.x == 0 && threadIdx.x < CHEM_XCDS) q.slab[threadIdx.x * QUEUE_SLAB_STRIDE] = 0u;
    unsigned att[ORDER_PER];
    double Tc[ORDER_PER];
#pragma unroll
    for (int j = 0; j < ORDER_PER; ++j) {
        const unsigned l = threadIdx.x + j * ORDER_THREADS;
        att[j] = l < nhere ? (unsigned)prev[c0 + l] : 0u;
        Tc[j] = T && l < nhere ? T[c0 + l] : 0.0;
    }
    unsigned u = 0;
#pragma unroll
    for (int j = 0; j < ORDER_PER; ++j)
        u += (unsigned)__popcll(
            __ballot(threadIdx.x + j * ORDER_THREADS < nhere && att[j] == 0u && Tc[j] > T_COLD_COOL));
    if (lane_id() == 0) nwarm[threadIdx.x >> 6] = u;
    __syncthreads();
    u = 0;
#pragma unroll
    for (int j = 0; j < ORDER_THREADS / 64; ++j) u += nwarm[j];
    const bool few = ORDER_FEW * u <= nhere;
    int key[ORDER_PER];
    unsigned rank[ORDER_PER];
#pragma unroll
    for (int j = 0; j < ORDER_PER; ++j) {
        const int cls = !(Tc[j] > T_COLD_COOL) ? 0 : Tc[j] <= T_COLD_HI ? 1 : Tc[j] <= T_COLD_HEII ? 2 : 3;
        // (no count yet, a state just set: warm gas may have long chains)
        const bool lng = att[j] >= (unsigned)TAIL_LONG_ATTEMPTS || (few && att[j] == 0u && cls);
        key[j] = lng ? ORDER_KEYS + (cls ? 1 : 0) : 8 * cls + order_bin(att[j]);
        rank[j] = threadIdx.x + j * ORDER_THREADS < nhere ? atomicAdd(&cnt[key[j]], 1u) : 0u;
    }
    __syncthreads();
    if (threadIdx.x < ORDER_KEYS) {
        unsigned s = cnt[threadIdx.x];
#pragma unroll
        for (int d = 1; d < ORDER_KEYS; d <<= 1) {
            const unsigned u = __shfl_up(s, d, 64);
            if ((int)threadIdx.x >= d) s += u;
        }
        beg[threadIdx.x] = s - cnt[threadIdx.x];
    } else if (threadIdx.x < ORDER_KEYS + 2) {
        const unsigned n = cnt[threadIdx.x];
        beg[threadIdx.x] = n ? atomicAdd(q.cnt[threadIdx.x - ORDER_KEYS], n) : 0u;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < ORDER_PER; ++j) {
        const unsigned l = threadIdx.x + j * ORDER_THREADS;
        if (l >= nhere) continue;
        const unsigned p = beg[key[j]] + rank[j];
        if (key[j] < ORDER_KEYS) place[p] = (uint16_t)l;
        else (key[j] == ORDER_KEYS ? q.acc : q.att)[p] = (int32_t)(c0 + l);
    }
    __syncthreads();
    const unsigned n = beg[ORDER_KEYS - 1] + cnt[ORDER_KEYS - 1];
#pragma unroll
    for (int j = 0; j < ORDER_PER; ++j) {
        const unsigned l = threadIdx.x + j * ORDER_THREADS;
        if (l < nhere) q.cell[c0 + l] = l < n ? (int32_t)(c0 + place[l]) : -1;
    }
}

// The chemistry of every cell in one persistent launch (the pass after a
// separate transport): each lane takes a cell, runs its attempts one per
// loop trip (an attempt that fails the photon check repeats at once with the
// halved substep), writes it when it has filled dt_RT and takes the next,
// from its wave's reservation of positions.  With ordered, positions run over
// the lists of k_order (the waves of long chains issue ahead of the others),
// then over its sorted pieces; otherwise over the grid.  Every cell goes
// through the same attempt code as in the head and tail passes, so results
// are those of the two-pass chemistry bit for bit; what changes is that a
// lane whose cell is done no longer idles until its wave's other lanes are.
template <typename R, int M, int V>
__global__ __launch_bounds__(CHEM_THREADS, CHEM_WAVES) void k_chem_all(const KChem *__restrict__ kp, double dt,
                                                                            ChemIO<R> io, QueueView q,
                                                                            bool ordered, unsigned slabs, unsigned piece,
                                                                            unsigned chunk,
                                                                            DevStats *__restrict__ st)
{
    const KChem &k = *kp;
    __shared__ double rt[rate_table_len<V>()];
    rate_table_to_lds<V>(k.rates, rt);
    constexpr bool SM = (V & V_SMOOTH) != 0;
    const size_t nc = io.ncell;
    // positions below n0 and n1: the lists of long chains
    const unsigned n0 = ordered ? *q.cnt[0] : 0u;
    const unsigned n1 = n0 + (ordered ? *q.cnt[1] : 0u);
    ChemState<V> s;
    // the cell's destination fluxes, loaded with the cell (not with smoothed
    // RT, which has two sets of them)
    constexpr bool PRE = !SM;
    R fpre[PRE ? 3 * M : 1];
    uint32_t cell = 0;
    CC cc{1.0, 0.0, 0.0, 10.0};
    bool active = false, exhausted = false, raised = false;
    // Positions this wave has reserved and not yet handed out: below n1 the
    // lists, from there the cells.  A wave takes its share of the lists, then
    // the cells of its XCD's slab (every eighth piece of the grid; workgroup b
    // is on XCD b % 8), so that the lines of a piece are read by one L2 only,
    // then what is left of the other slabs.  The first wave's width of each
    // needs no atomic, and is dealt out block by block so that a small grid's
    // waves spread over all CUs.
    const unsigned waves = blockDim.x >> 6, wave = threadIdx.x >> 6;
    const unsigned first0 = gridDim.x * waves * 64u;
    const unsigned npiece = ((unsigned)nc + piece - 1u) / piece;
    unsigned slab = blockIdx.x % slabs, left = slabs;
    unsigned rbase = (wave * gridDim.x + blockIdx.x) * 64u;
    unsigned ravail = rbase < n1 ? min(64u, n1 - rbase) : 0u;
    bool lists = n1 > first0, own = true;
    auto reserve = [&]() {
        ravail = 0u;
        if (lists) {
            unsigned at = 0;
            if (lane_id() == 0) at = atomicAdd(q.head, 64u);
            at = first0 + (unsigned)__builtin_amdgcn_readfirstlane(at);
            if (at < n1) {
                rbase = at;
                ravail = min(64u, n1 - at);
                return;
            }
            lists = false;
        }
        while (!exhausted) {
            // positions in the slab: the first widths of its waves, then by its counter
            const unsigned nb = (gridDim.x - slab + slabs - 1u) / slabs;
            unsigned at = nb * waves * 64u, take = 64u;
            if (own) {
                own = false;
                at = (wave * nb + blockIdx.x / slabs) * 64u;
            } else if (at / piece * slabs + slab < npiece) {
                unsigned got = 0;
                if (lane_id() == 0) got = atomicAdd(q.slab + slab * QUEUE_SLAB_STRIDE, chunk);
                at += (unsigned)__builtin_amdgcn_readfirstlane(got);
                take = chunk;
            }
            const unsigned pc = at / piece * slabs + slab;
            if (pc < npiece) {
                rbase = n1 + pc * piece + at % piece;
                ravail = take;
                return;
            }
            slab = (slab + 1u) % slabs;
            exhausted = --left == 0u;
        }
    };
    unsigned fl = 0, cfl = 0;        // flags of the lane, flags of its current cell
    unsigned long long a_acc = 0, a_att = 0;  // of this lane's cells (INT_MAX attempts each at most, any number of cells)
    unsigned a_max = 0;
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
        if constexpr (PRE) store_cell_with<R, M>(io, cell, s, T, fpre);
        else store_cell<R, M>(io, cell, s, T);
        if (io.hist) hist_add(s_hist, s.acc);
        a_acc += (unsigned long long)s.acc;
        a_att += (unsigned long long)s.att;
        a_max = a_max > (unsigned)s.att ? a_max : (unsigned)s.att;
    };
    // what a lane without a cell holds: an attempt on it ends at the photon
    // stage's cap, in cold gas
    auto idle = [&]() {
        s.att = k.max_att32;
        s.x = 0.5;
        s.y2 = s.y3 = 0.25;
        s.Tmu = 10.0;
    };
    idle();
    while (true) {
        if (!exhausted) {
            bool first = false;
            const bool need = !active;
            const unsigned long long m = __ballot(need);
            if (m) {
                const unsigned nneed = (unsigned)__popcll(m);
                const unsigned r = (unsigned)__popcll(m & ((1ull << lane_id()) - 1ull));
                unsigned t = rbase + r;
                bool got = need && r < ravail;
                if (ravail >= nneed) {
                    rbase += nneed;
                    ravail -= nneed;
                } else {
                    // what is left of the reservation goes first
                    const unsigned had = ravail, more = nneed - ravail;
                    reserve();
                    if (need && r >= had && r - had < ravail) {
                        t = rbase + (r - had);
                        got = true;
                    }
                    const unsigned used = min(more, ravail);
                    rbase += used;
                    ravail -= used;
                }
                got = got && t < n1 + (unsigned)nc;
                if (got) {
                    int32_t c = (int32_t)(t - n1);
                    if (ordered) {
                        c = t < n0 ? q.acc[t] : t < n1 ? q.att[t - n0] : q.cell[t - n1];
                        asm volatile("" : "+v"(c));  // (the wait for it: here, not in both branches' wake)
                        first = t < n1;
                    }
                    if (c != -1 || !ordered) {
                        cell = (uint32_t)c;
                        cfl = 0;
                        if (load(cell, true)) {
                            active = true;
                        } else {
                            // the cell is written back as loaded
                            cfl = chem_refused(k, s);
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
        // every lane attempts (an exec mask around it would copy the state)
        const bool done = chem_attempt<CM, V>(k, k.rates, rt, cc, s, cfl);
        if (active && done) {
            finish();
            active = false;
        }
        if (!active) idle();
    }
    if (io.hist) hist_flush(s_hist, io.hist);
    block_stats(st, a_acc, a_att, a_max, fl);
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
    // The one-pass chemistry orders the cells where there are more of them
    // than lanes (and scratch for it): with at most one cell per lane nothing
    // is refilled and the order only costs its launch (us per step, ordered /
    // not: 16^3 91.5 / 82.3, isothermal 32^3 65 / 61, 97 x 61 x 45 222 / 255,
    // 64^3 304 / 320).
    const bool more = a.io.ncell > (size_t)CHEM_BLOCKS * CHEM_THREADS;
    const bool ordered = more && a.io.prev_att && (size_t)a.q.stride >= a.io.ncell;
    const unsigned slabs = ordered ? CHEM_XCDS : 1u;
    // without the order: one counter for every wave, so more at a time
    const unsigned chunk = more && !ordered ? CHEM_SWEEP_CHUNK : 64u;
    QueueView qa = a.q;
    if (!ordered) qa.slab = a.q.head;
    // (with at most one cell per lane the one pass hands out its first widths
    // only and uses no counter: 4.5 us of a 16^3 step's 63)
    if (pass != CHEM_TAIL && (more || pass != CHEM_ALL))
        hipLaunchKernelGGL(k_zero_u32, dim3(1), dim3(64), 0, s, a.q.count, 65);
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
        // the order (where the scratch has room for it), then the persistent kernel
        if (ordered)
            hipLaunchKernelGGL(k_order, dim3((unsigned)((a.io.ncell + ORDER_CELLS - 1) / ORDER_CELLS)),
                               dim3(ORDER_THREADS), 0, s, a.io.prev_att, a.isothermal ? nullptr : a.io.T, a.io.ncell,
                               qa);
        hipLaunchKernelGGL((k_chem_all<R, M, V>), pb, dim3(CHEM_THREADS), 0, s, a.dk, a.dt, a.io, qa, ordered, slabs,
                           ordered ? (unsigned)ORDER_CELLS : chunk, chunk, a.st);
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

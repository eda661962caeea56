// rt_chem.h -- what the chemistry kernels (rt_chem.hip, one build per
// radiation type and method variant) and their dispatch share.
#pragma once
#include "rt_cell.h"

namespace rtm1 {

// Workgroups of the persistent chemistry kernels hold the rate table in LDS
// (75 KB, without OTSA 113 KB): one workgroup per CU, of two waves per SIMD.
// An attempt holds about 210 registers; at three waves per SIMD (168) 20 to
// 50 of them spill inside the subcycling loop (256^3 x 3 groups, 200 sources:
// 4.43 ms per step against 3.93 at two).
#ifndef RT_CHEM_WAVES
#define RT_CHEM_WAVES 2
#endif
constexpr int CHEM_WAVES = RT_CHEM_WAVES;
constexpr int CHEM_THREADS = CHEM_WAVES * 256;
constexpr int CHEM_BLOCKS = 256;
constexpr unsigned CHEM_XCDS = 8;

enum ChemPass { CHEM_HEAD, CHEM_FUSED_GLF, CHEM_FUSED_HLL, CHEM_TAIL, CHEM_ALL };

template <typename R>
struct ChemCall {
    KGrid g;
    const KChem *dk;
    double dt;
    R c, kdx;            // fused passes: the transport's light speed and dt/dx
    const R *Nin, *Fin;  // fused passes: the source set
    ChemIO<R> io;
    const R *tab;
    int nf, nth;
    QueueView q;
    int K;
    DevStats *st;
    bool isothermal;
};

template <typename R, int V>
void launch_chem_variant(ChemPass pass, int M, const ChemCall<R> &a, hipStream_t s);

}  // namespace rtm1

// Internal interface of the three-dimensional march (host launch code and
// kernels).
#pragma once

#include "tsq_internal.h"

namespace tsq {

// Kernel arguments of one pass of the three-dimensional march (one step per
// pass): mesh (nz, ny, nx), tiles of an x-strip x a slab of row pairs x a
// segment of plane pairs, and the rotation coefficients per axis.
template <class R>
struct March3Args {
    const void* src;
    void* dst;
    const void* ptab;
    int nx, ny, nz;
    int strip_sites, slab_pairs, seg_pairs;  // stored x-sites, row pairs, plane pairs per tile
    int nstrips, nslabs, nsegs;
    int strip_cols, pack_lanes;  // slab march: see SlabColumns
    R o1s[3], o1d[3];  // odd factors opening the pass (tau = dt/2 first pass, else dt), x y z
    R ehs[3], ehd[3];  // even factors and the closing odd factors, tau = dt/2, x y z
    // Slab march (tangent form, see MarchArgs): odd factors opening the
    // pass (x: s', d' of the delta form), tangents at dt and dt/2, closing odd x.
    R o1x[2], o1t[3], t2[3], t1[3], c1x[2];
    R table_unit;  // slab march, complex64: 1 per fixed-point unit of a table entry
};

constexpr int kWaves3 = 8;  // wavefronts per block of the 3D march (one row pair each)

struct Pass3Desc {
    const void* src;
    void* dst;
    const void* ptab;
    int nx, ny, nz;
    bool first;           // opening odd factors for dt/2 (else dt)
    bool close;           // a closing pass: only the final odd factors, dt/2
    int seg_pairs;        // plane pairs per tile
    int stages = 1, rp = 1;  // slab march
    Coef64 oh[3], o2[3];  // tau = dt/2 and tau = dt, per axis
};

// The slab march: one or two steps (d.stages) or, close, one step and the closing
// odd factors (two stages) in one pass, d.rp row pairs per wavefront.
hipError_t launch_slab(int dtype, const Pass3Desc& d, hipStream_t s);
// The closing odd factors alone, src to dst or in place.
hipError_t launch_close3(int dtype, const Pass3Desc& d, hipStream_t s);
// Bytes of a plane the slab march addresses with 32-bit offsets.
constexpr long long kMaxSlabPlane = 0x7fffffffLL;
// Stored x-sites and row pairs per block of the slab march.
constexpr int slab_strip(int stages) { return (kWaveSize - 2 * stages) * 2; }
constexpr int slab_pairs(int stages, int rp) { return kWaves3 * rp - 2 * stages; }
// Columns (blocks side by side) of the slab march on a plane: full strips x slabs,
// then the strip left over, whose few lanes (its sites and halo) serve several
// slabs in one block: `pack` lane groups of `pack_lanes`, a slab each.  A block of
// a narrow strip takes as long as one of a full strip, so this saves the blocks that
// a ragged width leaves mostly idle: 512^3 in complex64 has 93 columns instead of 110.
// us per step before and now, complex64 512^3 477 and 421, 128^3 17.2 and 13.8, 250 x
// 180 x 90 28.0 and 20.3, 192^3 (a rest of 68, one slab a block) 32.8 and 32.4;
// complex128 512^3 1164 and 1149, 128^3 31.0 and 23.7, 620 x 240 x 128 186 and 166.
struct SlabColumns {
    int full_strips, pack_lanes, pack, nslabs;
    long long strip_cols, columns;  // columns of full strips, and all
};
inline SlabColumns slab_columns(int nx, int ny, int stages, int rp) {
    const int strip = slab_strip(stages), slab = slab_pairs(stages, rp), rest = nx % strip;
    SlabColumns g{nx / strip, kWaveSize, 1, (ny / 2 + slab - 1) / slab, 0, 0};
    g.strip_cols = g.columns = (long long)g.full_strips * g.nslabs;
    if (rest) {
        g.pack_lanes = rest / 2 + 2 * stages;
        g.pack = kWaveSize / g.pack_lanes;
        g.columns += (g.nslabs + g.pack - 1) / g.pack;
    }
    return g;
}
// Plane pairs per tile of the slab march: the blocks go in rounds of one per compute
// unit, each marching a tile's Q pairs and its halo (a pair per stage and side, half of
// them without the second stage), and every tile reads its halo: the segment count with
// the least sum of the two, in pairs per unit.  At 512^3 complex64 two segments (186 tiles
// on 256 units).  Segment counts that give the same Q are passed over, and the search
// ends where no larger count can win: a few hundred counts for the longest mesh
// (2 x 2 x 2^29) instead of its 2^28, which took 2.9 s of every call.
long long slab_segment_pairs(long long columns, long long pairs, int stages, long long cus);
// log of the squared modulus a step's tangent-form factors multiply a site by.
template <class R>
double step3_log_sec2(const Coef64* oh, const Coef64* o2) {
    double L = 0.0;
    for (int ax = 0; ax < 3; ++ax)
        L += log_sec2(tangent<R>(o2[ax])) + 2.0 * log_sec2(tangent<R>(oh[ax]));
    return L;
}
// The modulus of the table's entries, exp(-step3_log_sec2 / 2), in two parts: one
// double's rounding of it would scale every site alike at every step (600 steps of 0.1
// rad a step and axis in complex128: a norm off by 4.7e-14, where the rounding of the
// entries themselves leaves 4e-16).
template <class R>
void slab_table_scale(const Coef64* oh, const Coef64* o2, TableScale& sc) {
    long double g2 = 1.0L;
    for (int ax = 0; ax < 3; ++ax) {
        const long double t2 = tangent<R>(o2[ax]), t1 = tangent<R>(oh[ax]);
        g2 *= (1.0L + t2 * t2) * (1.0L + t1 * t1) * (1.0L + t1 * t1);
    }
    const long double g = 1.0L / sqrtl(g2);
    sc.g = (double)g;
    sc.g_lo = (double)(g - sc.g);
}
// Fixed-point units per 1 of a complex64 table whose entries have the modulus
// g = exp(-L/2): the power of two that takes g to [2^30, 2^31), so an entry keeps 2^-31
// of itself at any angle, as one of modulus 1 does at 2^30 (at 2^30 for all, entries
// lose up to 3.8 bits near 1 rad a step, the same at every step).
inline double slab_table_unit(double L) {
    const double g = std::exp(-0.5 * L);
    int e = 30 - std::ilogb(g);
    if (std::ldexp(g, e) > 2147483647.0) --e;
    return std::ldexp(1.0, e);
}
hipError_t launch_pass3(int dtype, const Pass3Desc& d, hipStream_t s);
hipError_t launch_observables3(int dtype, const void* psi, const double* V, int nx, int ny, int nz,
                               double Jx, double Jy, double Jz, double eps0, double* partial,
                               int nblocks, double* result, hipStream_t s);

}  // namespace tsq

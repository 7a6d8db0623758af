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
    R o1s[3], o1d[3];  // odd factors opening the pass (tau = dt/2 first pass, else dt), x y z
    R ehs[3], ehd[3];  // even factors and the closing odd factors, tau = dt/2, x y z
    // Slab march (tangent form, see MarchArgs): odd factors opening the
    // pass (x: s', d' of the delta form), tangents at dt and dt/2, closing odd x.
    R o1x[2], o1t[3], t2[3], t1[3], c1x[2];
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
// log of the squared modulus a step's tangent-form factors multiply a site by.
template <class R>
double step3_log_sec2(const Coef64* oh, const Coef64* o2) {
    double L = 0.0;
    for (int ax = 0; ax < 3; ++ax)
        L += log_sec2(tangent<R>(o2[ax])) + 2.0 * log_sec2(tangent<R>(oh[ax]));
    return L;
}
hipError_t launch_pass3(int dtype, const Pass3Desc& d, hipStream_t s);
hipError_t launch_observables3(int dtype, const void* psi, const double* V, int nx, int ny, int nz,
                               double Jx, double Jy, double Jz, double eps0, double* partial,
                               int nblocks, double* result, hipStream_t s);

}  // namespace tsq

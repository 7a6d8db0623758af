// Tile kernels of the second-order Trotter-Suzuki step for small 2D meshes
// (Wittek & Cucchietti, Sec. 2), instantiated per dtype and variant in
// tile_<dtype>.hip.
//
// The march (tsq_march.hpp) runs the stages of one segment one behind the
// other in a single wavefront, which on a mesh of a few hundred rows is the
// whole pass: the other SIMDs are idle while (Q + K) K stage runs of 0.2 us
// follow each other.  Here a block of kTileWaves wavefronts holds one strip of
// kTileWaves * RP row pairs, RP pairs per wavefront, in registers (one load of
// psi and phase per site, all in flight together), and every step works on all
// its rows at once; the odd y-pairs that join two wavefronts swap their rows
// through LDS, one barrier a step.  Each step the outermost row pair on either
// side loses its neighbour, so after K stages the inner T - 2K of T pairs are
// stored (the x halo is the march's: K lanes per side).  Every site sees the
// march's operations in the march's order, so results are the march's, bit for
// bit.  What bounds it: at 256^2 complex128 two thirds of a launch are stage
// runs on the block's four SIMDs, the rest launch and memory latency.
//
// The number of steps is a kernel argument: nothing in registers depends on it.

#pragma once

#include "tsq_march.hpp"

namespace tsq {
namespace {

// Rows published for the odd y-pairs between wavefronts: [buffer][wavefront]
// [0 = first pair's top row, 1 = last pair's bottom row][16-byte part][lane].
template <class R>
struct TileExchange {
    static constexpr int kParts = 2 * sizeof(R) / 8;  // 16-byte parts of two complex sites
    float4 v[2][kTileWaves][2][kParts][kWaveSize];
};

// One pass of `a.tile_steps` steps (plus the closing odd factors if `a.tile_last`)
// over one strip and segment (a.seg_rows = 2 (T - 2K) stored rows).
template <class T, int RP, bool CLOSED, bool TD, bool U4>
__global__ void __launch_bounds__(kWaveSize * kTileWaves)
tile_kernel(const MarchArgs<typename T::R> a) {
    using R = typename T::R;
    using PT = PhaseT<T, TD>;
    using TT = TableT<T, TD>;
    static_assert(!U4 || (!CLOSED && !TD), "the fourth-order pass is periodic and static");
    constexpr int NT = kTileWaves * RP;  // row pairs of the block
    __shared__ TileExchange<R> xch;
    __shared__ double2 turns[TD ? kTurns : 1];
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const int S = a.tile_steps, K = S + (a.tile_last ? 1 : 0);
    const int nx = a.nx, ny = a.ny;

    // XCD-aware block order, segment-major, as in the march
    const int nb = gridDim.x, full = nb & ~7, b = blockIdx.x;
    const int lb = (b < full) ? ((b & 7) * (full >> 3) + (b >> 3)) : b;
    const int seg = lb / a.nstrips, strip = lb - seg * a.nstrips;

    // x: as in the march, one pair per lane, K halo lanes per side
    const long long xu = (long long)strip * a.strip_sites + (long long)(lane - K) * 2;
    const bool inner = lane >= K && lane < kWaveSize - K;
    const int col = CLOSED ? (int)xu : wrap(xu, nx);
    XPairs<1, CLOSED> xm;
    int ccol[2] = {0, 0};
    if constexpr (CLOSED) {
        auto in = [&](long long x) { return x >= 0 && x < nx; };
        xm.even[0] = in(xu) && in(xu + 1);
        xm.inner[0] = false;
        xm.left = in(xu - 1) && in(xu);
        xm.right = in(xu + 1) && in(xu + 2);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            xm.kx[i] = ((nx & 1) && xu + i == nx - 1) ? a.kxw : 1.0;
            ccol[i] = (int)(xu + i < 0 ? 0 : (xu + i >= nx ? nx - 1 : xu + i));
        }
    }

    // y: the block's pairs are q0 - K + p, p = 0 .. NT-1 (unwrapped); this
    // wavefront's are p = w RP + j
    const int hp = CLOSED ? (ny + 1) >> 1 : ny >> 1;
    const int q0 = seg * (a.seg_rows >> 1);
    const int q1 = min(q0 + (a.seg_rows >> 1), hp);
    const int p0 = w * RP;
    const int qw = q0 - K + p0;  // pair index of j = 0
    auto load_row = [&](int r, Row<R, 2>& v) {
        if constexpr (CLOSED) {
            const long long off = (long long)(r < 0 ? 0 : (r >= ny ? ny - 1 : r)) * nx;
#pragma unroll
            for (int i = 0; i < 2; ++i) load_site(a.src, off + ccol[i], v.re[i], v.im[i]);
        } else {
            load_pair(a.src, (long long)r * nx + col, v, 0);
        }
    };
    auto load_table = [&](const void* tab, int r, TT (&v)[2]) {
        const TT* P = reinterpret_cast<const TT*>(tab);
        if constexpr (CLOSED) {
            const long long off = (long long)(r < 0 ? 0 : (r >= ny ? ny - 1 : r)) * nx;
#pragma unroll
            for (int i = 0; i < 2; ++i) v[i] = P[off + ccol[i]];
        } else {
            const long long off = (long long)r * nx + col;
#pragma unroll
            for (int i = 0; i < 2; ++i) v[i] = P[off + i];
        }
    };

    PairRows<R, 2> h[RP];
    PhasePair<PT, 2> ph[RP], phm[U4 ? RP : 1];
    {
        TT tf[RP][2], tg[RP][2], mf[U4 ? RP : 1][2], mg[U4 ? RP : 1][2];
#pragma unroll
        for (int j = 0; j < RP; ++j) {
            // every pair is a row pair of the mesh (wrapped or clamped to it)
            const int r = CLOSED ? 2 * (qw + j) : wrap(2LL * (qw + j), ny);
            load_row(r, h[j].f);
            load_row(r + 1, h[j].g);
            load_table(a.ptab, r, tf[j]);
            load_table(a.ptab, r + 1, tg[j]);
            if constexpr (U4) {
                load_table(a.ptab2, r, mf[j]);
                load_table(a.ptab2, r + 1, mg[j]);
            }
        }
        if constexpr (TD) {
            constexpr int kThreads = kWaveSize * kTileWaves;
            static_assert(kTurns % kThreads == 0, "whole table entries per thread");
#pragma unroll
            for (int e = 0; e < kTurns / kThreads; ++e)
                turns[threadIdx.x + e * kThreads] =
                    reinterpret_cast<const double2*>(a.ptab2)[threadIdx.x + e * kThreads];
            // read after the first step's barrier
        }
#pragma unroll
        for (int j = 0; j < RP; ++j)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if constexpr (TD) {
                    ph[j].f[i] = tf[j][i];
                    ph[j].g[i] = tg[j][i];
                } else {
                    ph[j].f[i] = decode_phase(tf[j][i]);
                    ph[j].g[i] = decode_phase(tg[j][i]);
                    if constexpr (U4) {
                        phm[j].f[i] = decode_phase(mf[j][i]);
                        phm[j].g[i] = decode_phase(mg[j][i]);
                    }
                }
            }
    }

    int buf = 0;
    for (int k = 0; k < K; ++k, buf ^= 1) {
        // pairs [k, NT-1-k] hold the state after k steps; this stage completes
        // [k+1, NT-2-k].  Wavefront-uniform tests; every wavefront meets the
        // barrier.
        const bool has = p0 + RP - 1 >= k && p0 <= NT - 1 - k;
        R oxs, oxd, oys, oyd, ext, eyt;
        if constexpr (U4) {
            oxs = a.u4.xs[k]; oxd = a.u4.xd[k]; oys = a.u4.yt[k]; oyd = R(0);
            ext = a.u4.ext[k == 2 ? 1 : 0]; eyt = a.u4.eyt[k == 2 ? 1 : 0];
        } else {
            const bool first = k == 0, close = k == S;
            oxs = first ? a.o1xs : close ? a.c1xs : a.o2xs;
            oxd = first ? a.o1xd : close ? a.c1xd : a.o2xd;
            oys = first ? a.o1ys : close ? a.c1ys : a.o2ys;
            oyd = first ? a.o1yd : close ? a.c1yd : a.o2yd;
            ext = a.ehxs; eyt = a.ehys;
        }
        if (has) {
            if (CLOSED || U4 || k == 0 || k == S) {
#pragma unroll
                for (int j = 0; j < RP; ++j) {
                    odd_x<CLOSED>(h[j].f, oxs, oxd, xm);
                    odd_x<CLOSED>(h[j].g, oxs, oxd, xm);
                }
            } else if constexpr (!CLOSED && !U4) {
#pragma unroll
                for (int j = 0; j < RP; ++j) {
                    odd_x_t(h[j].f, oxs);
                    odd_x_t(h[j].g, oxs);
                }
            }
            put16(xch.v[buf][w][0], lane, h[0].f);
            put16(xch.v[buf][w][1], lane, h[RP - 1].g);
        }
        // one barrier a step: a buffer is written again two steps later, after
        // the barrier that every wavefront meets once it has read it
        __syncthreads();
        if (p0 + RP - 1 <= k || p0 >= NT - 1 - k) continue;  // completes no pair
        Row<R, 2> up{}, dn{};  // bottom row of the pair above, top row of the pair below
        if (w > 0) get16(xch.v[buf][w - 1][1], lane, up);
        if (w + 1 < kTileWaves) get16(xch.v[buf][w + 1][0], lane, dn);
        if constexpr (CLOSED) {
            // odd y-pair of pairs q and q+1: rows 2q+1, 2q+2
            auto oy = [&](int q) { return q >= 0 && 2 * q + 2 < ny; };
            side_y(h[0].f, up, oy(qw - 1) ? oys : R(0), oy(qw - 1) ? oyd : R(0));
#pragma unroll
            for (int j = 0; j + 1 < RP; ++j)
                pair_y(h[j].g, h[j + 1].f, oy(qw + j) ? oys : R(0), oy(qw + j) ? oyd : R(0));
            side_y(h[RP - 1].g, dn, oy(qw + RP - 1) ? oys : R(0), oy(qw + RP - 1) ? oyd : R(0));
        } else {
            (void)oyd;
            side_y_t(h[0].f, up, oys);
#pragma unroll
            for (int j = 0; j + 1 < RP; ++j) pair_y_t(h[j].g, h[j + 1].f, oys);
            side_y_t(h[RP - 1].g, dn, oys);
        }
        if (k == S) continue;
#pragma unroll
        for (int j = 0; j < RP; ++j) {
            PairRows<R, 2>& o = h[j];
            const int q = qw + j;
            const R et = (!CLOSED || (q >= 0 && 2 * q + 1 < ny)) ? eyt : R(0);
            even_x_t<CLOSED>(o.f, ext, xm);
            even_x_t<CLOSED>(o.g, ext, xm);
            pair_y_t(o.f, o.g, et);
            if constexpr (TD) {
                double kf = 1.0, kg = 1.0;
                const double* kx = nullptr;
                if constexpr (CLOSED) {
                    const bool odd_h = (ny & 1) != 0;
                    kf = (odd_h && 2 * q == ny - 1) ? a.kyw : 1.0;
                    kg = (odd_h && 2 * q + 1 == ny - 1) ? a.kyw : 1.0;
                    kx = xm.kx;
                }
                phase_rows_td<CLOSED>(o.f, o.g, ph[j].f, ph[j].g, a.g[k], turns, kx, kf, kg);
            } else if (U4 && k == 2) {
                phase_row(o.f, phm[U4 ? j : 0].f);
                phase_row(o.g, phm[U4 ? j : 0].g);
            } else {
                phase_row(o.f, ph[j].f);
                phase_row(o.g, ph[j].g);
            }
            pair_y_t(o.f, o.g, et);
            even_x_t<CLOSED>(o.f, ext, xm);
            even_x_t<CLOSED>(o.g, ext, xm);
        }
    }

#pragma unroll
    for (int j = 0; j < RP; ++j) {
        const int p = p0 + j, q = qw + j;
        if (p < K || p > NT - 1 - K || q >= q1) continue;  // wavefront-uniform
        const long long rf = 2LL * q, rg = rf + 1;
        if constexpr (CLOSED) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                if (inner && xu + i >= 0 && xu + i < nx) {
                    if (rf < ny) store_site(a.dst, rf * nx + xu + i, h[j].f.re[i], h[j].f.im[i]);
                    if (rg < ny) store_site(a.dst, rg * nx + xu + i, h[j].g.re[i], h[j].g.im[i]);
                }
            }
        } else if (inner && xu < nx) {
            store_pair(a.dst, rf * nx + col, h[j].f, 0);
            store_pair(a.dst, rg * nx + col, h[j].g, 0);
        }
    }
}

template <class T, int RP>
const void* pick_tile_rp(bool closed, bool td, bool u4) {
    if (u4) {
        if constexpr (RP == 1)
            return reinterpret_cast<const void*>(&tile_kernel<T, 1, false, false, true>);
        else
            return nullptr;
    }
    if (closed)
        return td ? reinterpret_cast<const void*>(&tile_kernel<T, RP, true, true, false>)
                  : reinterpret_cast<const void*>(&tile_kernel<T, RP, true, false, false>);
    return td ? reinterpret_cast<const void*>(&tile_kernel<T, RP, false, true, false>)
              : reinterpret_cast<const void*>(&tile_kernel<T, RP, false, false, false>);
}
template <class T>
const void* pick_tile(int rp, bool closed, bool td, bool u4) {
    return rp == 1 ? pick_tile_rp<T, 1>(closed, td, u4) : pick_tile_rp<T, 2>(closed, td, u4);
}

}  // namespace
}  // namespace tsq

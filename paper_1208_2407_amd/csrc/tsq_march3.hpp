// Three-dimensional march: the second-order step on a (nz, ny, nx) mesh, one
// time step per pass.  Sec. 2 splits the 2D mesh Hamiltonian into five parts
// (the diagonal and the even and odd pairs of each axis); this march extends
// that split to three axes, seven parts (Sec. 5 names three dimensions as
// future work).  Per step, first factor first:
//   Ox Oy Oz Ex Ey Ez P Ez Ey Ex Oz Oy Ox   (kinetic factors for dt/2)
// with consecutive steps sharing their odd factors as in the 2D march; a
// closing pass after the last step applies its final Oz Oy Ox.
//
// Tiling: a block of kWaves3 wavefronts owns an x-strip of 64 lanes (two
// x-sites per lane) times a slab of kWaves3 row pairs (wavefront w holds row
// pair w: each lane keeps rows a = 2m and b = 2m+1 of its two x-sites), and it
// marches along z over a segment of plane pairs with the 2D march's pipeline
// (planes in place of rows, F/G named by the direction of travel).  x-pairs
// are exchanged across lanes by DPP shifts; even y-pairs sit in a lane; odd
// y-pairs join row b of wavefront w with row a of wavefront w+1 through LDS,
// one block barrier per exchange; z-pairs sit in a lane.  The lanes and
// wavefronts at the tile edges are halo whose results are discarded (one pair
// per side, like the 2D halo).
#pragma once

#include "tsq_internal3.h"
#include "tsq_march.hpp"

namespace tsq {
namespace {

// A plane pair held by one lane: planes F and G, each with rows a and b of the
// lane's row pair ([0] = a, [1] = b), two x-sites per row.
template <class R>
struct PlanePair {
    Row<R, 2> f[2], g[2];
};

template <class PT>
struct PlanePhase {
    PT f[2][2], g[2][2];  // [row][site]
};

// LDS area of one block for the odd y exchange: [buffer][wavefront][plane]
// [row][component][lane]; components re0, im0, re1, im1 of the two sites.
template <class R>
struct Exchange3 {
    R v[2][kWaves3][2][2][4][kWaveSize];
};

// Wait for this wavefront's LDS writes, then meet the block at the barrier;
// global loads in flight are not waited for.
__device__ __forceinline__ void block_sync_lds() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

template <class R>
__device__ __forceinline__ void put_row(Exchange3<R>& x, int buf, int w, int plane, int row,
                                        int lane, const Row<R, 2>& r) {
    x.v[buf][w][plane][row][0][lane] = r.re[0];
    x.v[buf][w][plane][row][1][lane] = r.im[0];
    x.v[buf][w][plane][row][2][lane] = r.re[1];
    x.v[buf][w][plane][row][3][lane] = r.im[1];
}

template <class R>
__device__ __forceinline__ Row<R, 2> get_row(const Exchange3<R>& x, int buf, int w, int plane,
                                             int row, int lane) {
    Row<R, 2> r;
    r.re[0] = x.v[buf][w][plane][row][0][lane];
    r.im[0] = x.v[buf][w][plane][row][1][lane];
    r.re[1] = x.v[buf][w][plane][row][2][lane];
    r.im[1] = x.v[buf][w][plane][row][3][lane];
    return r;
}

// Odd y-pairs of two planes p and q: row b of wavefront w with row a of
// wavefront w+1.  Every wavefront publishes its rows, the block meets once,
// and each wavefront rotates its own rows with its neighbours' published
// (pre-factor) values; the wavefronts at the slab edges have no partner in the
// block (halo) and rotate with zeros.  Buffers alternate, so one barrier per
// exchange suffices: a buffer is written again only after every wavefront has
// passed the barrier of the exchange in between, hence finished reading it.
template <class R>
__device__ __forceinline__ void odd_y3(Row<R, 2> (&p)[2], Row<R, 2> (&q)[2], R s, R d,
                                       Exchange3<R>& x, int& buf, int w, int lane) {
    put_row(x, buf, w, 0, 0, lane, p[0]);
    put_row(x, buf, w, 0, 1, lane, p[1]);
    put_row(x, buf, w, 1, 0, lane, q[0]);
    put_row(x, buf, w, 1, 1, lane, q[1]);
    block_sync_lds();
    Row<R, 2> pb, pa, qb, qa;  // partners of p[1], p[0], q[1], q[0]
#pragma unroll
    for (int i = 0; i < 2; ++i) pb.re[i] = pb.im[i] = pa.re[i] = pa.im[i] = R(0);
    qb = pb;
    qa = pb;
    if (w + 1 < kWaves3) {
        pb = get_row(x, buf, w + 1, 0, 0, lane);
        qb = get_row(x, buf, w + 1, 1, 0, lane);
    }
    if (w > 0) {
        pa = get_row(x, buf, w - 1, 0, 1, lane);
        qa = get_row(x, buf, w - 1, 1, 1, lane);
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        rot_site(p[1].re[i], p[1].im[i], pb.re[i], pb.im[i], s, d);
        rot_site(p[0].re[i], p[0].im[i], pa.re[i], pa.im[i], s, d);
        rot_site(q[1].re[i], q[1].im[i], qb.re[i], qb.im[i], s, d);
        rot_site(q[0].re[i], q[0].im[i], qa.re[i], qa.im[i], s, d);
    }
    buf ^= 1;
}

// The single stage of a pass.  o is the older plane pair, n the newer one; the
// odd factors act on the boundary planes (o.g, n.f), then the even factors
// and the phase on o.  A closing pass (CLOSE, after the last step) applies
// only the closing odd factors, for dt/2.
template <bool CLOSE, class R, class PT>
__device__ __forceinline__ void stage3(PlanePair<R>& o, PlanePair<R>& n,
                                       const March3Args<R>& a, const XPairs<1, false>& xm,
                                       const PlanePhase<PT>& ph, Exchange3<R>& x, int& buf,
                                       int w, int lane) {
    const R oxs = CLOSE ? a.ehs[0] : a.o1s[0], oxd = CLOSE ? a.ehd[0] : a.o1d[0];
    const R oys = CLOSE ? a.ehs[1] : a.o1s[1], oyd = CLOSE ? a.ehd[1] : a.o1d[1];
    const R ozs = CLOSE ? a.ehs[2] : a.o1s[2], ozd = CLOSE ? a.ehd[2] : a.o1d[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        odd_x<false>(o.g[r], oxs, oxd, xm);
        odd_x<false>(n.f[r], oxs, oxd, xm);
    }
    odd_y3(o.g, n.f, oys, oyd, x, buf, w, lane);
#pragma unroll
    for (int r = 0; r < 2; ++r) pair_y(o.g[r], n.f[r], ozs, ozd);
    if constexpr (!CLOSE) {
        const R es[3] = {a.ehs[0], a.ehs[1], a.ehs[2]};
        const R ed[3] = {a.ehd[0], a.ehd[1], a.ehd[2]};
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            even_x<false>(o.f[r], es[0], ed[0], xm);
            even_x<false>(o.g[r], es[0], ed[0], xm);
        }
        pair_y(o.f[0], o.f[1], es[1], ed[1]);
        pair_y(o.g[0], o.g[1], es[1], ed[1]);
#pragma unroll
        for (int r = 0; r < 2; ++r) pair_y(o.f[r], o.g[r], es[2], ed[2]);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            phase_row(o.f[r], ph.f[r]);
            phase_row(o.g[r], ph.g[r]);
        }
#pragma unroll
        for (int r = 0; r < 2; ++r) pair_y(o.f[r], o.g[r], es[2], ed[2]);
        pair_y(o.f[0], o.f[1], es[1], ed[1]);
        pair_y(o.g[0], o.g[1], es[1], ed[1]);
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            even_x<false>(o.f[r], es[0], ed[0], xm);
            even_x<false>(o.g[r], es[0], ed[0], xm);
        }
    }
}

// One run of plane pairs [q0, q1) of one column (strip, slab) of one pass;
// wavefront w of the block.
// Register homes as in the 2D march: the plane pair entering in iteration j
// stays in home j mod 3 until stored one iteration later.  The phase of the
// pair stage 0 completes is loaded one iteration ahead into one register
// home, right after the stage has used the previous one: the phase of pair j
// is loaded in iteration j and used in iteration j+1.
template <class T, bool CLOSE>
__device__ __forceinline__ void march3_tile(const March3Args<typename T::R>& a, int strip,
                                            int slab, int q0, int q1, bool rev, int w, int lane,
                                            Exchange3<typename T::R>& x, int& buf) {
    using R = typename T::R;
    using PT = typename T::PT;
    constexpr int K = 1;           // one stage: one step, or the closing odd factors
    constexpr int HL = K;          // halo lanes (x) and halo wavefronts (y) per side
    constexpr int NH = K + 2;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const long long plane = (long long)nx * ny;

    // x: the lane's x-pair (wrapped) and whether it is stored
    const long long xu = (long long)strip * a.strip_sites + (long long)(lane - HL) * 2;
    const int col = wrap(xu, nx);
    const bool x_keep = lane >= HL && lane < kWaveSize - HL && xu < nx;
    // y: the wavefront's row pair (wrapped) and whether it is stored
    const long long yu = (long long)slab * a.slab_pairs + (w - HL);  // unwrapped row pair
    const int ya = wrap(2 * yu, ny);
    const bool y_keep = w >= HL && w < kWaves3 - HL && 2 * yu < ny;
    const bool keep = x_keep && y_keep;
    const long long rowa = (long long)ya * nx + col, rowb = (long long)(ya + 1) * nx + col;
    const XPairs<1, false> xm{};

    // z: output plane pairs [q0, q1), input [q0 - K, q1 - 1 + K], marched up
    // (rev) or down; rz* are the first planes of the next pairs to load.
    const int nit = (q1 - q0) + 2 * K;
    const int tstart = rev ? q1 - 1 + K : q0 - K;
    const int fo = rev ? 1 : 0;
    const int zstep = rev ? -2 : 2;
    int rz = wrap(2LL * tstart, nz);
    int rzp = rz;  // phase
    int qout = rev ? q1 - 1 + 2 * K : q0 - 2 * K;

    auto step_z = [&](int& z) {
        z += zstep;
        z = z < 0 ? z + nz : z;
        z = z >= nz ? z - nz : z;
    };
    auto load_plane = [&](int z, Row<R, 2> (&rows)[2]) {
        load_pair(a.src, z * plane + rowa, rows[0], 0);
        load_pair(a.src, z * plane + rowb, rows[1], 0);
    };
    auto load_psi = [&](PlanePair<R>& h) {
        load_plane(rz + fo, h.f);
        load_plane(rz + 1 - fo, h.g);
        step_z(rz);
    };
    auto load_phase_plane = [&](int z, PT (&v)[2][2]) {
        const typename T::TT* P = reinterpret_cast<const typename T::TT*>(a.ptab);
        v[0][0] = decode_phase(P[z * plane + rowa]);
        v[0][1] = decode_phase(P[z * plane + rowa + 1]);
        v[1][0] = decode_phase(P[z * plane + rowb]);
        v[1][1] = decode_phase(P[z * plane + rowb + 1]);
    };
    auto load_phase = [&](PlanePhase<PT>& ph) {
        load_phase_plane(rzp + fo, ph.f);
        load_phase_plane(rzp + 1 - fo, ph.g);
        step_z(rzp);
    };
    auto store_out = [&](const PlanePair<R>& h) {
        const int qo = qout;
        qout += rev ? -1 : 1;
        if (rev ? (qo >= q1) : (qo < q0)) return;  // warming up (wavefront-uniform)
        if (!keep) return;
        const long long zf = 2LL * qo + fo, zg = 2LL * qo + 1 - fo;
        store_pair(a.dst, zf * plane + rowa, h.f[0], 0);
        store_pair(a.dst, zf * plane + rowb, h.f[1], 0);
        store_pair(a.dst, zg * plane + rowa, h.g[0], 0);
        store_pair(a.dst, zg * plane + rowb, h.g[1], 0);
    };

    PlanePair<R> home[NH];
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                home[h].f[r].re[i] = home[h].f[r].im[i] = R(0);
                home[h].g[r].re[i] = home[h].g[r].im[i] = R(0);
            }
    PlanePhase<PT> ph;
#pragma unroll
    for (int r = 0; r < 2; ++r)
#pragma unroll
        for (int i = 0; i < 2; ++i) ph.f[r][i] = ph.g[r][i] = zero_phase<PT>();

    int q = rev ? tstart + 1 : tstart - 1;     // pair stage 0 completes this iteration
    const int qend = rev ? q - nit : q + nit;  // one past the last iteration
    load_psi(home[0]);
    auto iteration = [&](auto U) {
        constexpr int u = decltype(U)::value;
        load_psi(home[(u + 1) % NH]);  // the last iteration loads one pair more than it uses
        stage3<CLOSE>(home[(u - 1 + NH) % NH], home[u % NH], a, xm, ph, x, buf, w, lane);
        if constexpr (!CLOSE) load_phase(ph);  // the phase of the pair completed next
        store_out(home[(u - K + 2 * NH) % NH]);
        q += rev ? -1 : 1;
        return q != qend;
    };
    // no phase before the loop: iteration 0 completes a pair of the zero
    // warm-up (before the march start) and then loads the phase of pair 0
    while (static_all<NH>(iteration)) {
    }
}

template <class T, bool CLOSE>
__global__ void __launch_bounds__(kWaveSize * kWaves3)
march3_kernel(const March3Args<typename T::R> a) {
    __shared__ Exchange3<typename T::R> xch;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    // XCD-aware block order, as in the 2D march.  Tiles are dealt segment
    // fastest; the same segment of neighbouring columns marches the same
    // planes at the same time, so the halo rows two slabs share meet in L2.
    const int nb = gridDim.x;
    const int full = nb & ~7;
    const int b = blockIdx.x;
    const int lb = (b < full) ? ((b & 7) * (full >> 3) + (b >> 3)) : b;
    const long long ntiles = (long long)a.nstrips * a.nslabs * a.nsegs;
    if (lb >= ntiles) return;  // uniform per block
    const int seg = (int)(lb % a.nsegs);
    const long long rest = lb / a.nsegs;
    const int slab = (int)(rest % a.nslabs);
    const int strip = (int)(rest / a.nslabs);
    const int q0 = seg * a.seg_pairs;
    const int q1 = min(q0 + a.seg_pairs, a.nz >> 1);
    int buf = 0;
    march3_tile<T, CLOSE>(a, strip, slab, q0, q1, seg & 1, w, lane, xch, buf);
}

// ------------------------------------------------------------------ slab march, one or two steps per pass
//
// The pass of one step reads and writes the mesh once per step and is bound by
// that.  This march takes two steps (or one step and the closing odd factors)
// per read and write: two stages, the block a slab of kWaves3 * RP row pairs,
// RP of them per wavefront, of which K (the stages) per side are halo.
// complex64 takes RP = 2 (12 of 16 row pairs kept at two stages; four plane
// pairs of psi and one of phases are 160 registers, two wavefronts per SIMD),
// complex128 RP = 1 (4 of 8 kept: twice the bytes per register).  One stage
// serves single steps and small meshes, whose passes last as long as one
// block's iterations (RP = 1 there: half the work per iteration).  Rotations in
// the tangent form as on periodic 2D meshes, the cosines of a step in the phase
// table; stage 0 restores what the opening half factors differ by.
template <class R, int RP>
struct SlabPair {
    Row<R, 2> f[2 * RP], g[2 * RP];
};
template <class TT, int RP>
struct SlabPhase {
    TT f[2 * RP][2], g[2 * RP][2];  // [row][site], as the table stores them
};

// LDS of a block: the rows published for the odd y-pairs between wavefronts
// ([area][wavefront][plane][first or last row][16-byte part][lane]; two areas
// alternate and a stage meets one barrier, but for complex128 at two stages,
// which has room for one and meets two), and at two full stages the phases
// stage 0 has used, kept for stage 1 of the next iteration ([wavefront][row]
// [part][lane], as the table stores them: each lane reads what it wrote).
template <class R, int RP, bool PH>
struct SlabLds {
    static constexpr int kParts = 2 * sizeof(R) / 8;
    static constexpr int kAreas = PH && sizeof(R) == 8 ? 1 : 2;
    float4 v[kAreas][kWaves3][2][2][kParts][kWaveSize];
    float4 ph[PH ? kWaves3 : 1][4 * RP][kParts][kWaveSize];
};
__device__ __forceinline__ void put_phase(float4 (&v)[1][kWaveSize], int lane, const int2 (&t)[2]) {
    *reinterpret_cast<int4*>(&v[0][lane]) = make_int4(t[0].x, t[0].y, t[1].x, t[1].y);
}
__device__ __forceinline__ void get_phase(const float4 (&v)[1][kWaveSize], int lane, int2 (&t)[2]) {
    const int4 a = *reinterpret_cast<const int4*>(&v[0][lane]);
    t[0] = make_int2(a.x, a.y);
    t[1] = make_int2(a.z, a.w);
}
__device__ __forceinline__ void put_phase(float4 (&v)[2][kWaveSize], int lane, const double2 (&t)[2]) {
#pragma unroll
    for (int c = 0; c < 2; ++c) *reinterpret_cast<double2*>(&v[c][lane]) = t[c];
}
__device__ __forceinline__ void get_phase(const float4 (&v)[2][kWaveSize], int lane, double2 (&t)[2]) {
#pragma unroll
    for (int c = 0; c < 2; ++c) t[c] = *reinterpret_cast<const double2*>(&v[c][lane]);
}

// Stage K2: 0 or 1; CLOSE: stage 1 applies the closing odd factors only.
// `area` is the exchange area of this run.  `take(r, tf, tg)` yields the table
// entries of row r of both planes.
template <class T, int RP, int K2, bool CLOSE, class Lds, class Take>
__device__ __forceinline__ void slab_stage(SlabPair<typename T::R, RP>& o,
                                           SlabPair<typename T::R, RP>& n,
                                           const March3Args<typename T::R>& a,
                                           Lds& x, int& area, int w, int lane, Take&& take) {
    using R = typename T::R;
    constexpr int NR = 2 * RP;
    const XPairs<1, false> xm{};
    constexpr bool last = K2 == 1 && CLOSE;
    const R oxt = last ? a.c1x[0] : K2 == 0 ? a.o1x[0] : a.t2[0];
    const R oyt = last ? a.t1[1] : K2 == 0 ? a.o1t[1] : a.t2[1];
    const R ozt = last ? a.t1[2] : K2 == 0 ? a.o1t[2] : a.t2[2];
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        if constexpr (K2 == 0 || last) {
            const R xd = last ? a.c1x[1] : a.o1x[1];
            odd_x<false>(o.g[r], oxt, xd, xm);
            odd_x<false>(n.f[r], oxt, xd, xm);
        } else {
            odd_x_t(o.g[r], oxt);
            odd_x_t(n.f[r], oxt);
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    // Two areas, taken in turn by the runs as they come (the fill skips some): one
    // is written again only after the barrier of the run in between, which every
    // wavefront meets after its reads.  One area: a barrier before it is written.
    if constexpr (Lds::kAreas == 1) block_sync_lds();
    put16(x.v[area][w][0][0], lane, o.g[0]);
    put16(x.v[area][w][0][1], lane, o.g[NR - 1]);
    put16(x.v[area][w][1][0], lane, n.f[0]);
    put16(x.v[area][w][1][1], lane, n.f[NR - 1]);
    block_sync_lds();
#pragma unroll
    for (int r = 1; r + 1 < NR; r += 2) {
        pair_y_t(o.g[r], o.g[r + 1], oyt);
        pair_y_t(n.f[r], n.f[r + 1], oyt);
    }
    {
        // the block's first and last wavefronts have no partner there (halo)
        Row<R, 2> p{}, q{};
        if (w > 0) {
            get16(x.v[area][w - 1][0][1], lane, p);
            get16(x.v[area][w - 1][1][1], lane, q);
        }
        side_y_t(o.g[0], p, oyt);
        side_y_t(n.f[0], q, oyt);
    }
    __builtin_amdgcn_sched_barrier(0);
    {
        Row<R, 2> p{}, q{};
        if (w + 1 < kWaves3) {
            get16(x.v[area][w + 1][0][0], lane, p);
            get16(x.v[area][w + 1][1][0], lane, q);
        }
        side_y_t(o.g[NR - 1], p, oyt);
        side_y_t(n.f[NR - 1], q, oyt);
    }
    if constexpr (Lds::kAreas == 2) area ^= 1;
#pragma unroll
    for (int r = 0; r < NR; ++r) pair_y_t(o.g[r], n.f[r], ozt);
    if constexpr (!last) {
        const R ex = a.t1[0], ey = a.t1[1], ez = a.t1[2];
#pragma unroll
        for (int r = 0; r < NR; r += 2) {
#pragma unroll
            for (int i = r; i < r + 2; ++i) {
                even_x_t<false>(o.f[i], ex, xm);
                even_x_t<false>(o.g[i], ex, xm);
            }
            pair_y_t(o.f[r], o.f[r + 1], ey);
            pair_y_t(o.g[r], o.g[r + 1], ey);
#pragma unroll
            for (int i = r; i < r + 2; ++i) {
                __builtin_amdgcn_sched_barrier(0);  // one row's decoded phases at a time
                pair_y_t(o.f[i], o.g[i], ez);
                typename T::TT tf[2], tg[2];
                take(i, tf, tg);
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    // the entry is scaled before the product: as it is stored
                    // (2^30 and more), parts of psi beyond 1e29 would overflow
                    apply_phase(o.f[i].re[c], o.f[i].im[c], decode_phase(tf[c], a.table_unit));
                    apply_phase(o.g[i].re[c], o.g[i].im[c], decode_phase(tg[c], a.table_unit));
                }
                pair_y_t(o.f[i], o.g[i], ez);
            }
            pair_y_t(o.f[r], o.f[r + 1], ey);
            pair_y_t(o.g[r], o.g[r + 1], ey);
#pragma unroll
            for (int i = r; i < r + 2; ++i) {
                even_x_t<false>(o.f[i], ex, xm);
                even_x_t<false>(o.g[i], ex, xm);
            }
        }
    }
}

// v modulo n for v up to 2N outside [0, n), n even and at least 2: no division, of
// which a block of a small mesh, a handful of iterations long, would feel each.
template <int N>
__device__ __forceinline__ int wrap_near(int v, int n) {
#pragma unroll
    for (int i = 0; i < N; ++i) {
        v = v < 0 ? v + n : v;
        v = v >= n ? v - n : v;
    }
    return v;
}

template <class T, int RP, int NS, bool CLOSE>
__global__ void __launch_bounds__(kWaveSize * kWaves3)
slab_kernel(const March3Args<typename T::R> a) {
    using R = typename T::R;
    using TT = typename T::TT;
    static_assert(NS == 1 || NS == 2, "one or two stages");
    static_assert(!CLOSE || NS == 2, "the closing factors are a second stage");
    constexpr int K = NS, NH = K + 2, NR = 2 * RP;
    constexpr bool PH = NS == 2 && !CLOSE;
    using Lds = SlabLds<R, RP, PH>;
    __shared__ Lds xch;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x / kWaveSize);
    const int nb = gridDim.x, full = nb & ~7, b = blockIdx.x;
    const int lb = (b < full) ? ((b & 7) * (full >> 3) + (b >> 3)) : b;
    // XCD-aware: an XCD takes a run of neighbouring slabs of one segment, which read
    // each other's y halo (a third to all of what they keep) through one L2.  With a
    // column's segments next to each other instead, which share the smaller z halo, us
    // per step: complex64 512^3 421 (405 this way), 192^3 32.4 (28.8), complex128
    // 512^3 1149 (1046), 106^3 17.3 (15.5); 100 x 200 x 60, segments of two pairs,
    // 8.7 (9.3) and 15.7 (16.4).
    const int cols = gridDim.x / a.nsegs, seg = lb / cols, rest = lb % cols;
    const int q0 = seg * a.seg_pairs, q1 = min(q0 + a.seg_pairs, a.nz >> 1);
    const bool rev = (seg & 1) != 0;
    const int nx = a.nx, ny = a.ny, nz = a.nz;
    const long long plane = (long long)nx * ny;

    // A full strip of one slab, or the strip left over, a slab to each group of
    // pack_lanes lanes.  A group's outer K lanes are its halo as a wavefront's are, so
    // what the shifts bring from the next group is never stored; lanes past the last
    // group count on from it, so that they load what its halo does (below).
    int strip = rest / a.nslabs, slab = rest % a.nslabs;
    int glane = lane, glanes = kWaveSize;  // lane of the group, its lanes
    bool mine = true;
    if (rest >= a.strip_cols) {
        const int pack = kWaveSize / a.pack_lanes, sub = min(lane / a.pack_lanes, pack - 1);
        strip = a.nstrips;
        slab = (rest - a.strip_cols) * pack + sub;
        glanes = a.pack_lanes;
        glane = lane - sub * glanes;
        mine = slab < a.nslabs;
    }

    // Lanes (row pairs) further past the mesh than the halo of its last column
    // (row pair) load what that halo loads: nothing stored depends on them, and
    // a last strip or slab that is mostly empty costs no memory traffic.
    const int xu = strip * a.strip_sites + (glane - K) * 2;
    const int col = wrap_near<K>(min(xu, nx - 2 + 2 * K), nx);
    const bool x_keep = mine && glane >= K && glane < glanes - K && xu < nx;
    const int yu = slab * a.slab_pairs + w * RP - K;  // unwrapped first row pair
    // byte offset of each row pair's first row within a plane (psi and the table
    // have the same bytes per site); planes start at wavefront-uniform addresses
    constexpr unsigned E = 2 * sizeof(R);
    static_assert(sizeof(TT) == E, "psi and table sites of one size");
    unsigned row[RP];
    bool keep[RP];
#pragma unroll
    for (int j = 0; j < RP; ++j) {
        row[j] = ((unsigned)wrap_near<K>(2 * min(yu + j, (ny >> 1) - 1 + K), ny) * (unsigned)nx + (unsigned)col) * E;
        keep[j] = x_keep && w * RP + j >= K && w * RP + j < kWaves3 * RP - K && 2 * (yu + j) < ny;
    }
    const long long pbytes = plane * E, rbytes = (long long)nx * E;

    const int nit = (q1 - q0) + 2 * K;
    const int tstart = rev ? q1 - 1 + K : q0 - K;
    const int fo = rev ? 1 : 0, zstep = rev ? -2 : 2;
    int rz = wrap_near<K>(2 * tstart, nz);   // first plane of the next pair to load
    // ... of the next phase pair: one pair behind where every iteration loads the
    // phases it uses (two stages)
    int rzp = NS == 1 ? rz : wrap_near<K + 1>(2 * tstart - zstep, nz);
    int qout = rev ? q1 - 1 + 2 * K : q0 - 2 * K;
    auto step_z = [&](int& z) {
        z += zstep;
        z = z < 0 ? z + nz : z;
        z = z >= nz ? z - nz : z;
    };
    auto load_psi = [&](SlabPair<R, RP>& h) {
        const char* pf = static_cast<const char*>(a.src) + (rz + fo) * pbytes;
        const char* pg = static_cast<const char*>(a.src) + (rz + 1 - fo) * pbytes;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < RP; ++j) {
                load_pair(pf + i * rbytes + row[j], 0, h.f[2 * j + i], 0);
                load_pair(pg + i * rbytes + row[j], 0, h.g[2 * j + i], 0);
            }
        step_z(rz);
    };
    // table entries of row r of the phase pair at plane rzp; step_z(rzp) after the last
    auto load_phase = [&](SlabPhase<TT, RP>& ph, int r) {
        const long long off = (r & 1) * rbytes;
        const TT* f = reinterpret_cast<const TT*>(static_cast<const char*>(a.ptab) + (rzp + fo) * pbytes +
                                                  off + row[r >> 1]);
        const TT* g = reinterpret_cast<const TT*>(static_cast<const char*>(a.ptab) +
                                                  (rzp + 1 - fo) * pbytes + off + row[r >> 1]);
#pragma unroll
        for (int c = 0; c < 2; ++c) {
            ph.f[r][c] = f[c];
            ph.g[r][c] = g[c];
        }
    };
    auto store_out = [&](const SlabPair<R, RP>& h) {
        const int qo = qout;
        qout += rev ? -1 : 1;
        if (rev ? (qo >= q1) : (qo < q0)) return;  // warming up (wavefront-uniform)
        char* pf = static_cast<char*>(a.dst) + (2LL * qo + fo) * pbytes;
        char* pg = static_cast<char*>(a.dst) + (2LL * qo + 1 - fo) * pbytes;
#pragma unroll
        for (int j = 0; j < RP; ++j)
            if (keep[j]) {
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    store_pair(pf + i * rbytes + row[j], 0, h.f[2 * j + i], 0);
                    store_pair(pg + i * rbytes + row[j], 0, h.g[2 * j + i], 0);
                }
            }
    };

    SlabPair<R, RP> home[NH];
    SlabPhase<TT, RP> ph;
#pragma unroll
    for (int h = 0; h < NH; ++h)
#pragma unroll
        for (int r = 0; r < NR; ++r)
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                home[h].f[r].re[i] = home[h].f[r].im[i] = R(0);
                home[h].g[r].re[i] = home[h].g[r].im[i] = R(0);
            }
    load_psi(home[0]);
    int it = 0, area = 0;
    auto load_phases = [&]() {
#pragma unroll
        for (int r = 0; r < NR; ++r) load_phase(ph, r);
        step_z(rzp);
    };
    if constexpr (NS == 1) load_phases();
    // Iteration j (home index u = j mod NH) loads psi of pair j+1; stage k completes
    // pair j-1-k.  Stage k's runs before iteration 2k+1 feed nothing stored and are
    // skipped (block-uniform: the stages meet barriers).  One stage: a row of the
    // next pair's phases is loaded as soon as the stage has taken its own.  Two:
    // registers hold one pair's phases only from their load at the start of the
    // iteration to its end (loading them ahead spills 250 bytes a lane more), and
    // stage 1 takes its pair's from LDS, where the iteration before left them.
    auto iteration = [&](auto U) {
        constexpr int u = decltype(U)::value;
        if constexpr (NS == 2) load_phases();
        load_psi(home[(u + 1) % NH]);
        __builtin_amdgcn_sched_barrier(0);
        if (it > 0) {
            slab_stage<T, RP, 0, CLOSE>(home[(u - 1 + NH) % NH], home[u], a, xch, area, w, lane,
                                        [&](int r, TT (&tf)[2], TT (&tg)[2]) {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    tf[c] = ph.f[r][c];
                    tg[c] = ph.g[r][c];
                }
                if constexpr (NS == 1) load_phase(ph, r);
            });
            if constexpr (NS == 1) step_z(rzp);
        }
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (NS == 2) {
            if (it > 2)
                slab_stage<T, RP, 1, CLOSE>(home[(u - 2 + NH) % NH], home[(u - 1 + NH) % NH], a, xch,
                                            area, w, lane, [&](int r, TT (&tf)[2], TT (&tg)[2]) {
                    get_phase(xch.ph[w][2 * r], lane, tf);
                    get_phase(xch.ph[w][2 * r + 1], lane, tg);
                });
            __builtin_amdgcn_sched_barrier(0);
        }
        if constexpr (PH) {
#pragma unroll
            for (int r = 0; r < NR; ++r) {
                put_phase(xch.ph[w][2 * r], lane, ph.f[r]);
                put_phase(xch.ph[w][2 * r + 1], lane, ph.g[r]);
            }
        }
        store_out(home[(u - K + NH) % NH]);
        ++it;
        return it != nit;
    };
    while (static_all<NH>(iteration)) {
    }
}

// The closing odd factors alone (after an even count of steps).  The odd pairs
// of the three axes tile the mesh with 2 x 2 x 2 cubes that nothing leaves, so a
// thread reads one cube, rotates it and writes it, in place or to the other
// buffer: a pass at the rate of a copy, and no copy back.
template <class R>
struct alignas(2 * sizeof(R)) Site {
    R re, im;
};
template <class T>
__global__ void __launch_bounds__(256)
close3_kernel(const March3Args<typename T::R> a) {
    using R = typename T::R;
    const int hx = a.nx >> 1, hy = a.ny >> 1;
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i >= hx) return;
    const long long plane = (long long)a.nx * a.ny;
    const int x0 = 2 * i + 1, x1 = x0 + 1 == a.nx ? 0 : x0 + 1;
    for (int c = blockIdx.y; c < hy * (a.nz >> 1); c += gridDim.y) {
        const int j = c % hy, k = c / hy;
        const int y0 = 2 * j + 1, y1 = y0 + 1 == a.ny ? 0 : y0 + 1;
        const int z0 = 2 * k + 1, z1 = z0 + 1 == a.nz ? 0 : z0 + 1;
        const long long l[4] = {z0 * plane + (long long)y0 * a.nx, z0 * plane + (long long)y1 * a.nx,
                                z1 * plane + (long long)y0 * a.nx, z1 * plane + (long long)y1 * a.nx};
        const Site<R>* src = static_cast<const Site<R>*>(a.src);
        Site<R>* dst = static_cast<Site<R>*>(a.dst);
        Row<R, 2> r[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const Site<R> u = src[l[q] + x0], v = src[l[q] + x1];
            r[q].re[0] = u.re; r[q].im[0] = u.im;
            r[q].re[1] = v.re; r[q].im[1] = v.im;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q)
            rot_pair(r[q].re[0], r[q].im[0], r[q].re[1], r[q].im[1], a.c1x[0], a.c1x[1]);
        pair_y_t(r[0], r[1], a.t1[1]);
        pair_y_t(r[2], r[3], a.t1[1]);
        pair_y_t(r[0], r[2], a.t1[2]);
        pair_y_t(r[1], r[3], a.t1[2]);
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            dst[l[q] + x0] = Site<R>{r[q].re[0], r[q].im[0]};
            dst[l[q] + x1] = Site<R>{r[q].re[1], r[q].im[1]};
        }
    }
}
template <class T>
const void* pick_close3() {
    return reinterpret_cast<const void*>(&close3_kernel<T>);
}

// Instances: one stage with one row pair per wavefront, two stages with one or
// (complex64) two.
template <class T, int RP>
const void* pick_slab2(bool close) {
    return close ? reinterpret_cast<const void*>(&slab_kernel<T, RP, 2, true>)
                 : reinterpret_cast<const void*>(&slab_kernel<T, RP, 2, false>);
}
template <class T>
const void* pick_slab(int stages, int rp, bool close) {
    if (stages == 1)
        return rp == 1 && !close ? reinterpret_cast<const void*>(&slab_kernel<T, 1, 1, false>) : nullptr;
    if (rp == 1) return pick_slab2<T, 1>(close);
    if constexpr (sizeof(typename T::R) == 4) {
        if (rp == 2) return pick_slab2<T, 2>(close);
    }
    return nullptr;
}

template <class T>
const void* pick_kernel3(bool close) {
    return close ? reinterpret_cast<const void*>(&march3_kernel<T, true>)
                 : reinterpret_cast<const void*>(&march3_kernel<T, false>);
}

}  // namespace
}  // namespace tsq

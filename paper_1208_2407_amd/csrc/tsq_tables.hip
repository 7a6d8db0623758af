// HIP kernels for gfx950 around the step march (Wittek & Cucchietti, Sec. 2):
// the phase table of the diagonal part H0 (and the table of a time-dependent
// potential), and the FP64 norm and energy of the mesh Hamiltonian.

#include "tsq_internal.h"

#include <algorithm>

namespace tsq {
namespace {

struct C128 {};
struct C64 {};

// ------------------------------------------------------------------ phase table of H0 (Sec. 2)

// Bound by FP64 arithmetic with the library's sincos (its long reduction above all),
// by memory with the short one below: complex64 us, before and now, 2048 x 1024
// 16.9 and 9.7, 3000 x 2000 30.1 and 21.4, 4096^2 87.5 and 55.1 (268 MB read and
// written: 4.9 TB/s), 16384 x 8192 546 and 458; complex128 (the library's, whose
// last bits its table keeps) 2048 x 1024 18.0 and 12.2, 3000 x 2000 31.9 and 25.0,
// 4096^2 103 and 85, from the grid alone (see launch_phase_table).
//
// exp(-i phi_l) times the site's scale (the cosines the march's tangent-form
// factors leave out; see TableScale) for sites l = i, i + n/4... of each
// thread's four-site groups: the four loads of V are issued before the four
// sines and cosines.
__device__ __forceinline__ double site_scale(const TableScale& sc, long long l) {
    if (sc.wx < 0 && sc.wy0 < 0) return sc.g;
    const bool x = sc.wx >= 0 && l % sc.nx == sc.wx;
    const bool y = sc.wy0 >= 0 && l >= sc.wy0;
    return x ? (y ? sc.gxy : sc.gx) : (y ? sc.gy : sc.g);
}
// sin and cos for a table that rounds to 2^-31: x = j pi/2 + r with j the integer
// nearest x 2/pi, |r| <= pi/4, pi/2 in two parts (the first product is exact in its
// FMA), then the Taylor series of sin r through r^15 and cos r through r^16 (omitted
// below 4.7e-17 and 2.1e-18).  j comes from adding 1.5 * 2^52 in the FMA that forms
// x 2/pi, so the low bits of the sum hold it.  Within 1.5e-16 of the exact values
// for |x| < 2^30; larger angles, infinities and NaN take the library's.
__device__ __forceinline__ void sincos_table(double x, double* s, double* c) {
    if (!(fabs(x) < 0x1p30)) {
        sincos(x, s, c);
        return;
    }
    const double shifter = 0x1.8p52;
    const double t = __builtin_fma(x, 0x1.45f306dc9c883p-1, shifter);  // 2/pi
    const double j = t - shifter;
    const int q = __double2loint(t);
    double r = __builtin_fma(-j, 0x1.921fb54442d18p+0, x);  // pi/2 rounded, and the rest
    r = __builtin_fma(-j, 0x1.1a62633145c07p-54, r);
    const double z = r * r;
    double a = -1.0 / 1307674368000.0;  // sin r = r + r z a
    a = __builtin_fma(a, z, 1.0 / 6227020800.0);
    a = __builtin_fma(a, z, -1.0 / 39916800.0);
    a = __builtin_fma(a, z, 1.0 / 362880.0);
    a = __builtin_fma(a, z, -1.0 / 5040.0);
    a = __builtin_fma(a, z, 1.0 / 120.0);
    a = __builtin_fma(a, z, -1.0 / 6.0);
    const double sn = __builtin_fma(r * z, a, r);
    double b = 1.0 / 20922789888000.0;  // cos r = 1 + z b
    b = __builtin_fma(b, z, -1.0 / 87178291200.0);
    b = __builtin_fma(b, z, 1.0 / 479001600.0);
    b = __builtin_fma(b, z, -1.0 / 3628800.0);
    b = __builtin_fma(b, z, 1.0 / 40320.0);
    b = __builtin_fma(b, z, -1.0 / 720.0);
    b = __builtin_fma(b, z, 1.0 / 24.0);
    b = __builtin_fma(b, z, -0.5);
    const double cs = __builtin_fma(b, z, 1.0);
    const double sv = (q & 1) ? cs : sn, cv = (q & 1) ? sn : cs;
    *s = (q & 2) ? -sv : sv;
    *c = ((q + 1) & 2) ? -cv : cv;
}

// g cos x and g sin x, g = (g, g_lo) in two parts, each with one rounding: formed from
// a rounded cosine an entry would round twice, and its error repeats at every step
// (200 steps of 0.01 rad a step and axis on a random 3D state: 5.7e-15, this way 4.3e-15).
// The reduction of sincos_table with what it rounds off kept in r_lo (the angle's third
// part of pi/2 is below 1e-23), cos = 1 - r^2/2 and sin = r - r^3/6 with the rest of the
// series in a tail that is small beside them, and the products by g with their FMA
// remainders.
__device__ __forceinline__ void scaled_sincos(double x, double g, double g_lo, double* gs, double* gc) {
    if (!(fabs(x) < 0x1p30)) {
        double s, c;
        sincos(x, &s, &c);
        *gs = __builtin_fma(g, s, g_lo * s);
        *gc = __builtin_fma(g, c, g_lo * c);
        return;
    }
    const double shifter = 0x1.8p52;
    const double t = __builtin_fma(x, 0x1.45f306dc9c883p-1, shifter);  // 2/pi
    const double j = t - shifter;
    const int q = __double2loint(t);
    const double r0 = __builtin_fma(-j, 0x1.921fb54442d18p+0, x);  // exact
    const double low = j * 0x1.1a62633145c07p-54;
    const double r = r0 - low, b = r - r0;
    const double r_lo = (r0 - (r - b)) - (low + b);
    const double z = r * r, z_lo = __builtin_fma(r, r, -z);
    double a = 1.0 / 355687428096000.0;  // sin r = r - r^3/6 + r^3 z a, through r^17 (omitted: 8e-20)
    a = __builtin_fma(a, z, -1.0 / 1307674368000.0);
    a = __builtin_fma(a, z, 1.0 / 6227020800.0);
    a = __builtin_fma(a, z, -1.0 / 39916800.0);
    a = __builtin_fma(a, z, 1.0 / 362880.0);
    a = __builtin_fma(a, z, -1.0 / 5040.0);
    a = __builtin_fma(a, z, 1.0 / 120.0);
    double d = -1.0 / 6402373705728000.0;  // cos r = 1 - z/2 + z^2 d, through r^18 (3e-21)
    d = __builtin_fma(d, z, 1.0 / 20922789888000.0);
    d = __builtin_fma(d, z, -1.0 / 87178291200.0);
    d = __builtin_fma(d, z, 1.0 / 479001600.0);
    d = __builtin_fma(d, z, -1.0 / 3628800.0);
    d = __builtin_fma(d, z, 1.0 / 40320.0);
    d = __builtin_fma(d, z, -1.0 / 720.0);
    d = __builtin_fma(d, z, 1.0 / 24.0);
    const double h = 0.5 * z, w = 1.0 - h;
    const double c_tail = __builtin_fma(z * z, d, ((1.0 - w) - h) - 0.5 * z_lo - r * r_lo);
    const double c6 = -1.0 / 6.0, c6_lo = -9.2518585385429707656e-18;
    const double r3 = r * z, r3_lo = __builtin_fma(r, z, -r3) + r * z_lo;
    const double u = c6 * r3, u_lo = __builtin_fma(c6, r3, -u) + (c6 * r3_lo + c6_lo * r3);
    const double v = r + u;
    const double s_tail = __builtin_fma(r3 * z, a, ((r - v) + u) + u_lo + r_lo * w);
    const double pc = g * w, ps = g * v;
    const double cs = pc + (__builtin_fma(g, w, -pc) + __builtin_fma(g, c_tail, g_lo * w));
    const double sn = ps + (__builtin_fma(g, v, -ps) + __builtin_fma(g, s_tail, g_lo * v));
    const double sv = (q & 1) ? cs : sn, cv = (q & 1) ? sn : cs;
    *gs = (q & 2) ? -sv : sv;
    *gc = ((q + 1) & 2) ? -cv : cv;
}

// `store(site, angle)` for every site of the thread.
template <class Store>
__device__ __forceinline__ void phase_sites(const double* __restrict__ V, long long n, double dt,
                                            double eps0, double hbar, Store&& store) {
    const long long stride = (long long)gridDim.x * blockDim.x;
    long long l = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    auto phase = [&](double v, long long at) { store(at, dt * (v + eps0) / hbar); };
    for (; l + 3 * stride < n; l += 4 * stride) {
        double v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) v[k] = V[l + k * stride];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            phase(v[k], l + k * stride);
        }
    }
    for (; l < n; l += stride) phase(V[l], l);
}

__global__ void phase_table_c128(const double* __restrict__ V, double2* __restrict__ P,
                                 long long n, double dt, double eps0, double hbar, TableScale sc) {
    phase_sites(V, n, dt, eps0, hbar, [&](long long l, double x) {
        double s, c;
        sincos(x, &s, &c);
        const double g = site_scale(sc, l);
        P[l] = make_double2(g * c, -(g * s));
    });
}

// Meshes whose scale has two parts (3D).
__global__ void phase_table_c128_two(const double* __restrict__ V, double2* __restrict__ P,
                                     long long n, double dt, double eps0, double hbar, TableScale sc) {
    phase_sites(V, n, dt, eps0, hbar, [&](long long l, double x) {
        double s, c;
        scaled_sincos(x, sc.g, sc.g_lo, &s, &c);
        P[l] = make_double2(c, -s);
    });
}

// complex64: cos(phi) and -sin(phi) as 32-bit fixed point, value * sc.unit
// rounded to nearest (2^30 on 2D meshes: |value| <= 1, so it fits; error <= 2^-31
// per part; 3D meshes of the slab march: see slab_table_unit).
__global__ void phase_table_c64(const double* __restrict__ V, int2* __restrict__ P,
                                long long n, double dt, double eps0, double hbar, TableScale sc) {
    phase_sites(V, n, dt, eps0, hbar, [&](long long l, double x) {
        double s, c;
        sincos_table(x, &s, &c);
        const double g = site_scale(sc, l);
        P[l] = make_int2(__double2int_rn(g * c * sc.unit), __double2int_rn(-(g * s) * sc.unit));
    });
}

// Time-dependent potential V0 + f(t) W: per site theta0 = dt (V0 + eps0) / hbar
// and w = dt W / hbar; step n's phase is exp(-i (theta0 + f_n w)), formed in
// the march.
__global__ void td_table(const double* __restrict__ V0, const double* __restrict__ W,
                         double2* __restrict__ T, long long n, double dt, double eps0, double hbar) {
    for (long long l = (long long)blockIdx.x * blockDim.x + threadIdx.x; l < n;
         l += (long long)gridDim.x * blockDim.x)
        T[l] = make_double2(dt * (V0[l] + eps0) / hbar, dt * W[l] / hbar);
}

// The march's factors scale * exp(-i j pi/1024), j = 0 .. kTurns-1 (j / 1024
// is exact, so sincospi sees the angle without rounding).
__global__ void td_turns(double2* __restrict__ U, double scale) {
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= kTurns) return;
    double sn, cs;
    sincospi((double)j / 1024.0, &sn, &cs);
    U[j] = make_double2(scale * cs, -(scale * sn));
}

// ------------------------------------------------------------------ norm and energy (Sec. 2)

__device__ __forceinline__ void load_site(const void* psi, long long l, double& re, double& im, C128) {
    double2 v = reinterpret_cast<const double2*>(psi)[l];
    re = v.x;
    im = v.y;
}
__device__ __forceinline__ void load_site(const void* psi, long long l, double& re, double& im, C64) {
    float2 v = reinterpret_cast<const float2*>(psi)[l];
    re = (double)v.x;
    im = (double)v.y;
}

// Block b sums |psi|^2 and Re(conj(psi) (H psi)) over its share of the mesh:
// work items (column chunk of kReduceThreads columns, band of `band` rows),
// items b, b + gridDim.x, ...; each thread walks its column down the band with
// the rows above and below the current one in registers, so every psi and V
// value is read once from device memory (the x-neighbours come from the cache
// lines the wavefront has just read).  Rows go four at a time, their loads
// issued together.  Fixed item order, fixed row order per thread and a fixed
// in-block tree: the result is bitwise reproducible.
template <class T>
__device__ __forceinline__ void site_energy(double cr, double ci, double ur, double ui, double dr,
                                            double di, double r1, double i1, double r2, double i2,
                                            double v, double Jx, double Jy, double eps0,
                                            double& an, double& ae) {
    const double diag = v + eps0;
    const double hr = diag * cr - Jx * (r1 + r2) - Jy * (dr + ur);
    const double hi = diag * ci - Jx * (i1 + i2) - Jy * (di + ui);
    an += cr * cr + ci * ci;
    ae += cr * hr + ci * hi;
}

// A thread's sum over its rows with the rounding errors of the additions kept beside it
// (Knuth's two-sum), so a band's length does not show in the result: its rows come in
// groups of four, added in pairs first, so this costs 12 additions per group.
struct LongSum {
    double s = 0.0, c = 0.0;
    __device__ __forceinline__ void add(double x) {
        const double t = s + x, b = t - s;
        c += (s - (t - b)) + (x - b);
        s = t;
    }
    __device__ __forceinline__ double value() const {
        return isfinite(s) ? s + c : s;  // an infinite sum leaves NaN in c
    }
};

// five wavefronts a SIMD: left to itself the compiler takes 100 registers and four
// (closed 4096^2, complex128, 149 us against 130)
template <class T>
__global__ void __launch_bounds__(kReduceThreads, 5)
observables_partial(const void* __restrict__ psi, const double* __restrict__ V, int nx, int ny,
                    double Jx, double Jy, double eps0, int closed, int band,
                    double* __restrict__ partial) {
    __shared__ double sn[kReduceThreads], se[kReduceThreads];
    constexpr int U = 4;  // rows per step of the walk
    LongSum an, ae;
    const int chunks = (nx + kReduceThreads - 1) / kReduceThreads;
    const int bands = (ny + band - 1) / band;
    const long long items = (long long)chunks * bands;
    for (long long it = blockIdx.x; it < items; it += gridDim.x) {
        const int x = (int)(it % chunks) * kReduceThreads + (int)threadIdx.x;
        const int y0 = (int)(it / chunks) * band;
        const int y1 = min(y0 + band, ny);
        if (x >= nx) continue;
        // neighbours wrap on periodic meshes and are absent beyond closed walls
        const bool has_xp = !closed || x + 1 < nx, has_xm = !closed || x > 0;
        const int xp = (x + 1 == nx) ? 0 : x + 1;
        const int xm = (x == 0) ? nx - 1 : x - 1;
        auto load_row = [&](int y, double& dr, double& di, double& r1, double& i1, double& r2,
                            double& i2, double& v) {
            // row below y, the x-neighbours on row y, V on row y
            dr = di = r1 = i1 = r2 = i2 = 0.0;
            if (!closed || y + 1 < ny)
                load_site(psi, (long long)(y + 1 == ny ? 0 : y + 1) * nx + x, dr, di, T());
            const long long row = (long long)y * nx;
            if (has_xp) load_site(psi, row + xp, r1, i1, T());
            if (has_xm) load_site(psi, row + xm, r2, i2, T());
            v = V[row + x];
        };
        double ur = 0, ui = 0, cr, ci;  // row above, current row
        if (!closed || y0 > 0)
            load_site(psi, (long long)(y0 == 0 ? ny - 1 : y0 - 1) * nx + x, ur, ui, T());
        load_site(psi, (long long)y0 * nx + x, cr, ci, T());
        int y = y0;
        for (; y + U <= y1; y += U) {
            double dr[U], di[U], r1[U], i1[U], r2[U], i2[U], v[U];
#pragma unroll
            for (int k = 0; k < U; ++k) load_row(y + k, dr[k], di[k], r1[k], i1[k], r2[k], i2[k], v[k]);
            double rn[U] = {}, re[U] = {};
#pragma unroll
            for (int k = 0; k < U; ++k) {
                site_energy<T>(cr, ci, ur, ui, dr[k], di[k], r1[k], i1[k], r2[k], i2[k], v[k], Jx,
                               Jy, eps0, rn[k], re[k]);
                ur = cr; ui = ci;
                cr = dr[k]; ci = di[k];
            }
            an.add((rn[0] + rn[1]) + (rn[2] + rn[3]));
            ae.add((re[0] + re[1]) + (re[2] + re[3]));
        }
        for (; y < y1; ++y) {
            double dr, di, r1, i1, r2, i2, v, rn = 0.0, re = 0.0;
            load_row(y, dr, di, r1, i1, r2, i2, v);
            site_energy<T>(cr, ci, ur, ui, dr, di, r1, i1, r2, i2, v, Jx, Jy, eps0, rn, re);
            an.add(rn);
            ae.add(re);
            ur = cr; ui = ci;
            cr = dr; ci = di;
        }
    }
    sn[threadIdx.x] = an.value();
    se[threadIdx.x] = ae.value();
    __syncthreads();
    for (int w = kReduceThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            sn[threadIdx.x] += sn[threadIdx.x + w];
            se[threadIdx.x] += se[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = sn[0];
        partial[2 * blockIdx.x + 1] = se[0];
    }
}

// Periodic meshes with an even number of columns: each lane owns two
// neighbouring columns (16-byte loads of psi and V per row, as the march
// issues), and the x-neighbours outside its pair come from the lanes beside
// it by a DPP wavefront shift; only the first and last lanes of a wavefront
// (and the last lane holding columns when the row ends inside the wavefront)
// load theirs.  Work items are (chunk of 2 * kReduceThreads columns, band of
// rows), walked as in observables_partial; fixed order, bitwise reproducible.
__device__ __forceinline__ double lane_from_left(double v) {
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x138 /* wave_shr:1 */, 0xF, 0xF, true);
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x138, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}
__device__ __forceinline__ double lane_from_right(double v) {
    const int hi = __builtin_amdgcn_update_dpp(0, __double2hiint(v), 0x130 /* wave_shl:1 */, 0xF, 0xF, true);
    const int lo = __builtin_amdgcn_update_dpp(0, __double2loint(v), 0x130, 0xF, 0xF, true);
    return __hiloint2double(hi, lo);
}

// psi of sites l and l+1 (l even): complex128 two 16-byte loads, complex64 one.
__device__ __forceinline__ void load_pair2(const void* psi, long long l, double (&re)[2],
                                           double (&im)[2], C128) {
    const double2* q = reinterpret_cast<const double2*>(psi) + l;
    const double2 a = q[0], b = q[1];
    re[0] = a.x; im[0] = a.y; re[1] = b.x; im[1] = b.y;
}
__device__ __forceinline__ void load_pair2(const void* psi, long long l, double (&re)[2],
                                           double (&im)[2], C64) {
    const float4 a = *reinterpret_cast<const float4*>(reinterpret_cast<const float2*>(psi) + l);
    re[0] = a.x; im[0] = a.y; re[1] = a.z; im[1] = a.w;
}

template <class T>
__global__ void __launch_bounds__(kReduceThreads)
observables_pairs(const void* __restrict__ psi, const double* __restrict__ V, int nx, int ny,
                  double Jx, double Jy, double eps0, int band, double* __restrict__ partial) {
    __shared__ double sn[kReduceThreads], se[kReduceThreads];
    constexpr int U = 4;  // rows per step of the walk
    constexpr int W = 2 * kReduceThreads;  // columns per chunk
    LongSum an, ae;
    const int lane = threadIdx.x & (kWaveSize - 1);
    const int chunks = (nx + W - 1) / W;
    const int bands = (ny + band - 1) / band;
    const long long items = (long long)chunks * bands;
    for (long long it = blockIdx.x; it < items; it += gridDim.x) {
        const int x0 = (int)(it % chunks) * W + 2 * (int)threadIdx.x;
        const int y0 = (int)(it / chunks) * band;
        const int y1 = min(y0 + band, ny);
        // every lane takes part in the shifts; lanes past the row load nothing
        const bool live = x0 < nx;
        const bool edge_l = lane == 0;
        const bool edge_r = lane == kWaveSize - 1 || x0 + 2 >= nx;
        const int xl = x0 == 0 ? nx - 1 : x0 - 1;
        const int xr = x0 + 2 >= nx ? 0 : x0 + 2;
        const int xc = live ? x0 : 0;
        auto load_pairs = [&](int y, double (&re)[2], double (&im)[2]) {
            re[0] = re[1] = im[0] = im[1] = 0.0;
            if (live) load_pair2(psi, (long long)y * nx + xc, re, im, T());
        };
        double ur[2], ui[2], cr[2], ci[2];
        load_pairs(y0 == 0 ? ny - 1 : y0 - 1, ur, ui);
        load_pairs(y0, cr, ci);
        // one row: the row below is loaded by the caller, V and the edge
        // neighbours of row y here
        auto row = [&](int y, const double (&dr)[2], const double (&di)[2], double2 v, double& rn,
                       double& re) {
            rn = re = 0.0;
            double lr = lane_from_left(cr[1]), li = lane_from_left(ci[1]);
            double rr = lane_from_right(cr[0]), ri = lane_from_right(ci[0]);
            if (live && edge_l) load_site(psi, (long long)y * nx + xl, lr, li, T());
            if (live && edge_r) load_site(psi, (long long)y * nx + xr, rr, ri, T());
            if (live) {
                site_energy<T>(cr[0], ci[0], ur[0], ui[0], dr[0], di[0], cr[1], ci[1], lr, li, v.x,
                               Jx, Jy, eps0, rn, re);
                site_energy<T>(cr[1], ci[1], ur[1], ui[1], dr[1], di[1], rr, ri, cr[0], ci[0], v.y,
                               Jx, Jy, eps0, rn, re);
            }
        };
        auto load_v = [&](int y) {
            return live ? *reinterpret_cast<const double2*>(V + (long long)y * nx + xc)
                        : make_double2(0.0, 0.0);
        };
        int y = y0;
        for (; y + U <= y1; y += U) {
            double dr[U][2], di[U][2];
            double2 v[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                load_pairs(y + k + 1 == ny ? 0 : y + k + 1, dr[k], di[k]);
                v[k] = load_v(y + k);
            }
            double rn[U], re[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                row(y + k, dr[k], di[k], v[k], rn[k], re[k]);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    ur[i] = cr[i]; ui[i] = ci[i];
                    cr[i] = dr[k][i]; ci[i] = di[k][i];
                }
            }
            an.add((rn[0] + rn[1]) + (rn[2] + rn[3]));
            ae.add((re[0] + re[1]) + (re[2] + re[3]));
        }
        for (; y < y1; ++y) {
            double dr[2], di[2], rn, re;
            load_pairs(y + 1 == ny ? 0 : y + 1, dr, di);
            row(y, dr, di, load_v(y), rn, re);
            an.add(rn);
            ae.add(re);
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                ur[i] = cr[i]; ui[i] = ci[i];
                cr[i] = dr[i]; ci[i] = di[i];
            }
        }
    }
    sn[threadIdx.x] = an.value();
    se[threadIdx.x] = ae.value();
    __syncthreads();
    for (int w = kReduceThreads / 2; w > 0; w >>= 1) {
        if ((int)threadIdx.x < w) {
            sn[threadIdx.x] += sn[threadIdx.x + w];
            se[threadIdx.x] += se[threadIdx.x + w];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = sn[0];
        partial[2 * blockIdx.x + 1] = se[0];
    }
}

// One block sums the partial sums, four loads in flight a thread: latency alone
// bounds it (256 threads with one load in flight took 8.9 us for 8192 partial
// sums; a call at 3000 x 2000, complex64, 59.4 then and 54.8 with this).
constexpr int kFinalThreads = 1024;
constexpr long long kObservableItems = 1024;  // least work items of a large 2D mesh's sums
__global__ void __launch_bounds__(kFinalThreads)
observables_final(const double2* __restrict__ partial, int nblocks, double* __restrict__ result) {
    __shared__ double sn[kFinalThreads / kWaveSize], se[kFinalThreads / kWaveSize];
    double an = 0.0, ae = 0.0;
    for (int b = threadIdx.x; b < nblocks; b += 4 * kFinalThreads) {
        double2 v[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const int i = b + k * kFinalThreads;
            v[k] = i < nblocks ? partial[i] : make_double2(0.0, 0.0);
        }
        an += (v[0].x + v[1].x) + (v[2].x + v[3].x);
        ae += (v[0].y + v[1].y) + (v[2].y + v[3].y);
    }
    const int lane = threadIdx.x & (kWaveSize - 1), wave = threadIdx.x / kWaveSize;
    for (int w = kWaveSize / 2; w > 0; w >>= 1) {
        an += __shfl_down(an, w);
        ae += __shfl_down(ae, w);
    }
    if (lane == 0) {
        sn[wave] = an;
        se[wave] = ae;
    }
    __syncthreads();
    // the wavefronts' sums as a tree too: one behind the other they round 16 times
    constexpr int kWaves = kFinalThreads / kWaveSize;
    if (wave > 0) return;
    an = lane < kWaves ? sn[lane] : 0.0;
    ae = lane < kWaves ? se[lane] : 0.0;
    for (int w = kWaves / 2; w > 0; w >>= 1) {
        an += __shfl_down(an, w);
        ae += __shfl_down(ae, w);
    }
    if (lane == 0) {
        result[0] = an;
        result[1] = an > 0.0 ? ae / an : 0.0;
    }
}

}  // namespace

hipError_t launch_phase_table(int dtype, const double* V, void* ptab, long long sites,
                              double dt, double eps0, double hbar, const TableScale& scale,
                              hipStream_t s) {
    const int threads = 256;
    // four sites a thread, their loads in flight together, once that leaves every
    // compute unit 8 blocks (a round of resident wavefronts); one a thread below,
    // where latency counts and the wavefronts hide it (one a thread up to 8192
    // blocks: two or three loads in turn at 4M sites and more)
    const long long round = 2048;
    long long want = (sites + threads - 1) / threads;
    want = want <= round ? want : std::max(round, (want + 3) / 4);
    const int blocks = (int)(want < 8192 ? want : 8192);
    if (dtype == 1 && scale.g_lo != 0.0)
        hipLaunchKernelGGL(phase_table_c128_two, dim3(blocks), dim3(threads), 0, s, V,
                           reinterpret_cast<double2*>(ptab), sites, dt, eps0, hbar, scale);
    else if (dtype == 1)
        hipLaunchKernelGGL(phase_table_c128, dim3(blocks), dim3(threads), 0, s, V,
                           reinterpret_cast<double2*>(ptab), sites, dt, eps0, hbar, scale);
    else
        hipLaunchKernelGGL(phase_table_c64, dim3(blocks), dim3(threads), 0, s, V,
                           reinterpret_cast<int2*>(ptab), sites, dt, eps0, hbar, scale);
    return hipGetLastError();
}

hipError_t launch_td_table(const double* V0, const double* W, void* table, void* turns,
                           long long sites, double dt, double eps0, double hbar, double scale,
                           hipStream_t s) {
    const int threads = 256;
    long long want = (sites + threads - 1) / threads;
    const int blocks = (int)(want < 8192 ? want : 8192);
    hipLaunchKernelGGL(td_table, dim3(blocks), dim3(threads), 0, s, V0, W,
                       reinterpret_cast<double2*>(table), sites, dt, eps0, hbar);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(td_turns, dim3((kTurns + 255) / 256), dim3(256), 0, s,
                       reinterpret_cast<double2*>(turns), scale);
    return hipGetLastError();
}

hipError_t launch_observables_final(const double* partial, int nblocks, double* result,
                                    hipStream_t s) {
    hipLaunchKernelGGL(observables_final, dim3(1), dim3(kFinalThreads), 0, s,
                       reinterpret_cast<const double2*>(partial), nblocks, result);
    return hipGetLastError();
}

hipError_t launch_observables(int dtype, const void* psi, const double* V, int nx, int ny,
                              double Jx, double Jy, double eps0, bool closed, double* partial,
                              int nblocks, double* result, hipStream_t s) {
    const int cl = closed ? 1 : 0;
    // periodic meshes (even sides) with 16-byte aligned psi and V take the
    // two-column kernel
    const bool aligned = reinterpret_cast<uintptr_t>(psi) % 16 == 0 &&
                         reinterpret_cast<uintptr_t>(V) % 16 == 0;
    const bool pairs = !closed && (nx % 2) == 0 && aligned;
    const int width = pairs ? 2 * kReduceThreads : kReduceThreads;
    // bands of rows sized so there are about kObservableItems work items: 4 blocks a
    // compute unit.  More give bands of a few rows, which read half as many rows
    // again at their edges and never reach the walk of four.  A call, us, with 8192
    // | 4096 | 2048 | 1024 items: complex64 3000 x 2000 54.8 | 52.4 | 51.6 | 49.3,
    // 200 x 8000 47.4 | 42.1 | 37.6 | 35.9, 16384 x 8192 515 | 518 | 508 | 499;
    // complex128 4096^2 98 | 102 | 100 | 102, 16384 x 8192 656 | 655 | 640 | 566.  Bands
    // of more than 256 rows only past `nblocks` items: 32768^2 complex64 takes 3.4 ms
    // at 256 rows (8192 items) and 4.15 at 2048, whose blocks are far apart in memory.
    const long long chunks = (nx + width - 1) / width;
    long long bands = std::max(kObservableItems / chunks,
                               std::min(nblocks / chunks, (long long)(ny + 255) / 256));
    if (bands < 1) bands = 1;
    if (bands > ny) bands = ny;
    const int band = (int)((ny + bands - 1) / bands);
    const long long items = chunks * ((ny + band - 1) / band);
    if (items < nblocks) nblocks = (int)items;
    if (pairs && dtype == 1)
        hipLaunchKernelGGL(observables_pairs<C128>, dim3(nblocks), dim3(kReduceThreads), 0, s,
                           psi, V, nx, ny, Jx, Jy, eps0, band, partial);
    else if (pairs)
        hipLaunchKernelGGL(observables_pairs<C64>, dim3(nblocks), dim3(kReduceThreads), 0, s,
                           psi, V, nx, ny, Jx, Jy, eps0, band, partial);
    else if (dtype == 1)
        hipLaunchKernelGGL(observables_partial<C128>, dim3(nblocks), dim3(kReduceThreads), 0, s,
                           psi, V, nx, ny, Jx, Jy, eps0, cl, band, partial);
    else
        hipLaunchKernelGGL(observables_partial<C64>, dim3(nblocks), dim3(kReduceThreads), 0, s,
                           psi, V, nx, ny, Jx, Jy, eps0, cl, band, partial);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(observables_final, dim3(1), dim3(kFinalThreads), 0, s,
                       reinterpret_cast<const double2*>(partial), nblocks, result);
    return hipGetLastError();
}

}  // namespace tsq

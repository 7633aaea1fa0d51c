// fvna3d.hip -- the three-dimensional step (the paper's equations in three
// dimensions, which Sec. 5 says they allow) and its C ABI (include/fvna3d.h).
//
// State (R, M1, M2, M3) = (rho'/rho0, rho u1/(rho0 c0), ...), dimensionless
// with the mesh spacing as length unit.  One step: x1 sweep -> x2 sweep ->
// x3 sweep -> source (Godunov splitting, each sweep the high-resolution Roe
// scheme of Secs. 3.1-3.2 with a second passive shear wave), then the CFL
// decision of the opening of Sec. 4, all on the device:
//   k3_sweep12  x1 and x2 sweeps of one z-plane tile: lanes along x1 (the
//               left cell, the neighbour waves and the right flux over DPP
//               lane shifts, every x1 interface solved once), a register
//               march along x2 (every x2 interface solved once);
//   k3_sweep3s  x3 sweep and source of one x1-x2 tile: every thread marches
//               one column along x3 in registers, and the velocities of the
//               swept planes meet in LDS for the 7-point Laplacian.
// Three state buffers X0, X1, X2 and the device clock's cur = c in {0, 1}: the
// state's density is in X[1-c] and its momenta in X[c]; the x1-x2 sweep writes
// all four fields to X2, and the second kernel writes the new state into the
// planes the old one does not use (density X[c], momenta X[1-c]).  An accepted
// step flips c; a rejected one leaves the current state untouched.  The
// decision on an attempt (accept or reject, the next time step) is taken in
// the prologues of the attempt after it, as in two dimensions (step_begin).
// Steps are replayed from a captured HIP graph; the host waits once per
// fvna3_step call.
// Ghost values follow the side rule of their axis applied to the state of
// the stage that needs them (Q^n for x1, the x1-swept state for x2, the
// x2-swept state for x3, the x3-swept state for the source).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <string>

#include "../../include/fvna3d.h"
#include "fvna_device.hpp"
#include "fvna_reply.hpp"
#include "fvna_step.hpp"

using namespace fvna;

namespace {

constexpr int HALO12 = 2;                      // x1 stencil: two interfaces each side
constexpr int OUT12 = WAVE - 2 * HALO12;       // 60 output columns per x1-x2 wavefront

// Buffer roles for clock cur = c (see the file's header).
__device__ __forceinline__ int buf_rho(int c) { return c ^ 1; }
__device__ __forceinline__ int buf_mom(int c) { return c; }
constexpr int BUF_X12 = 2;

struct Desc3 {
    int n[3];                  // nx, ny, nz
    int pitch;                 // elements per x1 row (padded to 256 bytes)
    int strips12, segs12, rows12;   // x1-x2 tiles: 60-column strips, row segments of rows12
    int tailw12, tailp12, tailk12;  // packed tail (tailw12 > 0): the last nx mod 60 columns of
                                    // tailp12 planes per wavefront, lanes in segments of
                                    // tailw12 = that + 4; tailk12 plane groups
    int bx, by, ntx, nty;           // x3 and source tiles: bx x by threads, (bx - 2) x (by - 2)
                                    // columns of output, ntx x nty tiles
    int segs3, planes3;             // their z segments of planes3
    long long plane;           // elements per field = pitch * ny * nz
    int bc[6];
    int fixed_dt, max_retries;
    double beta, delta;        // delta~ = delta / (c0 dx)
    double cfl_target, cfl_max;
    void* buf[3];
    Clock* clk;
};

// Index m along axis a mapped to a stored index by the side rule of that
// axis; *neg is set when the momentum normal to the axis is mirrored.
__device__ __forceinline__ int side_map(const Desc3& d, int a, int m, bool& neg)
{
    const int n = d.n[a];
    neg = false;
    if (m < 0) {
        const int b = d.bc[2 * a];
        if (b == FVNA_BC_PERIODIC) m += n;
        else if (b == FVNA_BC_REFLECT) { m = -m - 1; neg = true; }
        else m = 0;
    } else if (m >= n) {
        const int b = d.bc[2 * a + 1];
        if (b == FVNA_BC_PERIODIC) m -= n;
        else if (b == FVNA_BC_REFLECT) { m = 2 * n - m - 1; neg = true; }
        else m = n - 1;
    }
    return min(max(m, 0), n - 1);
}

// ---------------------------------------------------------------------------
// Roe solver of one interface with two tangential momenta (a, b).
// ---------------------------------------------------------------------------
template <typename T> struct W4 { T s1, s2, s3, a1, a2, a3, a4, r1a, r2a, r1b, r2b; };
template <typename T> struct Q4 { T R, n, a, b; };

// Eigenvalues w + c, w - c, w, w; acoustic eigenvectors (1, s, ra, rb) with
// ra = za (s - 2 zn)/(Zbar^1 (s - w)) (likewise rb), shear eigenvectors
// (0, 0, 1, 0) and (0, 0, 0, 1); strengths from sum_p alpha^p r^p = Q_R - Q_L.
// The means are carried as sums of the two sides (every factor 2 cancels).
// Returns the interface's largest |s| in the form Cfl<T> reduces (FP32 as an
// excess over 1), the discriminant in D, and in parted whether |w| < c (roe_sh).
// h = 1/(2 + L.R + R.R) comes from the caller (rcp_pair).
template <typename T>
__device__ __forceinline__ T roe4(const Q4<T>& L, T unL, T uaL, T ubL, const Q4<T>& R, T unR, T uaR, T ubR,
                                  T beta, T h, W4<T>& w, T& D, bool& parted)
{
    const T Sr = L.R + R.R, Sn = unL + unR, Sa = uaL + uaR, Sb = ubL + ubR;
    const T wv = Sn * h;
    const T D1 = fma_(wv, wv - Sn, (beta - T(1)) * Sr);
    D = T(1) + D1;
    T c, ic;
    sqrt_pair(D, c, ic);
    T spd;
    if constexpr (sizeof(T) == 8) spd = c + abs_(wv);
    else spd = fma_(D1, rcp(T(1) + c), abs_(wv));
    parted = abs_(wv) < c;
    w.s1 = wv + c;
    w.s2 = wv - c;
    w.s3 = wv;
    const T hic = h * ic;
    const T ka = Sa * hic, kb = Sb * hic;
    const T e1 = w.s1 - Sn, e2 = w.s2 - Sn;
    w.r1a = ka * e1;
    w.r2a = -ka * e2;
    w.r1b = kb * e1;
    w.r2b = -kb * e2;
    const T d1 = R.R - L.R, d2 = R.n - L.n, d3 = R.a - L.a, d4 = R.b - L.b;
    w.a1 = T(0.5) * ic * fma_(-w.s2, d1, d2);
    w.a2 = d1 - w.a1;
    w.a3 = fma_(-w.a2, w.r2a, fma_(-w.a1, w.r1a, d3));
    w.a4 = fma_(-w.a2, w.r2b, fma_(-w.a1, w.r1b, d4));
    return spd;
}

// Upwind values of two neighbouring interfaces x (below) and y (above) for
// each other, as wave_cross in two dimensions: tx = alpha_x X for y, ty =
// alpha_y X for x, X = r^p_x . r^p_y for the acoustic families (entries 0, 1);
// entries 2, 3: the shear strengths alpha^3, alpha^4 (X = 1).
template <typename T>
__device__ __forceinline__ void cross4(const W4<T>& x, const W4<T>& y, T tx[4], T ty[4])
{
    const T x1 = fma_(x.r1b, y.r1b, fma_(x.r1a, y.r1a, fma_(x.s1, y.s1, T(1))));
    const T x2 = fma_(x.r2b, y.r2b, fma_(x.r2a, y.r2a, fma_(x.s2, y.s2, T(1))));
    tx[0] = x.a1 * x1; tx[1] = x.a2 * x2; tx[2] = x.a3; tx[3] = x.a4;
    ty[0] = y.a1 * x1; ty[1] = y.a2 * x2; ty[2] = y.a3; ty[3] = y.a4;
}

// Fluctuations plus limited corrections of one interface (eqs. fluc:m,
// fluc:p, limiter, fv-hr): Gm = A^- dQ + F~ for the cell on the low side,
// Gp = A^+ dQ - F~ for the cell on the high side.  lo/hi: upwind values t of
// the interface below/above (cross4).  The upwind interface is the one below
// for s >= 0.  The limited products and PARTED as in two dimensions (hr_split):
// FP64 from u = t / n with one reciprocal of n1 n2, FP32 from
// theta = t / (alpha n).
template <bool PARTED, typename T>
__device__ __forceinline__ void hr_split4(const W4<T>& w, const T lo[4], const T hi[4], T dt, T Gm[4], T Gp[4])
{
    const bool n3 = w.s3 < T(0);
    const T t1 = PARTED ? lo[0] : w.s1 < T(0) ? hi[0] : lo[0], t2 = PARTED ? hi[1] : w.s2 < T(0) ? hi[1] : lo[1];
    const T t3 = n3 ? hi[2] : lo[2], t4 = n3 ? hi[3] : lo[3];
    const T q1 = fma_(w.r1b, w.r1b, fma_(w.r1a, w.r1a, fma_(w.s1, w.s1, T(1))));
    const T q2 = fma_(w.r2b, w.r2b, fma_(w.r2a, w.r2a, fma_(w.s2, w.s2, T(1))));
    const T as1 = abs_(w.s1), as2 = abs_(w.s2), as3 = abs_(w.s3);
    T c1, c2, c3, c4;
    if constexpr (sizeof(T) == 8) {
        const T ip = rcp(q1 * q2);
        const T hdt = T(-0.5) * dt;
        const T f3 = fma_(hdt, as3, T(0.5)) * as3;
        c1 = (fma_(hdt, as1, T(0.5)) * as1) * mc_scaled(w.a1, t1 * (ip * q2));
        c2 = (fma_(hdt, as2, T(0.5)) * as2) * mc_scaled(w.a2, t2 * (ip * q1));
        c3 = f3 * mc_scaled(w.a3, t3);
        c4 = f3 * mc_scaled(w.a4, t4);
    } else {
        const T f3 = fma_(-dt, as3, T(1)) * as3;
        c1 = (fma_(-dt, as1, T(1)) * as1) * (mc_half(t1 * rcp(w.a1 * q1)) * w.a1);
        c2 = (fma_(-dt, as2, T(1)) * as2) * (mc_half(t2 * rcp(w.a2 * q2)) * w.a2);
        c3 = f3 * mc_unit(w.a3, t3);
        c4 = f3 * mc_unit(w.a4, t4);
    }
    const T m3 = min_(w.s3, T(0));
    const T e1 = PARTED ? c1 : fma_(min_(w.s1, T(0)), w.a1, c1);
    const T e2 = fma_(PARTED ? w.s2 : min_(w.s2, T(0)), w.a2, c2);
    const T e3 = fma_(m3, w.a3, c3);
    const T e4 = fma_(m3, w.a4, c4);
    const T g1 = fma_(w.s1, w.a1, -e1);
    const T g2 = fma_(w.s2, w.a2, -e2);
    const T g3 = fma_(w.s3, w.a3, -e3);
    const T g4 = fma_(w.s3, w.a4, -e4);
    Gm[0] = e1 + e2;
    Gm[1] = fma_(e1, w.s1, e2 * w.s2);
    Gm[2] = fma_(e1, w.r1a, fma_(e2, w.r2a, e3));
    Gm[3] = fma_(e1, w.r1b, fma_(e2, w.r2b, e4));
    Gp[0] = g1 + g2;
    Gp[1] = fma_(g1, w.s1, g2 * w.s2);
    Gp[2] = fma_(g1, w.r1a, fma_(g2, w.r2a, g3));
    Gp[3] = fma_(g1, w.r1b, fma_(g2, w.r2b, g4));
}

// State carried by a register march from one cell of the marching axis to
// the next (split-local components: R, normal, tangential a, tangential b).
template <typename T> struct March4 {
    Q4<T> q; T un, ua, ub;     // last cell pushed and its velocities
    W4<T> w;                   // interface below it
    bool parted;               // hr_split's PARTED holds there in every lane
    T lo[4];                   // upwind values t of the interface below it for it (cross4)
    Q4<T> part;                // previous cell minus dt Gp of its lower interface (awaiting its upper flux)
};

template <typename T>
__device__ __forceinline__ void march_zero(March4<T>& m)
{
    const T z = T(0);
    m.q = {z, z, z, z};
    m.un = m.ua = m.ub = z;
    m.w = {z, z, z, z, z, z, z, z, z, z, z};
    m.parted = false;
    m.lo[0] = m.lo[1] = m.lo[2] = m.lo[3] = z;
    m.part = {z, z, z, z};
}

// Push cell v (split-local q) through a march: solve interface v - 1/2,
// correct interface v - 3/2, and return cell v - 2 completed in `done`.
// Adds the speed of interface v - 1/2 to acc when `count`.
template <typename T>
__device__ __forceinline__ void march_push(const Q4<T>& q, const March4<T>& in, March4<T>& out, T beta, T dt,
                                           bool count, Cfl<T>& acc, Q4<T>& done)
{
    T ir, h;
    rcp_pair(T(1) + q.R, T(2) + (in.q.R + q.R), ir, h);
    ir = rcp_polish(T(1) + q.R, ir);
    const T un = q.n * ir, ua = q.a * ir, ub = q.b * ir;
    W4<T> wA;
    T D;
    bool parted;
    const T spd = roe4(in.q, in.un, in.ua, in.ub, q, un, ua, ub, beta, h, wA, D, parted);
    out.parted = all_lanes(parted);
    if (count) {
        if (__builtin_expect(out.parted, 1)) acc.add(spd);
        else acc.add(spd, D);
    }
    T tup[4], hi[4];
    cross4(in.w, wA, tup, hi);
    T Gm[4], Gp[4];
    if (__builtin_expect(in.parted, 1)) hr_split4<true>(in.w, in.lo, hi, dt, Gm, Gp);
    else hr_split4<false>(in.w, in.lo, hi, dt, Gm, Gp);
    done.R = fma_(-dt, Gm[0], in.part.R);
    done.n = fma_(-dt, Gm[1], in.part.n);
    done.a = fma_(-dt, Gm[2], in.part.a);
    done.b = fma_(-dt, Gm[3], in.part.b);
    out.part.R = fma_(-dt, Gp[0], in.q.R);
    out.part.n = fma_(-dt, Gp[1], in.q.n);
    out.part.a = fma_(-dt, Gp[2], in.q.a);
    out.part.b = fma_(-dt, Gp[3], in.q.b);
    out.q = q;
    out.un = un; out.ua = ua; out.ub = ub;
    out.w = wA;
    out.lo[0] = tup[0];
    out.lo[1] = tup[1];
    out.lo[2] = tup[2];
    out.lo[3] = tup[3];
}

// Wait for the loads of q here.  Loads and stores share one in-order counter,
// and after stores under a condition the compiler can only wait for a load by
// waiting for all but as many newer operations as are certain to have been
// issued: for the loads two rows ahead as well, the whole latency on every row.
// Placed ahead of a row's stores, the wait is for the next row's loads only.
template <typename T>
__device__ __forceinline__ void wait_loads(Q4<T>& q)
{
    asm volatile("" : "+v"(q.R), "+v"(q.n), "+v"(q.a), "+v"(q.b));
}

// Fold a block's CFL bookkeeping into the attempt's slot: over the wavefront,
// then in LDS (sh: two words per wavefront) over the block.  Every thread of the
// block calls it, after its last use of sh.
template <typename T>
__device__ __forceinline__ void cfl_commit(const Attempt& at, const Cfl<T>& acc, bool counted, T* sh)
{
    T m;
    bool nh, nf;
    acc.finish(counted, m, nh, nf);
    const int lane = threadIdx.x & (WAVE - 1), wave = threadIdx.x / WAVE, waves = blockDim.x / WAVE;
    for (int off = 32; off >= 1; off >>= 1) m = max_(m, perm(m, lane ^ off));
    const bool anyh = __any(nh), anyf = __any(nf);
    __syncthreads();
    if (lane == 0) {
        sh[2 * wave] = m;
        sh[2 * wave + 1] = (anyh ? T(1) : T(0)) + (anyf ? T(2) : T(0));
    }
    __syncthreads();
    if (threadIdx.x != 0) return;
    int fl = 0;
    for (int k = 0; k < waves; ++k) {
        m = max_(m, sh[2 * k]);
        fl |= (int)sh[2 * k + 1];
    }
    cfl_raise(at, cfl_speed<T>(m), (fl & 1) != 0, (fl & 2) != 0);
}

// ---------------------------------------------------------------------------
// x1 and x2 sweeps of one tile: 64 lanes over columns c0 - 2 .. c0 + 61 (the
// 60 outputs in lanes 2..61), rows r0 .. r1 - 1 of plane k.  Rows r0 - 2 ..
// r1 + 1 go through the x1 sweep and the x2 march; a row outside the grid is
// the x1 sweep of the row its side rule names (mirrored rows with M2
// negated), which is the side rule applied to the x1-swept state.
//
// Packed tail: the last nx mod 60 columns (rem) would fill a 60-column strip
// only in part (256 columns: 16 of 60).  Their tiles instead pack tailp12
// planes into one wavefront: lane segments of w = rem + 4 lanes, segment s
// holding columns c0 - 2 .. c0 + rem + 1 of plane kg tailp12 + s (a full
// strip is the case of one 64-lane segment, sweep12_lanes).  The lane shifts
// run across segment ends; what crosses them reaches only the two end lanes
// of a segment, which are its halo, exactly as at the ends of a full strip.
// Lanes of no segment or past the last plane read a real cell and store and
// count nothing.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void sweep12_lanes(const Desc3& d, int tile, int& seg, int& k, int& col, int& loc,
                                              int& w, bool& lane_ok)
{
    const int lane = threadIdx.x & (WAVE - 1);
    const int nfull = d.strips12 * d.segs12 * d.n[2];
    int c0, k0, np;
    if (tile < nfull) {
        const int strip = tile % d.strips12;
        seg = (tile / d.strips12) % d.segs12;
        k0 = tile / (d.strips12 * d.segs12);
        c0 = strip * OUT12;
        w = WAVE;
        np = 1;
    } else {
        const int t = tile - nfull;
        seg = t % d.segs12;
        k0 = (t / d.segs12) * d.tailp12;
        c0 = d.strips12 * OUT12;
        w = d.tailw12;
        np = d.tailp12;
    }
    const int sgm = lane / w;
    loc = lane - sgm * w;
    const int kk = k0 + sgm;
    lane_ok = sgm < np && kk < d.n[2];
    k = lane_ok ? kk : d.n[2] - 1;
    col = c0 - HALO12 + loc;
}

// The wavefronts of a block raise as one: each leaves its values in LDS and the
// last to come raises the attempt's (no barrier: they end when they end).  The
// wavefronts of a launch whose tiles are all equally tall end together, read the
// word before any has raised it, and wait for one another's atomics after all.
// us per step with each for itself / by blocks: 224 x 100 x 40 FP32 in
// 10-row tiles 54.6 / 45.0 (11-row tiles, the last of a plane shorter: 45.6 /
// 45.7), 128^3 FP32 in 8-row tiles 78.1 / 65.2, 90 x 75 x 64 FP64 in 5-row tiles
// 48.1 / 41.0.  (Not for the two-dimensional march, whose first and last segments
// end early: 1319 x 813 FP64 39.1 / 40.5, 4096^2 level.)
struct BlockCfl { unsigned long long smax; unsigned int flags, left; };

// By every thread of the block, before its wavefronts part; n of them will raise.
__device__ __forceinline__ void block_cfl_init(BlockCfl& b, int n)
{
    if (threadIdx.x == 0) { b.smax = 0ull; b.flags = 0u; b.left = (unsigned)n; }
    __syncthreads();
}

__device__ __forceinline__ void cfl_raise_block(const Attempt& at, BlockCfl& b, double speed, bool nonhyp, bool nonfin)
{
    atomicMax(&b.smax, (unsigned long long)__double_as_longlong(speed));
    const unsigned fl = (nonhyp ? FLAG_NONHYP : 0u) | (nonfin ? FLAG_NONFINITE : 0u);
    if (fl) atomicOr(&b.flags, fl);
    __threadfence_block();
    if (atomicSub(&b.left, 1u) != 1u) return;
    __threadfence_block();
    const unsigned all = atomicOr(&b.flags, 0u);
    cfl_raise(at, __longlong_as_double((long long)atomicMax(&b.smax, 0ull)), (all & FLAG_NONHYP) != 0,
              (all & FLAG_NONFINITE) != 0);
}

template <typename T>
__device__ __forceinline__ void sweep12_tile(const Desc3& d, int tile, const Attempt& at, BlockCfl& cfl)
{
    const int nx = d.n[0], ny = d.n[1];
    const int lane = threadIdx.x & (WAVE - 1);
    int seg, k, col, loc, w;
    bool lane_ok;
    sweep12_lanes(d, tile, seg, k, col, loc, w, lane_ok);
    const int r0 = seg * d.rows12, r1 = min(r0 + d.rows12, ny);
    const T dt = (T)at.dt;
    const T* inR = (const T*)d.buf[buf_rho(at.cur)];
    const T* inM = (const T*)d.buf[buf_mom(at.cur)];
    T* out = (T*)d.buf[BUF_X12];
    const T beta = (T)d.beta;
    const bool perx = d.bc[0] == FVNA_BC_PERIODIC, pery = d.bc[2] == FVNA_BC_PERIODIC;
    bool xneg;
    const int scol = side_map(d, 0, col, xneg);
    const T xs = xneg ? T(-1) : T(1);
    const size_t pl = (size_t)d.plane;
    const size_t zoff = (size_t)k * (size_t)ny * (size_t)d.pitch;
    const bool out_lane = lane_ok && loc >= HALO12 && loc < w - HALO12 && col < nx;
    Cfl<T> xacc, yacc;

    // x1 sweep of stored row sr (lane-parallel), components (R, M1, M2, M3)
    // raw Q^n of the row that row v stands for (side rule along x2)
    // this lane's plane and column, fixed over the march (the row offset
    // added per row is the same for every lane)
    const T* __restrict__ inR_l = inR + (zoff + (size_t)scol);
    const T* __restrict__ inM_l = inM + (zoff + (size_t)scol);
    T* __restrict__ out_l = out + (zoff + (size_t)(out_lane ? col : 0));
    auto load_row = [&](int v) -> Q4<T> {
        bool yneg;
        const int sr = side_map(d, 1, v, yneg);
        const size_t ro = (size_t)sr * (size_t)d.pitch;
        const T* m = inM_l + ro;
        return Q4<T>{inR_l[ro], m[pl], m[2 * pl], m[3 * pl]};
    };
    auto xsweep = [&](Q4<T> q) -> Q4<T> {
        q.n = xs * q.n;
        Q4<T> L;
        L.R = from_lo(q.R);
        T ir, h;
        rcp_pair(T(1) + q.R, T(2) + (L.R + q.R), ir, h);
        ir = rcp_polish(T(1) + q.R, ir);           // the first lane's left cell is another plane's in a packed tail
        const T un = q.n * ir, ua = q.a * ir, ub = q.b * ir;
        L.n = from_lo(q.n); L.a = from_lo(q.a); L.b = from_lo(q.b);
        const T unL = from_lo(un), uaL = from_lo(ua), ubL = from_lo(ub);
        W4<T> wv;
        T D;
        bool parted;
        const T spd = roe4(L, unL, uaL, ubL, q, un, ua, ub, beta, h, wv, D, parted);
        T hi[4], lo[4], Gm[4], Gp[4];
        if (__builtin_expect(all_lanes(parted), 1)) {
            xacc.add(spd);
            // family 1 meets the interface to the left, family 2 the one to the right
            const T x1 = fma_(from_lo(wv.r1b), wv.r1b,
                              fma_(from_lo(wv.r1a), wv.r1a, fma_(from_lo(wv.s1), wv.s1, T(1))));
            const T x2 = fma_(wv.r2b, from_hi(wv.r2b),
                              fma_(wv.r2a, from_hi(wv.r2a), fma_(wv.s2, from_hi(wv.s2), T(1))));
            lo[0] = from_lo(wv.a1) * x1;
            hi[1] = from_hi(wv.a2) * x2;
            lo[2] = from_lo(wv.a3); hi[2] = from_hi(wv.a3);
            lo[3] = from_lo(wv.a4); hi[3] = from_hi(wv.a4);
            hr_split4<true>(wv, lo, hi, dt, Gm, Gp);
        } else {
            xacc.add(spd, D);
            W4<T> wr;
            wr.a1 = from_hi(wv.a1); wr.s1 = from_hi(wv.s1); wr.r1a = from_hi(wv.r1a); wr.r1b = from_hi(wv.r1b);
            wr.a2 = from_hi(wv.a2); wr.s2 = from_hi(wv.s2); wr.r2a = from_hi(wv.r2a); wr.r2b = from_hi(wv.r2b);
            wr.a3 = from_hi(wv.a3);
            wr.a4 = from_hi(wv.a4);
            T tup[4];
            cross4(wv, wr, tup, hi);
            lo[0] = from_lo(tup[0]); lo[1] = from_lo(tup[1]); lo[2] = from_lo(tup[2]); lo[3] = from_lo(tup[3]);
            hr_split4<false>(wv, lo, hi, dt, Gm, Gp);
        }
        Q4<T> o2;
        o2.R = fma_(-dt, from_hi(Gm[0]) + Gp[0], q.R);
        o2.n = fma_(-dt, from_hi(Gm[1]) + Gp[1], q.n);
        o2.a = fma_(-dt, from_hi(Gm[2]) + Gp[2], q.a);
        o2.b = fma_(-dt, from_hi(Gm[3]) + Gp[3], q.b);
        return o2;
    };

    // x2 march over rows v = r0 - 2 .. r1 + 1; components (R, M2, M1, M3)
    March4<T> A, B;
    march_zero(A);
    const int v0 = r0 - HALO12, v1 = r1 + HALO12;
    auto step_row = [&](int v, const Q4<T>& raw, Q4<T>& next, const March4<T>& mi, March4<T>& mo) {
        bool yneg;
        (void)side_map(d, 1, v, yneg);
        const Q4<T> x = xsweep(raw);
        Q4<T> q;                                   // split-local for x2: normal = M2
        q.R = x.R;
        q.n = yneg ? -x.a : x.a;
        q.a = x.n;
        q.b = x.b;
        const bool cnt = v > v0 && (pery || (v >= 0 && v <= ny));
        Q4<T> dn;
        march_push(q, mi, mo, beta, dt, cnt, yacc, dn);
        wait_loads(next);
        const int j = v - 2;
        if (j >= r0 && out_lane) {
            T* o = out_l + (size_t)j * (size_t)d.pitch;
            o[0] = dn.R;
            o[pl] = dn.a;
            o[2 * pl] = dn.n;
            o[3 * pl] = dn.b;
        }
    };
    // two rows of loads in flight ahead of the row being swept (rows past
    // v1 - 1 are clamped by the side rule and never used)
    Q4<T> p0 = load_row(v0), p1 = load_row(v0 + 1);
    wait_loads(p0);
    int v = v0;
#pragma unroll 1
    for (; v + 1 < v1; v += 2) {
        Q4<T> r = p0;
        p0 = load_row(v + 2);
        step_row(v, r, p1, A, B);
        r = p1;
        p1 = load_row(v + 3);
        step_row(v + 1, r, p0, B, A);
    }
    if (v < v1) step_row(v, p0, p1, A, B);

    // x1 interfaces: a lane's lies between columns col - 1 and col (the
    // first lane of a segment has no left neighbour); x2 interfaces: lanes
    // with exact x1-swept values
    const bool real_col = perx || (col >= 0 && col < nx);
    const bool cnt_x = lane_ok && loc >= 1 && (perx || (col >= 0 && col <= nx));
    const bool cnt_y = lane_ok && loc >= HALO12 && loc < w - HALO12 && real_col;
    T sx, sy;
    bool hx, hy, fx, fy;
    xacc.finish(cnt_x, sx, hx, fx);
    yacc.finish(cnt_y, sy, hy, fy);
    T m = max_(sx, sy);
    for (int off = 32; off >= 1; off >>= 1) m = max_(m, perm(m, lane ^ off));
    const bool anyh = __any(hx || hy), anyf = __any(fx || fy);
    if (lane == 0) cfl_raise_block(at, cfl, cfl_speed<T>(m), anyh, anyf);
}

template <typename T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(Occupancy<T>::waves)))
void k3_sweep12(Desc3 d, int force, int pos, long long owed)
{
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int first = xcd_block(blockIdx.x, gridDim.x) * WAVES_PER_BLOCK, tile = first + wave;
    const int tiles = (d.strips12 * d.n[2] + d.tailk12) * d.segs12;
    __shared__ BlockCfl cfl;
    block_cfl_init(cfl, min(WAVES_PER_BLOCK, tiles - first));
    if (tile >= tiles) return;
    pos = max(pos, 0);
    Attempt at;
    if (step_begin(d, force, pos, owed, at)) sweep12_tile<T>(d, tile, at, cfl);
    if (tile == 0 && (threadIdx.x & (WAVE - 1)) == 0) step_end(d, pos, owed);
}

// ---------------------------------------------------------------------------
// x3 sweep and source (3-D form of eq. fs:source, forward Euler: M_c += dt
// delta~ lap(u_c), 7-point Laplacian of u_c = M_c / (1 + R)) in one pass.
//
// A block takes a tile of bx x by columns (thread t: row t / bx, column t mod
// bx, the outermost ones halo) and a segment of planes k0 .. k1 - 1.  Every
// thread marches its column through the x3 sweep in registers; planes k0 - 3 ..
// k1 + 2 are pushed (outside the grid by the x3 side rule applied to the
// x2-swept state), which completes planes k0 - 1 .. k1.  A completed plane's
// velocities go to LDS, and one plane later, when the plane above is known
// too, each thread finds its x1 and x2 neighbours there: the halo threads hold
// the neighbour columns, or by the side rule the ghosts (mirrored normal
// velocity).  Two LDS planes and one barrier per plane: neighbours are read
// before the barrier of the iteration that publishes the next plane.
//
// The two separate kernels this replaces moved the state over HBM twice
// (256^3, one step: x3 sweep 129 us and source 124 us FP32, both at 4.3 TB/s,
// 206 and 239 us FP64); here the swept state never leaves the CU, at the price
// of marching the halo columns (15 to 25% of the threads) and two more planes
// per segment.
// ---------------------------------------------------------------------------
template <typename T> struct Vel { T u1, u2, u3; };

// Threads of a block: FP32 four wavefronts per SIMD, FP64 two.
template <typename T> struct Sweep3 { static constexpr int threads = sizeof(T) == 8 ? 512 : 1024; };

template <typename T>
__global__ __launch_bounds__(Sweep3<T>::threads) void k3_sweep3s(Desc3 d, int force, int pos, long long owed)
{
    constexpr int N = Sweep3<T>::threads;
    __shared__ T ys[2][3][N];                          // [plane parity][component][thread]
    Attempt at;
    // the whole block: the same words
    if (!step_again(d, force, max(pos, 0), owed, at)) return;
    const int b = xcd_block(blockIdx.x, gridDim.x);
    const int tx = b % d.ntx, ty = (b / d.ntx) % d.nty, seg = b / (d.ntx * d.nty);
    const int nx = d.n[0], ny = d.n[1], nz = d.n[2];
    const int t = threadIdx.x, bx = d.bx, by = d.by;
    const int row = t / bx, cx = t - row * bx;
    const int gx = tx * (bx - 2) - 1 + cx, gy = ty * (by - 2) - 1 + row;
    bool xneg, yneg;
    const int sx = side_map(d, 0, gx, xneg), sy = side_map(d, 1, gy, yneg);
    const bool real = row < by && gx >= 0 && gx < nx && gy >= 0 && gy < ny;
    const bool out = real && cx >= 1 && cx < bx - 1 && row >= 1 && row < by - 1;
    const int k0 = seg * d.planes3, k1 = min(k0 + d.planes3, nz);
    const T dt = (T)at.dt, beta = (T)d.beta;
    const T kd = dt * (T)d.delta;
    const bool perz = d.bc[4] == FVNA_BC_PERIODIC;
    const size_t pl = (size_t)d.plane;
    const size_t zstride = (size_t)ny * (size_t)d.pitch;
    const T* __restrict__ in = (const T*)d.buf[BUF_X12];
    T* __restrict__ outR = (T*)d.buf[buf_rho(at.cur ^ 1)];
    T* __restrict__ outM = (T*)d.buf[buf_mom(at.cur ^ 1)];
    const unsigned cell = (unsigned)sy * (unsigned)d.pitch + (unsigned)sx;      // within a plane
    Cfl<T> acc;
    March4<T> A, B;
    march_zero(A);
    const int v0 = k0 - 3, v1 = k1 + 3;
    // raw x2-swept cell of the plane that plane v stands for, split-local for
    // x3 (normal = M3), the mirror applied
    auto load_plane = [&](int v) -> Q4<T> {
        bool zneg;
        const T* p = in + (size_t)side_map(d, 2, v, zneg) * zstride;
        Q4<T> q{p[cell], (p + 3 * pl)[cell], (p + pl)[cell], (p + 2 * pl)[cell]};
        if (zneg) q.n = -q.n;
        return q;
    };
    Vel<T> ub{T(0), T(0), T(0)}, uc{T(0), T(0), T(0)};
    Vel<T> mc{T(0), T(0), T(0)};                       // momenta of the plane awaiting its source
    auto step_plane = [&](int v, const Q4<T>& q, Q4<T>& next, const March4<T>& mi, March4<T>& mo) {
        Q4<T> dn;
        march_push(q, mi, mo, beta, dt, v > v0 && (perz || (v >= 0 && v <= nz)), acc, dn);
        const int m = v - 2, j = v - 3;                // completed plane, plane taking its source
        const T ir = rcp(T(1) + dn.R);
        const Vel<T> ua{dn.a * ir, dn.b * ir, dn.n * ir};
        Vel<T> xl, xh, yl, yh;
        const bool src = out && j >= k0;               // j < k1 always
        if (src) {
            const T (*s)[N] = ys[j & 1];
            xl = Vel<T>{s[0][t - 1], s[1][t - 1], s[2][t - 1]};
            xh = Vel<T>{s[0][t + 1], s[1][t + 1], s[2][t + 1]};
            yl = Vel<T>{s[0][t - bx], s[1][t - bx], s[2][t - bx]};
            yh = Vel<T>{s[0][t + bx], s[1][t + bx], s[2][t + bx]};
        }
        // a halo thread's cell stands in for the ghost beside its neighbour
        T (*w)[N] = ys[m & 1];
        w[0][t] = xneg ? -ua.u1 : ua.u1;
        w[1][t] = yneg ? -ua.u2 : ua.u2;
        w[2][t] = ua.u3;
        wait_loads(next);
        if (src) {
            Vel<T> zl = ub, zh = ua;
            if (!perz && j == 0) {
                zl = uc;
                if (d.bc[4] == FVNA_BC_REFLECT) zl.u3 = -zl.u3;
            }
            if (!perz && j == nz - 1) {
                zh = uc;
                if (d.bc[5] == FVNA_BC_REFLECT) zh.u3 = -zh.u3;
            }
            // the oracle's order: -6 u_c, then x-, x+, y-, y+, z-, z+
            auto lap = [&](T c, T a0, T a1, T a2, T a3, T a4, T a5) {
                return ((((((T(-6) * c + a0) + a1) + a2) + a3) + a4) + a5);
            };
            const T l1 = lap(uc.u1, xl.u1, xh.u1, yl.u1, yh.u1, zl.u1, zh.u1);
            const T l2 = lap(uc.u2, xl.u2, xh.u2, yl.u2, yh.u2, zl.u2, zh.u2);
            const T l3 = lap(uc.u3, xl.u3, xh.u3, yl.u3, yh.u3, zl.u3, zh.u3);
            T* o = outM + (size_t)j * zstride;
            (o + pl)[cell] = fma_(kd, l1, mc.u1);
            (o + 2 * pl)[cell] = fma_(kd, l2, mc.u2);
            (o + 3 * pl)[cell] = fma_(kd, l3, mc.u3);
        }
        if (out && m >= k0 && m < k1) (outR + (size_t)m * zstride)[cell] = dn.R;
        mc = Vel<T>{dn.a, dn.b, dn.n};
        ub = uc;
        uc = ua;
        __syncthreads();
    };
    // two planes of loads in flight ahead of the one being pushed
    Q4<T> p0 = load_plane(v0), p1 = load_plane(v0 + 1);
    wait_loads(p0);
    int v = v0;
#pragma unroll 1
    for (; v + 1 < v1; v += 2) {
        Q4<T> r = p0;
        p0 = load_plane(v + 2);
        step_plane(v, r, p1, A, B);
        r = p1;
        p1 = load_plane(v + 3);
        step_plane(v + 1, r, p0, B, A);
    }
    if (v < v1) step_plane(v, p0, p1, A, B);
    cfl_commit(at, acc, real, &ys[0][0][0]);
}

__global__ void k3_ctrl_fold(Desc3 d, int last, long long owed)
{
    if (threadIdx.x == 0) *d.clk = fold_decision(d, last, owed);
}

__global__ void k3_bump(Clock* c, long long n)
{
    if (threadIdx.x == 0) c->target += n;
}

// First time step from the speeds of every interface of the current state in
// all three directions (the sweeps run with dt = 0, which leaves the state
// unchanged, so each sweep sees Q^0).
__global__ void k3_dt0(Desc3 d)
{
    if (threadIdx.x != 0) return;
    Clock* c = d.clk;
    const double smax = __longlong_as_double((long long)c->smax_bits);
    const unsigned flags = c->flags;
    c->smax_bits = 0ull;
    c->flags = 0u;
    if (flags & FLAG_NONHYP) { c->status = ST_NONHYP; c->status_step = 0; return; }
    if ((flags & FLAG_NONFINITE) || !(smax > 0.0) || !(smax <= 1.7976931348623157e308)) {
        c->status = ST_NONFINITE;
        c->status_step = 0;
        return;
    }
    c->dt = d.cfl_target / smax;
}

__global__ void k3_clock(Clock* c, double t, double dt, int cur)
{
    if (threadIdx.x != 0) return;
    Clock h;
    __builtin_memset(&h, 0, sizeof(h));
    h.t = t;
    h.dt = dt;
    h.cur = cur;
    *c = h;
}

// Host doubles (SI, staged) <-> stored dimensionless field; rows r over
// ny * nz, grid-strided (gridDim.y is at most 65535).
template <typename T>
__global__ void k3_import(Desc3 d, const double* __restrict__ src, int field, double denom)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= d.pitch) return;
    const int rows = d.n[1] * d.n[2];
    for (int r = blockIdx.y; r < rows; r += gridDim.y) {
        // the state of clock cur = 0 (set after the import)
        T* dst = (T*)d.buf[field == 0 ? buf_rho(0) : buf_mom(0)] + (size_t)field * (size_t)d.plane +
                 (size_t)r * (size_t)d.pitch;
        dst[i] = i < d.n[0] ? (T)(src[(size_t)r * d.n[0] + i] / denom) : T(0);
    }
}

template <typename T>
__global__ void k3_export(Desc3 d, double* __restrict__ dst, int field, long long row0, long long nrows, double factor)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= d.n[0]) return;
    const int cur = d.clk->cur;
    const T* base = (const T*)d.buf[field == 0 ? buf_rho(cur) : buf_mom(cur)] + (size_t)field * (size_t)d.plane;
    for (long long r = blockIdx.y; r < nrows; r += gridDim.y)
        dst[(size_t)r * d.n[0] + i] = (double)base[(size_t)(row0 + r) * (size_t)d.pitch + i] * factor;
}

thread_local std::string g_err3 = "no error";

fvna_status fail3(fvna_status s, const std::string& msg)
{
    g_err3 = msg;
    return s;
}

#define HIP3(x)                                                                        \
    do {                                                                               \
        hipError_t e_ = (x);                                                           \
        if (e_ != hipSuccess) return fail3(FVNA_E_HIP, std::string(#x) + ": " + hipGetErrorString(e_)); \
    } while (0)

constexpr int GRAPH3_CHUNK = 32;    // attempts per captured graph

size_t elem(const fvna3_params* p) { return p->precision == FVNA_F64 ? 8 : 4; }
int pitch3(const fvna3_params* p) { const int per = 256 / (int)elem(p); return (p->nx + per - 1) / per * per; }

fvna_status validate3(const fvna3_params* p)
{
    if (!p) return fail3(FVNA_E_INVALID, "params is NULL");
    if (p->nx < 4 || p->ny < 4 || p->nz < 4) return fail3(FVNA_E_INVALID, "grid must have at least 4 cells per axis");
    if ((long long)p->nx * p->ny * p->nz > (1ll << 31)) return fail3(FVNA_E_INVALID, "grid too large");
    if (!(p->dx > 0) || !(p->c0 > 0) || !(p->rho0 > 0) || !(p->beta >= 1) || !(p->delta >= 0))
        return fail3(FVNA_E_INVALID, "need dx, c0, rho0 > 0, beta >= 1, delta >= 0");
    if (p->precision != FVNA_F64 && p->precision != FVNA_F32) return fail3(FVNA_E_INVALID, "precision must be F64 or F32");
    for (int s = 0; s < 6; ++s)
        if (p->bc[s] != FVNA_BC_PERIODIC && p->bc[s] != FVNA_BC_EXTRAP0 && p->bc[s] != FVNA_BC_REFLECT)
            return fail3(FVNA_E_INVALID, "sides must be PERIODIC, EXTRAP0 or REFLECT");
    for (int a = 0; a < 3; ++a)
        if ((p->bc[2 * a] == FVNA_BC_PERIODIC) != (p->bc[2 * a + 1] == FVNA_BC_PERIODIC))
            return fail3(FVNA_E_INVALID, "both sides of an axis must be periodic together");
    if (!(p->cfl_target > 0) || !(p->cfl_target < p->cfl_max)) return fail3(FVNA_E_INVALID, "need 0 < cfl_target < cfl_max");
    if (p->max_retries < 0) return fail3(FVNA_E_INVALID, "max_retries must be >= 0");
    return FVNA_OK;
}

// scratch layout: [Clock, ClockAux][staging of one field]
constexpr size_t OFF3_STAGE = 768;
static_assert(CLOCK_AUX_OFFSET + sizeof(ClockAux) <= OFF3_STAGE, "clock and shadow states before the staging area");

int cu_count3()
{
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 256;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) return 256;
    return n;
}

// Blocks of k3_sweep12 that a CU holds at once, as built.
template <typename T> int resident12()
{
    int n = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, k3_sweep12<T>, 256, 0) != hipSuccess || n <= 0) {
        (void)hipGetLastError();
        n = sizeof(T) == 8 ? 2 : 5;
    }
    return n;
}

// Tiles of k3_sweep3s: the width bx, with by = threads / bx rows, and the
// number of z segments of least cost, counted in planes pushed one after
// another: rounds of one block per CU, times planes per segment + 6.
void plan_sweep3(Desc3& d, int threads, int cus)
{
    double best = 1e30;
    const int nz = d.n[2];
    for (int bx = std::min(8, d.n[0] + 2); bx <= std::min(threads / 4, d.n[0] + 2); ++bx) {
        const int by = std::min(threads / bx, d.n[1] + 2);
        const long long ntx = (d.n[0] + bx - 3) / (bx - 2), nty = (d.n[1] + by - 3) / (by - 2), xy = ntx * nty;
        for (int segs = 1; segs <= nz; ++segs) {
            const int planes = (nz + segs - 1) / segs;
            const long long blocks = xy * ((nz + planes - 1) / planes);
            // rows of a tile shorter than a 128-byte line waste part of what they fetch
            const double cost = (double)((blocks + cus - 1) / cus) * (planes + 6) * (1.0 + 1.0 / bx);
            if (cost < best) {
                best = cost;
                d.bx = bx; d.by = by; d.ntx = (int)ntx; d.nty = (int)nty;
                d.planes3 = planes;
                d.segs3 = (nz + planes - 1) / planes;
            }
            if (planes <= 2 || blocks > 16ll * cus) break;
        }
    }
}

}  // namespace

struct fvna3_ctx {
    fvna3_params p;
    Desc3 d;
    hipStream_t s;
    hipStream_t cap;
    char* scratch;
    hipGraph_t graph = nullptr;
    hipGraphExec_t exec = nullptr;
    Reply reply;
    void (*attempt)(const Desc3&, int force, int pos, long long owed, hipStream_t) = nullptr;
};

namespace {

template <typename T>
void launch_attempt(const Desc3& d, int force, int pos, long long owed, hipStream_t s)
{
    const int t12 = (d.strips12 * d.n[2] + d.tailk12) * d.segs12;
    hipLaunchKernelGGL(k3_sweep12<T>, dim3((t12 + 3) / 4), dim3(256), 0, s, d, force, pos, owed);
    hipLaunchKernelGGL(k3_sweep3s<T>, dim3(d.ntx * d.nty * d.segs3), dim3(Sweep3<T>::threads), 0, s, d, force, pos,
                       owed);
}

// n attempts in a row and the closing decision (as launch_attempts in two
// dimensions).
void launch_attempts3(fvna3_ctx* c, int n, long long owed, hipStream_t s)
{
    if (n <= 0) return;
    for (int k = 0; k < n; ++k) c->attempt(c->d, 0, k, owed, s);
    hipLaunchKernelGGL(k3_ctrl_fold, dim3(1), dim3(64), 0, s, c->d, n - 1, owed);
}

void drop_graph3(fvna3_ctx* c)
{
    if (c->exec || c->graph) (void)hipStreamSynchronize(c->s);
    if (c->exec) (void)hipGraphExecDestroy(c->exec);
    if (c->graph) (void)hipGraphDestroy(c->graph);
    c->exec = nullptr;
    c->graph = nullptr;
}

fvna_status build_graph3(fvna3_ctx* c)
{
    if (c->exec) return FVNA_OK;
    HIP3(hipStreamBeginCapture(c->cap, hipStreamCaptureModeThreadLocal));
    launch_attempts3(c, GRAPH3_CHUNK, 0, c->cap);
    hipGraph_t g = nullptr;
    HIP3(hipStreamEndCapture(c->cap, &g));
    c->graph = g;
    HIP3(hipGraphInstantiate(&c->exec, g, nullptr, nullptr, 0));
    return FVNA_OK;
}

fvna_status enqueue3(fvna3_ctx* c, long long attempts, long long owed = 0)
{
    if (attempts >= GRAPH3_CHUNK) {
        const fvna_status s = build_graph3(c);
        if (s) return s;
        for (long long k = 0; k < attempts / GRAPH3_CHUNK; ++k) HIP3(hipGraphLaunch(c->exec, c->s));
    }
    launch_attempts3(c, (int)(attempts % GRAPH3_CHUNK), owed, c->s);
    HIP3(hipGetLastError());
    return FVNA_OK;
}

fvna_status read_clock3(fvna3_ctx* c, Clock* h)
{
    HIP3(read_words(c->reply, c->s, c->d.clk, h, sizeof(Clock)));
    return FVNA_OK;
}

fvna_status status3(int st)
{
    switch (st) {
    case 0: return FVNA_OK;
    case ST_NONHYP: return fail3(FVNA_E_NONHYPERBOLIC, "non-real Roe speeds (discriminant <= 0) in a step");
    case ST_NONFINITE: return fail3(FVNA_E_NONFINITE, "non-finite wave speed in a step");
    case ST_RETRIES: return fail3(FVNA_E_RETRIES, "too many rejected attempts in a row");
    default: return fail3(FVNA_E_STATE, "unknown device status");
    }
}

// Wait for the stream and top up the steps rejected attempts left owed.
fvna_status sync3(fvna3_ctx* c)
{
    Clock h;
    for (int guard = 0; guard < 1000; ++guard) {
        fvna_status s = read_clock3(c, &h);
        if (s) return s;
        if (h.status != 0 || h.accepted >= h.target) return status3(h.status);
        s = enqueue3(c, h.target - h.accepted);
        if (s) return s;
    }
    return fail3(FVNA_E_STATE, "steps still owed after many top-up rounds");
}

}  // namespace

extern "C" {

const char* fvna3_last_error(void) { return g_err3.c_str(); }

fvna_status fvna3_workspace_size(const fvna3_params* p, size_t* state_bytes, size_t* scratch_bytes)
{
    fvna_status s = validate3(p);
    if (s) return s;
    if (!state_bytes || !scratch_bytes) return fail3(FVNA_E_INVALID, "NULL argument");
    *state_bytes = 4 * (size_t)pitch3(p) * (size_t)p->ny * (size_t)p->nz * elem(p);
    *scratch_bytes = OFF3_STAGE + (size_t)p->nx * (size_t)p->ny * (size_t)p->nz * sizeof(double);
    return FVNA_OK;
}

fvna_status fvna3_create(const fvna3_params* p, void* buf_a, void* buf_b, void* buf_c, void* scratch, void* stream,
                         fvna3_ctx** out)
{
    if (!out) return fail3(FVNA_E_INVALID, "out is NULL");
    *out = nullptr;
    fvna_status s = validate3(p);
    if (s) return s;
    if (!buf_a || !buf_b || !buf_c || !scratch) return fail3(FVNA_E_INVALID, "NULL buffer");
    if (((uintptr_t)buf_a | (uintptr_t)buf_b | (uintptr_t)buf_c | (uintptr_t)scratch) % 256)
        return fail3(FVNA_E_INVALID, "device buffers must be 256-byte aligned");
    fvna3_ctx* c = new (std::nothrow) fvna3_ctx;
    if (!c) return fail3(FVNA_E_NOMEM, "out of host memory");
    c->p = *p;
    Desc3& d = c->d;
    std::memset(&d, 0, sizeof(d));
    d.n[0] = p->nx; d.n[1] = p->ny; d.n[2] = p->nz;
    d.pitch = pitch3(p);
    d.plane = (long long)d.pitch * p->ny * p->nz;
    const int cus = cu_count3();
    // x1-x2 tiles: full 60-column strips, and the remaining nx mod 60
    // columns packed several planes to a wavefront when at least two fit
    // (256^3 FP32: 3330 wavefronts instead of 3840)
    const int rem12 = p->nx % OUT12, tw = rem12 + 2 * HALO12;
#ifndef FVNA3_PACK_TAIL
#define FVNA3_PACK_TAIL 1
#endif
    if (FVNA3_PACK_TAIL && rem12 > 0 && WAVE / tw >= 2) {
        d.strips12 = p->nx / OUT12;
        d.tailw12 = tw;
        d.tailp12 = WAVE / tw;
        d.tailk12 = (p->nz + d.tailp12 - 1) / d.tailp12;
    } else {
        d.strips12 = (p->nx + OUT12 - 1) / OUT12;
        d.tailw12 = 0;
        d.tailp12 = 1;
        d.tailk12 = 0;
    }
    // row segments for about six x1-x2 tiles per SIMD: several rounds of
    // wavefronts let the dispatcher even out the load of the SIMDs, where
    // one round leaves some with a wavefront more than others (256^3, per
    // step: FP32 325 us with 43-row tiles, 333 with 64, 345 with 86, 371 with
    // 128; 332 with 25).  On a grid too small for that at 16 rows the CU with the
    // most blocks (of four tiles) ends the sweep: m blocks on it take a row 1,
    // 1.55, 2.15, ... = 0.35 + 0.6 m times as long as one (128^3 FP32: 0.93 us with
    // one, 1.37, 1.88, 2.42, 2.93), blocks past what is resident (FP64 two per CU,
    // FP32 five) take rounds, and the height of least (rows + 4 warm-up rows) x
    // that is taken, at least 4.  us per step, by the total of tiles before / by
    // blocks: 128^3 FP32 70 / 62 (16 / 19 rows), FP64 103 / 90, 180 x 160 x 140 FP32
    // 106 / 93 (32 / 24), 90 x 75 x 64 FP64 43 / 41 (10 / 5); FP64 with three blocks
    // taken as resident / two: 160^3 160 / 155 (27 / 40), 148 x 95 x 137 89 / 85
    // (12 / 19), 96^3 59.5 / 57.3 (6 / 10).
    {
        const long long units = (long long)d.strips12 * p->nz + d.tailk12;
        const long long simds = 4ll * cus, want = 6 * simds;
        const long long nseg = std::max(1ll, (want + units - 1) / units);
        long long rows = (p->ny + nseg - 1) / nseg;
        if (rows < 16) {
            const long long resident = p->precision == FVNA_F64 ? resident12<double>() : resident12<float>();
            auto row_time = [](long long m) { return m == 0 ? 0.0 : m == 1 ? 1.0 : 0.35 + 0.6 * (double)m; };
            double best = 1e30;
            for (long long r = std::min(4, p->ny); r <= p->ny; ++r) {
                const long long blocks = (units * ((p->ny + r - 1) / r) + 3) / 4, round = resident * cus;
                const double cost = (double)(r + 2 * HALO12) * ((double)(blocks / round) * row_time(resident) +
                                                                row_time((blocks % round + cus - 1) / cus));
                if (cost <= best) { best = cost; rows = r; }       // of equals the tallest: fewer warm-up rows
            }
        }
        d.rows12 = (int)std::min(rows, (long long)p->ny);
    }
    d.segs12 = (p->ny + d.rows12 - 1) / d.rows12;
    plan_sweep3(d, p->precision == FVNA_F64 ? Sweep3<double>::threads : Sweep3<float>::threads, cus);
    for (int k = 0; k < 6; ++k) d.bc[k] = p->bc[k];
    d.fixed_dt = p->fixed_dt ? 1 : 0;
    d.max_retries = p->max_retries;
    d.beta = p->beta;
    d.delta = p->delta / (p->c0 * p->dx);
    d.cfl_target = p->cfl_target;
    d.cfl_max = p->cfl_max;
    d.buf[0] = buf_a; d.buf[1] = buf_b; d.buf[2] = buf_c;
    d.clk = (Clock*)scratch;
    c->scratch = (char*)scratch;
    c->s = (hipStream_t)stream;
    c->attempt = p->precision == FVNA_F64 ? launch_attempt<double> : launch_attempt<float>;
    if (hipStreamCreateWithFlags(&c->cap, hipStreamNonBlocking) != hipSuccess) {
        delete c;
        return fail3(FVNA_E_HIP, "cannot create the capture stream");
    }
    const size_t sb = 4 * (size_t)d.plane * elem(p);
    for (int b = 0; b < 3; ++b)
        if (hipMemsetAsync(d.buf[b], 0, sb, c->s) != hipSuccess) {
            (void)hipStreamDestroy(c->cap);
            delete c;
            return fail3(FVNA_E_HIP, "cannot clear the state buffers");
        }
    hipLaunchKernelGGL(k3_clock, dim3(1), dim3(64), 0, c->s, d.clk, 0.0, 0.0, 0);
    if (hipStreamSynchronize(c->s) != hipSuccess) {
        (void)hipStreamDestroy(c->cap);
        delete c;
        return fail3(FVNA_E_HIP, "cannot initialise the clock");
    }
    *out = c;
    return FVNA_OK;
}

fvna_status fvna3_set_state(fvna3_ctx* c, const double* rho_p, const double* m1, const double* m2, const double* m3)
{
    if (!c || !rho_p || !m1 || !m2 || !m3) return fail3(FVNA_E_INVALID, "NULL argument");
    const fvna3_params& p = c->p;
    const Desc3& d = c->d;
    const double* src[4] = {rho_p, m1, m2, m3};
    const double denom[4] = {p.rho0, p.rho0 * p.c0, p.rho0 * p.c0, p.rho0 * p.c0};
    const size_t n = (size_t)p.nx * p.ny * p.nz;
    double* stage = (double*)(c->scratch + OFF3_STAGE);
    HIP3(hipStreamSynchronize(c->s));
    const dim3 grid((d.pitch + 255) / 256, std::min(p.ny * p.nz, 65535));
    for (int f = 0; f < 4; ++f) {
        HIP3(hipMemcpyAsync(stage, src[f], n * sizeof(double), hipMemcpyHostToDevice, c->s));
        if (p.precision == FVNA_F64) hipLaunchKernelGGL(k3_import<double>, grid, dim3(256), 0, c->s, d, stage, f, denom[f]);
        else hipLaunchKernelGGL(k3_import<float>, grid, dim3(256), 0, c->s, d, stage, f, denom[f]);
        HIP3(hipGetLastError());
    }
    const double dt0 = p.dt0 > 0 ? p.dt0 * p.c0 / p.dx : 0.0;
    hipLaunchKernelGGL(k3_clock, dim3(1), dim3(64), 0, c->s, d.clk, 0.0, dt0, 0);
    HIP3(hipGetLastError());
    if (!(dt0 > 0)) {
        // dt = 0: the x1, x2 and x3 sweeps see Q^0 and the source adds nothing
        c->attempt(d, 1, 0, 0, c->s);
        hipLaunchKernelGGL(k3_dt0, dim3(1), dim3(64), 0, c->s, d);
        HIP3(hipGetLastError());
    }
    // waits for the stream: the caller's arrays are free when this returns
    Clock h;
    fvna_status s = read_clock3(c, &h);
    if (s) return s;
    if (h.status == ST_NONHYP) return fail3(FVNA_E_NONHYPERBOLIC, "non-real Roe speeds in the initial state");
    if (h.status) return fail3(FVNA_E_NONFINITE, "no finite positive wave speed in the initial state");
    return FVNA_OK;
}

fvna_status fvna3_step(fvna3_ctx* c, int64_t nsteps)
{
    if (!c) return fail3(FVNA_E_INVALID, "ctx is NULL");
    if (nsteps < 0) return fail3(FVNA_E_INVALID, "nsteps must be >= 0");
    if (nsteps == 0) return FVNA_OK;
    const bool graph = nsteps >= GRAPH3_CHUNK;         // shorter runs carry their step count themselves
    if (graph) hipLaunchKernelGGL(k3_bump, dim3(1), dim3(64), 0, c->s, c->d.clk, (long long)nsteps);
    HIP3(hipGetLastError());
    fvna_status s = enqueue3(c, nsteps, graph ? 0 : nsteps);
    if (s) return s;
    return sync3(c);
}

fvna_status fvna3_get_state(fvna3_ctx* c, double* rho_p, double* m1, double* m2, double* m3)
{
    if (!c || !rho_p || !m1 || !m2 || !m3) return fail3(FVNA_E_INVALID, "NULL argument");
    const fvna3_params& p = c->p;
    const Desc3& d = c->d;
    double* dst[4] = {rho_p, m1, m2, m3};
    const double fac[4] = {p.rho0, p.rho0 * p.c0, p.rho0 * p.c0, p.rho0 * p.c0};
    const size_t n = (size_t)p.nx * p.ny * p.nz;
    double* stage = (double*)(c->scratch + OFF3_STAGE);
    const long long rows = (long long)p.ny * p.nz;
    auto fill = [&](int f, long long r0, long long nr, double* out) {
        const dim3 grid((p.nx + 255) / 256, (unsigned)std::min(nr, 65535ll));
        if (p.precision == FVNA_F64)
            hipLaunchKernelGGL(k3_export<double>, grid, dim3(256), 0, c->s, d, out, f, r0, nr, fac[f]);
        else hipLaunchKernelGGL(k3_export<float>, grid, dim3(256), 0, c->s, d, out, f, r0, nr, fac[f]);
    };
    hipError_t err;
    if (stream_out(c->reply, c->s, 4, rows, p.nx, stage, dst, fill, err)) {
        HIP3(err);
        return FVNA_OK;
    }
    HIP3(hipStreamSynchronize(c->s));
    for (int f = 0; f < 4; ++f) {
        fill(f, 0, rows, stage);
        HIP3(hipGetLastError());
        HIP3(hipMemcpyAsync(dst[f], stage, n * sizeof(double), hipMemcpyDeviceToHost, c->s));
        HIP3(hipStreamSynchronize(c->s));
    }
    return FVNA_OK;
}

fvna_status fvna3_get_stats(fvna3_ctx* c, fvna_stats* st)
{
    if (!c || !st) return fail3(FVNA_E_INVALID, "NULL argument");
    Clock h;
    fvna_status s = read_clock3(c, &h);
    if (s) return s;
    const double tu = c->p.dx / c->p.c0;
    std::memset(st, 0, sizeof(*st));
    st->t = h.t * tu;
    st->dt_next = h.dt * tu;
    st->nu_last = h.nu_last;
    st->nu_mean = h.nu_mean;
    st->nu_std = h.nu_count > 0 ? std::sqrt(h.nu_m2 / (double)h.nu_count) : 0.0;
    st->steps = h.accepted;
    st->rejected = h.rejected;
    st->status = h.status;
    st->status_step = h.status_step;
    return FVNA_OK;
}

fvna_status fvna3_time_step_kernels(fvna3_ctx* c, int32_t reps, double* ms)
{
    if (!c || !ms || reps < 1) return fail3(FVNA_E_INVALID, "bad argument");
    // back-to-back recomputations of the attempt the next step would make
    // (forced, no decision): the state and the clock are unchanged apart
    // from the attempt's speed maximum, which the next closing launch clears
    hipEvent_t e0, e1;
    HIP3(hipEventCreate(&e0));
    HIP3(hipEventCreate(&e1));
    c->attempt(c->d, 1, 0, 0, c->s);
    HIP3(hipEventRecord(e0, c->s));
    for (int r = 0; r < reps; ++r) c->attempt(c->d, 1, 0, 0, c->s);
    HIP3(hipGetLastError());
    HIP3(hipEventRecord(e1, c->s));
    HIP3(hipEventSynchronize(e1));
    float t = 0.0f;
    HIP3(hipEventElapsedTime(&t, e0, e1));
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    *ms = (double)t / reps;
    return FVNA_OK;
}

void fvna3_destroy(fvna3_ctx* c)
{
    if (!c) return;
    (void)hipStreamSynchronize(c->s);
    drop_graph3(c);
    (void)hipStreamDestroy(c->cap);
    delete c;
}

}  // extern "C"

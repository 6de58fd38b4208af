// pb_tree.hip -- the atoms x cut-points sums of the energy read-back, by multipole expansions.
//
//   S_F(i) = sum_p F_p / |r_p - a_i|      S_D(i) = sum_p u_p.(r_p - a_i) / |r_p - a_i|^3
//
// are potentials of point charges F_p and point dipoles u_p, so a box of cut points acts on a
// distant atom through one expansion in solid harmonics instead of point by point.  With the
// cut points of a box scaled to its centre and half-diagonal rs, and
//
//   q_mm = (x + iy)^m,   q_lm = z q_{l-1,m} - c_lm r^2 q_{l-2,m},   c_lm = ((l-1)^2 - m^2)/((2l-1)(2l-3))
//
// (solid harmonics whose z-polynomial has leading coefficient one),
//
//   1/|R - r| = sum_{l,m>=0} N_lm Re[q_lm(r) conj(q_lm(R))] / |R|^(2l+1),
//   N_lm = (2 - [m=0]) ((2l-1)!!)^2 / ((l-m)! (l+m)!).
//
// The expansion of a box has the coefficients M_lm = N_lm sum F q_lm for the charges and D_lm =
// -N_lm sum u.grad q_lm for the dipoles; the gradient of a q_lm is a combination of three of
// degree l-1, so the box sums needed are those of F q_lm, u_x q_lm, u_y q_lm and u_z q_lm.
//
// 60,000 atoms x 3.9e6 points (385^3): 136 ms by the direct sum; here 17.0 ms, of which box
// expansions 3.6, their sums 5.0 and the near points 8.4 (1.2e10 of 2.3e11 pairs).
//
// Boxes are B^3 lattice cells (about kBoxPoints cut points each); atoms are taken in groups of
// 64 along a Hilbert curve, one wave per group.  A box acts on a group through its expansion,
// truncated at the degree p where (rs/d)^(p+1) <= 1e-12 (d: distance of the box centre to the
// group's bounding box), when p <= kDegree and that costs less than the box's points; else the
// wave sums the box's points.  (rs/d)^(p+1) bounds the terms left out of the charges' series; the
// dipoles' have up to p + 1 times that.  Against extended precision, relative to the box's own sum
// of absolute values and at any admitted distance: points all over the box 1e-15 for the charges
// and 9e-14 for the dipoles, a plane patch 3e-15 and 3e-13, points in the corner that faces the atom
// alone 4e-13 and 2e-11.  Over an atom's whole sum, boxes on all sides, none of it is left: for globules,
// rods, two clusters, flat sheets, tilted sheets and hollow shells the errors, 2e-16 to 3e-14 of the sum
// of absolute values, are those of the direct sum in two digits.
//
// Everything is ordered: the cut points of a box keep their lattice order, a wave takes its
// boxes in index order and a chunk's partial sums are added in chunk order, so that a read-back
// gives the same bits each time.
#include "pb_tree.h"

#include <algorithm>
#include <cmath>

namespace pbk {

namespace {

constexpr int kDegree = 39;                               // largest degree of an expansion
constexpr int kRow = 4;                                   // terms per step of the far sum
constexpr int kBoxPoints = 1500, kMinBoxPoints = 400;      // cut points aimed at per box
constexpr int kBoxes = 700;                               // boxes that keep the device busy
constexpr int kMaxSide = 32;                              // most lattice cells along a box
constexpr int kMaxBits = 6;                               // bins per axis along the atoms' curve: 2^kMaxBits
constexpr int kCurveBits = 10;                            // ... and cells: 2^kCurveBits
constexpr int kGroup = 64;                                // atoms per group, one per lane
constexpr int kFarWaves = 16384, kNearBlocks = 8192;      // waves and blocks aimed at in the sums

// terms in rows m = 0, 1, ..., each l = m, m + 1, ... padded to whole steps of kRow terms (zeros)
__host__ __device__ constexpr int row_terms(int m) { return (kDegree - m + kRow) / kRow * kRow; }
__host__ __device__ constexpr int row_base(int m)
{
    int e = 0;
    for (int k = 0; k < m; ++k) e += row_terms(k);
    return e;
}
constexpr int kTerms = row_base(kDegree + 1);

struct Tables {
    double c[kTerms];           // c_lm
    double n[kTerms];           // N_lm (0: padding)
    short base[kDegree + 2];    // row_base
    unsigned char l[kTerms], m[kTerms];
};

constexpr Tables make_tables()
{
    Tables t{};
    for (int m = 0; m <= kDegree; ++m) {
        // N_mm = (2 - [m=0]) ((2m-1)!!)^2 / (2m)!, and N_{l,m} / N_{l-1,m} = (2l-1)^2 / (l^2 - m^2)
        double n = m == 0 ? 1.0 : 2.0;
        for (int k = 1; k <= m; ++k) n *= (double)(2 * k - 1) / (double)(2 * k);
        t.base[m] = (short)row_base(m);
        for (int l = m; l < m + row_terms(m); ++l) {
            const int e = row_base(m) + l - m;
            if (l > m) n *= (double)((2 * l - 1) * (2 * l - 1)) / (double)(l * l - m * m);
            t.n[e] = l <= kDegree ? n : 0.0;
            t.c[e] = l >= 2 ? (double)((l - 1) * (l - 1) - m * m) / (double)((2 * l - 1) * (2 * l - 3)) : 0.0;
            t.l[e] = (unsigned char)l;
            t.m[e] = (unsigned char)m;
        }
    }
    t.base[kDegree + 1] = (short)kTerms;
    return t;
}

__constant__ const Tables kTab = make_tables();

__device__ __forceinline__ int term(int l, int m) { return kTab.base[m] + l - m; }

// ---- cut points by box -------------------------------------------------------------------
// The cut list is in lattice order, so the cut points of one lattice row (i, j) inside a box are
// consecutive: a segment.  Segment r of box b (r = the row within the box) is seg[b * B^2 + r].

__device__ __forceinline__ int seg_of(const TreeGeom& t, int64_t key)
{
    const int64_t e = key >> 2, row = e / t.S;
    const int k = (int)(e - row * t.S) - Z0, j = (int)(row % t.ny), i = (int)(row / t.ny);
    int c[3] = {i - t.c0[0], j - t.c0[1], k - t.c0[2]}, b[3];
    for (int d = 0; d < 3; ++d) {
        c[d] = c[d] < 0 ? 0 : c[d];
        b[d] = c[d] / t.B;
        b[d] = b[d] < t.nb[d] ? b[d] : t.nb[d] - 1;
        c[d] -= b[d] * t.B;
        c[d] = c[d] < t.B ? c[d] : t.B - 1;
    }
    return ((b[0] * t.nb[1] + b[1]) * t.nb[2] + b[2]) * t.B * t.B + c[0] * t.B + c[1];
}

// first and one past the last cut point of every segment (cleared before)
__global__ void __launch_bounds__(256) k_tree_seg(TreeGeom t, int64_t ncut, const int64_t* __restrict__ cutkey,
                                                  int* __restrict__ first, int* __restrict__ last)
{
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= ncut) return;
    const int s = seg_of(t, cutkey[c]);
    if (c == 0 || seg_of(t, cutkey[c - 1]) != s) first[s] = (int)c;
    if (c == ncut - 1 || seg_of(t, cutkey[c + 1]) != s) last[s] = (int)c + 1;
}

// per box: shift[s] = the offset within the box of segment s's cut points minus the segment's
// first cut point, and the box's count
__global__ void __launch_bounds__(256) k_tree_box(TreeGeom t, const int* __restrict__ first, int* __restrict__ last,
                                                  int* __restrict__ count)
{
    __shared__ int sh[4];
    const int nseg = t.B * t.B, s0 = blockIdx.x * nseg;
    const int lane = (int)(threadIdx.x & 63), w = (int)(threadIdx.x >> 6);
    int carry = 0;
    for (int base = 0; base < nseg; base += 256) {
        const int r = base + (int)threadIdx.x;
        const int f = r < nseg ? first[s0 + r] : 0, v = r < nseg ? last[s0 + r] - f : 0;
        int incl = v;
        for (int o = 1; o < 64; o <<= 1) {
            const int u = __shfl_up(incl, o, 64);
            if (lane >= o) incl += u;
        }
        if (lane == 63) sh[w] = incl;
        __syncthreads();
        int before = carry;
        for (int q = 0; q < w; ++q) before += sh[q];
        carry += (sh[0] + sh[1]) + (sh[2] + sh[3]);
        if (r < nseg) last[s0 + r] = before + incl - v - f;
        __syncthreads();
    }
    if (threadIdx.x == 0) count[blockIdx.x] = carry;
}

// where cut point c goes: start[box] + shift[segment] + c
__global__ void __launch_bounds__(256) k_tree_pos(TreeGeom t, int64_t ncut, const int64_t* __restrict__ cutkey,
                                                  const int* __restrict__ shift, const int* __restrict__ start,
                                                  int* __restrict__ pos)
{
    const int64_t c = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (c >= ncut) return;
    const int s = seg_of(t, cutkey[c]);
    pos[c] = start[s / (t.B * t.B)] + shift[s] + (int)c;
}

// ---- atoms along a Hilbert curve ----------------------------------------------------------

// position along the Hilbert curve of a cube of 2^kCurveBits cells per axis: Skilling's transpose form
// (J. Skilling, Programming the Hilbert curve, AIP Conf. Proc. 707, 2004), then the interleave.  Its
// leading 3 b bits are the position along the curve of 2^b cells per axis.
__device__ __forceinline__ unsigned hilbert(const TreeGeom& t, const double* x)
{
    unsigned v[3];
    const int top = (1 << kCurveBits) - 1;
    for (int d = 0; d < 3; ++d) {
        const int q = (int)floor((x[d] - t.alo[d]) * t.ainv);
        v[d] = (unsigned)(q < 0 ? 0 : q > top ? top : q);
    }
    for (unsigned q = 1u << (kCurveBits - 1); q > 1; q >>= 1)
        for (int d = 0; d < 3; ++d) {
            if (v[d] & q) {
                v[0] ^= q - 1;
            } else {
                const unsigned e = (v[0] ^ v[d]) & (q - 1);
                v[0] ^= e;
                v[d] ^= e;
            }
        }
    v[1] ^= v[0];
    v[2] ^= v[1];
    unsigned e = 0;
    for (unsigned q = 1u << (kCurveBits - 1); q > 1; q >>= 1)
        if (v[2] & q) e ^= q - 1;
    unsigned code = 0;
    for (int b = kCurveBits - 1; b >= 0; --b)
        for (int d = 0; d < 3; ++d) code = (code << 1) | (((v[d] ^ e) >> b) & 1u);
    return code;
}

__device__ __forceinline__ int bin_of(const TreeGeom& t, unsigned code) { return (int)(code >> 3 * (kCurveBits - t.bits)); }

__global__ void __launch_bounds__(256) k_tree_acount(TreeGeom t, Atoms at, int* cnt)
{
    const int a = blockIdx.x * 256 + threadIdx.x;
    if (a < at.n) atomicAdd(&cnt[bin_of(t, hilbert(t, at.xyzr + 4 * a))], 1);
}

// position and atom into the atom's bin; leaves cursor[b] at the end of bin b
__global__ void __launch_bounds__(256) k_tree_ascatter(TreeGeom t, Atoms at, int* cursor,
                                                       unsigned long long* __restrict__ keys)
{
    const int a = blockIdx.x * 256 + threadIdx.x;
    if (a >= at.n) return;
    const unsigned code = hilbert(t, at.xyzr + 4 * a);
    keys[atomicAdd(&cursor[bin_of(t, code)], 1)] = (unsigned long long)code << 32 | (unsigned)a;
}

// The scatter's order depends on scheduling: each atom goes to its rank in its bin by position, then
// atom.  One thread per atom counts the smaller keys of the bin, an atom or two in a compact solute; bins
// can be long where one atom lies far from the rest (sorted by one thread per bin, 0.6 s of a read-back of
// 24,000 atoms with one 1,200 A away; 5 ms in all so).  The atoms then as the sums take them: -2a and |a|^2
// relative to the atoms' centre.
__global__ void __launch_bounds__(256) k_tree_aorder(TreeGeom t, Atoms at, const int* __restrict__ end,
                                                     const unsigned long long* __restrict__ keys, int* __restrict__ ids,
                                                     double* __restrict__ at4)
{
    const int u = blockIdx.x * 256 + threadIdx.x;
    if (u >= at.n) return;
    const unsigned long long key = keys[u];
    const int b = bin_of(t, (unsigned)(key >> 32));
    const int s = b > 0 ? end[b - 1] : 0, e = end[b];
    int place = s;
    for (int x = s; x < e; ++x) place += keys[x] < key ? 1 : 0;
    const int a = (int)(unsigned)key;
    ids[place] = a;
    const double* A = at.xyzr + 4 * a;
    const double x = A[0] - at.cx, y = A[1] - at.cy, z = A[2] - at.cz;
    double* o = at4 + 4 * place;
    o[0] = -2.0 * x;
    o[1] = -2.0 * y;
    o[2] = -2.0 * z;
    o[3] = fma(x, x, fma(y, y, z * z));
}

// ---- box expansions -------------------------------------------------------------------------
// One block per box, eight waves: the orders m < 16 and m >= 16, each for the real and the imaginary
// parts, and each of these for every other four points.  A wave works on four cut points at a time: lane m' + 16 k holds the z-recurrence of order
// m0 + m' at cut point k, and a 4x4x4 FP64 matrix instruction (A: 16 orders x 4 points, B: 4
// points x the weights F, u_x, u_y, u_z) adds the four points' products to the sums, which so stay
// in registers, one per lane and degree, with no reduction across lanes.  Per degree: four FP64
// instructions and a matrix instruction of 16 cycles (measured: at the vector units' FP64 rate).
// Both parts in one wave would save a quarter of the FP64 instructions, but its 80 sums per lane
// leave room for two waves per SIMD only.  3.9e6 points: 3.6 ms, matrix and vector pipes busy 0.70
// of the time; 3.9 ms with both parts in one wave.

using GPtr = const double* __restrict__;

// component k of cut point u: components lie ncut apart, so that a load takes the component's base
// from scalar registers and the lane's 32-bit offset
__device__ __forceinline__ double component(GPtr pts, int64_t ncut, int k, unsigned u)
{
    return *(const double*)((const char*)(pts + k * ncut) + u * 8u);
}

__device__ __forceinline__ void box_centre(const TreeGeom& t, int box, double* c)
{
    const int bz = box % t.nb[2], bxy = box / t.nb[2], by = bxy % t.nb[1], bx = bxy / t.nb[1];
    c[0] = t.ctr[0] + t.side * (double)bx;
    c[1] = t.ctr[1] + t.side * (double)by;
    c[2] = t.ctr[2] + t.side * (double)bz;
}

__device__ __forceinline__ void csq(double& r, double& i)
{
    const double t = fma(r, r, -(i * i));
    i = 2.0 * (r * i);
    r = t;
}

__device__ __forceinline__ void cmul(double& r, double& i, double a, double b)
{
    const double t = fma(r, a, -(i * b));
    i = fma(r, b, i * a);
    r = t;
}

constexpr int kOrders = (kDegree + 16) / 16 * 16;   // orders in whole sets of 16

// one part of the z-recurrences of orders M0 + m', from the seeds (x + iy)^m, into the sums: step
// t takes degree m + t of every order m (degrees past kDegree are formed and dropped).  cl: the
// table of c_{m+t,m} by t and m
template <int M0, int NL>
__device__ __forceinline__ void p2m_orders(const double* cl, double z, double r2, double w, int mloc, double seed,
                                           double (&acc)[NL])
{
    double q1 = seed, q2 = 0.0;
    int at = M0 + mloc;
    asm volatile("" : "+v"(at));   // keeps the c_lm from being held in registers over the point loop
    acc[0] = __builtin_amdgcn_mfma_f64_4x4x4f64(seed, w, acc[0], 0, 0, 0);
#pragma unroll
    for (int t = 1; t < NL; ++t) {
        const double q = fma(z, q1, -((cl[t * kOrders + at] * r2) * q2));
        acc[t] = __builtin_amdgcn_mfma_f64_4x4x4f64(q, w, acc[t], 0, 0, 0);
        q2 = q1;
        q1 = q;
    }
}

// a wave's sums to LDS: lane (j = lane & 3, order M0 + 4 ((lane >> 2) & 3) + (lane >> 4))
template <int M0, int NL>
__device__ __forceinline__ void p2m_store(double* G, int lane, int part, bool add, const double (&acc)[NL])
{
    const int j = lane & 3, m = M0 + 4 * ((lane >> 2) & 3) + (lane >> 4);
    if (m > kDegree) return;
    double* o = G + 8 * term(m, m) + 2 * j + part;
#pragma unroll
    for (int t = 0; t < NL; ++t)
        if (m + t <= kDegree) o[8 * t] = add ? o[8 * t] + acc[t] : acc[t];
}

__global__ void __launch_bounds__(512, 4) k_tree_p2m(TreeGeom t, int64_t ncut, const int* __restrict__ start, GPtr pts,
                                                     double* __restrict__ coef)
{
    static_assert((kDegree + 1) * kOrders <= 8 * kTerms, "table space");
    __shared__ double G[8 * kTerms];   // per term: the complex sums of F q, u_x q, u_y q, u_z q
    const int box = blockIdx.x;
    const int p0 = start[box], p1 = start[box + 1];
    if (p0 == p1) return;
    double c[3];
    box_centre(t, box, c);
    const int lane = (int)(threadIdx.x & 63);
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)), part = (w >> 1) & 1, half = w >> 2;
    const int mloc = lane & 15, pt = lane >> 4;
    // the component of this lane's weight: F, u_x, u_y or u_z
    const double* wp = pts + ((lane & 3) == 0 ? 6 : 2 + (lane & 3)) * ncut;
    double nx, ny, nz, nw;
    auto load = [&](int u) {
        const int at = min(u + pt, p1 - 1);
        nx = component(pts, ncut, 0, (unsigned)at);
        ny = component(pts, ncut, 1, (unsigned)at);
        nz = component(pts, ncut, 2, (unsigned)at);
        nw = wp[at];
        nw = u + pt < p1 ? nw : 0.0;
    };
    double x, y, z, r2, wt, sr, si;
    // the points of step u, from the loads before; (x + iy)^mloc in sr, si, (x + iy)^16 in x, y
    auto step = [&](int u) {
        x = (nx - c[0]) * t.rinv;
        y = (ny - c[1]) * t.rinv;
        z = (nz - c[2]) * t.rinv;
        wt = nw;
        load(u + 8);
        r2 = fma(x, x, fma(y, y, z * z));
        sr = 1.0;
        si = 0.0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            double tr = sr, ti = si;
            cmul(tr, ti, x, y);
            const bool on = (mloc >> b) & 1;
            sr = on ? tr : sr;
            si = on ? ti : si;
            csq(x, y);
        }
    };
    // c_lm in the space of the sums, which are written when all waves are through with it
    for (int e = (int)threadIdx.x; e < (kDegree + 1) * kOrders; e += 512) {
        const int m = e % kOrders, l = m + e / kOrders;
        G[e] = l >= 2 ? (double)((l - 1) * (l - 1) - m * m) / (double)((2 * l - 1) * (2 * l - 3)) : 0.0;
    }
    load(p0 + 4 * half);
    __syncthreads();
    const double* cl = G;
    if ((w & 1) == 0) {
        constexpr int NL = kDegree + 1;
        double acc[NL];
#pragma unroll
        for (int l = 0; l < NL; ++l) acc[l] = 0.0;
        for (int u = p0 + 4 * half; u < p1; u += 8) {
            step(u);
            p2m_orders<0, NL>(cl, z, r2, wt, mloc, part ? si : sr, acc);
        }
        __syncthreads();
        if (half == 0) p2m_store<0, NL>(G, lane, part, false, acc);
        __syncthreads();
        if (half == 1) p2m_store<0, NL>(G, lane, part, true, acc);
    } else {
        constexpr int N1 = kDegree + 1 - 16, N2 = kDegree + 1 - 32;   // degrees of the orders from 16 and from 32 on
        double a1[N1], a2[N2];
#pragma unroll
        for (int l = 0; l < N1; ++l) a1[l] = 0.0;
#pragma unroll
        for (int l = 0; l < N2; ++l) a2[l] = 0.0;
        for (int u = p0 + 4 * half; u < p1; u += 8) {
            step(u);
            cmul(sr, si, x, y);
            p2m_orders<16, N1>(cl, z, r2, wt, mloc, part ? si : sr, a1);
            cmul(sr, si, x, y);
            p2m_orders<32, N2>(cl, z, r2, wt, mloc, part ? si : sr, a2);
        }
        __syncthreads();
        if (half == 0) {
            p2m_store<16, N1>(G, lane, part, false, a1);
            p2m_store<32, N2>(G, lane, part, false, a2);
        }
        __syncthreads();
        if (half == 1) {
            p2m_store<16, N1>(G, lane, part, true, a1);
            p2m_store<32, N2>(G, lane, part, true, a2);
        }
    }
    __syncthreads();
    // coefficients: Re and Im of M_lm / rs, then of D_lm / rs^2
    double* out = coef + (int64_t)box * (4 * kTerms);
    for (int e = threadIdx.x; e < kTerms; e += 512) {
        const int l = kTab.l[e], m = kTab.m[e];
        if (l > kDegree) {
            for (int q = 0; q < 4; ++q) out[4 * e + q] = 0.0;
            continue;
        }
        const double nm = kTab.n[e] * t.rinv;
        double dr = 0.0, di = 0.0;
        if (l > 0) {
            const double q = 1.0 / (double)(2 * l - 1);
            if (m <= l - 1) {
                const double* g = G + 8 * term(l - 1, m);
                const double k = (double)((l - m) * (l + m)) * q;
                dr = k * g[6];
                di = k * g[7];
            }
            if (m + 1 <= l - 1) {
                // (u_x - i u_y) q_{l-1,m+1}
                const double* g = G + 8 * term(l - 1, m + 1);
                const double k = (double)((l - m) * (l - m - 1)) * q * (m == 0 ? 1.0 : 0.5);
                dr = fma(-k, g[2] + g[5], dr);
                if (m > 0) di = fma(-k, g[3] - g[4], di);
            }
            if (m > 0) {
                // (u_x + i u_y) q_{l-1,m-1}
                const double* g = G + 8 * term(l - 1, m - 1);
                const double k = (double)((l + m) * (l + m - 1)) * q * 0.5;
                dr = fma(k, g[2] - g[5], dr);
                di = fma(k, g[3] + g[4], di);
            }
        }
        out[4 * e] = nm * G[8 * e];
        out[4 * e + 1] = nm * G[8 * e + 1];
        out[4 * e + 2] = -nm * t.rinv * dr;
        out[4 * e + 3] = -nm * t.rinv * di;
    }
}

// ---- the sums -------------------------------------------------------------------------------
// How a box acts on a group: its cut points s0 .. s1, and the degree of its expansion (0: point by
// point).  Both kernels below choose by this, one box per lane.
struct BoxRole {
    int s0, s1, deg;
};

__device__ __forceinline__ BoxRole box_role(const TreeGeom& t, const int* __restrict__ start, int box,
                                            const double* lo, const double* hi)
{
    BoxRole r{0, 0, 0};
    if (box >= t.nb[0] * t.nb[1] * t.nb[2]) return r;
    r.s0 = start[box];
    r.s1 = start[box + 1];
    double c[3], d2 = 0.0;
    box_centre(t, box, c);
    for (int d = 0; d < 3; ++d) {
        const double v = fmax(fmax(lo[d] - c[d], c[d] - hi[d]), 0.0);
        d2 = fma(v, v, d2);
    }
    // (rs/d)^(p+1) <= 1e-12: p + 1 >= 2 * 39.87 / log2((d/rs)^2)
    const float lg = __log2f((float)(d2 * t.rinv * t.rinv));
    if (lg > 0.5f) {
        const int p = (int)(79.74f / lg);
        // a term costs 7 instructions and a degree about 14 more, a cut point about 18
        const int cost = (7 * (p + 1) * (p + 2) / 2 + 14 * (p + 1)) / 18;
        if (p <= kDegree && cost < r.s1 - r.s0) r.deg = p > 1 ? p : 1;
    }
    return r;
}

// block b runs on XCD b mod 8: gives each XCD a contiguous range of groups (neighbours along the
// Hilbert curve), whose near boxes are mostly the same
__device__ __forceinline__ int xcd_order(int b, int n)
{
    const int q = n >> 3, rem = n & 7, xcd = b & 7;
    return xcd * q + (xcd < rem ? xcd : rem) + (b >> 3);
}

// the bounding box of a group, from one atom per lane
__device__ __forceinline__ void group_box(double x, double y, double z, double* lo, double* hi)
{
    lo[0] = hi[0] = x;
    lo[1] = hi[1] = y;
    lo[2] = hi[2] = z;
    for (int o = 32; o > 0; o >>= 1)
        for (int d = 0; d < 3; ++d) {
            lo[d] = fmin(lo[d], __shfl_xor(lo[d], o, 64));
            hi[d] = fmax(hi[d], __shfl_xor(hi[d], o, 64));
        }
}

// Expansions.  Wave (group, chunk): the chunk's boxes b = chunk, chunk + nfar, ... in index order,
// one atom per lane.  The coefficients are the same for the whole wave: they come through the
// scalar cache and enter the FP64 instructions as scalar operands, so that they cost neither
// vector registers nor LDS.  Per term: three instructions of the recurrence in 1/|R| and four
// multiply-adds; whole steps of kRow terms, rows padded with zeros (with a remainder loop, whose
// every pass waits for its scalar loads, 5.8 ms for 60,000 atoms and 1,900 boxes; 5.0 now, vector
// pipes busy 0.71 of the time).
__global__ void __launch_bounds__(256) k_tree_far(TreeGeom t, int n, const int* __restrict__ ids, GPtr at4,
                                                  const int* __restrict__ start, GPtr coef,
                                                  double* __restrict__ partial)
{
    const int lane = (int)(threadIdx.x & 63);
    const int group = __builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    const int chunk = (int)blockIdx.y;
    if (group * kGroup >= n) return;
    const bool act = group * kGroup + lane < n;
    const int u = act ? group * kGroup + lane : n - 1;
    const double x = -0.5 * at4[4 * u], y = -0.5 * at4[4 * u + 1], z = -0.5 * at4[4 * u + 2];
    double lo[3], hi[3];
    group_box(x, y, z, lo, hi);
    double sf = 0.0, sd = 0.0;
    const int nbox = t.nb[0] * t.nb[1] * t.nb[2];
    for (int base = chunk; base < nbox; base += 64 * t.nfar) {
        const BoxRole mine = box_role(t, start, base + lane * t.nfar, lo, hi);
        unsigned long long todo = __ballot(mine.deg > 0);
        while (todo) {
            const int k = __builtin_ctzll(todo);
            todo &= todo - 1;
            const int p = __builtin_amdgcn_readlane(mine.deg, k);
            const int box = base + k * t.nfar;
            double c[3];
            box_centre(t, box, c);
            const double X = (x - c[0]) * t.rinv, Y = (y - c[1]) * t.rinv, Z = (z - c[2]) * t.rinv;
            double jm = rsqrt_fp64(fma(X, X, fma(Y, Y, Z * Z)));
            const double ir2 = jm * jm, zr = Z * ir2;
            double C = 1.0, S = 0.0;
            const double *cf = coef + (int64_t)box * (4 * kTerms), *ct = kTab.c;
            for (int m = 0; m <= p; ++m) {
                double j1 = jm, j2 = 0.0;
                double fc = 0.0, fs = 0.0, dc = 0.0, ds = 0.0;
                // degrees m .. p in whole steps (those past p up to the step's end are as good)
                const int steps = (p - m + kRow) / kRow;
                for (int q = 0; q < steps; ++q) {
#pragma unroll
                    for (int i = 0; i < kRow; ++i) {
                        const int e = kRow * q + i;
                        double j;
                        if (i == 0 && q == 0)
                            j = jm;
                        else
                            j = fma(zr, j1, -((ct[e] * ir2) * j2));
                        fc = fma(j, cf[4 * e], fc);
                        fs = fma(j, cf[4 * e + 1], fs);
                        dc = fma(j, cf[4 * e + 2], dc);
                        ds = fma(j, cf[4 * e + 3], ds);
                        j2 = q == 0 && i == 0 ? 0.0 : j1;
                        j1 = j;
                    }
                }
                sf = fma(C, fc, fma(S, fs, sf));
                sd = fma(C, dc, fma(S, ds, sd));
                cmul(C, S, X, Y);
                jm *= ir2;
                const int row = (kDegree - m + kRow) / kRow * kRow;
                cf += 4 * row;
                ct += row;
            }
        }
    }
    if (act) {
        double* o = partial + ((int64_t)chunk * n + ids[u]) * 2;
        o[0] = sf;
        o[1] = sd;
    }
}

// Cut points one by one.  Block (group, chunk): the chunk's boxes b = chunk, chunk + nnear, ...;
// wave w has eight atoms of the group, in scalar registers, and its lanes take 64 cut points at a
// time, so that a cut point's 80 bytes are loaded once for eight pairs (the eight waves read the
// same points together) and every operand of a pair is at hand.  The lanes' sums are added in a
// fixed order at the end.  Bound by the FP64 issue rate: 8.4 ms for 1.2e10 pairs, vector pipes busy
// 0.96 of the time.  With one atom per lane and the points through the scalar cache 21 ms, with
// records of 80 bytes per point in place of one array per component 14 ms, without the points
// loaded ahead 16.5 ms.
constexpr int kNearAtoms = 8;
constexpr int kNearWaves = kGroup / kNearAtoms;

// one cut point per lane
struct NearPoint {
    double px, py, pz, ux, uy, uz, f, pp, pu2;
    __device__ __forceinline__ void load(GPtr pts, int64_t ncut, unsigned u)
    {
        auto at = [&](int k) { return component(pts, ncut, k, u); };
        px = at(0);
        py = at(1);
        pz = at(2);
        ux = at(3);
        uy = at(4);
        uz = at(5);
        f = at(6);
        pp = at(7);
        pu2 = at(8);
    }
    __device__ __forceinline__ void clear() { ux = uy = uz = f = pu2 = 0.0; }
};

struct NearAtoms {
    double mx[kNearAtoms], my[kNearAtoms], mz[kNearAtoms], aa[kNearAtoms], sf[kNearAtoms], sd[kNearAtoms];
    __device__ __forceinline__ void add(const NearPoint& c)
    {
#pragma unroll
        for (int q = 0; q < kNearAtoms; ++q) {
            const double r2 = fma(mx[q], c.px, fma(my[q], c.py, fma(mz[q], c.pz, c.pp + aa[q])));
            const double dn2 = fma(mx[q], c.ux, fma(my[q], c.uy, fma(mz[q], c.uz, c.pu2)));
            const double r = rsqrt_nb(r2);
            sf[q] = fma(c.f, r, sf[q]);
            sd[q] = fma(dn2, (r * r) * r, sd[q]);
        }
    }
};

__global__ void __launch_bounds__(64 * kNearWaves) k_tree_near(TreeGeom t, int n, int64_t ncut, const int* __restrict__ ids, GPtr at4,
                                                               const int* __restrict__ start, GPtr pts,
                                                               double* __restrict__ partial)
{
    const int lane = (int)(threadIdx.x & 63), group = xcd_order((int)blockIdx.x, (int)gridDim.x), chunk = (int)blockIdx.y;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    double lo[3], hi[3];
    {
        const int u = min(group * kGroup + lane, n - 1);
        group_box(-0.5 * at4[4 * u], -0.5 * at4[4 * u + 1], -0.5 * at4[4 * u + 2], lo, hi);
    }
    const int a0 = group * kGroup + w * kNearAtoms;
    if (a0 >= n) return;
    NearAtoms N;
#pragma unroll
    for (int q = 0; q < kNearAtoms; ++q) {
        const double* A = at4 + 4 * min(a0 + q, n - 1);
        N.mx[q] = A[0];
        N.my[q] = A[1];
        N.mz[q] = A[2];
        N.aa[q] = A[3];
        N.sf[q] = N.sd[q] = 0.0;
    }
    const int nbox = t.nb[0] * t.nb[1] * t.nb[2];
    for (int base = chunk; base < nbox; base += 64 * t.nnear) {
        const BoxRole mine = box_role(t, start, base + lane * t.nnear, lo, hi);
        unsigned long long todo = __ballot(mine.deg == 0 && mine.s1 > mine.s0);
        while (todo) {
            const int k = __builtin_ctzll(todo);
            todo &= todo - 1;
            const int u0 = __builtin_amdgcn_readlane(mine.s0, k), u1 = __builtin_amdgcn_readlane(mine.s1, k);
            // 64 points are worked on while the next 64 are on their way (past the end: the last point,
            // with nothing on it)
            NearPoint p, q;
            p.load(pts, ncut, (unsigned)min(u0 + lane, u1 - 1));
            for (int u = u0;;) {
                q.load(pts, ncut, (unsigned)min(u + 64 + lane, u1 - 1));
                if (u + lane >= u1) p.clear();
                N.add(p);
                if ((u += 64) >= u1) break;
                p.load(pts, ncut, (unsigned)min(u + 64 + lane, u1 - 1));
                if (u + lane >= u1) q.clear();
                N.add(q);
                if ((u += 64) >= u1) break;
            }
        }
    }
#pragma unroll
    for (int q = 0; q < kNearAtoms; ++q) {
        for (int o = 32; o > 0; o >>= 1) {
            N.sf[q] += __shfl_xor(N.sf[q], o, 64);
            N.sd[q] += __shfl_xor(N.sd[q], o, 64);
        }
        if (lane == q && a0 + q < n) {
            double* o = partial + ((int64_t)(t.nfar + chunk) * n + ids[a0 + q]) * 2;
            o[0] = N.sf[q];
            o[1] = 0.5 * N.sd[q];
        }
    }
}

inline unsigned nblk(int64_t n, int bs) { return (unsigned)((n + bs - 1) / bs); }
inline size_t up(size_t b) { return (b + 255) & ~(size_t)255; }

// the arrays of a plan in its work space: partial sums first (the reduction reads them there)
struct Arrays {
    double *partial, *coef, *at4;
    unsigned long long* keys;
    int *first, *last, *count, *start, *pos, *ids, *abin;
    size_t bytes;
};

Arrays arrays(const TreePlan& t, char* w)
{
    const TreeGeom& G = t.geom;
    const size_t nbox = (size_t)G.nb[0] * G.nb[1] * G.nb[2], nseg = nbox * G.B * G.B;
    const size_t nbin = (size_t)1 << 3 * G.bits;
    size_t o = 0;
    auto take = [&](size_t b) {
        char* p = w ? w + o : nullptr;
        o += up(b);
        return p;
    };
    Arrays A;
    A.partial = (double*)take(sizeof(double) * (size_t)energy_partial_doubles(t.n, G.nfar + G.nnear));
    A.coef = (double*)take(sizeof(double) * 4 * kTerms * nbox);
    A.at4 = (double*)take(sizeof(double) * 4 * (size_t)t.n);
    A.keys = (unsigned long long*)take(sizeof(unsigned long long) * (size_t)t.n);
    A.first = (int*)take(sizeof(int) * nseg);
    A.last = (int*)take(sizeof(int) * nseg);
    A.count = (int*)take(sizeof(int) * nbox);
    A.start = (int*)take(sizeof(int) * (nbox + 1));
    A.pos = (int*)take(sizeof(int) * (size_t)t.ncut);
    A.ids = (int*)take(sizeof(int) * (size_t)t.n);
    A.abin = (int*)take(sizeof(int) * (nbin + 1));
    A.bytes = o;
    return A;
}

}  // namespace

bool tree_plan(const Grid& g, const Atoms& at, const double* lo, const double* hi, double rmax, int64_t ncut,
               size_t bytes, TreePlan* out)
{
    TreePlan t;
    t.n = at.n;
    t.ncut = ncut;
    if (at.n < kTreeMinAtoms || (double)at.n * (double)ncut < kTreeMinPairs || ncut >= (int64_t)1 << 28) return false;
    TreeGeom& G = t.geom;
    G.S = g.S;
    G.ny = g.ny;
    // the lattice cells that hold cut points: those the balls reach, with one cell to spare
    const double org[3] = {g.ox, g.oy, g.oz}, c[3] = {at.cx, at.cy, at.cz};
    const int nn[3] = {g.nx, g.ny, g.nz};
    int cells[3];
    double vol = 1.0, ext[3];
    for (int d = 0; d < 3; ++d) {
        const double f0 = std::floor((lo[d] - rmax - org[d]) / g.h) - g.off[d] - 1.0;
        const double f1 = std::floor((hi[d] + rmax - org[d]) / g.h) - g.off[d] + 1.0;
        G.c0[d] = (int)std::min(std::max(f0, 0.0), (double)(nn[d] - 2));
        cells[d] = (int)std::min(std::max(f1, (double)G.c0[d]), (double)(nn[d] - 2)) - G.c0[d] + 1;
        ext[d] = hi[d] - lo[d];
        vol *= ext[d] + 2.0 * rmax;
    }
    // at most two bins per atom, down to about 2.5 A (an atom or two each)
    const double longest = std::max(ext[0], std::max(ext[1], ext[2]));
    G.bits = 1;
    while (G.bits < kMaxBits && longest > 2.5 * (double)(1 << G.bits) && 8 << 3 * G.bits <= 2 * at.n) ++G.bits;
    G.ainv = (double)(1 << kCurveBits) / std::max(longest, 1e-3);
    for (int d = 0; d < 3; ++d) G.alo[d] = lo[d];
    const int64_t groups = (at.n + kGroup - 1) / kGroup;
    auto split = [&](int64_t want) { return (int)std::min<int64_t>(64, std::max<int64_t>(1, (want + groups - 1) / groups)); };
    G.nfar = split(kFarWaves);
    G.nnear = split(kNearBlocks);
    // boxes of about kBoxPoints cut points where the bounding box is full to pi/6, as a globule
    // fills its own, smaller ones where those would be too few to share the work of the expansions
    // (5000 atoms, 3.5e5 points: 1.39 ms with 700 points per box, 1.57 with 1500), and larger ones
    // where the work space asks for fewer
    const double aim = std::min((double)kBoxPoints, std::max((double)kMinBoxPoints, (double)ncut / kBoxes));
    const double side = std::cbrt(vol * 0.5236 * aim / (double)ncut);
    int B = (int)std::min(std::max(std::floor(side / g.h + 0.5), 2.0), (double)kMaxSide);
    for (; B <= kMaxSide; ++B) {
        G.B = B;
        int64_t nbox = 1;
        for (int d = 0; d < 3; ++d) {
            G.nb[d] = (cells[d] + B - 1) / B;
            nbox *= G.nb[d];
        }
        if (nbox * B * B >= (int64_t)1 << 30) continue;
        if (arrays(t, nullptr).bytes <= bytes) break;
    }
    if (B > kMaxSide) return false;
    G.side = g.h * (double)B;
    // A box acts on a group by its expansion from about twice its half-diagonal on.  Where the balls fill
    // little of the bounding box (an atom far from the rest), or the work space asks for large boxes, that
    // distance and the group's own extent can take in most of the solute; the direct sum is the faster one
    // from half of it on.  Direct sum and expansions in ms by that share: 0.28 2.20 and 1.64, 0.41 5.67
    // and 4.28, 0.45 4.98 and 3.98, 0.56 2.13 and 2.39, 0.67 9.4 and 10.2, 0.95 1.59 and 3.18.
    const double occupied = 0.5236 * std::min(vol, (double)at.n * 8.0 * rmax * rmax * rmax);
    const double near = 1.74 * G.side + std::cbrt(kGroup * occupied / (double)at.n);
    if (4.19 * near * near * near > 0.5 * occupied) return false;
    for (int d = 0; d < 3; ++d)
        G.ctr[d] = (org[d] - c[d]) + g.h * ((double)(G.c0[d] + g.off[d]) + 0.5 * (double)B);
    G.rinv = 1.0 / (0.5 * std::sqrt(3.0) * G.side * (1.0 + 1e-9));
    *out = t;
    return true;
}

hipError_t launch_tree_order(hipStream_t s, const TreePlan& t, const Atoms& at, const int64_t* cutkey, void* work,
                             const int** pos)
{
    const TreeGeom& G = t.geom;
    const Arrays A = arrays(t, (char*)work);
    const int nbox = G.nb[0] * G.nb[1] * G.nb[2];
    const int nbin = 1 << 3 * G.bits;
    hipError_t e = launch_fill(s, A.first, (size_t)((char*)A.count - (char*)A.first));
    if (e != hipSuccess) return e;
    k_tree_seg<<<nblk(t.ncut, 256), 256, 0, s>>>(G, t.ncut, cutkey, A.first, A.last);
    k_tree_box<<<nbox, 256, 0, s>>>(G, A.first, A.last, A.count);
    e = launch_scan1(s, A.count, nbox, A.start);
    if (e != hipSuccess) return e;
    k_tree_pos<<<nblk(t.ncut, 256), 256, 0, s>>>(G, t.ncut, cutkey, A.last, A.start, A.pos);
    e = launch_fill(s, A.abin, up(sizeof(int) * (size_t)(nbin + 1)));
    if (e != hipSuccess) return e;
    k_tree_acount<<<nblk(at.n, 256), 256, 0, s>>>(G, at, A.abin);
    e = launch_scan1(s, A.abin, nbin, A.abin);
    if (e != hipSuccess) return e;
    k_tree_ascatter<<<nblk(at.n, 256), 256, 0, s>>>(G, at, A.abin, A.keys);
    k_tree_aorder<<<nblk(at.n, 256), 256, 0, s>>>(G, at, A.abin, A.keys, A.ids, A.at4);
    *pos = A.pos;
    return hipGetLastError();
}

hipError_t launch_tree_sums(hipStream_t s, const TreePlan& t, const double* pts, void* work)
{
    const TreeGeom& G = t.geom;
    const Arrays A = arrays(t, (char*)work);
    k_tree_p2m<<<G.nb[0] * G.nb[1] * G.nb[2], 512, 0, s>>>(G, t.ncut, A.start, pts, A.coef);
    k_tree_far<<<dim3(nblk(t.n, 4 * kGroup), (unsigned)G.nfar), 256, 0, s>>>(G, t.n, A.ids, A.at4, A.start, A.coef,
                                                                            A.partial);
    k_tree_near<<<dim3(nblk(t.n, kGroup), (unsigned)G.nnear), 64 * kNearWaves, 0, s>>>(G, t.n, t.ncut, A.ids, A.at4, A.start,
                                                                                      pts, A.partial);
    return hipGetLastError();
}

}  // namespace pbk

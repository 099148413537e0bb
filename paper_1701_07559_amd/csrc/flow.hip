// Wilson gradient flow of the gauge links (the smearing the paper applies to
// its ensembles before the valence solves, Sec. III, at flow time t_gf = 1),
// in FP64 on canonical links U[t][z][y][x][mu][3][3].
//
// Flow equation (Luscher's Wilson flow, cited in Sec. III):
//   dV/dt = Z(V) V,  Z_mu(x) = -1/2 (O - O^+) + 1/6 tr(O - O^+),
//   O_mu(x) = U_mu(x) * (sum of the six staples of the link),
// integrated with the third-order Runge-Kutta scheme of the same reference
// in its low-storage form: per stage i, E_i = a_i eps Z(W_i) + b_i E_{i-1}
// and W_{i+1} = exp(E_i) W_i with (a, b) = (1/4, 0), (8/9, -17/9), (3/4, -1).
//
// One kernel launch per stage, on fields laid out [mu][entry][site] between the
// first and the last: a wave owns one direction of 64 consecutive sites, so each
// of its loads is 64 adjacent entries.  A thread reads the stage's input field
// (its link and the six staples; staple links by their first two rows), writes
// E_i for that link (its eight independent reals) and the updated link into a
// second buffer, so every staple sees the stage's input.
#include <cmath>
#include <cstdio>
#include <vector>

#include "ctx.h"

namespace mdwf {
namespace {

constexpr int kFlowBlock = 256;
// largest entry of U U^+ - 1 and of det U - 1 the flow accepts
constexpr double kSu3Tol = 1e-10;

struct Su3 {
    cx<double> m[9];
};

__device__ __forceinline__ cx<double> ld(const double2* p) {
    const double2 v = *p;
    return {v.x, v.y};
}
// stored past L2, which the stage's links need
__device__ __forceinline__ void st_past(double2* p, double a, double b) {
    __builtin_nontemporal_store(nd2{a, b}, reinterpret_cast<nd2*>(p));
}
__device__ __forceinline__ Su3 ld_link(const double2* U, long link) {
    Su3 r;
    const double2* p = U + link * 9;
#pragma unroll
    for (int k = 0; k < 9; ++k) r.m[k] = ld(p + k);
    return r;
}

// A staple link from its first two rows: for U in SU(3) (unitary, det U = 1)
// the third row is the complex conjugate of the cross product of the first
// two, so six of the nine entries are loaded and three are computed.  The
// flow keeps every link in SU(3) up to rounding, and the staple gathers, not
// the arithmetic, bound the stage.
__device__ __forceinline__ cx<double> conj_cross(cx<double> a, cx<double> b, cx<double> c, cx<double> d) {
    const cx<double> v = cmadd(cmul(a, b), cx<double>{-c.re, -c.im}, d);   // a b - c d
    return {v.re, -v.im};
}
__device__ __forceinline__ void third_row(Su3& r) {
    r.m[6] = conj_cross(r.m[1], r.m[5], r.m[2], r.m[4]);
    r.m[7] = conj_cross(r.m[2], r.m[3], r.m[0], r.m[5]);
    r.m[8] = conj_cross(r.m[0], r.m[4], r.m[1], r.m[3]);
}

// The Runge-Kutta accumulator E is traceless antihermitian: eight reals per
// link, stored as four double2 (Im E00, Im E11; E01; E02; E12).
// complete_alg fills in the other entries from those eight.
__device__ __forceinline__ void complete_alg(Su3& r) {
    r.m[0].re = 0.0;
    r.m[4].re = 0.0;
    r.m[8] = {0.0, -(r.m[0].im + r.m[4].im)};
    r.m[3] = {-r.m[1].re, r.m[1].im};
    r.m[6] = {-r.m[2].re, r.m[2].im};
    r.m[7] = {-r.m[5].re, r.m[5].im};
}
// a b, a b^+
__device__ __forceinline__ Su3 mul(const Su3& a, const Su3& b) {
    Su3 r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cx<double> s = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < 3; ++k) s = cmadd(s, a.m[i * 3 + k], b.m[k * 3 + j]);
            r.m[i * 3 + j] = s;
        }
    return r;
}
__device__ __forceinline__ Su3 mul_nd(const Su3& a, const Su3& b) {   // a b^+
    Su3 r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            cx<double> s = {0.0, 0.0};
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const cx<double> bc = {b.m[j * 3 + k].re, -b.m[j * 3 + k].im};
                s = cmadd(s, a.m[i * 3 + k], bc);
            }
            r.m[i * 3 + j] = s;
        }
    return r;
}

// exp(X) for a traceless antihermitian X: scale by 2^-k until the Frobenius
// norm is at most 1/4, Taylor polynomial of degree 12 by Horner's rule, then
// square k times (truncation below 1e-17 relative).  By Cayley and Hamilton
// X^3 = t X + det X with t = tr X^2 / 2 real and det X = i e imaginary, so
// Horner's R = 1 + X R / d runs on the three complex coefficients of
// R = r0 + r1 X + r2 X^2: some ten operations a step for a product of matrices.
__device__ __forceinline__ Su3 expm_small(Su3 X) {
    // off-diagonal moduli; X_kk = i a_k
    auto n2 = [](cx<double> v) { return v.re * v.re + v.im * v.im; };
    double t = -0.5 * (X.m[0].im * X.m[0].im + X.m[4].im * X.m[4].im + X.m[8].im * X.m[8].im) -
               (n2(X.m[1]) + n2(X.m[2]) + n2(X.m[5]));
    int sq = 0;
    double scale = 1.0;
    const double n = sqrt(-2.0 * t);
    while (n * scale > 0.25 && sq < 40) {
        scale *= 0.5;
        ++sq;
    }
#pragma unroll
    for (int k = 0; k < 9; ++k) X.m[k] = scale * X.m[k];
    t *= scale * scale;
    const double a0 = X.m[0].im, a1 = X.m[4].im, a2 = X.m[8].im;
    const double n01 = n2(X.m[1]), n02 = n2(X.m[2]), n12 = n2(X.m[5]);
    const cx<double> p = cmul(X.m[1], X.m[5]);   // X01 X12
    // det X = i e
    const double e = a0 * n12 + a1 * n02 + a2 * n01 - a0 * a1 * a2 - 2.0 * (p.im * X.m[2].re - p.re * X.m[2].im);
    // X^2, hermitian
    const double d0 = -(a0 * a0 + n01 + n02), d1 = -(a1 * a1 + n01 + n12), d2 = -(a2 * a2 + n02 + n12);
    auto ti = [](double a, cx<double> v) { return cx<double>{-a * v.im, a * v.re}; };   // i a v
    auto cj = [](cx<double> v) { return cx<double>{v.re, -v.im}; };
    const cx<double> q01 = cmadd(ti(a0 + a1, X.m[1]), X.m[2], X.m[7]);
    const cx<double> q02 = ti(a0 + a2, X.m[2]) + p;
    const cx<double> q12 = cmadd(ti(a1 + a2, X.m[5]), X.m[3], X.m[2]);
    cx<double> r0 = {1.0, 0.0}, r1 = {0.0, 0.0}, r2 = {0.0, 0.0};
#pragma unroll
    for (int d = 12; d >= 1; --d) {
        const double inv = 1.0 / d;
        const cx<double> s1 = inv * (r0 + t * r2);
        r0 = {1.0 - inv * e * r2.im, inv * e * r2.re};
        r2 = inv * r1;
        r1 = s1;
    }
    Su3 R;
    const cx<double> q[9] = {{d0, 0.0}, q01, q02, cj(q01), {d1, 0.0}, q12, cj(q02), cj(q12), {d2, 0.0}};
#pragma unroll
    for (int k = 0; k < 9; ++k) {
        cx<double> v = cmul(r1, X.m[k]);
        if (k % 4 == 0) v = v + r0 + q[k].re * r2;
        else v = cmadd(v, r2, q[k]);
        R.m[k] = v;
    }
    for (int s = 0; s < sq; ++s) R = mul(R, R);
    return R;
}

struct FlowGeo {
    int X, Y, Z, T;
};

__device__ __forceinline__ long nbr(const FlowGeo& g, int x, int y, int z, int t, int mu, int d) {
    if (mu == 0) x = (x + d + g.X) % g.X;
    else if (mu == 1) y = (y + d + g.Y) % g.Y;
    else if (mu == 2) z = (z + d + g.Z) % g.Z;
    else t = (t + d + g.T) % g.T;
    return long(x) + long(g.X) * (y + long(g.Y) * (z + long(g.Z) * t));
}

__device__ __forceinline__ uint32_t sel4(int d, int a, int b, int c, int e) {
    int v = d == 1 ? b : a;
    v = d == 2 ? c : v;
    return uint32_t(d == 3 ? e : v);
}

constexpr int kFlowSites = 64;    // sites of a workgroup, one per lane; a wave per direction
constexpr int kSitePitch = 37;    // double2 of a site's four links in LDS, padded off the banks

// Traversal of a stage: slabs of bz planes, t inside, then z, y, x; every XCD
// sweeps one contiguous part, so a slab's time planes stay in its L2.
struct FlowTrav {
    FastDiv slab, plane, xy, x;   // sites of a slab (bz planes), of one time plane of it, X Y, X
    int bz;
    uint32_t nsites;
};

// one Runge-Kutta stage for every link: E = a Z(Win) + b E, Wout = exp(E) Win.
// CANON: Wout in the canonical layout (through LDS), otherwise [mu][entry][site].
//
// A link's six staples take 18 neighbouring links.  Read from the canonical
// layout each lane of a load touches its own cache line; that, the address
// unit's rate, and products of full matrices made this stage 1077 us at
// 24^3 x 64.  Here adjacent lanes read adjacent entries, only two rows of every
// SU(3) product are computed, and the four directions of a site, a wave each,
// share what they can through LDS: U_nu(x), U_nu(x-nu) (three waves) and
// U_nu(x+mu) (the waves of mu and nu, which go through the planes in step).
// That leaves 73 loads a link of 121, and some 430 us, FP64 issue busy
// over half the time.
// Three waves a SIMD (168 registers, 48 KB a workgroup) are worth more than
// loads ahead of their use: with the next staple's in flight, 204 registers
// and two waves, it runs 9 % slower.
template <bool CANON>
__global__ void __launch_bounds__(4 * kFlowSites) k_flow_stage(const FlowGeo g, const FlowTrav tv, const double2* Win,
                                                               double2* Wout, double2* E, double a, double b) {
    __shared__ double2 lds[2 * 24 * kFlowSites];
    double2* own = lds;                       // [mu][entry][lane]: rows of U_mu(x)
    double2* ex = lds + 24 * kFlowSites;      // of U_mu(x-mu), then of the links the waves exchange
    const int lane = threadIdx.x & 63;
    const int mu = __builtin_amdgcn_readfirstlane(int(threadIdx.x >> 6));
    const uint32_t V = tv.nsites;
    const uint32_t first = uint32_t(xcd_logical_block(blockIdx.x, gridDim.x)) * kFlowSites;
    const bool valid = first + lane < V;
    const uint32_t pos = valid ? first + lane : V - 1;   // idle lanes repeat the last site, storing nothing
    const uint32_t sl = tv.slab.div(pos), in = pos - sl * tv.slab.d;
    const int z0 = int(sl) * tv.bz;
    // the last slab may be thinner
    const bool whole = z0 + tv.bz <= g.Z;
    const uint32_t pl = whole ? tv.plane.d : uint32_t(g.Z - z0) * tv.xy.d;
    const int t = int(whole ? tv.plane.div(in) : in / pl);
    const uint32_t r = in - uint32_t(t) * pl;
    const uint32_t zz = tv.xy.div(r), r2 = r - zz * tv.xy.d;
    const int y = int(tv.x.div(r2)), x = int(r2 - uint32_t(y) * tv.x.d), z = z0 + int(zz);
    const int sy = g.X, sz = g.X * g.Y, sT = sz * g.Z;
    const uint32_t site = uint32_t(x + sy * y + sz * z) + uint32_t(sT) * uint32_t(t);
    // site offsets of the neighbours
    const int f0 = x == g.X - 1 ? 1 - g.X : 1, f1 = y == g.Y - 1 ? (1 - g.Y) * sy : sy;
    const int f2 = z == g.Z - 1 ? (1 - g.Z) * sz : sz, f3 = t == g.T - 1 ? (1 - g.T) * sT : sT;
    const int b0 = x == 0 ? g.X - 1 : -1, b1 = y == 0 ? (g.Y - 1) * sy : -sy;
    const int b2 = z == 0 ? (g.Z - 1) * sz : -sz, b3 = t == 0 ? (g.T - 1) * sT : -sT;
    auto entry = [&](int d, int k, uint32_t i) {
        return ld(reinterpret_cast<const double2*>(reinterpret_cast<const char*>(Win + size_t(d * 9 + k) * V) +
                                                   i * 16u));
    };
    auto rows = [&](int d, uint32_t i) {   // the first two rows
        Su3 r;
#pragma unroll
        for (int k = 0; k < 6; ++k) r.m[k] = entry(d, k, i);
        return r;
    };
    auto put = [&](double2* p, int d, const Su3& v) {
#pragma unroll
        for (int k = 0; k < 6; ++k) p[(d * 6 + k) * kFlowSites + lane] = make_double2(v.m[k].re, v.m[k].im);
    };
    auto get = [&](const double2* p, int d) {
        Su3 r;
#pragma unroll
        for (int k = 0; k < 6; ++k) r.m[k] = ld(p + (d * 6 + k) * kFlowSites + lane);
        return r;
    };
    const uint32_t xp = site + sel4(mu, f0, f1, f2, f3);
    put(ex, mu, rows(mu, site + sel4(mu, b0, b1, b2, b3)));
    put(own, mu, rows(mu, site));
    __syncthreads();
    Su3 S;
#pragma unroll
    for (int k = 0; k < 9; ++k) S.m[k] = {0.0, 0.0};
    // a staple is in SU(3): its third row follows from the first two, as a link's does
#pragma unroll 1
    for (int j = 1; j < 4; ++j) {   // lower staples (U_mu(x-nu) U_nu(x+mu-nu))^+ U_nu(x-nu)
        const int nu = mu ^ j;
        const uint32_t dn = sel4(nu, b0, b1, b2, b3);
        Su3 A = rows(nu, xp + dn), B = rows(mu, site + dn), C = get(ex, nu);
        third_row(B);
        A.m[6] = conj_cross(A.m[1], A.m[5], A.m[2], A.m[4]);
        A.m[7] = conj_cross(A.m[2], A.m[3], A.m[0], A.m[5]);
        cx<double> Q[6];   // the first two columns of U_mu U_nu
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                cx<double> v = {0.0, 0.0};
#pragma unroll
                for (int k = 0; k < 3; ++k) v = cmadd(v, B.m[l * 3 + k], A.m[k * 3 + i]);
                Q[i * 3 + l] = v;
            }
        third_row(C);
        Su3 s2;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                cx<double> v = {0.0, 0.0};
#pragma unroll
                for (int k = 0; k < 3; ++k) v = cjmadd(v, Q[i * 3 + k], C.m[k * 3 + l]);
                s2.m[i * 3 + l] = v;
            }
        third_row(s2);
#pragma unroll
        for (int k = 0; k < 9; ++k) S.m[k] = S.m[k] + s2.m[k];
    }
#pragma unroll 1
    for (int j = 1; j < 4; ++j) {   // upper staples U_nu(x+mu) U_mu(x+nu)^+ U_nu(x)^+
        const int nu = mu ^ j;
        const Su3 A = rows(nu, xp);   // the wave of nu needs it too and loads U_mu(x+nu)
        __syncthreads();
        put(ex, mu, A);
        __syncthreads();
        Su3 B = get(ex, nu), C = get(own, nu);
        third_row(B);
        cx<double> P[6];
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                cx<double> v = {0.0, 0.0};
#pragma unroll
                for (int k = 0; k < 3; ++k) v = cjmadd(v, B.m[l * 3 + k], A.m[i * 3 + k]);
                P[i * 3 + l] = v;
            }
        third_row(C);
        Su3 s1;
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int l = 0; l < 3; ++l) {
                cx<double> v = {0.0, 0.0};
#pragma unroll
                for (int k = 0; k < 3; ++k) v = cjmadd(v, C.m[l * 3 + k], P[i * 3 + k]);
                s1.m[i * 3 + l] = v;
            }
        third_row(s1);
#pragma unroll
        for (int k = 0; k < 9; ++k) S.m[k] = S.m[k] + s1.m[k];
    }
    Su3 U = get(own, mu);
#pragma unroll
    for (int k = 6; k < 9; ++k) U.m[k] = entry(mu, k, site);
    const Su3 O = mul(U, S);
    // Z = -1/2 (O - O^+) + 1/6 tr(O - O^+); tr(O - O^+) = 2 i Im tr O.
    // The eight independent entries of E (upper triangle, first two
    // diagonal ones); the rest follow from antihermiticity and zero trace
    const double itr = (O.m[0].im + O.m[4].im + O.m[8].im) / 3.0;
    Su3 Ev;
    double2* Ep = E + size_t(mu * 4) * V + site;
    Ev.m[0] = {0.0, a * (itr - O.m[0].im)};
    Ev.m[4] = {0.0, a * (itr - O.m[4].im)};
    Ev.m[1] = {-0.5 * a * (O.m[1].re - O.m[3].re), -0.5 * a * (O.m[1].im + O.m[3].im)};
    Ev.m[2] = {-0.5 * a * (O.m[2].re - O.m[6].re), -0.5 * a * (O.m[2].im + O.m[6].im)};
    Ev.m[5] = {-0.5 * a * (O.m[5].re - O.m[7].re), -0.5 * a * (O.m[5].im + O.m[7].im)};
    if (b != 0.0 && valid) {
        const double2 d = Ep[0];
        Ev.m[0].im += b * d.x;
        Ev.m[4].im += b * d.y;
        Ev.m[1] = Ev.m[1] + b * ld(Ep + V);
        Ev.m[2] = Ev.m[2] + b * ld(Ep + 2 * size_t(V));
        Ev.m[5] = Ev.m[5] + b * ld(Ep + 3 * size_t(V));
    }
    if (valid) {
        st_past(Ep, Ev.m[0].im, Ev.m[4].im);
        st_past(Ep + V, Ev.m[1].re, Ev.m[1].im);
        st_past(Ep + 2 * size_t(V), Ev.m[2].re, Ev.m[2].im);
        st_past(Ep + 3 * size_t(V), Ev.m[5].re, Ev.m[5].im);
    }
    complete_alg(Ev);
    const Su3 Wn = mul(expm_small(Ev), U);
    if constexpr (!CANON) {
        if (valid) {
#pragma unroll
            for (int k = 0; k < 9; ++k)
                st_past(Wout + size_t(mu * 9 + k) * V + site, Wn.m[k].re, Wn.m[k].im);
        }
    } else {
        __shared__ uint32_t at[kFlowSites];
        __syncthreads();   // every wave has read the links
        if (mu == 0) at[lane] = site;
#pragma unroll
        for (int k = 0; k < 9; ++k) lds[lane * kSitePitch + mu * 9 + k] = make_double2(Wn.m[k].re, Wn.m[k].im);
        __syncthreads();
        const uint32_t n = min(uint32_t(kFlowSites), V - first);
        for (uint32_t e = threadIdx.x; e < n * 36; e += 4 * kFlowSites) {
            const uint32_t i = e / 36, k = e - 36 * i;
            Wout[size_t(at[i]) * 36 + k] = lds[i * kSitePitch + k];
        }
    }
}

// The links between the canonical layout and [mu][entry][site] (TO_SOA or back).
template <bool TO_SOA>
__global__ void __launch_bounds__(4 * kFlowSites) k_flow_layout(const double2* in, double2* out, uint32_t V) {
    __shared__ double2 sh[kFlowSites * kSitePitch];
    const int lane = threadIdx.x & 63, mu = threadIdx.x >> 6;
    const uint32_t s0 = blockIdx.x * kFlowSites;
    const uint32_t n = min(uint32_t(kFlowSites), V - s0);
    if constexpr (TO_SOA) {
        for (uint32_t e = threadIdx.x; e < n * 36; e += 4 * kFlowSites)
            sh[(e / 36) * kSitePitch + e % 36] = in[size_t(s0) * 36 + e];
        __syncthreads();
        if (uint32_t(lane) < n)
#pragma unroll
            for (int k = 0; k < 9; ++k) out[size_t(mu * 9 + k) * V + s0 + lane] = sh[lane * kSitePitch + mu * 9 + k];
    } else {
        if (uint32_t(lane) < n)
#pragma unroll
            for (int k = 0; k < 9; ++k) sh[lane * kSitePitch + mu * 9 + k] = in[size_t(mu * 9 + k) * V + s0 + lane];
        __syncthreads();
        for (uint32_t e = threadIdx.x; e < n * 36; e += 4 * kFlowSites)
            out[size_t(s0) * 36 + e] = sh[(e / 36) * kSitePitch + e % 36];
    }
}

// sum over the six planes of Re tr U_mu nu(x), block partials in a fixed order
__global__ void __launch_bounds__(kFlowBlock) k_plaquette(const FlowGeo g, const double2* U, double* partials,
                                                          long nsites) {
    const long site = long(blockIdx.x) * blockDim.x + threadIdx.x;
    double v = 0.0;
    if (site < nsites) {
        const int x = int(site % g.X);
        const int y = int((site / g.X) % g.Y);
        const int z = int((site / (long(g.X) * g.Y)) % g.Z);
        const int t = int(site / (long(g.X) * g.Y * g.Z));
        for (int mu = 0; mu < 4; ++mu)
            for (int nu = mu + 1; nu < 4; ++nu) {
                const Su3 a = mul(ld_link(U, site * 4 + mu), ld_link(U, nbr(g, x, y, z, t, mu, 1) * 4 + nu));
                const Su3 c = mul_nd(a, ld_link(U, nbr(g, x, y, z, t, nu, 1) * 4 + mu));
                const Su3 p = mul_nd(c, ld_link(U, site * 4 + nu));
                v += p.m[0].re + p.m[4].re + p.m[8].re;
            }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v += __shfl_xor(v, off, 64);
    __shared__ double ws[kFlowBlock / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) ws[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double s = 0.0;
#pragma unroll
        for (int w = 0; w < kFlowBlock / 64; ++w) s += ws[w];
        partials[blockIdx.x] = s;
    }
}

// Largest deviation from SU(3) of the links of a block of sites: max over
// each site's four links of the entries of U U^+ - 1 and of det U - 1 (re
// and im parts), so a field the flow stage's two-row staple loads would
// misread is refused.  NaN propagates into the partial.
__device__ __forceinline__ double max_nan(double v, double x) { return (x > v || x != x) ? x : v; }

__global__ void __launch_bounds__(kFlowBlock) k_su3_deviation(const double2* U, double* partials, long nsites) {
    const long site = long(blockIdx.x) * blockDim.x + threadIdx.x;
    double v = 0.0;
    if (site < nsites) {
        for (int mu = 0; mu < 4; ++mu) {
            const Su3 a = ld_link(U, site * 4 + mu);
            const Su3 p = mul_nd(a, a);   // U U^+
#pragma unroll
            for (int k = 0; k < 9; ++k) {
                v = max_nan(v, fabs(p.m[k].re - ((k % 4 == 0) ? 1.0 : 0.0)));
                v = max_nan(v, fabs(p.m[k].im));
            }
            // det U = row 2 . (row 0 x row 1)
            const cx<double> c0 = cmadd(cmul(a.m[1], a.m[5]), cx<double>{-a.m[2].re, -a.m[2].im}, a.m[4]);
            const cx<double> c1 = cmadd(cmul(a.m[2], a.m[3]), cx<double>{-a.m[0].re, -a.m[0].im}, a.m[5]);
            const cx<double> c2 = cmadd(cmul(a.m[0], a.m[4]), cx<double>{-a.m[1].re, -a.m[1].im}, a.m[3]);
            const cx<double> det = cmadd(cmadd(cmul(a.m[6], c0), a.m[7], c1), a.m[8], c2);
            v = max_nan(v, fabs(det.re - 1.0));
            v = max_nan(v, fabs(det.im));
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) v = max_nan(v, __shfl_xor(v, off, 64));
    __shared__ double ws[kFlowBlock / 64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) ws[wave] = v;
    __syncthreads();
    if (threadIdx.x == 0) {
        double m = 0.0;
#pragma unroll
        for (int w = 0; w < kFlowBlock / 64; ++w) m = max_nan(m, ws[w]);
        partials[blockIdx.x] = m;
    }
}

mdwf_status check_geom(const mdwf_geometry* g) {
    if (!g) return fail(nullptr, MDWF_ERR_ARG, "null geometry");
    if (g->X < 2 || g->Y < 2 || g->Z < 2 || g->T < 2) return fail(nullptr, MDWF_ERR_ARG, "extents must be >= 2");
    return MDWF_OK;
}

// average plaquette of the device field U into *plaq (synchronous on st)
mdwf_status plaquette_dev(const FlowGeo& fg, const double2* U, double* part, double* hpart, long nsites, int nblk,
                          hipStream_t st, double* plaq) {
    hipLaunchKernelGGL(k_plaquette, dim3(nblk), dim3(kFlowBlock), 0, st, fg, U, part, nsites);
    mdwf_status s = hip_check(nullptr, hipGetLastError(), "plaquette kernel");
    if (s) return s;
    if ((s = hip_check(nullptr, hipMemcpyAsync(hpart, part, sizeof(double) * nblk, hipMemcpyDeviceToHost, st),
                       "plaquette D2H")))
        return s;
    if ((s = hip_check(nullptr, hipStreamSynchronize(st), "plaquette"))) return s;
    double tot = 0.0;
    for (int k = 0; k < nblk; ++k) tot += hpart[k];
    *plaq = tot / (3.0 * 6.0 * double(nsites));
    return MDWF_OK;
}

}  // namespace
}  // namespace mdwf

using namespace mdwf;

extern "C" {

mdwf_status mdwf_plaquette_dev(const mdwf_geometry* geom, const double* U_dev, void* stream, double* plaq) {
    mdwf_status s = check_geom(geom);
    if (s) return s;
    if (!U_dev || !plaq) return fail(nullptr, MDWF_ERR_ARG, "null argument");
    const FlowGeo fg{geom->X, geom->Y, geom->Z, geom->T};
    const long nsites = long(fg.X) * fg.Y * fg.Z * fg.T;
    const int nblk = int((nsites + kFlowBlock - 1) / kFlowBlock);
    double* part = nullptr;
    if ((s = hip_check(nullptr, hipMalloc(&part, sizeof(double) * nblk), "plaquette partials"))) return s;
    std::vector<double> hpart(nblk);
    s = plaquette_dev(fg, reinterpret_cast<const double2*>(U_dev), part, hpart.data(), nsites, nblk,
                      static_cast<hipStream_t>(stream), plaq);
    (void)hipFree(part);
    return s;
}

mdwf_status mdwf_wilson_flow_dev(const mdwf_geometry* geom, double* U_dev, double eps, int nsteps, void* stream,
                                 double* plaq) {
    mdwf_status s = check_geom(geom);
    if (s) return s;
    if (!U_dev) return fail(nullptr, MDWF_ERR_ARG, "null gauge field");
    if (!(eps > 0.0) || !std::isfinite(eps) || nsteps < 0)
        return fail(nullptr, MDWF_ERR_ARG, "need eps > 0 and nsteps >= 0");
    hipStream_t st = static_cast<hipStream_t>(stream);
    const FlowGeo fg{geom->X, geom->Y, geom->Z, geom->T};
    const long nsites = long(fg.X) * fg.Y * fg.Z * fg.T, nlinks = 4 * nsites;
    const size_t bytes = size_t(nlinks) * 9 * sizeof(double2);
    // the stages address an entry by a 32-bit byte offset; two such fields
    // are beyond the device's memory anyway
    if (nsites >= (1L << 28)) return fail(nullptr, MDWF_ERR_OOM, "flow buffer");
    const int nblk_p = int((nsites + kFlowBlock - 1) / kFlowBlock);
    double2 *W2 = nullptr, *E = nullptr;
    double* part = nullptr;
    if ((s = hip_check(nullptr, hipMalloc(&W2, bytes), "flow buffer"))) return s;
    if ((s = hip_check(nullptr, hipMalloc(&E, size_t(nlinks) * 4 * sizeof(double2)), "flow buffer"))) {
        (void)hipFree(W2);
        return s;
    }
    if ((s = hip_check(nullptr, hipMalloc(&part, sizeof(double) * nblk_p), "plaquette partials"))) {
        (void)hipFree(W2);
        (void)hipFree(E);
        return s;
    }
    std::vector<double> hpart(nblk_p);
    double2* W[2] = {reinterpret_cast<double2*>(U_dev), W2};
    {   // the links must be SU(3) (the stage rebuilds staple links' third rows)
        hipLaunchKernelGGL(k_su3_deviation, dim3(nblk_p), dim3(kFlowBlock), 0, st, W[0], part, nsites);
        s = hip_check(nullptr, hipGetLastError(), "SU(3) check kernel");
        if (!s) s = hip_check(nullptr, hipMemcpyAsync(hpart.data(), part, sizeof(double) * nblk_p,
                                                      hipMemcpyDeviceToHost, st), "SU(3) check D2H");
        if (!s) s = hip_check(nullptr, hipStreamSynchronize(st), "SU(3) check");
        double dev = 0.0;
        for (int k = 0; k < nblk_p && !s; ++k) dev = (hpart[k] > dev || hpart[k] != hpart[k]) ? hpart[k] : dev;
        if (!s && !(dev <= kSu3Tol)) {
            char msg[160];
            std::snprintf(msg, sizeof msg, "gauge links are not SU(3): deviation %.3e > %.0e", dev, kSu3Tol);
            s = fail(nullptr, MDWF_ERR_ARG, msg);
        }
    }
    if (!s && plaq) s = plaquette_dev(fg, W[0], part, hpart.data(), nsites, nblk_p, st, plaq);
    const double ca[3] = {0.25, 8.0 / 9.0, 0.75}, cb[3] = {0.0, -17.0 / 9.0, -1.0};
    // stages 0, 2, .. read W2 and write U_dev's memory, in the stage's layout;
    // the last one writes it in the canonical layout or, an even one, W2
    const uint32_t V = uint32_t(nsites);
    const unsigned grid = unsigned((nsites + kFlowSites - 1) / kFlowSites);
    FlowTrav tv;
    tv.bz = fg.Z / 8 > 1 ? fg.Z / 8 : 1;
    tv.xy = FastDiv(uint32_t(fg.X * fg.Y));
    tv.x = FastDiv(uint32_t(fg.X));
    tv.plane = FastDiv(uint32_t(fg.X * fg.Y * tv.bz));
    tv.slab = FastDiv(uint32_t(fg.X * fg.Y * tv.bz) * uint32_t(fg.T));
    tv.nsites = V;
    if (!s && nsteps) {
        hipLaunchKernelGGL(k_flow_layout<true>, dim3(grid), dim3(4 * kFlowSites), 0, st, W[0], W[1], V);
        s = hip_check(nullptr, hipGetLastError(), "flow layout kernel");
    }
    const long nstages = 3L * nsteps;
    for (long n = 0; n < nstages && !s; ++n) {
        const double2* in = W[1 - n % 2];
        double2* out = W[n % 2];
        const int i = int(n % 3);
        if (n == nstages - 1 && n % 2 == 0)
            hipLaunchKernelGGL(k_flow_stage<true>, dim3(grid), dim3(4 * kFlowSites), 0, st, fg, tv, in, out, E,
                               ca[i] * eps, cb[i]);
        else
            hipLaunchKernelGGL(k_flow_stage<false>, dim3(grid), dim3(4 * kFlowSites), 0, st, fg, tv, in, out, E,
                               ca[i] * eps, cb[i]);
        s = hip_check(nullptr, hipGetLastError(), "flow kernel");
    }
    if (!s && nstages && nstages % 2 == 0) {
        hipLaunchKernelGGL(k_flow_layout<false>, dim3(grid), dim3(4 * kFlowSites), 0, st, W[1], W[0], V);
        s = hip_check(nullptr, hipGetLastError(), "flow layout kernel");
    }
    if (!s && plaq) s = plaquette_dev(fg, W[0], part, hpart.data(), nsites, nblk_p, st, plaq + 1);
    if (!s) s = hip_check(nullptr, hipStreamSynchronize(st), "flow");
    (void)hipFree(W2);
    (void)hipFree(E);
    (void)hipFree(part);
    return s;
}

mdwf_status mdwf_wilson_flow(const mdwf_geometry* geom, int hip_device, double* U, double eps, int nsteps,
                             double* plaq) {
    mdwf_status s = check_geom(geom);
    if (s) return s;
    if (!U) return fail(nullptr, MDWF_ERR_ARG, "null gauge field");
    if ((s = hip_check(nullptr, hipSetDevice(hip_device), "hipSetDevice"))) return s;
    const size_t bytes = size_t(4) * geom->X * geom->Y * geom->Z * geom->T * 9 * sizeof(double2);
    double* d = nullptr;
    if ((s = hip_check(nullptr, hipMalloc(&d, bytes), "flow field"))) return s;
    s = hip_check(nullptr, hipMemcpy(d, U, bytes, hipMemcpyHostToDevice), "flow H2D");
    if (!s) s = mdwf_wilson_flow_dev(geom, d, eps, nsteps, nullptr, plaq);
    if (!s) s = hip_check(nullptr, hipMemcpy(U, d, bytes, hipMemcpyDeviceToHost), "flow D2H");
    (void)hipFree(d);
    return s;
}

}  // extern "C"

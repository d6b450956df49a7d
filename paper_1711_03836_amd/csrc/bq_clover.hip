// Clover term of Eq. 2 on the device: field strength from the four-leaf
// clover, the two Hermitian 6x6 blocks per site and their inverses.
//
// In the chiral basis sigma_{mu nu} is block diagonal; with the Hermitian
// field strengths G_{mu nu} = -i F_{mu nu} (mu,nu = 0..3 for x,y,z,t) the
// clover matrix T = 1 + kappa c_SW sum_{mu<nu} sigma_{mu nu} (x) G_{mu nu} is
//   block +/- = 1 + ck [ s3 (x) (G01 -/+ G23) + s2 (x) (G02 +/- G13) + s1 (x) (G12 -/+ G03) ]
// (s1,s2,s3 Pauli matrices acting on the two spins of the block), i.e.
//   [[ 1 + ck X3,  ck (X1 - i X2) ], [ ck (X1 + i X2),  1 - ck X3 ]].
// Blocks are inverted with a complex Cholesky factorisation, which also
// checks positive definiteness.
#include <algorithm>

#include "bq_kernels.h"

namespace bq {
namespace {

using c64 = cx<double>;

struct M3 {
    c64 m[9];
};

struct LinkTable {
    const double2* U[8];
};

// The points of a plane (mu, nu) around site s, mu and nu uniform over the wavefront: a link m steps in
// mu and n in nu (-1, 0, 1; periodic) away is at lexicographic index l0 + xm sm + xn sn, and on parity
// p + m + n (the extents are even), so its array is uniform as well.
struct Plane {
    int parity, Lm, Ln, sm, sn;  // uniform
    int l0, xm, xn;
    __device__ __forceinline__ Plane(const Geom& g, const Site& s, int par, int mu, int nu)
    {
        parity = par;
        Lm = g.L[mu];
        Ln = g.L[nu];
        sm = sn = 1;
#pragma unroll
        for (int k = 0; k < 3; k++) {
            sm *= k < mu ? g.L[k] : 1;
            sn *= k < nu ? g.L[k] : 1;
        }
        const int c[4] = {s.x, s.y, s.z, s.t};
        xm = xn = 0;
#pragma unroll
        for (int k = 0; k < 4; k++) {
            xm += k == mu ? c[k] : 0;
            xn += k == nu ? c[k] : 0;
        }
        l0 = s.x + g.L[0] * (s.y + g.L[1] * (s.z + g.L[2] * s.t)) - xm * sm - xn * sn;
    }
    __device__ __forceinline__ int index(int m, int n) const  // in its parity
    {
        int a = xm + m, b = xn + n;
        a = a < 0 ? a + Lm : (a >= Lm ? a - Lm : a);
        b = b < 0 ? b + Ln : (b >= Ln ? b - Ln : b);
        return (l0 + a * sm + b * sn) >> 1;
    }
    __device__ __forceinline__ M3 link(const LinkTable& t, int dir, int m, int n) const
    {
        const int j = index(m, n);
        const double2* u = t.U[((parity + m + n) & 1) * 4 + dir];
        M3 r;
#pragma unroll
        for (int k = 0; k < 9; k++) {
            const double2 v = at(u, j, k, 9);
            r.m[k] = {v.x, v.y};
        }
        return r;
    }
};

// Products are taken in place, row by row (a = a b, a = a b^dag), so that a chain of links needs the
// registers of one running product and one link.  hold() keeps the compiler from loading the links of
// the next products before this one is done (359 registers spilled without it).
__device__ __forceinline__ void hold(M3& a)
{
#pragma unroll
    for (int k = 0; k < 9; k++) asm volatile("" : "+v"(a.m[k].re), "+v"(a.m[k].im));
    asm volatile("" ::: "memory");
}
__device__ __forceinline__ void m3_mul_by(M3& a, const M3& b)
{
#pragma unroll
    for (int i = 0; i < 3; i++) {
        const c64 r0 = a.m[i * 3], r1 = a.m[i * 3 + 1], r2 = a.m[i * 3 + 2];
#pragma unroll
        for (int k = 0; k < 3; k++) {
            c64 s = cmul(r0, b.m[k]);
            s = cmac(s, r1, b.m[3 + k]);
            s = cmac(s, r2, b.m[6 + k]);
            a.m[i * 3 + k] = s;
        }
    }
    hold(a);
}
__device__ __forceinline__ void m3_mul_by_dag(M3& a, const M3& b)
{
#pragma unroll
    for (int i = 0; i < 3; i++) {
        const c64 r0 = a.m[i * 3], r1 = a.m[i * 3 + 1], r2 = a.m[i * 3 + 2];
#pragma unroll
        for (int k = 0; k < 3; k++) {
            c64 s = {0, 0};
            s = cmac(s, r0, c64{b.m[k * 3 + 0].re, -b.m[k * 3 + 0].im});
            s = cmac(s, r1, c64{b.m[k * 3 + 1].re, -b.m[k * 3 + 1].im});
            s = cmac(s, r2, c64{b.m[k * 3 + 2].re, -b.m[k * 3 + 2].im});
            a.m[i * 3 + k] = s;
        }
    }
    hold(a);
}
// a = a^dag b
__device__ __forceinline__ void m3_dag_mul_by(M3& a, const M3& b)
{
    M3 t;
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int k = 0; k < 3; k++) t.m[i * 3 + k] = a.m[k * 3 + i];
#pragma unroll
    for (int i = 0; i < 3; i++)
#pragma unroll
        for (int k = 0; k < 3; k++) {
            c64 s = {0, 0};
            s = cmacc(s, t.m[i * 3 + 0], b.m[0 * 3 + k]);
            s = cmacc(s, t.m[i * 3 + 1], b.m[1 * 3 + k]);
            s = cmacc(s, t.m[i * 3 + 2], b.m[2 * 3 + k]);
            a.m[i * 3 + k] = s;
        }
    hold(a);
}
__device__ __forceinline__ void m3_add(M3& a, const M3& b)
{
#pragma unroll
    for (int k = 0; k < 9; k++) a.m[k] = cadd(a.m[k], b.m[k]);
    hold(a);
}

// the planes mu < nu in order
__device__ __forceinline__ void plane_of(int p, int& mu, int& nu)
{
    mu = p < 3 ? 0 : (p < 5 ? 1 : 2);
    nu = p < 3 ? p + 1 : (p < 5 ? p - 1 : 3);
}

// A tile's links U_mu(x) and U_mu(x - mu) in LDS, [2 mu + (1 for x - mu)][entry][lane]
typedef double2 TileLinks[8][9][kTile];

__device__ __forceinline__ M3 lds_link(const double2 (&t)[9][kTile], int lane)
{
    M3 r;
#pragma unroll
    for (int k = 0; k < 9; k++) {
        const double2 v = t[k][lane];
        r.m[k] = {v.x, v.y};
    }
    return r;
}

// Hermitian traceless G = (Q - Q^dag)/(8i) of the four leaves in a plane: its three diagonal reals, then
// its lower triangle (1,0), (2,0), (2,1)
__device__ __forceinline__ void field_strength(const Plane& x, const LinkTable& U, const TileLinks& t, int lane, int mu,
                                               int nu, double (&out)[9])
{
    // leaf 1: U_mu(x) U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
    M3 Q = lds_link(t[2 * mu], lane);
    m3_mul_by(Q, x.link(U, nu, 1, 0));
    m3_mul_by_dag(Q, x.link(U, mu, 0, 1));
    m3_mul_by_dag(Q, lds_link(t[2 * nu], lane));
    // leaf 2: U_nu(x) U_mu(x+nu-mu)^dag U_nu(x-mu)^dag U_mu(x-mu)
    {
        M3 a = lds_link(t[2 * nu], lane);
        m3_mul_by_dag(a, x.link(U, mu, -1, 1));
        m3_mul_by_dag(a, x.link(U, nu, -1, 0));
        m3_mul_by(a, lds_link(t[2 * mu + 1], lane));
        m3_add(Q, a);
    }
    // leaf 3: U_mu(x-mu)^dag U_nu(x-mu-nu)^dag U_mu(x-mu-nu) U_nu(x-nu)
    {
        // U_mu(x-mu)^dag U_nu(x-mu-nu)^dag = (U_nu(x-mu-nu) U_mu(x-mu))^dag
        M3 a = x.link(U, nu, -1, -1);
        m3_mul_by(a, lds_link(t[2 * mu + 1], lane));
        M3 ad;
#pragma unroll
        for (int i = 0; i < 3; i++)
#pragma unroll
            for (int k = 0; k < 3; k++) ad.m[i * 3 + k] = {a.m[k * 3 + i].re, -a.m[k * 3 + i].im};
        m3_mul_by(ad, x.link(U, mu, -1, -1));
        m3_mul_by(ad, lds_link(t[2 * nu + 1], lane));
        m3_add(Q, ad);
    }
    // leaf 4: U_nu(x-nu)^dag U_mu(x-nu) U_nu(x-nu+mu) U_mu(x)^dag
    {
        M3 a = lds_link(t[2 * nu + 1], lane);
        m3_dag_mul_by(a, x.link(U, mu, 0, -1));
        m3_mul_by(a, x.link(U, nu, 1, -1));
        m3_mul_by_dag(a, lds_link(t[2 * mu], lane));
        m3_add(Q, a);
    }
    // G = (Q - Q^dag) / (8 i): G_ik = -i (Q_ik - conj(Q_ki)) / 8
    auto G = [&](int i, int k) {
        const c64 d = {Q.m[i * 3 + k].re - Q.m[k * 3 + i].re, Q.m[i * 3 + k].im + Q.m[k * 3 + i].im};
        return c64{d.im * 0.125, -d.re * 0.125};
    };
    const double g0 = G(0, 0).re, g1 = G(1, 1).re, g2 = G(2, 2).re;
    const double tr = (g0 + g1 + g2) / 3.0;
    out[0] = g0 - tr;
    out[1] = g1 - tr;
    out[2] = g2 - tr;
    const c64 l10 = G(1, 0), l20 = G(2, 0), l21 = G(2, 1);
    out[3] = l10.re;
    out[4] = l10.im;
    out[5] = l20.re;
    out[6] = l20.im;
    out[7] = l21.re;
    out[8] = l21.im;
}

// dense Hermitian 6x6 block helpers
struct H6 {
    c64 a[36];
};

// where one clover field (T or its inverse) goes in each storage precision; null: nowhere
struct CloverOut {
    double2* d;
    float2* f;
    uint2* h;
};

__device__ __forceinline__ void pack_store(const CloverOut& T, int j, int blk, const H6& A)
{
    c64 c[18];
    c[0] = {A.a[0].re, A.a[7].re};
    c[1] = {A.a[14].re, A.a[21].re};
    c[2] = {A.a[28].re, A.a[35].re};
#pragma unroll
    for (int i = 1; i < 6; i++)
#pragma unroll
        for (int k = 0; k < i; k++) c[3 + i * (i - 1) / 2 + k] = A.a[i * 6 + k];
    if (T.d)
#pragma unroll
        for (int k = 0; k < 18; k++) st_stream(&at(T.d, j, blk * 18 + k, 36), make_double2(c[k].re, c[k].im));
    if (T.f)
#pragma unroll
        for (int k = 0; k < 18; k += 2)  // units 2m and 2m + 1 of a site lie side by side
            *(float4*)&at(T.f, j, blk * 18 + k, 36) =
                make_float4((float)c[k].re, (float)c[k].im, (float)c[k + 1].re, (float)c[k + 1].im);
    if (T.h)
#pragma unroll
        for (int k = 0; k < 18; k += 2)
            at(T.h, j, blk * 9 + k / 2, 18) = CxIO<P16, 2>::pack(cx<float>{(float)c[k].re, (float)c[k].im},
                                                                 cx<float>{(float)c[k + 1].re, (float)c[k + 1].im});
}

__device__ __forceinline__ H6 pack_load(const double2* T, int j, int blk)
{
    H6 A;
    double2 d0 = at(T, j, blk * 18 + 0, 36), d1 = at(T, j, blk * 18 + 1, 36), d2 = at(T, j, blk * 18 + 2, 36);
    const double d[6] = {d0.x, d0.y, d1.x, d1.y, d2.x, d2.y};
#pragma unroll
    for (int i = 0; i < 6; i++) A.a[i * 6 + i] = {d[i], 0.0};
#pragma unroll
    for (int i = 1; i < 6; i++)
#pragma unroll
        for (int k = 0; k < i; k++) {
            double2 t = at(T, j, blk * 18 + 3 + i * (i - 1) / 2 + k, 36);
            A.a[i * 6 + k] = {t.x, t.y};
            A.a[k * 6 + i] = {t.x, -t.y};
        }
    return A;
}

// inverse of a Hermitian positive-definite 6x6 block by Cholesky A = L L^dag; returns false if not HPD
__device__ bool hpd_inverse(const H6& A, H6& Ai)
{
    c64 L[36];
#pragma unroll
    for (int k = 0; k < 36; k++) L[k] = {0, 0};
    bool ok = true;
#pragma unroll
    for (int j = 0; j < 6; j++) {
        double s = A.a[j * 6 + j].re;
#pragma unroll
        for (int k = 0; k < j; k++) s -= cnorm2(L[j * 6 + k]);
        ok = ok && (s > 0.0) && isfinite(s);
        const double ljj = sqrt(s > 0.0 ? s : 1.0);
        const double inv = 1.0 / ljj;
        L[j * 6 + j] = {ljj, 0.0};
#pragma unroll
        for (int i = j + 1; i < 6; i++) {
            c64 t = A.a[i * 6 + j];
#pragma unroll
            for (int k = 0; k < j; k++) {
                // t -= L[i][k] * conj(L[j][k])
                const c64 a = L[i * 6 + k], b = L[j * 6 + k];
                t.re -= a.re * b.re + a.im * b.im;
                t.im -= a.im * b.re - a.re * b.im;
            }
            L[i * 6 + j] = cscale(inv, t);
        }
    }
    // W = L^-1 (lower triangular)
    c64 W[36];
#pragma unroll
    for (int k = 0; k < 36; k++) W[k] = {0, 0};
#pragma unroll
    for (int i = 0; i < 6; i++) {
        const double inv = 1.0 / L[i * 6 + i].re;
        W[i * 6 + i] = {inv, 0.0};
#pragma unroll
        for (int j = 0; j < i; j++) {
            c64 s = {0, 0};
#pragma unroll
            for (int k = j; k < i; k++) s = cmac(s, L[i * 6 + k], W[k * 6 + j]);
            W[i * 6 + j] = cscale(-inv, s);
        }
    }
    // A^-1 = W^dag W
#pragma unroll
    for (int i = 0; i < 6; i++)
#pragma unroll
        for (int j = 0; j <= i; j++) {
            c64 s = {0, 0};
#pragma unroll
            for (int k = i; k < 6; k++) s = cmacc(s, W[k * 6 + i], W[k * 6 + j]);
            Ai.a[i * 6 + j] = s;
            Ai.a[j * 6 + i] = {s.re, -s.im};
        }
#pragma unroll
    for (int i = 0; i < 6; i++) Ai.a[i * 6 + i].im = 0.0;
    return ok;
}

// B (the clover blocks without identity and kappa c_SW) of one tile per workgroup, one wavefront per
// plane: its field strengths meet in LDS, then wavefront 3 * block + part assembles and stores six of
// the block's 18 packed units.  Bound by the fills of the L1: the leaves of six planes read 96 links
// per site, 48 of them the links U_mu(x) and U_mu(x - mu) that three planes each read twice; those
// come from LDS here (24^3x48, both parities: 808 us with one thread per site for all planes, 790 with
// one wavefront per plane, 545 with the eight links in LDS).
__global__ __launch_bounds__(6 * kTile) __attribute__((amdgpu_waves_per_eu(3, 8))) void k_clover_build(
    const Geom g, const LinkTable U, double2* __restrict__ B0, double2* __restrict__ B1)
{
    __shared__ TileLinks sl;
    double(*sg)[9][kTile] = (double(*)[9][kTile])sl;  // after the links: [plane][real of G][lane]
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> kTileLog), lane = threadIdx.x & (kTile - 1);
    const int lb = xcd_remap(blockIdx.x, gridDim.x);  // the two parities of a tile side by side
    const int parity = lb & 1;
    const int j = (lb >> 1) * kTile + lane;
    double2* __restrict__ B = parity ? B1 : B0;
    const bool in = j < g.Vh;
    const Site s = site_of(g, parity, in ? j : 0);
    for (int h = w; h < 8; h += 6) {
        const int mu = h >> 1, bw = h & 1;
        const double2* u = U.U[(parity ^ bw) * 4 + mu];
        const int jl = Plane(g, s, parity, mu, (mu + 1) & 3).index(-bw, 0);
#pragma unroll
        for (int k = 0; k < 9; k++) sl[h][k][lane] = at(u, jl, k, 9);
    }
    __syncthreads();
    {
        int mu, nu;
        plane_of(w, mu, nu);
        double G[9];
        field_strength(Plane(g, s, parity, mu, nu), U, sl, lane, mu, nu, G);
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 9; k++) sg[w][k][lane] = G[k];
    }
    __syncthreads();
    if (!in) return;
    // block 0: X3 = G01 - G23, X2 = G02 + G13, X1 = G12 - G03; block 1 with the other signs
    const int blk = w / 3, part = w % 3;
    const double sgn = blk == 0 ? -1.0 : +1.0;
    auto low = [&](int p, int a, int b) {  // G_p[a][b]
        if (a == b) return c64{sg[p][a][lane], 0.0};
        const int e = a > b ? (a == 1 ? 3 : (b == 0 ? 5 : 7)) : (b == 1 ? 3 : (a == 0 ? 5 : 7));
        const double re = sg[p][e][lane], im = sg[p][e + 1][lane];
        return c64{re, a > b ? im : -im};
    };
    auto X3 = [&](int a, int b) {
        const c64 u = low(0, a, b), v = low(5, a, b);
        return c64{u.re + sgn * v.re, u.im + sgn * v.im};
    };
    auto X21 = [&](int a, int b) {  // X1 + i X2
        const c64 u = low(1, a, b), v = low(4, a, b), p = low(3, a, b), q = low(2, a, b);
        const c64 x2 = {u.re - sgn * v.re, u.im - sgn * v.im}, x1 = {p.re + sgn * q.re, p.im + sgn * q.im};
        return c64{x1.re - x2.im, x1.im + x2.re};
    };
    auto put = [&](int unit, c64 v) { st_stream(&at(B, j, blk * 18 + unit, 36), make_double2(v.re, v.im)); };
    if (part == 0) {  // diagonal (x3, -x3) and the lower triangle of rows 1, 2
        const double d0 = X3(0, 0).re, d1 = X3(1, 1).re, d2 = X3(2, 2).re;
        put(0, {d0, d1});
        put(1, {d2, -d0});
        put(2, {-d1, -d2});
        put(3, X3(1, 0));
        put(4, X3(2, 0));
        put(5, X3(2, 1));
    } else if (part == 1) {  // rows 3, 4, columns 0..2
#pragma unroll
        for (int b = 0; b < 3; b++) put(3 + 3 + b, X21(0, b));
#pragma unroll
        for (int b = 0; b < 3; b++) put(3 + 6 + b, X21(1, b));
    } else {  // row 5, columns 0..2, and -X3 below the diagonal of rows 4, 5
#pragma unroll
        for (int b = 0; b < 3; b++) put(3 + 10 + b, X21(2, b));
        const c64 a = X3(1, 0), b = X3(2, 0), c = X3(2, 1);
        put(3 + 9, {-a.re, -a.im});
        put(3 + 13, {-b.re, -b.im});
        put(3 + 14, {-c.re, -c.im});
    }
}

// T = 1 + ck B and its inverse in every storage precision asked for, one thread per site and block.
// Bound by HBM: with the conversions as passes of their own over the FP64 results, 24^3x48 took 381
// us per parity for the three precisions, now 154 (860 MB, 5.6 TB/s).
__global__ __launch_bounds__(64) void k_clover_from_B(const Geom g, const double2* __restrict__ B, double ck, CloverOut T,
                                                      CloverOut Tinv, int* bad)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= g.Vh) return;
    const int blk = blockIdx.y;
    H6 A = pack_load(B, j, blk);
#pragma unroll
    for (int k = 0; k < 36; k++) A.a[k] = cscale(ck, A.a[k]);
#pragma unroll
    for (int i = 0; i < 6; i++) A.a[i * 6 + i].re += 1.0;
    pack_store(T, j, blk, A);
    if (Tinv.d || Tinv.f || Tinv.h) {
        H6 Ai;
        const bool ok = hpd_inverse(A, Ai);
        pack_store(Tinv, j, blk, Ai);
        if (!ok && bad) *bad = 1;
    }
}

struct CloverCols {
    const void* p[kMaxCols];
};

// y = (block of the clover) x, the block packed in 18 values
template <typename T>
__device__ __forceinline__ void block_mul(const cx<T> (&cb)[18], const cx<T>* v, cx<T>* y)
{
    const T d[6] = {cb[0].re, cb[0].im, cb[1].re, cb[1].im, cb[2].re, cb[2].im};
#pragma unroll
    for (int i = 0; i < 6; i++) y[i] = cscale(d[i], v[i]);
#pragma unroll
    for (int i = 1; i < 6; i++)
#pragma unroll
        for (int k = 0; k < i; k++) {
            const cx<T> A = cb[3 + i * (i - 1) / 2 + k];
            y[i] = cmac(y[i], A, v[k]);
            y[k] = cmacc(y[k], A, v[i]);
        }
}

// the packed values of block blk of site j
template <class P>
__device__ __forceinline__ void load_block(const typename P::unit* C, int j, int blk, cx<typename P::real> (&cb)[18])
{
    if constexpr (P::id == PREC_F16) {
#pragma unroll
        for (int u = 0; u < 9; u++) CxIO<P16, 2>::unpack(at(C, j, blk * 9 + u, 18), cb[2 * u], cb[2 * u + 1]);
    } else {
#pragma unroll
        for (int k = 0; k < 18; k++) {
            const auto t = at(C, j, blk * 18 + k, 36);
            cb[k] = {t.x, t.y};
        }
    }
}

// out = C in, one column of one tile per wavefront
template <class P>
__global__ __launch_bounds__(128) void k_clover_apply(const Geom g, const typename P::unit* C0, SpinorPtr<P> in,
                                                      SpinorPtr<P> out, int percol, const CloverCols cc, const int* status,
                                                      int statmask)
{
    using T = typename P::real;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (j >= g.Vh || (status && !col_selected(status, statmask, c))) return;
    const typename P::unit* C = percol ? (const typename P::unit*)cc.p[c] : C0;
    cx<T> v[12], y[12];
    load_spinor(in, c, j, v);
#pragma unroll
    for (int b = 0; b < 2; b++) {
        cx<T> cb[18];
        load_block<P>(C, j, b, cb);
        block_mul(cb, v + 6 * b, y + 6 * b);
    }
    store_spinor(out, c, j, y);
}

// The same for the columns c0 .. c0 + cols - 1.  A shared clover is read once for all of them and kept in
// registers: one of its two blocks per wavefront (blockIdx.z) in FP64 and FP32, both in FP16, whose
// spinors have one scale for the site.  Bound by HBM; read once per column the clover was most of the
// traffic: 24^3x48 x 12, both parities: FP64 1174 -> 678 us, FP32 555 -> 345, FP16 285 -> 197.
template <class P>
__global__ __launch_bounds__(128) void k_clover_apply_cols(const Geom g, const typename P::unit* C0, SpinorPtr<P> in,
                                                           SpinorPtr<P> out, int ncol, int cols, int percol,
                                                           const CloverCols cc, const int* status, int statmask)
{
    using T = typename P::real;
    constexpr int NB = P::id == PREC_F16 ? 2 : 1;  // blocks per wavefront
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= g.Vh) return;
    const int c0 = blockIdx.y * cols, c1 = min(ncol, c0 + cols);
    const int b0 = NB == 2 ? 0 : blockIdx.z;
    cx<T> cb[NB][18];
    const auto load_clover = [&](const typename P::unit* C) {
#pragma unroll
        for (int b = 0; b < NB; b++) load_block<P>(C, j, b0 + b, cb[b]);
    };
    if (!percol) load_clover(C0);
    for (int c = c0; c < c1; c++) {
        if (status && !col_selected(status, statmask, c)) continue;
        if (percol) load_clover((const typename P::unit*)cc.p[c]);
        if constexpr (NB == 2) {
            cx<T> v[12], y[12];
            load_spinor(in, c, j, v);
#pragma unroll
            for (int b = 0; b < 2; b++) block_mul(cb[b], v + 6 * b, y + 6 * b);
            store_spinor(out, c, j, y);
        } else {
            const typename P::unit* ib = in.d + c * in.cstride;
            typename P::unit* ob = out.d + c * out.cstride;
            cx<T> v[6], y[6];
#pragma unroll
            for (int k = 0; k < 6; k++) {
                auto t = at(ib, j, b0 * 6 + k, 12);
                v[k] = {t.x, t.y};
            }
            block_mul(cb[0], v, y);
#pragma unroll
            for (int k = 0; k < 6; k++) at(ob, j, b0 * 6 + k, 12) = {y[k].re, y[k].im};
        }
    }
}

// sum over the 6 planes of Re tr U_{mu nu}(x) / 3, one FP64 partial per tile; one wavefront per plane, the
// planes of a site summed in order.  The tile's own four links are read once, into LDS (24^3x48: 227 ->
// 126 us).
__global__ __launch_bounds__(6 * kTile) void k_plaquette(const Geom g, const LinkTable U, double* partial, int nwaves)
{
    __shared__ double2 own[4][9][kTile];
    __shared__ double sp[6][kTile];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> kTileLog), lane = threadIdx.x & (kTile - 1);
    const int lb = xcd_remap(blockIdx.x, gridDim.x);  // the two parities of a tile side by side
    const int parity = lb & 1, tile = lb >> 1;
    const int j = tile * kTile + lane;
    const bool in = j < g.Vh;
    if (w < 4) {
        const double2* u = U.U[parity * 4 + w];
#pragma unroll
        for (int k = 0; k < 9; k++) own[w][k][lane] = at(u, in ? j : 0, k, 9);
    }
    __syncthreads();
    {
        const Site s = site_of(g, parity, in ? j : 0);
        int mu, nu;
        plane_of(w, mu, nu);
        const Plane x(g, s, parity, mu, nu);
        M3 a = lds_link(own[mu], lane);
        m3_mul_by(a, x.link(U, nu, 1, 0));
        m3_mul_by_dag(a, x.link(U, mu, 0, 1));
        m3_mul_by_dag(a, lds_link(own[nu], lane));
        sp[w][lane] = (a.m[0].re + a.m[4].re + a.m[8].re) / 3.0;
    }
    __syncthreads();
    if (w != 0) return;
    double acc = 0.0;
    if (in)
#pragma unroll
        for (int p = 0; p < 6; p++) acc += sp[p][lane];
    acc = wave_sum(acc);
    if (lane == 0 && tile < nwaves) partial[parity * nwaves + tile] = acc;
}

}  // namespace

hipError_t launch_plaquette(const Geom& g, const double2* const U64[8], double* partial, int nparts, hipStream_t st)
{
    // partial: 2 * (padded Vh / 64) entries, parity 0 first
    LinkTable t;
    for (int k = 0; k < 8; k++) t.U[k] = U64[k];
    const int nw = pad_sites(g.Vh) / kTile;
    if (nparts < 2 * nw) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_plaquette, dim3(2 * nw), dim3(6 * kTile), 0, st, g, t, partial, nw);
    return hipGetLastError();
}

hipError_t launch_clover_build(const Geom& g, const double2* const U64[8], double2* const B[2], hipStream_t st)
{
    LinkTable t;
    for (int k = 0; k < 8; k++) t.U[k] = U64[k];
    hipLaunchKernelGGL(k_clover_build, dim3(2 * g.ntiles), dim3(6 * kTile), 0, st, g, t, B[0], B[1]);
    return hipGetLastError();
}

hipError_t launch_clover_from_B(const Geom& g, const double2* B, double ck, void* const T[3], void* const Tinv[3],
                                int* bad, hipStream_t st)
{
    const CloverOut t = {(double2*)T[PREC_F64], (float2*)T[PREC_F32], (uint2*)T[PREC_F16]};
    const CloverOut ti = {(double2*)Tinv[PREC_F64], (float2*)Tinv[PREC_F32], (uint2*)Tinv[PREC_F16]};
    hipLaunchKernelGGL(k_clover_from_B, dim3(g.ntiles, 2), dim3(kTile), 0, st, g, B, ck, t, ti, bad);
    return hipGetLastError();
}

hipError_t launch_clover_apply(int prec, const Geom& g, const void* clov, FieldArg in, FieldArg out, int ncol,
                               hipStream_t st, const void* const* cclov, const int* status, int statmask)
{
    const int bs = 128, nz = prec == PREC_F16 ? 1 : 2;
    CloverCols cc{};
    const int percol = cclov != nullptr;
    if (percol) {
        if (ncol > kMaxCols) return hipErrorInvalidValue;
        for (int c = 0; c < ncol; c++) cc.p[c] = cclov[c];
    }
    // columns per wavefront: all that share the clover, but at least 4096 wavefronts where there are as
    // many (four per SIMD)
    const int tiles = pad_sites(g.Vh) / kTile;
    const int groups = percol ? ncol : std::max(1, std::min(ncol, 4096 / (tiles * nz)));
    const int cols = (ncol + groups - 1) / groups;
    // One column and both blocks per wavefront instead: FP16 with nothing to share, or whose clover the L2s
    // hold (16^3x32 x 6 20.2 us against 22.7, x 10 27.9 and 30; 20^3x40 x 4 47 and 34); FP32 on a few tiles
    // (6x10x14x18 x 12 10.5 against 11.3; 16^4 x 6 17.9 and 16.6); one column in long streams (32^3x64 FP64
    // 382 against 399; 20^3x40 58 and 49)
    const bool single = prec == PREC_F16 ? percol || ncol == 1 || tiles < 2048
                                         : (ncol == 1 && tiles >= 8192) || (prec == PREC_F32 && tiles < 256);
    const int blocks = (g.Vh + bs - 1) / bs;
#define CA(P, U)                                                                                                     \
    {                                                                                                                \
        const SpinorPtr<P> i{(U*)in.d, in.s, in.cstride, in.sstride}, o{(U*)out.d, out.s, out.cstride, out.sstride}; \
        if (single)                                                                                                  \
            hipLaunchKernelGGL(k_clover_apply<P>, dim3(blocks, ncol), dim3(bs), 0, st, g, (const U*)clov, i, o, percol, cc, \
                               status, statmask);                                                                    \
        else                                                                                                         \
            hipLaunchKernelGGL(k_clover_apply_cols<P>, dim3(blocks, (ncol + cols - 1) / cols, nz), dim3(bs), 0, st, g, \
                               (const U*)clov, i, o, ncol, cols, percol, cc, status, statmask);                      \
    }
    switch (prec) {
    case PREC_F64: CA(P64, double2) break;
    case PREC_F32: CA(P32, float2) break;
    case PREC_F16: CA(P16, uint2) break;
    default: return hipErrorInvalidValue;
    }
#undef CA
    return hipGetLastError();
}

}  // namespace bq

// Layout conversion, BLAS-1 updates, deterministic FP64 reductions and the
// per-column CG finalisation kernels.
//
// Reductions: every kernel that reduces writes one FP64 partial per wavefront
// of 64 consecutive sites (a butterfly inside the wave), and a finalisation
// kernel sums a column's partials in a fixed order in one workgroup.  The
// partials depend only on which 64 sites a wave covers, so a column's result
// is the same bit for bit whatever the block size, column tile or batch it
// was computed in.
#include <type_traits>

#include "bq_kernels.h"

namespace bq {
namespace {

template <class P>
__host__ __device__ SpinorPtr<P> sp(const FieldArg& f)
{
    return SpinorPtr<P>{(typename P::unit*)f.d, f.s, f.cstride, f.sstride};
}

__device__ __forceinline__ int lex_of(const Geom& g, int parity, int j)
{
    const Site s = site_of(g, parity, j);
    return s.x + g.L[0] * (s.y + g.L[1] * (s.z + g.L[2] * s.t));
}

// --------------------------------------------------------------------------
// layout conversion between the canonical lexicographic complex128 arrays and
// the site-tiled checkerboard storage
// --------------------------------------------------------------------------

// The link arrays [parity * 4 + mu] of one storage form.
template <class U>
struct LinkOut {
    U* p[8];
};

// units 2m and 2m + 1 of a site lie side by side in 8-byte units: N of them, a last odd one alone
template <int N>
__device__ __forceinline__ void store_pairs(float2* b, int j, const float2 (&v)[N])
{
#pragma unroll
    for (int c = 0; c + 1 < N; c += 2) *(float4*)&at(b, j, c, N) = make_float4(v[c].x, v[c].y, v[c + 1].x, v[c + 1].y);
    if constexpr (N & 1) at(b, j, N - 1, N) = v[N - 1];
}

// Canonical links into the 18-real forms, with the largest distance from SU(3): per link max over
// max_ab |(U U^dag - 1)_ab| and |det U - 1|, infinite if an entry is not finite, one partial maximum per
// workgroup (k_fin_max takes their maximum).  One wavefront per tile, parity and direction, turned around in LDS as
// k_spinor_turn does (a link's 9 values are an odd number of 16-byte words already).  Bound by HBM:
// reading the canonical links once for the check and once for each of five forms and two parities took
// 1122 us at 24^3x48, now 161 (955 MB, 5.9 TB/s) and 122 in k_links_rows.
__global__ __launch_bounds__(4 * kTile) void k_links_take(const double2* __restrict__ canon, const Geom g, LinkOut<double2> d,
                                                          LinkOut<float2> f, double* partial)
{
    __shared__ double2 turn[4][kTile * 9];
    __shared__ double wm[4];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> kTileLog), lane = threadIdx.x & (kTile - 1);
    const int tile = blockIdx.x * 2 + (w >> 1), par = w & 1, mu = blockIdx.y;
    double2* t = turn[w];
    const int j = tile * kTile + lane;
    const bool in = j < g.Vh;
    const Site s = site_of(g, par, in ? j : 0);
    const unsigned long long odd = __ballot(s.x & 1);
    const int nu = 9 * min(kTile, g.Vh - tile * kTile);
    const double2* can = canon + (size_t)mu * 2 * g.Vh * 9;
    const size_t site0 = 2 * (size_t)tile * kTile;
#pragma unroll
    for (int i = 0; i < 9; i++) {
        const int u = i * kTile + lane;
        if (u < nu) {
            const int l = u / 9;
            t[u] = ld_stream(can + (site0 + 2 * l + ((odd >> l) & 1)) * 9 + (u - 9 * l));
        }
    }
    __syncthreads();
    double dev = 0.0;
    if (in) {
        cx<double> u[9];
#pragma unroll
        for (int e = 0; e < 9; e++) {
            const double2 x = t[lane * 9 + e];
            u[e] = {x.x, x.y};
        }
        double mag = 0.0;  // not finite if an entry is not (fmax below would drop a NaN)
#pragma unroll
        for (int e = 0; e < 9; e++) mag += fabs(u[e].re) + fabs(u[e].im);
        double2* db = d.p[par * 4 + mu];  // uniform over the wavefront
        float2* fb = f.p[par * 4 + mu];
        float2 v[9];
#pragma unroll
        for (int e = 0; e < 9; e++) {
            at(db, j, e, 9) = make_double2(u[e].re, u[e].im);
            v[e] = make_float2((float)u[e].re, (float)u[e].im);
        }
        store_pairs<9>(fb, j, v);
#pragma unroll
        for (int a = 0; a < 3; a++)
#pragma unroll
            for (int b = 0; b < 3; b++) {
                cx<double> q = {0.0, 0.0};
#pragma unroll
                for (int c = 0; c < 3; c++) q = cmacc(q, u[b * 3 + c], u[a * 3 + c]);  // sum_c U_ac conj(U_bc)
                if (a == b) q.re -= 1.0;
                dev = fmax(dev, fmax(fabs(q.re), fabs(q.im)));
            }
        const cx<double> m0 = csub(cmul(u[4], u[8]), cmul(u[5], u[7]));
        const cx<double> m1 = csub(cmul(u[5], u[6]), cmul(u[3], u[8]));
        const cx<double> m2 = csub(cmul(u[3], u[7]), cmul(u[4], u[6]));
        cx<double> det = cmul(u[0], m0);
        det = cmac(det, u[1], m1);
        det = cmac(det, u[2], m2);
        det.re -= 1.0;
        dev = fmax(dev, sqrt(cnorm2(det)));
        if (!isfinite(mag) || !isfinite(dev)) dev = INFINITY;
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) dev = fmax(dev, __shfl_xor(dev, off, 64));
    if (lane == 0) wm[w] = dev;
    __syncthreads();
    if (threadIdx.x == 0) partial[blockIdx.y * gridDim.x + blockIdx.x] = fmax(fmax(wm[0], wm[1]), fmax(wm[2], wm[3]));
}

// The two-row forms of the precisions that keep one, from the FP64 18-real form in one pass.
__global__ __launch_bounds__(256) void k_links_rows(LinkOut<double2> src, int Vh, LinkOut<double2> d, LinkOut<float2> f,
                                                    LinkOut<uint2> h)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= Vh) return;
    const double2* sb = src.p[blockIdx.y];
    double2* db = d.p[blockIdx.y];
    float2* fb = f.p[blockIdx.y];
    uint2* hb = h.p[blockIdx.y];
    double2 u[6];
    float2 v[6];
#pragma unroll
    for (int e = 0; e < 6; e++) {
        u[e] = ld_stream(&at(sb, j, e, 9));
        v[e] = make_float2((float)u[e].x, (float)u[e].y);
    }
    if (db)
#pragma unroll
        for (int e = 0; e < 6; e++) at(db, j, e, 6) = u[e];
    if (fb) store_pairs<6>(fb, j, v);
    if (hb)
#pragma unroll
        for (int e = 0; e < 3; e++)
            at(hb, j, e, 3) = CxIO<P16, 2>::pack(cx<float>{v[2 * e].x, v[2 * e].y}, cx<float>{v[2 * e + 1].x, v[2 * e + 1].y});
}

// Spinors between the canonical array and the tiles: one wavefront per tile, parity and column.
// The 64 sites j of a tile are the canonical sites 2j + (0 or 1), of 12 consecutive 16-byte values
// each.  A lane that read or wrote its own site would touch 64 lines with every access, one per
// lane; so the canonical side is walked in its own order, value u = 12 site + component by lane u mod
// 64 (192-byte runs), and the wavefront turns the tile around in LDS, in rows of 13 values to keep
// the lanes' rows in different banks.  Both parities of a tile run in one workgroup and share the
// lines that their sites halve.  Both sides stream (non-temporal), except that FP32 and FP16 leave
// the lines of both parities to meet in the L2 on the way out (32^3x64 x 12 FP16: 1346 -> 1190 us).
// Bound by HBM: 24^3x48 x 12 columns in FP64, 3.06 GB, import 713 -> 583 us, export 793 -> 554 us
// (5.5 TB/s; a plain copy reaches 6.6); 32^3x64 x 12 in FP32, odd sites only, export 1180 -> 750 us.
constexpr int kTurnRow = 13;  // values per site in LDS

// canonical value index (site * 12 + component) of value u of the wavefront's tile; odd: bit l set
// if lane l's site is the odd one of its pair
__device__ __forceinline__ size_t canon_of(size_t site0, int u, unsigned long long odd)
{
    const int l = u / 12;
    return (site0 + 2 * l + ((odd >> l) & 1)) * 12 + (u - 12 * l);
}

typedef double bq_d2 __attribute__((ext_vector_type(2)));

// NP parities per workgroup (p0 .. p0 + NP - 1), f: the first one's field, hs / hss: units / scales between them
template <class P, int NP, bool IMPORT>
__global__ __launch_bounds__(kTile * 4) void k_spinor_turn(double2* __restrict__ canon, const Geom g, int p0, SpinorPtr<P> f,
                                                           size_t hs, size_t hss)
{
    using T = typename P::real;
    using C = typename std::conditional<sizeof(T) == 8, double2, float2>::type;
    __shared__ C turn[4][kTile * kTurnRow];
    const int w = threadIdx.x >> kTileLog, lane = threadIdx.x & (kTile - 1);
    const int tile = blockIdx.x * (4 / NP) + w / NP;
    const int c = blockIdx.y;
    const int par = p0 + w % NP;
    C* t = turn[w];
    const int j = tile * kTile + lane;
    const bool in = j < g.Vh;
    const Site s = site_of(g, par, in ? j : 0);
    const unsigned long long odd = __ballot(s.x & 1);
    const int nu = 12 * min(kTile, g.Vh - tile * kTile);  // values of the tile (its last sites may be padding)
    double2* can = canon + (size_t)c * 2 * g.Vh * 12;
    const size_t site0 = 2 * (size_t)tile * kTile;
    f.d += (w % NP) * hs;
    if constexpr (P::id == PREC_F16) f.s += (w % NP) * hss;
    cx<T> v[12];
    if constexpr (IMPORT) {
        // all twelve loads are on their way before the first is used (a part-filled tile reads its last
        // value again: a test around each load would have made them wait for one another)
        bq_d2 x[12];
        if (nu > 0)
#pragma unroll
            for (int i = 0; i < 12; i++)
                x[i] = __builtin_nontemporal_load((const bq_d2*)can + canon_of(site0, min(i * kTile + lane, nu - 1), odd));
#pragma unroll
        for (int i = 0; i < 12; i++) {
            const int u = i * kTile + lane;
            if (u < nu) t[u + u / 12 * (kTurnRow - 12)] = C{(T)x[i].x, (T)x[i].y};
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const C x = t[lane * kTurnRow + k];
            v[k] = {x.x, x.y};
        }
        if (in) store_spinor<P, true>(f, c, j, v);
    } else {
        if (in) {
            if constexpr (P::id == PREC_F64) CxIO<P, 12>::load_stream(f.d + c * f.cstride, j, v);
            else load_spinor(f, c, j, v);
#pragma unroll
            for (int k = 0; k < 12; k++) t[lane * kTurnRow + k] = C{v[k].re, v[k].im};
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < 12; i++) {
            const int u = i * kTile + lane;
            if (u < nu) {
                const C x = t[u + u / 12 * (kTurnRow - 12)];
                const bq_d2 y = {(double)x.x, (double)x.y};
                bq_d2* to = (bq_d2*)can + canon_of(site0, u, odd);
                if constexpr (NP == 1 || P::id == PREC_F64) __builtin_nontemporal_store(y, to);
                else *to = y;
            }
        }
    }
}

// --------------------------------------------------------------------------
// BLAS-1 over n sites (a parity half, or both halves of a full field)
// --------------------------------------------------------------------------

template <class PS, class PD>
__global__ void k_convert(SpinorPtr<PS> src, SpinorPtr<PD> dst, int n, const int* status, int statmask)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (j >= n || !col_selected(status, statmask, c)) return;
    cx<typename PS::real> a[12];
    cx<typename PD::real> b[12];
    load_spinor(src, c, j, a);
#pragma unroll
    for (int k = 0; k < 12; k++) b[k] = {(typename PD::real)a[k].re, (typename PD::real)a[k].im};
    store_spinor(dst, c, j, b);
}

template <class P>
__global__ void k_zero(SpinorPtr<P> x, int n, const int* status, int statmask)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (j >= n || !col_selected(status, statmask, c)) return;
    cx<typename P::real> z[12];
#pragma unroll
    for (int k = 0; k < 12; k++) z[k] = {0, 0};
    store_spinor(x, c, j, z);
}

template <class P>
__global__ void k_norm2(SpinorPtr<P> x, int n, double* partial, int nwaves)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    double s = 0.0;
    if (j < n) {
        cx<typename P::real> v[12];
        load_spinor(x, c, j, v);
#pragma unroll
        for (int k = 0; k < 12; k++) s += (double)v[k].re * v[k].re + (double)v[k].im * v[k].im;
    }
    s = wave_sum(s);
    const int w = j >> kTileLog;
    if ((threadIdx.x & 63) == 0 && w < nwaves) partial[(size_t)c * nwaves + w] = s;
}

// <x, y> = sum conj(x) y (G5: <x, gamma_5 y>, gamma_5 = diag(1,1,-1,-1) in spin), FP64 fields;
// partials [col][re/im][wave]
template <bool G5>
__global__ void k_dot(SpinorPtr<P64> x, SpinorPtr<P64> y, int n, double* partial, int nwaves)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    double re = 0.0, im = 0.0;
    if (j < n) {
        cx<double> a[12], b[12];
        load_spinor(x, c, j, a);
        load_spinor(y, c, j, b);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            const double sg = (G5 && k >= 6) ? -1.0 : 1.0;  // components 6..11 are spins 2 and 3
            re += sg * (a[k].re * b[k].re + a[k].im * b[k].im);
            im += sg * (a[k].re * b[k].im - a[k].im * b[k].re);
        }
    }
    re = wave_sum(re);
    im = wave_sum(im);
    const int w = j >> kTileLog;
    if ((threadIdx.x & 63) == 0 && w < nwaves) {
        partial[((size_t)c * 2 + 0) * nwaves + w] = re;
        partial[((size_t)c * 2 + 1) * nwaves + w] = im;
    }
}

// x += alpha p (active and just-stopped columns); p = r + beta p (active columns)
template <class PX, class PP, class PR>
__global__ void k_cg_update(SpinorPtr<PX> x, SpinorPtr<PP> p, SpinorPtr<PR> r, int n, const double* alpha,
                            const double* beta, const int* status)
{
    using TX = typename PX::real;
    using TP = typename PP::real;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    const int st = status ? status[c] : COL_ACTIVE;
    if (j >= n || (st != COL_ACTIVE && st != COL_JUST_STOPPED)) return;
    cx<TP> pv[12];
    load_spinor(p, c, j, pv);
    {
        const TX a = (TX)alpha[c];
        cx<TX> xv[12];
        load_spinor(x, c, j, xv);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            xv[k].re = fmadd(a, (TX)pv[k].re, xv[k].re);
            xv[k].im = fmadd(a, (TX)pv[k].im, xv[k].im);
        }
        store_spinor(x, c, j, xv);
    }
    if (st == COL_ACTIVE) {
        const TP b = (TP)beta[c];
        cx<typename PR::real> rv[12];
        load_spinor(r, c, j, rv);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            pv[k].re = fmadd(b, pv[k].re, (TP)rv[k].re);
            pv[k].im = fmadd(b, pv[k].im, (TP)rv[k].im);
        }
        store_spinor(p, c, j, pv);
    }
}

// y64 += x ; x = 0
template <class PX>
__global__ void k_accum(SpinorPtr<PX> x, SpinorPtr<P64> y, int n, const int* status, int statmask)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (j >= n || !col_selected(status, statmask, c)) return;
    cx<typename PX::real> xv[12];
    cx<double> yv[12];
    load_spinor(x, c, j, xv);
    load_spinor(y, c, j, yv);
#pragma unroll
    for (int k = 0; k < 12; k++) {
        yv[k].re += (double)xv[k].re;
        yv[k].im += (double)xv[k].im;
        xv[k] = {0, 0};
    }
    store_spinor(y, c, j, yv);
    store_spinor(x, c, j, xv);
}

// rs = lowp(r64) ; p = rs + beta p   (columns with flag set)
template <class PRS, class PP>
__global__ void k_restart(SpinorPtr<P64> r64, SpinorPtr<PRS> rs, SpinorPtr<PP> p, int n, const double* beta,
                          const int* flag, int write_rs)
{
    using TP = typename PP::real;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (j >= n || !flag[c]) return;
    cx<double> rv[12];
    load_spinor(r64, c, j, rv);
    if (write_rs) {
        cx<typename PRS::real> t[12];
#pragma unroll
        for (int k = 0; k < 12; k++) t[k] = {(typename PRS::real)rv[k].re, (typename PRS::real)rv[k].im};
        store_spinor(rs, c, j, t);
#pragma unroll
        for (int k = 0; k < 12; k++) rv[k] = {(double)t[k].re, (double)t[k].im};
    }
    const TP b = (TP)beta[c];
    cx<TP> pv[12];
    load_spinor(p, c, j, pv);
#pragma unroll
    for (int k = 0; k < 12; k++) {
        pv[k].re = fmadd(b, pv[k].re, (TP)rv[k].re);
        pv[k].im = fmadd(b, pv[k].im, (TP)rv[k].im);
    }
    store_spinor(p, c, j, pv);
}

// complex Z2 noise from SplitMix64 used as a counter-based generator:
// output k of stream `seed` is mix(seed + (k+1) * 0x9E3779B97F4A7C15);
// component (noise n, lexicographic site i, spin s, colour c) uses k = (n*V + i)*12 + 3s + c,
// bit 63 -> sign of the real part, bit 62 -> sign of the imaginary part, |eta| = 1.
__device__ __forceinline__ uint64_t mix64(uint64_t z)
{
    z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
    z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
    return z ^ (z >> 31);
}

__global__ void k_z2_noise(uint64_t seed, long n0, const Geom g, int parity, SpinorPtr<P64> f)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (j >= g.Vh) return;
    const uint64_t V = 2 * (uint64_t)g.Vh;
    const uint64_t lex = (uint64_t)lex_of(g, parity, j);
    const double h = 0.70710678118654752440;
    cx<double> v[12];
#pragma unroll
    for (int k = 0; k < 12; k++) {
        const uint64_t ctr = ((uint64_t)(n0 + c) * V + lex) * 12 + k;
        const uint64_t z = mix64(seed + (ctr + 1) * 0x9E3779B97F4A7C15ull);
        v[k] = {(z >> 63) & 1 ? -h : h, (z >> 62) & 1 ? -h : h};
    }
    store_spinor(f, c, j, v);
}

// --------------------------------------------------------------------------
// per-column finalisation (one workgroup of 256 threads per column)
// --------------------------------------------------------------------------

__device__ double block_sum(const double* __restrict__ part, int n)
{
    // eight independent partial sums per thread keep eight loads in flight; which element goes
    // to which sum depends on n only, so the result is deterministic for a given lattice
    __shared__ double w[4];
    double a[8] = {0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0, 0.0};
    int i = threadIdx.x;
    for (; i + 7 * 256 < n; i += 8 * 256) {
#pragma unroll
        for (int k = 0; k < 8; k++) a[k] += part[i + k * 256];
    }
    for (; i < n; i += 256) a[0] += part[i];
    double s = ((a[0] + a[1]) + (a[2] + a[3])) + ((a[4] + a[5]) + (a[6] + a[7]));
    s = wave_sum(s);
    __syncthreads();  // a previous call's readers of w are done before it is overwritten
    if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = s;
    __syncthreads();
    return (w[0] + w[1]) + (w[2] + w[3]);
}

__global__ void k_fin_sum(const double* partial, int nwaves, double* out)
{
    const int c = blockIdx.x;
    const double s = block_sum(partial + (size_t)c * nwaves, nwaves);
    if (threadIdx.x == 0) out[c] = s;
}

// out[0] = the largest of n partial maxima
__global__ __launch_bounds__(256) void k_fin_max(const double* partial, int n, double* out)
{
    __shared__ double w[4];
    double m = 0.0;
    for (int i = threadIdx.x; i < n; i += 256) m = fmax(m, partial[i]);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m = fmax(m, __shfl_xor(m, off, 64));
    if ((threadIdx.x & 63) == 0) w[threadIdx.x >> 6] = m;
    __syncthreads();
    if (threadIdx.x == 0) out[0] = fmax(fmax(w[0], w[1]), fmax(w[2], w[3]));
}

__global__ void k_fin_alpha(const CgScalars s, const double* partial, int nwaves)
{
    const int c = blockIdx.x;
    const int st = s.status[c];
    if (st != COL_ACTIVE && st != COL_JUST_STOPPED) return;  // uniform per block
    const double pAp = st == COL_ACTIVE ? block_sum(partial + (size_t)c * nwaves, nwaves) : 0.0;
    if (threadIdx.x != 0) return;
    if (st == COL_JUST_STOPPED) {
        s.status[c] = COL_STOPPED;
        return;
    }
    s.pAp[c] = pAp;
    if (!(pAp > 0.0) || !isfinite(pAp)) {
        s.alpha[c] = 0.0;
        s.status[c] = COL_FAILED;
    } else {
        s.alpha[c] = s.rho[c] / pAp;
    }
}

__global__ void k_fin_beta(const CgScalars s, const double* partial, int nwaves)
{
    const int c = blockIdx.x;
    if (s.status[c] != COL_ACTIVE) return;
    const double rho = block_sum(partial + (size_t)c * nwaves, nwaves);
    if (threadIdx.x != 0) return;
    s.iters[c] += 1;
    if (!isfinite(rho)) {
        s.status[c] = COL_FAILED;
    } else if (rho <= s.stop2[c] || (s.delta2 > 0.0 && rho <= s.delta2 * s.rmax2[c])) {
        s.status[c] = COL_JUST_STOPPED;  // x still takes this iteration's alpha*p
    } else {
        s.beta[c] = rho / s.rho[c];
        s.rho[c] = rho;
        if (rho > s.rmax2[c]) s.rmax2[c] = rho;
    }
}

// k_fin_beta and k_cg_update in one: every workgroup takes its column's |r|^2 and decides for itself; the
// first one writes the states after the iteration to `next`, since the others still read `cur`.  On
// small lattices a launch of its own for one sum costs as much as a stencil: 8^4, FP32, 2.3 us and a
// gap of about one, of 30 per iteration.
template <class PX, class PP, class PR>
__global__ __launch_bounds__(256) void k_cg_update_beta(SpinorPtr<PX> x, SpinorPtr<PP> p, SpinorPtr<PR> r, int n,
                                                        const CgScalars cur, const CgScalars next, const double* partial,
                                                        int nwaves)
{
    using TX = typename PX::real;
    using TP = typename PP::real;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    const bool first = blockIdx.x == 0 && threadIdx.x == 0;
    const int st = cur.status[c];
    double rho = cur.rho[c], rmax2 = cur.rmax2[c];
    const double pAp = cur.pAp[c];
    const bool broken = st == COL_ACTIVE && (!(pAp > 0.0) || !isfinite(pAp));
    if (st != COL_ACTIVE || broken) {  // uniform over the workgroup
        if (first) {
            // (a column that stopped in the last iteration has taken its last update of x)
            next.status[c] = broken ? COL_FAILED : (st == COL_JUST_STOPPED ? COL_STOPPED : st);
            next.iters[c] = cur.iters[c];
            next.rho[c] = rho;
            next.rmax2[c] = rmax2;
        }
        return;
    }
    cx<TP> pv[12];
    cx<TX> xv[12];
    cx<typename PR::real> rv[12];
    if (j < n) {
        load_spinor(p, c, j, pv);
        load_spinor(x, c, j, xv);
        load_spinor(r, c, j, rv);
    }
    const double r2 = block_sum(partial + (size_t)c * nwaves, nwaves);
    int nst = COL_ACTIVE;
    double beta = 0.0;
    if (!isfinite(r2)) {
        nst = COL_FAILED;
    } else if (r2 <= cur.stop2[c] || (cur.delta2 > 0.0 && r2 <= cur.delta2 * rmax2)) {
        nst = COL_JUST_STOPPED;  // x still takes this iteration's alpha*p
    } else {
        beta = r2 / rho;
        rho = r2;
        if (r2 > rmax2) rmax2 = r2;
    }
    if (first) {
        next.status[c] = nst;
        next.iters[c] = cur.iters[c] + 1;
        next.rho[c] = rho;
        next.rmax2[c] = rmax2;
    }
    if (nst == COL_FAILED || j >= n) return;
    const TX a = (TX)cur.alpha[c];
#pragma unroll
    for (int k = 0; k < 12; k++) {
        xv[k].re = fmadd(a, (TX)pv[k].re, xv[k].re);
        xv[k].im = fmadd(a, (TX)pv[k].im, xv[k].im);
    }
    store_spinor(x, c, j, xv);
    if (nst != COL_ACTIVE) return;
    const TP b = (TP)beta;
#pragma unroll
    for (int k = 0; k < 12; k++) {
        pv[k].re = fmadd(b, pv[k].re, (TP)rv[k].re);
        pv[k].im = fmadd(b, pv[k].im, (TP)rv[k].im);
    }
    store_spinor(p, c, j, pv);
}

__global__ void k_fin_reliable(const CgScalars s, const double* partial, int nwaves)
{
    const int c = blockIdx.x;
    const int st = s.status[c];
    const bool sel = st == COL_JUST_STOPPED || st == COL_STOPPED;
    const double r2 = sel ? block_sum(partial + (size_t)c * nwaves, nwaves) : 0.0;
    if (threadIdx.x != 0) return;
    s.restart[c] = 0;
    if (!sel) return;
    s.nrel[c] += 1;
    if (!isfinite(r2)) {
        s.status[c] = COL_FAILED;
    } else if (r2 <= s.stop2[c]) {
        s.rho[c] = r2;
        s.status[c] = COL_DONE;
    } else {
        s.beta[c] = r2 / s.rho[c];
        s.rho[c] = r2;
        s.rmax2[c] = r2;
        s.status[c] = COL_ACTIVE;
        s.restart[c] = 1;
    }
}

// ---------------------------------------------------------------------------
// dispatch helpers
// ---------------------------------------------------------------------------

constexpr int kBS = 256;

inline dim3 grid2(int n, int ncol) { return dim3((n + kBS - 1) / kBS, ncol); }

inline bool prec_ok(int prec) { return prec == PREC_F64 || prec == PREC_F32 || prec == PREC_F16; }

}  // namespace

int links_take_parts(const Geom& g) { return (g.ntiles + 1) / 2 * 4; }

hipError_t launch_links_take(const double2* canon, const Geom& g, const void* const d18[8], const void* const f18[8],
                             double* partial, hipStream_t st)
{
    LinkOut<double2> d;
    LinkOut<float2> f;
    for (int k = 0; k < 8; k++) {
        d.p[k] = (double2*)d18[k];
        f.p[k] = (float2*)f18[k];
    }
    hipLaunchKernelGGL(k_links_take, dim3((g.ntiles + 1) / 2, 4), dim3(4 * kTile), 0, st, canon, g, d, f, partial);
    return hipGetLastError();
}

hipError_t launch_links_rows(const void* const d18[8], int Vh, const void* const d12[8], const void* const f12[8],
                             const void* const h12[8], hipStream_t st)
{
    LinkOut<double2> src, d;
    LinkOut<float2> f;
    LinkOut<uint2> h;
    for (int k = 0; k < 8; k++) {
        src.p[k] = (double2*)d18[k];
        d.p[k] = (double2*)d12[k];
        f.p[k] = (float2*)f12[k];
        h.p[k] = (uint2*)h12[k];
    }
    hipLaunchKernelGGL(k_links_rows, dim3((Vh + kBS - 1) / kBS, 8), dim3(kBS), 0, st, src, Vh, d, f, h);
    return hipGetLastError();
}

// canonical array <-> np parities (from p0) of a field whose parities lie half_units / half_sites apart
template <bool IMPORT>
static hipError_t spinor_turn(double2* canon, int ncol, const Geom& g, int p0, int np, int prec, const FieldArg& f,
                              size_t half_units, size_t half_sites, hipStream_t st)
{
    if (np < 1 || np > 2 || p0 < 0 || p0 + np > 2) return hipErrorInvalidValue;
    const int tpb = 4 / np;  // tiles per workgroup
    const dim3 grid((g.ntiles + tpb - 1) / tpb, ncol), block(4 * kTile);
#define TURN(P)                                                                                                       \
    if (np == 2)                                                                                                      \
        hipLaunchKernelGGL((k_spinor_turn<P, 2, IMPORT>), grid, block, 0, st, canon, g, p0, sp<P>(f), half_units, half_sites); \
    else                                                                                                              \
        hipLaunchKernelGGL((k_spinor_turn<P, 1, IMPORT>), grid, block, 0, st, canon, g, p0, sp<P>(f), half_units, half_sites)
    switch (prec) {
    case PREC_F64: TURN(P64); break;
    case PREC_F32: TURN(P32); break;
    case PREC_F16: TURN(P16); break;
    default: return hipErrorInvalidValue;
    }
#undef TURN
    return hipGetLastError();
}

hipError_t launch_spinor_import(const double2* canon, int ncol, const Geom& g, int p0, int np, int prec, FieldArg dst,
                                size_t half_units, size_t half_sites, hipStream_t st)
{
    return spinor_turn<true>(const_cast<double2*>(canon), ncol, g, p0, np, prec, dst, half_units, half_sites, st);
}

hipError_t launch_spinor_export(FieldArg src, int ncol, const Geom& g, int p0, int np, int prec, size_t half_units,
                                size_t half_sites, double2* canon, hipStream_t st)
{
    return spinor_turn<false>(canon, ncol, g, p0, np, prec, src, half_units, half_sites, st);
}

hipError_t launch_convert(int sprec, FieldArg src, int dprec, FieldArg dst, int n, int ncol, const int* status,
                          int statmask, hipStream_t st)
{
    const dim3 grid = grid2(n, ncol);
#define CV(PS, PD) hipLaunchKernelGGL((k_convert<PS, PD>), grid, dim3(kBS), 0, st, sp<PS>(src), sp<PD>(dst), n, status, statmask)
    if (!prec_ok(sprec) || !prec_ok(dprec)) return hipErrorInvalidValue;
    const int key = sprec * 3 + dprec;
    switch (key) {
    case PREC_F64 * 3 + PREC_F64: CV(P64, P64); break;
    case PREC_F64 * 3 + PREC_F32: CV(P64, P32); break;
    case PREC_F64 * 3 + PREC_F16: CV(P64, P16); break;
    case PREC_F32 * 3 + PREC_F64: CV(P32, P64); break;
    case PREC_F32 * 3 + PREC_F32: CV(P32, P32); break;
    case PREC_F32 * 3 + PREC_F16: CV(P32, P16); break;
    case PREC_F16 * 3 + PREC_F64: CV(P16, P64); break;
    case PREC_F16 * 3 + PREC_F32: CV(P16, P32); break;
    case PREC_F16 * 3 + PREC_F16: CV(P16, P16); break;
    default: return hipErrorInvalidValue;
    }
#undef CV
    return hipGetLastError();
}

hipError_t launch_norm2(int prec, FieldArg x, int n, int ncol, double* partial, int nwaves, hipStream_t st)
{
    const dim3 grid = grid2(n, ncol);
    switch (prec) {
    case PREC_F64: hipLaunchKernelGGL(k_norm2<P64>, grid, dim3(kBS), 0, st, sp<P64>(x), n, partial, nwaves); break;
    case PREC_F32: hipLaunchKernelGGL(k_norm2<P32>, grid, dim3(kBS), 0, st, sp<P32>(x), n, partial, nwaves); break;
    case PREC_F16: hipLaunchKernelGGL(k_norm2<P16>, grid, dim3(kBS), 0, st, sp<P16>(x), n, partial, nwaves); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Plain copy of n 16-byte words, one word per thread, non-temporal on both sides: the reference
// rate against which the stencils' HBM bandwidth is read.
__global__ __launch_bounds__(256) void k_copy16(const bq_u4v* __restrict__ src, bq_u4v* __restrict__ dst, size_t n)
{
    const size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) __builtin_nontemporal_store(__builtin_nontemporal_load(src + i), dst + i);
}

hipError_t launch_copy16(const void* src, void* dst, size_t n, hipStream_t st)
{
    const size_t blocks = (n + 255) / 256;
    if (blocks > 0x7fffffff) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_copy16, dim3((unsigned)blocks), dim3(256), 0, st, (const bq_u4v*)src, (bq_u4v*)dst, n);
    return hipGetLastError();
}

hipError_t launch_zero(int prec, FieldArg x, int n, int ncol, const int* status, int statmask, hipStream_t st)
{
    const dim3 grid = grid2(n, ncol);
    switch (prec) {
    case PREC_F64: hipLaunchKernelGGL(k_zero<P64>, grid, dim3(kBS), 0, st, sp<P64>(x), n, status, statmask); break;
    case PREC_F32: hipLaunchKernelGGL(k_zero<P32>, grid, dim3(kBS), 0, st, sp<P32>(x), n, status, statmask); break;
    case PREC_F16: hipLaunchKernelGGL(k_zero<P16>, grid, dim3(kBS), 0, st, sp<P16>(x), n, status, statmask); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_dot(int prec, FieldArg x, FieldArg y, int n, int ncol, double* partial, int nwaves, hipStream_t st,
                      int gamma5)
{
    if (prec != PREC_F64) return hipErrorInvalidValue;
    if (gamma5)
        hipLaunchKernelGGL(k_dot<true>, grid2(n, ncol), dim3(kBS), 0, st, sp<P64>(x), sp<P64>(y), n, partial, nwaves);
    else
        hipLaunchKernelGGL(k_dot<false>, grid2(n, ncol), dim3(kBS), 0, st, sp<P64>(x), sp<P64>(y), n, partial, nwaves);
    return hipGetLastError();
}

hipError_t launch_cg_update(int xprec, FieldArg x, int pprec, FieldArg p, int rprec, FieldArg r, int n, int ncol,
                            const double* alpha, const double* beta, const int* status, hipStream_t st)
{
    const dim3 grid = grid2(n, ncol);
#define UP(PX, PP, PR) \
    hipLaunchKernelGGL((k_cg_update<PX, PP, PR>), grid, dim3(kBS), 0, st, sp<PX>(x), sp<PP>(p), sp<PR>(r), n, alpha, beta, status)
    if (xprec == PREC_F64 && pprec == PREC_F64 && rprec == PREC_F64) UP(P64, P64, P64);
    else if (xprec == PREC_F32 && pprec == PREC_F32 && rprec == PREC_F32) UP(P32, P32, P32);
    else if (xprec == PREC_F32 && pprec == PREC_F16 && rprec == PREC_F32) UP(P32, P16, P32);
    else return hipErrorInvalidValue;
#undef UP
    return hipGetLastError();
}

hipError_t launch_cg_update_beta(int xprec, FieldArg x, int pprec, FieldArg p, int rprec, FieldArg r, int n, int ncol,
                                 const CgScalars& cur, const CgScalars& next, const double* partial, int nwaves,
                                 hipStream_t st)
{
    if (nwaves > kFusedParts) return hipErrorInvalidValue;
    const dim3 grid = grid2(n, ncol);
#define UP(PX, PP, PR)                                                                                              \
    hipLaunchKernelGGL((k_cg_update_beta<PX, PP, PR>), grid, dim3(kBS), 0, st, sp<PX>(x), sp<PP>(p), sp<PR>(r), n, cur, next, \
                       partial, nwaves)
    if (xprec == PREC_F64 && pprec == PREC_F64 && rprec == PREC_F64) UP(P64, P64, P64);
    else if (xprec == PREC_F32 && pprec == PREC_F32 && rprec == PREC_F32) UP(P32, P32, P32);
    else if (xprec == PREC_F32 && pprec == PREC_F16 && rprec == PREC_F32) UP(P32, P16, P32);
    else return hipErrorInvalidValue;
#undef UP
    return hipGetLastError();
}

hipError_t launch_accum(int xprec, FieldArg x, FieldArg y64, int n, int ncol, const int* status, int statmask,
                        hipStream_t st)
{
    const dim3 grid = grid2(n, ncol);
    if (xprec == PREC_F32)
        hipLaunchKernelGGL(k_accum<P32>, grid, dim3(kBS), 0, st, sp<P32>(x), sp<P64>(y64), n, status, statmask);
    else if (xprec == PREC_F64)
        hipLaunchKernelGGL(k_accum<P64>, grid, dim3(kBS), 0, st, sp<P64>(x), sp<P64>(y64), n, status, statmask);
    else
        return hipErrorInvalidValue;
    return hipGetLastError();
}

hipError_t launch_restart(FieldArg r64, int rsprec, FieldArg rs, int pprec, FieldArg p, int n, int ncol,
                          const double* beta, const int* flag, hipStream_t st)
{
    const dim3 grid = grid2(n, ncol);
    const int write_rs = rs.d != r64.d;
#define RS(PRS, PP) \
    hipLaunchKernelGGL((k_restart<PRS, PP>), grid, dim3(kBS), 0, st, sp<P64>(r64), sp<PRS>(rs), sp<PP>(p), n, beta, flag, write_rs)
    if (rsprec == PREC_F64 && pprec == PREC_F64) RS(P64, P64);
    else if (rsprec == PREC_F32 && pprec == PREC_F32) RS(P32, P32);
    else if (rsprec == PREC_F32 && pprec == PREC_F16) RS(P32, P16);
    else return hipErrorInvalidValue;
#undef RS
    return hipGetLastError();
}

hipError_t launch_z2_noise(uint64_t seed, long n0, const Geom& g, int parity, FieldArg dst, int ncol, hipStream_t st)
{
    hipLaunchKernelGGL(k_z2_noise, grid2(g.Vh, ncol), dim3(kBS), 0, st, seed, n0, g, parity, sp<P64>(dst));
    return hipGetLastError();
}

hipError_t launch_fin_alpha(const CgScalars& s, const double* partial, int nwaves, int ncol, hipStream_t st)
{
    hipLaunchKernelGGL(k_fin_alpha, dim3(ncol), dim3(256), 0, st, s, partial, nwaves);
    return hipGetLastError();
}

hipError_t launch_fin_beta(const CgScalars& s, const double* partial, int nwaves, int ncol, hipStream_t st)
{
    hipLaunchKernelGGL(k_fin_beta, dim3(ncol), dim3(256), 0, st, s, partial, nwaves);
    return hipGetLastError();
}

hipError_t launch_fin_reliable(const CgScalars& s, const double* partial, int nwaves, int ncol, hipStream_t st)
{
    hipLaunchKernelGGL(k_fin_reliable, dim3(ncol), dim3(256), 0, st, s, partial, nwaves);
    return hipGetLastError();
}

hipError_t launch_fin_sum(const double* partial, int nwaves, int ncol, double* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_fin_sum, dim3(ncol), dim3(256), 0, st, partial, nwaves, out);
    return hipGetLastError();
}

hipError_t launch_fin_max(const double* partial, int n, double* out, hipStream_t st)
{
    hipLaunchKernelGGL(k_fin_max, dim3(1), dim3(256), 0, st, partial, n, out);
    return hipGetLastError();
}

// --------------------------------------------------------------------------
// multishift CG
// --------------------------------------------------------------------------

namespace {

__global__ void k_axpy_norm(SpinorPtr<P64> x, SpinorPtr<P64> y, double a, int n, double* partial, int nwaves)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    double s = 0.0;
    if (j < n) {
        cx<double> xv[12], yv[12];
        load_spinor(x, c, j, xv);
        load_spinor(y, c, j, yv);
#pragma unroll
        for (int k = 0; k < 12; k++) {
            yv[k].re = fmadd(a, xv[k].re, yv[k].re);
            yv[k].im = fmadd(a, xv[k].im, yv[k].im);
            s += yv[k].re * yv[k].re + yv[k].im * yv[k].im;
        }
        store_spinor(y, c, j, yv);
    }
    s = wave_sum(s);
    const int w = j >> kTileLog;
    if ((threadIdx.x & 63) == 0 && w < nwaves) partial[(size_t)c * nwaves + w] = s;
}

__global__ void k_ms_init(const MsState s, int ncol, double tol2)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncol) return;
    const double r2 = s.cur.rho[c];
    s.stop2[c] = tol2 * r2;
    s.cur.alpha_prev[c] = 1.0;
    s.cur.beta_prev[c] = 0.0;
    s.cur.iters[c] = 0;
    const int st = !isfinite(r2) ? COL_FAILED : (r2 > 0.0 ? COL_ACTIVE : COL_DONE);
    s.cur.status[c] = st;
    for (int k = 0; k < s.nshift; k++) {
        const int i = c * s.nshift + k;
        s.cur.zeta[i] = s.cur.zeta_prev[i] = s.zeta_new[i] = 1.0;
        s.ak[i] = 0.0;
        s.cur.act[i] = st == COL_ACTIVE;
        s.cur.kiters[i] = 0;
    }
}

// The vector work of a multishift iteration in two launches.  Every workgroup takes its column's sums
// itself (block_sum, the order of a launch of their own) and the first one of a column writes the
// scalars that others read later.  The shifts' x_k wait for the second launch, which has their p_k in
// registers anyway: 37 vectors are read or written for 8 shifts instead of 44, in one workgroup per
// 256 sites and shift instead of one for all shifts.  Bound by memory: 16^3x32, 8 shifts: 49.2 + 25.7 us,
// with the two launches for the scalars 87.7, now 14.7 + 51.0.
__global__ __launch_bounds__(256) void k_ms_residual(const MsState s, const MsFields f, const double* pq, const double* pp,
                                                     int nparts, double sigma_b, int n, double* partial, int nwaves)
{
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    const int c = blockIdx.y;
    if (s.cur.status[c] != COL_ACTIVE) return;  // uniform per block
    const SpinorPtr<P64> r = sp<P64>(f.r), w = sp<P64>(f.w), p = sp<P64>(f.p);
    cx<double> rv[12], wv[12], pv[12];
    if (j < n) {
        load_spinor(r, c, j, rv);
        load_spinor(w, c, j, wv);
        if (sigma_b != 0.0) load_spinor(p, c, j, pv);
    }
    const double qq = block_sum(pq + (size_t)c * nparts, nparts);
    const double ppn = sigma_b != 0.0 ? block_sum(pp + (size_t)c * nparts, nparts) : 0.0;
    const double pAp = qq + sigma_b * ppn;
    const bool first = blockIdx.x == 0 && threadIdx.x == 0;
    if (!(pAp > 0.0) || !isfinite(pAp)) {  // every workgroup of the column finds the same
        if (first) s.cur.status[c] = COL_FAILED;
        return;
    }
    const double al = s.cur.rho[c] / pAp;
    if (first) {
        const double ap = s.cur.alpha_prev[c], bp = s.cur.beta_prev[c];
        s.alpha[c] = al;
        for (int k = 0; k < s.nshift; k++) {
            const int i = c * s.nshift + k;
            if (!s.cur.act[i]) continue;
            const double z = s.cur.zeta[i], zp = s.cur.zeta_prev[i];
            const double zn = z * zp * ap / (al * bp * (zp - z) + zp * ap * (1.0 + s.shift[k] * al));
            s.zeta_new[i] = zn;
            s.ak[i] = al * zn / z;
        }
    }
    double nr = 0.0;
    if (j < n) {
#pragma unroll
        for (int k = 0; k < 12; k++) {
            if (sigma_b != 0.0) {
                wv[k].re = fmadd(sigma_b, pv[k].re, wv[k].re);
                wv[k].im = fmadd(sigma_b, pv[k].im, wv[k].im);
            }
            rv[k].re = fmadd(-al, wv[k].re, rv[k].re);
            rv[k].im = fmadd(-al, wv[k].im, rv[k].im);
            nr += rv[k].re * rv[k].re + rv[k].im * rv[k].im;
        }
        store_spinor(r, c, j, rv);
    }
    nr = wave_sum(nr);
    const int wave = j >> kTileLog;
    if ((threadIdx.x & 63) == 0 && wave < nwaves) partial[(size_t)c * nwaves + wave] = nr;
}

// a shift has converged in this iteration: |zeta_{j+1} r_{j+1}| <= tol |b| (or its recurrence broke down)
__device__ __forceinline__ bool ms_done(const MsState& s, int c, int i, double rho)
{
    const double zn = s.zeta_new[i];
    return zn * zn * rho <= s.stop2[c] || !isfinite(zn);
}

__global__ __launch_bounds__(256) void k_ms_directions(const MsState s, const MsFields f, const double* pr, int nparts,
                                                       int n, double* partial, int nwaves)
{
    const int c = blockIdx.y;
    // the shifts of the same sites side by side on one XCD: they share r in its L2
    const int lb = xcd_remap(blockIdx.x, gridDim.x);
    const int blk = lb / s.nshift, q = lb - blk * s.nshift;
    const int j = blk * 256 + threadIdx.x;
    const bool first = lb == 0 && threadIdx.x == 0;
    const int st = s.cur.status[c];
    const MsSet &cu = s.cur, &nx = s.next;
    if (st != COL_ACTIVE) {  // uniform per block
        if (first) {
            nx.rho[c] = cu.rho[c];
            nx.alpha_prev[c] = cu.alpha_prev[c];
            nx.beta_prev[c] = cu.beta_prev[c];
            nx.status[c] = st;
            nx.iters[c] = cu.iters[c];
            for (int k = 0; k < s.nshift; k++) {
                const int i = c * s.nshift + k;
                nx.zeta[i] = cu.zeta[i];
                nx.zeta_prev[i] = cu.zeta_prev[i];
                nx.act[i] = cu.act[i];
                nx.kiters[i] = cu.kiters[i];
            }
        }
        return;
    }
    const int iq = c * s.nshift + q;
    const bool act = cu.act[iq], base = q == s.base;
    const SpinorPtr<P64> X = sp<P64>(f.x[q]), P = sp<P64>(base ? f.p : f.pk[q]);
    cx<double> xv[12], pk[12], rv[12];
    if ((act || base) && j < n) {
        load_spinor(P, c, j, pk);
        if (act) load_spinor(X, c, j, xv);
        load_spinor(sp<P64>(f.r), c, j, rv);
    }
    const double rho0 = cu.rho[c];
    const double rho = block_sum(pr + (size_t)c * nparts, nparts);
    const bool ok = isfinite(rho);
    const double be = rho / rho0;
    bool any = false;
    for (int k = 0; k < s.nshift; k++) {
        const int i = c * s.nshift + k;
        any = any || (cu.act[i] && !ms_done(s, c, i, rho));
    }
    if (first) {
        nx.iters[c] = cu.iters[c] + 1;
        nx.alpha_prev[c] = ok ? s.alpha[c] : cu.alpha_prev[c];
        nx.beta_prev[c] = ok ? be : cu.beta_prev[c];
        nx.rho[c] = ok ? rho : rho0;
        nx.status[c] = !ok ? COL_FAILED : (any ? COL_ACTIVE : COL_DONE);
        for (int k = 0; k < s.nshift; k++) {
            const int i = c * s.nshift + k;
            const bool a = cu.act[i], go = a && ok && !ms_done(s, c, i, rho);
            nx.act[i] = ok ? go : (int)a;
            nx.kiters[i] = cu.kiters[i] + (a && ok);
            nx.zeta_prev[i] = go ? cu.zeta[i] : cu.zeta_prev[i];
            nx.zeta[i] = go ? s.zeta_new[i] : cu.zeta[i];
        }
    }
    double np = 0.0;
    if (j < n) {
        if (act) {
            const double a = s.ak[iq];
#pragma unroll
            for (int k = 0; k < 12; k++) {
                xv[k].re = fmadd(a, pk[k].re, xv[k].re);
                xv[k].im = fmadd(a, pk[k].im, xv[k].im);
            }
            store_spinor(X, c, j, xv);
        }
        if (ok && any && base) {
#pragma unroll
            for (int k = 0; k < 12; k++) {
                pk[k].re = fmadd(be, pk[k].re, rv[k].re);
                pk[k].im = fmadd(be, pk[k].im, rv[k].im);
                np += pk[k].re * pk[k].re + pk[k].im * pk[k].im;
            }
            store_spinor(P, c, j, pk);
        } else if (ok && act && !base && !ms_done(s, c, iq, rho)) {
            const double z = s.zeta_new[iq], g = z / cu.zeta[iq], b = be * g * g;
#pragma unroll
            for (int k = 0; k < 12; k++) {
                pk[k].re = fmadd(b, pk[k].re, z * rv[k].re);
                pk[k].im = fmadd(b, pk[k].im, z * rv[k].im);
            }
            store_spinor(P, c, j, pk);
        }
    }
    if (!base) return;  // uniform per block
    np = wave_sum(np);
    const int w = j >> kTileLog;
    if ((threadIdx.x & 63) == 0 && w < nwaves) partial[(size_t)c * nwaves + w] = np;
}

}  // namespace

hipError_t launch_axpy_norm(FieldArg x, FieldArg y, double a, int n, int ncol, double* partial, int nwaves,
                            hipStream_t st)
{
    hipLaunchKernelGGL(k_axpy_norm, grid2(n, ncol), dim3(kBS), 0, st, sp<P64>(x), sp<P64>(y), a, n, partial, nwaves);
    return hipGetLastError();
}

hipError_t launch_ms_init(const MsState& s, int ncol, double tol2, hipStream_t st)
{
    hipLaunchKernelGGL(k_ms_init, dim3((ncol + 63) / 64), dim3(64), 0, st, s, ncol, tol2);
    return hipGetLastError();
}

hipError_t launch_ms_residual(const MsState& s, const MsFields& f, const double* pq, const double* pp, int nparts,
                              double sigma_b, int n, int ncol, double* partial, int nwaves, hipStream_t st)
{
    if (s.nshift < 1 || s.nshift > kMaxShifts) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_ms_residual, grid2(n, ncol), dim3(kBS), 0, st, s, f, pq, pp, nparts, sigma_b, n, partial, nwaves);
    return hipGetLastError();
}

hipError_t launch_ms_directions(const MsState& s, const MsFields& f, const double* pr, int nparts, int n, int ncol,
                                double* partial, int nwaves, hipStream_t st)
{
    if (s.nshift < 1 || s.nshift > kMaxShifts) return hipErrorInvalidValue;
    hipLaunchKernelGGL(k_ms_directions, dim3((n + kBS - 1) / kBS * s.nshift, ncol), dim3(kBS), 0, st, s, f, pr, nparts, n,
                       partial, nwaves);
    return hipGetLastError();
}

}  // namespace bq

namespace bq {
namespace {
__global__ void k_cg_init(const CgScalars s, int ncol, double tol2, const int* sel, const double* tol2c,
                          const double* rho_src)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= ncol || (sel && !sel[c])) return;
    if (rho_src) s.rho[c] = rho_src[c];
    const double r2 = s.rho[c];
    s.stop2[c] = (tol2c ? tol2c[c] : tol2) * r2;
    s.rmax2[c] = r2;
    s.iters[c] = 0;
    s.nrel[c] = 0;
    s.restart[c] = 0;
    s.alpha[c] = 0.0;
    s.beta[c] = 0.0;
    s.status[c] = !isfinite(r2) ? COL_FAILED : (r2 > 0.0 ? COL_ACTIVE : COL_DONE);
}
}  // namespace

hipError_t launch_cg_init(const CgScalars& s, int ncol, double tol2, hipStream_t st, const int* sel,
                          const double* tol2c, const double* rho_src)
{
    hipLaunchKernelGGL(k_cg_init, dim3((ncol + 63) / 64), dim3(64), 0, st, s, ncol, tol2, sel, tol2c, rho_src);
    return hipGetLastError();
}

__global__ void k_set_status(int* status, const int* sel, int ncol, int value)
{
    const int c = blockIdx.x * blockDim.x + threadIdx.x;
    if (c < ncol && sel[c]) status[c] = value;
}

hipError_t launch_set_status(int* status, const int* sel, int ncol, int value, hipStream_t st)
{
    hipLaunchKernelGGL(k_set_status, dim3((ncol + 63) / 64), dim3(64), 0, st, status, sel, ncol, value);
    return hipGetLastError();
}
}  // namespace bq

// Quenched gauge configurations for the plaquette action, the ensembles of
// the paper's study (Sec. 3.1: beta = 6.0 and 5.7 on 16^4 and 32^4):
//   S = beta * sum_P (1 - Re tr U_P / 3),
//   U_P(x) = U_mu(x) U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag.
// A link U_mu(x) sees the staple sum
//   A = sum_{nu != mu} U_nu(x+mu) U_mu(x+nu)^dag U_nu(x)^dag
//                    + U_nu(x+mu-nu)^dag U_mu(x-nu)^dag U_nu(x-nu)
// and the action -beta/3 Re tr(U A).  One launch updates the links of one
// direction on the sites of one parity (their staples do not contain each
// other), FP64.
//
// Heatbath (Cabibbo-Marinari): U <- R U with R in the SU(2) subgroups on
// rows (0,1), (0,2), (1,2) in turn, drawn from exp(beta/3 Re tr(R W)),
// W = U A.  The 2x2 block r of W enters through Re tr(X r) = k Re tr(X V^dag)
// (X, V in SU(2), k >= 0), so R = Y V with y0 of Y from
// sqrt(1 - y0^2) exp(2 beta k/3 y0): y0 = 1 - delta, delta Gamma(3/2) from
// two logarithms and a cosine, accepted with probability sqrt(1 - delta/2)
// (Kennedy-Pendleton); the rest of Y uniform on the sphere of radius
// sqrt(1 - y0^2).  Over-relaxation: R = V^2 (Re tr(R r) unchanged).
// Random numbers: SplitMix64 of counters, uniform in (0, 1]:
//   key = mix(seed K1 + sweep K2), u(c) = mix(key + (c + 1) golden),
//   c = ((lex * 4 + mu) * 3 + subgroup) * 4096 + draw;
// attempt t uses draws 4t .. 4t+3, the direction draws 4000 and 4001; a link
// without acceptance in 1000 attempts keeps that subgroup unchanged.
//
// During a call the links are kept, in the caller's buffer, in tiles of 32 site
// pairs (2k, 2k+1) with the site index fastest (slot_of): in the canonical
// layout every lane of a load touches a cache line of its own.
#include "dwf_internal.h"
#include "blas.h"
#include "gauge.h"

namespace dwf {

namespace {

constexpr int GT = 256;
constexpr unsigned long long GOLD = 0x9E3779B97F4A7C15ull;
constexpr unsigned long long GK1 = 0x2545F4914F6CDD1Dull;
constexpr unsigned long long GK2 = 0x632BE59BD9B4E019ull;

__host__ __device__ inline unsigned long long mix64(unsigned long long z) {
    z ^= z >> 30;
    z *= 0xBF58476D1CE4E5B9ull;
    z ^= z >> 27;
    z *= 0x94D049BB133111EBull;
    z ^= z >> 31;
    return z;
}

__device__ inline double uniform01(unsigned long long key, unsigned long long c) {
    const unsigned long long z = mix64(key + (c + 1ull) * GOLD);
    return ((double)(z >> 11) + 1.0) * (1.0 / 9007199254740992.0);
}

struct M3 {
    double2 e[9];
};

__device__ inline double2 cadd(double2 a, double2 b) { return make_double2(a.x + b.x, a.y + b.y); }
__device__ inline double2 cmul(double2 a, double2 b) { return make_double2(a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x); }
// s + a b, four multiply-adds
__device__ inline double2 cmac(double2 s, double2 a, double2 b) {
    return make_double2(fma(-a.y, b.y, fma(a.x, b.x, s.x)), fma(a.y, b.x, fma(a.x, b.y, s.y)));
}
__device__ inline double2 cconj(double2 a) { return make_double2(a.x, -a.y); }

__device__ inline M3 load_link(const double2* U, long lex, int mu) {
    M3 m;
    const double2* p = U + (lex * 4 + mu) * 9;
#pragma unroll
    for (int k = 0; k < 9; ++k) m.e[k] = p[k];
    return m;
}

__device__ inline M3 dag(const M3& a) {
    M3 r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) r.e[i * 3 + j] = cconj(a.e[j * 3 + i]);
    return r;
}

__device__ inline M3 mul(const M3& a, const M3& b) {
    M3 r;
#pragma unroll
    for (int i = 0; i < 3; ++i)
#pragma unroll
        for (int j = 0; j < 3; ++j) {
            double2 s = cmul(a.e[i * 3], b.e[j]);
            s = cmac(s, a.e[i * 3 + 1], b.e[3 + j]);
            s = cmac(s, a.e[i * 3 + 2], b.e[6 + j]);
            r.e[i * 3 + j] = s;
        }
    return r;
}

struct Geo {
    int L[4];
    __device__ long lex(const int c[4]) const { return c[0] + (long)L[0] * (c[1] + (long)L[1] * (c[2] + (long)L[2] * c[3])); }
    __device__ void coords(long x, int c[4]) const {
        for (int mu = 0; mu < 4; ++mu) {
            c[mu] = (int)(x % L[mu]);
            x /= L[mu];
        }
    }
    __device__ long shift(const int c[4], int mu, int step) const {
        int d[4] = {c[0], c[1], c[2], c[3]};
        d[mu] = (d[mu] + step + L[mu]) % L[mu];
        return lex(d);
    }
};

// Links in tiles: pair k = lex / 2 (Lx is even: one site of each parity),
// element e = mu * 9 + row * 3 + col, at
//   tile * 32 * 72 + (e * 2 + parity) * n + k % 32,  tile = k / 32,
// n = 32 pairs (fewer in the last tile): a wave's same-parity sites are
// consecutive, and a tile occupies the bytes of its 64 canonical sites, so the
// conversion works in place.
constexpr int TPAIRS = 32, TELEM = 72 * TPAIRS;
struct Slot {
    size_t base;
    unsigned stride;   // element e at base + e * stride
};
__device__ inline Slot slot_of(unsigned lex, int parity, unsigned npairs) {
    const unsigned k = lex >> 1, t = k / TPAIRS, first = t * TPAIRS;
    const unsigned n = min((unsigned)TPAIRS, npairs - first);
    return {(size_t)t * TELEM + (unsigned)parity * n + (k - first), 2u * n};
}

// A link projected onto SU(3), element e at p[e * stride]: rows 0, 1 normalised and
// orthogonalised, row 2 = conj(row0 x row1).
__device__ __forceinline__ void project_su3(double2* p, unsigned stride) {
    double2 a[3], b[3];
    double na = 0.0, nb = 0.0;
#pragma unroll
    for (unsigned k = 0; k < 3; ++k) {
        a[k] = p[k * stride];
        b[k] = p[(3 + k) * stride];
        na += a[k].x * a[k].x + a[k].y * a[k].y;
    }
    na = sqrt(na);
    double2 dot = make_double2(0.0, 0.0);
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        a[k] = make_double2(a[k].x / na, a[k].y / na);
        dot = cadd(dot, cmul(cconj(a[k]), b[k]));
    }
#pragma unroll
    for (int k = 0; k < 3; ++k) {
        const double2 t = cmul(dot, a[k]);
        b[k] = make_double2(b[k].x - t.x, b[k].y - t.y);
        nb += b[k].x * b[k].x + b[k].y * b[k].y;
    }
    nb = sqrt(nb);
#pragma unroll
    for (int k = 0; k < 3; ++k) b[k] = make_double2(b[k].x / nb, b[k].y / nb);
#pragma unroll
    for (unsigned k = 0; k < 3; ++k) {
        const unsigned i = (k + 1) % 3, j = (k + 2) % 3;
        const double2 u = cmul(a[i], b[j]), v = cmul(a[j], b[i]);
        p[k * stride] = a[k];
        p[(3 + k) * stride] = b[k];
        p[(6 + k) * stride] = make_double2(u.x - v.x, -(u.y - v.y));
    }
}

// The links after a sweep, in tiles: a thread per link, site fastest.  Bound by
// memory: 16^4 10.9 us (75 MB at 5.8 TB/s without the third rows' reads).  After
// the call's last sweep the conversion back does it, in the time of its own
// (15.6 us).
__global__ __launch_bounds__(GT) void gauge_project_kernel(double2* __restrict__ U, unsigned npairs) {
    const unsigned l = blockIdx.x * GT + threadIdx.x, t = l / (2 * TPAIRS), mu = blockIdx.y;
    if (l >= 2 * npairs) return;
    const unsigned n = min((unsigned)TPAIRS, npairs - t * TPAIRS);
    project_su3(U + (size_t)t * TELEM + (size_t)(mu * 9) * (2 * n) + (l - t * (2 * TPAIRS)), 2 * n);
}

// canonical -> tiles (TO_TILES), or back with the links projected, in place, one
// tile per block
template <bool TO_TILES>
__global__ __launch_bounds__(GT) void gauge_tiles_kernel(double2* __restrict__ U, Geo g, unsigned npairs) {
    __shared__ double2 buf[TELEM];
    const unsigned first = blockIdx.x * TPAIRS, n = min((unsigned)TPAIRS, npairs - first);
    double2* p = U + (size_t)blockIdx.x * TELEM;
    for (unsigned e = threadIdx.x; e < 72u * n; e += GT) buf[e] = p[e];
    __syncthreads();
    if (!TO_TILES) {
        static_assert(GT == 2 * TPAIRS * 4, "a thread per link of the tile");
        const unsigned l = threadIdx.x % (2u * TPAIRS), mu = threadIdx.x / (2u * TPAIRS);
        if (l < 2u * n) project_su3(buf + mu * 9u * (2u * n) + l, 2u * n);
        __syncthreads();
    }
    for (unsigned e = threadIdx.x; e < 72u * n; e += GT) {
        // e walks the destination; site q of the tile's 2 n sites, element m of 36
        unsigned q, m, src;
        if (TO_TILES) {
            const unsigned mp = e / n, k = e - mp * n;
            m = mp >> 1;
            const unsigned pair = first + k;
            const unsigned row = 2u * pair / (unsigned)g.L[0], r2 = row / (unsigned)g.L[1];
            const unsigned odd = (row % (unsigned)g.L[1] + r2 % (unsigned)g.L[2] + r2 / (unsigned)g.L[2]) & 1u;
            q = 2u * k + ((odd + mp) & 1u);   // the site of parity mp & 1
            src = q * 36u + m;
        } else {
            q = e / 36u;
            m = e - q * 36u;
            const unsigned k = q >> 1, pair = first + k;
            const unsigned row = 2u * pair / (unsigned)g.L[0], r2 = row / (unsigned)g.L[1];
            const unsigned odd = (row % (unsigned)g.L[1] + r2 % (unsigned)g.L[2] + r2 / (unsigned)g.L[2]) & 1u;
            src = (m * 2u + ((odd + q) & 1u)) * n + k;
        }
        p[e] = buf[src];
    }
}

// value of lane `from` of the quad (a constant after unrolling)
template <int P0, int P1, int P2, int P3>
__device__ inline double quad(double v) {
    constexpr int ctl = P0 | (P1 << 2) | (P2 << 4) | (P3 << 6);
    const int lo = __builtin_amdgcn_mov_dpp(__double2loint(v), ctl, 0xf, 0xf, true);
    const int hi = __builtin_amdgcn_mov_dpp(__double2hiint(v), ctl, 0xf, 0xf, true);
    return __hiloint2double(hi, lo);
}
template <int P0, int P1, int P2, int P3>
__device__ inline double2 quad(double2 v) { return make_double2(quad<P0, P1, P2, P3>(v.x), quad<P0, P1, P2, P3>(v.y)); }
__device__ inline double quad_sum(double v) {
    v += quad<1, 0, 3, 2>(v);
    return v + quad<2, 3, 0, 1>(v);
}

__device__ inline M3 load_m3(const double2* __restrict__ U, Slot s, int mu) {
    M3 m;
#pragma unroll
    for (int k = 0; k < 9; ++k) m.e[k] = (U + s.base)[(unsigned)(mu * 9 + k) * s.stride];
    return m;
}

// column `lane` of a row (by value: a select of references would put the row
// into scratch memory); lane 3 repeats column 0
__device__ inline double2 column(int lane, const double2 a, const double2 b, const double2 c) {
    return make_double2(lane == 1 ? b.x : (lane == 2 ? c.x : a.x), lane == 1 ? b.y : (lane == 2 ? c.y : a.y));
}

// Subgroup (a, b) of one link: w, u = column c of W and of the link on lane c
template <bool HB, int A, int B>
__device__ inline void update_subgroup(double2 (&w)[3], double2 (&u)[3], double beta, unsigned long long key,
                                       unsigned long long c0) {
    const double2 r00 = quad<A, A, A, A>(w[A]), r10 = quad<A, A, A, A>(w[B]);
    const double2 r01 = quad<B, B, B, B>(w[A]), r11 = quad<B, B, B, B>(w[B]);
    double q[4] = {0.5 * (r00.x + r11.x), -0.5 * (r01.y + r10.y), -0.5 * (r01.x - r10.x), -0.5 * (r00.y - r11.y)};
    const double k = sqrt(q[0] * q[0] + q[1] * q[1] + q[2] * q[2] + q[3] * q[3]);
    const double rk = k > 0.0 ? 1.0 / k : 1.0;
#pragma unroll
    for (int t = 0; t < 4; ++t) q[t] *= rk;
    double x[4];   // R as a quaternion
    if constexpr (HB) {
        const double alpha = k > 0.0 ? 2.0 * beta * k / 3.0 : 1e-300;
        const double ralpha = 1.0 / alpha;
        bool ok = false;
        double y0 = 1.0;
        for (int t = 0; t < 1000 && !ok; ++t) {
            const unsigned long long cb = c0 + 4ull * (unsigned long long)t;
            const double u1 = uniform01(key, cb), u2 = uniform01(key, cb + 1), u3 = uniform01(key, cb + 2),
                         u4 = uniform01(key, cb + 3);
            const double cs = cospi(2.0 * u2);
            const double delta = -(log(u1) + cs * cs * log(u3)) * ralpha;
            if (u4 * u4 <= 1.0 - 0.5 * delta) {
                y0 = 1.0 - delta;
                ok = true;
            }
        }
        const double cth = 2.0 * uniform01(key, c0 + 4000) - 1.0;
        double sp, cp;
        sincospi(2.0 * uniform01(key, c0 + 4001), &sp, &cp);
        const double rad = sqrt(fmax(0.0, 1.0 - y0 * y0));
        const double rs = rad * sqrt(fmax(0.0, 1.0 - cth * cth));
        const double y1 = rs * cp, y2 = rs * sp, y3 = rad * cth;
        // (y0 + i y.sigma)(q0 + i q.sigma) = y0 q0 - y.q + i (y0 q + q0 y - y x q).sigma
        x[0] = ok ? y0 * q[0] - y1 * q[1] - y2 * q[2] - y3 * q[3] : 1.0;
        x[1] = ok ? y0 * q[1] + q[0] * y1 - (y2 * q[3] - y3 * q[2]) : 0.0;
        x[2] = ok ? y0 * q[2] + q[0] * y2 - (y3 * q[1] - y1 * q[3]) : 0.0;
        x[3] = ok ? y0 * q[3] + q[0] * y3 - (y1 * q[2] - y2 * q[1]) : 0.0;
    } else {
        x[0] = q[0] * q[0] - q[1] * q[1] - q[2] * q[2] - q[3] * q[3];
#pragma unroll
        for (int t = 1; t < 4; ++t) x[t] = 2.0 * q[0] * q[t];
    }
    // rows a, b of both columns: [[x0 + i x3, x2 + i x1], [-x2 + i x1, x0 - i x3]]
    const double2 R00 = make_double2(x[0], x[3]), R01 = make_double2(x[2], x[1]), R10 = make_double2(-x[2], x[1]),
                  R11 = make_double2(x[0], -x[3]);
    const double2 wa = w[A], wb = w[B], ua = u[A], ub = u[B];
    w[A] = cmac(cmul(R00, wa), R01, wb);
    w[B] = cmac(cmul(R10, wa), R11, wb);
    u[A] = cmac(cmul(R00, ua), R01, ub);
    u[B] = cmac(cmul(R10, ua), R11, ub);
}

// One update of U_mu on the sites of one parity.  Four lanes per link: lane nu forms the two staples of
// direction nu, then lane c (0..2) carries column c of the link and of W
// through the subgroups.  On 16^4 (131072 lanes, two waves per SIMD) a launch is bound
// by its own chain (loads, ~650 FP64 instructions, square roots): 13.5 us, and
// 23.4 us for the heatbath; one thread per link in the canonical layout took
// 29 us.  A step of one heatbath and four over-relaxation sweeps: 16^4 1.33 ->
// 0.65 ms, 24^3x48 16.2 -> 5.6 ms (0.61 and 5.2 with the projection at the end of
// each update instead, but then the staples of a sweep see its links projected,
// which is another update for links that are not exactly SU(3)).
constexpr int GU = 256;
template <bool HB>
__global__ __launch_bounds__(GU) __attribute__((amdgpu_waves_per_eu(2))) void gauge_update_kernel(
    double2* __restrict__ U, Geo g, int mu, int parity, double beta, unsigned long long key, unsigned npairs) {
    // blocks are dealt to the 8 XCDs in turn, each with an L2 of its own: XCD x
    // takes one contiguous eighth of the lattice
    const unsigned nb = gridDim.x, bx = blockIdx.x & 7u, bq = nb >> 3, br = nb & 7u;
    const unsigned blk = bx * bq + min(bx, br) + (blockIdx.x >> 3);
    const unsigned pair = (blk * GU + threadIdx.x) >> 2;
    const bool live = pair < npairs;
    const unsigned pr = live ? pair : npairs - 1;   // spare quads repeat the last link and store nothing
    const int lane = threadIdx.x & 3, nu = lane;
    const unsigned L0 = g.L[0], L1 = g.L[1], L2 = g.L[2], L3 = g.L[3];
    const unsigned row = 2u * pr / L0, r2 = row / L1, c3 = r2 / L2;
    const unsigned c1 = row - r2 * L1, c2 = r2 - c3 * L2;
    const unsigned c0 = 2u * pr - row * L0 + (((unsigned)parity + c1 + c2 + c3) & 1u);
    const unsigned x = row * L0 + c0;
    // coordinate, extent and stride of direction mu and of this lane's nu
    auto pick = [](int d, unsigned v0, unsigned v1, unsigned v2, unsigned v3) -> unsigned {
        const unsigned a = d & 1 ? v1 : v0, b = d & 1 ? v3 : v2;
        return d & 2 ? b : a;
    };
    const unsigned S2 = L0 * L1, S3 = S2 * L2;
    const unsigned cm = pick(mu, c0, c1, c2, c3), em = pick(mu, L0, L1, L2, L3), tm = pick(mu, 1u, L0, S2, S3);
    const unsigned cn = pick(nu, c0, c1, c2, c3), en = pick(nu, L0, L1, L2, L3), tn = pick(nu, 1u, L0, S2, S3);
    const unsigned up_m = cm + 1 == em ? 0u - (em - 1) * tm : tm, up_n = cn + 1 == en ? 0u - (en - 1) * tn : tn;
    const unsigned dn_n = cn == 0 ? (en - 1) * tn : 0u - tn;
    const int q = 1 - parity;
    const Slot sx = slot_of(x, parity, npairs);
    const M3 Ul = load_m3(U, sx, mu);
    M3 A;
#pragma unroll
    for (int k = 0; k < 9; ++k) A.e[k] = make_double2(0.0, 0.0);
    if (nu != mu) {
        const unsigned xm = x + up_m, xn = x + up_n, xb = x + dn_n, xmb = xb + up_m;   // (mod 2^32)
        const Slot sm = slot_of(xm, q, npairs), sn = slot_of(xn, q, npairs), sb = slot_of(xb, q, npairs),
                   smb = slot_of(xmb, parity, npairs);
        const M3 up = mul(mul(load_m3(U, sm, nu), dag(load_m3(U, sn, mu))), dag(load_m3(U, sx, nu)));
        const M3 dn = mul(mul(dag(load_m3(U, smb, nu)), dag(load_m3(U, sb, mu))), load_m3(U, sb, nu));
#pragma unroll
        for (int k = 0; k < 9; ++k) A.e[k] = cadd(up.e[k], dn.e[k]);
    }
    // sum over the quad; lane c keeps column c of A, of the link and of W = U A
    double2 w[3], u[3], ac[3];
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        double2 t[3];
#pragma unroll
        for (int c = 0; c < 3; ++c) t[c] = make_double2(quad_sum(A.e[i * 3 + c].x), quad_sum(A.e[i * 3 + c].y));
        ac[i] = column(lane, t[0], t[1], t[2]);
        u[i] = column(lane, Ul.e[i * 3], Ul.e[i * 3 + 1], Ul.e[i * 3 + 2]);
    }
#pragma unroll
    for (int i = 0; i < 3; ++i)
        w[i] = cmac(cmac(cmul(Ul.e[i * 3], ac[0]), Ul.e[i * 3 + 1], ac[1]), Ul.e[i * 3 + 2], ac[2]);
    const unsigned long long cbase = ((unsigned long long)x * 4ull + (unsigned long long)mu) * 3ull;
    update_subgroup<HB, 0, 1>(w, u, beta, key, cbase * 4096ull);
    update_subgroup<HB, 0, 2>(w, u, beta, key, (cbase + 1ull) * 4096ull);
    update_subgroup<HB, 1, 2>(w, u, beta, key, (cbase + 2ull) * 4096ull);
    if (live && lane < 3) {
#pragma unroll
        for (int i = 0; i < 3; ++i) (U + sx.base)[(unsigned)(mu * 9 + i * 3 + lane) * sx.stride] = u[i];
    }
}

// Sum of Re tr over the plaquettes of 64 sites, one plane per wave.  Bound by the
// latency of its loads (a lane's links lie 576 bytes apart) and by their number;
// the six planes of a site share the cache lines: 16^4 42 us, 52 us with
// one thread for all planes of a site.
constexpr int PLAQ_SITES = 64, PLAQ_PLANES = 6;
__global__ __launch_bounds__(PLAQ_SITES * PLAQ_PLANES) void gauge_plaquette_kernel(const double2* __restrict__ U, Geo g,
                                                                                  long V, double* __restrict__ partial) {
    __shared__ double red[PLAQ_PLANES];
    const long x = (long)blockIdx.x * PLAQ_SITES + (threadIdx.x & 63);
    const int plane = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int mu = plane < 3 ? 0 : (plane < 5 ? 1 : 2), nu = plane < 3 ? plane + 1 : (plane < 5 ? plane - 1 : 3);
    double acc = 0.0;
    if (x < V) {
        int c[4];
        g.coords(x, c);
        const long xpmu = g.shift(c, mu, +1), xpnu = g.shift(c, nu, +1);
        const M3 P = mul(mul(mul(load_link(U, x, mu), load_link(U, xpmu, nu)), dag(load_link(U, xpnu, mu))),
                         dag(load_link(U, x, nu)));
        acc = P.e[0].x + P.e[4].x + P.e[8].x;
    }
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if ((threadIdx.x & 63) == 0) red[plane] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < PLAQ_PLANES; ++w) t += red[w];
        partial[blockIdx.x] = t;
    }
}

Geo geo_of(const int dims[4]) {
    Geo g;
    for (int mu = 0; mu < 4; ++mu) g.L[mu] = dims[mu];
    return g;
}

}  // namespace

void gauge_sweeps(void* U, const int dims[4], double beta, int nsweeps, int n_or, unsigned long long seed,
                  long long sweep0, hipStream_t st) {
    if (nsweeps <= 0) return;
    const long V = (long)dims[0] * dims[1] * dims[2] * dims[3];
    DWF_REQUIRE(V < (1L << 31), DWF_EDIMS, "lattice too large for 32-bit site indices");
    const unsigned npairs = (unsigned)(V / 2), tiles = (npairs + TPAIRS - 1) / TPAIRS;
    const unsigned blocks = (unsigned)((4L * npairs + GU - 1) / GU);
    const Geo g = geo_of(dims);
    double2* u = static_cast<double2*>(U);
    hipLaunchKernelGGL(gauge_tiles_kernel<true>, dim3(tiles), dim3(GT), 0, st, u, g, npairs);
    for (int k = 0; k < nsweeps; ++k) {
        const unsigned long long key = mix64(seed * GK1 + (unsigned long long)(sweep0 + k) * GK2);
        for (int o = 0; o <= n_or; ++o) {
            for (int mu = 0; mu < 4; ++mu)
                for (int p = 0; p < 2; ++p) {
                    if (o == 0)
                        hipLaunchKernelGGL(gauge_update_kernel<true>, dim3(blocks), dim3(GU), 0, st, u, g, mu, p, beta,
                                           key, npairs);
                    else
                        hipLaunchKernelGGL(gauge_update_kernel<false>, dim3(blocks), dim3(GU), 0, st, u, g, mu, p, beta,
                                           key, npairs);
                }
            if (o < n_or || k + 1 < nsweeps)
                hipLaunchKernelGGL(gauge_project_kernel, dim3((2 * npairs + GT - 1) / GT, 4), dim3(GT), 0, st, u, npairs);
        }
    }
    hipLaunchKernelGGL(gauge_tiles_kernel<false>, dim3(tiles), dim3(GT), 0, st, u, g, npairs);
    DWF_HIP(hipGetLastError());
}

int gauge_plaquette_partials(const int dims[4]) {
    const long V = (long)dims[0] * dims[1] * dims[2] * dims[3];
    return (int)((V + PLAQ_SITES - 1) / PLAQ_SITES);
}

void gauge_plaquette(const void* U, const int dims[4], double* partial, double* out_dev, hipStream_t st) {
    const long V = (long)dims[0] * dims[1] * dims[2] * dims[3];
    const int nb = gauge_plaquette_partials(dims);
    hipLaunchKernelGGL(gauge_plaquette_kernel, dim3(nb), dim3(PLAQ_SITES * PLAQ_PLANES), 0, st, static_cast<const double2*>(U),
                       geo_of(dims), V, partial);
    DWF_HIP(hipGetLastError());
    finalize(partial, nb, 1, out_dev, 0, st);
}

}  // namespace dwf

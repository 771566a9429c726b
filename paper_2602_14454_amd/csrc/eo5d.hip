// Kernels of the five-dimensional even-odd split (layout and operator in
// eo5d.h).  One lane per (site, s) of the output half field: the 5D
// blocks have no dense fifth-dimension part, so there is nothing for MFMA
// here; the hop is the spin-projected Wilson hop of the fused kernel's
// conventions, with the K and 1 / M_ss scalings folded into per-slice,
// per-chirality factors.
#include <type_traits>

#include "eo5d.h"
#include "precision.h"

namespace dwf {

namespace {

// Chiral basis: gamma_mu = [[0, B],[B^dag, 0]] with B = -i sigma_1, -i sigma_2,
// -i sigma_3, 1 for mu = x, y, z, t.  (1 + SG gamma_mu) psi = (w, SG B^dag w),
// w = psi_up + SG B psi_lo.  Components: index spin * 3 + colour, re/im pairs.
// The input enters with its chirality's factor c[0], c[1]; the products of the
// lower components are rounded, those of the upper ones are not.
template <int MU, class T>
__device__ __forceinline__ void project(T sg, const T (&p)[24], const T (&c)[2], T (&w)[12]) {
    // w[h * 6 + a * 2 + reim] for half-spinor row h = 0, 1
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const T l0r = c[1] * p[(2 * 3 + a) * 2], l0i = c[1] * p[(2 * 3 + a) * 2 + 1];
        const T l1r = c[1] * p[(3 * 3 + a) * 2], l1i = c[1] * p[(3 * 3 + a) * 2 + 1];
        T b0r, b0i, b1r, b1i;   // B psi_lo
        if (MU == 0) {          // -i sigma_1: (-i l1, -i l0)
            b0r = l1i; b0i = -l1r; b1r = l0i; b1i = -l0r;
        } else if (MU == 1) {   // -i sigma_2 = [[0,-1],[1,0]]: (-l1, l0)
            b0r = -l1r; b0i = -l1i; b1r = l0r; b1i = l0i;
        } else if (MU == 2) {   // -i sigma_3: (-i l0, i l1)
            b0r = l0i; b0i = -l0r; b1r = -l1i; b1i = l1r;
        } else {                // 1
            b0r = l0r; b0i = l0i; b1r = l1r; b1i = l1i;
        }
        w[0 * 6 + a * 2] = fma(c[0], p[(0 * 3 + a) * 2], sg * b0r);
        w[0 * 6 + a * 2 + 1] = fma(c[0], p[(0 * 3 + a) * 2 + 1], sg * b0i);
        w[1 * 6 + a * 2] = fma(c[0], p[(1 * 3 + a) * 2], sg * b1r);
        w[1 * 6 + a * 2 + 1] = fma(c[0], p[(1 * 3 + a) * 2 + 1], sg * b1i);
    }
}

// acc_up += v, acc_lo += SG B^dag v for v = U w (two half-spinor rows)
template <int MU, class T>
__device__ __forceinline__ void reconstruct(T sg, const T (&v)[12], T (&acc)[24]) {
#pragma unroll
    for (int a = 0; a < 3; ++a) {
        const T v0r = v[0 * 6 + a * 2], v0i = v[0 * 6 + a * 2 + 1];
        const T v1r = v[1 * 6 + a * 2], v1i = v[1 * 6 + a * 2 + 1];
        acc[(0 * 3 + a) * 2] += v0r;
        acc[(0 * 3 + a) * 2 + 1] += v0i;
        acc[(1 * 3 + a) * 2] += v1r;
        acc[(1 * 3 + a) * 2 + 1] += v1i;
        T c0r, c0i, c1r, c1i;   // B^dag v
        if (MU == 0) {          // i sigma_1: (i v1, i v0)
            c0r = -v1i; c0i = v1r; c1r = -v0i; c1i = v0r;
        } else if (MU == 1) {   // [[0,1],[-1,0]]: (v1, -v0)
            c0r = v1r; c0i = v1i; c1r = -v0r; c1i = -v0i;
        } else if (MU == 2) {   // i sigma_3: (i v0, -i v1)
            c0r = -v0i; c0i = v0r; c1r = v1i; c1i = -v1r;
        } else {
            c0r = v0r; c0i = v0i; c1r = v1r; c1i = v1i;
        }
        acc[(2 * 3 + a) * 2] += sg * c0r;
        acc[(2 * 3 + a) * 2 + 1] += sg * c0i;
        acc[(3 * 3 + a) * 2] += sg * c1r;
        acc[(3 * 3 + a) * 2 + 1] += sg * c1i;
    }
}

}  // namespace

// the 12 components of slice s at site j
template <class T>
__device__ __forceinline__ void load_site(const void* f, int s, long j, int Ls, T (&v)[24]) {
#pragma unroll
    for (int g = 0; g < 3; ++g) {
        T q[8];
        load4<T>(f, gidx(s * 3 + g, j, Ls * 3), q);
#pragma unroll
        for (int k = 0; k < 8; ++k) v[8 * g + k] = q[k];
    }
}

template <int MU, class T>
__device__ __forceinline__ void eo5_direction(const Eo5Params& P, const void* lk, int d, T sg, int s, int q, long i,
                                              const T (&cin)[2], T (&acc)[24]) {
    constexpr int CB = 2 * (int)sizeof(T), LP = link_lp(CB), NG = link_ng(CB);
    const long j = P.nbr[(long)q * 8 * P.Vhp + gidx(d, i, 8)];
    T p[24], u[18], w[12], v[12];
    load_site<T>(P.in, s, j, P.Ls, p);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
        static_assert(LP * CB == 16, "16-byte link groups expected");
        const u32x4 x = static_cast<const u32x4*>(lk)[gidx(d * NG + g, i, 8 * NG)];
        decode_link_group<T>(x, g, u);
    }
    project<MU, T>(sg, p, cin, w);
    // U w; every complex product rounded before it is added
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            T re = 0, im = 0;
#pragma unroll
            for (int b = 0; b < 3; ++b) {
                const T ur = u[(a * 3 + b) * 2], ui = u[(a * 3 + b) * 2 + 1];
                const T xr = w[h * 6 + b * 2], xi = w[h * 6 + b * 2 + 1];
                const T tr = fma(ur, xr, -(ui * xi)), ti = fma(ur, xi, ui * xr);
                re = b ? re + tr : tr;
                im = b ? im + ti : ti;
            }
            v[h * 6 + a * 2] = re;
            v[h * 6 + a * 2 + 1] = im;
        }
    reconstruct<MU, T>(sg, v, acc);
}

// A block takes 64 sites of one 4D parity and four of the slices (s, s + 2, ...)
// that have this parity in the output: its waves read the same links.  Blocks
// go to the 8 XCDs in contiguous ranges of sites, and an XCD sweeps its sites
// for four slices before the next four, so that neighbouring sites are still in
// its L2.  16^4, Ls = 16, FP32: 73 us a launch (the 142 to 192 MB it must move
// take 25 to 33 us at the copy rate; neither more waves per SIMD nor eight
// unrolled directions changed it), 106 us with one block per slice and 8-byte
// loads.
template <class T>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(sizeof(T) == 8 ? 2 : 4))) void eo5_kernel(
    Eo5Params P, int tiles, int groups) {
    const long Vh = P.Vh;
    const int xcd = blockIdx.x & 7, n = (int)blockIdx.x >> 3;
    const int t0 = tiles * xcd / 8, nt = tiles * (xcd + 1) / 8 - t0;
    if (n >= nt * 2 * groups) return;
    const int sel = n / nt;
    const int s = (sel & 1) + 2 * ((sel >> 1) * 4 + ((int)threadIdx.x >> 6));
    const long i = (long)(t0 + n % nt) * 64 + (threadIdx.x & 63);
    if (s >= P.Ls || i >= Vh) return;
    const int q = (P.par + s) & 1;   // 4D parity of the output site
    const double* KD = P.coef + EO5_KD;
    const double* MINV = P.coef + EO5_MINV;
    const double* MM = P.coef + EO5_M;

    // scalings of the hop's input (slice s) and of its result, per chirality
    T cin[2], cout[2];
#pragma unroll
    for (int chi = 0; chi < 2; ++chi) {
        const T mi = P.pre ? T(MINV[chi * 16 + s]) : T(1);
        cin[chi] = P.dagger ? mi : T(KD[chi * 16 + s]) * mi;
        cout[chi] = P.dagger ? T(KD[chi * 16 + s]) : T(1);
    }

    T acc[24];
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] = 0;
    const void* lk = static_cast<const char*>(P.links) + (size_t)q * P.lpar * 2 * sizeof(T);
    for (int h = 0; h < 8; h += 4) {
        // forward hop (x + mu) carries (1 - gamma), backward (1 + gamma);
        // the adjoint (gamma_5 H gamma_5) flips both
        const T sg = (h == 0) != (P.dagger != 0) ? T(-1) : T(1);
        eo5_direction<0, T>(P, lk, h, sg, s, q, i, cin, acc);
        eo5_direction<1, T>(P, lk, h + 1, sg, s, q, i, cin, acc);
        eo5_direction<2, T>(P, lk, h + 2, sg, s, q, i, cin, acc);
        eo5_direction<3, T>(P, lk, h + 3, sg, s, q, i, cin, acc);
    }
    // -1/2 H (times K on the output side for the adjoint)
#pragma unroll
    for (int k = 0; k < 24; ++k) acc[k] *= T(-0.5) * (k < 12 ? cout[0] : cout[1]);

    // shift in s at the same site: (M - diag M) per chirality, rows s and
    // columns s -/+ 1 (transposed for the adjoint)
    const int Ls = P.Ls;
    const int qm = (s + Ls - 1) % Ls, qp = (s + 1) % Ls;
    int qs[2], nq = 0;   // distinct neighbouring slices (one for Ls = 2, none for Ls = 1)
    if (qm != s) qs[nq++] = qm;
    if (qp != s && qp != qm) qs[nq++] = qp;
    for (int n = 0; n < nq; ++n) {
        const int sq = qs[n];
        T c[2];
#pragma unroll
        for (int chi = 0; chi < 2; ++chi) {
            const double m = P.dagger ? MM[(chi * 16 + sq) * 16 + s] : MM[(chi * 16 + s) * 16 + sq];
            c[chi] = T(m) * (P.pre ? T(MINV[chi * 16 + sq]) : T(1));
        }
        T v[24];
        load_site<T>(P.in, sq, i, Ls, v);
#pragma unroll
        for (int k = 0; k < 24; ++k) acc[k] = fma(k < 12 ? c[0] : c[1], v[k], acc[k]);
    }
    const T mo[2] = {T(MINV[0 * 16 + s]), T(MINV[1 * 16 + s])};
    const T sgn = T(P.sgn), a = T(P.a);
    T l[24];
    if (P.loc) load_site<T>(P.loc, s, i, Ls, l);
#pragma unroll
    for (int g = 0; g < 3; ++g) {
        T o[8];
#pragma unroll
        for (int k8 = 0; k8 < 8; ++k8) {
            const int k = 8 * g + k8, chi = k < 12 ? 0 : 1;
            const T hs = P.post_hop ? mo[chi] : T(1);
            T r = sgn * hs * acc[k];
            if (P.loc) {
                const T ls = a * (P.post_loc ? mo[chi] : T(1));
                r = fma(ls, l[k], r);
            }
            o[k8] = r;
        }
        store4<T>(P.out, gidx(s * 3 + g, i, Ls * 3), o);
    }
}

__global__ __launch_bounds__(256) void eo5_diag_kernel(double2* out, const double2* in, const double* coef, long n,
                                                       int Ls) {
    const long t = (long)blockIdx.x * 256 + threadIdx.x;
    if (t >= n) return;
    const int row = (int)((t >> 4) % (Ls * 12));
    const int s = row / 12, k = row - s * 12;
    const int chi = k < 6 ? 0 : 1;
    const double m = coef[EO5_M + (chi * 16 + s) * 16 + s];
    out[t] = make_double2(m * in[t].x, m * in[t].y);
}

static unsigned grid_of(long work) { return (unsigned)((work + 255) / 256); }

void launch_eo5(int kind, const Eo5Params& P, hipStream_t st) {
    DWF_REQUIRE(P.Ls >= 1 && P.Ls <= LS_MAX, DWF_EDIMS, "Ls out of range for the 5D even-odd split");
    if (P.Vh == 0) return;
    const int tiles = (int)((P.Vh + 63) / 64), groups = ((P.Ls + 1) / 2 + 3) / 4;
    const unsigned blocks = 8u * (unsigned)((tiles + 7) / 8) * 2u * (unsigned)groups;
    if (kind == ST_F64) hipLaunchKernelGGL(eo5_kernel<double>, dim3(blocks), dim3(256), 0, st, P, tiles, groups);
    else if (kind == ST_F32) hipLaunchKernelGGL(eo5_kernel<float>, dim3(blocks), dim3(256), 0, st, P, tiles, groups);
    else throw Error{DWF_EINVAL, "the 5D even-odd split runs in FP64 or FP32"};
    DWF_HIP(hipGetLastError());
}

void eo5_diag(void* out, const void* in, const double* coef, long Vhp, int Ls, hipStream_t st) {
    const long n = (long)Ls * 12 * Vhp;
    if (n == 0) return;
    hipLaunchKernelGGL(eo5_diag_kernel, dim3(grid_of(n)), dim3(256), 0, st, static_cast<double2*>(out),
                       static_cast<const double2*>(in), coef, n, Ls);
    DWF_HIP(hipGetLastError());
}

}  // namespace dwf

// Kernels of the learned preconditioner: a linear, gauge-equivariant
// parallel-transport convolution (PTC) network (layers, weight gradients,
// loss, Adam).  Fields are FP32 internal half fields (precision.h), one per
// channel, channel after channel.
//
// One layer, for the sites x of one parity p:
//   out^a(x, s) = sum_b [ sum_{q in 0, +s, -s} W_q^{ab} in_loc^b(x, s + shift_q)
//                       + sum_{d = 0..7}     W_{1+d}^{ab} L_d(x) in_hop^b(nbr_d(x), s) ]
// where L_d(x) is the hop link of direction d (U_mu(x) forward, U_mu(x-mu)^dag
// backward, boundary phase folded; the same tables as the Wilson hop), W is
// a complex 4x4 spin matrix and in_loc / in_hop live on parity p / 1 - p.
// Path numbering: 0 identity, 1..8 = direction d + 1, 9 = +s, 10 = -s.
//
// The network is linear, and a weight (spin) commutes with a transport
// (colour, site), so the two layers are one sum over pairs of paths:
//   M r = sum_{q, q'} E_{qq'} T_q T_q' r,   E_{qq'} = sum_b W2_q^b W1_q'^b  (4x4),
// q, q' both local (even hidden sites) or both links (odd hidden sites).  Its
// cost does not depend on the number of hidden channels, and neither does that
// of the gradient, which needs the 4x4 correlations dL/dE_{qq'} =
// sum (T_q^dag g) (T_q' r)^dag and then only products of small matrices:
//   dL/dW2_q^b = sum_q' dL/dE_{qq'} W1_q'^b^dag,  dL/dW1_q'^b = sum_q W2_q^b^dag dL/dE_{qq'}.
// E is summed in FP64 and rounded once.
#include <algorithm>

#include "dwf_internal.h"
#include "precision.h"
#include "ptc.h"

namespace dwf {

constexpr int PT = 256;

__device__ __forceinline__ void cfma(float2& acc, float2 a, float2 b) {
    acc.x += a.x * b.x - a.y * b.y;
    acc.y += a.x * b.y + a.y * b.x;
}

// v (12 complex, spin-major) of slice s at internal site i
__device__ __forceinline__ void load12(const float2* f, int s, long i, int Ls, float2 (&v)[12]) {
#pragma unroll
    for (int q = 0; q < 6; ++q) {
        const float4 a = reinterpret_cast<const float4*>(f)[gidx(s * 6 + q, i, Ls * 6)];
        v[2 * q] = make_float2(a.x, a.y);
        v[2 * q + 1] = make_float2(a.z, a.w);
    }
}

__device__ __forceinline__ void store12(float2* f, int s, long i, int Ls, const float2 (&v)[12]) {
#pragma unroll
    for (int q = 0; q < 6; ++q)
        reinterpret_cast<float4*>(f)[gidx(s * 6 + q, i, Ls * 6)] =
            make_float4(v[2 * q].x, v[2 * q].y, v[2 * q + 1].x, v[2 * q + 1].y);
}

// the link of direction d at site i (9 complex; pairs, one 16-byte load each)
__device__ __forceinline__ void load_link(const float2* links, int d, long i, float2 (&L)[10]) {
#pragma unroll
    for (int g = 0; g < 5; ++g) {
        const float4 a = reinterpret_cast<const float4*>(links)[gidx(d * 5 + g, i, 40)];
        L[2 * g] = make_float2(a.x, a.y);
        L[2 * g + 1] = make_float2(a.z, a.w);
    }
}

// t = L v on every spin
__device__ __forceinline__ void transport(const float2 (&L)[10], const float2 (&v)[12], float2 (&t)[12]) {
#pragma unroll
    for (int sp = 0; sp < 4; ++sp)
#pragma unroll
        for (int a = 0; a < 3; ++a) {
            float2 acc = make_float2(0.f, 0.f);
#pragma unroll
            for (int b = 0; b < 3; ++b) cfma(acc, L[a * 3 + b], v[sp * 3 + b]);
            t[sp * 3 + a] = acc;
        }
}

// acc += W v  (W: 4x4 complex on spin, row-major; v, acc: 12 complex)
__device__ __forceinline__ void spin_apply(const float2* __restrict__ W, const float2 (&v)[12], float2 (&acc)[12]) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float2 w = W[i * 4 + j];
#pragma unroll
            for (int c = 0; c < 3; ++c) cfma(acc[i * 3 + c], w, v[j * 3 + c]);
        }
}

// One layer from one channel to one: one thread per (site, slice).
__global__ __launch_bounds__(PT) void ptc_layer_kernel(PtcLayerParams P) {
    const long i = (long)blockIdx.x * PT + threadIdx.x;
    if (i >= P.Vh) return;
    const int s = blockIdx.y;
    const int Ls = P.Ls;
    float2 acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = make_float2(0.f, 0.f);
    // local paths: 0 (same slice), 9 (s + 1), 10 (s - 1)
    if (P.in_loc) {
        for (int qi = 0; qi < 3; ++qi) {
            const int q = qi == 0 ? 0 : 8 + qi;
            const int ss = qi == 0 ? s : (qi == 1 ? s + 1 : s - 1);
            if (ss < 0 || ss >= P.Ls) continue;
            float2 t[12];
            load12(P.in_loc, ss, i, Ls, t);
            spin_apply(P.W + q * 16, t, acc);
        }
    }
    // link paths 1..8
    if (P.in_hop) {
        for (int d = 0; d < 8; ++d) {
            const long y = P.nbr[gidx(d, i, 8)];
            float2 v[12], t[12];
            load12(P.in_hop, s, y, Ls, v);
            float2 L[10];
            load_link(P.links, d, i, L);
            transport(L, v, t);
            spin_apply(P.W + (1 + d) * 16, t, acc);
        }
    }
    store12(P.out, s, i, Ls, acc);
}

// ---------------------------------------------------------------------
// the two layers as one (E_{qq'} above)
// ---------------------------------------------------------------------
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v4f __attribute__((ext_vector_type(4)));

// Link part of E as the MFMA A operand of ptc_mid_kernel, then the local part:
//   el[((d' * 4 + j) * 2 + tile) * 64 + lane], lane = 32 h + 4 d + i:
//     the factor of (re, im)[h] of t_{d', j} in (re, im)[tile] of g_{d, i}
//   al[k * 16 + i * 4 + j]: k = 0..3 the factor of r(s - 2), r(s - 1), r(s + 1),
//     r(s + 2); k = 4 + c that of r(s), with the term through s + 1 and back if
//     c & 1 and the one through s - 1 if c & 2 (present where that slice is);
//     al[AL + ..] what rounding these to FP32 left (they hold the identity that
//     a trained network stays near: their rounding would be the same at every
//     site, and the gradients' error against 64 bits 15 % larger with it).
// A chain of latencies: four lanes share the sum of an element (8^4, Ls = 8: one
// application 66.7 -> 64.9 us with 8 hidden channels, 79.9 -> 68.5 with 32).
constexpr int AL = 8 * 16;
__global__ __launch_bounds__(PT) void ptc_pair_weights(const float2* __restrict__ W1, const float2* __restrict__ W2,
                                                       int H, float* __restrict__ el, float2* __restrict__ al) {
    const int t = (blockIdx.x * PT + threadIdx.x) >> 2, k4 = threadIdx.x & 3;   // four lanes, one per inner spin
    if (t >= 1024 + AL) return;
    int q[3] = {0, 0, 0}, p[3] = {0, 0, 0}, n = 1, i, j;
    if (t < 1024) {   // t = d' * 128 + j * 32 + d * 4 + i
        i = t & 3;
        q[0] = 1 + ((t >> 2) & 7);
        j = (t >> 5) & 3;
        p[0] = 1 + (t >> 7);
    } else {
        const int k = (t - 1024) >> 4;
        i = ((t - 1024) >> 2) & 3;
        j = t & 3;
        if (k == 0) { q[0] = 10; p[0] = 10; }
        if (k == 1) { q[0] = 0; p[0] = 10; q[1] = 10; p[1] = 0; n = 2; }
        if (k == 2) { q[0] = 0; p[0] = 9; q[1] = 9; p[1] = 0; n = 2; }
        if (k == 3) { q[0] = 9; p[0] = 9; }
        if (k == 5 || k == 7) { q[1] = 9; p[1] = 10; n = 2; }
        if (k == 6 || k == 7) { q[n] = 10; p[n] = 9; ++n; }
    }
    double re = 0.0, im = 0.0;
    for (int m = 0; m < n; ++m)
#pragma unroll 4
        for (int b = 0; b < H; ++b) {
            const float2 x = W2[((long)q[m] * H + b) * 16 + i * 4 + k4], y = W1[((long)p[m] * H + b) * 16 + k4 * 4 + j];
            re += (double)x.x * y.x - (double)x.y * y.y;
            im += (double)x.x * y.y + (double)x.y * y.x;
        }
#pragma unroll
    for (int off = 1; off <= 2; off <<= 1) {
        re += __shfl_xor(re, off, 64);
        im += __shfl_xor(im, off, 64);
    }
    if (k4) return;
    if (t < 1024) {
        const int d = q[0] - 1, ks = (p[0] - 1) * 4 + j;
        float* o = el + (long)ks * 128 + 4 * d + i;
        o[0] = (float)re;
        o[32] = (float)-im;
        o[64] = (float)im;
        o[96] = (float)re;
    } else {
        const float2 hi = make_float2((float)re, (float)im);
        al[t - 1024] = hi;
        al[t - 1024 + AL] = make_float2((float)(re - hi.x), (float)(im - hi.y));
    }
}

// g_d(y, s) = sum_{d'} E_{dd'} (T_d' r)(y, s) for the eight d at the sites y of
// one parity (odd), as 32 x 32 complex times 32 x (sites x colours) on
// v_mfma_f32_32x32x2: a wave takes 32 sites of one slice, and the two halves
// of its lanes hold the real and the imaginary part of the same t, which is
// the B operand (column = site, k = re/im).  A lane ends up with four of the
// eight g_d of its site.  Links, neighbours and E are in LDS for the block's
// 32 sites and all slices.  Bound by the matrix cores (12288 multiply-adds per
// site and slice), 56 % busy, and by a last round of blocks that fills two thirds
// of the chip: 358 us on 16^3x32, Ls = 16 (72 TFLOP/s; a large FP32 product reaches
// 152); 412 us with the next slice's first loads behind this slice's stores.
// NT: non-temporal stores, for a g that the last-level cache (256 MB) does not
// hold anyway; ptc_out then finds more of what it reads besides (16^3x32, 805 MB:
// 226 us with, 264 without, and 371 against 357 here; 16^4, Ls = 8, 201 MB: 62
// against 53, and 84 against 87 here).  The whole network on 16^3x32: 0.59 ms for any
// number of channels; two layers of 8 channels, one thread per site and slice, took
// 2.5 to 2.8 ms.
template <bool NT>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void ptc_mid_kernel(
    const float2* __restrict__ r, float2* __restrict__ g, const float2* __restrict__ links,
    const int* __restrict__ nbr, const float* __restrict__ el, long Vh, long Vhp, int Ls) {
    __shared__ u32x4 lnk[8 * 5 * 32];
    __shared__ u32x4 ew4[1024];
    __shared__ int lnb[8 * 32];
    const long tile = xcd_block(blockIdx.x, gridDim.x);
    const int nthr = blockDim.x;
    for (int e = threadIdx.x; e < 8 * 5 * 32; e += nthr) {
        const long site = tile * 32 + (e & 31);
        lnk[e] = reinterpret_cast<const u32x4*>(links)[gidx(e >> 5, site < Vh ? site : Vh - 1, 40)];
    }
    for (int e = threadIdx.x; e < 8 * 32; e += nthr) {
        const long site = tile * 32 + (e & 31);
        lnb[e] = (int)gidx(0, nbr[gidx(e >> 5, site < Vh ? site : Vh - 1, 8)], Ls * 6);   // of a field's 16-byte groups
    }
    for (int e = threadIdx.x; e < 1024; e += nthr) ew4[e] = reinterpret_cast<const u32x4*>(el)[e];
    __syncthreads();
    const float* ew = reinterpret_cast<const float*>(ew4);
    const int lane = threadIdx.x & 63, j = lane & 31, h = lane >> 5;
    const long site = tile * 32 + j;
    const long n = (long)Ls * 12 * Vhp;
    const float4* r4 = reinterpret_cast<const float4*>(r);
    float4 nx[6];
#pragma unroll
    for (int q = 0; q < 6; ++q) nx[q] = r4[lnb[j] + ((int)(threadIdx.x >> 6) * 6 + q) * 16];
    for (int s = threadIdx.x >> 6; s < Ls; s += nthr >> 6) {
        v16f acc[3][2];
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int k = 0; k < 16; ++k) { acc[c][0][k] = 0.f; acc[c][1][k] = 0.f; }
#pragma unroll 1
        for (int d = 0; d < 8; ++d) {
            // real lanes use (re, -im) of the spinor, imaginary lanes (im, re)
            float a[12], b[12];
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                a[2 * q] = h ? nx[q].y : nx[q].x;
                b[2 * q] = h ? nx[q].x : -nx[q].y;
                a[2 * q + 1] = h ? nx[q].w : nx[q].z;
                b[2 * q + 1] = h ? nx[q].z : -nx[q].w;
            }
            // the next direction's spinor, in flight meanwhile; after the last one the next
            // slice's first, requested before this slice's stores (a load is waited for
            // with every store that was issued before it)
            const int y = lnb[((d + 1) & 7) * 32 + j], sn = d < 7 ? s : min(s + (nthr >> 6), Ls - 1);
#pragma unroll
            for (int q = 0; q < 6; ++q) nx[q] = r4[y + (sn * 6 + q) * 16];
            __builtin_amdgcn_sched_barrier(0);
            float U[20];
#pragma unroll
            for (int k = 0; k < 5; ++k) {
                const u32x4 w = lnk[(d * 5 + k) * 32 + j];
                U[4 * k] = __uint_as_float(w.x);
                U[4 * k + 1] = __uint_as_float(w.y);
                U[4 * k + 2] = __uint_as_float(w.z);
                U[4 * k + 3] = __uint_as_float(w.w);
            }
#pragma unroll
            for (int sp = 0; sp < 4; ++sp) {
                const float e0 = ew[((d * 4 + sp) * 2) * 64 + lane], e1 = ew[((d * 4 + sp) * 2 + 1) * 64 + lane];
#pragma unroll
                for (int c = 0; c < 3; ++c) {
                    float t = U[6 * c] * a[sp * 3];
                    t = __builtin_fmaf(U[6 * c + 1], b[sp * 3], t);
#pragma unroll
                    for (int k = 1; k < 3; ++k) {
                        t = __builtin_fmaf(U[6 * c + 2 * k], a[sp * 3 + k], t);
                        t = __builtin_fmaf(U[6 * c + 2 * k + 1], b[sp * 3 + k], t);
                    }
                    acc[c][0] = __builtin_amdgcn_mfma_f32_32x32x2f32(e0, t, acc[c][0], 0, 0, 0);
                    acc[c][1] = __builtin_amdgcn_mfma_f32_32x32x2f32(e1, t, acc[c][1], 0, 0, 0);
                }
            }
        }
        if (site < Vh) {
            // rows of accumulator slot 4 k + i: 8 k + 4 h + i = 4 (2 k + h) + i, spin i of direction 2 k + h
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                float2* gd = g + (long)(2 * k + h) * n;
#pragma unroll
                for (int q = 0; q < 6; ++q) {
                    const int c0 = (2 * q) % 3, s0 = (2 * q) / 3, c1 = (2 * q + 1) % 3, s1 = (2 * q + 1) / 3;
                    const v4f o = {acc[c0][0][4 * k + s0], acc[c0][1][4 * k + s0], acc[c1][0][4 * k + s1],
                                   acc[c1][1][4 * k + s1]};
                    v4f* to = reinterpret_cast<v4f*>(gd) + gidx(s * 6 + q, site, Ls * 6);
                    if constexpr (NT) __builtin_nontemporal_store(o, to);
                    else *to = o;
                }
            }
        }
    }
}

// out(x, s) = local pairs of r + sum_d L_d(x) g_d(nbr_d(x), s) at the even
// sites; one thread per (site, slice), one slice per wave.  Bound by memory (every
// g_d is read once, 8 fields; r and the links come from cache) and by half as much
// arithmetic.  The slices of 64 sites follow each other on one XCD: 226 us on
// 16^3x32, Ls = 16 (1.05 GB at 4.6 TB/s); 288 us with the sites of four slices in sequence
// over all XCDs and with the two terms through s + 1 and s - 1 and back as matrices
// of their own.  Two slices per thread, with the links read once, were no faster.
__global__ __launch_bounds__(256) void ptc_out_kernel(const float2* __restrict__ r, const float2* __restrict__ g,
                                                      float2* __restrict__ out, const float2* __restrict__ links,
                                                      const int* __restrict__ nbr, const float2* __restrict__ al,
                                                      long Vh, long Vhp, int Ls, int groups) {
    const int b = xcd_block(blockIdx.x, gridDim.x);
    const long i = (long)(b / groups) * 64 + (threadIdx.x & 63);
    const int s = __builtin_amdgcn_readfirstlane(b % groups * 4 + (int)(threadIdx.x >> 6));
    if (s >= Ls || i >= Vh) return;
    const long n = (long)Ls * 12 * Vhp;
    float2 acc[12];
#pragma unroll
    for (int k = 0; k < 12; ++k) acc[k] = make_float2(0.f, 0.f);
#pragma unroll 2
    for (int d = 0; d < 8; ++d) {
        const long y = nbr[gidx(d, i, 8)];
        float2 L[10], m[12], t[12];
        load_link(links, d, i, L);
        load12(g + d * n, s, y, Ls, m);
        transport(L, m, t);
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            acc[k].x += t[k].x;
            acc[k].y += t[k].y;
        }
    }
#pragma unroll 1
    for (int k = -2; k <= 2; ++k) {
        if (s + k < 0 || s + k >= Ls) continue;
        float2 v[12];
        load12(r, s + k, i, Ls, v);
        const float2* a = al + 16 * (k < 0 ? k + 2 : (k > 0 ? k + 1 : 4 + (s + 1 < Ls ? 1 : 0) + (s > 0 ? 2 : 0)));
        spin_apply(a + AL, v, acc);
        spin_apply(a, v, acc);
    }
    store12(out, s, i, Ls, acc);
}

// Correlations C[a][b] = sum_{site, s, colour} u_a conj(t_b), a, b = 0..31 = 4 x
// slot + spin, of one parity's sites:
//   links (LOCAL 0, odd sites): u slot d = T_d g, t slot d = T_d r;
//   local (LOCAL 1, even sites): t slots 0..4 = r(s + slot - 2), u slots 0..2 =
//   g everywhere, where slice s + 1 exists, where s - 1 exists; others zero.
// A block forms both sides for 32 sites of one slice (a thread per site and
// slot; a link serves both), passes them through LDS, and its four waves
// multiply a quarter of the 96 (site, colour) terms each on
// v_mfma_f32_32x32x2.  Sums of 24 terms are kept in FP32, everything beyond
// in FP64 (a fixed order: the same bits on every run).  16^4, Ls = 8: 107 and
// 83 us, against 2.5 ms for the weight gradients of 8 channels path by path.  The LDS row stride of
// 33 puts the 32 sites of a write on different banks.
template <int LOCAL>
__global__ __launch_bounds__(256) void ptc_corr_kernel(const float2* __restrict__ r, const float2* __restrict__ g,
                                                       const float2* __restrict__ links, const int* __restrict__ nbr,
                                                       long Vh, int Ls, long ntiles,
                                                       double* __restrict__ partial) {
    constexpr int NK = 96, ST = 33;
    __shared__ double smem[4 * NK * ST / 2];
    float* ur = reinterpret_cast<float*>(smem);
    float *ui = ur + NK * ST, *tr = ui + NK * ST, *ti = tr + NK * ST;
    const int j = threadIdx.x & 31, slot = threadIdx.x >> 5;
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    double cr[16], ci[16];
#pragma unroll
    for (int k = 0; k < 16; ++k) { cr[k] = 0.0; ci[k] = 0.0; }
    for (long tl = blockIdx.x; tl < ntiles; tl += gridDim.x) {
        const int s = (int)(tl % Ls);
        const long site = tl / Ls * 32 + j;
        float2 t[12], u[12];
#pragma unroll
        for (int k = 0; k < 12; ++k) {
            t[k] = make_float2(0.f, 0.f);
            u[k] = make_float2(0.f, 0.f);
        }
        if (site < Vh) {
            if constexpr (LOCAL) {
                const int ss = s + slot - 2;
                if (slot < 5 && ss >= 0 && ss < Ls) load12(r, ss, site, Ls, t);
                if (slot == 0 || (slot == 1 && s + 1 < Ls) || (slot == 2 && s > 0)) load12(g, s, site, Ls, u);
            } else {
                const long y = nbr[gidx(slot, site, 8)];
                float2 v[12], v2[12];
                load12(r, s, y, Ls, v);
                load12(g, s, y, Ls, v2);
                float2 L[10];
                load_link(links, slot, site, L);
                transport(L, v, t);
                transport(L, v2, u);
            }
        }
        __syncthreads();   // the previous tile's reads
#pragma unroll
        for (int c = 0; c < 3; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int at = (j * 3 + c) * ST + slot * 4 + i;
                ur[at] = u[i * 3 + c].x;
                ui[at] = u[i * 3 + c].y;
                tr[at] = t[i * 3 + c].x;
                ti[at] = t[i * 3 + c].y;
            }
        __syncthreads();
        v16f ar, ai;
#pragma unroll
        for (int k = 0; k < 16; ++k) { ar[k] = 0.f; ai[k] = 0.f; }
#pragma unroll
        for (int m = 0; m < NK / 8; ++m) {
            const int at = (2 * (w * (NK / 8) + m) + (lane >> 5)) * ST + (lane & 31);
            const float xr = ur[at], xi = ui[at], yr = tr[at], yi = ti[at];
            ar = __builtin_amdgcn_mfma_f32_32x32x2f32(xr, yr, ar, 0, 0, 0);
            ai = __builtin_amdgcn_mfma_f32_32x32x2f32(xi, yr, ai, 0, 0, 0);
            ar = __builtin_amdgcn_mfma_f32_32x32x2f32(xi, yi, ar, 0, 0, 0);
            ai = __builtin_amdgcn_mfma_f32_32x32x2f32(-xr, yi, ai, 0, 0, 0);
        }
#pragma unroll
        for (int k = 0; k < 16; ++k) {
            cr[k] += (double)ar[k];
            ci[k] += (double)ai[k];
        }
    }
    // the four waves in turn; accumulator slot k of a lane: row 8 (k / 4) + 4 (lane / 32) + k % 4, column lane % 32
    double* red = smem;   // [re, im][32][32]
    for (int ww = 0; ww < 4; ++ww) {
        __syncthreads();
        if (w == ww) {
#pragma unroll
            for (int k = 0; k < 16; ++k) {
                const int at = (8 * (k / 4) + 4 * (lane >> 5) + k % 4) * 32 + (lane & 31);
                red[at] = (ww ? red[at] : 0.0) + cr[k];
                red[1024 + at] = (ww ? red[1024 + at] : 0.0) + ci[k];
            }
        }
    }
    __syncthreads();
    for (int e = threadIdx.x; e < 2048; e += 256) partial[(long)blockIdx.x * 2048 + e] = red[e];
}

// c[set][e] = sum over blocks, e < 2048; eight threads per value, fixed order
__global__ __launch_bounds__(256) void ptc_corr_finalize(const double* __restrict__ partial, int nblocks,
                                                         double* __restrict__ c) {
    __shared__ double red[8][32];
    const int e = threadIdx.x & 31, part = threadIdx.x >> 5;
    const double* p = partial + (long)blockIdx.y * nblocks * 2048 + blockIdx.x * 32 + e;
    double a = 0.0;
#pragma unroll 4
    for (int b = part; b < nblocks; b += 8) a += p[(long)b * 2048];
    red[part][e] = a;
    __syncthreads();
    if (part == 0) {
        for (int k = 1; k < 8; ++k) a += red[k][e];
        c[(long)blockIdx.y * 2048 + blockIdx.x * 32 + e] = a;
    }
}

// dL/dE_{qq'}[i][j] from the correlations (set 0: links, set 1: local)
__device__ __forceinline__ double2 pair_grad(const double* c, int q, int p, int i, int j) {
    int set, a, b;
    if (q >= 1 && q <= 8) {
        // g meets T_d at the far end: T_d^dag = T of the reversed direction
        set = 0;
        a = (q - 1) ^ 4;
        b = p - 1;
    } else {
        set = 1;
        const int dq = q == 0 ? 0 : (q == 9 ? 1 : -1), dp = p == 0 ? 0 : (p == 9 ? 1 : -1);
        a = dq * dp == -1 ? (q == 9 ? 1 : 2) : 0;
        b = dq + dp + 2;
    }
    const long at = (long)set * 2048 + (a * 4 + i) * 32 + b * 4 + j;
    return make_double2(c[at], c[at + 1024]);
}

// weight gradients of both layers (products of 4x4 matrices, FP64)
__global__ __launch_bounds__(PT) void ptc_weight_grad(const double* __restrict__ c, const float2* __restrict__ W1,
                                                      const float2* __restrict__ W2, int H, float2* __restrict__ G1,
                                                      float2* __restrict__ G2) {
    const int t = blockIdx.x * PT + threadIdx.x;
    if (t >= 2 * 11 * H * 16) return;
    const int layer = t / (11 * H * 16), w = t % (11 * H * 16);
    const int j = w & 3, i = (w >> 2) & 3, b = (w >> 4) % H, q = (w >> 4) / H;
    const bool link = q >= 1 && q <= 8;
    double re = 0.0, im = 0.0;
    for (int m = 0; m < (link ? 8 : 3); ++m) {
        const int p = link ? 1 + m : (m == 0 ? 0 : 8 + m);
        for (int k = 0; k < 4; ++k) {
            // layer 2: dE_{qp}[i][k] conj(W1_p[j][k]); layer 1: conj(W2_p[k][i]) dE_{pq}[k][j]
            const double2 e = layer ? pair_grad(c, q, p, i, k) : pair_grad(c, p, q, k, j);
            const float2 x = layer ? W1[((long)p * H + b) * 16 + j * 4 + k] : W2[((long)p * H + b) * 16 + k * 4 + i];
            re += e.x * x.x + e.y * x.y;
            im += e.y * x.x - e.x * x.y;
        }
    }
    (layer ? G2 : G1)[w] = make_float2((float)re, (float)im);
}

// partial sums of |y - e|^2 and |e|^2 (FP64) over one half field
__global__ __launch_bounds__(PT) void ptc_loss_partial(const float2* y, const float2* e, long n, double* partial) {
    __shared__ double red[2][PT / 64];
    double d2 = 0.0, e2 = 0.0;
    for (long k = (long)blockIdx.x * PT + threadIdx.x; k < n; k += (long)gridDim.x * PT) {
        const float2 a = y[k], b = e[k];
        const double dx = (double)a.x - b.x, dy = (double)a.y - b.y;
        d2 += dx * dx + dy * dy;
        e2 += (double)b.x * b.x + (double)b.y * b.y;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        d2 += __shfl_xor(d2, off, 64);
        e2 += __shfl_xor(e2, off, 64);
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) { red[0][w] = d2; red[1][w] = e2; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0, b = 0;
        for (int k = 0; k < PT / 64; ++k) { a += red[0][k]; b += red[1][k]; }
        partial[2 * blockIdx.x] = a;
        partial[2 * blockIdx.x + 1] = b;
    }
}

// out[0] = |y-e|^2 / |e|^2 (loss), out[1] = |e|^2, out[2] = |y-e|^2
__global__ __launch_bounds__(PT) void ptc_loss_finalize(const double* partial, int nparts, double* out) {
    __shared__ double red[2][PT / 64];
    double a = 0, b = 0;
    for (int k = threadIdx.x; k < nparts; k += PT) { a += partial[2 * k]; b += partial[2 * k + 1]; }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        a += __shfl_xor(a, off, 64);
        b += __shfl_xor(b, off, 64);
    }
    if ((threadIdx.x & 63) == 0) { red[0][threadIdx.x >> 6] = a; red[1][threadIdx.x >> 6] = b; }
    __syncthreads();
    if (threadIdx.x != 0) return;
    for (int k = 1; k < PT / 64; ++k) { a += red[0][k]; b += red[1][k]; }
    out[0] = b > 0 ? a / b : 0.0;
    out[1] = b;
    out[2] = a;
}

// g = 2 (y - e) / |e|^2
__global__ __launch_bounds__(PT) void ptc_loss_grad(const float2* y, const float2* e, long n, const double* stats,
                                                    float2* g) {
    const double e2 = stats[1];
    const float sc = e2 > 0 ? (float)(2.0 / e2) : 0.f;
    for (long k = (long)blockIdx.x * PT + threadIdx.x; k < n; k += (long)gridDim.x * PT) {
        const float2 a = y[k], b = e[k];
        g[k] = make_float2(sc * (a.x - b.x), sc * (a.y - b.y));
    }
}

// residual loss: out[0] = |u|^2 / |r|^2, out[1] = |r|^2, out[2] = |u|^2 (partials as ptc_loss_partial)
__global__ __launch_bounds__(PT) void ptc_norms_partial(const float2* u, const float2* r, long n, double* partial) {
    __shared__ double red[2][PT / 64];
    double u2 = 0.0, r2 = 0.0;
    for (long k = (long)blockIdx.x * PT + threadIdx.x; k < n; k += (long)gridDim.x * PT) {
        const float2 a = u[k], b = r[k];
        u2 += (double)a.x * a.x + (double)a.y * a.y;
        r2 += (double)b.x * b.x + (double)b.y * b.y;
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) {
        u2 += __shfl_xor(u2, off, 64);
        r2 += __shfl_xor(r2, off, 64);
    }
    const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
    if (lane == 0) { red[0][w] = u2; red[1][w] = r2; }
    __syncthreads();
    if (threadIdx.x == 0) {
        double a = 0, b = 0;
        for (int k2 = 0; k2 < PT / 64; ++k2) { a += red[0][k2]; b += red[1][k2]; }
        partial[2 * blockIdx.x] = a;
        partial[2 * blockIdx.x + 1] = b;
    }
}

// d = y - e
__global__ __launch_bounds__(PT) void ptc_sub(const float2* y, const float2* e, long n, float2* d) {
    for (long k = (long)blockIdx.x * PT + threadIdx.x; k < n; k += (long)gridDim.x * PT) {
        const float2 a = y[k], b = e[k];
        d[k] = make_float2(a.x - b.x, a.y - b.y);
    }
}

// g = (2 / stats[1]) w
__global__ __launch_bounds__(PT) void ptc_scale_grad(const float2* w, long n, const double* stats, float2* g) {
    const double r2 = stats[1];
    const float sc = r2 > 0 ? (float)(2.0 / r2) : 0.f;
    for (long k = (long)blockIdx.x * PT + threadIdx.x; k < n; k += (long)gridDim.x * PT) {
        const float2 a = w[k];
        g[k] = make_float2(sc * a.x, sc * a.y);
    }
}

// Adam on n real parameters (Kingma and Ba); bc1 = 1 - b1^t, bc2 = 1 - b2^t
__global__ __launch_bounds__(PT) void ptc_adam_kernel(float* w, const float* g, float* m, float* v, int n, float lr,
                                                      float b1, float b2, float eps, float bc1, float bc2) {
    const int k = blockIdx.x * PT + threadIdx.x;
    if (k >= n) return;
    const float gk = g[k];
    const float mk = b1 * m[k] + (1.f - b1) * gk;
    const float vk = b2 * v[k] + (1.f - b2) * gk * gk;
    m[k] = mk;
    v[k] = vk;
    w[k] -= lr * (mk / bc1) / (sqrtf(vk / bc2) + eps);
}

// ---------------------------------------------------------------------
void ptc_layer(const PtcLayerParams& P, hipStream_t st) {
    DWF_REQUIRE(P.Ls >= 1 && P.Vh >= 1, DWF_EINVAL, "bad PTC layer shape");
    hipLaunchKernelGGL(ptc_layer_kernel, dim3((unsigned)((P.Vh + PT - 1) / PT), (unsigned)P.Ls), dim3(PT), 0, st, P);
    DWF_HIP(hipGetLastError());
}

void ptc_pairs_forward(const PtcPairParams& P, const float2* r, float2* out, hipStream_t st) {
    DWF_REQUIRE(P.Ls >= 1 && P.Vh >= 1 && P.H >= 1, DWF_EINVAL, "bad PTC shape");
    hipLaunchKernelGGL(ptc_pair_weights, dim3((4 * (1024 + AL) + PT - 1) / PT), dim3(PT), 0, st, P.W1, P.W2, P.H, P.el,
                       P.al);
    const dim3 mid_grid((unsigned)((P.Vh + 31) / 32)), mid_block(64 * (P.Ls < 4 ? P.Ls : 4));
    if ((double)P.Ls * 12 * P.Vhp * 8 * sizeof(float2) > 256e6)
        hipLaunchKernelGGL(ptc_mid_kernel<true>, mid_grid, mid_block, 0, st, r, P.mid, P.links[1], P.nbr[1], P.el, P.Vh,
                           P.Vhp, P.Ls);
    else
        hipLaunchKernelGGL(ptc_mid_kernel<false>, mid_grid, mid_block, 0, st, r, P.mid, P.links[1], P.nbr[1], P.el, P.Vh,
                           P.Vhp, P.Ls);
    const int groups = (P.Ls + 3) / 4;
    hipLaunchKernelGGL(ptc_out_kernel, dim3((unsigned)((P.Vh + 63) / 64 * groups)), dim3(256), 0, st, r, P.mid, out,
                       P.links[0], P.nbr[0], P.al, P.Vh, P.Vhp, P.Ls, groups);
    DWF_HIP(hipGetLastError());
}

static long corr_tiles(const PtcPairParams& P) { return (P.Vh + 31) / 32 * P.Ls; }
static int corr_blocks(const PtcPairParams& P) { return (int)std::min<long>(corr_tiles(P), 768); }
size_t ptc_corr_bytes(const PtcPairParams& P) { return ((size_t)2 * corr_blocks(P) + 2) * 2048 * sizeof(double); }

void ptc_pairs_gradient(const PtcPairParams& P, const float2* r, const float2* g, double* corr, float2* G1,
                        float2* G2, hipStream_t st) {
    const int nb = corr_blocks(P);
    double* c = corr + (size_t)2 * nb * 2048;
    hipLaunchKernelGGL(ptc_corr_kernel<0>, dim3(nb), dim3(256), 0, st, r, g, P.links[1], P.nbr[1], P.Vh, P.Ls,
                       corr_tiles(P), corr);
    hipLaunchKernelGGL(ptc_corr_kernel<1>, dim3(nb), dim3(256), 0, st, r, g, P.links[0], P.nbr[0], P.Vh, P.Ls,
                       corr_tiles(P), corr + (size_t)nb * 2048);
    hipLaunchKernelGGL(ptc_corr_finalize, dim3(64, 2), dim3(256), 0, st, corr, nb, c);
    hipLaunchKernelGGL(ptc_weight_grad, dim3((2 * 11 * P.H * 16 + PT - 1) / PT), dim3(PT), 0, st, c, P.W1, P.W2, P.H, G1,
                       G2);
    DWF_HIP(hipGetLastError());
}

int ptc_loss_blocks(long n) {
    long b = (n + PT - 1) / PT;
    return (int)(b > 1024 ? 1024 : (b < 1 ? 1 : b));
}

void ptc_loss(const float2* y, const float2* e, long n, double* partial, double* stats, float2* g, hipStream_t st) {
    const int nb = ptc_loss_blocks(n);
    hipLaunchKernelGGL(ptc_loss_partial, dim3(nb), dim3(PT), 0, st, y, e, n, partial);
    hipLaunchKernelGGL(ptc_loss_finalize, dim3(1), dim3(PT), 0, st, partial, nb, stats);
    if (g) hipLaunchKernelGGL(ptc_loss_grad, dim3(nb), dim3(PT), 0, st, y, e, n, stats, g);
    DWF_HIP(hipGetLastError());
}

void ptc_sub(const float2* y, const float2* e, long n, float2* d, hipStream_t st) {
    hipLaunchKernelGGL(ptc_sub, dim3(ptc_loss_blocks(n)), dim3(PT), 0, st, y, e, n, d);
    DWF_HIP(hipGetLastError());
}

void ptc_norms(const float2* u, const float2* r, long n, double* partial, double* stats, hipStream_t st) {
    const int nb = ptc_loss_blocks(n);
    hipLaunchKernelGGL(ptc_norms_partial, dim3(nb), dim3(PT), 0, st, u, r, n, partial);
    hipLaunchKernelGGL(ptc_loss_finalize, dim3(1), dim3(PT), 0, st, partial, nb, stats);
    DWF_HIP(hipGetLastError());
}

void ptc_scale_grad(const float2* w, long n, const double* stats, float2* g, hipStream_t st) {
    hipLaunchKernelGGL(ptc_scale_grad, dim3(ptc_loss_blocks(n)), dim3(PT), 0, st, w, n, stats, g);
    DWF_HIP(hipGetLastError());
}

void ptc_adam(float* w, const float* g, float* m, float* v, int n, float lr, float b1, float b2, float eps, int step,
              hipStream_t st) {
    const float bc1 = 1.f - std::pow(b1, (float)step), bc2 = 1.f - std::pow(b2, (float)step);
    hipLaunchKernelGGL(ptc_adam_kernel, dim3((n + PT - 1) / PT), dim3(PT), 0, st, w, g, m, v, n, lr, b1, b2, eps, bc1,
                       bc2);
    DWF_HIP(hipGetLastError());
}

}  // namespace dwf

// Single-lattice launches of the fused hop (hop_tile.h), the local s-mix and
// the streaming copy.
#include <algorithm>
#include <cstdlib>

#include "hop_tile.h"

namespace dwf {

template <class S, int KK, int TAG = 0, int PM = 1, int EK = -1>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(hop_waves_per_eu<S, PM>())))
void hop_mfma_kernel(HopParams P) {
    extern __shared__ u32x4 hop_smem[];
    hop_tile<S, KK, PM, EK>(P, xcd_block(blockIdx.x, gridDim.x), blockIdx.y,
                    P.partial ? P.partial + (long)blockIdx.y * gridDim.x + blockIdx.x : nullptr,
                    reinterpret_cast<unsigned char*>(hop_smem));
}

// ---------------------------------------------------------------------
// Local dense s-mix on one half field: out = A . in (per chirality),
// same lane layout and MFMA use as the hop epilogue.  Optional reduction.
// ---------------------------------------------------------------------
template <class S, int KK>
__global__ __launch_bounds__(256) void mix_mfma_kernel(MixParams P) {
    using R = typename Traits<S>::R;
    using V = typename Vec4<R>::T;
    const int lane = threadIdx.x & 63;
    const int j = lane & 15, sc = lane >> 4;
    const long Vh = P.Vh;
    const int Ls = P.Ls;
    const long site = ((long)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6)) * 16 + j;
    const bool valid = site < Vh;
    const long sx = valid ? site : Vh - 1;
    const long rows = (long)Ls * 12, roff = (long)blockIdx.y * rows * P.Vhp;
    const R* A = static_cast<const R*>(P.mat);
    R a[2][KK];
#pragma unroll
    for (int chi = 0; chi < 2; ++chi)
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) a[chi][kk] = A[(chi * 16 + j) * 16 + 4 * kk + sc];
    double nrm = 0.0;
#pragma unroll
    for (int cp = 0; cp < 12; ++cp) {
        const int chi = cp / 6;
        V cr = {0, 0, 0, 0}, ci = {0, 0, 0, 0};
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            const int s = sc + 4 * kk;
            R xr = 0, xi = 0;
            if (s < Ls) cload<S>(P.in, roff + fidx((long)s * 12 + cp, sx, rows, fpack<S>()), xr, xi);
            cr = mfma4(a[chi][kk], xr, cr);
            ci = mfma4(a[chi][kk], xi, ci);
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int s = out_row<R>(sc, i);
            if (valid && s < Ls) {
                cstore<S>(P.out, roff + fidx((long)s * 12 + cp, site, rows, fpack<S>()), cr[i], ci[i]);
                nrm += double(cr[i]) * double(cr[i]) + double(ci[i]) * double(ci[i]);
            }
        }
    }
    if (P.partial) {
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) nrm += __shfl_xor(nrm, off, 64);
        __shared__ double red[4];
        if (lane == 0) red[threadIdx.x >> 6] = nrm;
        __syncthreads();
        if (threadIdx.x == 0) {
            double t = 0.0;
            for (int w = 0; w < (int)(blockDim.x >> 6); ++w) t += red[w];
            P.partial[(long)blockIdx.y * gridDim.x + blockIdx.x] = t;
        }
    }
}

// ---------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------
int hop_grid_blocks(long Vh) { return (int)((Vh + 15) / 16); }
int mix_grid_blocks(long Vh) { return (int)((Vh + 63) / 64); }

// Minimum shared memory per hop block ($DWF_HOP_MIN_LDS bytes, default 0):
// a larger request caps the blocks resident per CU (160 KB of LDS each),
// i.e. the sites an XCD has in flight, without changing the code.
static unsigned hop_min_lds() {
    static const unsigned v = [] {
        const char* e = std::getenv("DWF_HOP_MIN_LDS");
        const long x = e ? std::atol(e) : 0;
        return (unsigned)std::min<long>(std::max<long>(x, 0), 160 * 1024);
    }();
    return v;
}

template <class S, int TAG, int PM, int EK>
static void launch_hop_ek(const HopParams& P, int nrhs, hipStream_t st) {
    const int KK = (P.Ls + 3) / 4;
    DWF_REQUIRE(!P.sum || (EK == EK_UPDS && KK > 1), DWF_EINVAL, "this form of the hop reads alpha");
    dim3 grid(hop_grid_blocks(P.Vh), nrhs), block(64 * hop_waves(KK, sizeof(S) == 8));
    const unsigned smem_b = std::max(hop_smem_bytes<S>(KK, P.loc != nullptr), hop_min_lds());
    switch (KK) {
        // Ls <= 4: the generic kernel (the specialised chained stage spills there)
        case 1: hipLaunchKernelGGL((hop_mfma_kernel<S, 1, TAG, PM, -1>), grid, block, smem_b, st, P); break;
        case 2: hipLaunchKernelGGL((hop_mfma_kernel<S, 2, TAG, PM, EK>), grid, block, smem_b, st, P); break;
        case 3: hipLaunchKernelGGL((hop_mfma_kernel<S, 3, TAG, PM, EK>), grid, block, smem_b, st, P); break;
        case 4: hipLaunchKernelGGL((hop_mfma_kernel<S, 4, TAG, PM, EK>), grid, block, smem_b, st, P); break;
        default: throw Error{DWF_EDIMS, "Ls > 16 not supported by the fused hop"};
    }
    DWF_HIP(hipGetLastError());
}

// Epilogue kinds compiled per pre-mix mode: those of the operators' launches
// (a pre-mixing hop is plain or has a dense local term; FP64 pre-mixing hops
// keep the generic form); the stand-alone benchmark instance only as the plain
// mode-1 hop it times.
template <class S, int TAG, int PM>
static void launch_hop_pm(const HopParams& P, int nrhs, hipStream_t st) {
    const int ek = epilogue_kind(P);
    if constexpr (sizeof(S) == 8 && TAG == 0)
        if (launch_hop_few(P, nrhs, ek, st)) return;
    if constexpr ((TAG == 1 && PM != 1) || (sizeof(S) == 8 && PM != 0)) {
        // (FP64 pre-mixing hops: the specialised plain form spills one value)
        launch_hop_ek<S, TAG, PM, -1>(P, nrhs, st);
    } else if constexpr (TAG == 1) {
        if (ek == EK_PLAIN) launch_hop_ek<S, TAG, PM, EK_PLAIN>(P, nrhs, st);
        else launch_hop_ek<S, TAG, PM, -1>(P, nrhs, st);
    } else if constexpr (PM != 0) {
        switch (ek) {
            case EK_PLAIN: launch_hop_ek<S, TAG, PM, EK_PLAIN>(P, nrhs, st); break;
            case EK_LOCD: launch_hop_ek<S, TAG, PM, EK_LOCD>(P, nrhs, st); break;
            default: launch_hop_ek<S, TAG, PM, -1>(P, nrhs, st); break;
        }
    } else {
        switch (ek) {
            case EK_PLAIN: launch_hop_ek<S, TAG, PM, EK_PLAIN>(P, nrhs, st); break;
            case EK_CHAIN: launch_hop_ek<S, TAG, PM, EK_CHAIN>(P, nrhs, st); break;
            case EK_UPD: launch_hop_ek<S, TAG, PM, EK_UPD>(P, nrhs, st); break;
            case EK_UPDS: launch_hop_ek<S, TAG, PM, EK_UPDS>(P, nrhs, st); break;
            case EK_LOCD: launch_hop_ek<S, TAG, PM, EK_LOCD>(P, nrhs, st); break;
            case EK_LOCI: launch_hop_ek<S, TAG, PM, EK_LOCI>(P, nrhs, st); break;
            case EK_CHAINN: launch_hop_ek<S, TAG, PM, EK_CHAINN>(P, nrhs, st); break;
            default: launch_hop_ek<S, TAG, PM, -1>(P, nrhs, st); break;
        }
    }
}

template <class S, int TAG>
static void launch_hop_t(const HopParams& P, int nrhs, hipStream_t st) {
    switch (P.pre_mode) {
        case 0: launch_hop_pm<S, TAG, 0>(P, nrhs, st); break;
        case 1: launch_hop_pm<S, TAG, 1>(P, nrhs, st); break;
        case 2: launch_hop_pm<S, TAG, 2>(P, nrhs, st); break;
        default: throw Error{DWF_EINVAL, "bad pre-mix mode"};
    }
}

void launch_hop(int kind, const HopParams& P, int nrhs, hipStream_t st, int bench_tag) {
    switch (kind) {
        case ST_F64:
            if (bench_tag) launch_hop_t<double, 1>(P, nrhs, st); else launch_hop_t<double, 0>(P, nrhs, st);
            break;
        case ST_F32:
            if (bench_tag) launch_hop_t<float, 1>(P, nrhs, st); else launch_hop_t<float, 0>(P, nrhs, st);
            break;
        case ST_BF16:
            if (bench_tag) launch_hop_t<bf16s, 1>(P, nrhs, st); else launch_hop_t<bf16s, 0>(P, nrhs, st);
            break;
        default: throw Error{DWF_EINVAL, "bad storage kind"};
    }
}

// Plain streaming copy (16-byte vectors), used to calibrate memory counters
// and as the measured streaming ceiling: every lane moves four 16-byte
// vectors whose loads are all issued before the first store, one block per
// 4 x 256 vectors (no grid-stride loop), the form that kept the most bytes
// in flight in a sweep of vectors per lane and block counts.
constexpr int COPY_VPL = 4;
__global__ __launch_bounds__(256) void copy_kernel(float4* __restrict__ dst, const float4* __restrict__ src, long n) {
    const long base = (long)blockIdx.x * (256 * COPY_VPL) + threadIdx.x;
    float4 v[COPY_VPL];
#pragma unroll
    for (int k = 0; k < COPY_VPL; ++k) {
        const long i = base + (long)k * 256;
        if (i < n) v[k] = src[i];
    }
#pragma unroll
    for (int k = 0; k < COPY_VPL; ++k) {
        const long i = base + (long)k * 256;
        if (i < n) dst[i] = v[k];
    }
}

void launch_copy(void* dst, const void* src, size_t bytes, hipStream_t st) {
    const long n = (long)(bytes / 16);
    const long blocks = (n + 256 * COPY_VPL - 1) / (256 * COPY_VPL);
    DWF_REQUIRE(blocks < (1L << 31), DWF_EINVAL, "copy too large");
    if (blocks == 0) return;
    hipLaunchKernelGGL(copy_kernel, dim3((unsigned)blocks), dim3(256), 0, st, (float4*)dst, (const float4*)src, n);
    DWF_HIP(hipGetLastError());
}

template <class S>
static void launch_mix_t(const MixParams& P, int nrhs, hipStream_t st) {
    dim3 grid(mix_grid_blocks(P.Vh), nrhs), block(256);
    const int KK = (P.Ls + 3) / 4;
    switch (KK) {
        case 1: hipLaunchKernelGGL((mix_mfma_kernel<S, 1>), grid, block, 0, st, P); break;
        case 2: hipLaunchKernelGGL((mix_mfma_kernel<S, 2>), grid, block, 0, st, P); break;
        case 3: hipLaunchKernelGGL((mix_mfma_kernel<S, 3>), grid, block, 0, st, P); break;
        case 4: hipLaunchKernelGGL((mix_mfma_kernel<S, 4>), grid, block, 0, st, P); break;
        default: throw Error{DWF_EDIMS, "Ls > 16 not supported"};
    }
    DWF_HIP(hipGetLastError());
}

void launch_mix(int kind, const MixParams& P, int nrhs, hipStream_t st) {
    switch (kind) {
        case ST_F64: launch_mix_t<double>(P, nrhs, st); break;
        case ST_F32: launch_mix_t<float>(P, nrhs, st); break;
        case ST_BF16: launch_mix_t<bf16s>(P, nrhs, st); break;
        default: throw Error{DWF_EINVAL, "bad storage kind"};
    }
}

}  // namespace dwf

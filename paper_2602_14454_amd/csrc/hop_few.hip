// FP64 launches of the fused hop (hop_tile.h) on small lattices.
#include "hop_tile.h"

namespace dwf {

// With so few blocks that every wave has a SIMD to itself, a launch is a chain
// of latencies: pre-mix and s-mix coefficients, links, eight directions, local
// term, old residual, one after the other in the form that several waves per
// SIMD want (3 waves, rolled direction loop).  Here everything that does not
// depend on another load is requested before the direction loop, and the
// spinors of four directions (two with the general pre-mix) are in flight, in
// 256 VGPRs and about 100 AGPRs.  FP64 only: FP32 and BF16 pipeline the
// directions already and gained nothing from a deeper one.
template <int KK, int PM, int EK>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void hop_few_kernel(HopParams P) {
    extern __shared__ u32x4 hop_smem[];
    hop_tile<double, KK, PM, EK, true>(P, blockIdx.x, blockIdx.y,
                                       P.partial ? P.partial + (long)blockIdx.y * gridDim.x + blockIdx.x : nullptr,
                                       reinterpret_cast<unsigned char*>(hop_smem));
}

// Waves of a launch up to which this form is used: three quarters of the 1024
// SIMDs.  Normal operator with layout conversion, general form / this one: 16
// waves (4^4, Ls = 8) 52.6 / 39.6 us, 256 (8^4, Ls = 8) 59.9 / 46.6, 512 (8^4,
// Ls = 16) 63.2 / 55.5, 768 (8^3x16, Ls = 12, c != 0) 67.1 / 64.4, 1024 (8^3x16,
// Ls = 16) 70.6 / 74.9, 2048 (8^2x16^2, Ls = 16) 125.4 / 128.5.
#ifndef DWF_HOP_FEW_WAVES
#define DWF_HOP_FEW_WAVES 768
#endif

template <int PM, int EK>
static bool launch_few(const HopParams& P, int nrhs, hipStream_t st) {
    const int KK = (P.Ls + 3) / 4;
    dim3 grid(hop_grid_blocks(P.Vh), nrhs), block(64 * hop_waves(KK, true));
    const unsigned smem_b = hop_smem_bytes<double>(KK, P.loc != nullptr);
    switch (KK) {
        case 1: hipLaunchKernelGGL((hop_few_kernel<1, PM, EK>), grid, block, smem_b, st, P); break;
        case 2: hipLaunchKernelGGL((hop_few_kernel<2, PM, EK>), grid, block, smem_b, st, P); break;
        case 3: hipLaunchKernelGGL((hop_few_kernel<3, PM, EK>), grid, block, smem_b, st, P); break;
        case 4: hipLaunchKernelGGL((hop_few_kernel<4, PM, EK>), grid, block, smem_b, st, P); break;
        default: return false;
    }
    DWF_HIP(hipGetLastError());
    return true;
}

bool launch_hop_few(const HopParams& P, int nrhs, int ek, hipStream_t st) {
    if ((long)hop_grid_blocks(P.Vh) * nrhs * hop_waves((P.Ls + 3) / 4, true) > DWF_HOP_FEW_WAVES) return false;
    switch (P.pre_mode * 8 + ek) {
        case EK_PLAIN: return launch_few<0, EK_PLAIN>(P, nrhs, st);
        case EK_CHAIN: return launch_few<0, EK_CHAIN>(P, nrhs, st);
        case EK_UPD: return launch_few<0, EK_UPD>(P, nrhs, st);
        case EK_UPDS: return launch_few<0, EK_UPDS>(P, nrhs, st);
        case EK_LOCD: return launch_few<0, EK_LOCD>(P, nrhs, st);
        case EK_LOCI: return launch_few<0, EK_LOCI>(P, nrhs, st);
        case EK_CHAINN: return launch_few<0, EK_CHAINN>(P, nrhs, st);
        case 8 + EK_PLAIN: return launch_few<1, EK_PLAIN>(P, nrhs, st);
        case 8 + EK_LOCD: return launch_few<1, EK_LOCD>(P, nrhs, st);
        case 16 + EK_PLAIN: return launch_few<2, EK_PLAIN>(P, nrhs, st);
        case 16 + EK_LOCD: return launch_few<2, EK_LOCD>(P, nrhs, st);
        default: return false;
    }
}

}  // namespace dwf

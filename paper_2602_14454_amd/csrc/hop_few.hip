// FP64 launches of the fused hop (hop_tile.h) on small lattices.
#include "hop_tile.h"

namespace dwf {

// With so few blocks that every wave has a SIMD to itself, a launch is a chain
// of latencies: pre-mix and s-mix coefficients, links, eight directions, local
// term, old residual, one after the other in the form that several waves per
// SIMD want (3 waves, rolled direction loop).  Here everything that does not
// depend on another load is requested before the direction loop, and the
// spinors of four directions (two with the general pre-mix, or when four waves
// share them) are in flight, in 256 VGPRs and about 100 AGPRs.  FP64 only: FP32 and BF16 pipeline the
// directions already and gained nothing from a deeper one.
template <int KK, int PM, int EK, int DS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(1, 1))) void hop_few_kernel(HopParams P) {
    extern __shared__ u32x4 hop_smem[];
    hop_tile<double, KK, PM, EK, true, DS>(P, blockIdx.x, blockIdx.y,
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

// Blocks up to which the one or two waves of a block (Ls <= 8) become four, one
// per SIMD of its CU, by sharing out the eight directions (DS): one block per CU,
// since two blocks of such waves do not fit one.  Three or four waves (Ls > 8)
// have no free SIMD.  Normal operator with layout conversion, before / after: 4^4,
// Ls = 8 (8 blocks) 55.2 / 50.1 us, 8^4, Ls = 8 (128) 61.7 / 58.6, 8^3x16, Ls = 8
// (256) 67.0 / 64.5; Ls = 4: 2^4 53.5 / 38.6, 8^4 60.8 / 47.4, 8^3x16 64.7 / 51.3.
#ifndef DWF_HOP_SPLIT_BLOCKS
#define DWF_HOP_SPLIT_BLOCKS 256
#endif

template <int KK, int PM, int EK, int DS>
static void launch_few_kk(const HopParams& P, int nrhs, hipStream_t st) {
    const dim3 grid(hop_grid_blocks(P.Vh), nrhs), block(64 * hop_waves(KK, true) * DS);
    const unsigned smem_b = HopSmem<double, KK, DS>::bytes(P.loc != nullptr);
    hipLaunchKernelGGL((hop_few_kernel<KK, PM, EK, DS>), grid, block, smem_b, st, P);
}

template <int PM, int EK>
static bool launch_few(const HopParams& P, int nrhs, hipStream_t st) {
    const bool split = (long)hop_grid_blocks(P.Vh) * nrhs <= DWF_HOP_SPLIT_BLOCKS;
    switch ((P.Ls + 3) / 4) {
        case 1:
            if constexpr (EK == EK_UPDS) return false;   // Ls <= 4: cg_few has no such launch
            else if (split) launch_few_kk<1, PM, EK, 4>(P, nrhs, st);
            else launch_few_kk<1, PM, EK, 1>(P, nrhs, st);
            break;
        case 2:
            if (split) launch_few_kk<2, PM, EK, 2>(P, nrhs, st);
            else launch_few_kk<2, PM, EK, 1>(P, nrhs, st);
            break;
        case 3: launch_few_kk<3, PM, EK, 1>(P, nrhs, st); break;
        case 4: launch_few_kk<4, PM, EK, 1>(P, nrhs, st); break;
        default: return false;
    }
    DWF_HIP(hipGetLastError());
    return true;
}

// Forms compiled per pre-mix mode: the operators' launches have no others.  Any
// other pair, ek = -1 (no compiled epilogue) among them, takes the general form.
template <int PM>
static bool launch_few_pm(const HopParams& P, int nrhs, int ek, hipStream_t st) {
    switch (ek) {
        case EK_PLAIN: return launch_few<PM, EK_PLAIN>(P, nrhs, st);
        case EK_LOCD: return launch_few<PM, EK_LOCD>(P, nrhs, st);
        default: break;
    }
    if constexpr (PM == 0) {
        switch (ek) {
            case EK_CHAIN: return launch_few<0, EK_CHAIN>(P, nrhs, st);
            case EK_UPD: return launch_few<0, EK_UPD>(P, nrhs, st);
            case EK_UPDS: return launch_few<0, EK_UPDS>(P, nrhs, st);
            case EK_LOCI: return launch_few<0, EK_LOCI>(P, nrhs, st);
            case EK_CHAINN: return launch_few<0, EK_CHAINN>(P, nrhs, st);
            default: break;
        }
    }
    return false;
}

bool launch_hop_few(const HopParams& P, int nrhs, int ek, hipStream_t st) {
    if ((long)hop_grid_blocks(P.Vh) * nrhs * hop_waves((P.Ls + 3) / 4, true) > DWF_HOP_FEW_WAVES) return false;
    switch (P.pre_mode) {
        case 0: return launch_few_pm<0>(P, nrhs, ek, st);
        case 1: return launch_few_pm<1>(P, nrhs, ek, st);
        case 2: return launch_few_pm<2>(P, nrhs, ek, st);
        default: return false;
    }
}

}  // namespace dwf

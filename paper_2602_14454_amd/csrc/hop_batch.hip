// Work-list launches of the fused hop (hop_tile.h) for batched solves.
#include "hop_tile.h"

namespace dwf {

// Work-list form for batches: one launch covers several operators (lattices
// of any size with the same ceil(Ls/4)) and all their right-hand sides.
// meta[0..n] is the prefix sum of the blocks of each item, meta[n+1+i] its
// number of right-hand sides.  Item i takes ceil(nrhs/nrb) x tiles blocks;
// a block computes one tile for nrb consecutive right-hand sides, so the
// tile's links and neighbour indices are fetched from HBM once and re-read
// from cache for the others.  order 0 sweeps tiles fastest (neighbour reuse
// across tiles of one RHS), order 1 sweeps RHS chunks fastest (link reuse
// across chunks).  A right-hand side whose done flag is set is skipped
// (its partial is written as 0).
// PM as in hop_batch1_kernel below (the same arithmetic path, so that every
// schedule gives the same bits).
template <class S, int KK, int PM>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(sizeof(S) == 8 ? DWF_HOP_WAVES_PER_EU64_BATCH : DWF_HOP_BATCHN_WPE)))
void hop_batch_kernel(const HopParams* __restrict__ items, const int* __restrict__ meta, int nitems, int nrb,
                      int order) {
    extern __shared__ u32x4 hop_smem[];
    const int b = xcd_block(blockIdx.x, gridDim.x);
    int i = 0;
    while (i + 1 < nitems && b >= meta[i + 1]) ++i;
    const HopParams& P = items[i];   // read in place (wave-uniform address: scalar loads)
    const int nrhs = meta[nitems + 1 + i];
    const long tiles = (P.Vh + 15) / 16;
    const int chunks = (nrhs + nrb - 1) / nrb;
    const long local = b - meta[i];
    const long tile = order == 0 ? local % tiles : local / chunks;
    const int chunk = order == 0 ? (int)(local / tiles) : (int)(local % chunks);
    for (int q = 0; q < nrb; ++q) {
        const int r = chunk * nrb + q;
        if (r >= nrhs) break;
        double* part = P.partial ? P.partial + (long)r * P.pstride + tile : nullptr;
        if (P.done && P.done[(long)r * P.done_stride] != 0.0) {
            if (part && threadIdx.x == 0) *part = 0.0;
            continue;
        }
        hop_tile<S, KK, PM>(P, tile, r, part, reinterpret_cast<unsigned char*>(hop_smem));
        __syncthreads();   // shared memory is reused by the next right-hand side
    }
}

// The same work list with one right-hand side per block (nrb = 1): no loop
// around the tile, so nothing is live across right-hand sides.
#ifndef DWF_HOP_BATCH1_WPE
#define DWF_HOP_BATCH1_WPE 5
#endif
// PM >= 0: every item of the launch has that pre-mix mode (compiled in, with
// the single-lattice kernel's pipelined direction loop and occupancy);
// PM = -1: mixed modes, read per item.
template <class S, int PM>
constexpr int hop_batch1_waves_per_eu() {
    if (PM >= 0) return hop_waves_per_eu<S, PM>();
    return sizeof(S) == 8 ? DWF_HOP_WAVES_PER_EU64_BATCH : DWF_HOP_BATCH1_WPE;
}

template <class S, int KK, int PM, int EK = -1>
__global__ __launch_bounds__(256)
__attribute__((amdgpu_waves_per_eu(hop_batch1_waves_per_eu<S, PM>())))
void hop_batch1_kernel(const HopParams* __restrict__ items, const int* __restrict__ meta, int nitems, int order) {
    extern __shared__ u32x4 hop_smem[];
    const int b = xcd_block(blockIdx.x, gridDim.x);
    int i = 0;
    while (i + 1 < nitems && b >= meta[i + 1]) ++i;
    const HopParams& P = items[i];   // read in place (wave-uniform address: scalar loads)
    const int nrhs = meta[nitems + 1 + i];
    const int tiles = (int)((P.Vh + 15) / 16);
    int tile = b - meta[i], r = 0;
    if (order == 0) {
        // tiles fastest: a uniform subtraction loop (nrhs steps at most)
        // keeps tile and r in scalar registers, where a division would be
        // expanded on the vector unit
        while (tile >= tiles) { tile -= tiles; ++r; }
    } else {
        r = tile % nrhs;
        tile /= nrhs;
    }
    double* part = P.partial ? P.partial + (long)r * P.pstride + tile : nullptr;
    if (P.done && P.done[(long)r * P.done_stride] != 0.0) {
        if (part && threadIdx.x == 0) *part = 0.0;
        return;
    }
    hop_tile<S, KK, PM, EK>(P, tile, r, part, reinterpret_cast<unsigned char*>(hop_smem));
}

// The work list with NR right-hand sides per block sharing the tile's
// staged links and neighbour indices: group r of the block's NR groups of
// hop_waves(KK) waves computes right-hand side chunk * NR + r of the tile in
// its own shared-memory region (`region` bytes each).  Block -> (tile,
// chunk) as in hop_batch1_kernel with chunks of NR right-hand sides.
template <class S, int KK, int PM, int NR>
__global__ __launch_bounds__(1024)
__attribute__((amdgpu_waves_per_eu(hop_batch1_waves_per_eu<S, PM>())))
void hop_multi_kernel(const HopParams* __restrict__ items, const int* __restrict__ meta, int nitems, int order,
                      unsigned region) {
    extern __shared__ u32x4 hop_smem[];
    const int b = xcd_block(blockIdx.x, gridDim.x);
    int i = 0;
    while (i + 1 < nitems && b >= meta[i + 1]) ++i;
    const HopParams& P = items[i];
    const int nrhs = meta[nitems + 1 + i];
    const int tiles = (int)((P.Vh + 15) / 16);
    const int chunks = (nrhs + NR - 1) / NR;
    int tile = b - meta[i], chunk = 0;
    if (order == 0) {
        while (tile >= tiles) { tile -= tiles; ++chunk; }
    } else {
        chunk = tile % chunks;
        tile /= chunks;
    }
    const int sub = (int)threadIdx.x / (64 * hop_waves(KK, sizeof(S) == 8));   // wave-uniform
    const int r = chunk * NR + sub;
    const bool in_range = r < nrhs;
    const int rr = in_range ? r : nrhs - 1;   // scalar reads of an out-of-range group stay in bounds
    const bool active = in_range && !(P.done && P.done[(long)rr * P.done_stride] != 0.0);
    // a converged right-hand side writes a zero partial (its loads read zeros)
    double* part = (P.partial && in_range) ? P.partial + (long)rr * P.pstride + tile : nullptr;
    hop_tile<S, KK, PM>(P, tile, rr, part, reinterpret_cast<unsigned char*>(hop_smem), sub, region, active);
}

// ---------------------------------------------------------------------
// launchers
// ---------------------------------------------------------------------
template <class S, int PM, int EK>
static void launch_hop_batch1_ek(int KK, dim3 grid, dim3 block, unsigned smem_b, const HopParams* items,
                                 const int* meta, int nitems, int order, hipStream_t st) {
    switch (KK) {
        // Ls <= 4: the generic kernel, as for single lattices
        case 1: hipLaunchKernelGGL((hop_batch1_kernel<S, 1, PM, -1>), grid, block, smem_b, st, items, meta, nitems, order); break;
        case 2: hipLaunchKernelGGL((hop_batch1_kernel<S, 2, PM, EK>), grid, block, smem_b, st, items, meta, nitems, order); break;
        case 3: hipLaunchKernelGGL((hop_batch1_kernel<S, 3, PM, EK>), grid, block, smem_b, st, items, meta, nitems, order); break;
        case 4: hipLaunchKernelGGL((hop_batch1_kernel<S, 4, PM, EK>), grid, block, smem_b, st, items, meta, nitems, order); break;
        default: throw Error{DWF_EDIMS, "Ls > 16 not supported by the fused hop"};
    }
}

// ek: the items' common epilogue kind (-1: mixed or none), compiled in on
// the same terms as for single-lattice launches
template <class S, int PM>
static void launch_hop_batch1_pm(int KK, dim3 grid, dim3 block, unsigned smem_b, const HopParams* items,
                                 const int* meta, int nitems, int order, int ek, hipStream_t st) {
    if constexpr (PM < 0 || (sizeof(S) == 8 && PM != 0)) {
        launch_hop_batch1_ek<S, PM, -1>(KK, grid, block, smem_b, items, meta, nitems, order, st);
    } else if constexpr (PM != 0) {
        if (ek == EK_PLAIN) launch_hop_batch1_ek<S, PM, EK_PLAIN>(KK, grid, block, smem_b, items, meta, nitems, order, st);
        else launch_hop_batch1_ek<S, PM, -1>(KK, grid, block, smem_b, items, meta, nitems, order, st);
    } else {
        switch (ek) {
            case EK_PLAIN: launch_hop_batch1_ek<S, PM, EK_PLAIN>(KK, grid, block, smem_b, items, meta, nitems, order, st); break;
            case EK_CHAIN: launch_hop_batch1_ek<S, PM, EK_CHAIN>(KK, grid, block, smem_b, items, meta, nitems, order, st); break;
            case EK_UPD: launch_hop_batch1_ek<S, PM, EK_UPD>(KK, grid, block, smem_b, items, meta, nitems, order, st); break;
            default: launch_hop_batch1_ek<S, PM, -1>(KK, grid, block, smem_b, items, meta, nitems, order, st); break;
        }
    }
}

template <class S, int PM>
static void launch_hop_batchn_pm(int KK, dim3 grid, dim3 block, unsigned smem_b, const HopParams* items,
                                 const int* meta, int nitems, int nrb, int order, hipStream_t st) {
    switch (KK) {
        case 1: hipLaunchKernelGGL((hop_batch_kernel<S, 1, PM>), grid, block, smem_b, st, items, meta, nitems, nrb, order); break;
        case 2: hipLaunchKernelGGL((hop_batch_kernel<S, 2, PM>), grid, block, smem_b, st, items, meta, nitems, nrb, order); break;
        case 3: hipLaunchKernelGGL((hop_batch_kernel<S, 3, PM>), grid, block, smem_b, st, items, meta, nitems, nrb, order); break;
        case 4: hipLaunchKernelGGL((hop_batch_kernel<S, 4, PM>), grid, block, smem_b, st, items, meta, nitems, nrb, order); break;
        default: throw Error{DWF_EDIMS, "Ls > 16 not supported by the fused hop"};
    }
}

template <class S, int PM, int NR>
static void launch_hop_multi_pm(int KK, dim3 grid, unsigned region, const HopParams* items, const int* meta,
                                int nitems, int order, hipStream_t st) {
    const dim3 block(64 * hop_waves(KK, sizeof(S) == 8) * NR);
    const unsigned smem_b = region * NR;
    switch (KK) {
        case 1: hipLaunchKernelGGL((hop_multi_kernel<S, 1, PM, NR>), grid, block, smem_b, st, items, meta, nitems, order, region); break;
        case 2: hipLaunchKernelGGL((hop_multi_kernel<S, 2, PM, NR>), grid, block, smem_b, st, items, meta, nitems, order, region); break;
        case 3: hipLaunchKernelGGL((hop_multi_kernel<S, 3, PM, NR>), grid, block, smem_b, st, items, meta, nitems, order, region); break;
        case 4: hipLaunchKernelGGL((hop_multi_kernel<S, 4, PM, NR>), grid, block, smem_b, st, items, meta, nitems, order, region); break;
        default: throw Error{DWF_EDIMS, "Ls > 16 not supported by the fused hop"};
    }
}

// shared-link kernel for FP32 with 2 or 4 right-hand sides per block when
// the block (<= 1024 threads) and its shared memory fit; false otherwise
template <class S>
static bool launch_hop_multi(int KK, int blocks, int nrb, int order, bool loc, int pm, const HopParams* items,
                             const int* meta, int nitems, hipStream_t st) {
    if constexpr (!std::is_same<S, float>::value) {
        return false;
    } else {
        if (nrb != 2 && nrb != 4) return false;
        if (64 * hop_waves(KK, false) * nrb > 1024) return false;
        static const int max_lds = [] {
            int dev = 0, v = 65536;
            if (hipGetDevice(&dev) == hipSuccess &&
                hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess)
                v = 65536;
            return v;
        }();
        const unsigned region = (hop_smem_bytes<S>(KK, loc) + 15u) & ~15u;
        if ((long)region * nrb > (long)max_lds) return false;
        const dim3 grid(blocks);
#define DWF_MULTI(PMV)                                                                                   \
    (nrb == 2 ? launch_hop_multi_pm<S, PMV, 2>(KK, grid, region, items, meta, nitems, order, st)        \
              : launch_hop_multi_pm<S, PMV, 4>(KK, grid, region, items, meta, nitems, order, st))
        switch (pm) {
            case 0: DWF_MULTI(0); break;
            case 1: DWF_MULTI(1); break;
            case 2: DWF_MULTI(2); break;
            default: DWF_MULTI(-1); break;
        }
#undef DWF_MULTI
        DWF_HIP(hipGetLastError());
        return true;
    }
}

template <class S>
static void launch_hop_batch_t(int KK, const HopParams* items, const int* meta, int nitems, int blocks, int nrb,
                               int order, bool loc, int pm, int ek, hipStream_t st) {
    if (launch_hop_multi<S>(KK, blocks, nrb, order, loc, pm, items, meta, nitems, st)) return;
    dim3 grid(blocks), block(64 * hop_waves(KK, sizeof(S) == 8));
    const unsigned smem_b = hop_smem_bytes<S>(KK, loc);
    if (nrb == 1) {
        switch (pm) {
            case 0: launch_hop_batch1_pm<S, 0>(KK, grid, block, smem_b, items, meta, nitems, order, ek, st); break;
            case 1: launch_hop_batch1_pm<S, 1>(KK, grid, block, smem_b, items, meta, nitems, order, ek, st); break;
            case 2: launch_hop_batch1_pm<S, 2>(KK, grid, block, smem_b, items, meta, nitems, order, ek, st); break;
            default: launch_hop_batch1_pm<S, -1>(KK, grid, block, smem_b, items, meta, nitems, order, ek, st); break;
        }
        DWF_HIP(hipGetLastError());
        return;
    }
    switch (pm) {
        case 0: launch_hop_batchn_pm<S, 0>(KK, grid, block, smem_b, items, meta, nitems, nrb, order, st); break;
        case 1: launch_hop_batchn_pm<S, 1>(KK, grid, block, smem_b, items, meta, nitems, nrb, order, st); break;
        case 2: launch_hop_batchn_pm<S, 2>(KK, grid, block, smem_b, items, meta, nitems, nrb, order, st); break;
        default: launch_hop_batchn_pm<S, -1>(KK, grid, block, smem_b, items, meta, nitems, nrb, order, st); break;
    }
    DWF_HIP(hipGetLastError());
}

int hop_epilogue_kind(const HopParams& P) { return epilogue_kind(P); }

void launch_hop_batch(int kind, int KK, const HopParams* items, const int* meta, int nitems, int blocks, int nrb,
                      int order, bool has_loc, int pm, int ek, hipStream_t st) {
    if (blocks <= 0) return;
    switch (kind) {
        case ST_F64: launch_hop_batch_t<double>(KK, items, meta, nitems, blocks, nrb, order, has_loc, pm, ek, st); break;
        case ST_F32: launch_hop_batch_t<float>(KK, items, meta, nitems, blocks, nrb, order, has_loc, pm, ek, st); break;
        case ST_BF16: launch_hop_batch_t<bf16s>(KK, items, meta, nitems, blocks, nrb, order, has_loc, pm, ek, st); break;
        default: throw Error{DWF_EINVAL, "bad storage kind"};
    }
}

}  // namespace dwf

// Launch interface of the parallel-transport convolution kernels (ptc_kernels.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace dwf {

// One layer (one channel to one) for the sites of one parity; see ptc_kernels.hip.
struct PtcLayerParams {
    const float2* in_loc;   // field on the output parity (paths 0, +s, -s), or nullptr
    const float2* in_hop;   // field on the other parity (the 8 link paths), or nullptr
    float2* out;            // field on the output parity
    const float2* W;        // [11][4][4] complex
    const float2* links;    // FP32 hop links of the output parity
    const int* nbr;         // neighbour table of the output parity
    long Vh, Vhp;
    int Ls;
};

void ptc_layer(const PtcLayerParams& P, hipStream_t st);
// Both layers as one sum over pairs of paths (see ptc_kernels.hip): FP32 even
// half fields in and out.
struct PtcPairParams {
    const float2 *W1, *W2;       // [11][H][4][4] each
    const float2* links[2];      // FP32 hop links and neighbour table by output parity
    const int* nbr[2];
    long Vh, Vhp;
    int Ls, H;
    float2* mid;                 // 8 half fields
    float* el;                   // 4096 floats: pair weights of the links
    float2* al;                  // 2 * 8 * 16: pair weights of the local paths and their rounding
};
void ptc_pairs_forward(const PtcPairParams& P, const float2* r, float2* out, hipStream_t st);
// dL/dW of both layers from r and g = dL/d(out); corr: ptc_corr_bytes of scratch
size_t ptc_corr_bytes(const PtcPairParams& P);
void ptc_pairs_gradient(const PtcPairParams& P, const float2* r, const float2* g, double* corr, float2* G1,
                        float2* G2, hipStream_t st);
int ptc_loss_blocks(long n);
// stats[0] = |y-e|^2/|e|^2, stats[1] = |e|^2, stats[2] = |y-e|^2; g = 2(y-e)/|e|^2 (if g)
void ptc_loss(const float2* y, const float2* e, long n, double* partial, double* stats, float2* g, hipStream_t st);
// d = y - e;  stats[0] = |u|^2/|r|^2, stats[1] = |r|^2, stats[2] = |u|^2;  g = 2 w / stats[1]
void ptc_sub(const float2* y, const float2* e, long n, float2* d, hipStream_t st);
void ptc_norms(const float2* u, const float2* r, long n, double* partial, double* stats, hipStream_t st);
void ptc_scale_grad(const float2* w, long n, const double* stats, float2* g, hipStream_t st);
void ptc_adam(float* w, const float* g, float* m, float* v, int n, float lr, float b1, float b2, float eps, int step,
              hipStream_t st);

}  // namespace dwf

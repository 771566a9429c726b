// Quenched gauge-field generation (gauge.hip).
#pragma once

#include <hip/hip_runtime.h>

namespace dwf {

// nsweeps times (one heatbath sweep keyed by seed and sweep0 + k, n_or
// over-relaxation sweeps) over every link of a canonical complex128 field
// U[lex][mu][3][3] (device), links re-projected onto SU(3) after every sweep.
// The field is rearranged in place while the work runs on the stream.
void gauge_sweeps(void* U, const int dims[4], double beta, int nsweeps, int n_or, unsigned long long seed,
                  long long sweep0, hipStream_t st);
// sum of Re tr U_P over sites and planes (FP64 reduction) in out_dev; partial: device scratch of
// gauge_plaquette_partials(dims) + 1 doubles
int gauge_plaquette_partials(const int dims[4]);
void gauge_plaquette(const void* U, const int dims[4], double* partial, double* out_dev, hipStream_t st);

}  // namespace dwf

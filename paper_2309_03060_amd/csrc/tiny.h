// Matrix-vector products of the smallest operators in one launch (host interface).
#pragma once
#include "common.h"

namespace cola {

struct TinyArgs {
    int32_t F, J;              // modes (2 or 3), terms
    int32_t dims[3];
    int32_t nrhs;
    const void* K[3];          // factor of mode m, term j at K[m] + j * dims[m]^2 elements
    const void* X;             // nrhs * n
    void* Y;                   // may be X
    const void* dvec;          // n or null
    double sigma2;
};

// Operators and right-hand sides that k_tiny_mvm takes (elements of `es` bytes).
bool tiny_mvm_supported(int F, int J, const int64_t* dims, int nrhs, int es);

// y = A x for every right-hand side; prec FP64 or FP32.
hipError_t launch_tiny_mvm(int prec, const TinyArgs& a, hipStream_t s);

}  // namespace cola

// Matrix-vector products of the smallest operators in one launch.
//
// An operator of a few thousand entries is all launches: one per mode (or one for two modes and one
// for the third), each of a few microseconds of which the products take a fraction.  Here one
// workgroup holds a right-hand side, the factors of every term and the intermediates in LDS and walks
// all modes, all terms of a mode together; the waves' FMAs suffice at this size.  A thread forms four
// outputs along the contracted mode at a time (one read of the vector and one of the transposed factor
// for four products, k upwards); what is left is the chain of one load from memory and one LDS loop
// and barrier per mode, which more threads do not shorten.
//
// 12 x 10 x 14, FP32, calls back to back: 1 right-hand side 10.2 -> 6.4 us (6.3 on the GPU), 64 16.0 -> 6.8,
// 512 70.8 -> 9.0; 8 x 8 x 8, four terms, FP64: 13.8 -> 7.1 us, 64 right-hand sides 60 -> 7.5 (two
// of these microseconds are the call's, which lost them by itself).
#include "tiny.h"

namespace cola {
namespace {

constexpr int kTinyThreads = 512;
constexpr int kTinyLds = 64 * 1024;

int64_t up4(int64_t v) { return (v + 3) / 4 * 4; }

// LDS elements: the vector, F - 1 intermediates of every term, the factors
int64_t tiny_elems(int F, int J, const int64_t* dims) {
    int64_t n = 1, k = 0;
    for (int m = 0; m < F; ++m) {
        n *= dims[m];
        k += dims[m] * up4(dims[m]);
    }
    return up4(n) + (F - 1) * up4(J * n) + J * k;
}

template <typename T, int F>
__global__ __launch_bounds__(kTinyThreads) void k_tiny_mvm(TinyArgs a) {
    typedef T V4 __attribute__((ext_vector_type(4)));
    constexpr int U = 4;                                     // loads in flight per operand
    extern __shared__ __attribute__((aligned(32))) char smem[];
    const uint32_t tid = threadIdx.x;
    uint32_t n = 1, off[F], most = 0;                        // off: of mode m's factors in kt, [term][k][row, padded]
    uint32_t at = 0;
#pragma unroll
    for (int m = 0; m < F; ++m) {
        const uint32_t nk = a.dims[m];
        n *= nk;
        off[m] = at;
        at += a.J * nk * ((nk + 3) & ~3u);
        most = a.J * nk * nk > most ? a.J * nk * nk : most;
    }
    most = n > most ? n : most;
    T* const xs = (T*)smem;
    T* const buf = xs + ((n + 3) & ~3u);
    const uint32_t bn = (a.J * n + 3) & ~3u;
    T* const kt = buf + (F - 1) * bn;
    const T* X = (const T*)a.X + (int64_t)blockIdx.x * n;
    T* Y = (T*)a.Y + (int64_t)blockIdx.x * n;
    for (uint32_t e0 = tid; e0 < most; e0 += U * kTinyThreads) {
        T x[U], k[F][U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t e = e0 + u * kTinyThreads;
            x[u] = X[e < n ? e : n - 1];
#pragma unroll
            for (int m = 0; m < F; ++m) {
                const uint32_t end = a.J * a.dims[m] * a.dims[m];
                k[m][u] = ((const T*)a.K[m])[e < end ? e : end - 1];
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint32_t e = e0 + u * kTinyThreads;
            if (e < n) xs[e] = x[u];
#pragma unroll
            for (int m = 0; m < F; ++m) {
                const uint32_t nk = a.dims[m], mp = (nk + 3) & ~3u;
                if (e < a.J * nk * nk) {
                    const uint32_t q = e / nk, l = e % nk, j = q / nk, i = q % nk;
                    kt[off[m] + (j * nk + l) * mp + i] = k[m][u];
                }
            }
        }
    }
    __syncthreads();

    // rows beyond a mode hold whatever LDS did: their products are not stored
    const T* in = xs;
    uint32_t trail = 1, in_term = 0;
#pragma unroll
    for (int m = F - 1; m >= 0; --m) {
        const uint32_t nk = a.dims[m], mp = (nk + 3) & ~3u, nb = mp / 4;
        const uint32_t groups = n / nk * nb, all = m > 0 ? groups * a.J : groups;
        T* const out = buf + (F - 1 - m) * bn;
        for (uint32_t e = tid; e < all; e += kTinyThreads) {
            const uint32_t j0 = e / groups, r = e % groups;
            const uint32_t b = r % trail, q = r / trail, ib = q % nb, g = q / nb;
            const uint32_t first = (g * nk + ib * 4) * trail + b;
            V4 acc = V4{0, 0, 0, 0};
            for (uint32_t j = m > 0 ? j0 : 0; j < (m > 0 ? j0 + 1 : (uint32_t)a.J); ++j) {
                const T* x = in + j * in_term + g * nk * trail + b;
                const T* K = kt + off[m] + j * nk * mp + ib * 4;
#pragma unroll 8
                for (uint32_t l = 0; l < nk; ++l) {
                    const V4 k4 = *(const V4*)(K + l * mp);
                    const T v = x[l * trail];
#pragma unroll
                    for (int c = 0; c < 4; ++c) acc[c] = __builtin_elementwise_fma((T)k4[c], v, acc[c]);
                }
            }
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                if (ib * 4 + c >= nk) continue;
                const uint32_t i = first + c * trail;
                if (m == 0) Y[i] = acc[c] + ((T)a.sigma2 + (a.dvec ? ((const T*)a.dvec)[i] : (T)0)) * xs[i];
                else out[j0 * n + i] = acc[c];
            }
        }
        __syncthreads();
        in = out;
        in_term = n;
        trail *= nk;
    }
}

template <typename T>
void launch_tiny(const TinyArgs& a, size_t lds, hipStream_t s) {
    if (a.F == 2) hipLaunchKernelGGL((k_tiny_mvm<T, 2>), dim3((unsigned)a.nrhs), dim3(kTinyThreads), lds, s, a);
    else hipLaunchKernelGGL((k_tiny_mvm<T, 3>), dim3((unsigned)a.nrhs), dim3(kTinyThreads), lds, s, a);
}

}  // namespace

// Up to 512 right-hand sides (beyond, the mode products fill the chip by themselves), 64 KB of LDS, and
// a bound on the longest thread's steps along k.  Measured on the GPU alone, in us, mode products
// against this kernel, one right-hand side: two modes, FP32: 58 steps (50 x 8) 6.2 / 5.2, 80 (40 x 40)
// 6.7 / 6.3, 94 (64 x 30) 6.1 / 7.9; FP64: 58 6.8 / 5.7, 70 (30 x 40) 6.9 / 7.3; three modes, FP32: 36
// (12 x 10 x 14) 10.1 / 6.3, 96 (16 x 16 x 16) 10.3 / 11.1, but at 64 right-hand sides 17.9 / 11.3 and
// 164 steps (20 x 20 x 6, two terms) 36.3 / 14.9; FP64: 36 12.8 / 7.0.
bool tiny_mvm_supported(int F, int J, const int64_t* dims, int nrhs, int es) {
    if (F < 2 || F > 3 || nrhs > 512) return false;
    int64_t n = 1;
    for (int m = 0; m < F; ++m) {
        if (dims[m] > 256 || J > 256) return false;          // no product below leaves 64 bits
        n *= dims[m];
    }
    int64_t steps = 0;
    for (int m = 0; m < F; ++m) {
        const int64_t groups = n / dims[m] * (up4(dims[m]) / 4);
        const int64_t iters = ((m > 0 ? groups * J : groups) + kTinyThreads - 1) / kTinyThreads;
        steps += iters * dims[m] * (m > 0 ? 1 : J);
    }
    const int64_t most = F == 3 ? (nrhs >= 64 ? 170 : 80) : (es == 8 ? 60 : 80);
    return steps <= most && tiny_elems(F, J, dims) * es <= kTinyLds;
}

hipError_t launch_tiny_mvm(int prec, const TinyArgs& a, hipStream_t s) {
    const int64_t dims[3] = {a.dims[0], a.dims[1], a.dims[2]};
    const int es = prec == COLA_PREC_FP64 ? 8 : 4;
    if (!tiny_mvm_supported(a.F, a.J, dims, a.nrhs, es)) return hipErrorInvalidValue;
    const size_t lds = (size_t)tiny_elems(a.F, a.J, dims) * es;
    if (prec == COLA_PREC_FP64) launch_tiny<double>(a, lds, s);
    else launch_tiny<float>(a, lds, s);
    return hipGetLastError();
}

}  // namespace cola

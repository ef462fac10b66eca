// Eigendecomposition of Kronecker factors for the Kronecker-eigen solve.
//
// A single Kronecker term K1 (x) .. (x) KF + sigma2 I with symmetric factors
// K_k = Q_k diag(lam_k) Q_k^T has eigenvectors Q1 (x) .. (x) QF and
// eigenvalues lam1 (x) .. (x) lamF + sigma2 (the Kronecker eigenvalue rule of
// the paper's appendix on Kronecker products).  The factors are decomposed
// here with one-sided (Hestenes) Jacobi in FP64: columns of U = A V are
// orthogonalised pairwise by plane rotations accumulated into V, all n/2 pairs of
// one round-robin step at a time.  Factors of up to 140 points are decomposed side
// by side: one workgroup per factor holds U in LDS and runs a whole sweep per launch
// (16 lanes a pair), and the next launch applies the sweep's rotations to the rows of
// Q.  Larger factors take one launch per step and one workgroup per pair.
#include "eig.h"

#include <algorithm>
#include <climits>
#include <cmath>
#include <vector>

#include "vector.h"

namespace cola {

namespace {

// Player at table position `pos` in round-robin step `step` (m players, m even):
// player 0 stays, the others rotate, so every pair meets once in m - 1 steps.
__device__ inline int rr_player(int pos, int step, int m) {
    return pos == 0 ? 0 : 1 + (pos - 1 + step) % (m - 1);
}

__global__ __launch_bounds__(kThreads) void k_jacobi_step(double* U, double* V, int64_t n, int m, int step,
                                                          double tol, unsigned long long* off_bits) {
    __shared__ double red[4];
    int p = rr_player(blockIdx.x, step, m);
    int q = rr_player(m - 1 - blockIdx.x, step, m);
    if (p >= n || q >= n) return;                          // the idle player of an odd n
    if (p > q) { const int t = p; p = q; q = t; }
    double* up = U + (int64_t)p * n;
    double* uq = U + (int64_t)q * n;
    double a = 0.0, b = 0.0, g = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += kThreads) {
        const double x = up[i], y = uq[i];
        a = __builtin_fma(x, x, a);
        b = __builtin_fma(y, y, b);
        g = __builtin_fma(x, y, g);
    }
    a = block_sum(a, red);
    b = block_sum(b, red);
    g = block_sum(g, red);
    const double ab = sqrt(a * b);
    const double rel = ab > 0.0 ? fabs(g) / ab : 0.0;
    if (threadIdx.x == 0 && rel > 0.0) {
        // non-negative doubles order like their bit patterns
        atomicMax(off_bits, (unsigned long long)__double_as_longlong(rel));
    }
    if (!(rel > tol)) return;
    // rotation that makes columns p and q orthogonal (smaller root of t^2 + 2 zeta t - 1 = 0)
    const double zeta = (b - a) / (2.0 * g);
    const double t = (zeta >= 0.0 ? 1.0 : -1.0) / (fabs(zeta) + sqrt(1.0 + zeta * zeta));
    const double c = 1.0 / sqrt(1.0 + t * t), s = c * t;
    double* vp = V + (int64_t)p * n;
    double* vq = V + (int64_t)q * n;
    for (int64_t i = threadIdx.x; i < n; i += kThreads) {
        const double x = up[i], y = uq[i];
        up[i] = c * x - s * y;
        uq[i] = s * x + c * y;
        const double xv = vp[i], yv = vq[i];
        vp[i] = c * xv - s * yv;
        vq[i] = s * xv + c * yv;
    }
}

// U = A (column-major copy of a symmetric matrix), V = I.
__global__ void k_jacobi_init(const double* A, double* U, double* V, int64_t n) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < n * n; e += (int64_t)gridDim.x * blockDim.x) {
        U[e] = A[e];
        V[e] = (e / n == e % n) ? 1.0 : 0.0;
    }
}

// One pair of columns of U in LDS by 16 lanes (lane l: rows l, l + 16, ..; R of them): rotate them
// orthogonal and return the rotation.
template <int R>
__device__ inline double2 jacobi_pair(double* up, double* uq, int n, int l, double tol, bool& rotated) {
    double x[R], y[R];
    double a = 0.0, b = 0.0, g = 0.0;
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const bool in = r + 1 < R || l + 16 * r < n;
        x[r] = in ? up[l + 16 * r] : 0.0;
        y[r] = in ? uq[l + 16 * r] : 0.0;
        a = __builtin_fma(x[r], x[r], a);
        b = __builtin_fma(y[r], y[r], b);
        g = __builtin_fma(x[r], y[r], g);
    }
    a = row_sum16(a);
    b = row_sum16(b);
    g = row_sum16(g);
    // |u_p . u_q| against tol |u_p| |u_q|, by the squares: a root of a b first is one more link of the chain
    // (120 x 90 x 100 direct solve 5.97 ms with it, 5.51 without)
    if (!(g * g > tol * tol * a * b)) return double2{1.0, 0.0};
    rotated = true;
    // t, the smaller root of t^2 + 2 zeta t - 1 = 0 with zeta = d / h, as h / (d + sign(d) |(d, h)|), and c, s
    // from it.  Roots and divisions are the full ones: with v_sqrt_f64, v_rcp_f64 and a Newton step the solve
    // took 5.24 ms, but the angle had fewer bits, and in c the bias let the columns' norms drift over the
    // sweeps.  Residuals of 200 16^3 RBF solves, median and 99 % quantile: 1.95e-12 and 4.75e-12, the per-step
    // kernel above 1.91e-12 and 5.08e-12.
    double d = b - a, h = 2.0 * g;
    const int ex = -__builtin_amdgcn_frexp_exp(fmax(fabs(d), fabs(h)));    // their squares stay in range
    d = ldexp(d, ex);
    h = ldexp(h, ex);
    const double t = (d >= 0.0 ? h : -h) / (fabs(d) + sqrt(__builtin_fma(d, d, h * h)));
    const double c = 1.0 / sqrt(__builtin_fma(t, t, 1.0));
    const double s = c * t;
#pragma unroll
    for (int r = 0; r < R; ++r)
        if (r + 1 < R || l + 16 * r < n) {
            up[l + 16 * r] = c * x[r] - s * y[r];
            uq[l + 16 * r] = s * x[r] + c * y[r];
        }
    return double2{c, s};
}

constexpr int kJacThreads = 1024;
constexpr int kJacPad = 1;                                  // columns n + 1 doubles apart: spreads the LDS banks

template <int R>
__device__ inline bool jacobi_sweep(double* U, int n, double2* rot, double tol) {
    const int tid = threadIdx.x, l = tid & 15, grp = tid >> 4;
    const int m = n + (n & 1), np = m / 2, ld = n + kJacPad;
    bool rotated = false;
    for (int step = 0; step < m - 1; ++step) {
        for (int k = grp; k < np; k += kJacThreads / 16) {
            int p = rr_player(k, step, m), q = rr_player(m - 1 - k, step, m);
            double2 cs{1.0, 0.0};
            if (p < n && q < n) {                           // not the idle player of an odd n
                if (p > q) { const int t = p; p = q; q = t; }
                cs = jacobi_pair<R>(U + p * ld, U + q * ld, n, l, tol, rotated);
            }
            if (l == 0) rot[(int64_t)step * np + k] = cs;
        }
        __syncthreads();
    }
    return rotated;
}

__device__ inline bool jacobi_sweep_n(double* U, int n, double2* rot, double tol) {
    switch ((n + 15) / 16) {
        case 1: return jacobi_sweep<1>(U, n, rot, tol);
        case 2: return jacobi_sweep<2>(U, n, rot, tol);
        case 3: return jacobi_sweep<3>(U, n, rot, tol);
        case 4: return jacobi_sweep<4>(U, n, rot, tol);
        case 5: return jacobi_sweep<5>(U, n, rot, tol);
        case 6: return jacobi_sweep<6>(U, n, rot, tol);
        case 7: return jacobi_sweep<7>(U, n, rot, tol);
        case 8: return jacobi_sweep<8>(U, n, rot, tol);
        default: return jacobi_sweep<9>(U, n, rot, tol);
    }
}

// What the lanes of a wave wrote to LDS before is what they read after it.
__device__ inline void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Row i of Q: the rotations of one sweep in order, one wave (v: its row in LDS).
__device__ inline void jacobi_row(double* v, double* q, int n, int i, const double2* rot, bool first) {
    const int lane = threadIdx.x & 63;
    for (int j = lane; j < n; j += 64) v[j] = first ? (j == i ? 1.0 : 0.0) : q[(int64_t)i * n + j];
    wave_sync();
    const int m = n + (n & 1), np = m / 2;
    constexpr int NK = (kJacobiLds / 2 + 63) / 64;          // pairs per lane
    double2 next[NK];
#pragma unroll
    for (int u = 0; u < NK; ++u) next[u] = lane + 64 * u < np ? rot[lane + 64 * u] : double2{1.0, 0.0};
    for (int step = 0; step < m - 1; ++step) {
        double2 cs[NK];
#pragma unroll
        for (int u = 0; u < NK; ++u) {
            cs[u] = next[u];
            if (step + 2 < m && lane + 64 * u < np) next[u] = rot[(int64_t)(step + 1) * np + lane + 64 * u];
        }
#pragma unroll
        for (int u = 0; u < NK; ++u) {
            const int k = lane + 64 * u;
            if (k >= np) continue;
            int p = rr_player(k, step, m), q2 = rr_player(m - 1 - k, step, m);
            if (p >= n || q2 >= n) continue;
            if (p > q2) { const int t = p; p = q2; q2 = t; }
            const double x = v[p], y = v[q2];
            v[p] = cs[u].x * x - cs[u].y * y;
            v[q2] = cs[u].y * x + cs[u].x * y;
        }
        wave_sync();                                        // the next step's pairs hold other lanes' columns
    }
    for (int j = lane; j < n; j += 64) q[(int64_t)i * n + j] = v[j];
}

// Sweep `sweep` of every unfinished factor (the first nitems workgroups; not when `last`), and the
// previous sweep's rotations on the rows of Q (the others: rows / 16 per factor).
__global__ __launch_bounds__(kJacThreads) void k_jacobi_round(const JacobiItem* items, JacobiState* state, int nitems,
                                                              int sweep, int last, double tol) {
    __shared__ double U[kJacobiLds * (kJacobiLds + kJacPad)];
    __shared__ int s_rotated, s_exponent;
    const int b = blockIdx.x, tid = threadIdx.x, now = sweep & 1;
    if (b >= nitems) {
        const int f = (b - nitems) % nitems, i = (b - nitems) / nitems * (kJacThreads / 64) + (tid >> 6);
        const JacobiItem it = items[f];
        if (i >= it.n || !(sweep == 1 || state[f].rotated[now ^ 1])) return;    // sweep 0 starts Q in any case
        jacobi_row(U + (tid >> 6) * kJacobiLds, it.q, it.n, i, it.rot + (now ^ 1) * jacobi_rotations(it.n),
                   sweep == 1);
        return;
    }
    if (last) return;
    JacobiState& st = state[b];
    if (sweep > 0 && st.done) {
        if (tid == 0) st.rotated[now] = 0;
        return;
    }
    const JacobiItem it = items[b];
    const int n = it.n, ld = n + kJacPad;
    if (tid == 0) {
        s_rotated = 0;
        s_exponent = INT_MIN;
    }
    __syncthreads();
    if (sweep == 0) {
        // Scaled by a power of two (exactly) to entries of at most 1: unscaled, the squares of columns
        // beyond 1e77 overflowed, no pair looked worth a rotation and A's own basis was returned.
        int top = INT_MIN;
        for (int e = tid; e < n * n; e += kJacThreads) {
            const double v = it.A[e];
            if (v != 0.0 && finite_d(v)) top = max(top, __builtin_amdgcn_frexp_exp(v));
        }
        if (top != INT_MIN) atomicMax(&s_exponent, top);
        __syncthreads();
        const int ex = s_exponent == INT_MIN ? 0 : s_exponent;
        for (int e = tid; e < n * n; e += kJacThreads) U[(e / n) * ld + e % n] = ldexp(it.A[e], -ex);
        if (tid == 0) st.exponent = ex;
    } else {
        for (int e = tid; e < n * n; e += kJacThreads) U[(e / n) * ld + e % n] = it.u[e];
    }
    __syncthreads();
    if (jacobi_sweep_n(U, n, it.rot + now * jacobi_rotations(n), tol)) s_rotated = 1;
    __syncthreads();
    for (int e = tid; e < n * n; e += kJacThreads) it.u[e] = U[(e / n) * ld + e % n];
    if (tid == 0) {
        st.done = !s_rotated;
        st.rotated[now] = s_rotated;
    }
}

// Q^T and the eigenvalues of every factor: lam_j = v_j . u_j (scaled back), one wave a column.
__global__ __launch_bounds__(kThreads) void k_jacobi_finish(const JacobiItem* items, const JacobiState* state) {
    const JacobiItem it = items[blockIdx.y];
    const int n = it.n, lane = threadIdx.x & 63, j = blockIdx.x * 4 + (threadIdx.x >> 6);
    if (j >= n) return;
    double s = 0.0;
    for (int i = lane; i < n; i += 64) {
        const double v = it.q[(int64_t)i * n + j];
        it.vt[(int64_t)j * n + i] = v;
        s = __builtin_fma(it.u[(int64_t)j * n + i], v, s);
    }
    s = wave_sum(s);
    if (lane == 0) it.lam[j] = ldexp(s, state[blockIdx.y].exponent);
}

// lam_j = v_j . u_j = v_j^T A v_j (the Rayleigh quotient of the converged column).
__global__ __launch_bounds__(kThreads) void k_jacobi_values(const double* U, const double* V, int64_t n, double* lam) {
    __shared__ double red[4];
    const int64_t j = blockIdx.x;
    double s = 0.0;
    for (int64_t i = threadIdx.x; i < n; i += kThreads) s = __builtin_fma(U[j * n + i], V[j * n + i], s);
    s = block_sum(s, red);
    if (threadIdx.x == 0) lam[j] = s;
}

__global__ void k_transpose_f64(const double* in, double* out, int64_t n) {
    __shared__ double tile[32][33];
    const int64_t bx = (int64_t)blockIdx.x * 32, by = (int64_t)blockIdx.y * 32;
    const int tx = threadIdx.x & 31, ty = threadIdx.x >> 5;        // 256 threads: 32 x 8
    for (int r = ty; r < 32; r += 8) {
        const int64_t i = by + r, j = bx + tx;
        if (i < n && j < n) tile[r][tx] = in[i * n + j];
    }
    __syncthreads();
    for (int r = ty; r < 32; r += 8) {
        const int64_t i = bx + r, j = by + tx;
        if (i < n && j < n) out[i * n + j] = tile[tx][r];
    }
}

__global__ void k_eig_scale(const double* Y, double* Z, int64_t total, int64_t n, int64_t n2, int64_t n3,
                            const double* l1, const double* l2, const double* l3, double sigma2) {
    for (int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; e < total; e += (int64_t)gridDim.x * blockDim.x) {
        const int64_t rest = e % n;
        const int64_t i3 = rest % n3, i2 = (rest / n3) % n2, i1 = rest / (n2 * n3);
        double lam = l1[i1] * l2[i2];
        if (l3) lam *= l3[i3];
        Z[e] = Y[e] / (lam + sigma2);
    }
}

}  // namespace

int32_t jacobi_eig(const double* A, int64_t n, double* V, double* lam, double* work, double* off, double tol,
                   int max_sweeps, hipStream_t s) {
    if (n < 1 || n > (1 << 20)) return COLA_ERR_INVALID_ARG;
    hipLaunchKernelGGL(k_jacobi_init, dim3((unsigned)std::min<int64_t>((n * n + 255) / 256, 65536)), dim3(256), 0,
                       s, A, work, V, n);
    if (hipGetLastError() != hipSuccess) return COLA_ERR_HIP;
    const int m = (int)(n + (n & 1));                      // even number of players
    unsigned long long* bits = (unsigned long long*)off;
    for (int sweep = 0; sweep < max_sweeps && n > 1; ++sweep) {
        if (fill_f64(off, 0.0, 1, s) != hipSuccess) return COLA_ERR_HIP;
        for (int step = 0; step < m - 1; ++step)
            hipLaunchKernelGGL(k_jacobi_step, dim3((unsigned)(m / 2)), dim3(kThreads), 0, s, work, V, n, m, step,
                               tol, bits);
        if (hipGetLastError() != hipSuccess) return COLA_ERR_HIP;
        double h = 0.0;
        if (hipMemcpyAsync(&h, off, sizeof(double), hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return COLA_ERR_HIP;
        if (!std::isfinite(h)) return COLA_ERR_NONFINITE;
        if (h <= tol) break;
    }
    hipLaunchKernelGGL(k_jacobi_values, dim3((unsigned)n), dim3(kThreads), 0, s, work, V, n, lam);
    return hipGetLastError() == hipSuccess ? COLA_OK : COLA_ERR_HIP;
}

int32_t jacobi_eig_batch(const JacobiItem* items, JacobiState* state, int nitems, int nmax, double tol,
                         int max_sweeps, hipStream_t s) {
    if (nitems < 1 || nitems > 65535 || nmax > kJacobiLds) return COLA_ERR_INVALID_ARG;
    const unsigned blocks = (unsigned)nitems * (1 + (nmax + kJacThreads / 64 - 1) / (kJacThreads / 64));
    std::vector<JacobiState> h(nitems);
    constexpr int kAhead = 6;                               // sweeps enqueued between two looks at the state
    for (int sweep = 0; sweep < max_sweeps;) {
        for (int u = 0; u < kAhead && sweep < max_sweeps; ++u, ++sweep)
            hipLaunchKernelGGL(k_jacobi_round, dim3(sweep == 0 ? (unsigned)nitems : blocks), dim3(kJacThreads), 0, s,
                               items, state, nitems, sweep, 0, tol);
        if (hipGetLastError() != hipSuccess) return COLA_ERR_HIP;
        const bool end = sweep >= max_sweeps;
        if (hipMemcpyAsync(h.data(), state, sizeof(JacobiState) * nitems, hipMemcpyDeviceToHost, s) != hipSuccess ||
            hipStreamSynchronize(s) != hipSuccess)
            return COLA_ERR_HIP;
        bool done = true;
        for (const JacobiState& st : h) done = done && st.done;
        if (done || end) {                                  // the last sweep's rotations (none if all are done)
            hipLaunchKernelGGL(k_jacobi_round, dim3(blocks), dim3(kJacThreads), 0, s, items, state, nitems, sweep, 1,
                               tol);
            break;
        }
    }
    const dim3 rows((unsigned)((nmax + 3) / 4), (unsigned)nitems);
    hipLaunchKernelGGL(k_jacobi_finish, rows, dim3(kThreads), 0, s, items, state);
    return hipGetLastError() == hipSuccess ? COLA_OK : COLA_ERR_HIP;
}

hipError_t eig_scale(const double* Y, double* Z, int64_t nrhs, int F, const int64_t* dims,
                     const double* const* lam, double sigma2, hipStream_t s) {
    int64_t d[3] = {1, 1, 1};
    for (int k = 0; k < F; ++k) d[k] = dims[k];
    const int64_t n = d[0] * d[1] * d[2];
    const int64_t total = nrhs * n;
    const unsigned grid = (unsigned)std::max<int64_t>(1, std::min<int64_t>((total + 255) / 256, 65536));
    hipLaunchKernelGGL(k_eig_scale, dim3(grid), dim3(256), 0, s, Y, Z, total, n, d[1], d[2], lam[0], lam[1],
                       F == 3 ? lam[2] : nullptr, sigma2);
    return hipGetLastError();
}

hipError_t transpose_f64(const double* in, double* out, int64_t n, hipStream_t s) {
    const unsigned g = (unsigned)((n + 31) / 32);
    hipLaunchKernelGGL(k_transpose_f64, dim3(g, g), dim3(256), 0, s, in, out, n);
    return hipGetLastError();
}

}  // namespace cola

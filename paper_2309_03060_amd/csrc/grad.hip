// Adjoint backward of the solve, and the contraction-tile autotuner.
//
// App. B.2 (autograd rule 1): with lambda = A^{-1} dL/dx, the gradient of the
// loss with respect to any operator parameter theta is
//     -sum_r lambda_r^T (dA/dtheta) x_r.
// For a factor K_jk of a Kronecker term this is a contraction of the mode-k
// unfoldings of Lambda and of Z = X multiplied along every other mode by the
// term's factors:  dK_jk = -sum_r Lambda_r,(k) Z_r,(k)^T  (n_k x n_k), a GEMM
// whose inner dimension is nrhs * n / n_k.  It runs as a split-K FP64 MFMA
// kernel (each block a slice of the inner dimension), and a second kernel
// sums the slices in fixed order.  The diagonal and sigma2 gradients are
// -sum_r lambda_r * x_r and its total.
#include <algorithm>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include "grad.h"

#include "gemm.h"
#include "gemm3.h"
#include "modepass.h"
#include "vector.h"

namespace cola {

// out[c][a][i] = scale * sum over (g, t) in chunk c of L[g, a, t] * Z[g, i, t]
//
// A GEMM of nk x nk outputs whose inner dimension (all other modes and right-hand sides) is cut into
// slices of 16 (of t within one g; of g where t has one value) and chunks of slices, one per block and
// tile.  The next slice is on its way in registers while the present one, in one of two LDS stages, is
// multiplied (one barrier per slice); loads are clamped, not branched around, and what lies beyond the
// range becomes zero on the way to LDS.  Tiles of 128 x 128 halve the loads per product of 64 x 64 ones,
// whose 4.3 GB through L2 bounded the largest: 1024 x 1024 outputs, inner dimension 16384, 1149 / 1106 us
// (t / g slices) staged in turn with 64 x 64 tiles, 621 / 612 us now (0.48 ms of products); 128 uneven
// systems of 16 .. 128 points, 16.1 -> 7.3 us a launch on average; 200 x 200 outputs, inner dimension
// 2880, 41.8 -> 18.5 us.
template <int WM, bool TRAIL1>
__global__ __launch_bounds__(kThreads, WM > 2 ? 2 : 4) void k_grad_gemm(const double* L, const double* Z, int64_t G, int nk,
                                                           int64_t T, int64_t slices, int64_t per_chunk, double scale,
                                                           double* out) {
    constexpr int MT = 32 * WM, KT = 16;
    constexpr int KP = KT + 2, MP = MT + 16;                 // pitches of an [m][k] and of a [k][m] stage
    constexpr int EL = TRAIL1 ? KT * MP : MT * KP;
    constexpr int NV = MT * KT / kThreads;                   // elements of each operand per thread and slice
    __shared__ double lds[2 * 2 * EL];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, lr = lane & 15, lq = lane >> 4;
    const int wm = wave >> 1, wn = wave & 1;
    const int nt = (nk + MT - 1) / MT;
    const int a0 = (int)(blockIdx.x / nt) * MT, i0 = (int)(blockIdx.x % nt) * MT;
    const int64_t c = blockIdx.y;
    const int64_t sbeg = c * per_chunk, send = sbeg + per_chunk < slices ? sbeg + per_chunk : slices;
    const int64_t per_g = TRAIL1 ? 1 : (T + KT - 1) / KT;

    // element e of a thread: row and k of the stage (consecutive threads along the contiguous index)
    auto em = [&](int e) { return TRAIL1 ? tid % MT : tid / KT + e * (kThreads / KT); };
    auto ek = [&](int e) { return TRAIL1 ? tid / MT + e * (kThreads / MT) : tid % KT; };
    int64_t g = TRAIL1 ? 0 : sbeg / per_g, k0 = TRAIL1 ? sbeg * KT : (sbeg - g * per_g) * KT;   // the slice loaded next
    const int64_t kmax = (TRAIL1 ? G : T) - 1;
    double av[NV], bv[NV];
    int valid;                                               // elements of k in the loaded slice
    auto load = [&]() {
        const double* Lg = L + (TRAIL1 ? k0 * nk : g * nk * T + k0);
        const double* Zg = Z + (TRAIL1 ? k0 * nk : g * nk * T + k0);
        valid = (int)(kmax + 1 - k0 < KT ? kmax + 1 - k0 : KT);
#pragma unroll
        for (int e = 0; e < NV; ++e) {
            const int k = ek(e) < valid ? ek(e) : valid - 1;
            const int ma = a0 + em(e) < nk ? a0 + em(e) : nk - 1, mi = i0 + em(e) < nk ? i0 + em(e) : nk - 1;
            av[e] = Lg[TRAIL1 ? (int64_t)k * nk + ma : ma * T + k];
            bv[e] = Zg[TRAIL1 ? (int64_t)k * nk + mi : mi * T + k];
        }
        k0 += KT;
        if (!TRAIL1 && k0 >= T) {
            k0 = 0;
            ++g;
        }
    };
    auto store = [&](double* As) {
        double* Bs = As + EL;
#pragma unroll
        for (int e = 0; e < NV; ++e) {
            const int at = TRAIL1 ? ek(e) * MP + em(e) : em(e) * KP + ek(e);
            As[at] = ek(e) < valid ? av[e] : 0.0;
            Bs[at] = ek(e) < valid ? bv[e] : 0.0;
        }
    };

    doublex4 acc[WM][WM];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WM; ++j) acc[i][j] = doublex4{0, 0, 0, 0};
    load();
    for (int64_t s = sbeg; s < send; ++s) {
        double* As = lds + ((s - sbeg) & 1) * 2 * EL;
        const double* Bs = As + EL;
        store(As);
        // the barrier also covers the other stage: every wave read it before it came here
        __syncthreads();
        if (s + 1 < send) load();
#pragma unroll
        for (int kk = 0; kk < KT; kk += 4) {
            double x[WM], y[WM];
#pragma unroll
            for (int i = 0; i < WM; ++i) {
                const int m = (wm * WM + i) * 16 + lr, n = (wn * WM + i) * 16 + lr;
                x[i] = As[TRAIL1 ? (kk + lq) * MP + m : m * KP + kk + lq];
                y[i] = Bs[TRAIL1 ? (kk + lq) * MP + n : n * KP + kk + lq];
            }
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WM; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f64_16x16x4f64(x[i], y[j], acc[i][j], 0, 0, 0);
        }
    }
    double* o = out + c * (int64_t)nk * nk;
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WM; ++j)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int a = a0 + (wm * WM + i) * 16 + 4 * v + lq, ii = i0 + (wn * WM + j) * 16 + lr;
                if (a < nk && ii < nk) o[(int64_t)a * nk + ii] = scale * acc[i][j][v];
            }
}

// dK = sum_c partial[c]: 64 entries a block, a quarter of the chunks per wave, summed in fixed order.
__global__ __launch_bounds__(kThreads) void k_grad_reduce(const double* partial, int64_t nchunks, int64_t nn, double* dK) {
    __shared__ double red[kThreads];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int64_t e = (int64_t)blockIdx.x * 64 + lane, ec = e < nn ? e : nn - 1;
    double s = 0.0;
#pragma unroll 4
    for (int64_t c = wave; c < nchunks; c += 4) s += partial[c * nn + ec];
    red[threadIdx.x] = s;
    __syncthreads();
    if (wave == 0 && e < nn) dK[e] = (red[lane] + red[64 + lane]) + (red[128 + lane] + red[192 + lane]);
}

template <int WM>
void launch_grad_gemm(bool trail1, int64_t tiles, int64_t chunks, const double* L, const double* Z, int64_t G, int64_t nk,
                      int64_t T, int64_t slices, int64_t per_chunk, double scale, double* out, hipStream_t st) {
    const dim3 grid((unsigned)tiles, (unsigned)chunks);
    if (trail1)
        hipLaunchKernelGGL((k_grad_gemm<WM, true>), grid, dim3(kThreads), 0, st, L, Z, G, (int)nk, T, slices, per_chunk,
                           scale, out);
    else
        hipLaunchKernelGGL((k_grad_gemm<WM, false>), grid, dim3(kThreads), 0, st, L, Z, G, (int)nk, T, slices, per_chunk,
                           scale, out);
}

// dd[e] = scale * (-sum_r lambda_r[e] x_r[e]);  dsigma2 = scale * (-sum_e sum_r lambda_r[e] x_r[e])
__global__ __launch_bounds__(kThreads) void k_grad_diag(const double* X, const double* Lam, int64_t n, int nrhs,
                                                        double* dd, double* dsigma2, double* partials,
                                                        uint32_t* counter, double scale) {
    __shared__ double red[4];
    double tot_local = 0.0;
    for (int64_t e = (int64_t)blockIdx.x * kThreads + threadIdx.x; e < n; e += (int64_t)gridDim.x * kThreads) {
        double s = 0.0;
#pragma unroll 4
        for (int r = 0; r < nrhs; ++r) s += Lam[(int64_t)r * n + e] * X[(int64_t)r * n + e];
        if (dd) dd[e] = -s * scale;
        tot_local += s;
    }
    const double b = block_sum(tot_local, red);
    double tot;
    if (last_block_reduce(b, partials, counter, gridDim.x, blockIdx.x, &tot, red) && threadIdx.x == 0 && dsigma2)
        *dsigma2 = -tot * scale;
}

// ---------------------------------------------------------------------------
int32_t apply_modes_f64(cola_op_s* op, const SysInfo& s, int term, int skip, const double* X, int nrhs,
                        double* out, hipStream_t st) {
    // ping-pong between out and inter[1]; the final product lands in `out`
    std::vector<int> modes;
    for (int m = s.Fv - 1; m >= 0; --m)
        if (m != skip && !(s.F == 1 && m == 0)) modes.push_back(m);
    if (modes.empty()) {
        if (hipMemcpyAsync(out, X, sizeof(double) * (size_t)nrhs * s.n, hipMemcpyDeviceToDevice, st) != hipSuccess)
            return COLA_ERR_HIP;
        return COLA_OK;
    }
    double* bufs[2] = {out, (double*)op->ws.inter[1]};
    int cur = (modes.size() % 2 == 1) ? 0 : 1;  // so that the last pass writes `out`
    const double* in = X;
    for (size_t q = 0; q < modes.size(); ++q) {
        const int m = modes[q];
        const int64_t nk = s.dims[m];
        int64_t lead = 1, trail = 1;
        for (int u = 0; u < m; ++u) lead *= s.dims[u];
        for (int u = m + 1; u < s.Fv; ++u) trail *= s.dims[u];
        PassArgs a;
        std::memset(&a, 0, sizeof(a));
        a.nk = (int32_t)nk;
        a.nsum = 1;
        a.nout = 1;
        a.K = op->fac64 + s.fac_off[m] + (int64_t)term * nk * nk;
        a.k_tstride = nk * nk;
        a.X = in;
        a.Y = bufs[cur];
        a.epi = EPI_STORE;
        const bool rows = (trail == 1);
        a.G = (int64_t)nrhs * lead;
        a.B = rows ? 1 : trail;
        a.a_per_rhs = lead;
        const TileCfg cfg = rows ? mode_tile(true, nk, a.G, nk, 1) : mode_tile(false, nk, nk, trail, a.G);
        if (launch_contract(COLA_PREC_FP64, rows, a, cfg, st) != hipSuccess) return COLA_ERR_HIP;
        in = bufs[cur];
        cur ^= 1;
    }
    return COLA_OK;
}

int32_t grad_system(cola_op_s* op, const SysInfo& s, const double* X, const double* Lam, int nrhs,
                    void* const* dfactors, void* ddiag, double* dsigma2, hipStream_t st, double scale) {
    if (op->ws.nrhs < nrhs) return COLA_ERR_INVALID_ARG;    // staging buffers must hold nrhs vectors
    if (dfactors) {
        double* Z = (double*)op->ws.inter[0];
        for (int j = 0; j < s.J; ++j)
            for (int k = 0; k < s.F; ++k) {
                double* dK = (double*)dfactors[j * s.F + k];
                if (!dK) continue;
                const int kv = (s.F == 1) ? 1 : k;
                int32_t rc = apply_modes_f64(op, s, j, kv, X, nrhs, Z, st);
                if (rc != COLA_OK) return rc;
                const int64_t nk = s.dims[kv];
                int64_t lead = 1, trail = 1;
                for (int u = 0; u < kv; ++u) lead *= s.dims[u];
                for (int u = kv + 1; u < s.Fv; ++u) trail *= s.dims[u];
                const int64_t G = (int64_t)nrhs * lead;
                // 128 x 128 tiles where they still fill the CUs, 32 x 32 for the smallest modes.  About two
                // blocks per CU, of at least 8 slices each (short ones cost the sum more than they save); the
                // chunks' outputs use the last workspace vector, as many as fit it, and a single chunk writes
                // the gradient itself.
                const int64_t slices = trail == 1 ? (G + 15) / 16 : G * ((trail + 15) / 16);
                const int64_t room = std::max<int64_t>(1, (int64_t)op->ws.nrhs * op->nmax / (nk * nk));
                int wm = 4;
                int64_t tiles = 1, chunks = 1;
                for (;; wm /= 2) {
                    const int64_t side = (nk + 32 * wm - 1) / (32 * wm);
                    tiles = side * side;
                    chunks = std::max<int64_t>(1, std::min<int64_t>({512 / tiles, slices / 8, room}));
                    if (wm == 1 || (nk >= 64 * (wm / 2) * (wm / 2) && (wm == 2 || tiles * chunks >= 256))) break;
                }
                const int64_t per_chunk = (slices + chunks - 1) / chunks;
                chunks = (slices + per_chunk - 1) / per_chunk;
                double* out = chunks == 1 ? dK : (double*)op->ws.vq;
                if (wm == 4)
                    launch_grad_gemm<4>(trail == 1, tiles, chunks, Lam, Z, G, nk, trail, slices, per_chunk, -scale, out, st);
                else if (wm == 2)
                    launch_grad_gemm<2>(trail == 1, tiles, chunks, Lam, Z, G, nk, trail, slices, per_chunk, -scale, out, st);
                else
                    launch_grad_gemm<1>(trail == 1, tiles, chunks, Lam, Z, G, nk, trail, slices, per_chunk, -scale, out, st);
                if (hipGetLastError() != hipSuccess) return COLA_ERR_HIP;
                if (chunks > 1) {
                    const int64_t nn = nk * nk;
                    hipLaunchKernelGGL(k_grad_reduce, dim3((unsigned)((nn + 63) / 64)), dim3(kThreads), 0, st, out, chunks,
                                       nn, dK);
                    if (hipGetLastError() != hipSuccess) return COLA_ERR_HIP;
                }
            }
    }
    if (ddiag || dsigma2) {
        // a thread's chain is its right-hand sides' loads: two entries a thread, at most 512 blocks
        // (36000 x 16: 40.7 us with eight entries)
        const unsigned blocks = (unsigned)std::min<int64_t>(512, std::max<int64_t>(1, (s.n + 511) / 512));
        hipLaunchKernelGGL(k_grad_diag, dim3(blocks), dim3(kThreads), 0, st, X, Lam, s.n, nrhs, (double*)ddiag,
                           dsigma2, op->ws.partials, op->ws.counters, scale);
        if (hipGetLastError() != hipSuccess) return COLA_ERR_HIP;
    }
    return COLA_OK;
}

// ---------------------------------------------------------------------------
// Autotuner: for each contraction pass of each system (at this nrhs), time
// every tile candidate over a few launches with HIP events and keep the
// fastest in the op's tile table.
int32_t autotune_op(cola_op_s* op, int nrhs, hipStream_t st) {
    int32_t rc = ensure_workspace(op, nrhs, st);
    if (rc != COLA_OK) return rc;
    const TileCfg cands[] = {{1, 1}, {1, 2}, {2, 1}, {2, 2}, {4, 2}, {2, 4}, {4, 4}, {1, 4}, {4, 1}};
    hipEvent_t e0, e1;
    if (hipEventCreate(&e0) != hipSuccess || hipEventCreate(&e1) != hipSuccess) return COLA_ERR_HIP;
    std::vector<int> precs = {COLA_PREC_FP64};
    if (op->prec != COLA_PREC_FP64) precs.push_back(op->prec);
    for (const SysInfo& s : op->sys) {
        for (int prec : precs) {
            if ((op->use_gemm2 && gemm2_supported(prec, s.Fv, s.dims)) ||
                (op->use_gemm3 && gemm3_supported(prec, s.Fv, s.J, s.dims)))
                continue;                                                         // fixed GEMM tiles
            for (int k = s.Fv - 1; k >= 0; --k) {
                const int64_t nk = s.dims[k];
                int64_t lead = 1, trail = 1;
                for (int u = 0; u < k; ++u) lead *= s.dims[u];
                for (int u = k + 1; u < s.Fv; ++u) trail *= s.dims[u];
                const bool rows = (k == s.Fv - 1);
                PassKey key{prec, rows ? 1 : 0, nk, rows ? 1 : trail, lead};
                float best = 1e30f;
                TileCfg bestc = cands[1];
                for (const TileCfg& c : cands) {
                    PassArgs a;
                    std::memset(&a, 0, sizeof(a));
                    a.nk = (int32_t)nk;
                    a.nsum = (k == 0) ? s.J : 1;
                    a.nout = (k == 0) ? 1 : s.J;
                    a.G = (int64_t)nrhs * lead;
                    a.B = rows ? 1 : trail;
                    a.a_per_rhs = lead;
                    a.X = op->ws.vx;
                    a.x_tstride = 0;
                    a.Y = op->ws.inter[0];
                    a.y_tstride = (int64_t)nrhs * s.n;
                    a.K = (prec == COLA_PREC_FP64) ? (const void*)(op->fac64 + s.fac_off[k])
                          : (prec == COLA_PREC_FP32) ? (const void*)(op->fac32 + s.fac_off[k])
                                                     : (const void*)(op->facbf + s.fac_off[k]);
                    a.k_tstride = nk * nk;
                    a.k_plane = op->fac_elems;
                    a.epi = EPI_STORE;
                    if (launch_contract(prec, rows, a, c, st) != hipSuccess) return COLA_ERR_HIP;  // warm
                    (void)hipEventRecord(e0, st);
                    for (int rep = 0; rep < 5; ++rep)
                        if (launch_contract(prec, rows, a, c, st) != hipSuccess) return COLA_ERR_HIP;
                    (void)hipEventRecord(e1, st);
                    if (hipEventSynchronize(e1) != hipSuccess) return COLA_ERR_HIP;
                    float ms = 0.f;
                    (void)hipEventElapsedTime(&ms, e0, e1);
                    if (ms < best) {
                        best = ms;
                        bestc = c;
                    }
                }
                op->tiles[key] = bestc;
                if (std::getenv("COLA_VERBOSE"))
                    std::fprintf(stderr, "cola_autotune: prec %d %s nk %lld B %lld lead %lld -> tile %dx%d (%.1f us)\n",
                                 prec, rows ? "rows" : "cols", (long long)nk, (long long)(rows ? 1 : trail),
                                 (long long)lead, 32 * bestc.wm, 32 * bestc.wn, 1e3 * best / 5);
            }
        }
    }
    (void)hipEventDestroy(e0);
    (void)hipEventDestroy(e1);
    op->tiles_version += 1;
    return COLA_OK;
}

}  // namespace cola

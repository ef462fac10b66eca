// Resident batched CG: many independent small systems in one persistent launch.
//
// CoLA solves blocks of right-hand sides together and stops when all have
// converged (App. D.5); here the block is a batch of independent systems
// K1 (x) K2 + diag(d) + sigma2 I of uneven sizes (mode sizes up to 128).
// Each (system, RHS) item is owned by one workgroup of eight waves for as long
// as it iterates.  The batch ends with its longest solves, one CU each, so what
// counts is the time of an iteration of a large system, which is bound by its
// FP32 MFMAs (13.7 us at 128 x 128 on one CU):
//   - x, r and p stay in registers, in the layout of the second product's output;
//     P and T = P K2^T pass through LDS, and both products are formed so that
//     every LDS access moves four consecutive elements of k (T is written
//     transposed straight from the accumulators, Q comes out transposed);
//   - the factors are read as fragments from L2, a step of 16 k ahead, so no
//     barrier separates slices: four barriers an iteration (two for the exchange
//     of P and T, one for each dot product);
//   - 16 x 16 tiles, dealt to the SIMDs along the mode that balances them.
// Workgroups pull items from an atomic queue ordered largest-first, so uneven
// iteration counts balance across the chip, and every workgroup leaves once the
// queue is empty.  When an item's FP32 residual has dropped by delta (or
// converged), its workgroup folds x into the FP64 solution, forms b - A x with the
// FP64 factors, replaces r and resumes the same CG (reliable updates), so items
// do not wait for one another.
// 128 uneven systems (modes 16 to 128, 216 iterations on average and up to 670),
// two solves and their gradients: 56 ms with the factors staged through LDS in
// 32-column chunks (two barriers a chunk, x in memory: 36 us an iteration at 128 x
// 128), 31 ms with the iteration above, 29 ms with the residuals in the same
// launch (before, a launch for every round of all items and one for its residuals).
#include "resident.h"

namespace cola {

constexpr int kResThreads = 512;                 // 8 waves per item
constexpr int kResWaves = kResThreads / 64;
constexpr int RPS = kResMax + 4;                 // LDS row stride of P and T^T (floats): conflict-free 16-byte accesses
constexpr int PX = kResMax + 2;                  // pitch of the FP64 X: conflict-free A-operand reads
constexpr size_t kResLds = 2 * sizeof(float) * kResMax * RPS > sizeof(double) * kResMax * PX
                               ? 2 * sizeof(float) * kResMax * RPS : sizeof(double) * kResMax * PX;
typedef float floatx4u __attribute__((ext_vector_type(4), aligned(4)));

// Sum over the WAVES waves of a workgroup with a single barrier.  A caller
// that sums again must use another slot array (or pass a barrier) before it
// writes these slots again: other waves may still be reading them.
template <int WAVES>
__device__ inline double block_sum_once(double v, double* smem) {
    v = wave_sum(v);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (lane == 0) smem[wave] = v;
    __syncthreads();
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < WAVES; ++i) s += smem[i];
    return s;
}

__global__ __launch_bounds__(kThreads) void k_resident_prepare(ResArgs a, double tol, int max_iters, double delta) {
    __shared__ double red[4];
    const int item = blockIdx.x;
    const ResSys sy = a.sys[item / a.nrhs];
    const int rhs = item % a.nrhs;
    const int64_t base = (int64_t)a.nrhs * sy.vec_off + (int64_t)rhs * sy.n;
    double sb = 0.0, sr = 0.0;
    for (int64_t e = threadIdx.x; e < sy.n; e += kThreads) {
        const double v = a.b64[base + e];
        const float f = (float)v;
        a.r[base + e] = f;
        a.x[base + e] = 0.f;
        a.p[base + e] = 0.f;
        a.x64[base + e] = 0.0;
        sb += v * v;
        sr += (double)f * (double)f;
    }
    sb = block_sum(sb, red);
    sr = block_sum(sr, red);
    if (threadIdx.x == 0) {
        CgState& st = a.st[item];
        st.rho = sr;
        st.bnorm2 = sb;
        st.tol2 = tol * tol * sb;
        st.alpha = 0.0;
        st.beta = 0.0;
        st.iters = 0;
        st.max_iters = max_iters;
        st.delta = delta < 0.0 ? -delta : delta;
        st.restart_dir = delta < 0.0;
        st.rmax = sqrt(sr);
        st.rho_true = sb;
        st.need_update = 0;
        st.fails = 0;
        st.updates = 0;
        if (!finite_d(sb) || !finite_d(sr)) {
            st.status = COLA_ERR_NONFINITE;
            st.active = 0;
        } else if (sb <= st.tol2) {                 // b = 0: x = 0 after zero iterations
            st.status = COLA_OK;
            st.active = 0;
        } else {
            st.status = COLA_NOT_CONVERGED;
            st.active = 1;
            atomicAdd(&a.cnt->num_active, 1);
        }
    }
}

__device__ inline floatx4 mma4(const floatx4& a, const floatx4& b, floatx4 c) {
#pragma unroll
    for (int k = 0; k < 4; ++k) c = __builtin_amdgcn_mfma_f32_16x16x4f32(a[k], b[k], c, 0, 0, 0);
    return c;
}

// Fragments of the 16 factor rows of N tiles: lane l holds row l % 16, elements k0 + 4 (l / 16) .. + 3
// (the factor buffer is padded past its last row; elements beyond the row are zeroed by `cut`).
template <int N>
struct FactorRows {
    const float* row[N];
    int nk, kl;                                             // mode size, this lane's first k of a step
    floatx4 v[N];
    __device__ void start(const float* K, int n, int first_tile, int tile_step) {
        const int lane = threadIdx.x & 63;
        nk = n;
        kl = 4 * (lane >> 4);
#pragma unroll
        for (int t = 0; t < N; ++t) {
            int r = 16 * (first_tile + tile_step * t) + (lane & 15);
            if (r >= n) r = n - 1;                          // its outputs are masked
            row[t] = K + r * n + kl;
        }
    }
    __device__ void load(int k0) {
#pragma unroll
        for (int t = 0; t < N; ++t) v[t] = *(const floatx4u*)(row[t] + k0);
    }
    __device__ void cut(int k0) {
        if (k0 + 16 <= nk) return;
#pragma unroll
        for (int t = 0; t < N; ++t)
#pragma unroll
            for (int c = 0; c < 4; ++c) v[t][c] = k0 + kl + c < nk ? v[t][c] : 0.f;
    }
};

// The iterations of one item.  This wave owns the 16 x 16 tiles (wi + GI a, wj + GJ b), a < WI,
// b < WJ; its lane holds the elements i = 16 (wi + GI a) + lane % 16, j = 16 (wj + GJ b) + 4 (lane / 16) + v.
template <int WI, int WJ>
__device__ inline void resident_item(const ResArgs& a, int item, float* Ps, float* Ts, double* red_pq,
                                     double* red_rr) {
    constexpr int GI = 8 / WI, GJ = 8 / WJ;                 // 8 x 8 tiles at most: 8 waves
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lr = lane & 15, lq = lane >> 4;
    // wave % 4 is the SIMD: it goes along the mode with four wave columns
    const int wi = GI == 4 ? wave & 3 : wave >> 2, wj = GJ == 4 ? wave & 3 : wave >> 2;
    CgState* stp = &a.st[item];
    const ResSys sy = a.sys[item / a.nrhs];
    const int rhs = item % a.nrhs;
    const int n1 = sy.n1, n2 = sy.n2;
    const int t1 = (n1 + 15) / 16, t2 = (n2 + 15) / 16;     // tiles, and k steps of 16
    const int na = (t1 - wi + GI - 1) / GI, nb = (t2 - wj + GJ - 1) / GJ;    // this wave's
    const int64_t base = (int64_t)a.nrhs * sy.vec_off + (int64_t)rhs * sy.n;
    const float* dgv = sy.diag_off >= 0 ? a.diag32 + sy.diag_off : nullptr;
    const float s2 = (float)sy.sigma2;
    FactorRows<WJ> k2;
    FactorRows<WI> k1;
    k2.start(a.fac32 + sy.k2_off, n2, wj, GJ);
    k1.start(a.fac32 + sy.k1_off, n1, wi, GI);
    auto row_of = [&](int ta) { return 16 * (wi + GI * ta) + lr; };
    auto col_of = [&](int tb) { return 16 * (wj + GJ * tb) + 4 * lq; };
    auto in = [&](int ta, int tb, int v) { return row_of(ta) < n1 && col_of(tb) + v < n2; };

    // scalars (read by every thread; only thread 0 writes them back)
    double rho = stp->rho, beta = stp->beta;
    const double tol2 = stp->tol2, delta = stp->delta, rmax = stp->rmax;
    int iters = stp->iters;
    const int max_iters = stp->max_iters;
    int status = stp->status, active = 1, need_update = 0;

    floatx4 x[WI][WJ], r[WI][WJ], p[WI][WJ];
#pragma unroll
    for (int ta = 0; ta < WI; ++ta)
#pragma unroll
        for (int tb = 0; tb < WJ; ++tb)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const bool ok = in(ta, tb, v);
                const int64_t e = base + (ok ? (int64_t)row_of(ta) * n2 + col_of(tb) + v : 0);
                x[ta][tb][v] = ok ? a.x[e] : 0.f;
                r[ta][tb][v] = ok ? a.r[e] : 0.f;
                p[ta][tb][v] = ok ? a.p[e] : 0.f;
            }

    for (;;) {
        k2.load(0);
        const float bf = (float)beta;
#pragma unroll
        for (int ta = 0; ta < WI; ++ta)
#pragma unroll
            for (int tb = 0; tb < WJ; ++tb) {
#pragma unroll
                for (int v = 0; v < 4; ++v) p[ta][tb][v] = __builtin_fmaf(bf, p[ta][tb][v], r[ta][tb][v]);
                if (ta < na && tb < nb) *(floatx4*)(Ps + row_of(ta) * RPS + col_of(tb)) = p[ta][tb];
            }
        __syncthreads();                                    // P complete
        floatx4 acc[WI][WJ];
#pragma unroll
        for (int ta = 0; ta < WI; ++ta)
#pragma unroll
            for (int tb = 0; tb < WJ; ++tb) acc[ta][tb] = floatx4{0, 0, 0, 0};
        // T = P K2^T (A: rows of P, B: rows of K2)
        for (int u = 0; u < t2; ++u) {
            FactorRows<WJ> now = k2;
            now.cut(16 * u);
            k2.load(u + 1 < t2 ? 16 * (u + 1) : 0);         // a step ahead
            floatx4 pa[WI];
#pragma unroll
            for (int ta = 0; ta < WI; ++ta) pa[ta] = *(const floatx4*)(Ps + row_of(ta) * RPS + 16 * u + 4 * lq);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ta = 0; ta < WI; ++ta)
#pragma unroll
                for (int tb = 0; tb < WJ; ++tb)
                    if (ta < na && tb < nb) acc[ta][tb] = mma4(pa[ta], now.v[tb], acc[ta][tb]);
        }
        k1.load(0);
        // accumulator element v of a lane: row 16 (wi + GI a) + 4 lq + v, column 16 (wj + GJ b) + lr
#pragma unroll
        for (int ta = 0; ta < WI; ++ta)
#pragma unroll
            for (int tb = 0; tb < WJ; ++tb)
                if (ta < na && tb < nb)
                    *(floatx4*)(Ts + (16 * (wj + GJ * tb) + lr) * RPS + 16 * (wi + GI * ta) + 4 * lq) = acc[ta][tb];
        __syncthreads();                                    // T^T complete
#pragma unroll
        for (int ta = 0; ta < WI; ++ta)
#pragma unroll
            for (int tb = 0; tb < WJ; ++tb) acc[ta][tb] = floatx4{0, 0, 0, 0};
        // Q^T = T^T K1^T (A: rows of T^T, B: rows of K1)
        for (int u = 0; u < t1; ++u) {
            FactorRows<WI> now = k1;
            now.cut(16 * u);
            k1.load(u + 1 < t1 ? 16 * (u + 1) : 0);
            floatx4 tt[WJ];
#pragma unroll
            for (int tb = 0; tb < WJ; ++tb)
                tt[tb] = *(const floatx4*)(Ts + (16 * (wj + GJ * tb) + lr) * RPS + 16 * u + 4 * lq);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int ta = 0; ta < WI; ++ta)
#pragma unroll
                for (int tb = 0; tb < WJ; ++tb)
                    if (ta < na && tb < nb) acc[ta][tb] = mma4(tt[tb], now.v[ta], acc[ta][tb]);
        }
        // q = K1 T + (sigma2 + d) p;  mu = p.q
        double mu_l = 0.0;
#pragma unroll
        for (int ta = 0; ta < WI; ++ta)
#pragma unroll
            for (int tb = 0; tb < WJ; ++tb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const bool ok = in(ta, tb, v);
                    const float d = dgv && ok ? dgv[row_of(ta) * n2 + col_of(tb) + v] : 0.f;
                    const float pe = p[ta][tb][v];
                    const float qv = ok ? acc[ta][tb][v] + (s2 + d) * pe : 0.f;
                    acc[ta][tb][v] = qv;
                    mu_l += (double)pe * (double)qv;
                }
        const double mu = block_sum_once<kResWaves>(mu_l, red_pq);
        if (!(mu > 0.0) || !finite_d(mu)) {
            status = finite_d(mu) ? COLA_ERR_NOT_SPD : COLA_ERR_NONFINITE;
            active = 0;
            break;
        }
        const float af = (float)(rho / mu);
        double rho_l = 0.0;
#pragma unroll
        for (int ta = 0; ta < WI; ++ta)
#pragma unroll
            for (int tb = 0; tb < WJ; ++tb)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    x[ta][tb][v] = __builtin_fmaf(af, p[ta][tb][v], x[ta][tb][v]);
                    r[ta][tb][v] = __builtin_fmaf(-af, acc[ta][tb][v], r[ta][tb][v]);
                    rho_l += (double)r[ta][tb][v] * (double)r[ta][tb][v];
                }
        const double rn = block_sum_once<kResWaves>(rho_l, red_rr);
        ++iters;
        bool stop = false;
        if (!finite_d(rn)) {
            status = COLA_ERR_NONFINITE;
            active = 0;
            stop = true;
        } else if (rn <= tol2) {                            // pause; the FP64 residual decides
            need_update = 1;
            active = 0;
            stop = true;
        } else if (iters >= max_iters) {
            status = COLA_NOT_CONVERGED;
            active = 0;
            stop = true;
        } else if (rn < delta * delta * rmax * rmax) {
            need_update = 1;
            stop = true;
        }
        beta = rn / rho;
        rho = rn;
        if (stop) break;
    }
    // write the state back
#pragma unroll
    for (int ta = 0; ta < WI; ++ta)
#pragma unroll
        for (int tb = 0; tb < WJ; ++tb)
#pragma unroll
            for (int v = 0; v < 4; ++v)
                if (in(ta, tb, v)) {
                    const int64_t e = base + (int64_t)row_of(ta) * n2 + col_of(tb) + v;
                    a.x[e] = x[ta][tb][v];
                    a.r[e] = r[ta][tb][v];
                    a.p[e] = p[ta][tb][v];
                }
    if (tid == 0) {
        stp->rho = rho;
        stp->beta = beta;
        stp->iters = iters;
        stp->status = status;
        stp->need_update = need_update;
        if (!active) {
            stp->active = 0;
            atomicSub(&a.cnt->num_active, 1);
        }
    }
    __syncthreads();
}

// FP64 residual of one item: fold the FP32 iterate into the FP64 solution,
// r = b - (K1 X K2^T + (sigma2 + d) x) with the FP64 factors, r_lo = r; returns
// ||r||^2 in every thread.
// Both mode products run on the FP64 matrix cores (v_mfma_f64_16x16x4f64;
// lane l supplies A[l % 16][l / 16] and B[l / 16][l % 16], accumulator
// element v sits at row 4 v + l / 16, column l % 16).  X stays in LDS (padded rows, zero beyond the
// system), the factors and T = X K2^T come from L2.  Each wave computes groups of 1 x 4 output
// tiles (16 x 64) that share the A fragment.

__device__ inline doublex4 mma_f64(double a, double b, doublex4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}

template <int WAVES>
__device__ inline double resident_residual(const ResArgs& a, int item, double* Xs, double* red) {
    constexpr int kThr = 64 * WAVES;
    const ResSys sy = a.sys[item / a.nrhs];
    const int rhs = item % a.nrhs;
    const int n1 = sy.n1, n2 = sy.n2;
    const int64_t base = (int64_t)a.nrhs * sy.vec_off + (int64_t)rhs * sy.n;
    const double* K1 = a.fac64 + sy.k1_off;
    const double* K2 = a.fac64 + sy.k2_off;
    const double* dgv = sy.diag_off >= 0 ? a.diag64 + sy.diag_off : nullptr;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lk = lane >> 4;
    const int n1p = (n1 + 15) & ~15, n2p = (n2 + 15) & ~15;       // 16 x 16 tile extents
    // fold the FP32 correction into x64 and stage X (zero in the padding)
    for (int e = tid; e < n1p * n2p; e += kThr) {
        const int row = e / n2p, col = e % n2p;
        double v = 0.0;
        if (row < n1 && col < n2) {
            const int64_t g = base + (int64_t)row * n2 + col;
            v = a.x64[g] + (double)a.x[g];
            a.x64[g] = v;
            a.x[g] = 0.f;
        }
        Xs[row * PX + col] = v;
    }
    __syncthreads();
    const int nt1 = n1p / 16, nt2 = n2p / 16, ng2 = (nt2 + 3) / 4;
    // T[i][j] = sum_l X[i][l] K2[j][l]
    for (int g = wave; g < nt1 * ng2; g += WAVES) {
        const int i0 = (g / ng2) * 16, j0 = (g % ng2) * 64;
        doublex4 acc[4] = {};
        for (int k = 0; k < n2p; k += 4) {
            const int kk = k + lk;
            const double av = Xs[(i0 + lr) * PX + kk];
            double bv[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int col = j0 + 16 * t + lr;
                bv[t] = (col < n2 && kk < n2) ? K2[(int64_t)col * n2 + kk] : 0.0;
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = mma_f64(av, bv[t], acc[t]);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = i0 + 4 * v + lk, col = j0 + 16 * t + lr;
                if (row < n1 && col < n2) a.t64[base + (int64_t)row * n2 + col] = acc[t][v];
            }
    }
    __syncthreads();                                    // T complete
    // q = K1 T + (sigma2 + d) x,  r = b - q
    double rr = 0.0;
    for (int g = wave; g < nt1 * ng2; g += WAVES) {
        const int i0 = (g / ng2) * 16, j0 = (g % ng2) * 64;
        doublex4 acc[4] = {};
        const int arow = i0 + lr;
        for (int k = 0; k < n1p; k += 4) {
            const int kk = k + lk;
            const double av = (arow < n1 && kk < n1) ? K1[(int64_t)arow * n1 + kk] : 0.0;
            double bv[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                const int col = j0 + 16 * t + lr;
                bv[t] = (col < n2 && kk < n1) ? a.t64[base + (int64_t)kk * n2 + col] : 0.0;
            }
#pragma unroll
            for (int t = 0; t < 4; ++t) acc[t] = mma_f64(av, bv[t], acc[t]);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int row = i0 + 4 * v + lk, col = j0 + 16 * t + lr;
                if (row < n1 && col < n2) {
                    const int64_t e = (int64_t)row * n2 + col;
                    const double dg = sy.sigma2 + (dgv ? dgv[e] : 0.0);
                    const double rv = a.b64[base + e] - (acc[t][v] + dg * Xs[row * PX + col]);
                    a.r[base + e] = (float)rv;
                    rr += rv * rv;
                }
            }
    }
    return block_sum_once<WAVES>(rr, red);
}

// Every item from the queue to its end: iterations until it asks for an FP64 residual, the residual
// and the reliable-update decision, and on until it is finished (or max_rounds residuals were formed).
__global__ __launch_bounds__(kResThreads, 2) void k_resident_cg(ResArgs a) {
    __shared__ __attribute__((aligned(16))) char smem[kResLds];
    float* Ps = (float*)smem;                  // direction P
    float* Ts = Ps + kResMax * RPS;            // (P K2^T)^T
    __shared__ double red_pq[kResWaves];       // slots of the p.q sums
    __shared__ double red_rr[kResWaves];       // slots of the r.r sums (every other barrier of the
                                               // iteration lies between one sum's reads and its next write)
    __shared__ int s_item;
    for (;;) {
        if (threadIdx.x == 0) s_item = (int)atomicAdd(a.queue, 1u);
        __syncthreads();
        const int q = s_item;
        __syncthreads();
        if (q >= a.nitems) break;
        const int item = a.order[q];
        if (!a.st[item].active) continue;
        // four wave columns along one mode, two along the other: the deal whose fullest SIMD has fewer tiles
        const ResSys& sy = a.sys[item / a.nrhs];
        const int t1 = (sy.n1 + 15) / 16, t2 = (sy.n2 + 15) / 16;
        const bool wide = (t1 + 3) / 4 * t2 <= (t2 + 3) / 4 * t1;
        for (int round = 0; round < a.max_rounds; ++round) {
            if (wide) resident_item<2, 4>(a, item, Ps, Ts, red_pq, red_rr);
            else resident_item<4, 2>(a, item, Ps, Ts, red_pq, red_rr);
            if (!a.st[item].need_update) break;            // the iteration limit, or a breakdown
            const double rr = resident_residual<kResWaves>(a, item, (double*)smem, red_rr);
            if (threadIdx.x == 0) {
                a.st[item].rho_true = rr;
                reliable_finish(a.st[item], a.cnt);
            }
            __syncthreads();
            if (!a.st[item].active) break;
        }
    }
}

// Final pass: the true residual of the items without a certified one (status not OK); a converged
// item was certified by its last update and its x has not changed since.
constexpr int kResidWaves = 16;
__global__ __launch_bounds__(64 * kResidWaves) void k_resident_final(ResArgs a) {
    __shared__ double Xs[kResMax * PX];
    __shared__ double red[kResidWaves];
    if (a.st[blockIdx.x].status == COLA_OK) return;
    const double rr = resident_residual<kResidWaves>(a, blockIdx.x, Xs, red);
    if (threadIdx.x == 0) a.st[blockIdx.x].rho_true = rr;
}


hipError_t launch_resident_prepare(const ResArgs& a, double tol, int max_iters, double delta, hipStream_t s) {
    hipLaunchKernelGGL(k_resident_prepare, dim3(a.nitems), dim3(kThreads), 0, s, a, tol, max_iters, delta);
    return hipGetLastError();
}
hipError_t launch_resident_cg(const ResArgs& a, int grid, hipStream_t s) {
    hipLaunchKernelGGL(k_resident_cg, dim3(grid), dim3(kResThreads), 0, s, a);
    return hipGetLastError();
}
hipError_t launch_resident_final(const ResArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(k_resident_final, dim3(a.nitems), dim3(64 * kResidWaves), 0, s, a);
    return hipGetLastError();
}

}  // namespace cola

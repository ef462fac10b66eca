// Mode products of the Kronecker MVM in FP64 and FP32 (one mode per pass).
//
//   ROWS (last mode):   Y[g, i]    = sum_l X[g, l] K[i, l]      (g: all leading indices)
//   COLS (other modes): Y[g, i, b] = sum_l K[i, l] X[g, l, b]   (b: trailing indices)
//
// Each is a batched GEMM with a short inner dimension (the mode size, tens to a
// few hundred): a block walks few k slices, so it is bound by the latency of its
// loads unless they overlap the products.  Two slices are on their way in
// registers while a third, in one of two LDS stages, is multiplied (one barrier
// per slice); the loads carry no branches, because a branch makes the compiler
// wait for everything in flight.  Rows and panels are loaded as 16-byte vectors
// at the elements' own alignment (mode sizes are arbitrary).  Four waves of
// (16 WM) x (16 WN) outputs each on 16x16x4 MFMAs; k runs upwards in steps of
// four, so products do not depend on the tile.  The epilogues work straight from
// the accumulators.
//
// Kernel times (rocprofv3), with one slice staged after the other, element loads
// where a row was not 16-byte aligned and the epilogue through LDS, and now:
// 97 x 101 x 89, 4 right-hand sides, FP32: last / middle / first mode 29 / 45 / 47
// -> 15 / 22 / 23 us; 91 x 75 x 61, 4 right-hand sides, FP64 CG: 30 / 33 / 78 ->
// 12 / 13 / 20 us; 200 x 180, 16 right-hand sides, FP64 CG: 19 / 54 -> 10 / 13 us.
#include "modepass.h"

#include <algorithm>
#include <type_traits>

#include "modeslice.h"

namespace cola {
namespace {

struct ModeF64 {
    using V = double; using Acc = doublex4;
    typedef double Vec __attribute__((ext_vector_type(2)));                     // 16 bytes
    typedef double VecU __attribute__((ext_vector_type(2), aligned(8)));        // the same at element alignment
    static constexpr int VW = 2, KT = 16, NPAD = 16;     // 128-byte k slices; panel pitch 32 (mod 64) banks
};
struct ModeF32 {
    using V = float; using Acc = floatx4;
    typedef float Vec __attribute__((ext_vector_type(4)));
    typedef float VecU __attribute__((ext_vector_type(4), aligned(4)));
    static constexpr int VW = 4, KT = 32, NPAD = 16;
};

// acc += A-row fragment x B-column fragment.  FP64: element v of a lane is row 4 v + lane / 16,
// column lane % 16.  FP32: the product is formed transposed, so a lane holds four consecutive
// columns 4 (lane / 16) + v of row lane % 16.
__device__ inline doublex4 mode_mma(double a, double b, doublex4 c) {
    return __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, 0, 0, 0);
}
__device__ inline floatx4 mode_mma(float a, float b, floatx4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x4f32(b, a, c, 0, 0, 0);
}

// Right-hand side of batch or row i (a 32-bit division wherever the numbers allow it).
__device__ inline int64_t rhs_of(const PassArgs& a, int64_t i) {
    if (a.G <= 0x7fffffff) return (uint32_t)i / (uint32_t)a.a_per_rhs;
    return i / a.a_per_rhs;
}

// Block index with the blocks of one XCD contiguous (blocks go to the 8 XCDs round robin), so
// that the tiles that share an input panel share an L2.
__device__ inline uint32_t xcd_order(uint32_t b, uint32_t T) {
    const uint32_t q = T / 8, r = T % 8, x = b % 8;
    return x * q + (x < r ? x : r) + b / 8;
}

// Waves per SIMD to leave registers for: as many blocks as the LDS stages allow.
constexpr int mode_waves(int wm, int wn) { return wm + wn <= 4 ? 4 : (wm + wn <= 5 ? 3 : (wm * wn <= 8 ? 2 : 1)); }

// ROWS or COLS layout; PNEW (ROWS): the vector operand is R + beta X; EK (COLS): the kind of epilogue,
// 0 EPI_STORE, 1 one with vector operands, 2 EPI_EIG; GENERAL: 64-bit indexes and
// element loads, for inputs of fewer elements than one vector and tiles that span 2 GB.
template <class P, int WM, int WN, bool ROWS, bool PNEW, int EK, bool GENERAL>
__global__ __launch_bounds__(kThreads, mode_waves(WM, WN)) void k_mode(PassArgs a, uint32_t nMt, uint32_t nNt, uint32_t total) {
    using V = typename P::V; using Acc = typename P::Acc; using Vec = typename P::Vec; using VecU = typename P::VecU;
    constexpr int MT = 32 * WM, NT = 32 * WN, VW = P::VW;
    constexpr int KT = P::KT;
    constexpr int KP = KT + VW;                              // pitch of a k-contiguous row: 4 (mod 64) banks
    constexpr int NTP = NT + P::NPAD;                        // pitch of a COLS panel row
    constexpr int A_EL = MT * KP, B_EL = ROWS ? NT * KP : KT * NTP;
    constexpr bool F64 = sizeof(V) == 8, FULL = EK == 1;
    __shared__ __attribute__((aligned(16))) V lds[2 * (A_EL + B_EL)];
    __shared__ double red[4];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1, lr = lane & 15, lq = lane >> 4;
    const int nk = a.nk;

    uint32_t L = xcd_order(blockIdx.x, total);
    int64_t g = 0, m0, n0;
    int tout;
    uint32_t mt, nt;
    if constexpr (ROWS) {                                    // the factor tiles of one row panel together
        nt = L % nNt; L /= nNt;
        mt = L % nMt; tout = (int)(L / nMt);
        m0 = (int64_t)mt * MT;
        n0 = (int64_t)nt * NT;
        if (a.gate) {
            const int64_t last = (m0 + MT < a.G ? m0 + MT : a.G) - 1;
            bool any = false;
            for (int64_t r = rhs_of(a, m0); r <= rhs_of(a, last); ++r) any |= a.gate[r * a.gate_stride] != 0;
            if (!any) return;
        }
    } else {                                                 // the factor tiles of one column panel together
        mt = L % nMt; L /= nMt;
        nt = L % nNt; L /= nNt;
        g = (int64_t)(L % (uint32_t)a.G); tout = (int)(L / (uint32_t)a.G);
        m0 = (int64_t)mt * MT;
        n0 = (int64_t)nt * NT;
        if (a.gate && a.gate[rhs_of(a, g) * a.gate_stride] == 0) return;
    }
    const int64_t Mrows = ROWS ? a.G : nk;                   // rows and columns of the output matrix
    const int64_t Ncols = ROWS ? nk : a.B;
    // This thread's vectors, as 32-bit byte offsets from a uniform base that moves from slice to slice
    // (modeslice.h says where they lie and why they stay inside the input).  Nothing branches between a
    // slice's loads (a branch would make the compiler wait for the loads in flight).  What the clamps of
    // the last slice moved, and what lies beyond nk, is put right on the way to LDS.
    constexpr int ES = sizeof(V);
    using Slices = ModeSlices<VW, KT, WM, WN, ROWS>;
    const Slices sl{nk, a.B, a.G, m0, n0, g};
    constexpr int AV = Slices::AV, BV = Slices::BV, XV = Slices::XV, FV = Slices::FV;
    constexpr int RQ = Slices::RQ, PQ = Slices::PQ;
    const int k_last = sl.k_last();                          // k0 of a term's last slice
    const int arow0 = sl.row(tid, 0), akc = sl.row_k(tid);   // k-contiguous vector q: row arow0 + q RQ
    const int bk0 = sl.panel_k(tid, 0), bn = sl.panel_col(tid);          // panel vector q: k bk0 + q PQ
    const int64_t x_end = sl.x_end(GENERAL ? 1 : VW), x_end_last = sl.x_end_last(GENERAL ? 1 : VW);
    const int64_t xstep = sl.x_step(), to_last = sl.x_to_last();
    const int steps = sl.slices() * a.nsum;                  // k slices of all terms
    uint32_t xoff[XV], xlast[XV], foff[FV];
#pragma unroll
    for (int q = 0; q < XV; ++q) {
        xoff[q] = (uint32_t)(sl.x_at(tid, q) * ES);
        xlast[q] = (uint32_t)((sl.x_last(tid, q) + VW) * ES);            // from VW elements before it
    }
#pragma unroll
    for (int q = 0; q < FV; ++q) foff[q] = (uint32_t)(sl.f_at(tid, q) * ES);
    double beta[PNEW ? AV : 1];
    if constexpr (PNEW) {
#pragma unroll
        for (int q = 0; q < AV; ++q) beta[q] = a.cg[rhs_of(a, m0 + sl.row_at(sl.row(tid, q), m0, a.G))].beta;
    }
    const bool tail = sl.x_clamped();                        // some vector of the last slice was read early
    const bool idle = sl.x_idle_early();

    struct Slice { Vec a[AV], r[PNEW ? AV : 1], b[BV]; };
    auto ldv = [&](const char* base, uint32_t off) -> Vec { return *(const VecU*)(base + off); };
    // GENERAL: 64-bit indexes, by elements
    auto ld_elem = [&](const V* base, int64_t i, int64_t end) -> Vec {
        Vec v;
#pragma unroll
        for (int c = 0; c < VW; ++c) v[c] = base[i + c < end ? i + c : end];
        return v;
    };
    // the slice the next load takes: bases of its operands, k0
    const int64_t t0 = a.nsum > 1 ? 0 : tout;
    const char* Fl = (const char*)((const V*)a.K + t0 * a.k_tstride + (ROWS ? n0 : m0) * nk);
    const char* Xl = (const char*)((const V*)a.X + t0 * a.x_tstride + sl.x_base());
    const char* Rl = (const char*)((const V*)a.R + t0 * a.x_tstride + sl.x_base());
    int kl = 0, left = steps;
    auto load_slice = [&](Slice& v) {
        // past the last slice every lane loads one address, or the last slice again (nothing uses it)
        const uint32_t keep = left > 0 || !idle ? 0xffffffffu : 0u;
        const bool last = kl == k_last;
        auto& vx = [&]() -> auto& { if constexpr (ROWS) return v.a; else return v.b; }();
        auto& vf = [&]() -> auto& { if constexpr (ROWS) return v.b; else return v.a; }();
        if constexpr (GENERAL) {
            const int64_t end = x_end - (int64_t)(kl / KT) * xstep;
#pragma unroll
            for (int q = 0; q < XV; ++q) {
                const int64_t i = left > 0 ? (last ? sl.x_last_wanted(tid, q) : sl.x_at(tid, q)) : 0;
                vx[q] = ld_elem((const V*)Xl, i, end);
                if constexpr (PNEW) v.r[q] = ld_elem((const V*)Rl, i, end);
            }
#pragma unroll
            for (int q = 0; q < FV; ++q)
                vf[q] = *(const VecU*)((const V*)Fl + (left > 0 ? sl.f_at(tid, q) : 0));
        } else {
            const int back = last ? VW * ES : 0;
#pragma unroll
            for (int q = 0; q < XV; ++q) {
                const uint32_t o = (last ? xlast[q] : xoff[q]) & keep;
                vx[q] = ldv(Xl - back, o);
                if constexpr (PNEW) v.r[q] = ldv(Rl - back, o);
            }
#pragma unroll
            for (int q = 0; q < FV; ++q) vf[q] = ldv(Fl, foff[q] & keep);
        }
        if (--left <= 0) return;                             // the bases stay on the last slice
        kl += KT;
        if (!last) {
            Fl += KT * ES;
            Xl += xstep * ES;
            if constexpr (PNEW) Rl += xstep * ES;
        } else {                                             // the next term
            Fl += (a.k_tstride - k_last) * ES;
            Xl += (a.x_tstride - to_last) * ES;
            if constexpr (PNEW) Rl += (a.x_tstride - to_last) * ES;
            kl = 0;
        }
    };
    // a vector read `sh` elements early: its elements back in place
    auto unshift = [&](Vec& v, int64_t sh) {
        if (sh <= 0) return;
#pragma unroll
        for (int c = 0; c < VW; ++c) {
            V w = (V)0;
#pragma unroll
            for (int e = c; e < VW; ++e) w = e - c == sh ? v[e] : w;
            v[c] = w;
        }
    };
    // the loaded slice: direction update and zeros beyond nk, then into its LDS stage
    int ks = 0;                                              // k0 of the slice stored next
    auto store_slice = [&](Slice& v, V* As, V* Bs) {
        const int k0 = ks;
        ks = k0 == k_last ? 0 : k0 + KT;
        if (!GENERAL && tail && k0 == k_last) {
#pragma unroll
            for (int q = 0; q < XV; ++q) {
                const int64_t sh = sl.x_last_wanted(tid, q) - x_end_last;
                if constexpr (ROWS) unshift(v.a[q], sh);
                else unshift(v.b[q], sh);
                if constexpr (PNEW) unshift(v.r[q], sh);
            }
        }
        if constexpr (PNEW) {
#pragma unroll
            for (int q = 0; q < AV; ++q)
#pragma unroll
                for (int c = 0; c < VW; ++c) v.a[q][c] = pnew_of(v.r[q][c], v.a[q][c], beta[q]);
        }
        if (k0 + KT > nk) {
#pragma unroll
            for (int c = 0; c < VW; ++c) {
                const bool out = k0 + akc + c >= nk;
#pragma unroll
                for (int q = 0; q < AV; ++q) v.a[q][c] = out ? (V)0 : v.a[q][c];
                if constexpr (ROWS) {
#pragma unroll
                    for (int q = 0; q < BV; ++q) v.b[q][c] = out ? (V)0 : v.b[q][c];
                }
            }
            if constexpr (!ROWS) {
#pragma unroll
                for (int q = 0; q < BV; ++q)
#pragma unroll
                    for (int c = 0; c < VW; ++c) v.b[q][c] = k0 + bk0 + q * PQ >= nk ? (V)0 : v.b[q][c];
            }
        }
#pragma unroll
        for (int q = 0; q < AV; ++q) *(Vec*)(As + (arow0 + q * RQ) * KP + akc) = v.a[q];
#pragma unroll
        for (int q = 0; q < BV; ++q) {
            if constexpr (ROWS) *(Vec*)(Bs + (arow0 + q * RQ) * KP + akc) = v.b[q];
            else *(Vec*)(Bs + (bk0 + q * PQ) * NTP + bn) = v.b[q];
        }
    };

    Acc acc[WM][WN];
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
        for (int j = 0; j < WN; ++j) acc[i][j] = Acc{0, 0, 0, 0};

    Slice set[2];                                            // slices s and s + 1 on their way
    auto step = [&](auto parity) {
        constexpr int b = decltype(parity)::value;
        V* As = lds + b * (A_EL + B_EL);
        V* Bs = As + A_EL;
        store_slice(set[b], As, Bs);
        // the barrier also covers the other stage: every wave read it before it came here
        __syncthreads();
        load_slice(set[b]);
        __builtin_amdgcn_sched_barrier(0);                   // the loads stay ahead of the products
#pragma unroll
        for (int kk = 0; kk < KT; kk += 4) {
            V av[WM], bv[WN];
#pragma unroll
            for (int i = 0; i < WM; ++i) av[i] = As[((wm * WM + i) * 16 + lr) * KP + kk + lq];
#pragma unroll
            for (int j = 0; j < WN; ++j) {
                if constexpr (ROWS) bv[j] = Bs[((wn * WN + j) * 16 + lr) * KP + kk + lq];
                else bv[j] = Bs[(kk + lq) * NTP + (wn * WN + j) * 16 + lr];
            }
#pragma unroll
            for (int i = 0; i < WM; ++i)
#pragma unroll
                for (int j = 0; j < WN; ++j) acc[i][j] = mode_mma(av[i], bv[j], acc[i][j]);
        }
    };
    load_slice(set[0]);
    load_slice(set[1]);
    for (int s = 0; s + 1 < steps; s += 2) {
        step(std::integral_constant<int, 0>{});
        step(std::integral_constant<int, 1>{});
    }
    if (steps & 1) step(std::integral_constant<int, 0>{});

    // ---- epilogue, straight from the accumulators: FP64 lanes hold one column of four rows (128-byte
    // lines across the lanes), FP32 lanes four consecutive columns of one row ----
    double dot = 0.0;
    V* Y = (V*)a.Y + (int64_t)tout * a.y_tstride + (ROWS ? 0 : g * (int64_t)nk * a.B);
    const int epi = FULL ? a.epi : (int)EPI_STORE;
    constexpr bool need_p = FULL;
    const bool need_r = epi == EPI_CG || epi == EPI_RESID || epi == EPI_RESID_CG;
    const V* Ep = need_p ? (const V*)a.Ep + g * (int64_t)nk * a.B : nullptr;
    const V* Er = need_r ? (const V*)a.Er + g * (int64_t)nk * a.B : nullptr;
    V* Po = epi == EPI_CG ? (V*)a.Epout + g * (int64_t)nk * a.B : nullptr;
    const V* Dv = need_p ? (const V*)a.dvec : nullptr;
    const double beta_e = epi == EPI_CG ? a.cg[g].beta : 0.0;
    const V s2 = (V)a.sigma2;
    constexpr int CW = F64 ? 1 : 4;                          // consecutive columns per access
    constexpr int NA = 4 / CW;                               // accesses per accumulator tile
    const bool full = n0 + NT <= Ncols && m0 + MT <= Mrows;
    constexpr int JB = !FULL || !F64 ? WN : (WN > 2 ? 2 : 1);           // tiles whose operands are in registers at once
#pragma unroll
    for (int ij = 0; ij < WM * WN; ij += JB) {
        const int i = ij / WN, j0 = ij % WN;
        const int64_t mb = m0 + (wm * WM + i) * 16;
        V u[JB][4], w[JB][4], d[JB][4];
        auto at = [&](int j, int x, int64_t& m, int64_t& n) {
            m = mb + (F64 ? 4 * x + lq : lr);
            n = n0 + (wn * WN + j0 + j) * 16 + (F64 ? lr : 4 * lq);
        };
        auto ldw = [&](const V* p, int64_t m, int64_t n, V* o) {
            if constexpr (CW == 1) {
                const int64_t mc = full ? m : (m < Mrows ? m : Mrows - 1), nc = full ? n : (n < Ncols ? n : Ncols - 1);
                o[0] = p[mc * Ncols + nc];
            } else if (full || (m < Mrows && n + CW <= Ncols)) {
                const VecU v = *(const VecU*)(p + m * Ncols + n);
#pragma unroll
                for (int c = 0; c < CW; ++c) o[c] = v[c];
            } else {
                const int64_t mc = m < Mrows ? m : Mrows - 1;
#pragma unroll
                for (int c = 0; c < CW; ++c) o[c] = p[mc * Ncols + (n + c < Ncols ? n + c : Ncols - 1)];
            }
        };
        auto stw = [&](V* p, int64_t m, int64_t n, const V* o) {
            if constexpr (CW == 1) {
                if (full || (m < Mrows && n < Ncols)) p[m * Ncols + n] = o[0];
            } else if (full || (m < Mrows && n + CW <= Ncols)) {
                VecU v;
#pragma unroll
                for (int c = 0; c < CW; ++c) v[c] = o[c];
                *(VecU*)(p + m * Ncols + n) = v;
            } else if (m < Mrows) {
#pragma unroll
                for (int c = 0; c < CW; ++c)
                    if (n + c < Ncols) p[m * Ncols + n + c] = o[c];
            }
        };
        if (need_p) {                                        // all loads before the first use
#pragma unroll
            for (int j = 0; j < JB; ++j)
#pragma unroll
                for (int x = 0; x < NA; ++x) {
                    int64_t m, n;
                    at(j, x, m, n);
                    ldw(Ep, m, n, &u[j][x * CW]);
                    if (need_r) ldw(Er, m, n, &w[j][x * CW]);
                    if (Dv) ldw(Dv, m, n, &d[j][x * CW]);
                }
        }
#pragma unroll
        for (int j = 0; j < JB; ++j)
#pragma unroll
            for (int x = 0; x < NA; ++x) {
                int64_t m, n;
                at(j, x, m, n);
                V out[CW], pn[CW];
#pragma unroll
                for (int c = 0; c < CW; ++c) {
                    const int e = x * CW + c;
                    const V val = (V)acc[i][j0 + j][e];
                    const bool in = full || (m < Mrows && n + c < Ncols);
                    if constexpr (EK == 2) {                 // the order of products of k_eig_scale
                        const uint32_t nc = (uint32_t)(n < Ncols ? n : Ncols - 1), n3 = (uint32_t)a.lam_n3;
                        double lam = a.lam[0][m < Mrows ? m : Mrows - 1] * a.lam[1][nc / n3];
                        if (a.lam[2]) lam *= a.lam[2][nc % n3];
                        out[c] = val / (lam + a.lam_shift);
                        continue;
                    }
                    if constexpr (!FULL) {
                        out[c] = val;
                        continue;
                    }
                    const V dg = s2 + (Dv ? d[j][e] : (V)0);
                    if (epi == EPI_CG) {
                        pn[c] = pnew_of(w[j][e], u[j][e], beta_e);
                        out[c] = val + dg * pn[c];
                        if (in) dot += (double)pn[c] * (double)out[c];
                    } else if (epi == EPI_MATVEC) {
                        out[c] = val + dg * u[j][e];
                    } else {
                        out[c] = w[j][e] - (val + dg * u[j][e]);
                        if (in) dot += (double)out[c] * (double)out[c];
                    }
                }
                stw(Y, m, n, out);
                if (epi == EPI_CG) stw(Po, m, n, pn);
            }
    }

    if constexpr (FULL) {
        if (epi == EPI_CG || epi == EPI_RESID || epi == EPI_RESID_CG) {
            const double s = block_sum(dot, red);
            double tot;
            if (last_block_reduce(s, a.partials + g * a.part_stride, a.counters + g * kCounterStride, (int)(nNt * nMt),
                                  (int)(nt + nNt * mt), &tot, red) && tid == 0) {
                if (epi == EPI_CG) {
                    CgState& st = a.cg[g];
                    if (!(tot > 0.0) || !finite_d(tot)) {
                        st.status = finite_d(tot) ? COLA_ERR_NOT_SPD : COLA_ERR_NONFINITE;
                        st.active = 0;
                        atomicSub(&a.cnt->num_active, 1);
                    } else {
                        st.alpha = st.rho / tot;
                    }
                } else if (epi == EPI_RESID_CG) {
                    a.cg[g].rho_true = tot;
                } else {
                    outer_residual(a.outer[g], tot, a.cnt);
                }
            }
        }
    }
}

template <class P, int WM, int WN, bool ROWS, bool PNEW, int EK, bool GENERAL>
hipError_t launch_v(const PassArgs& a, hipStream_t s) {
    const int64_t M = ROWS ? a.G : a.nk, N = ROWS ? a.nk : a.B;
    const int64_t nMt = (M + 32 * WM - 1) / (32 * WM), nNt = (N + 32 * WN - 1) / (32 * WN);
    const int64_t total = nMt * nNt * a.nout * (ROWS ? 1 : a.G);
    if (total < 1 || total > 0x7fffffff || (!ROWS && a.G > 0x7fffffff)) return hipErrorInvalidValue;
    hipLaunchKernelGGL((k_mode<P, WM, WN, ROWS, PNEW, EK, GENERAL>), dim3((unsigned)total), dim3(kThreads), 0, s, a,
                       (uint32_t)nMt, (uint32_t)nNt, (uint32_t)total);
    return hipGetLastError();
}

template <class P>
bool needs_general(bool rows, const PassArgs& a) {
    return mode_needs_general<P::VW, P::KT>(rows, a.nk, a.B, a.G, sizeof(typename P::V));
}

template <class P, int WM, int WN, bool GENERAL>
hipError_t launch_cols(const PassArgs& a, hipStream_t s) {
    if (a.epi == EPI_STORE) return launch_v<P, WM, WN, false, false, 0, GENERAL>(a, s);
    if constexpr (sizeof(typename P::V) == 8)
        if (a.epi == EPI_EIG) return launch_v<P, WM, WN, false, false, 2, GENERAL>(a, s);
    if (a.epi == EPI_EIG) return hipErrorInvalidValue;
    return launch_v<P, WM, WN, false, false, 1, GENERAL>(a, s);
}

template <class P, int WM, int WN, bool ROWS>
hipError_t launch_t(const PassArgs& a, hipStream_t s) {
    const bool elem = needs_general<P>(ROWS, a);
    if constexpr (ROWS) {
        if constexpr (WM == 1 && WN == 1)
            if (elem) return a.pnew ? launch_v<P, 1, 1, true, true, 0, true>(a, s)
                                    : launch_v<P, 1, 1, true, false, 0, true>(a, s);
        return a.pnew ? launch_v<P, WM, WN, true, true, 0, false>(a, s)
                      : launch_v<P, WM, WN, true, false, 0, false>(a, s);
    } else {
        if constexpr (WM == 1 && WN == 1)
            if (elem) return launch_cols<P, 1, 1, true>(a, s);
        return launch_cols<P, WM, WN, false>(a, s);
    }
}

// The factor's side of the tile (rows in COLS, columns in ROWS) shrinks to 96 where that still takes
// as few tiles, e.g. one of 96 instead of one of 128 for a mode of 91.
int trim(int w, int64_t nk) {
    return (w == 4 && (nk + 95) / 96 == (nk + 127) / 128) ? 3 : w;
}

template <class P>
hipError_t launch_p(bool rows, const PassArgs& a, TileCfg c, hipStream_t s) {
    if (needs_general<P>(rows, a)) c = TileCfg{1, 1};        // the only tile built that way
    if (rows) {
        const int wn = trim(c.wn, a.nk);
#define COLA_ROWS(M, N) \
    if (c.wm == M && wn == N) return launch_t<P, M, N, true>(a, s);
        COLA_ROWS(1, 1) COLA_ROWS(1, 2) COLA_ROWS(1, 3) COLA_ROWS(1, 4)
        COLA_ROWS(2, 1) COLA_ROWS(2, 2) COLA_ROWS(2, 3) COLA_ROWS(2, 4)
        COLA_ROWS(4, 1) COLA_ROWS(4, 2) COLA_ROWS(4, 3) COLA_ROWS(4, 4)
#undef COLA_ROWS
    } else {
        const int wm = trim(c.wm, a.nk);
#define COLA_COLS(M, N) \
    if (wm == M && c.wn == N) return launch_t<P, M, N, false>(a, s);
        COLA_COLS(1, 1) COLA_COLS(2, 1) COLA_COLS(3, 1) COLA_COLS(4, 1)
        COLA_COLS(1, 2) COLA_COLS(2, 2) COLA_COLS(3, 2) COLA_COLS(4, 2)
        COLA_COLS(1, 4) COLA_COLS(2, 4) COLA_COLS(3, 4) COLA_COLS(4, 4)
#undef COLA_COLS
    }
    return hipErrorInvalidValue;
}

}  // namespace

// Tiles of few outputs load more per product; tiles of many leave CUs without blocks and pad the
// edges.  The cost of a tile is its products, its loads (one row or column panel each) and a fixed
// part, times the number of blocks, of which fewer than four per CU take as long as four; tiles over
// 64 x 64 leave room for fewer blocks on a CU (a factor of 1.3).  Measured (us with the events around
// a launch, 256 CUs): 97 x 8989 outputs, K = 97, 4 batches, FP64: 32x32 37, 64x32 33, 64x64 35, 128x64
// 48; 200 x 180, K = 200, 16 batches, FP64: 32x32 16, 64x32 17, 64x64 20, 128x128 51; 64 x 4096, K =
// 64, 32 batches, FP64: 64x32 45, 64x64 42, 64x128 48; 64 x 64, K = 64, 2048 batches, FP32: 32x32 24,
// 64x32 21, 64x64 21, 128x64 29.
TileCfg mode_tile(bool rows, int64_t nk, int64_t M, int64_t N, int64_t batch) {
    TileCfg best{1, 1};
    double cost = 1e300;
    for (int wm : {1, 2, 4})
        for (int wn : {1, 2, 4}) {
            const int m = rows ? wm : trim(wm, nk), n = rows ? trim(wn, nk) : wn;
            const double blocks = (double)((M + 32 * m - 1) / (32 * m)) * (double)((N + 32 * n - 1) / (32 * n)) *
                                  (double)batch;
            const double c = std::max(blocks, 1024.0) * (m * n + m + n + 1) * (m * n > 4 ? 1.3 : 1.0);
            if (c < cost) {
                cost = c;
                best = TileCfg{wm, wn};
            }
        }
    return best;
}

hipError_t launch_mode_pass(int prec, bool rows, const PassArgs& a, TileCfg cfg, hipStream_t s) {
    return prec == COLA_PREC_FP64 ? launch_p<ModeF64>(rows, a, cfg, s) : launch_p<ModeF32>(rows, a, cfg, s);
}

}  // namespace cola

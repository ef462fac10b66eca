// Where the loads of one tile of a mode product (modepass.hip) lie in its operands.  Plain arithmetic,
// callable on the host: tests/test_mode_slices.py holds every load to its buffer over all small shapes.
#pragma once
#include <stdint.h>

#ifdef __HIPCC__
#define COLA_HD __host__ __device__ inline
#else
#define COLA_HD inline
#endif

namespace cola {

// A block of 256 threads walks the contracted mode (nk) in slices of KT and loads vectors of VW elements:
// the input's tile (ROWS: MT rows of the G x nk input from row m0 on; COLS: the nk x B input of batch g of
// G, columns n0 .. n0 + NT) and the factor's (from row n0 or m0 on).  Offsets are in elements, from a base that
// moves by xstep() from slice to slice.
//
// Rows of the output tile beyond the matrix repeat its last row and columns beyond it hold other
// elements: neither is stored.  What keeps the input's loads inside the input:
//   ROWS  a slice before the last lies inside its row; the last one may pass the row's end.
//   COLS  a vector that starts beyond the row (its columns are not stored) reads column n0 of its own
//         row instead, and one that starts inside passes the row's end by VW - 1 elements at most: a
//         slice before the last has (nk - k_last) B elements after its last row, so only B or a last slice
//         too small for that is left to the element-wise variant (mode_needs_general).
//   the last slice  rows beyond nk repeat row nk - 1, and a vector past the input's end is read early, at
//         the input's last vector (the kernel puts its elements back in place).
//   after the last slice  every lane loads one vector, just before the last slice's base (which may be
//         nearer to the input's end than a vector), or the last slice again where the input starts there.
// Factor vectors may run past the end of their matrix by part of a slice (the factor buffers are padded
// by a slice's 128 bytes).
template <int VW, int KT, int WM, int WN, bool ROWS>
struct ModeSlices {
    static constexpr int THREADS = 256, MT = 32 * WM, NT = 32 * WN;
    static constexpr int RV = KT / VW, RQ = THREADS / RV;    // vectors per k-contiguous row, rows per step of q
    static constexpr int PR = NT / VW, PQ = THREADS / PR;    // COLS: the same of a panel row of NT columns
    static constexpr int AV = MT * RV / THREADS, BV = NT * KT / VW / THREADS;    // vectors per thread and slice
    static constexpr int XV = ROWS ? AV : BV, FV = ROWS ? BV : AV;               // of the input and of the factor

    int nk;
    int64_t B, G;                                            // B: COLS only
    int64_t m0, n0, g;                                       // g: COLS only

    COLA_HD int slices() const { return (int)((uint32_t)(nk + KT - 1) / KT); }
    COLA_HD int k_last() const { return (int)((uint32_t)(nk - 1) / KT * KT); }         // first k of the last slice
    // vector q of a thread: in a k-contiguous row (row of the tile, k of the slice), in a panel (k, column)
    COLA_HD int row(int tid, int q) const { return tid / RV + q * RQ; }
    COLA_HD int row_k(int tid) const { return tid % RV * VW; }
    COLA_HD int panel_k(int tid, int q) const { return tid / PR + q * PQ; }
    COLA_HD int panel_col(int tid) const { return tid % PR * VW; }
    // tile row `r`, clamped to the matrix of `rows` rows whose row `first` is the tile's first
    COLA_HD int64_t row_at(int r, int64_t first, int64_t rows) const {
        const int64_t m = first + r;
        return (m < rows ? m : rows - 1) - first;
    }

    // the input: first slice's base, step between slices, and the last vector of VW elements (GENERAL: the
    // last element) from the first and from the last slice's base
    COLA_HD int64_t x_base() const { return ROWS ? m0 * nk : g * nk * B + n0; }
    COLA_HD int64_t x_step() const { return ROWS ? KT : (int64_t)KT * B; }
    COLA_HD int64_t x_end(int width) const { return (ROWS ? G * nk : G * nk * B) - width - x_base(); }
    COLA_HD int64_t x_to_last() const { return k_last() * (ROWS ? 1 : B); }      // to the last slice's base
    COLA_HD int64_t x_end_last(int width) const { return x_end(width) - x_to_last(); }

    // vector q in a slice before the last
    COLA_HD int64_t x_at(int tid, int q) const {
        if (ROWS) return row_at(row(tid, q), m0, G) * nk + row_k(tid);
        const int col = panel_col(tid);
        return (int64_t)panel_k(tid, q) * B + (n0 + col < B ? col : 0);
    }
    // vector q in the last slice, before and after the clamp to the input's end
    COLA_HD int64_t x_last_wanted(int tid, int q) const {
        if (ROWS) return row_at(row(tid, q), m0, G) * nk + row_k(tid);
        const int k = panel_k(tid, q);
        return (int64_t)(k_last() + k < nk ? k : nk - 1 - k_last()) * B + panel_col(tid);
    }
    COLA_HD int64_t x_last(int tid, int q) const {
        const int64_t w = x_last_wanted(tid, q), e = x_end_last(VW);
        return w < e ? w : e;
    }
    // whether some vector of the last slice may be read early
    COLA_HD bool x_clamped() const {
        return x_end_last(VW) < (ROWS ? (int64_t)(MT - 1) * nk + KT : (int64_t)(nk - 1 - k_last()) * B + NT);
    }
    // the load after the last slice: from a vector before that slice's base, or the last slice's own again
    // where that is before the input (x_idle_at for the thread and vector it is asked for)
    COLA_HD bool x_idle_early() const { return x_base() + x_to_last() >= VW; }
    COLA_HD int64_t x_idle_at(int tid, int q) const { return x_idle_early() ? -VW : x_last(tid, q); }
    // the factor: vector q from row n0 (ROWS) or m0 (COLS) on
    COLA_HD int64_t f_at(int tid, int q) const {
        return row_at(row(tid, q), ROWS ? n0 : m0, nk) * nk + row_k(tid);
    }
};

// Passes for the variant with 64-bit indexes and element loads: fewer elements than one vector, 128 rows (a
// slice of panel rows) that span 2 GB, or panels whose slices before the last have less than a
// vector's tail after them.
template <int VW, int KT>
COLA_HD bool mode_needs_general(bool rows, int64_t nk, int64_t B, int64_t G, int64_t es) {
    if ((rows ? G * nk : G * nk * B) < VW || (128 * nk + 128) * es > 0x7fffffff) return true;
    if (rows) return false;
    const int64_t k_last = (nk + KT - 1) / KT * KT - KT;
    return (KT * B + 128) * es > 0x7fffffff || (k_last > 0 && (nk - k_last) * B < VW - 1);
}

}  // namespace cola

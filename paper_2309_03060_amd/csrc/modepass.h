// Mode products of the Kronecker MVM in FP64 and FP32 (host interface).
#pragma once
#include "contract.h"

namespace cola {

// Tile of a pass with nothing tuned for it: M x N outputs in each of `batch` independent products,
// the factor's mode (nk) along M (COLS) or N (ROWS).
TileCfg mode_tile(bool rows, int64_t nk, int64_t M, int64_t N, int64_t batch);

// One pass of PassArgs (contract.h) in FP64 or FP32; `rows` selects the ROWS layout.
hipError_t launch_mode_pass(int prec, bool rows, const PassArgs& a, TileCfg cfg, hipStream_t s);

}  // namespace cola

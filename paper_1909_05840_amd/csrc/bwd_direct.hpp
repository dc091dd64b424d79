// The backward without a staging area (bwd_direct.hip), as the dispatch in bwd_bf16.hip sees it.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace qb {

struct DirectArgs {
    const uint16_t *dY;
    const int8_t *Xq;
    const uint8_t *packed;
    const float *h, *q0;          // q0: asymmetric ranges (h holds Delta then), else null
    const float *X, *W, *m;       // clamp masks of dX (X) and dW (W with its ranges m), or null
    uint16_t *dX;
    float *dW;
    int T, N, K, rows_per_group;
    float clip, scale;
    // filled by bwd_direct_run
    float rcp_rows;
    int tiles_x, tiles_w, dw_first, quad_ok;
};

// Teams per workgroup (1, 2 or 4) with which a call of this size should take bwd_direct_run, or 0 if the staged path is
// the faster one or the sizes do not fit.
int bwd_direct_teams(int64_t T, int64_t N, int64_t K, bool dx, bool dw);

void bwd_direct_run(DirectArgs g, int teams, int bits, hipStream_t st);

}  // namespace qb

// Row-tile bookkeeping shared by the two batch-1 GEMV kernels.
//
// Work decomposition (both kernels): a "team" of LPR lanes (64 or 32) owns a
// whole weight row at a time.  Lane l of the team owns the groups
// g = i*LPR + l, i < GPL, of every row, so that one load instruction of the
// team reads LPR consecutive 16-byte groups (1 KiB or 512 B of one row), and
// the activation values of those groups stay in the lane's registers for the
// whole kernel.  Teams walk row tiles of U rows in a grid-stride loop and
// fetch the next tile before computing the current one.
#pragma once

#include "nvq_internal.h"

namespace nvq {

// 16 bytes that are read once (weights): a non-temporal load.
__device__ __forceinline__ uint4 stream_load16(const uint4 *p) {
    typedef uint32_t u32x4_nt __attribute__((ext_vector_type(4)));
    const u32x4_nt v = __builtin_nontemporal_load(reinterpret_cast<const u32x4_nt *>(p));
    return make_uint4(v.x, v.y, v.z, v.w);
}

struct RowRef {
    const uint4 *qw;     // first group of the row
    const uint16_t *sc;  // first scale of the row
    void *y;             // output vector of the row's segment
    int32_t *dbg;        // accumulator dump of the row's segment (or nullptr)
    int N;               // rows in the segment
    int n;               // row index inside the segment
    int y_dtype;
    bool valid;
};

// Map a global row number to its segment.  Rows past the end are clamped to
// the last row so that loads stay in bounds; `valid` masks the stores.  SEGS is
// a (possibly address-space qualified) GemvSegs.
template <typename SEGS>
__device__ __forceinline__ RowRef locate_row(SEGS &S, int row, int G) {
    RowRef r;
    r.valid = row < S.total_rows;
    if (!r.valid) row = S.total_rows - 1;
    // select chain instead of indexing: the segment table lives in kernel
    // arguments and a dynamic index would force it through scratch memory
    int first = 0;
    r.qw = S.qw[0];
    r.sc = S.sc[0];
    r.y = S.y[0];
    r.dbg = S.dbg[0];
    r.N = S.N[0];
    r.y_dtype = S.y_dtype[0];
#pragma unroll
    for (int i = 1; i < kMaxSeg; ++i) {
        if (i < S.nseg && row >= S.row_end[i - 1]) {
            first = S.row_end[i - 1];
            r.qw = S.qw[i];
            r.sc = S.sc[i];
            r.y = S.y[i];
            r.dbg = S.dbg[i];
            r.N = S.N[i];
            r.y_dtype = S.y_dtype[i];
        }
    }
    r.n = row - first;
    r.qw += (int64_t)r.n * G;
    r.sc += (int64_t)r.n * G;
    return r;
}

// Resident workgroups per compute unit of the batch-1 kernels (measured on a 295 MB
// layer: 2 -> 3 workgroups 68 -> 60 us, 4 and 6 no better).
constexpr int kM1WgPerCu = 3;

// Rows per tile (1, 2, 4 or 8).  One while every row gets a team of its own that is resident: the
// call is then one trip to memory by as many waves as there are rows (2048 x 2048, W4A16: 2.7 us
// with one, 2.7, 3.6 and 5.3 with two, four and eight; 1024 x 3072 2.9 against 3.7 with two; cold
// weights, W4A8, 2048 x 8192 4.5 against 4.6).  Beyond, with two to four groups per lane, two (4096
// x 4096 4.4 against 4.8 with one and 4.7 with four, 14336 x 4096 9.0, 10.7 and 9.9, 28672 x 4096
// 14.8, 19.8 and 15.8); with one, whose rows are a load each, as many as make every tile resident
// (8192 x 2048 with four 4.5, with two 4.8; 128256 x 2048 with eight 42, with two 47).
static inline int tile_rows(int gpl, int rows, int teams_per_wg) {
    const int most = gpl == 1 ? 8 : gpl <= 4 ? 2 : 1, teams = device_cu_count() * kM1WgPerCu * teams_per_wg;
    int u = 1;
    while (u < most && (rows + u - 1) / u > teams) u *= 2;
    return u;
}

// Whether a call whose sums are added in sixty-four chains (gemv_slice.h) goes to a kernel with
// a wave per row instead of a workgroup per 16 rows.  Up to three tokens and few rows: the row
// tiles leave compute units idle and every one of them takes K by eight waves only, while the
// inputs of a few tokens cost little to read again for every row.  One token (K > 16384), W4A16:
// 16 x 65536 11.8 us against 29.6, 3000 x 16416 10.1 against 11.1, 6000 x 16416 21.3 against
// 21.1, 7000 x 65536 98 against 68, 12000 x 16416 38 against 32.  W4A8, whatever the rows: 16 x
// 65536 9.2 against 24.7, 4200 x 16416 11.6 against 17.2, 8192 x 16416 21.2 against 20.5, 10000
// x 65536 72 against 78, 20000 x 16416 45 against 47 and 20000 x 65536 148 against 176 (both go
// up in steps of 8192 rows; just above a step the row tiles are ahead, 12000 x 16416 33 against
// 28, and a little further on behind again).  Two tokens: 1024 x 16416 9.2 against 10.8 and 8.2
// against 9.4, 2048 x 2720 4.8 against 4.3 and 4.1 against 4.2, 3000 x 16416 15.9 against 11.3
// and 10.1 against 9.8; W4A8 where the scales of a block are not one load (K % 256 != 0), 3000 x
// 3616 5.0 against 5.3, 4200 x 5568 6.6 against 7.5 (a scale per group: 8.1), 5000 x 8256 9.4
// against 10.1, 6100 x 12352 16.2 against 15.3, 6600 x 5600 9.4 against 8.6; where they are, 3072 x
// 8192 6.9 against 6.9; with K beyond 16384 3000 x 20544 14.4 against 12.4, 5000 x 20544 20.5
// against 22.5.  Three: 700 x 8000 6.5 against 6.7 and 5.7 against 6.0, 2048 x 2720 5.6 against
// 4.7, 3000 x 8256 8.7 against 7.3 (W4A8).  Four: 512 x 2720 4.8 against 4.1.
static inline bool gemv_wave_per_row(const GemvSegs &S, int K, int M, int precision, bool per_group) {
    if (!per_group && gemv_mfma_supported(S, K, M)) return false;  // column chains
    const int cus = device_cu_count();
    if (M == 1) return precision == NVQ_W4A8 || S.total_rows <= 16 * cus;
    if (M == 2 && precision == NVQ_W4A8) return S.total_rows <= (K % 256 != 0 && K <= 16384 ? 24 : 8) * cus;
    return M <= 3 && M * S.total_rows <= 8 * cus;
}

// Grid size for a batch-1 GEMV: enough workgroups of `teams_per_wg` teams to
// give every tile a team, at most `wg_per_cu` resident workgroups per
// compute unit (the kernels are grid-stride beyond that).
static inline int gemv_grid(int tiles, int teams_per_wg, int wg_per_cu) {
    int want = (tiles + teams_per_wg - 1) / teams_per_wg;
    const int cus = device_cu_count();
    if (want < 1) want = 1;
    if (want <= cus * wg_per_cu) return want;
    // A whole number k of workgroups per compute unit; the work takes ceil(want / grid)
    // rounds, and a round costs a compute unit k / efficiency(k) (measured: two resident
    // workgroups stream at 0.85, one at 0.6 of the rate of three or more).  1024
    // workgroups' worth of tiles are better served by 512 (two even rounds) than by
    // 768 (two rounds, the second a third full).
    int best = cus;
    double best_cost = 1e30;
    for (int k = 1; k <= wg_per_cu; ++k) {
        const double eff = k == 1 ? 0.6 : k == 2 ? 0.85 : 1.0;
        const int rounds = (want + cus * k - 1) / (cus * k);
        const double cost = rounds * (k / eff);
        if (cost < best_cost) {
            best_cost = cost;
            best = cus * k;
        }
    }
    return best;
}

}  // namespace nvq

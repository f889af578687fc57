// Internal declarations shared by the translation units of libnvq (host side
// and gfx950 device helpers).  Not installed; the public ABI is include/nvq.h.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "nvq.h"

namespace nvq {

// ---- host helpers ---------------------------------------------------------
void set_hip_error(hipError_t e, const char *where);
int device_cu_count();  // compute units of the current device (cached)

#define NVQ_HIP_TRY(expr)                                   \
    do {                                                    \
        hipError_t e_ = (expr);                             \
        if (e_ != hipSuccess) {                             \
            ::nvq::set_hip_error(e_, #expr);                \
            return NVQ_ERR_HIP;                             \
        }                                                   \
    } while (0)

static inline bool aligned(const void *p, size_t a) {
    return (reinterpret_cast<uintptr_t>(p) & (a - 1)) == 0;
}

// Up to four weight matrices that read the same input can be served by one
// GEMV launch (q/k/v, gate/up).  Rows are numbered consecutively across the
// segments; row_end[i] is the first row after segment i.
constexpr int kMaxSeg = 4;
struct GemvSegs {
    const uint4 *qw[kMaxSeg];     // [N_i][G] one uint4 = one group of 32 nibbles
    const uint16_t *sc[kMaxSeg];  // [N_i][G] fp16 bits
    void *y[kMaxSeg];             // [M][N_i]
    int32_t *dbg[kMaxSeg];        // [M][N_i][G] or nullptr
    int N[kMaxSeg];
    int row_end[kMaxSeg];
    int y_dtype[kMaxSeg];
    int nseg;
    int total_rows;
};

// Internal launchers (validated arguments; enqueue only).
int launch_quant_act(const uint16_t *x, int M, int K, int act_group, int8_t *xq, float *xscale,
                     int32_t *xgsum, hipStream_t st);
// The inputs of n <= kMaxMerge layers with the same K, for M tokens, in one launch where K allows:
// a layer's transform (if any) and, with `quant`, its codes, scales and (unless xgsum is null) code
// sums; without it the transformed values go to xt (plain input: nothing).  xt is scratch either
// way.
constexpr int kMaxMerge = 2;
struct PrepTarget {
    uint16_t *xt;
    int8_t *xq;
    float *xscale;
    int32_t *xgsum;
};
int launch_prep(const nvq_linear *const *e, const PrepTarget *to, int n, int M, int act_group, bool quant,
                hipStream_t st);
int launch_gemv_w4a8(const GemvSegs &segs, int K, const int8_t *xq, const float *xscale,
                     const int32_t *xgsum, int act_group, int M, hipStream_t st);
int launch_gemv_w4a16(const GemvSegs &segs, int K, const uint16_t *x, int M, hipStream_t st);
// Up to 32 tokens, any K that is a whole number of groups (gemv_slice.h).  One launch takes up to
// kMaxMerge phases of the same K that do not depend on each other, each with its own input, if
// gemv_slice_merges says so.
struct SliceWork {
    int n;
    const GemvSegs *segs[kMaxMerge];
    const void *x[kMaxMerge];          // codes or bf16
    const float *xscale[kMaxMerge];    // W4A8
};
// Whether the multi-token kernel takes a phase (of the walk or a single call), and whether it takes
// two of them in one launch with every result added as in a launch of its own.
bool gemv_slice_takes(const GemvSegs &segs, int K, int M, int precision, int act_group);
bool gemv_slice_merges(const GemvSegs &a, const GemvSegs &b, int K, int M, int precision, int act_group);
int launch_gemv_slice_w4a16(const SliceWork &w, int K, int M, hipStream_t st);
int launch_gemv_slice_w4a8(const SliceWork &w, int K, int act_group, int M, hipStream_t st);
// Whether the grouped matrix-core launches take a phase: 2 <= M <= 32 tokens, per-token
// activation scale, K a multiple of 128, scale rows 8-byte aligned.
bool gemv_mfma_supported(const GemvSegs &segs, int K, int M);

// One phase of a grouped small-batch launch (lives in device memory): the
// activation quantisation of all its tokens (W4A8) and the matrix-core product
// of its row tiles run in grids shared with the other phases of its batch.
struct GroupPhase {
    GemvSegs segs;           // accumulator dumps unused
    const uint16_t *x_bf16;  // [M][K] input
    int8_t *xq;              // [M][K]   codes      (W4A8 phases, workspace)
    float *xscale;           // [M]      scales
    int32_t *xgsum;          // [M][K/32] code sums
    char *xa;                // operand image of the persistent kernel (either precision, workspace)
    int G, precision;
    int unit_begin;          // first grid unit of the phase in its batch
    int unit_count;          // its units
    int img_begin;           // first image unit of the phase in its batch (launch_operand_images)
};
// jobs[j] names the (W4A8) phase whose M tokens grid blocks j*M .. j*M+M-1 quantise; xgsum may
// be null.  The first eight words at `clear` (unless null) are set to zero, also without jobs.
int launch_quant_act_group(const GroupPhase *tab, const uint16_t *jobs, int njobs, int M,
                           uint32_t *clear, hipStream_t st);
// The operand images `xa` of the phases named in `jobs` (per-token scales of
// the W4A8 ones first, then the images: img_units[u] names the phase of image
// unit u, a token tile times eight 128-input columns; image_units(M, K) of
// them per phase, numbered from GroupPhase::img_begin).  Per tile of 16
// tokens, column c and piece i one KiB whose 16 bytes number 16 * kb + n are,
// for token n of the tile, the int8 codes 32 * kb + 16 * i .. + 15 of the
// column (W4A8, two pieces; xscale as in launch_quant_act_group, no code sums)
// or the bf16 inputs 32 * i + 8 * kb .. + 7 of the column, copied (W4A16, four
// pieces).  Token slots past M are left as they are.
int image_units(int M, int K);
int launch_operand_images(const GroupPhase *tab, const uint16_t *jobs, int njobs,
                          const uint16_t *img_units, int nimg, int M, hipStream_t st);
// unit_phase[u] names the phase of grid unit u; a unit is group_row_tiles(M)
// consecutive 16-row tiles, which share their activation operands (as many as
// fit the registers next to one or two token tiles).
static inline int group_row_tiles(int M) { (void)M; return 2; }
int launch_gemv_mfma_group(const GroupPhase *tab, const uint16_t *unit_phase, int nunits, int M,
                           hipStream_t st);
// The same work as one persistent grid of teams (a loader wave feeding four
// consumer waves through LDS rings); needs K % 512 == 0 and 16-byte aligned
// scale rows in every phase, and the operand images of launch_quant_act_group.
// The batch is cut into `nparts` = ring_parts(grid) parts of equal weight bytes
// that the workgroups of one XCD each work off together; part_tab (device
// memory): nparts + 1 unit indices, the cuts, then nparts + 1 phase indices,
// the phase of the unit at each cut.  A wait inside the kernel that gives up
// sets *status.
constexpr int kRingMaxParts = 8;
bool gemv_mfma_ring_supported(const GemvSegs &segs, int K);
int ring_grid(int M, int nunits);
int ring_parts(int grid);
int launch_gemv_mfma_ring(const GroupPhase *tab, const uint32_t *part_tab, int nparts, int grid,
                          int M, uint32_t *status, hipStream_t st);

// The same work for long lists of 2 to 32 tokens, from the inputs themselves (codes and scales of
// launch_quant_act_group for the W4A8 phases); grid: rows_grid() of its groups; tickets: eight words that
// are zero.  order: nparts + 1 indices into what follows, then the phases of every part in the order
// they are taken in (null: as they stand).
int rows_groups(int units);  // of one phase in one part
int rows_resident(int M);    // workgroups that are at work together
int rows_grid(int groups, int nparts, int M);  // groups: of the part with the most of them
int launch_gemv_rows(const GroupPhase *tab, const uint32_t *part_tab, int nparts, const uint32_t *order, int grid,
                     int M, uint32_t *tickets, hipStream_t st);

// From so many tokens on a batch of a plan may run as launches phase by phase (before: as the per-tile grid).
constexpr int kPhasesMinTokens = 17;

// ---- device helpers -------------------------------------------------------
#if defined(__HIPCC__)

__device__ __forceinline__ float bf16_bits_to_float(uint32_t h) {
    return __uint_as_float(h << 16);
}

// fp32 -> bf16 bits, round to nearest even: the hardware's conversion
// (v_cvt_pk_bf16_f32, one instruction for two values).
__device__ __forceinline__ uint16_t float_to_bf16_bits(float f) {
    return __builtin_bit_cast(uint16_t, (__bf16)f);
}
typedef __bf16 nvq_bf16x2 __attribute__((ext_vector_type(2)));
// ... two at a time, `lo` in the low half of the word.
__device__ __forceinline__ uint32_t pack_bf16x2(float lo, float hi) {
    const nvq_bf16x2 v = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, v);
}

__device__ __forceinline__ float half_bits_to_float(uint16_t h) {
    _Float16 v = __builtin_bit_cast(_Float16, h);
    return (float)v;
}

// op(value, value of lane i ^ D) without a trip through LDS, op symmetric.  D = 4 and 8 rotate
// within sixteen lanes: for 8 that is the exchange, for 4 it is where lanes 8 apart agree.
template <int D, typename T, typename OP>
__device__ __forceinline__ T with_lane_xor(T v, OP op) {
    static_assert(sizeof(T) == 4, "one register");
    const uint32_t b = __builtin_bit_cast(uint32_t, v);
    if constexpr (D >= 16) {
        const auto r = D == 32 ? __builtin_amdgcn_permlane32_swap(b, b, false, false)
                               : __builtin_amdgcn_permlane16_swap(b, b, false, false);
        const uint32_t even = r[0], odd = r[1];  // (a bit cast of an element in place takes element 0)
        return op(__builtin_bit_cast(T, even), __builtin_bit_cast(T, odd));
    } else {
        constexpr int kCtrl = D == 8 ? 0x128 : D == 4 ? 0x124 : D == 2 ? 0x4e : 0xb1;
        return op(v, __builtin_bit_cast(T, __builtin_amdgcn_update_dpp(b, b, kCtrl, 0xf, 0xf, false)));
    }
}

struct AddOp {
    template <typename T>
    __device__ T operator()(T a, T b) const { return a + b; }
};

// Sum across the LPR (64 or 32) lanes of an aligned lane group, those LPR / 2 apart first; every lane
// gets the sum.
template <int LPR>
__device__ __forceinline__ float group_sum(float v) {
    static_assert(LPR == 64 || LPR == 32, "");
    if (LPR == 64) v = with_lane_xor<32>(v, AddOp());
    v = with_lane_xor<16>(v, AddOp());
    v = with_lane_xor<8>(v, AddOp());
    v = with_lane_xor<4>(v, AddOp());
    v = with_lane_xor<2>(v, AddOp());
    return with_lane_xor<1>(v, AddOp());
}

__device__ __forceinline__ void store_out(void *y, int y_dtype, int64_t idx, float v) {
    if (y_dtype == NVQ_F32)
        reinterpret_cast<float *>(y)[idx] = v;
    else
        reinterpret_cast<uint16_t *>(y)[idx] = float_to_bf16_bits(v);
}

#endif  // __HIPCC__

}  // namespace nvq

// W4A16 instances of the small-batch kernel (gemv_slice.h).
#include "gemv_slice.h"

namespace nvq {

namespace {

template <int TOK, int RT, int W, int NG, int V>
int go(const SliceWork &w, int G, int M, hipStream_t st) {
    const int scb = slice_scale_bytes(w, G);
    if constexpr (V == 64) {
        if (scb >= 4) return slice_go<NVQ_W4A16, false, TOK, RT, W, NG, V, 4>(w, G, M, st);
        return slice_go<NVQ_W4A16, false, TOK, RT, W, NG, V, 2>(w, G, M, st);
    } else {  // (scales aligned to 8 bytes)
        if constexpr (NG == 8)
            if (scb == 16) return slice_go<NVQ_W4A16, false, TOK, RT, W, NG, V, 16>(w, G, M, st);
        return slice_go<NVQ_W4A16, false, TOK, RT, W, NG, V, 4>(w, G, M, st);
    }
}

template <int TOK>
int go_chains(const SliceWork &w, int G, int M, hipStream_t st) {
    const int v = slice_chains(*w.segs[0], G, M, false), rows = slice_rows(w);
    constexpr int NG = TOK == 32 ? 4 : 8;
    if constexpr (TOK == 8)
        if (v == 64 && slice_many(rows)) return go<TOK, 1, 4, 8, 64>(w, G, M, st);
    if (v == 64) return go<TOK, 1, 8, TOK == 8 ? 8 : 4, 64>(w, G, M, st);
    if constexpr (TOK == 16)
        if (v == 16 && slice_shared(rows)) return go<TOK, 1, 8, 4, 16>(w, G, M, st);
    if (v == 16) return go<TOK, 1, 8, NG, 16>(w, G, M, st);
    if (slice_row_tiles(rows) == 2) return go<TOK, 2, 4, NG, 8>(w, G, M, st);
    if (slice_eight_waves(rows, TOK)) return go<TOK, 1, 8, 4, 8>(w, G, M, st);
    if constexpr (TOK < 32) return go<TOK, 1, 4, 8, 8>(w, G, M, st);
    return NVQ_OK;  // (not reached)
}

}  // namespace

int launch_gemv_slice_w4a16(const SliceWork &w, int K, int M, hipStream_t st) {
    const int G = K / 32;
    if (M <= 8) return go_chains<8>(w, G, M, st);
    if (M <= 16) return go_chains<16>(w, G, M, st);
    return go_chains<32>(w, G, M, st);
}

}  // namespace nvq

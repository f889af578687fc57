// W4A16 instances of the small-batch kernel (gemv_slice.h).
#include "gemv_slice.h"

namespace nvq {

namespace {

template <int TOK, int RT, int W, int NG, int V>
int go(const GemvSegs &S, int G, int M, const uint16_t *x, hipStream_t st) {
    const int scb = slice_scale_bytes(S, G);
    if constexpr (V == 64) {
        if (scb >= 4) return slice_go<NVQ_W4A16, false, TOK, RT, W, NG, V, 4>(S, G, M, x, nullptr, st);
        return slice_go<NVQ_W4A16, false, TOK, RT, W, NG, V, 2>(S, G, M, x, nullptr, st);
    } else {  // (scales aligned to 8 bytes)
        if constexpr (NG == 8)
            if (scb == 16) return slice_go<NVQ_W4A16, false, TOK, RT, W, NG, V, 16>(S, G, M, x, nullptr, st);
        return slice_go<NVQ_W4A16, false, TOK, RT, W, NG, V, 4>(S, G, M, x, nullptr, st);
    }
}

template <int TOK>
int go_chains(const GemvSegs &S, int G, int M, const uint16_t *x, hipStream_t st) {
    const int v = slice_chains(S, G, M, false), rows = S.total_rows;
    constexpr int NG = TOK == 32 ? 4 : 8;
    if constexpr (TOK == 8)
        if (v == 64 && slice_many(rows)) return go<TOK, 1, 4, 8, 64>(S, G, M, x, st);
    if (v == 64) return go<TOK, 1, 8, TOK == 8 ? 8 : 4, 64>(S, G, M, x, st);
    if constexpr (TOK == 16)
        if (v == 16 && slice_shared(rows)) return go<TOK, 1, 8, 4, 16>(S, G, M, x, st);
    if (v == 16) return go<TOK, 1, 8, NG, 16>(S, G, M, x, st);
    if (slice_row_tiles(rows) == 2) return go<TOK, 2, 4, NG, 8>(S, G, M, x, st);
    if (slice_eight_waves(rows, TOK)) return go<TOK, 1, 8, 4, 8>(S, G, M, x, st);
    if constexpr (TOK < 32) return go<TOK, 1, 4, 8, 8>(S, G, M, x, st);
    return NVQ_OK;  // (not reached)
}

}  // namespace

int launch_gemv_slice_w4a16(const GemvSegs &S, int K, const uint16_t *x, int M, hipStream_t st) {
    const int G = K / 32;
    if (M <= 8) return go_chains<8>(S, G, M, x, st);
    if (M <= 16) return go_chains<16>(S, G, M, x, st);
    return go_chains<32>(S, G, M, x, st);
}

}  // namespace nvq

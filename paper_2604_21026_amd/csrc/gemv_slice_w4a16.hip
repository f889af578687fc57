// W4A16 instances of the small-batch kernel (gemv_slice.h).
#include "gemv_slice.h"

namespace nvq {

namespace {

template <int TOK, int RT>
int go(const GemvSegs &S, int G, int M, const uint16_t *x, hipStream_t st) {
    const int scb = slice_scale_bytes(S, G);
    if constexpr (TOK < 32)
        if (scb == 16) return slice_go<NVQ_W4A16, false, TOK, RT, 16>(S, G, M, x, nullptr, st);
    if (scb >= 4) return slice_go<NVQ_W4A16, false, TOK, RT, 4>(S, G, M, x, nullptr, st);
    return slice_go<NVQ_W4A16, false, TOK, RT, 2>(S, G, M, x, nullptr, st);
}

template <int TOK>
int go_rows(const GemvSegs &S, int G, int M, const uint16_t *x, hipStream_t st) {
    if (slice_row_tiles(S.total_rows) == 2) return go<TOK, 2>(S, G, M, x, st);
    return go<TOK, 1>(S, G, M, x, st);
}

}  // namespace

int launch_gemv_slice_w4a16(const GemvSegs &S, int K, const uint16_t *x, int M, hipStream_t st) {
    const int G = K / 32;
    if (M <= 8) return go_rows<8>(S, G, M, x, st);
    if (M <= 16) return go_rows<16>(S, G, M, x, st);
    return go_rows<32>(S, G, M, x, st);
}

}  // namespace nvq

// W4A8 instances of the small-batch kernel (gemv_slice.h).
#include "gemv_slice.h"

namespace nvq {

namespace {

template <bool PG, int TOK, int RT, int W, int NG, int V>
int go(const GemvSegs &S, int G, int M, const int8_t *xq, const float *xscale, bool debug, hipStream_t st) {
    // the accumulator dump: the same order of additions, the instance that takes any scales
    if (debug) return slice_go<NVQ_W4A8, PG, TOK, RT, W, NG, V, 2, true>(S, G, M, xq, xscale, st);
    const int scb = slice_scale_bytes(S, G);
    if constexpr (V == 64) {
        if constexpr (PG && NG == 8)
            if (scb == 16) return slice_go<NVQ_W4A8, PG, TOK, RT, W, NG, V, 16>(S, G, M, xq, xscale, st);
        if (scb >= 4) return slice_go<NVQ_W4A8, PG, TOK, RT, W, NG, V, 4>(S, G, M, xq, xscale, st);
        return slice_go<NVQ_W4A8, PG, TOK, RT, W, NG, V, 2>(S, G, M, xq, xscale, st);
    } else {  // (scales aligned to 8 bytes)
        if constexpr (NG == 8)
            if (scb == 16) return slice_go<NVQ_W4A8, PG, TOK, RT, W, NG, V, 16>(S, G, M, xq, xscale, st);
        return slice_go<NVQ_W4A8, PG, TOK, RT, W, NG, V, 4>(S, G, M, xq, xscale, st);
    }
}

template <bool PG, int TOK>
int go_chains(const GemvSegs &S, int G, int M, const int8_t *xq, const float *xscale, hipStream_t st) {
    bool debug = false;
    for (int i = 0; i < S.nseg; ++i) debug |= S.dbg[i] != nullptr;
    const int v = slice_chains(S, G, M, PG), rows = S.total_rows;
    if constexpr (!PG) {
        if constexpr (TOK == 32)
            if (v == 16 && slice_shared(rows)) return go<PG, TOK, 1, 8, 4, 16>(S, G, M, xq, xscale, debug, st);
        if (v == 16) return go<PG, TOK, 1, 8, 8, 16>(S, G, M, xq, xscale, debug, st);
        if (v == 8 && slice_row_tiles(rows) == 2) return go<PG, TOK, 2, 4, 8, 8>(S, G, M, xq, xscale, debug, st);
        if (v == 8 && slice_eight_waves(rows, TOK)) return go<PG, TOK, 1, 8, 4, 8>(S, G, M, xq, xscale, debug, st);
        if constexpr (TOK < 32)
            if (v == 8) return go<PG, TOK, 1, 4, 8, 8>(S, G, M, xq, xscale, debug, st);
    }
    if constexpr (TOK == 8)
        if (slice_many(rows)) return go<PG, TOK, 1, 4, 8, 64>(S, G, M, xq, xscale, debug, st);
    return go<PG, TOK, 1, 8, 8, 64>(S, G, M, xq, xscale, debug, st);
}

template <bool PG>
int go_tokens(const GemvSegs &S, int G, int M, const int8_t *xq, const float *xscale, hipStream_t st) {
    if (M <= 8) return go_chains<PG, 8>(S, G, M, xq, xscale, st);
    if (M <= 16) return go_chains<PG, 16>(S, G, M, xq, xscale, st);
    return go_chains<PG, 32>(S, G, M, xq, xscale, st);
}

}  // namespace

int launch_gemv_slice_w4a8(const GemvSegs &S, int K, const int8_t *xq, const float *xscale,
                           int act_group, int M, hipStream_t st) {
    return act_group == 32 ? go_tokens<true>(S, K / 32, M, xq, xscale, st)
                           : go_tokens<false>(S, K / 32, M, xq, xscale, st);
}

}  // namespace nvq

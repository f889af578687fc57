// W4A8 instances of the small-batch kernel (gemv_slice.h).
#include "gemv_slice.h"

namespace nvq {

namespace {

template <bool PG, int TOK, int RT>
int go(const GemvSegs &S, int G, int M, const int8_t *xq, const float *xscale, hipStream_t st) {
    const int scb = slice_scale_bytes(S, G);
    if (scb == 16) return slice_go<NVQ_W4A8, PG, TOK, RT, 16>(S, G, M, xq, xscale, st);
    if (scb == 4) return slice_go<NVQ_W4A8, PG, TOK, RT, 4>(S, G, M, xq, xscale, st);
    return slice_go<NVQ_W4A8, PG, TOK, RT, 2>(S, G, M, xq, xscale, st);
}

template <bool PG, int TOK>
int go_rows(const GemvSegs &S, int G, int M, const int8_t *xq, const float *xscale, hipStream_t st) {
    bool debug = false;
    for (int i = 0; i < S.nseg; ++i) debug |= S.dbg[i] != nullptr;
    const int rt = slice_row_tiles(S.total_rows);
    if (debug) {  // the accumulator dump: the same order of additions, the instances that take any K
        if (rt == 2) return slice_go<NVQ_W4A8, PG, TOK, 2, 2, true>(S, G, M, xq, xscale, st);
        return slice_go<NVQ_W4A8, PG, TOK, 1, 2, true>(S, G, M, xq, xscale, st);
    }
    if (rt == 2) return go<PG, TOK, 2>(S, G, M, xq, xscale, st);
    return go<PG, TOK, 1>(S, G, M, xq, xscale, st);
}

template <bool PG>
int go_tokens(const GemvSegs &S, int G, int M, const int8_t *xq, const float *xscale, hipStream_t st) {
    if (M <= 8) return go_rows<PG, 8>(S, G, M, xq, xscale, st);
    if (M <= 16) return go_rows<PG, 16>(S, G, M, xq, xscale, st);
    return go_rows<PG, 32>(S, G, M, xq, xscale, st);
}

}  // namespace

int launch_gemv_slice_w4a8(const GemvSegs &S, int K, const int8_t *xq, const float *xscale,
                           int act_group, int M, hipStream_t st) {
    return act_group == 32 ? go_tokens<true>(S, K / 32, M, xq, xscale, st)
                           : go_tokens<false>(S, K / 32, M, xq, xscale, st);
}

}  // namespace nvq

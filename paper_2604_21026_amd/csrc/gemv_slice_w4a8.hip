// W4A8 instances of the small-batch kernel (gemv_slice.h).
#include "gemv_slice.h"

namespace nvq {

namespace {

template <bool PG, int TOK, int RT, int W, int NG, int V>
int go(const SliceWork &w, int G, int M, bool debug, hipStream_t st) {
    // the accumulator dump: the same order of additions, the instance that takes any scales
    if (debug) return slice_go<NVQ_W4A8, PG, TOK, RT, W, NG, V, 2, true>(w, G, M, st);
    const int scb = slice_scale_bytes(w, G);
    if constexpr (V == 64) {
        if constexpr (PG && NG == 8)
            if (scb == 16) return slice_go<NVQ_W4A8, PG, TOK, RT, W, NG, V, 16>(w, G, M, st);
        if (scb >= 4) return slice_go<NVQ_W4A8, PG, TOK, RT, W, NG, V, 4>(w, G, M, st);
        return slice_go<NVQ_W4A8, PG, TOK, RT, W, NG, V, 2>(w, G, M, st);
    } else {  // (scales aligned to 8 bytes)
        if constexpr (NG == 8)
            if (scb == 16) return slice_go<NVQ_W4A8, PG, TOK, RT, W, NG, V, 16>(w, G, M, st);
        return slice_go<NVQ_W4A8, PG, TOK, RT, W, NG, V, 4>(w, G, M, st);
    }
}

template <bool PG, int TOK>
int go_chains(const SliceWork &w, int G, int M, hipStream_t st) {
    bool debug = false;
    for (int k = 0; k < w.n; ++k)
        for (int i = 0; i < w.segs[k]->nseg; ++i) debug |= w.segs[k]->dbg[i] != nullptr;
    const int v = slice_chains(*w.segs[0], G, M, PG), rows = slice_rows(w);
    if constexpr (!PG) {
        if constexpr (TOK == 32)
            if (v == 16 && slice_shared(rows)) return go<PG, TOK, 1, 8, 4, 16>(w, G, M, debug, st);
        if (v == 16) return go<PG, TOK, 1, 8, 8, 16>(w, G, M, debug, st);
        if (v == 8 && slice_row_tiles(rows) == 2) return go<PG, TOK, 2, 4, 8, 8>(w, G, M, debug, st);
        if (v == 8 && slice_eight_waves(rows, TOK)) return go<PG, TOK, 1, 8, 4, 8>(w, G, M, debug, st);
        if constexpr (TOK < 32)
            if (v == 8) return go<PG, TOK, 1, 4, 8, 8>(w, G, M, debug, st);
    }
    if constexpr (TOK == 8)
        if (slice_many(rows)) return go<PG, TOK, 1, 4, 8, 64>(w, G, M, debug, st);
    return go<PG, TOK, 1, 8, 8, 64>(w, G, M, debug, st);
}

template <bool PG>
int go_tokens(const SliceWork &w, int G, int M, hipStream_t st) {
    if (M <= 8) return go_chains<PG, 8>(w, G, M, st);
    if (M <= 16) return go_chains<PG, 16>(w, G, M, st);
    return go_chains<PG, 32>(w, G, M, st);
}

}  // namespace

bool gemv_slice_takes(const GemvSegs &S, int K, int M, int precision, int act_group) {
    if (M == 1 && K <= 16384) return false;
    return !gemv_wave_per_row(S, K, M, precision, precision == NVQ_W4A8 && act_group == 32);
}

// The order of a result's additions is the phase's own (slice_chains); rows, waves and row tiles of
// a launch go by all its rows.
bool gemv_slice_merges(const GemvSegs &a, const GemvSegs &b, int K, int M, int precision, int act_group) {
    const bool pg = precision == NVQ_W4A8 && act_group == 32;
    return gemv_slice_takes(a, K, M, precision, act_group) && gemv_slice_takes(b, K, M, precision, act_group) &&
           slice_chains(a, K / 32, M, pg) == slice_chains(b, K / 32, M, pg);
}

int launch_gemv_slice_w4a8(const SliceWork &w, int K, int act_group, int M, hipStream_t st) {
    return act_group == 32 ? go_tokens<true>(w, K / 32, M, st) : go_tokens<false>(w, K / 32, M, st);
}

}  // namespace nvq

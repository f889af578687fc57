// Products of 2 to 32 tokens with one phase's weight rows, any K that is a whole number
// of groups, activation scales per token or per group: the kernel behind the single calls
// and the per-phase walk (up to three tokens and few rows: see gemv_wave_per_row).  Paper:
// the W4A8 / W4A16 kernel descriptions; the arithmetic is that of mfma_act.h (one 16x16x32
// MFMA per quantisation group, 16 tokens times 16 rows, the constant nibble offset of W4A16 removed
// by a second MFMA; W4A8 weights enter as signed bytes 16 (n - 8)).
//
// A workgroup of W waves owns 16 RT consecutive rows; the waves share out K in blocks of
// NG groups (eight: 256 inputs, a whole 128-byte line of every row), wave w the blocks w, w
// + W, ..., and the partial sums are added through LDS at the end.  Until then the waves do
// not meet.  Each copies what it needs of a block (the rows' weights and scales, the tokens'
// inputs) straight from global memory into its own piece of LDS, takes it into registers,
// asks for its next block and only then multiplies; what covers the memory's latency are
// the workgroups that share a compute unit (see SliceBlock for how many).
//
// The order of a result's additions is a property of the call, not of W, NG and RT: V
// chains of groups, each added from the first group to the last, whose sums then meet.
//   V = 8, 16  chain v holds the columns (four groups) v, v + V, ...; the chains are added
//              in order.  K a multiple of 128, scales aligned to 8 bytes, and a scale per
//              token (or none).
//   V = 64     chain v holds the groups v, v + 64, ...; the chains are added in pairs, those
//              32 apart first.  Everything else.
// (One chain per wave, as its blocks follow each other, is a shorter way to the sum; but the
// sums get longer, four to eight times in parts, and a chain of layers amplifies the bits that
// differ from the other kernels' to a hundredth of the result.)
//
// What bounds it: a launch, and then the instructions of a compute unit's waves.  4096 x 4096 at 8 tokens
// (W4A16, 4.1 us between launches): the first load leaves 0.6 us after a workgroup's start, the first block
// arrives after 1.4, the last 2.4, and 0.9 go by with the slowest wave's products and the sums; between the
// loads memory is near its rate.  28672 x 4096 at 8 tokens takes 14.5 (W4A8) to 16.7 us (W4A16), a compute
// unit with 4 workgroups 2 us longer than one with 3; the per-tile grid that loaded straight into
// registers took 25 and 31.  A product takes 8 to 10 vector instructions and one or two LDS reads with up to 8
// tokens (11 to 13 and three when the products of a pair of groups were brought together by lane
// exchanges: 17.2 us instead of 16.7, 8192 x 2048 4.4 instead of 4.1, the 8B chain 188.4 instead of 183.2).
// The sixty-four chains cost registers
// and a longer way through LDS: with a scale per group 16384 x 3072 takes 9.2 us at 4 tokens
// (8.6 in one chain per wave; a wave per row, which served these calls before, 18.7), 28672 x
// 4096 20, 27 and 57 us at 8, 16 and 32 tokens (that: 63, 111 and 202).  Two to four blocks in
// flight per wave instead of one were no faster, with the same number of workgroups per compute unit either
// (4096 x 14336 11.4 us against 10.8), nor were priorities of any kind.
//
// W, NG: eight waves with blocks of eight groups, or where that is better
//  - four waves, in eight column chains (see slice_eight_waves), and with a scale per group and up to
//    eight tokens from two row tiles per compute unit on (28672 x 4096: 20.4 against 21.6;
//    4096 x 14336 14.5 against 10.2, so not below);
//  - blocks of four groups.  They load half lines, which costs 5-15 % where nothing else
//    changes, and are taken where eight leave room in LDS for one workgroup only: W4A16 at 17
//    tokens and more (16384 x 3072, 32 tokens: 12.9 us against 17.5), W4A16 at 9 to 16 and W4A8
//    at 17 and more tokens with more row tiles than compute units (8192 x 4096: 8.3 against 9.0
//    and 9.5 against 11.7; with fewer tiles 14.6 against 13.5 at K = 14336); and where eight
//    waves in eight chains need them (slice_eight_waves).
//
// SCB: bytes per scale load.  16: K is a multiple of 256 and the scales are aligned to
// that (one load per row and block); 4 or 2: any other K, scales aligned to 4 bytes and an
// even number of groups, or not; the last block may then end early (its missing groups
// are loaded as the last one again and not multiplied).
#pragma once

#include <type_traits>

#include "gemv_tile.h"
#include "mfma_act.h"

namespace nvq {

namespace {

typedef __attribute__((address_space(3))) void *slice_lds_ptr;

// The value of lane i ^ 1 or i ^ 2.
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e;
template <int CTRL>
__device__ __forceinline__ float dpp_f32(float v) {
    const int i = __builtin_bit_cast(int, v);
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(i, i, CTRL, 0xf, 0xf, false));
}

constexpr int slice_vmcnt(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0f70; }

// What a block of NG groups takes in a wave's ring: TOK tokens (8, 16 or 32), RT 16-row tiles.
template <int PREC, bool PG, int TOK, int RT, int NG, int SCB>
struct SliceBlock {
    static_assert(SCB != 16 || NG == 8, "16 bytes are the scales of eight groups");
    static constexpr int kTokenBytes = NG * (PREC == NVQ_W4A8 ? 32 : 64);
    // scales: [16 bytes of a row], or words of 4 bytes, [pair of groups or group][row]
    static constexpr int kScOps = SCB == 16 ? 1 : NG == 4 && SCB == 4 && RT == 1 ? 1 : RT * (SCB == 4 ? 1 : 2) * NG / 8;
    static constexpr int kScBytes = SCB == 16 ? RT * 256 : kScOps * 256;
    static constexpr int kPieces = kTokenBytes / 16, kMixed = (kPieces < 16 ? kPieces : 16) - 1;
    static constexpr int kAOps = TOK * kTokenBytes / 1024;
    static constexpr int kXsOps = PG ? TOK * NG / 64 : 0;  // 64 lanes x 4 bytes, NG scales per token
    static constexpr int kWOps = RT * NG / 4, kWTile = 256 * NG;
    static constexpr int kW = 0, kSc = kW + RT * kWTile, kA = kSc + kScBytes;
    static constexpr int kXs = kA + TOK * kTokenBytes, kBytes = kXs + kXsOps * 256;

    // With up to eight tokens lane rows 2 and 3 of a product hold no token.  The products of groups i and
    // i + 4 of a block are therefore added into one register each: group i multiplies the tokens as rows 0
    // to 7 of the operand, group i + 4 as rows 8 to 15, and what the other rows read in LDS is zero.  A pair of
    // groups then costs 4 conversions (W4A8) and 4 fmaf instead of 8 and 8, with half the registers.
    static constexpr bool kPair = TOK == 8 && NG == 8;
    static constexpr int kZero = kPair ? 16 : 0;  // bytes of zeros behind the rings, for those
    static constexpr int group_half(int kb) { return kPair ? kb >> 1 : 0; }  // whose groups lane row kb adds

    // Where lane row kb finds the scales of its first token, and a token's place among the
    // activations: what stands for tokens that are not there is read from another's.
    static constexpr int xs_place(int kb) {
        return 16 * NG * (TOK < 16 ? kb & (TOK / 4 - 1) : kb) + 16 * group_half(kb);
    }
    static constexpr int token_place(int n) { return (TOK < 16 ? n & (TOK - 1) : n) * kTokenBytes; }
    // The last byte that the reads of a block touch lies inside the piece it belongs to.
    static constexpr int kTiles = (TOK + 15) / 16, kRowBytes = 16 * NG;
    static constexpr int kScWords = SCB == 2 ? NG : NG / 2;  // words with the scales of a row
    static constexpr int kScRead = kPair ? kScWords / 2 : kScWords, kXsRead = kPair ? 1 : NG / 4;  // per lane
    static constexpr int kScStep = SCB == 16 ? 4 : 64 * RT;  // from word to word
    static constexpr int largest(int (*place)(int), int n) {
        int m = 0;
        for (int i = 0; i < n; ++i) m = place(i) > m ? place(i) : m;
        return m;
    }
    static_assert(15 * kRowBytes + 16 * (NG - 1) + 16 <= kWTile, "weights");
    static_assert((SCB == 16 ? RT * 256 : kScWords * 16 * RT * 4) <= kScBytes, "scales");
    static_assert(largest(token_place, 16) + (kTiles - 1) * 16 * kTokenBytes + kTokenBytes <= TOK * kTokenBytes,
                  "activations");
    static_assert(!PG || largest(xs_place, 4) + ((kTiles - 1) * 16 + 3) * 4 * NG + 16 * kXsRead <= kXsOps * 256,
                  "activation scales");
};

// A phase of a launch.  Arguments cost time twice: the host writes them into device memory (a call
// with 512 bytes of them takes 0.5 us longer than with 224), and they are cold memory in every
// launch.  So they are few, there are two phases only where a launch has two, and the kernel asks
// for all lines of a phase together (one after the other, where they are needed, the last of
// them, where the results go, was waited for when everything else was done; W4A16, 4096 x 4096 at 8
// tokens: 5.1 us against 4.5).  SEGS: room for kMaxSeg matrices, or for the one of a single call, which
// then has fewer lines of them and no matrix to select for its rows and results (W4A16, 16 tokens: 4096 x
// 4096 4.6 us with four, 4.2 with one, 5000 x 96 3.8 and 3.1; 3 tokens, 300 x 1024 2.7 and 2.5).
// A workgroup's rows belong to one matrix (a matrix that ends inside a row tile leaves the rest of it
// empty), so that everything but a lane's place in the tile is in scalar registers: when every lane
// found the matrix of its own rows, a third of a wave's vector instructions at K = 4096 were spent
// before its first load and behind its last product (four 8B blocks as a chain at 8 tokens: 191.4 us, now
// 189.6).
template <int SEGS, bool DEBUG>
struct SlicePhase {
    const uint4 *qw[SEGS];
    const uint16_t *sc[SEGS];
    void *y[SEGS];
    const char *x;
    const float *xscale;
    int N[SEGS];  // of the whole matrix
    int G, M;
    uint32_t bf16;  // bit i: matrix i has bf16 results; bit 8 + i: its workgroups have 16 rows each
    // (with one matrix all that is read lies in one line)
    int rows[SEGS];      // of it here
    int unit_end[SEGS];  // workgroups up to this matrix; of those that are not there: as the last one's
    int32_t *dbg[DEBUG ? SEGS : 1];
};
// What of a phase a workgroup keeps: the matrix its rows belong to.
struct SliceMatrix {
    const uint4 *qw;
    const uint16_t *sc;
    void *y;
    int32_t *dbg;
    int N, rows;
    bool bf16, half;
};
template <int NP, int SEGS, bool DEBUG>
struct SliceArgs {
    SlicePhase<SEGS, DEBUG> phase[NP];  // the first phase's workgroups come first
};
static_assert(sizeof(SlicePhase<kMaxSeg, false>) == 184 && kMaxMerge == 2, "three lines; one comparison finds a workgroup's phase");

// Two workgroups of eight waves per compute unit with a scale per group and 16 tokens: 128 registers, which
// the compiler would pass by two.
constexpr int slice_min_waves(bool pg, int tok, int scb, bool debug) { return pg && tok == 16 && scb >= 4 && !debug ? 4 : 1; }

template <int PREC, bool PG, int TOK, int RT, int W, int NG, int V, int SCB, int NP, int SEGS, bool DEBUG>
__global__ __launch_bounds__(W * 64) __attribute__((amdgpu_waves_per_eu(slice_min_waves(PG, TOK, SCB, DEBUG)))) void
gemv_slice_kernel(SliceArgs<NP, SEGS, DEBUG>) {
    typedef Act<PREC> A;
    typedef SliceBlock<PREC, PG, TOK, RT, NG, SCB> B;
    constexpr bool TAIL = SCB != 16;
    constexpr int MT = B::kTiles;
    constexpr int kTile = RT * MT * 4;  // result registers per lane
    // The chains that meet in a wave: C of every block, and the blocks take turns over U sets
    // of them (block b belongs to set b % U).  Chain of set u, place c: (C (w + W u) + c) % V.
    constexpr bool kByGroup = V == 64;
    constexpr int C = kByGroup ? NG : NG / 4, U = V / (C * W);
    constexpr int CR = B::kPair ? C / 2 : C;  // their registers: place c + C / 2 in the upper half
    static_assert(U * C * W == V && (U == 1 || U == 2), "every chain has one place");
    constexpr int SH = W / 2;  // by group: lanes that share a result
    static_assert(!kByGroup || SH == 2 || SH == 4, "128 results at a time");
    constexpr int kRing = W * B::kBytes, kLds = kRing + B::kZero, kRedStride = 128 + 64 / SH;
    constexpr int kRed = kByGroup ? W * C * kRedStride * 4 : V * kTile * 256;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kLds > kRed ? kLds : kRed];

    typedef const __attribute__((address_space(4))) SlicePhase<SEGS, DEBUG> CPhase;
    typedef const __attribute__((address_space(4))) uint32_t CWord;
    // (through the segment's pointer: indexed as a parameter the struct would be copied to scratch; it is
    // the kernel's only parameter, so the segment begins with it)
    CPhase *phase = (CPhase *)__builtin_amdgcn_kernarg_segment_ptr();
    int unit = (int)blockIdx.x;
    if constexpr (NP > 1) {
        static_assert(SEGS == kMaxSeg, "the lines asked for here");
        CWord *a = (CWord *)phase;
        constexpr int kNext = sizeof(SlicePhase<SEGS, DEBUG>) / 4;
        const uint32_t l0 = a[0], l1 = a[16], l2 = a[32], l3 = a[kNext], l4 = a[kNext + 16], l5 = a[NP * kNext - 1];
        const int units = phase->unit_end[SEGS - 1];
        asm volatile("" ::"s"(l0), "s"(l1), "s"(l2), "s"(l3), "s"(l4), "s"(l5), "s"(units));
        if (unit >= units) {
            unit -= units;
            ++phase;
        }
    }
    // (Copies in scalar registers that the compiler takes for values of its own: it would select among
    // the fields' addresses and load again.)
    const uint4 *qw[SEGS];
    const uint16_t *sc[SEGS];
    void *y[SEGS];
    int N[SEGS], rows[SEGS], unit_end[SEGS];
#pragma unroll
    for (int i = 0; i < SEGS; ++i) {
        qw[i] = phase->qw[i];
        sc[i] = phase->sc[i];
        y[i] = phase->y[i];
        N[i] = phase->N[i];
        asm volatile("" : "+s"(qw[i]), "+s"(sc[i]), "+s"(y[i]), "+s"(N[i]));
        rows[i] = SEGS > 1 ? phase->rows[i] : N[i];
        unit_end[i] = SEGS > 1 ? phase->unit_end[i] : 0;
        if (SEGS > 1) asm volatile("" : "+s"(rows[i]), "+s"(unit_end[i]));
    }
    const int G = phase->G, M = phase->M;
    const char *const xin = phase->x;
    const float *const xscale = phase->xscale;
    const uint32_t bits = phase->bf16;
    SliceMatrix S = {qw[0], sc[0], y[0], phase->dbg[0], N[0], rows[0], (bits & 1u) != 0, (bits >> 8 & 1u) != 0};
    int first = 0;  // the matrix's first workgroup
#pragma unroll
    for (int i = 1; i < SEGS; ++i) {
        if (unit < unit_end[i - 1]) continue;
        S = {qw[i], sc[i], y[i], phase->dbg[DEBUG ? i : 0], N[i], rows[i], (bits >> i & 1u) != 0, (bits >> (8 + i) & 1u) != 0};
        first = unit_end[i - 1];
    }
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n = lane & 15, kb = lane >> 4;
    const bool one_tile = RT == 2 && TOK == 8 && SEGS > 1 && S.half;
    const int row0 = (unit - first) * (one_tile ? 16 : 16 * RT);
    // the last of the tile's rows: others are read as this one
    const int last = one_tile && S.rows - row0 > 16 ? 15 : S.rows - 1 - row0;
    const char *const qrow = reinterpret_cast<const char *>(S.qw + (int64_t)row0 * G);
    const char *const srow = reinterpret_cast<const char *>(S.sc + (int64_t)row0 * G);
    const int NB = (G + NG - 1) / NG;
    const int nblk = NB > w ? (NB - w + W - 1) / W : 0;
    unsigned char *const slot = lds + w * B::kBytes;

    // Sources, at the start of the row: weights (a row's NG pieces of 16 bytes side by
    // side, permuted against the neighbouring rows'), scales, activations.
    uint32_t woff[B::kWOps], soff[B::kScOps];
    constexpr int kWRows = 64 / NG;  // rows per weight load
    int wc[2];                       // the piece, even and odd j
#pragma unroll
    for (int j = 0; j < 2; ++j) wc[j] = (lane % NG) ^ (((kWRows * j + lane / NG) / (16 / NG)) % NG);
#pragma unroll
    for (int j = 0; j < B::kWOps; ++j) {
        const int r = kWRows * j + lane / NG;
        woff[j] = (uint32_t)(r < last ? r : last) * (uint32_t)(G * 16) + (TAIL ? 0u : 16u * (uint32_t)wc[j & 1]);
    }
    constexpr int kRows = 16 * RT;
    int sg[B::kScOps];  // first group of the lane's word
#pragma unroll
    for (int k = 0; k < B::kScOps; ++k) {
        const int word = k * 64 + lane;
        sg[k] = SCB == 16 ? 0 : (word / kRows * (SCB / 2)) % NG;
        const int r = word % kRows;
        soff[k] = (uint32_t)(r < last ? r : last) * (uint32_t)(G * 2);
    }
    // activations: 2 or 4 tokens per instruction, pieces permuted against each other
    constexpr int kPieces = B::kPieces;
    uint32_t aoff[B::kAOps];
    int apiece[B::kAOps];
#pragma unroll
    for (int j = 0; j < B::kAOps; ++j) {
        const int m = j * (64 / kPieces) + lane / kPieces;
        const int p = (lane % kPieces) ^ (m & B::kMixed);
        aoff[j] = (uint32_t)(m < M ? m : M - 1) * (uint32_t)(G * 32 * A::kBytes) + (TAIL ? 0u : 16u * (uint32_t)p);
        apiece[j] = p;
    }
    uint32_t xsoff[PG ? B::kXsOps : 1];  // word l: scale l % NG of token l / NG
    if (PG) {
#pragma unroll
        for (int j = 0; j < B::kXsOps; ++j) {
            const int m = j * (64 / NG) + lane / NG;
            xsoff[j] = (uint32_t)(m < M ? m : M - 1) * (uint32_t)G;
        }
    }
    auto clamp_g = [&](int g) { return g < G ? g : G - 1; };
    auto issue = [&](int b) {
        const int g0 = NG * (w + W * b);
#pragma unroll
        for (int j = 0; j < B::kWOps; ++j) {
            const char *p = TAIL ? qrow + (woff[j] + 16u * (uint32_t)clamp_g(g0 + wc[j & 1])) : qrow + (size_t)g0 * 16 + woff[j];
            __builtin_amdgcn_global_load_lds((const void *)p, (slice_lds_ptr)(slot + B::kW + j * 1024), 16, 0, 0);
        }
#pragma unroll
        for (int k = 0; k < B::kScOps; ++k) {
            if (SCB == 16) {
                const char *p = srow + (size_t)g0 * 2 + soff[k];
                if (lane < kRows)
                    __builtin_amdgcn_global_load_lds((const void *)p, (slice_lds_ptr)(slot + B::kSc), 16, 0, 0);
            } else if (SCB == 4) {  // (a pair of groups is inside the row or outside it)
                const int g = g0 + sg[k];
                const char *p = srow + (soff[k] + 2u * (uint32_t)(g < G ? g : G - 2));
                __builtin_amdgcn_global_load_lds((const void *)p, (slice_lds_ptr)(slot + B::kSc + k * 256), 4, 0, 0);
            } else {
                const char *p = srow + (soff[k] + 2u * (uint32_t)clamp_g(g0 + sg[k]));
                __builtin_amdgcn_global_load_lds((const void *)p, (slice_lds_ptr)(slot + B::kSc + k * 256), 2, 0, 0);
            }
        }
#pragma unroll
        for (int j = 0; j < B::kAOps; ++j) {
            const char *p;
            if (TAIL) {
                const int pg = kPieces / NG;  // pieces per group
                p = xin + (aoff[j] + (uint32_t)clamp_g(g0 + apiece[j] / pg) * (uint32_t)(32 * A::kBytes) +
                           16u * (uint32_t)(apiece[j] % pg));
            } else {
                p = xin + (size_t)g0 * (32 * A::kBytes) + aoff[j];
            }
            __builtin_amdgcn_global_load_lds((const void *)p, (slice_lds_ptr)(slot + B::kA + j * 1024), 16, 0, 0);
        }
        if (PG) {
#pragma unroll
            for (int j = 0; j < B::kXsOps; ++j) {
                const char *p = reinterpret_cast<const char *>(xscale) + 4u * (xsoff[j] + (uint32_t)clamp_g(g0 + lane % NG));
                __builtin_amdgcn_global_load_lds((const void *)p, (slice_lds_ptr)(slot + B::kXs + j * 256), 4, 0, 0);
            }
        }
    };

    float f[U][CR][RT][MT][4];
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
        for (int c = 0; c < CR; ++c)
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) f[u][c][r][mt][jj] = 0.0f;

    // The lane's places in its piece of LDS, for group i of the block.  Weights: dword kb of
    // piece i of row n (what the MFMA's weight operand of group i wants), 64 different banks;
    // activations: for W4A16 half a piece twice (inputs 4 kb .. + 3 and 16 + 4 kb .. + 3 of
    // the group), for W4A8 a dword twice.
    const uint32_t at = (uint32_t)(uintptr_t)slot;
    const int mn = TOK < 16 ? n & (TOK - 1) : n;
    // The permutations leave the rest of an address alone: another piece is one xor away.  With more
    // than 8 tokens and a scale per group the addresses are made anew for every block, so that
    // the registers suffice, up to 16 tokens for two workgroups per compute unit (28672 x 4096: 27 us
    // against 36); elsewhere they stay in registers.
    constexpr bool kFresh = PG && TOK > 8;
    const uint32_t wpos0 = at + n * (16 * NG) + 16 * ((n / (16 / NG)) % NG) + 4 * kb;
    const uint32_t apos0 = B::token_place(n) + (PREC == NVQ_W4A8 ? 16 * (mn & B::kMixed) + 4 * kb
                                                                : 16 * ((kb >> 1) ^ mn) + 8 * (kb & 1));
    auto wpiece = [&](uint32_t p0, int i) { return p0 ^ (uint32_t)(16 * i); };
    auto apiece_at = [&](uint32_t p0, int i, int h) {
        return at + (p0 ^ (uint32_t)(16 * (PREC == NVQ_W4A8 ? 2 * i + h : 4 * i + 2 * h)));
    };
    // pairs: rows 0 to 7 of the operand of groups 0 to 3, rows 8 to 15 of that of 4 to 7, and zeros
    const uint32_t zero = (uint32_t)(uintptr_t)lds + kRing;
    if (B::kPair) asm volatile("ds_write_b32 %0, %1" ::"v"(zero + 4 * (n & 3)), "v"(0) : "memory");
    auto pair_at = [&](uint32_t p0, int i, int h) {
        return (n < 8) == (i < 4) ? B::kA + apiece_at(p0, i, h) : zero;
    };
    const int half = B::group_half(kb);
    const uint32_t spos = at + (SCB == 16 ? 16 : 4) * n + half * B::kScRead * B::kScStep;
    const uint32_t xspos = at + B::xs_place(kb);  // token 4 kb, 4 NG bytes per token

    if (nblk > 0) issue(0);
    // The scales of the tokens whose results the lane holds, or (by group) stores at the end (W4A8,
    // a scale per token): asked for here, they arrive with the first block (at the end, one wait
    // after the other, they took 0.4 to 0.5 us of every launch).
    constexpr bool kTokenScale = PREC == NVQ_W4A8 && !PG;
    constexpr int kRegs = B::kPair ? 4 : 2, kRounds = kByGroup ? kTile / kRegs : 1;  // (see the end)
    const int share = (int)threadIdx.x % SH, result = (int)threadIdx.x / SH;
    auto stored_reg = [&](int round) { return kRegs * round + (B::kPair ? result >> 5 : result >> 6); };
    auto stored_token = [&](int reg) {
        return 16 * ((reg >> 2) % MT) + 4 * ((result >> 4) & (B::kPair ? 1 : 3)) + (reg & 3);
    };
    constexpr int kXsc = kByGroup ? kRounds : MT * 4;
    // W4A8 weights enter as 16 (n - 8) (see weights, below).  The factor leaves with a scale per token on the
    // chain's sum (in the scale it would cost bits of those below 2^-122); with a scale per group before that:
    // left in the chains it would overflow for results beyond 2^124.  There a product starts at the bits
    // of 786432.0f, whose last place is a sixteenth, so that what it ends at is a float that is
    // one subtraction from the product, no more than a conversion costs.  (For a scale per token too it
    // would cost four registers, and with 8 waves and 8 tokens a sixth of the waves.)
    constexpr float kWeightUnit = kTokenScale ? 0.0625f : 1.0f;
    constexpr int kStart = PG ? 0x49400000 : 0;
    float xsc[kXsc];
    if (kTokenScale) {
#pragma unroll
        for (int i = 0; i < kXsc; ++i) {
            const int m = kByGroup ? stored_token(stored_reg(i)) : (i >> 2) * 16 + (B::kPair ? kb & 1 : kb) * 4 + (i & 3);
            xsc[i] = as_global<float>(xscale)[m < M ? m : M - 1];
        }
    }

    // (up to eight tokens in registers before the first block arrives; with more the compiler's own choice is
    // up to 4 % faster)
    uint32_t wplace[kFresh ? 1 : NG], pplace[kFresh || !B::kPair ? 1 : NG][2];
    if constexpr (!kFresh) {
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            wplace[i] = wpiece(wpos0, i);
            if (TOK == 8) asm volatile("" : "+v"(wplace[i]));
            if constexpr (B::kPair) {
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    pplace[i][h] = pair_at(apos0, i, h);
                    asm volatile("" : "+v"(pplace[i][h]));
                }
            }
        }
    }
#define NVQ_RD32(dst_, addr_, off_) asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(dst_) : "v"(addr_), "n"(off_))
#define NVQ_RD64(dst_, addr_, off_) asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(dst_) : "v"(addr_), "n"(off_))
#define NVQ_RDROWS(dst_, addr_, off_) asm volatile("ds_read2st64_b32 %0, %1 offset0:0 offset1:%2" : "=v"(dst_) : "v"(addr_), "n"(off_))
#define NVQ_RD128(dst_, addr_, off_) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst_) : "v"(addr_), "n"(off_))
    // block b of set u
    auto block = [&](int b, auto set) {
        constexpr int u = decltype(set)::value;
        __builtin_amdgcn_s_waitcnt(slice_vmcnt(0));
        asm volatile("" ::: "memory");
        if (kTokenScale) {
#pragma unroll
            for (float &v : xsc) asm volatile("" : "+v"(v));  // (not to be asked for later)
        }

        constexpr int kSc = B::kScRead;
        uint32_t q[RT][NG], sc[RT][kSc];
        uint32_t wpos = wpos0, apos = apos0;
        if (kFresh) asm volatile("" : "+v"(wpos), "+v"(apos));
        constexpr bool kRows = B::kPair && RT == 2;
        uint2v q2[kRows ? NG : 1], s2[B::kPair && SCB == 16 ? RT : 1];  // weights of both row tiles; scales
        uint2v a2[PREC == NVQ_W4A8 ? 1 : MT][NG][2];
        uint32_t a1[PREC == NVQ_W4A8 ? MT : 1][NG][2];
        float4v xs4[PG ? MT : 1][4][B::kXsRead];
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            if constexpr (kRows) {
                NVQ_RDROWS(q2[i], (kFresh ? wpiece(wpos, i) : wplace[kFresh ? 0 : i]), B::kWTile / 256);
            } else {
#pragma unroll
                for (int r = 0; r < RT; ++r) NVQ_RD32(q[r][i], (kFresh ? wpiece(wpos, i) : wplace[kFresh ? 0 : i]), B::kW + r * B::kWTile);
            }
        }
#pragma unroll
        for (int r = 0; r < RT; ++r) {
            if constexpr (B::kPair && SCB == 16) {
                NVQ_RD64(s2[r], spos, B::kSc + r * 256);
            } else {
#pragma unroll
                for (int k = 0; k < kSc; ++k)
                    NVQ_RD32(sc[r][k], spos, B::kSc + r * (SCB == 16 ? 256 : 64) + k * B::kScStep);
            }
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < NG; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const uint32_t from = B::kPair ? (kFresh ? pair_at(apos, i, h) : pplace[kFresh || !B::kPair ? 0 : i][h])
                                                   : B::kA + apiece_at(apos, i, h);
                    if (PREC == NVQ_W4A8)
                        NVQ_RD32(a1[mt][i][h], from, mt * 16 * B::kTokenBytes);
                    else
                        NVQ_RD64(a2[mt][i][h], from, mt * 16 * B::kTokenBytes);
                }
        if (PG) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                    for (int h = 0; h < B::kXsRead; ++h)
                        NVQ_RD128(xs4[mt][jj][h], xspos, B::kXs + (mt * 16 + jj) * 4 * NG + h * 16);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int r = 0; r < RT; ++r) {
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                if constexpr (kRows) {
                    if (r == 0) asm volatile("" : "+v"(q2[i]));
                } else {
                    asm volatile("" : "+v"(q[r][i]));
                }
            }
            if constexpr (B::kPair && SCB == 16) {
                asm volatile("" : "+v"(s2[r]));
                sc[r][0] = s2[r].x;
                sc[r][1] = s2[r].y;
            } else {
#pragma unroll
                for (int k = 0; k < kSc; ++k) asm volatile("" : "+v"(sc[r][k]));
            }
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                if (PREC == NVQ_W4A8)
                    asm volatile("" : "+v"(a1[mt][i][0]), "+v"(a1[mt][i][1]));
                else
                    asm volatile("" : "+v"(a2[mt][i][0]), "+v"(a2[mt][i][1]));
                if (PG && i < 4 * B::kXsRead) asm volatile("" : "+v"(xs4[mt][i & 3][i >> 2]));
            }
        if (b + 1 < nblk) issue(b + 1);

        const int g0 = NG * (w + W * b);
        auto activation = [&](int mt, int i) {
            if constexpr (PREC == NVQ_W4A8) {
                return (long)((uint64_t)a1[mt][i][0] | ((uint64_t)a1[mt][i][1] << 32));
            } else {
                const uint4v v = {a2[mt][i][0].x, a2[mt][i][0].y, a2[mt][i][1].x, a2[mt][i][1].y};
                return __builtin_bit_cast(bf16x8, v);
            }
        };
        // W4A8: no correction of the offset, the weights enter as 16 (n - 8): the nibble in the high half of
        // its byte, its top bit flipped (see kWeightUnit)
        auto weights = [&](int r, int i) {
            uint32_t v;
            if constexpr (kRows)
                v = q2[i][r];
            else
                v = q[r][i];
            if constexpr (PREC == NVQ_W4A8) {
                const uint32_t lo = ((v << 4) & 0xf0f0f0f0u) ^ 0x80808080u, hi = (v & 0xf0f0f0f0u) ^ 0x80808080u;
                return (long)((uint64_t)lo | ((uint64_t)hi << 32));
            } else {
                return A::weights(v);
            }
        };
        // groups i, and i + 4 in the upper half of a pair
        auto dump = [&](const typename A::offset_t &raw, int i, int r, int mt) {
            const int row = row0 + 16 * r + n, g = g0 + i + 4 * half;
            if (row >= S.rows || !S.dbg || g >= G) return;
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const int m = mt * 16 + (B::kPair ? kb & 1 : kb) * 4 + jj;
                if (m < M) S.dbg[((int64_t)m * S.N + row) * G + g] = ((int)raw[jj] - kStart) / 16;
            }
        };
        // what the lane adds in round i: group i, or i + 4 in the upper half of a pair
        auto add = [&](const float4v &p, int i, int r, int mt) {
            const uint32_t sb = SCB == 2 ? sc[r][i] : sc[r][i >> 1] >> (16 * (i & 1));
            const float sw = half_bits_to_float((uint16_t)sb);
            float (&sum)[4] = f[u][kByGroup ? i : i >> 2][r][mt];
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const float sj = PG ? sw * xs4[PG ? mt : 0][jj][i >> 2][i & 3] : sw;
                sum[jj] = fmaf(sj, p[jj], sum[jj]);
            }
        };
        // A branch ends the last block of a tail early, and others write the sums of a test.  The
        // wait costs up to 5% (W4A8, 32 tokens, 16400 x 2720: 31.0 -> 32.5 us) and nothing at
        // 4096 x 4096.
        constexpr bool kBranches = TAIL || DEBUG;
        // Group i, or the pair of groups i and i + 4: its product with row tile r and token tile mt.
        auto product = [&](int i, int r, int mt, const typename A::offset_t &off) {
            if constexpr (B::kPair) {
                const typename A::offset_t p = A::multiply(activation(0, i), weights(r, i), off);
                return A::multiply(activation(0, i + 4), weights(r, i + 4), p);
            } else {
                return A::multiply(activation(mt, i), weights(r, i), off);
            }
        };
        // W4A16: the constant offset of its weights, for all row tiles
        auto correction = [&](int i, int mt) {
            if constexpr (PREC == NVQ_W4A8)
                return typename A::offset_t{kStart, kStart, kStart, kStart};
            else if constexpr (B::kPair)
                return A::offset(activation(0, i + 4), A::offset(activation(0, i)));
            else
                return A::offset(activation(mt, i));
        };
        auto value = [&](const typename A::offset_t &p) {
            if constexpr (PG)
                return __builtin_bit_cast(float4v, p) - 786432.0f;
            else
                return A::value(p);
        };
        constexpr int kRounds = B::kPair ? 4 : NG;
        if constexpr (PREC == NVQ_W4A8 && MT * RT == 1 && !kBranches) {
            // the products of a round are used when those of the next are on their way (3072 x 8192 at 16 tokens
            // 6.5 us, so 6.3; with more tiles there are enough of them)
            typename A::offset_t p = product(0, 0, 0, correction(0, 0));
#pragma unroll
            for (int i = 0; i < kRounds; ++i) {
                const typename A::offset_t now = p;
                if (i + 1 < kRounds) p = product(i + 1, 0, 0, correction(i + 1, 0));
                add(value(now), i, 0, 0);
            }
        } else {
#pragma unroll
            for (int i = 0; i < kRounds; ++i) {
                if (TAIL && g0 + i >= G) break;  // the last block may end early
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const auto off = correction(i, mt);
#pragma unroll
                    for (int r = 0; r < RT; ++r) {
                        typename A::offset_t p = product(i, r, mt, off);
                        if constexpr (kBranches) wait_written(p);
                        if (DEBUG && PREC == NVQ_W4A8) dump(p, i, r, mt);
                        if (!TAIL || !B::kPair || g0 + i + 4 * half < G) add(value(p), i, r, mt);
                    }
                }
            }
        }
    };
    for (int b = 0; b < nblk; b += U) {
        block(b, std::integral_constant<int, 0>());
        if (U == 2 && b + 1 < nblk) block(b + 1, std::integral_constant<int, U - 1>());
    }
#undef NVQ_RD32
#undef NVQ_RD64
#undef NVQ_RD128
#undef NVQ_RDROWS

    // (row of the tile)
    auto store = [&](int row, int m, float sum) {
        if (row <= last && m < M) store_global(S.y, S.bf16 ? NVQ_BF16 : NVQ_F32, (int64_t)m * S.N + (row0 + row), sum);
    };
    __syncthreads();  // the blocks' LDS is free
    if constexpr (!kByGroup) {
        // the chains one after the other
        float (*const red)[kTile][64] = reinterpret_cast<float (*)[kTile][64]>(lds);
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) {
                const float xs = kTokenScale ? xsc[kByGroup ? 0 : mt * 4 + jj] : 1.0f;
#pragma unroll
                for (int u = 0; u < U; ++u)
#pragma unroll
                    for (int c = 0; c < CR; ++c)
#pragma unroll
                        for (int r = 0; r < RT; ++r)
                            red[C * (w + W * u) + c + half * (C / 2)][(r * MT + mt) * 4 + jj][B::kPair ? lane & 31 : lane] =
                                (kWeightUnit * f[u][c][r][mt][jj]) * xs;
            }
        __syncthreads();
#pragma unroll
        for (int pass = 0; pass < (kTile + W - 1) / W; ++pass) {
            const int reg = pass * W + w;
            if (reg < kTile) {
                float sum = 0.0f;
#pragma unroll
                for (int k = 0; k < V; ++k) sum += red[k][reg][B::kPair ? lane & 31 : lane];
                const int r = reg / (MT * 4), mt = (reg >> 2) % MT, jj = reg & 3;
                store(16 * r + n, mt * 16 + kb * 4 + jj, sum);
            }
        }
    } else {
        // Chain 64 u / U + C w + c.  Those 64 / U apart meet in their wave's registers; then 128
        // results of every chain at a time (two registers of all lanes, or, in pairs, four of half
        // of them) go to LDS, and SH neighbouring lanes share a result: lane t of them adds the
        // chains SH q + t, in pairs, and their sums meet in the lanes.
        constexpr int NQ = W * C / SH;
        float (*const red)[kRedStride] = reinterpret_cast<float (*)[kRedStride]>(lds);
#pragma unroll
        for (int round = 0; round < kRounds; ++round) {
            if (round > 0) __syncthreads();
#pragma unroll
            for (int c = 0; c < CR; ++c)
#pragma unroll
                for (int p = 0; p < kRegs; ++p) {
                    const int reg = kRegs * round + p, r = reg / (MT * 4), mt = (reg >> 2) % MT, jj = reg & 3;
                    const float v = U == 2 ? f[0][c][r][mt][jj] + f[U - 1][c][r][mt][jj] : f[0][c][r][mt][jj];
                    red[C * w + c + half * (C / 2)][B::kPair ? 32 * p + (lane & 31) : 64 * p + lane] = v;
                }
            __syncthreads();
            {
                float v[NQ];
#pragma unroll
                for (int q = 0; q < NQ; ++q) v[q] = red[SH * q + share][result];
#pragma unroll
                for (int apart = NQ / 2; apart > 0; apart >>= 1)
#pragma unroll
                    for (int q = 0; q < apart; ++q) v[q] += v[q + apart];
                if (SH == 4) v[0] += dpp_f32<kDppXor2>(v[0]);
                v[0] += dpp_f32<kDppXor1>(v[0]);
                const int reg = stored_reg(round), r = reg / (MT * 4);
                if (share == 0)
                    store(16 * r + (result & 15), stored_token(reg), (kWeightUnit * v[0]) * (kTokenScale ? xsc[round] : 1.0f));
            }
        }
    }
}

// Two row tiles per workgroup: how many of a phase's tiles get a workgroup of their own, so that every
// compute unit has the same rows.  With a tile or less per unit left over by whole workgroups, those
// of two tiles would give some units two more and others none (28672 rows on 256 units: 128 rows or 96,
// with halves 112; a chain of four such blocks at 8 tokens 190.4 us, so 188.4).  Up to eight tokens: a workgroup
// of one tile multiplies as much as one of two, which is what counts beyond (two 8B blocks, W4A16, 16 tokens:
// 105 us, with halves 108).
inline int slice_halves(const GemvSegs &S) {
    int tiles = 0;
    for (int k = 0; k < S.nseg; ++k) tiles += (S.N[k] + 15) / 16;
    const int cus = device_cu_count(), rest = tiles % (2 * cus);
    return rest <= cus ? rest : 0;
}
// The rows of matrix k in workgroups of two tiles: it has a share of the `halves`, at its end.
inline int slice_whole(const GemvSegs &S, int k, int halves) {
    const int before = k > 0 ? S.row_end[k - 1] : 0, end = S.row_end[k];
    auto share = [&](int rows) { return (int)((int64_t)halves * rows / S.total_rows); };
    const int tiles = (S.N[k] + 15) / 16, whole = (tiles - (share(end) - share(before))) / 2 * 32;
    return whole < S.N[k] ? whole : S.N[k];
}

template <int PREC, bool PG, int TOK, int RT, int W, int NG, int V, int SCB, int NP, int SEGS, bool DEBUG>
int slice_launch(const SliceWork &w, int G, int M, hipStream_t st) {
    SliceArgs<NP, SEGS, DEBUG> a = {};
    int units = 0;
    for (int i = 0; i < NP; ++i) {
        SlicePhase<SEGS, DEBUG> &p = a.phase[i];
        const GemvSegs &S = *w.segs[i];
        int end = 0, seg = 0;
        // rows from .. to - 1 of matrix k, in workgroups of `unit` rows
        auto matrix = [&](int k, int from, int to, int unit) {
            if (to <= from) return;
            p.qw[seg] = S.qw[k] + (int64_t)from * G;
            p.sc[seg] = S.sc[k] + (int64_t)from * G;
            p.y[seg] = static_cast<char *>(S.y[k]) + (int64_t)from * (S.y_dtype[k] == NVQ_BF16 ? 2 : 4);
            p.N[seg] = S.N[k];
            p.rows[seg] = to - from;
            if (S.y_dtype[k] == NVQ_BF16) p.bf16 |= 1u << seg;
            if (unit < 16 * RT) p.bf16 |= 1u << (8 + seg);
            if (DEBUG) p.dbg[DEBUG ? seg : 0] = S.dbg[k];
            end += (to - from + unit - 1) / unit;
            p.unit_end[seg++] = end;
        };
        const int halves = RT == 2 && TOK == 8 && 2 * S.nseg <= SEGS ? slice_halves(S) : 0;
        for (int k = 0; k < S.nseg; ++k) matrix(k, 0, halves ? slice_whole(S, k, halves) : S.N[k], 16 * RT);
        for (int k = 0; k < S.nseg && halves; ++k) matrix(k, slice_whole(S, k, halves), S.N[k], 16);
        for (; seg < SEGS; ++seg) p.unit_end[seg] = end;
        p.x = reinterpret_cast<const char *>(w.x[i]);
        p.xscale = w.xscale[i];
        p.G = G;
        p.M = M;
        units += end;
    }
    hipLaunchKernelGGL((gemv_slice_kernel<PREC, PG, TOK, RT, W, NG, V, SCB, NP, SEGS, DEBUG>), dim3(units), dim3(W * 64), 0,
                       st, a);
    NVQ_HIP_TRY(hipGetLastError());
    return NVQ_OK;
}

template <int PREC, bool PG, int TOK, int RT, int W, int NG, int V, int SCB, bool DEBUG = false>
int slice_go(const SliceWork &w, int G, int M, hipStream_t st) {
    if constexpr (!DEBUG) {  // (only a single call asks for accumulators)
        if (w.n == 2) return slice_launch<PREC, PG, TOK, RT, W, NG, V, SCB, 2, kMaxSeg, false>(w, G, M, st);
        if (w.segs[0]->nseg > 1)
            return slice_launch<PREC, PG, TOK, RT, W, NG, V, SCB, 1, kMaxSeg, false>(w, G, M, st);
    }
    return slice_launch<PREC, PG, TOK, RT, W, NG, V, SCB, 1, 1, DEBUG>(w, G, M, st);
}

// Whether a phase has more than two row tiles per compute unit.
inline bool slice_many(int rows) { return (rows + 15) / 16 > 2 * device_cu_count(); }

// How many chains a result is added in (see above): sixteen where there are at most two row
// tiles per compute unit, so that eight waves share a tile, and every chain still gets two
// columns (8 tokens, 4096 x 14336: 9.5 us against 16.9 with four waves and two tiles each).
inline int slice_chains(const GemvSegs &S, int G, int M, bool per_group) {
    if (per_group || !gemv_mfma_supported(S, G * 32, M)) return 64;
    return G >= 128 && !slice_many(S.total_rows) ? 16 : 8;
}

// Row tiles per workgroup of four waves (eight chains): two where those still make two
// workgroups per compute unit and the tokens' inputs, which every workgroup reads, count.  28672
// x 4096, W4A16: 18.9, 21.7 and 32.0 us at 8, 16 and 32 tokens against 20.4, 26.2 and 39.8 with
// one, W4A8 17.1, 19.2, 26.6 against 17.9, 21.9, 33.3; 16384 x 3072 8.8 to 12.8 against 8.3 to
// 15.4; 12288 x 2048 6.6 to 9.7 against 5.7 to 9.7, and below that one is better at any number of
// tokens (5120 x 3072: 5.2 against 6.1).
inline int slice_row_tiles(int rows) { return rows >= 64 * device_cu_count() ? 2 : 1; }

// Whether a phase has more row tiles than compute units, so that two workgroups share one.
inline bool slice_shared(int rows) { return (rows + 15) / 16 > device_cu_count(); }

// Eight column chains and one row tile: eight waves with half blocks instead of four with whole
// ones, where a compute unit has no second row tile (2048 x 2048, 16 tokens: 3.5 us against 4.0;
// 12288 x 3072 7.6 against 7.1), and at 17 tokens and more (3072 x 3072: 5.7 against 6.7).
inline bool slice_eight_waves(int rows, int tokens) { return tokens > 16 || !slice_shared(rows); }

// The scale loads the phases of a launch allow (see SCB).
inline int slice_scale_bytes(const SliceWork &w, int G) {
    int b = (G & 7) == 0 ? 16 : (G & 1) == 0 ? 4 : 2;
    for (int k = 0; k < w.n; ++k)
        for (int i = 0; i < w.segs[k]->nseg; ++i) {
            if (b == 16 && !aligned(w.segs[k]->sc[i], 16)) b = 4;
            if (b == 4 && !aligned(w.segs[k]->sc[i], 4)) b = 2;
        }
    return b;
}

inline int slice_rows(const SliceWork &w) {
    int rows = 0;
    for (int i = 0; i < w.n; ++i) rows += w.segs[i]->total_rows;
    return rows;
}

}  // namespace

}  // namespace nvq

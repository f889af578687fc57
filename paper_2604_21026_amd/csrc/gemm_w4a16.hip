// nvq_gemm_w4a16: the prefill / large-batch product.  Paper: kernel table (the
// weights are dequantised to 16-bit values, a dense GEMM follows) and the
// remark in the limitations that large batches are bound by compute.  Here the
// two are one kernel: Y[m][n] = sum_k X[m][k] * Wd[n][k] with Wd[n][k] =
// bf16(code[n][k] * scale[n][k/32]) (what nvq_dequant_bf16 stores), bf16 x bf16
// products accumulated in fp32 on the matrix cores; the dense weights never
// exist in memory, a wave dequantises the nibbles it is about to multiply.
//
// v_mfma_f32_32x32x16_bf16: operand A = 32 tokens x 16 inputs, operand B = 16
// inputs x 32 weight rows, lane (i, b) = (lane % 32, lane / 32) supplies eight
// inputs of token / row i.  Which eight is free as long as both operands agree,
// and since the scale is folded into the bf16 weight an MFMA may mix two
// quantisation groups: the kernel advances by pairs of groups (64 inputs), lane
// (i, b) takes its eight inputs from group 2 p + b of pair p, inputs 8 s .. 8 s
// + 7 of that group in MFMA step s = 0..3.  For the activations that is 16
// contiguous bytes; for the weights the lane loads the group's 16 packed bytes
// once (adjacent to the other lane's group: 32 contiguous bytes per row) and
// step s uses the low (s < 2) or high nibbles of bytes 8 (s % 2) .. + 7.
// Nibble -> fp32 (n - 8) * s, exact, round to bf16.
//
// Two kernels, which add the products of a slice of K in the same order:
//  - tiles of 256 tokens x 256 rows ("wide", K a multiple of 256), whose waves dequantise
//    a weight once per 256 tokens: the best rate, if the output has enough of them;
//  - smaller tiles (second half of this file), 32 to 128 tokens x 32 to 256 rows, whose
//    waves share out rows and slices of K, for everything else.
// gemm_choose weighs them by what they were measured to take; with it goes the order of the
// additions (one, two, four or eight slices of K), which therefore depends on the number of tokens.
#include "nvq_internal.h"

#include <cstdlib>
#include <cstring>

namespace nvq {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef float floatx2 __attribute__((ext_vector_type(2)));
typedef _Float16 halfx2 __attribute__((ext_vector_type(2)));
typedef unsigned uint4v __attribute__((ext_vector_type(4)));

constexpr int kGemmThreads = 256;

__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
    const floatx2 f = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f, bf16x2));  // nearest even
}

// ---- wide tiles --------------------------------------------------------------
// 256 tokens x 256 weight rows per workgroup, four waves, one per SIMD with the
// whole register file (the 8 x 2 accumulator tiles of a wave fill 256
// registers): a wave multiplies all 256 tokens by its own 64 rows, so that a
// weight is dequantised once per workgroup and serves eight MFMAs.  K must be a
// multiple of 256 (a pair of groups per step, blocks of four pairs below).
//
// Everything comes from global memory straight into LDS, 16 bytes per lane:
//  - the activations of a pair of groups (256 tokens x 128 bytes, three buffers
//    shared by the waves; 1 KiB = eight whole lines per load instruction);
//  - the packed weights of a wave's 64 rows for two pairs (64 bytes per row:
//    16 half lines per instruction, two buffers per wave) and their scales for
//    four pairs (16 bytes per row, two buffers per wave).  Loaded by the lane
//    that needs them (lane i = row i, 16 bytes of one group) a load instruction
//    touches 32 lines for 1 KiB and the wave stands still while it is taken
//    apart: with the weight loads pointed at one row the kernel ran 25-30 %
//    faster, which is what the detour through LDS is for.
// A row's 16-byte pieces are stored permuted so that the 16 lanes of a quarter
// wave, reading the same piece of 16 consecutive rows, touch every LDS bank once:
// piece c of activation row r at position c ^ ((r / 2) % 8), piece c of weight
// row r at position c ^ ((r / 4) % 4).
typedef __attribute__((address_space(3))) void *lds_void_ptr;

constexpr int kWideTokens = 256, kWideRows = 256;
constexpr int kWideBuf = kWideTokens * 128;  // bytes of one activation buffer
constexpr int kWideBw = 64 * 64;             // a wave's packed weights of two pairs
constexpr int kWideBs = 64 * 16;             // a wave's scales of four pairs
constexpr int kWideLds = 3 * kWideBuf + 4 * 2 * (kWideBw + kWideBs);

// s_waitcnt immediate that waits for vmcnt <= n only
constexpr int wide_vmcnt(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0f70; }

// Whether bf16 results leave as 16 bytes per lane: N rows of a launch, ldy from token to token.  (A launch of
// part of the rows can have whole eights of them where the result's rows are no multiple of 16 bytes apart.)
__host__ __device__ inline bool gemm_whole_stores(int N, int ldy, const void *y) {
    return ((N | ldy) & 7) == 0 && (reinterpret_cast<uintptr_t>(y) & 15) == 0;
}

template <bool F32>
__global__ __launch_bounds__(kGemmThreads) __attribute__((amdgpu_waves_per_eu(1, 1))) void
gemm_w4a16_wide_kernel(const unsigned char *__restrict__ qw, const unsigned char *__restrict__ sc,
                       int N, int G, const unsigned char *__restrict__ x, int M,
                       void *__restrict__ y, int ldy) {
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kWideLds];
    unsigned char *const xa = lds;
    const int t = threadIdx.x, lane = t & 63;
    const int wave = __builtin_amdgcn_readfirstlane(t >> 6);
    unsigned char *const bw = lds + 3 * kWideBuf + wave * 2 * kWideBw;
    unsigned char *const bs = lds + 3 * kWideBuf + 4 * 2 * kWideBw + wave * 2 * kWideBs;
    const int li = lane & 31, lb = lane >> 5;
    // Tiles in token-major order, weight rows fastest.  (Giving each XCD, with its
    // own L2, a contiguous eighth of the tiles, so that its workgroups share one or
    // two token tiles, changed the time by -1..+3 %; starting every workgroup at a
    // different place along K made it 3-7 % slower; reading the inputs from LDS two
    // steps ahead instead of one changed nothing.)
    const int nx = (N + kWideRows - 1) / kWideRows;
    const int tile = (int)blockIdx.x;
    const int m0 = (tile / nx) * kWideTokens, n0 = (tile % nx) * kWideRows;
    const int P = G >> 1;  // pairs of groups, a multiple of 4

    // Activation loads: instruction j of this wave fills rows 8 (8 wave + j) ..
    // + 7 of a buffer, lane l the position l % 8 of row l / 8 of those (rows past
    // the last token: the last token again; those results are not stored).
    // Addresses are a base common to the wave plus a 32-bit offset per lane (the
    // form a load instruction takes without any address arithmetic in the lanes).
    const unsigned char *const xbase = x + (size_t)m0 * (size_t)(G * 64);
    uint32_t xo[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int r = 8 * (8 * wave + j) + (lane >> 3);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        const int rc = m0 + r < M ? r : M - 1 - m0;
        xo[j] = (uint32_t)rc * (uint32_t)(G * 64) + 16u * (uint32_t)c;
    }
    auto issue_a1 = [&](unsigned char *buf, int p, int j) {
        __builtin_amdgcn_global_load_lds((const void *)(xbase + (size_t)p * 128 + xo[j]),
                                         (lds_void_ptr)(buf + (8 * wave + j) * 1024), 16, 0, 0);
    };
    // Weight loads: instruction j fills rows 16 j .. + 15 of a weight buffer, lane l
    // the position l % 4 of row l / 4 of those (rows past the last one: the last one
    // again).  Scale load: lane l the 16 bytes of row l.
    const int nw = n0 + wave * 64 < N ? n0 + wave * 64 : N - 1;  // the wave's first row
    const unsigned char *const qbase = qw + (size_t)nw * (size_t)(G * 16);
    const unsigned char *const sbase = sc + (size_t)nw * (size_t)(G * 2);
    uint32_t qo[4], so;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const int r = 16 * j + (lane >> 2);
        const int c = (lane & 3) ^ ((r >> 2) & 3);
        const int rc = nw + r < N ? r : N - 1 - nw;
        qo[j] = (uint32_t)rc * (uint32_t)(G * 16) + 16u * (uint32_t)c;
    }
    so = (uint32_t)(nw + lane < N ? lane : N - 1 - nw) * (uint32_t)(G * 2);
    // block b2 = pairs 2 b2, 2 b2 + 1 into weight buffer `sel`; block b4 = pairs 4 b4 .. + 3
    auto issue_bw1 = [&](int b2, int sel, int j) {
        __builtin_amdgcn_global_load_lds((const void *)(qbase + (size_t)b2 * 64 + qo[j]),
                                         (lds_void_ptr)(bw + sel * kWideBw + j * 1024), 16, 0, 0);
    };
    auto issue_bs = [&](int b4, int sel) {
        __builtin_amdgcn_global_load_lds((const void *)(sbase + (size_t)b4 * 16 + so),
                                         (lds_void_ptr)(bs + sel * kWideBs), 16, 0, 0);
    };

    floatx16 acc[8][2];
#pragma unroll
    for (int tt = 0; tt < 8; ++tt)
#pragma unroll
        for (int rt = 0; rt < 2; ++rt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[tt][rt][r] = 0.0f;

    // The lane's LDS positions.  Activations: row li of a token tile, piece 4 lb +
    // st in MFMA step st.  Weights: row li of a row tile, the group lb of the first
    // pair of a block (the second pair: the position ^ 2); scales: row li, group lb
    // of the first pair of a block of four.
    const uint32_t xa0 = (uint32_t)(uintptr_t)xa;
    uint32_t apos[4];
#pragma unroll
    for (int st = 0; st < 4; ++st) apos[st] = li * 128 + 16 * ((4 * lb + st) ^ ((li >> 1) & 7));
    const uint32_t bwpos = (uint32_t)(uintptr_t)bw + li * 64 + 16 * (lb ^ ((li >> 2) & 3));
    const uint32_t bspos = (uint32_t)(uintptr_t)bs + li * 16 + 2 * lb;

    // The loop is a chain of MFMA steps (four per pair of groups, 16 inputs per
    // lane half each).  Everything else is dealt between the sixteen MFMAs of a
    // step, a little after each, so that the matrix core never waits for more
    // than a few instructions: the eight LDS reads of the next step's inputs, the
    // conversion of the next step's sixteen weights (byte -> fp32, one FMA with
    // the scale, every other time the rounding of two to bf16), in step 1 the LDS
    // reads of the next pair's packed weights, in step 2 their unpacking and in
    // step 3 the loads from global memory.  The step after step 3 is step 0 of the
    // next pair.  LDS accesses are written as instructions with their own waits:
    // before an LDS access it knows of, the compiler waits for every load in flight.
    struct BRaw {  // the lane's packed weights and scales of a pair, per row tile
        uint4v w[2];
        uint32_t h[2];
    };
    struct Nibbles {  // one nibble per byte, [row tile][low, high][dword]; the high ones times 16
        uint32_t d[2][2][4];
        float s[2][2];  // scale for the low nibbles, scale / 16 for the high ones
        float m8[2];    // -8 * scale
    };
    // piece k of 10: the low and high nibbles of a dword (k < 8), the scale of a row tile
    auto unpack1 = [&](const BRaw &b, Nibbles &nb, int k) {
        if (k < 8) {
            const int rt = k >> 2, i = k & 3;
            const uint32_t d = b.w[rt][i];
            nb.d[rt][0][i] = d & 0x0f0f0f0fu;
            nb.d[rt][1][i] = d & 0xf0f0f0f0u;
            // the bytes are converted one by one; seen through, the compiler
            // extracts each nibble from d again with an instruction of its own
            asm("" : "+v"(nb.d[rt][0][i]));
            asm("" : "+v"(nb.d[rt][1][i]));
        } else {
            const int rt = k - 8;
            nb.s[rt][0] = half_bits_to_float((uint16_t)b.h[rt]);
            nb.s[rt][1] = 0.0625f * nb.s[rt][0];  // exact
            nb.m8[rt] = -8.0f * nb.s[rt][0];
        }
    };
    // weight i (0..15) of MFMA step st: row tile i / 8, input i % 8 of the step
    auto weight = [&](const Nibbles &nb, int st, int i) -> float {
        const int rt = i >> 3, e = i & 7;
        const uint32_t d = nb.d[rt][st >> 1][2 * (st & 1) + (e >> 2)];
        return fmaf((float)((d >> (8 * (e & 3))) & 0xffu), nb.s[rt][st >> 1], nb.m8[rt]);
    };
    auto read_input = [&](uint32_t addr, int tt, uint4v &a) {
        switch (tt) {
#define NVQ_RD(t_) case t_: asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(a) : "v"(addr), "n"(t_ * 4096)); break;
            NVQ_RD(0) NVQ_RD(1) NVQ_RD(2) NVQ_RD(3) NVQ_RD(4) NVQ_RD(5) NVQ_RD(6) NVQ_RD(7)
#undef NVQ_RD
        }
    };
    // piece 0, 1: the packed weights of row tile 0, 1 (32 rows = 2 KiB further); 2, 3: the scales
    auto read_b1 = [&](uint32_t waddr, uint32_t saddr, BRaw &b, int piece) {
        switch (piece) {
            case 0: asm volatile("ds_read_b128 %0, %1" : "=v"(b.w[0]) : "v"(waddr)); break;
            case 1: asm volatile("ds_read_b128 %0, %1 offset:2048" : "=v"(b.w[1]) : "v"(waddr)); break;
            case 2: asm volatile("ds_read_u16 %0, %1" : "=v"(b.h[0]) : "v"(saddr)); break;
            case 3: asm volatile("ds_read_u16 %0, %1 offset:512" : "=v"(b.h[1]) : "v"(saddr)); break;
        }
    };
    uint4v a[2][8];
    uint32_t bo[2][2][4];  // [step parity][row tile] bf16 x 8
    BRaw braw;             // of the next pair
    Nibbles nba, nbb;      // of the pair being multiplied and of the next one, in turn
    auto arrived = [&](uint4v (&v)[8]) {
        asm volatile("s_waitcnt lgkmcnt(0)"
                     : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(v[4]), "+v"(v[5]),
                       "+v"(v[6]), "+v"(v[7]), "+v"(braw.w[0]), "+v"(braw.w[1]), "+v"(braw.h[0]),
                       "+v"(braw.h[1]));
    };

    // The loads from global memory that belong to pair p: the activations of pair p +
    // 3 (eight instructions), for even p before them the weight block p / 2 + 2
    // (four), for p % 4 == 0 before those the scale block p / 4 + 1 (one): a list of
    // `kind` = 13, 8, 12 or 8 instructions.  They are dealt over four steps (step 3
    // of pair p, where the buffer of pair p becomes free, and steps 0..2 of pair p +
    // 1), a quarter of the list each, one every fourth MFMA: a load instruction holds
    // up the wave that issues it while the address unit is busy, and the four waves
    // of a workgroup issue theirs at the same time.
    auto load_op = [&](int kind, int quarter, int m, unsigned char *abuf, int pa, int b2, int wsel,
                       int b4, int ssel) {
        const int first = kind == 13 ? (quarter == 0 ? 0 : 1 + 3 * quarter) : (kind / 4) * quarter;
        const int count = kind == 13 ? (quarter == 0 ? 4 : 3) : kind / 4;
        if (m >= count) return;
        int k = first + m;
        if (kind == 13) {
            if (k == 0) {
                issue_bs(b4, ssel);
                return;
            }
            k -= 1;
        }
        if (kind >= 12) {
            if (k < 4) {
                issue_bw1(b2, wsel, k);
                return;
            }
            k -= 4;
        }
        issue_a1(abuf, pa, k);
    };

    // Step `st` of the pair in registers (a[st % 2], bo[st % 2]) while the operands
    // of step `nst` of the pair at `nbuf` with the nibbles `wn` are made.  extra =
    // 1: also reads the next pair's packed weights from LDS (at waddr / saddr);
    // extra = 2: also unpacks them into wnext.  Every step issues a quarter of a list
    // of loads (kind, quarter): the activations of pair pa into abuf, the weight
    // block b2 into buffer wsel, the scale block b4 into buffer ssel.
    auto step = [&](int st, uint32_t nbuf, const Nibbles &wn, Nibbles &wnext, int nst, int extra,
                    uint32_t waddr, uint32_t saddr, int kind, int quarter, unsigned char *abuf, int pa,
                    int b2, int wsel, int b4, int ssel) {
        const int c = st & 1, n = c ^ 1;
        const uint32_t addr = nbuf + apos[nst];
        float prev = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const int tt = i >> 1, rt = i & 1;
            acc[tt][rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_bit_cast(bf16x8, a[c][tt]),
                __builtin_bit_cast(bf16x8, make_uint4(bo[c][rt][0], bo[c][rt][1], bo[c][rt][2], bo[c][rt][3])),
                acc[tt][rt], 0, 0, 0);
            if (i < 8) read_input(addr, i, a[n][i]);
            const float w = weight(wn, nst, i);
            if (i & 1) bo[n][i >> 3][(i & 7) >> 1] = pack_bf16(prev, w);
            prev = w;
            if (extra == 1 && i >= 8 && i < 12) read_b1(waddr, saddr, braw, i - 8);
            if (extra == 2 && i >= 4 && i < 14) unpack1(braw, wnext, i - 4);
            if ((i & 3) == 2) load_op(kind, quarter, i >> 2, abuf, pa, b2, wsel, b4, ssel);
            __builtin_amdgcn_sched_barrier(0);
        }
        arrived(a[n]);
    };

#define NVQ_PIN asm volatile("" ::: "memory")
    // Before the loop: the activations of pairs 0 and 1 and the first quarter of
    // those of pair 2 (the rest follows in steps 0..2 of pair 0, as in every turn of
    // the loop), the weights of pairs 0..3 and their scales; pair 0 unpacked and its
    // first operands in registers.
    const int last2 = (P >> 1) - 1, last4 = (P >> 2) - 1;
    auto pair_or_last = [&](int q) { return q < P ? q : P - 1; };
    issue_bs(0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) issue_bw1(0, 0, j);
#pragma unroll
    for (int j = 0; j < 4; ++j) issue_bw1(1 < last2 ? 1 : last2, 1, j);
#pragma unroll
    for (int q = 0; q < 2; ++q)
#pragma unroll
        for (int j = 0; j < 8; ++j) issue_a1(xa + q * kWideBuf, pair_or_last(q), j);
#pragma unroll
    for (int j = 0; j < 2; ++j) issue_a1(xa + 2 * kWideBuf, pair_or_last(2), j);
    NVQ_PIN;
    __builtin_amdgcn_s_waitcnt(wide_vmcnt(0));
    __builtin_amdgcn_s_barrier();
    NVQ_PIN;
#pragma unroll
    for (int piece = 0; piece < 4; ++piece) read_b1(bwpos, bspos, braw, piece);
#pragma unroll
    for (int tt = 0; tt < 8; ++tt) read_input(xa0 + apos[0], tt, a[0][tt]);
    arrived(a[0]);
#pragma unroll
    for (int k = 0; k < 10; ++k) unpack1(braw, nba, k);
    {
        float prev = 0.0f;
#pragma unroll
        for (int i = 0; i < 16; ++i) {
            const float w = weight(nba, 0, i);
            if (i & 1) bo[0][i >> 3][(i & 7) >> 1] = pack_bf16(prev, w);
            prev = w;
        }
    }

    // Four pairs per turn (a block of scales, two blocks of weights); pair p = 4 k +
    // i has a list of 13, 8, 12, 8 loads for i = 0..3.  The wait before step 3 of pair
    // p lets the list of pair p - 1 (begun in step 3 of that pair, ended in step 2 of
    // this one) stay in flight and ends all older loads: A(p + 1), read right after the
    // barrier, is in the list of pair p - 2, and the weights and scales of pair p + 2,
    // read from LDS in step 1 of pair p + 1, are in that of pair p - 2 or older.
    int cur = 0, prv = 2 * kWideBuf;  // byte offsets of the activation buffers of pairs p and p - 1
    int ssel = 0;                     // scale buffer of the pairs 4 k .. 4 k + 3
    for (int p = 0; p < P; p += 4) {
        // i_: place of the pair in the turn; kprev_, kind_: the lists of pairs p - 1 and p
#define NVQ_PAIR(i_, kprev_, kind_, nb, nnb)                                                     \
    do {                                                                                         \
        const int q_ = (i_) + 1; /* the next pair's place in its blocks */                       \
        const uint32_t waddr_ = (bwpos + ((q_ >> 1) & 1) * kWideBw) ^ ((q_ & 1) * 32);           \
        const uint32_t saddr_ = bspos + (((q_ >> 2) ? ssel ^ 1 : ssel)) * kWideBs + (q_ & 3) * 4; \
        const int nxt_ = cur + kWideBuf == 3 * kWideBuf ? 0 : cur + kWideBuf;                    \
        /* the list of the pair before: its activations go to that pair's buffer */             \
        const int pp_ = p + (i_) - 1;                                                            \
        const int pa_ = pair_or_last(pp_ + 3);                                                   \
        const int pb2_ = (pp_ >> 1) + 2 < last2 ? (pp_ >> 1) + 2 : last2;                        \
        const int pb4_ = (p >> 2) + 1 < last4 ? (p >> 2) + 1 : last4;                            \
        const int pws_ = (((i_) + 3) >> 1) & 1; /* ((i - 1) / 2) % 2 for i = 1..3 */             \
        step(0, xa0 + cur, nb, nnb, 1, 0, 0, 0, kprev_, 1, xa + prv, pa_, pb2_, pws_, pb4_,      \
             ssel ^ 1);                                                                          \
        step(1, xa0 + cur, nb, nnb, 2, 1, waddr_, saddr_, kprev_, 2, xa + prv, pa_, pb2_, pws_,  \
             pb4_, ssel ^ 1);                                                                    \
        step(2, xa0 + cur, nb, nnb, 3, 2, 0, 0, kprev_, 3, xa + prv, pa_, pb2_, pws_, pb4_,      \
             ssel ^ 1);                                                                          \
        __builtin_amdgcn_s_waitcnt(wide_vmcnt(kprev_));                                          \
        __builtin_amdgcn_s_barrier();                                                            \
        NVQ_PIN;                                                                                 \
        {                                                                                        \
            const int b2_ = ((p + (i_)) >> 1) + 2;                                               \
            step(3, xa0 + nxt_, nnb, nb, 0, 0, 0, 0, kind_, 0, xa + cur, pair_or_last(p + (i_) + 3), \
                 b2_ < last2 ? b2_ : last2, ((i_) >> 1) & 1, pb4_, ssel ^ 1);                    \
        }                                                                                        \
        NVQ_PIN;                                                                                 \
        prv = cur;                                                                               \
        cur = nxt_;                                                                              \
    } while (0)
        NVQ_PAIR(0, 8, 13, nba, nbb);
        NVQ_PAIR(1, 13, 8, nbb, nba);
        NVQ_PAIR(2, 8, 12, nba, nbb);
        NVQ_PAIR(3, 12, 8, nbb, nba);
#undef NVQ_PAIR
        ssel ^= 1;
    }
#undef NVQ_PIN
    // no load into LDS may outlive the wave
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    // Result tile: lane (j, b) holds weight row j; register r holds token
    // 8 * (r / 4) + 4 * b + r % 4 of a 32 x 32 tile.
    if (!F32 && gemm_whole_stores(N, ldy, y)) {
        // bf16 results pass through LDS (free now), so that they leave as whole
        // 128-byte lines, 16 bytes per lane, instead of 2 bytes per lane: a wave's
        // 256 tokens x 64 rows in 32 KiB, a row of 128 bytes per token with its
        // 16-byte pieces permuted (piece c at position c ^ ((token / 4) % 8): the two
        // halves of the wave write tokens four apart).
        __builtin_amdgcn_s_barrier();  // every wave has left the loop: nothing reads or fills LDS
        unsigned char *const out = lds + wave * (kWideTokens * 128);
#pragma unroll
        for (int tt = 0; tt < 8; ++tt)
#pragma unroll
            for (int rt = 0; rt < 2; ++rt)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int tok = tt * 32 + 8 * (r >> 2) + 4 * lb + (r & 3);
                    const int nl = rt * 32 + li;
                    const int pos = (nl >> 3) ^ ((tok >> 2) & 7);
                    *reinterpret_cast<uint16_t *>(out + tok * 128 + pos * 16 + (nl & 7) * 2) =
                        float_to_bf16_bits(acc[tt][rt][r]);
                }
        // the wave reads back what it wrote itself
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        const int nb0 = n0 + wave * 64;
#pragma unroll 4
        for (int i = 0; i < 32; ++i) {
            const int idx = i * 64 + lane;
            const int tok = idx >> 3, pos = idx & 7;
            const int c = pos ^ ((tok >> 2) & 7);
            const uint4 v = *reinterpret_cast<const uint4 *>(out + tok * 128 + pos * 16);
            const int m = m0 + tok, n = nb0 + c * 8;
            if (m < M && n < N)
                *reinterpret_cast<uint4 *>(reinterpret_cast<uint16_t *>(y) + (size_t)m * ldy + n) = v;
        }
        return;
    }
#pragma unroll
    for (int tt = 0; tt < 8; ++tt)
#pragma unroll
        for (int rt = 0; rt < 2; ++rt) {
            const int n = n0 + wave * 64 + rt * 32 + li;
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int m = m0 + tt * 32 + 8 * (r >> 2) + 4 * lb + (r & 3);
                if (m < M && n < N) {
                    if (F32)
                        reinterpret_cast<float *>(y)[(size_t)m * ldy + n] = acc[tt][rt][r];
                    else
                        reinterpret_cast<uint16_t *>(y)[(size_t)m * ldy + n] =
                            float_to_bf16_bits(acc[tt][rt][r]);
                }
            }
        }
}

// ---- smaller tiles -----------------------------------------------------------
// For outputs too small to give every compute unit a 256 x 256 tile: a workgroup of four or
// eight waves owns 32 TT tokens x 32 RT WN weight rows; WN waves lie side by side along
// the rows (each 32 RT of them, all the tokens) and WK share out K in blocks of
// two pairs of groups (128 inputs), slice k the blocks k, k + WK, ...; the partial tiles
// are added through LDS in slice order at the end.  As with the wide tiles everything
// goes straight from global memory into LDS, 16 bytes per lane,
//  - the activations of a slice's pair (128 bytes per token, three buffers; the WN waves
//    of a slice load and read them together, one barrier per pair, none for WN = 1),
//  - a wave's packed weights of a block (64 bytes per row, two buffers; an instruction
//    covers 16 rows: loaded by the lane that needs them it touches 32 lines, which took a
//    third of the time),
//  - its scales of a block (two buffers; 4 bytes per row and pair, or 2 per row and group with
//    TAIL; a row's lie with neighbouring lanes, since what a load costs is the lines that its lanes
//    touch: with each row's in 64 lines of two loads a 48-token prompt waited as long for 6 % of the
//    bytes as for the weights.  48 x 2048 x 2048: 6.2 -> 5.4 us, 48 x 2048 x 8192 12.9 -> 11.4; with TAIL
//    48 x 2048 x 8224 12.4 -> 11.9, but 100 x 8192 x 2880 in 128 x 64 17.7 -> 18.1: with four token
//    tiles TAIL keeps a lane's own scales),
// in the wide kernel's permuted order, and everything besides the MFMAs is dealt between
// them.  TAIL: the number of groups is no multiple of four (a block then ends past the
// row: the last group again, with scale 0) or the scales are not aligned to 4 bytes.
//
// What bounds it: the activations' way from L2 into the compute units (about 50 bytes
// per ns and unit with all of them busy: a 64 x 64 tile moves 10 KiB per 0.5 MFLOP and is
// held by that, at 580 TFLOP/s; 128 x 128 moves half as much per FLOP, 128 x 256 with one
// slice a third) and the vector work of the dequantisation, which serves 64 or 128 tokens;
// against both stands the number of tiles, which has to fill 256 compute units.  One 64 x
// 64 tile, in us: 4.2 + 0.6 per pair.  1024 tokens x 4096 rows x K = 4096: 39 us, against
// 78 of the wide tiles (64 of them); 333 x 3072 x 3072: 17 against 69 of the 256 x 128
// tiles that took these before; 48 x 2048 x 8192: 16 against 173.
//
// Eight waves instead of four, so that two share a SIMD, where that was measured to be faster: with
// TAIL 128 x 256 and 128 x 128, whose addresses cost more instructions per load (1300 x 17280 x 2880:
// 179 -> 159 us, 900 x 4288 x 2880 47 -> 40, 600 x 2880 x 8640 at 128 x 128 64.6 -> 57.0; without TAIL
// a call alone gains 2-5 %, a prompt's calls one after the other, at the clock the power limit
// leaves, nothing: 704 tokens of 3B 183 -> 187); and 32 x 32 with K in eight slices, for prompts
// that four slices of 64 tokens leave on a quarter of the machine (48 x 2048 x 8192: 17.2 -> 13.8, 40 x
// 4096 x 14336: 26.8 -> 21.9).  Not for the others: two waves that share rows dequantise them twice
// (128 x 64 12.1 -> 14.0, 64 x 32 7.2 -> 8.9), and 32 rows per wave instead of 64 read the
// activations twice from LDS (64 x 64 8.8 -> 9.5).
//
// Nibble -> weight: a nibble under the bits of the fp16 number 1024 is 1024 + n (in bits
// 4-7: 1024 + 16 n), two per instruction, and a mixed-precision FMA takes the fp16 halves
// as they are: (1024 + n) * s - 1032 * s, one rounding of a number that needs none (n - 8
// has 4, s 11 significant bits).  17 instructions per 8 weights against 23 through bytes.
constexpr int kBand = 4;

template <bool F32, int TT, int RT, int WN, int WK, bool TAIL>
__global__ __launch_bounds__(WN * WK * 64) __attribute__((amdgpu_waves_per_eu(WN * WK / 4, WN * WK / 4))) void
gemm_w4a16_tile_kernel(const unsigned char *__restrict__ qw, const unsigned char *__restrict__ sc,
                         int N, int G, const unsigned char *__restrict__ x, int M, int row_tiles,
                         int token_tiles, void *__restrict__ y, int ldy) {
    constexpr int kWaves = WN * WK;
    constexpr int NM = TT * RT;           // MFMAs of a step (16 inputs per lane half)
    constexpr int kTokens = 32 * TT, kBufA = kTokens * 128;  // bytes of an activation buffer
    constexpr int NA = 4 * TT / WN;       // activation loads of a wave and pair
    static_assert(NA * WN == 4 * TT && kWaves % 4 == 0, "whole instructions; waves on every SIMD");
    constexpr int kW = RT * 32 * 64;      // packed weights of a block
    constexpr int kS = TAIL ? RT * 512 : RT * 256;  // scales of a block
    constexpr int kLds = WK * 3 * kBufA + kWaves * (2 * kW + 2 * kS);
    constexpr int kRegs = TT * RT * 16;   // result registers per lane
    constexpr bool kNear = !TAIL || TT < 4;  // neighbouring lanes load the scales of one row
    constexpr int kScOps = TAIL ? 2 * RT : RT, kWOps = 2 * RT;
    constexpr int kEven = kWOps + kScOps + NA, kOdd = NA;  // loads of an even and an odd pair's list
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kLds];

    // Tiles are numbered along the tokens first, beyond eight token tiles in bands of kBand of them; workgroup b
    // runs on XCD b % 8 and takes one of that XCD's eighth of the numbers, so that its 32 workgroups share
    // a few token tiles and a few row ranges in their L2.  Without the bands an XCD's workgroups all
    // read other activations where there are 32 token tiles: 128 x 64 then waited for the memory behind
    // L2 (4096 tokens, 2560 rows, K = 8192: 372 us, 203 with bands of 4; 128 x 128 212 -> 185, 128 x
    // 256 224 -> 222).  Bands of 8: within 2 %; 2 and 16: up to 4 and 7 % slower.  Five to eight token tiles
    // are one band: cut in two the second is a narrow one that reads its weights for few tokens (259 x 1472 x 4320
    // 13.5 us, so 12.3, 148 x 1536 x 4992 10.0 and 9.2; 213 drawn products of so many tiles 1 % faster on average).
    const int tiles = row_tiles * token_tiles, per_xcd = (tiles + 7) >> 3;
    const int tile = ((int)blockIdx.x & 7) * per_xcd + ((int)blockIdx.x >> 3);
    if (tile >= tiles) return;
    int band0 = 0, width = token_tiles, in_band = tile;
    if (token_tiles > 2 * kBand) {
        band0 = tile / (row_tiles * kBand) * kBand;
        width = token_tiles - band0 < kBand ? token_tiles - band0 : kBand;
        in_band = tile - row_tiles * band0;
    }
    const int row_tile = in_band / width, token_tile = band0 + in_band % width;

    const int t = threadIdx.x, lane = t & 63;
    const int w = __builtin_amdgcn_readfirstlane(t >> 6);
    const int li = lane & 31, lb = lane >> 5;
    const int m0 = token_tile * kTokens;
    const int wn = w % WN, wk = w / WN;  // the wave's rows and slice of K
    const int n0 = row_tile * (32 * RT * WN) + wn * (32 * RT) < N ? row_tile * (32 * RT * WN) + wn * (32 * RT)
                                                                   : N - 1;  // the wave's first row
    unsigned char *const xa = lds + wk * 3 * kBufA;
    unsigned char *const bw = lds + WK * 3 * kBufA + w * (2 * kW + 2 * kS);
    unsigned char *const bs = bw + 2 * kW;

    const int NB = (G + 3) >> 2;  // blocks
    // Blocks of this wave's slice, and of the longest (waves that share activations meet at
    // barriers, of which all of the workgroup must see as many).  Nothing is multiplied past
    // the end of K except by the zero scale of an odd last group's missing partner.
    const int nblk = NB > wk ? (NB - wk + WK - 1) / WK : 0, nblk_max = (NB + WK - 1) / WK;

    // Activation loads: instruction j fills rows 8 j .. + 7 of a buffer, lane l position
    // l % 8 of row l / 8 (past the last token: the last token again; not stored).  Weight
    // loads: instruction j rows 16 j .. + 15, lane l position l % 4 of row l / 4.
    const unsigned char *const xbase = x + (size_t)m0 * (size_t)(G * 64);
    uint32_t xo[NA];
#pragma unroll
    for (int j = 0; j < NA; ++j) {
        const int r = 8 * (NA * wn + j) + (lane >> 3);
        const int c = (lane & 7) ^ ((r >> 1) & 7);
        xo[j] = (uint32_t)(m0 + r < M ? r : M - 1 - m0) * (uint32_t)(G * 64) + (TAIL ? 0u : 16u * (uint32_t)c);
    }
    const int xc0 = (lane & 7) ^ (lane >> 4), xc1 = xc0 ^ 4;  // the piece, even and odd j
    const unsigned char *const qbase = qw + (size_t)n0 * (size_t)(G * 16);
    const unsigned char *const sbase = sc + (size_t)n0 * (size_t)(G * 2);
    const int qc = (lane & 3) ^ ((lane >> 4) & 3);
    uint32_t qo[2 * RT], so[kScOps];
#pragma unroll
    for (int j = 0; j < 2 * RT; ++j) {
        const int r = 16 * j + (lane >> 2);
        qo[j] = (uint32_t)(n0 + r < N ? r : N - 1 - n0) * (uint32_t)(G * 16) + (TAIL ? 0u : 16u * (uint32_t)qc);
    }
#pragma unroll
    for (int k = 0; k < kScOps; ++k) {
        // lane l the scales of pair l % 2 of row l / 2; TAIL: of group l % 4 of row l / 4, or its own of pair k / RT
        const int r = !TAIL ? 32 * k + (lane >> 1) : kNear ? 16 * k + (lane >> 2) : 32 * (k % RT) + li;
        so[k] = (uint32_t)(n0 + r < N ? r : N - 1 - n0) * (uint32_t)(G * 2) + (TAIL ? 0u : 4u * (uint32_t)(lane & 1));
    }
    const int last = nblk > 0 ? nblk - 1 : 0;
    auto group_of = [&](int b) { return 4 * (wk + WK * (b < last ? b : last)); };  // first group of block b
    auto clamp_g = [&](int g) { return g < G ? g : G - 1; };
    auto issue_a1 = [&](unsigned char *buf, int q, int j) {  // of the wave's pair q
        const int g0 = group_of(q >> 1) + 2 * (q & 1);
        const unsigned char *src;
        if (TAIL) {
            const int c = ((NA * wn + j) & 1) ? xc1 : xc0;
            src = xbase + (xo[j] + 64u * (uint32_t)clamp_g(g0 + (c >> 2)) + 16u * (uint32_t)(c & 3));
        } else {
            src = xbase + (size_t)g0 * 64 + xo[j];
        }
        __builtin_amdgcn_global_load_lds((const void *)src, (lds_void_ptr)(buf + (NA * wn + j) * 1024), 16, 0, 0);
    };
    auto issue_w1 = [&](int b, int sel, int j) {
        const int g0 = group_of(b);
        const unsigned char *src = TAIL ? qbase + (qo[j] + 16u * (uint32_t)clamp_g(g0 + qc))
                                        : qbase + (size_t)g0 * 16 + qo[j];
        __builtin_amdgcn_global_load_lds((const void *)src, (lds_void_ptr)(bw + sel * kW + j * 1024), 16, 0, 0);
    };
    auto issue_s1 = [&](int b, int sel, int k) {
        const int g0 = group_of(b);
        if (TAIL) {
            const unsigned char *src = sbase + (so[k] + 2u * (uint32_t)clamp_g(g0 + (kNear ? lane & 3 : 2 * (k / RT) + lb)));
            __builtin_amdgcn_global_load_lds((const void *)src, (lds_void_ptr)(bs + sel * kS + k * 256), 2, 0, 0);
        } else {
            const unsigned char *src = sbase + (size_t)g0 * 2 + so[k];
            __builtin_amdgcn_global_load_lds((const void *)src, (lds_void_ptr)(bs + sel * kS + k * 256), 4, 0, 0);
        }
    };
    // op k of the list of pair q: even q the weights and scales of block q / 2 + 2 and the
    // activations of pair q + 3, odd q those alone; quarter `qu` of the list
    auto load_op = [&](int q, bool even, int sel, unsigned char *abuf, int k) {
        if (even) {
            if (k < kWOps) return issue_w1((q >> 1) + 2, sel, k);
            k -= kWOps;
            if (k < kScOps) return issue_s1((q >> 1) + 2, sel, k);
            k -= kScOps;
        }
        issue_a1(abuf, q + 3, k);
    };

    floatx16 acc[TT][RT];
#pragma unroll
    for (int tt = 0; tt < TT; ++tt)
#pragma unroll
        for (int rt = 0; rt < RT; ++rt)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[tt][rt][r] = 0.0f;

    const uint32_t xa0 = (uint32_t)(uintptr_t)xa;
    uint32_t apos[4];
#pragma unroll
    for (int st = 0; st < 4; ++st) apos[st] = xa0 + li * 128 + 16 * ((4 * lb + st) ^ ((li >> 1) & 7));
    const uint32_t bwpos = (uint32_t)(uintptr_t)bw + li * 64 + 16 * (lb ^ ((li >> 2) & 3));
    const uint32_t bspos = (uint32_t)(uintptr_t)bs + (!TAIL ? 8 * li : kNear ? 16 * li + 4 * lb : 4 * lane);
    uint32_t mask_lo = 0x000f000fu, mask_hi = 0x00f000f0u, magic = 0x64006400u;
    asm("" : "+s"(mask_lo));
    asm("" : "+s"(mask_hi));
    asm("" : "+v"(magic));

    struct BRaw {
        uint4v w[RT];
        uint32_t h[RT];
    };
    struct Nibbles {
        uint32_t d[RT][4], e[RT][4];  // packed words, and shifted by 8
        float s[RT][2], c[RT][2];     // scale and offset for low and high nibbles
    };
    uint4v a[2][TT];
    uint32_t bo[2][RT][4];
    BRaw braw;
    Nibbles nba, nbb;
    auto read_a = [&](uint32_t addr, uint4v (&v)[TT]) {
        asm volatile("ds_read_b128 %0, %1" : "=v"(v[0]) : "v"(addr));
        if (TT > 1) asm volatile("ds_read_b128 %0, %1 offset:4096" : "=v"(v[TT > 1 ? 1 : 0]) : "v"(addr));
        if (TT == 4) {
            asm volatile("ds_read_b128 %0, %1 offset:8192" : "=v"(v[TT - 2]) : "v"(addr));
            asm volatile("ds_read_b128 %0, %1 offset:12288" : "=v"(v[TT - 1]) : "v"(addr));
        }
    };
    auto read_b = [&](uint32_t waddr, uint32_t saddr) {
        asm volatile("ds_read_b128 %0, %1" : "=v"(braw.w[0]) : "v"(waddr));
        if (RT == 2) asm volatile("ds_read_b128 %0, %1 offset:2048" : "=v"(braw.w[RT - 1]) : "v"(waddr));
        asm volatile("ds_read_b32 %0, %1" : "=v"(braw.h[0]) : "v"(saddr));
        if (RT == 2) {
            if (TAIL && kNear)
                asm volatile("ds_read_b32 %0, %1 offset:512" : "=v"(braw.h[RT - 1]) : "v"(saddr));
            else
                asm volatile("ds_read_b32 %0, %1 offset:256" : "=v"(braw.h[RT - 1]) : "v"(saddr));
        }
    };
    // (every register that is on its way is named by the wait: nothing of it moves before)
    auto arrived_a = [&](uint4v (&v)[TT]) {
        if constexpr (TT == 4)
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]));
        else if constexpr (TT == 2)
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(v[1]));
        else
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]));
    };
    auto arrived_b = [&](uint4v (&v)[TT]) {
        if constexpr (TT == 4 && RT == 2)
            asm volatile("s_waitcnt lgkmcnt(0)"
                         : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(braw.w[0]), "+v"(braw.w[1]),
                           "+v"(braw.h[0]), "+v"(braw.h[1]));
        else if constexpr (TT == 4)
            asm volatile("s_waitcnt lgkmcnt(0)"
                         : "+v"(v[0]), "+v"(v[1]), "+v"(v[2]), "+v"(v[3]), "+v"(braw.w[0]), "+v"(braw.h[0]));
        else if constexpr (TT == 2 && RT == 2)
            asm volatile("s_waitcnt lgkmcnt(0)"
                         : "+v"(v[0]), "+v"(v[1]), "+v"(braw.w[0]), "+v"(braw.w[1]), "+v"(braw.h[0]), "+v"(braw.h[1]));
        else if constexpr (TT == 2)
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(v[1]), "+v"(braw.w[0]), "+v"(braw.h[0]));
        else
            asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(v[0]), "+v"(braw.w[0]), "+v"(braw.h[0]));
    };
    static_assert(RT == 1 || (RT == 2 && TT > 1), "the waits above");
    // row tile rt of the pair whose first group is g
    auto unpack = [&](Nibbles &nb, int rt, int g) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            nb.d[rt][i] = braw.w[rt][i];
            nb.e[rt][i] = braw.w[rt][i] >> 8;
        }
        uint32_t hb = braw.h[rt];
        if (TAIL)
            hb = g + lb < G ? hb : 0u;
        else
            hb >>= 16 * lb;
        const float s = half_bits_to_float((uint16_t)hb);
        nb.s[rt][0] = s;
        nb.s[rt][1] = 0.0625f * s;
        nb.c[rt][0] = -1032.0f * s;
        nb.c[rt][1] = -72.0f * s;
    };
    // four weights (words 2 h, 2 h + 1 of the operand) of row tile rt, MFMA step st
    auto dequant4 = [&](const Nibbles &nb, int st, int rt, int h, uint32_t (&o)[4]) {
        const int hi = st >> 1, i = 2 * (st & 1) + h;
        const uint32_t mask = hi ? mask_hi : mask_lo;
        const halfx2 ev = __builtin_bit_cast(halfx2, (nb.d[rt][i] & mask) | magic);
        const halfx2 od = __builtin_bit_cast(halfx2, (nb.e[rt][i] & mask) | magic);
        const float s = nb.s[rt][hi], c = nb.c[rt][hi];
        o[2 * h] = pack_bf16(fmaf((float)ev.x, s, c), fmaf((float)od.x, s, c));
        o[2 * h + 1] = pack_bf16(fmaf((float)ev.y, s, c), fmaf((float)od.y, s, c));
    };

    // Step st of the pair in registers while the operands of step nst of the pair at LDS
    // offset `nbuf` with the nibbles wn are made.  extra = 1: also reads the next pair's
    // packed weights; 2: also unpacks them.  A quarter of the load list of pair lq.
    auto step = [&](int st, uint32_t nbuf, const Nibbles &wc, int nst, int extra, uint32_t waddr,
                    uint32_t saddr, Nibbles &wnext, int gnext, int lq, bool even, int quarter, int sel,
                    unsigned char *abuf) {
        const int c = st & 1, n = c ^ 1;
        const int ops = even ? kEven : kOdd;
        const int first = ops * quarter / 4, count = ops * (quarter + 1) / 4 - first;
#pragma unroll
        for (int i = 0; i < NM; ++i) {
            const int tt = i / RT, rt = i % RT;
            acc[tt][rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                __builtin_bit_cast(bf16x8, a[c][tt]),
                __builtin_bit_cast(bf16x8, make_uint4(bo[c][rt][0], bo[c][rt][1], bo[c][rt][2], bo[c][rt][3])),
                acc[tt][rt], 0, 0, 0);
            if (i == 0) read_a(apos[nst] + nbuf, a[n]);
            if (extra == 1 && i == 0) read_b(waddr, saddr);
            if (NM == RT) {
                dequant4(wc, nst, i, 0, bo[n][i]);
                dequant4(wc, nst, i, 1, bo[n][i]);
            } else if (NM == 2 * RT)
                dequant4(wc, nst, i >> 1, i & 1, bo[n][i >> 1]);
            else if (!(i & 1))
                dequant4(wc, nst, i >> 2, (i >> 1) & 1, bo[n][i >> 2]);
            if (extra == 2 && i < RT) unpack(wnext, i, gnext);
#pragma unroll
            for (int m = 0; m < count; ++m)
                if (m * NM / count == i) load_op(lq, even, sel, abuf, first + m);
            __builtin_amdgcn_sched_barrier(0);
        }
        if (extra == 1)
            arrived_b(a[n]);
        else
            arrived_a(a[n]);
    };
#define NVQ_PIN asm volatile("" ::: "memory")
    if (nblk > 0) {
        // weights of blocks 0 and 1, activations of pairs 0 and 1 and a quarter of pair 2's
#pragma unroll
        for (int k = 0; k < kWOps; ++k) issue_w1(0, 0, k);
#pragma unroll
        for (int k = 0; k < kScOps; ++k) issue_s1(0, 0, k);
#pragma unroll
        for (int j = 0; j < NA; ++j) issue_a1(xa, 0, j);
#pragma unroll
        for (int j = 0; j < NA; ++j) issue_a1(xa + kBufA, 1, j);
#pragma unroll
        for (int k = 0; k < kWOps; ++k) issue_w1(1, 1, k);
#pragma unroll
        for (int k = 0; k < kScOps; ++k) issue_s1(1, 1, k);
#pragma unroll
        for (int j = 0; j < NA / 4; ++j) issue_a1(xa + 2 * kBufA, 2, j);
        NVQ_PIN;
        __builtin_amdgcn_s_waitcnt(wide_vmcnt(NA + kWOps + kScOps + NA / 4));
        if (WN > 1) __builtin_amdgcn_s_barrier();
        NVQ_PIN;
        read_b(bwpos, bspos);
        read_a(apos[0], a[0]);
        arrived_b(a[0]);
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) unpack(nba, rt, group_of(0));
#pragma unroll
        for (int i = 0; i < 2 * RT; ++i) dequant4(nba, 0, i >> 1, i & 1, bo[0][i >> 1]);

        // Pair q: the wait before step 3 lets the list of pair q - 1 stay in flight and ends
        // all older loads: the activations of pair q + 1, read next, are in the list of pair
        // q - 2, its weights in that of pair q - 2 or older.
        int cur = 0, prv = 2 * kBufA, wsel = 0;
        for (int b = 0; b < nblk; ++b) {
#define NVQ_PAIR(odd_, nb, nnb)                                                                    \
    do {                                                                                           \
        const int q_ = 2 * b + (odd_);                                                             \
        const int nsel_ = (odd_) ? wsel ^ 1 : wsel; /* weight buffer of the next pair */           \
        const uint32_t waddr_ = (bwpos + nsel_ * kW) ^ ((odd_) ? 0 : 32);                          \
        const uint32_t saddr_ = bspos + nsel_ * kS + ((odd_) ? 0 : !TAIL ? 4 : kNear ? 8 : RT * 256); \
        const int gnext_ = (odd_) ? group_of(b + 1) : group_of(b) + 2;                             \
        const int nxt_ = cur + kBufA == 3 * kBufA ? 0 : cur + kBufA;                                  \
        step(0, cur, nb, 1, 0, 0, 0, nnb, 0, q_ - 1, (odd_), 1, wsel, xa + prv);                   \
        step(1, cur, nb, 2, 1, waddr_, saddr_, nnb, 0, q_ - 1, (odd_), 2, wsel, xa + prv);         \
        step(2, cur, nb, 3, 2, 0, 0, nnb, gnext_, q_ - 1, (odd_), 3, wsel, xa + prv);              \
        __builtin_amdgcn_s_waitcnt(wide_vmcnt((odd_) ? kEven : kOdd));                             \
        if (WN > 1) __builtin_amdgcn_s_barrier();                                                  \
        NVQ_PIN;                                                                                   \
        step(3, nxt_, nnb, 0, 0, 0, 0, nb, 0, q_, !(odd_), 0, wsel, xa + cur);                     \
        NVQ_PIN;                                                                                   \
        prv = cur;                                                                                 \
        cur = nxt_;                                                                                \
    } while (0)
            NVQ_PAIR(0, nba, nbb);
            if (TAIL && group_of(b) + 2 >= G) {  // the last block has one pair only
                if (WN > 1) __builtin_amdgcn_s_barrier();
                break;
            }
            NVQ_PAIR(1, nbb, nba);
#undef NVQ_PAIR
            wsel ^= 1;
        }
    } else if (WN > 1) {
        __builtin_amdgcn_s_barrier();
    }
    if (WN > 1)
        for (int b = 2 * nblk; b < 2 * nblk_max; ++b) __builtin_amdgcn_s_barrier();
#undef NVQ_PIN
    // no load into LDS may outlive the loop
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");

    // Result tile: lane (j, b) holds weight row j; register r token 8 (r / 4) + 4 b + r % 4.
    // The partial tiles of the slices are added through LDS: of the WK waves with the same
    // rows, wave u owns registers u kMine .. and the others hand theirs over, four registers
    // (16 bytes) per lane at a time; the sum is taken in slice order.
    constexpr int kOwners = WK < kRegs / 4 ? WK : kRegs / 4;  // waves that own a part, whole registers of 16 bytes
    constexpr int kMine = kRegs / kOwners;
    constexpr int kOwnRt = kMine >= 16 * RT ? RT : 1;  // row tiles and tokens a wave owns
    constexpr int kOwnTok = kMine * 2 / kOwnRt;
    constexpr int kRed = WN * kRegs * 256 * (WK - 1), kOut = kMine * 128;
    static_assert(kRed + kWaves * kOut <= kLds, "partial tiles and results fit");
    float v[kMine];
    __syncthreads();  // every wave has left the loop
    if (WK > 1) {
        auto part = [&](int owner, int from) {  // where `from` leaves its part for `owner`
            const int slot = from < owner ? from : from - 1;
            return reinterpret_cast<floatx4 *>(lds) + (((wn * kOwners + owner) * (WK - 1) + slot) * (kMine / 4)) * 64 + lane;
        };
#pragma unroll
        for (int u = 0; u < kOwners; ++u) {
            if (u == wk) continue;
            floatx4 *const dst = part(u, wk);
#pragma unroll
            for (int i = 0; i < kMine / 4; ++i) {
                const int k = u * kMine + 4 * i, tt = k / (16 * RT), rt = (k >> 4) % RT, r = k & 15;
                const floatx4 f = {acc[tt][rt][r], acc[tt][rt][r + 1], acc[tt][rt][r + 2], acc[tt][rt][r + 3]};
                dst[i * 64] = f;
            }
        }
        __syncthreads();
        if (kOwners < WK && wk >= kOwners) return;
#pragma unroll
        for (int i = 0; i < kMine; ++i) v[i] = 0.0f;
#pragma unroll
        for (int u = 0; u < WK; ++u) {
            if (u == wk) {
#pragma unroll
                for (int i = 0; i < kMine; ++i) {
                    const int k = u * kMine + i;
                    v[i] += acc[k / (16 * RT)][(k >> 4) % RT][k & 15];
                }
            } else {
                const floatx4 *const src = part(wk, u);
#pragma unroll
                for (int i = 0; i < kMine / 4; ++i) {
                    const floatx4 f = src[i * 64];
                    v[4 * i] += f.x;
                    v[4 * i + 1] += f.y;
                    v[4 * i + 2] += f.z;
                    v[4 * i + 3] += f.w;
                }
            }
        }
    } else {
#pragma unroll
        for (int i = 0; i < kMine; ++i) v[i] = acc[i / (16 * RT)][(i >> 4) % RT][i & 15];
    }
    // first token and row of what this wave owns
    const int k0 = wk * kMine;
    const int mo = m0 + (k0 / (16 * RT)) * 32 + 2 * (k0 & 15);
    const int no = row_tile * (32 * RT * WN) + wn * (32 * RT) + (kOwnRt == RT ? 0 : ((k0 >> 4) % RT) * 32);
    auto token_of = [&](int i) { return (i / (16 * kOwnRt)) * 32 + 8 * ((i & 15) >> 2) + 4 * lb + (i & 3); };
    if (!F32 && gemm_whole_stores(N, ldy, y)) {
        // bf16 results leave as 16 bytes per lane, whole lines where a wave owns 64 rows: through
        // LDS, pieces permuted as in the wide kernel; the wave reads back what it wrote itself
        constexpr int kPieces = kOwnRt * 4;
        unsigned char *const out = lds + kRed + w * kOut;
#pragma unroll
        for (int i = 0; i < kMine; ++i) {
            const int tok = token_of(i), nl = ((i >> 4) % kOwnRt) * 32 + li;
            const int pos = (nl >> 3) ^ ((tok >> 2) & (kPieces - 1));
            *reinterpret_cast<uint16_t *>(out + (tok * kPieces + pos) * 16 + (nl & 7) * 2) = float_to_bf16_bits(v[i]);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int i = 0; i < (kOwnTok * kPieces + 63) / 64; ++i) {
            const int idx = i * 64 + lane;
            if (kOwnTok * kPieces < 64 && idx >= kOwnTok * kPieces) break;
            const int tok = idx / kPieces, pos = idx % kPieces;
            const int c = pos ^ ((tok >> 2) & (kPieces - 1));
            const uint4v q = *reinterpret_cast<const uint4v *>(out + idx * 16);
            const int m = mo + tok, n = no + c * 8;
            if (m < M && n < N)
                *reinterpret_cast<uint4v *>(reinterpret_cast<uint16_t *>(y) + (size_t)m * ldy + n) = q;
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < kMine; ++i) {
        const int m = mo + token_of(i), n = no + ((i >> 4) % kOwnRt) * 32 + li;
        if (m < M && n < N) store_out(y, F32 ? NVQ_F32 : NVQ_BF16, (int64_t)m * ldy + n, v[i]);
    }
}

// The tiles a product can be cut into, and what a launch of them takes (us): kGemmLaunch, and for each
// round of all compute units `fixed` and per pair of groups and slice `pair` plus `busy` times the
// share of the compute units that are at work (they share the L2 caches and the power); `tail`: for
// kernels with TAIL.  Fitted to 480 products of 36 to 4096 tokens, 512 to 28672 rows and K from 960 to
// 14336 (2.5 to 4.6 % rms per kind).
struct GemmCost {
    float fixed, pair, busy;
};
struct GemmTile {
    int tokens, rows, slices;
    GemmCost whole, tail;
    const char *name;  // for NVQ_GEMM_TILE
};
constexpr GemmTile kGemmTiles[] = {
    {256, 256, 1, {9.96f, 0.959f, 0.575f}, {}, "wide"},
    {128, 256, 1, {5.02f, 0.693f, 0.256f}, {4.10f, 0.642f, 0.408f}, "128x256"},
    {128, 128, 2, {4.81f, 0.681f, 0.276f}, {3.14f, 0.679f, 0.414f}, "128x128"},
    {128, 64, 2, {2.98f, 0.450f, 0.145f}, {3.00f, 0.503f, 0.164f}, "128x64"},
    {64, 64, 4, {3.11f, 0.518f, 0.144f}, {3.07f, 0.566f, 0.147f}, "64x64"},
    {64, 32, 4, {2.16f, 0.378f, 0.087f}, {2.17f, 0.375f, 0.083f}, "64x32"},
    {32, 32, 8, {2.21f, 0.475f, 0.115f}, {2.19f, 0.442f, 0.146f}, "32x32"},
};
constexpr double kGemmLaunch = 2.5, kGemmSplitGain = 0.925;
constexpr int kGemmTileKinds = (int)(sizeof(kGemmTiles) / sizeof(kGemmTiles[0]));

// n / d up, for d a power of two
int64_t up_div(int64_t n, int d) { return (n + d - 1) >> __builtin_ctz((unsigned)d); }

int64_t gemm_tiles(const GemmTile &k, int64_t N, int64_t M) { return up_div(N, k.rows) * up_div(M, k.tokens); }

// A round with this share of the compute units at work.
double gemm_round(const GemmTile &k, int64_t G, bool tail, double share) {
    const GemmCost &c = tail ? k.tail : k.whole;
    return c.fixed + (double)up_div((G + 1) / 2, k.slices) * (c.pair + c.busy * share);
}

// (a narrow division where it will do: a call makes up to a few dozen)
int64_t whole_rounds(int64_t tiles, int64_t cus) {
    return tiles <= 0xffffffffll ? (int64_t)((uint32_t)tiles / (uint32_t)cus) : tiles / cus;
}

// Estimated time of a launch: whole rounds of all compute units, then the rest, which has the caches and
// the power to itself.
double gemm_cost(const GemmTile &k, int64_t N, int64_t G, int64_t M, int64_t cus, bool tail) {
    const int64_t n = gemm_tiles(k, N, M), full = whole_rounds(n, cus);
    double us = kGemmLaunch + (double)full * gemm_round(k, G, tail, 1.0);
    if (n > full * cus) us += gemm_round(k, G, tail, (double)(n - full * cus) / (double)cus);
    return us;
}

// The kind of tile with the smallest estimated time.  Over those 480 products the choice costs 0.05 %
// on average and 3.6 % at worst against the fastest kind (0.03 and 6 % over 194 others); counting the rest at the price of a full
// round it cost 3.7 % and up to 54 %.
int gemm_choose(int64_t N, int64_t G, int64_t M, int64_t cus, bool can_wide, bool tail, double *us) {
    int best = -1;
    for (int i = can_wide ? 0 : 1; i < kGemmTileKinds; ++i) {
        const double t = gemm_cost(kGemmTiles[i], N, G, M, cus, tail);
        if (best < 0 || t < *us) {
            best = i;
            *us = t;
        }
    }
    return best;
}

// A product as one launch of tiles, or as two: the whole rounds of one kind, and the rest of the rows or
// of the tokens in the kind that is best for what is left.
struct GemmPlan {
    int kind;
    int64_t rows, tokens;  // of the first launch
    int rest;              // kind of the second; < 0: none
};

// Large tiles are the cheaper ones per product, but their last round takes a whole round's time however
// few compute units it keeps busy: smaller tiles fill the chip with what is left.  Two launches where
// they are estimated 8 % faster: of 138 such products (100 to 4096 tokens) 12 % faster on average, the
// worst 5 % slower (333 x 6144 x 14336: 86.2 -> 90.9 us; 6000 x 3072 x 3072: 148 -> 112, 3072 x 6144 x
// 4096: 188 -> 151, 1300 x 3072 x 4096: 57 -> 44, 4096 x 6144 x 4096: 199 -> 188).  From an
// estimate of 2 % on: 6 % on average, but 28 of 271 lost 3 to 10 %.  Cuts elsewhere than at the end
// of the whole rounds, all of them tried with the estimate, gain 0.2 % more.
GemmPlan gemm_plan(int64_t N, int64_t G, int64_t M, int64_t cus, bool can_wide, bool tail) {
    double one = 0.0;
    GemmPlan best = {gemm_choose(N, G, M, cus, can_wide, tail, &one), N, M, -1};
    double best_us = kGemmSplitGain * one;
    for (int i = can_wide ? 0 : 1; i < kGemmTileKinds; ++i) {
        const GemmTile &k = kGemmTiles[i];
        const int64_t full = whole_rounds(gemm_tiles(k, N, M), cus);
        // (what is left takes at least another launch)
        if (full == 0 || 2 * kGemmLaunch + (double)full * gemm_round(k, G, tail, 1.0) >= best_us) continue;
        for (int by_rows = 0; by_rows < 2; ++by_rows) {
            const int64_t across = by_rows ? up_div(M, k.tokens) : up_div(N, k.rows);
            const int64_t first = full * cus / across * (by_rows ? k.rows : k.tokens);
            if (first == 0 || first >= (by_rows ? N : M)) continue;
            const int64_t n1 = by_rows ? first : N, m1 = by_rows ? M : first;
            double us = 0.0;
            const int rest = gemm_choose(by_rows ? N - n1 : N, G, by_rows ? M : M - m1, cus, can_wide, tail, &us);
            us += gemm_cost(k, n1, G, m1, cus, tail);
            if (us < best_us) {
                best_us = us;
                best = {i, n1, m1, rest};
            }
        }
    }
    return best;
}

// Whether blocks of two pairs do not fit K, or the scales' words their alignment (TAIL).
bool gemm_tail(int64_t G, const unsigned char *scales) { return (G & 3) != 0 || !aligned(scales, 4); }

template <bool F32, int TT, int RT, int WN, int WK, bool TAIL>
void launch_tile(dim3 grid, hipStream_t st, const unsigned char *q, const unsigned char *s, int N, int G,
                 const unsigned char *x, int M, int row_tiles, int token_tiles, void *y, int ldy) {
    hipLaunchKernelGGL((gemm_w4a16_tile_kernel<F32, TT, RT, WN, WK, TAIL>), grid, dim3(WN * WK * 64), 0, st, q, s, N,
                       G, x, M, row_tiles, token_tiles, y, ldy);
}

template <bool F32>
void launch_gemm(int kind, const unsigned char *q, const unsigned char *s, int N, int G,
                 const unsigned char *x, int M, void *y, int ldy, hipStream_t st) {
    const GemmTile &k = kGemmTiles[kind];
    const int64_t tiles = gemm_tiles(k, N, M);
    if (kind == 0) {
        hipLaunchKernelGGL(gemm_w4a16_wide_kernel<F32>, dim3((unsigned)tiles), dim3(kGemmThreads), 0, st, q, s,
                           N, G, x, M, y, ldy);
    } else {
        const int rt = (int)((N + (int64_t)k.rows - 1) / k.rows), tt = (M + k.tokens - 1) / k.tokens;
        const dim3 grid((unsigned)((tiles + 7) / 8 * 8));
        const bool tail = gemm_tail(G, s);
        switch (kind) {
#define NVQ_TILE(TAIL_, TT_, RT_, WN_, WK_) launch_tile<F32, TT_, RT_, WN_, WK_, TAIL_>(grid, st, q, s, N, G, x, M, rt, tt, y, ldy)
#define NVQ_TILES(TT_, RT_, WN_, WK_) \
    if (tail) NVQ_TILE(true, TT_, RT_, WN_, WK_); else NVQ_TILE(false, TT_, RT_, WN_, WK_)
            case 1:
                if (tail) NVQ_TILE(true, 4, 1, 8, 1); else NVQ_TILE(false, 4, 2, 4, 1);
                break;
            case 2:
                if (tail) NVQ_TILE(true, 4, 1, 4, 2); else NVQ_TILE(false, 4, 2, 2, 2);
                break;
            case 3: NVQ_TILES(4, 1, 2, 2); break;
            case 4: NVQ_TILES(2, 2, 1, 4); break;
            case 5: NVQ_TILES(2, 1, 1, 4); break;
            default: NVQ_TILES(1, 1, 1, 8); break;
#undef NVQ_TILES
#undef NVQ_TILE
        }
    }
}

template <bool F32>
int launch_plan(const GemmPlan &p, const unsigned char *q, const unsigned char *s, int N, int G,
                const unsigned char *x, int M, void *y, hipStream_t st) {
    const int n1 = (int)p.rows, m1 = (int)p.tokens;
    launch_gemm<F32>(p.kind, q, s, n1, G, x, m1, y, N, st);
    if (p.rest >= 0) {
        const bool by_rows = n1 < N;
        const size_t n0 = by_rows ? n1 : 0, m0 = by_rows ? 0 : m1;
        launch_gemm<F32>(p.rest, q + n0 * (size_t)(G * 16), s + n0 * (size_t)(G * 2), N - (int)n0, G,
                         x + m0 * (size_t)(G * 64), M - (int)m0,
                         static_cast<unsigned char *>(y) + (m0 * (size_t)N + n0) * (F32 ? 4 : 2), N, st);
    }
    NVQ_HIP_TRY(hipGetLastError());
    return NVQ_OK;
}

bool gemm_sizes(int64_t N, int64_t K, int64_t M) {
    return N > 0 && M > 0 && K > 0 && (K % 32) == 0 && K <= NVQ_MAX_K && N <= (1 << 24) && M <= (1 << 24);
}

// The launches of a product of such sizes.
int gemm_launches(int64_t N, int64_t K, int64_t M, const uint16_t *scales, GemmPlan *out) {
    // The wide tiles take whole blocks of K and move 16 bytes of scales at a time.  The
    // environment variable NVQ_GEMM_TILE (the name of a tile; "narrow" for 128x256) overrides
    // the choice where the kernel can run (the tests reach all of them on small shapes).
    const bool can_wide = (K % 256) == 0 && aligned(scales, 16);
    const bool tail = gemm_tail(K / 32, reinterpret_cast<const unsigned char *>(scales));
    const int64_t cus = device_cu_count();
    GemmPlan plan = gemm_plan(N, K / 32, M, cus, can_wide, tail);
    if (const char *force = getenv("NVQ_GEMM_TILE")) {
        if (strcmp(force, "narrow") == 0) force = "128x256";
        for (int i = can_wide ? 0 : 1; i < kGemmTileKinds; ++i)
            if (strcmp(force, kGemmTiles[i].name) == 0) plan = {i, N, M, -1};
    }
    // a grid holds so many workgroups
    auto fits = [](int kind, int64_t n, int64_t m) { return gemm_tiles(kGemmTiles[kind], n, m) <= (int64_t)0x7ffffff8; };
    if (plan.rest >= 0 && !(fits(plan.kind, plan.rows, plan.tokens) &&
                            fits(plan.rest, plan.rows < N ? N - plan.rows : N, plan.rows < N ? M : M - plan.tokens))) {
        double us;
        plan = {gemm_choose(N, K / 32, M, cus, can_wide, tail, &us), N, M, -1};
    }
    if (!fits(plan.kind, plan.rows, plan.tokens)) return NVQ_ERR_SHAPE;
    *out = plan;
    return NVQ_OK;
}

}  // namespace

}  // namespace nvq

extern "C" int nvq_gemm_w4a16(const uint8_t *qweight, const uint16_t *scales, int64_t N, int64_t K,
                              const uint16_t *x_bf16, int64_t M, void *y, int y_dtype,
                              void *stream) {
    using namespace nvq;
    if (!qweight || !scales || !x_bf16 || !y) return NVQ_ERR_INVALID_ARG;
    if (y_dtype != NVQ_F32 && y_dtype != NVQ_BF16) return NVQ_ERR_INVALID_ARG;
    if (!gemm_sizes(N, K, M)) return NVQ_ERR_SHAPE;
    if (!aligned(qweight, 16) || !aligned(scales, 2) || !aligned(x_bf16, 16) ||
        !aligned(y, y_dtype == NVQ_F32 ? 4 : 2))
        return NVQ_ERR_ALIGN;
    GemmPlan plan;
    const int rc = gemm_launches(N, K, M, scales, &plan);
    if (rc != NVQ_OK) return rc;
    const unsigned char *const sb = reinterpret_cast<const unsigned char *>(scales);
    const unsigned char *const xb = reinterpret_cast<const unsigned char *>(x_bf16);
    if (y_dtype == NVQ_F32)
        return launch_plan<true>(plan, qweight, sb, (int)N, (int)(K / 32), xb, (int)M, y, (hipStream_t)stream);
    return launch_plan<false>(plan, qweight, sb, (int)N, (int)(K / 32), xb, (int)M, y, (hipStream_t)stream);
}

extern "C" int nvq_gemm_describe(const uint16_t *scales, int64_t N, int64_t K, int64_t M, const void *y, int y_dtype,
                                 int32_t *out, int out_words) {
    using namespace nvq;
    if (!out || (y_dtype != NVQ_F32 && y_dtype != NVQ_BF16)) return NVQ_ERR_INVALID_ARG;
    if (!gemm_sizes(N, K, M)) return NVQ_ERR_SHAPE;
    if (!aligned(scales, 2) || !aligned(y, y_dtype == NVQ_F32 ? 4 : 2)) return NVQ_ERR_ALIGN;
    GemmPlan plan;
    const int rc = gemm_launches(N, K, M, scales, &plan);
    if (rc != NVQ_OK) return rc;
    const int launches = plan.rest < 0 ? 1 : 2;
    if (out_words < 1 + 7 * launches) return NVQ_ERR_WORKSPACE;
    *out++ = launches;
    const bool by_rows = plan.rows < N;
    for (int i = 0; i < launches; ++i) {
        const GemmTile &k = kGemmTiles[i == 0 ? plan.kind : plan.rest];
        const int64_t n0 = i > 0 && by_rows ? plan.rows : 0, m0 = i > 0 && !by_rows ? plan.tokens : 0;
        const int64_t n = i == 0 ? plan.rows : N - n0, m = i == 0 ? plan.tokens : M - m0;
        const int size = y_dtype == NVQ_F32 ? 4 : 2;
        const char *const at = static_cast<const char *>(y) + (m0 * N + n0) * size;
        const int64_t words[7] = {k.tokens, k.rows, n0, n, m0, m,
                                  y_dtype == NVQ_BF16 && gemm_whole_stores((int)n, (int)N, at) ? 16 : size};
        for (int64_t w : words) *out++ = (int32_t)w;
    }
    return NVQ_OK;
}

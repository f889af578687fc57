// Products of 2 to 32 tokens with one phase's weight rows, any K that is a whole number
// of groups, activation scales per token or per group: the kernel behind the single calls
// and the per-phase walk.  Paper: the W4A8 / W4A16 kernel descriptions; the arithmetic is
// that of mfma_act.h (one 16x16x32 MFMA per quantisation group, 16 tokens times 16 rows,
// the constant nibble offset removed by a second MFMA).
//
// A workgroup of W waves owns 16 RT consecutive rows; the waves share out K in blocks of
// eight groups (256 inputs: a whole 128-byte line of every row), wave w the blocks w, w +
// W, ..., and the partial tiles are added through LDS, in pairs, at the end.  Until
// then the waves do not meet.  Each copies what it needs of a block (the rows' weights and
// scales, the tokens' 256 inputs) straight from global memory into its own piece of LDS,
// takes it into registers, asks for its next block and only then multiplies; what covers
// the memory's latency are the three or four workgroups that share a compute unit.
//
// What bounds it: neither memory nor arithmetic alone.  28672 x 4096 at 8 tokens takes 18.2
// us (3.6 TB/s; 33 with a workgroup per 16 rows that loaded straight into registers);
// without the loads it takes 12, the vector ALUs busy three quarters of that (18
// instructions per 16 x 16 x 32 product), without either 6.  Two to four blocks in flight
// per wave instead of one, with fewer workgroups per compute unit, were no faster; blocks
// of four groups, whose loads move half lines, 5-15 % slower.
//
// SCB: bytes per scale load.  16: K is a multiple of 256 and the scales are aligned to
// that (one load per row and block); 4 or 2: any other K, scales aligned to 4 bytes and an
// even number of groups, or not; the last block may then end early (its missing groups
// are loaded as the last one again and not multiplied).
#pragma once

#include "gemv_tile.h"
#include "mfma_act.h"

namespace nvq {

namespace {

typedef __attribute__((address_space(3))) void *slice_lds_ptr;

constexpr int slice_vmcnt(int n) { return (n & 15) | ((n >> 4) << 14) | 0x0f70; }

// What a block takes in a wave's ring: TOK tokens (8, 16 or 32), RT 16-row tiles.
template <int PREC, bool PG, int TOK, int RT, int SCB>
struct SliceBlock {
    // groups per block: half as many where the activations would fill the ring
    static constexpr int NG = PREC == NVQ_W4A16 && TOK == 32 ? 4 : 8;
    static_assert(SCB != 16 || NG == 8, "16 bytes are the scales of eight groups");
    static constexpr int kTokenBytes = NG * (PREC == NVQ_W4A8 ? 32 : 64);
    // scales: [16 bytes of a row], or words of 4 bytes, [pair of groups or group][row]
    static constexpr int kScOps = SCB == 16 ? (RT + 3) / 4 : NG == 4 && SCB == 4 && RT == 1 ? 1 : RT * (SCB == 4 ? 1 : 2) * NG / 8;
    static constexpr int kScBytes = SCB == 16 ? RT * 256 : kScOps * 256;
    static constexpr int kAOps = TOK * kTokenBytes / 1024;
    static constexpr int kXsOps = PG ? TOK / 8 : 0;  // 64 lanes x 4 bytes, eight scales per token
    static constexpr int kWOps = RT * NG / 4, kWTile = 256 * NG;
    static constexpr int kW = 0, kSc = kW + RT * kWTile, kA = kSc + kScBytes;
    static constexpr int kXs = kA + TOK * kTokenBytes, kBytes = kXs + kXsOps * 256;
    static constexpr int kOps = kWOps + kScOps + kAOps + kXsOps;

    // Where lane row kb finds the scales of its first token, and its token's place among the
    // activations: what stands for tokens that are not there is read from another's.
    static constexpr int xs_place(int kb) { return 128 * (TOK < 16 ? kb & (TOK / 4 - 1) : kb); }
    static constexpr int token_place(int n) { return (TOK < 16 ? n & (TOK - 1) : n) * kTokenBytes; }
    // The last byte that the reads of a block touch lies inside the piece it belongs to.
    static constexpr int kTiles = (TOK + 15) / 16, kRowBytes = 16 * NG;
    static constexpr int kScWords = SCB == 2 ? NG : NG / 2;  // words with the scales of a row
    static constexpr int largest(int (*place)(int), int n) {
        int m = 0;
        for (int i = 0; i < n; ++i) m = place(i) > m ? place(i) : m;
        return m;
    }
    static_assert(15 * kRowBytes + 16 * (NG - 1) + 16 <= kWTile, "weights");
    static_assert((SCB == 16 ? RT * 256 : kScWords * 16 * RT * 4) <= kScBytes, "scales");
    static_assert(largest(token_place, 16) + (kTiles - 1) * 16 * kTokenBytes + kTokenBytes <= TOK * kTokenBytes,
                  "activations");
    static_assert(!PG || largest(xs_place, 4) + ((kTiles - 1) * 16 + 3) * 32 + 32 <= kXsOps * 256,
                  "activation scales");
};

// Waves per workgroup.
constexpr int slice_waves(int RT) { return RT == 1 ? 8 : 4; }

template <int PREC, bool PG, int TOK, int RT, int SCB, bool DEBUG>
__global__ __launch_bounds__(slice_waves(RT) * 64) void gemv_slice_kernel(
    GemvSegs S, int G, int M, const char *__restrict__ xin, const float *__restrict__ xscale) {
    typedef Act<PREC> A;
    typedef SliceBlock<PREC, PG, TOK, RT, SCB> B;
    constexpr bool TAIL = SCB != 16;
    constexpr int NG = B::NG, W = slice_waves(RT), MT = (TOK + 15) / 16;
    constexpr int kTile = RT * MT * 4;  // result registers per lane
    constexpr int kRing = W * B::kBytes, kRed = W * kTile * 256;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[kRing > kRed ? kRing : kRed];

    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n = lane & 15, kb = lane >> 4;
    const int row0 = (int)blockIdx.x * (16 * RT);
    const int NB = (G + NG - 1) / NG;
    const int nblk = NB > w ? (NB - w + W - 1) / W : 0;
    unsigned char *const slot = lds + w * B::kBytes;

    // Sources, at the start of the row: weights (a row's NG pieces of 16 bytes side by
    // side, permuted against the neighbouring rows'), scales, activations.
    const char *wsrc[B::kWOps], *ssrc[B::kScOps];
    constexpr int kWRows = 64 / NG;  // rows per weight load
    int wc[2];                       // the piece, even and odd j
#pragma unroll
    for (int j = 0; j < 2; ++j) wc[j] = (lane % NG) ^ (((kWRows * j + lane / NG) / (16 / NG)) % NG);
#pragma unroll
    for (int j = 0; j < B::kWOps; ++j)
        wsrc[j] = reinterpret_cast<const char *>(locate_row(S, row0 + kWRows * j + lane / NG, G).qw) +
                  (TAIL ? 0 : 16 * wc[j & 1]);
    constexpr int kRows = 16 * RT;
    int sg[B::kScOps];  // first group of the lane's word
#pragma unroll
    for (int k = 0; k < B::kScOps; ++k) {
        const int word = k * 64 + lane;
        sg[k] = SCB == 16 ? 0 : (word / kRows * (SCB / 2)) % NG;
        ssrc[k] = reinterpret_cast<const char *>(locate_row(S, row0 + word % kRows, G).sc);
    }
    // activations: 2 or 4 tokens per instruction, pieces permuted against each other
    constexpr int kPieces = B::kTokenBytes / 16;  // 16 or 32
    uint32_t aoff[B::kAOps];
    int apiece[B::kAOps];
#pragma unroll
    for (int j = 0; j < B::kAOps; ++j) {
        const int m = j * (64 / kPieces) + lane / kPieces;
        const int p = (lane % kPieces) ^ (m & 15);
        aoff[j] = (uint32_t)(m < M ? m : M - 1) * (uint32_t)(G * 32 * A::kBytes) + (TAIL ? 0u : 16u * (uint32_t)p);
        apiece[j] = p;
    }
    uint32_t xsoff[PG ? B::kXsOps : 1];  // word l: scale l % 8 of token l / 8
    if (PG) {
#pragma unroll
        for (int j = 0; j < B::kXsOps; ++j) {
            const int m = j * 8 + (lane >> 3);
            xsoff[j] = (uint32_t)(m < M ? m : M - 1) * (uint32_t)G;
        }
    }
    auto clamp_g = [&](int g) { return g < G ? g : G - 1; };
    auto issue = [&](int b) {
        const int g0 = NG * (w + W * b);
#pragma unroll
        for (int j = 0; j < B::kWOps; ++j) {
            const char *p = wsrc[j] + (TAIL ? (size_t)clamp_g(g0 + wc[j & 1]) * 16 : (size_t)g0 * 16);
            __builtin_amdgcn_global_load_lds((const void *)p, (slice_lds_ptr)(slot + B::kW + j * 1024), 16, 0, 0);
        }
#pragma unroll
        for (int k = 0; k < B::kScOps; ++k) {
            if (SCB == 16) {
                const char *p = ssrc[k] + (size_t)g0 * 2;
                if (RT == 4 || lane < kRows)
                    __builtin_amdgcn_global_load_lds((const void *)p, (slice_lds_ptr)(slot + B::kSc), 16, 0, 0);
            } else if (SCB == 4) {  // (a pair of groups is inside the row or outside it)
                const int g = g0 + sg[k];
                const char *p = ssrc[k] + (size_t)(g < G ? g : G - 2) * 2;
                __builtin_amdgcn_global_load_lds((const void *)p, (slice_lds_ptr)(slot + B::kSc + k * 256), 4, 0, 0);
            } else {
                const char *p = ssrc[k] + (size_t)clamp_g(g0 + sg[k]) * 2;
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
                const float *p = xscale + (xsoff[j] + (uint32_t)clamp_g(g0 + (lane & 7)));
                __builtin_amdgcn_global_load_lds((const void *)p, (slice_lds_ptr)(slot + B::kXs + j * 256), 4, 0, 0);
            }
        }
    };

    float f[RT][MT][4];
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) f[r][mt][jj] = 0.0f;

    // The lane's places in its piece of LDS, for group i of the block.  Weights: dword kb of
    // piece i of row n (what the MFMA's weight operand of group i wants), 64 different banks;
    // activations: for W4A16 half a piece twice (inputs 4 kb .. + 3 and 16 + 4 kb .. + 3 of
    // the group), for W4A8 a dword twice.
    const uint32_t at = (uint32_t)(uintptr_t)slot;
    const int mn = TOK < 16 ? n & (TOK - 1) : n;
    uint32_t wpos[NG], apos[NG][2];
#pragma unroll
    for (int i = 0; i < NG; ++i) {
        wpos[i] = at + n * (16 * NG) + 16 * (i ^ ((n / (16 / NG)) % NG)) + 4 * kb;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            if (PREC == NVQ_W4A8)
                apos[i][h] = at + B::token_place(n) + 16 * ((2 * i + h) ^ mn) + 4 * kb;
            else
                apos[i][h] = at + B::token_place(n) + 16 * ((4 * i + 2 * h + (kb >> 1)) ^ mn) + 8 * (kb & 1);
        }
    }
    const uint32_t spos = at + (SCB == 16 ? 16 : 4) * n;
    const uint32_t xspos = at + B::xs_place(kb);  // token 4 kb, 32 bytes per token

#define NVQ_RD32(dst_, addr_, off_) asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(dst_) : "v"(addr_), "n"(off_))
#define NVQ_RD64(dst_, addr_, off_) asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(dst_) : "v"(addr_), "n"(off_))
#define NVQ_RD128(dst_, addr_, off_) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst_) : "v"(addr_), "n"(off_))
    if (nblk > 0) issue(0);
    for (int b = 0; b < nblk; ++b) {
        __builtin_amdgcn_s_waitcnt(slice_vmcnt(0));
        asm volatile("" ::: "memory");

        constexpr int kSc = B::kScWords;
        uint32_t q[RT][NG], sc[RT][kSc];
        uint2v a2[PREC == NVQ_W4A8 ? 1 : MT][NG][2];
        uint32_t a1[PREC == NVQ_W4A8 ? MT : 1][NG][2];
        float4v xs4[PG ? MT : 1][4][2];
#pragma unroll
        for (int i = 0; i < NG; ++i)
#pragma unroll
            for (int r = 0; r < RT; ++r) NVQ_RD32(q[r][i], wpos[i], B::kW + r * B::kWTile);
#pragma unroll
        for (int r = 0; r < RT; ++r)
#pragma unroll
            for (int k = 0; k < kSc; ++k)
                NVQ_RD32(sc[r][k], spos, B::kSc + (SCB == 16 ? r * 256 + k * 4 : (k * kRows + 16 * r) * 4));
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < NG; ++i)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    if (PREC == NVQ_W4A8)
                        NVQ_RD32(a1[mt][i][h], apos[i][h], B::kA + mt * 16 * B::kTokenBytes);
                    else
                        NVQ_RD64(a2[mt][i][h], apos[i][h], B::kA + mt * 16 * B::kTokenBytes);
                }
        if (PG) {
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        NVQ_RD128(xs4[mt][jj][h], xspos, B::kXs + (mt * 16 + jj) * 32 + h * 16);
        }
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
        for (int r = 0; r < RT; ++r) {
#pragma unroll
            for (int i = 0; i < NG; ++i) asm volatile("" : "+v"(q[r][i]));
#pragma unroll
            for (int k = 0; k < kSc; ++k) asm volatile("" : "+v"(sc[r][k]));
        }
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int i = 0; i < NG; ++i) {
                if (PREC == NVQ_W4A8)
                    asm volatile("" : "+v"(a1[mt][i][0]), "+v"(a1[mt][i][1]));
                else
                    asm volatile("" : "+v"(a2[mt][i][0]), "+v"(a2[mt][i][1]));
                if (PG) asm volatile("" : "+v"(xs4[mt][i & 3][i >> 2]));
            }
        if (b + 1 < nblk) issue(b + 1);

        // With a scale per group the products are rounded and the sums have no low zero bits to
        // lose: half a block is summed by itself first, so that fewer terms meet the large sum
        // (relative error 0.9e-7 instead of 1.5e-7 at K = 14336).
        float fb[PG ? RT : 1][PG ? MT : 1][4];
        if (PG) {
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) fb[PG ? r : 0][PG ? mt : 0][jj] = 0.0f;
        }
        const int g0 = NG * (w + W * b);
#pragma unroll
        for (int i = 0; i < NG; ++i) {
            if (TAIL && g0 + i >= G) break;  // the last block may end early
            if (PG && (i & 3) == 0 && i > 0) {
#pragma unroll
                for (int r = 0; r < RT; ++r)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                        for (int jj = 0; jj < 4; ++jj) {
                            f[r][mt][jj] += fb[PG ? r : 0][PG ? mt : 0][jj];
                            fb[PG ? r : 0][PG ? mt : 0][jj] = 0.0f;
                        }
            }
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                typename A::operand act;
                if constexpr (PREC == NVQ_W4A8) {
                    act = (long)((uint64_t)a1[mt][i][0] | ((uint64_t)a1[mt][i][1] << 32));
                } else {
                    const uint4v v = {a2[mt][i][0].x, a2[mt][i][0].y, a2[mt][i][1].x, a2[mt][i][1].y};
                    act = __builtin_bit_cast(bf16x8, v);
                }
                const typename A::offset_t off = A::offset(act);
#pragma unroll
                for (int r = 0; r < RT; ++r) {
                    const uint32_t sb = SCB == 2 ? sc[r][i] : sc[r][i >> 1] >> (16 * (i & 1));
                    const float sw = half_bits_to_float((uint16_t)sb);
                    int4v raw;
                    float4v p = A::product(act, A::weights(q[r][i]), off, raw);
                    if (PG) {
                        p.x *= xs4[mt][0][i >> 2][i & 3];
                        p.y *= xs4[mt][1][i >> 2][i & 3];
                        p.z *= xs4[mt][2][i >> 2][i & 3];
                        p.w *= xs4[mt][3][i >> 2][i & 3];
                    }
                    float (&sum)[4] = PG ? fb[PG ? r : 0][PG ? mt : 0] : f[r][mt];
                    sum[0] = fmaf(sw, p.x, sum[0]);
                    sum[1] = fmaf(sw, p.y, sum[1]);
                    sum[2] = fmaf(sw, p.z, sum[2]);
                    sum[3] = fmaf(sw, p.w, sum[3]);
                    if (DEBUG && PREC == NVQ_W4A8) {
                        const RowRef o = locate_row(S, row0 + 16 * r + n, G);
                        if (o.valid && o.dbg) {
                            const int acc[4] = {raw.x, raw.y, raw.z, raw.w};
#pragma unroll
                            for (int jj = 0; jj < 4; ++jj) {
                                const int m = mt * 16 + kb * 4 + jj;
                                if (m < M) o.dbg[((int64_t)m * o.N + o.n) * G + g0 + i] = acc[jj];
                            }
                        }
                    }
                }
            }
        }
        if (PG) {
#pragma unroll
            for (int r = 0; r < RT; ++r)
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) f[r][mt][jj] += fb[PG ? r : 0][PG ? mt : 0][jj];
        }
    }
#undef NVQ_RD32
#undef NVQ_RD64
#undef NVQ_RD128

    // Sum the slices.
    float xs[MT][4];
#pragma unroll
    for (int mt = 0; mt < MT; ++mt)
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
            const int m = mt * 16 + kb * 4 + jj;
            xs[mt][jj] = (PREC == NVQ_W4A8 && !PG && m < M) ? as_global<float>(xscale)[m] : 1.0f;
        }
    float (*const red)[kTile][64] = reinterpret_cast<float (*)[kTile][64]>(lds);
    __syncthreads();
#pragma unroll
    for (int r = 0; r < RT; ++r)
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) red[w][(r * MT + mt) * 4 + jj][lane] = f[r][mt][jj] * xs[mt][jj];
    __syncthreads();
#pragma unroll
    for (int pass = 0; pass < (kTile + W - 1) / W; ++pass) {
        const int reg = pass * W + w;
        if (reg < kTile) {
            float part[W];  // added in pairs
#pragma unroll
            for (int k = 0; k < W; ++k) part[k] = red[k][reg][lane];
#pragma unroll
            for (int step = 1; step < W; step *= 2)
#pragma unroll
                for (int k = 0; k < W; k += 2 * step) part[k] += part[k + step];
            const float sum = part[0];
            const int r = reg / (MT * 4), mt = (reg >> 2) % MT, jj = reg & 3;
            const int m = mt * 16 + kb * 4 + jj;
            const RowRef o = locate_row(S, row0 + 16 * r + n, G);
            if (o.valid && m < M) store_global(o.y, o.y_dtype, (int64_t)m * o.N + o.n, sum);
        }
    }
}

template <int PREC, bool PG, int TOK, int RT, int SCB, bool DEBUG = false>
int slice_go(const GemvSegs &S, int G, int M, const void *x, const float *xscale, hipStream_t st) {
    const int units = (S.total_rows + 16 * RT - 1) / (16 * RT);
    hipLaunchKernelGGL((gemv_slice_kernel<PREC, PG, TOK, RT, SCB, DEBUG>), dim3(units),
                       dim3(slice_waves(RT) * 64), 0, st, S, G, M, reinterpret_cast<const char *>(x), xscale);
    NVQ_HIP_TRY(hipGetLastError());
    return NVQ_OK;
}

// Row tiles per workgroup.  Sixteen rows and eight waves where there are few rows (8 tokens,
// 4096 x 14336: 10.7 us against 16.9 with 32 rows; 6144 x 4096: 6.6 against 7.6), 32 where
// those make about two workgroups per compute unit and the tokens' inputs, which every
// workgroup reads, count (28672 x 4096: 18.2 against 21.7 us, at 16 tokens 21.8 against
// 32.0; 16384 x 3072, 4 tokens: 8.8 against 9.3).
inline int slice_row_tiles(int rows) { return rows >= 48 * device_cu_count() ? 2 : 1; }

// The scale loads a phase allows (see SCB).
inline int slice_scale_bytes(const GemvSegs &S, int G) {
    int b = (G & 7) == 0 ? 16 : (G & 1) == 0 ? 4 : 2;
    for (int i = 0; i < S.nseg; ++i) {
        if (b == 16 && !aligned(S.sc[i], 16)) b = 4;
        if (b == 4 && !aligned(S.sc[i], 4)) b = 2;
    }
    return b;
}

}  // namespace

}  // namespace nvq

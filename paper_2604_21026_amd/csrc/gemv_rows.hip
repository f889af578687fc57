// Small batches of 2 to 32 tokens through many independent phases as one persistent
// grid (plans whose K are all multiples of 512).  Paper: the W4A8 / W4A16 kernel
// descriptions; the arithmetic is that of mfma_act.h.
//
// With two token tiles 32 weight rows need 3.6 times their own bytes of bf16 activations, and a
// kernel whose waves each fetch their own (the ring kernel) stands at 3 TB/s of weights.  So a workgroup takes 128 rows at a
// time: four waves, each with 32 rows of its own (two 16-row tiles, a unit of the batch) and all of K, share the activations
// through LDS, and no sums cross the waves.  K advances by 256 inputs (a whole 128-byte
// line of a row); per step a wave asks for its quarter of the next step's activations (two
// buffers) and, once the current step's weights and scales are in registers, for its next
// weights, all straight from global memory into LDS; one barrier per step says that the
// activations have arrived and that the other buffer is free.  Three workgroups share a
// compute unit, four where one token tile does (36 KiB of LDS): up to 16 tokens the rings wait for
// their sums across waves and for the operand images made beforehand: four blocks of 8B at 2, 8 and 16 tokens
// 134, 133 and 142 us there, 117, 120 and 124 here.
//
// The batch is cut into parts, one per XCD (the compute units of an XCD advance through
// the phases together, so that the activations they all read stay in their L2), of equal bytes or, where all
// groups are resident together, of as many groups as an XCD holds workgroups; the
// workgroups of a part take its groups of four units, the phases with the largest K first, first come
// first served from a counter, which the quantisation launch in front has cleared.
//
// What bounds it: 8B layers at 32 tokens take 1,021 us (4.1 TB/s), 20 of them the quantisation.
// Without the loads 700, without the products 960: memory, whose queue runs dry while a workgroup waits for
// a step, crosses the barrier and copies its weights.  What brought it there from 1,133: the phases in the order of
// their K (see order_phases; 60 us), two steps' scales per load (16 bytes of a row per load were a
// request each, 20), the matrix core and the vector instructions interleaved unit by unit with
// addresses that need no arithmetic per group (from 92 vector instructions per KiB of weights to 89), a
// higher priority for the waves that ask for operands (10).  Not faster: two steps of weights in flight with
// four barriers per step (the activations in quarters, for the room: 1,140), eight waves per workgroup, weights
// loaded into registers (they spill), plain loads of the weights (2.5 %).
#include <type_traits>

#include "gemv_tile.h"
#include "mfma_act.h"

namespace nvq {

namespace {

typedef __attribute__((address_space(3))) void *rows_lds_ptr;
// tables that do not change during the kernel, on scalar loads
typedef const __attribute__((address_space(4))) GroupPhase CGroup;
typedef const __attribute__((address_space(4))) uint32_t CWord;

constexpr int kRowsWaves = 4;      // waves per workgroup = units per group
constexpr int rows_per_cu(int mt) { return mt == 2 ? 3 : 4; }  // workgroups, for mt token tiles
constexpr int kRowsW = 2 * 2048;   // a wave's weights of a step: 32 rows x 128 bytes
constexpr int kRowsSc = 1024;      // and the scales of two, 32 bytes per row

// A part of the batch: the units begin .. end - 1, in groups of up to four of one phase, phase by phase in
// the order given or as they stand in the batch.  (Groups across phases made a workgroup of four small
// phases keep all of K four times: 32 phases of up to 8192 rows and 14 x 512 inputs 118 us.)
struct RowsPart {
    CWord *order;  // its phases, or null: first, first + 1, ...
    int first, phases;
    int begin, end;
};
// A bundle: up to four consecutive units of one phase.
struct RowsBundle {
    int p;            // phase
    int unit, count;  // first unit (of the phase) and how many; none: the part has no such group
    int at, base;     // the phase's place in the order, groups of the part before it
};

// Group t of the part, not before `from`'s phase.
__device__ __forceinline__ RowsBundle rows_bundle(CGroup *tab, const RowsPart &P, const RowsBundle &from, int t) {
    RowsBundle b = from;
    b.count = 0;
    for (; b.at < P.phases; ++b.at) {
        b.p = P.order ? (int)P.order[b.at] : P.first + b.at;
        const int lo = tab[b.p].unit_begin, hi = lo + tab[b.p].unit_count;
        const int first = lo < P.begin ? P.begin : lo, units = (hi < P.end ? hi : P.end) - first;
        const int groups = (units + kRowsWaves - 1) / kRowsWaves;  // (none, if units < 0)
        if (t < b.base + groups) {
            const int u = (t - b.base) * kRowsWaves;
            b.unit = first - lo + u;
            b.count = units - u < kRowsWaves ? units - u : kRowsWaves;
            break;
        }
        b.base += groups > 0 ? groups : 0;
    }
    return b;
}

// Where a wave finds its operands of a bundle.
struct RowsSource {
    const char *w, *s;  // the wave's first row: weights, scales
    const char *a;      // the phase's activations, [M][K] codes or bf16
    int p, row0;        // phase, the wave's first row there
    int G, precision;
    bool active;        // the wave has a unit of the bundle
    bool whole;         // its 32 rows follow each other in memory (one matrix, none missing)
};

// MT: tiles of 16 tokens
template <int MT>
__global__ __launch_bounds__(kRowsWaves * 64) __attribute__((amdgpu_waves_per_eu(rows_per_cu(MT)))) void
gemv_rows_kernel(const GroupPhase *__restrict__ tab_, const uint32_t *__restrict__ part_tab_, int nparts,
                 const uint32_t *__restrict__ order_, int M, uint32_t *__restrict__ tickets) {
    constexpr int R = 2;  // row tiles of a wave
    constexpr int kRowsBlock = 2048 * MT;   // a block of activations: 128 bytes of every token
    constexpr int kRowsA = 4 * kRowsBlock;  // a buffer: a step's 256 inputs as bf16 (codes fill half of it)
    constexpr int kWaveLds = kRowsW + kRowsSc;
    __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * kRowsA + kRowsWaves * kWaveLds];
    __shared__ int ticket_word;
    CGroup *tab = (CGroup *)tab_;
    CWord *part_tab = (CWord *)part_tab_;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    unsigned char *const slot = lds + 2 * kRowsA + w * kWaveLds;

    const int part = (int)blockIdx.x % nparts;
    const int part_wgs = ((int)gridDim.x - 1 - part) / nparts + 1;
    RowsPart P;
    P.begin = (int)part_tab[part];
    P.end = (int)part_tab[part + 1];
    P.first = (int)part_tab[nparts + 1 + part];
    P.phases = (int)part_tab[nparts + 1 + part + 1] + 1 - P.first;
    P.order = nullptr;
    if (order_) {
        CWord *const order = (CWord *)order_;
        P.order = order + nparts + 1 + order[part];
        P.phases = (int)(order[part + 1] - order[part]);
    }
    int t = (int)blockIdx.x / nparts;  // the group
    auto source = [&](const RowsBundle &b) {
        RowsSource s;
        CGroup &P = tab[b.p];
        s.G = P.G;
        s.precision = P.precision;
        s.a = P.precision == NVQ_W4A8 ? reinterpret_cast<const char *>(P.xq)
                                      : reinterpret_cast<const char *>(P.x_bf16);
        s.active = w < b.count;
        s.p = b.p;
        s.row0 = (b.unit + (s.active ? w : 0)) * 32;
        const RowRef o = locate_row(P.segs, s.row0, s.G), e = locate_row(P.segs, s.row0 + 31, s.G);
        s.w = reinterpret_cast<const char *>(o.qw);
        s.s = reinterpret_cast<const char *>(o.sc);
        s.whole = e.valid && e.n == o.n + 31 && e.y == o.y;
        return s;
    };

    // The lane's number, opaque: what follows from it is made anew where it is used.  Kept, it would cost
    // registers across the whole loop, and a spill's reload waits for every load in flight.
    auto fresh_lane = [&]() {
        uint32_t l = threadIdx.x & 63;
        asm volatile("" : "+v"(l));
        return l;
    };

    // The wave's share of step c's activations: a block is 128 bytes of every token, four tokens' 64
    // bytes per load; W4A16 has four blocks in a step, W4A8 two.
    auto issue_a = [&](const RowsSource &s, int c, int buf) {
        const bool codes = s.precision == NVQ_W4A8;
        const int lane = (int)fresh_lane();
        const uint32_t row = (uint32_t)(s.G * (codes ? 32 : 64));
        const int block = codes ? w >> 1 : w;
        const char *src = s.a + (size_t)c * (codes ? 256 : 512) + block * 128;
        unsigned char *const dst = lds + buf * kRowsA + block * kRowsBlock;
        const uint32_t piece = 16u * (uint32_t)((lane & 3) ^ ((lane >> 4) & 3));
#pragma unroll
        for (int j = 0; j < 2 * MT; ++j) {
            if (codes && (MT == 2 ? j >> 1 : j) != (w & 1)) continue;
            const int m = 16 * (j >> 1) + (lane >> 2);
            __builtin_amdgcn_global_load_lds(
                (const void *)(src + ((uint32_t)(m < M ? m : M - 1) * row + piece + 64u * (uint32_t)(j & 1))),
                (rows_lds_ptr)(dst + j * 1024), 16, 0, 0);
        }
    };
    // Weights, load j: rows 8 j .. + 7 of the wave's 32, lane l piece (l % 8) ^ (row / 2 % 8)
    // of row l / 8.
    auto issue_w = [&](const RowsSource &s, int c) {
        if (!s.active) return;
        const int wrow = (int)fresh_lane() >> 3, piece = (int)fresh_lane() & 7;
        const uint32_t row_bytes = (uint32_t)s.G * 16;  // a multiple of 256
        if (s.whole) {
            const uint32_t lo = (uint32_t)wrow * row_bytes + 16u * (uint32_t)(piece ^ (wrow >> 1));
#pragma unroll
            for (int j = 0; j < 4; ++j)
                __builtin_amdgcn_global_load_lds(
                    (const void *)(s.w + ((size_t)c * 128 + (size_t)(8 * j) * row_bytes) + ((j & 1) ? lo ^ 64u : lo)),
                    (rows_lds_ptr)(slot + j * 1024), 16, 0, 2);
        } else {
            CGroup &P = tab[s.p];
            for (int j = 0; j < 4; ++j) {
                const char *row = reinterpret_cast<const char *>(locate_row(P.segs, s.row0 + 8 * j + wrow, s.G).qw);
                const int pc = piece ^ ((4 * j + (wrow >> 1)) & 7);
                __builtin_amdgcn_global_load_lds((const void *)(row + (size_t)c * 128 + 16 * pc),
                                                 (rows_lds_ptr)(slot + j * 1024), 16, 0, 2);
            }
        }
    };
    // Scales of steps c and c + 1 (c even): 32 bytes of every row, in two pieces.
    auto issue_s = [&](const RowsSource &s, int c) {
        if (!s.active) return;
        const uint32_t l = fresh_lane(), row = l >> 1, piece = l & 1;
        const char *a;
        if (s.whole)
            a = s.s + ((size_t)c * 16 + (row * (uint32_t)s.G * 2u + 16u * piece));
        else
            a = reinterpret_cast<const char *>(locate_row(tab[s.p].segs, s.row0 + (int)row, s.G).sc) + (size_t)c * 16 +
                16 * piece;
        __builtin_amdgcn_global_load_lds((const void *)a, (rows_lds_ptr)(slot + kRowsW), 16, 0, 0);
    };

    // The lane's places.  Weights: dword kb of piece i of row n, piece i at position i ^ (n / 2
    // % 8).  Activations, [tile][half line][token][position], piece p of a half line at position
    // p ^ (n / 4): W4A16 half a piece twice (pieces 4 g + 2 h + kb / 2 of a block), W4A8 a dword
    // twice (pieces 2 g + h).
    const uint32_t at = (uint32_t)(uintptr_t)slot, abase = (uint32_t)(uintptr_t)lds;

    // A result's sum in three levels: the eight groups of a step, eight steps, all of K.  (One
    // chain over all of K had up to twice the error of the four that the ring kernel adds, registers
    // for four would be 64; for 2 % more vector instructions this is as close as those at K = 2048 (rms of
    // W4A8 results against 64 bits 6.4e-8, there 6.3e-8) and closer beyond: K = 14336 8.5e-8, there 1.5e-7.)
    float f[R][MT][4], total[R][MT][4], sums[R][MT][4];
    auto clear = [&](float (&v)[R][MT][4]) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) v[r][mt][jj] = 0.0f;
    };
    auto add = [&](float (&to)[R][MT][4], const float (&v)[R][MT][4]) {
#pragma unroll
        for (int r = 0; r < R; ++r)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) to[r][mt][jj] += v[r][mt][jj];
    };

#define NVQ_RD2(dst_, addr_) asm volatile("ds_read2st64_b32 %0, %1 offset0:0 offset1:8" : "=v"(dst_) : "v"(addr_))
#define NVQ_RD128(dst_, addr_, off_) asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(dst_) : "v"(addr_), "n"(off_))
#define NVQ_RD32(dst_, addr_, off_) asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(dst_) : "v"(addr_), "n"(off_))
#define NVQ_RD64(dst_, addr_, off_) asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(dst_) : "v"(addr_), "n"(off_))
    RowsBundle cur = rows_bundle(tab, P, RowsBundle{}, t);
    if (cur.count == 0) return;
    RowsSource src = source(cur);
    int buf = 0;
    issue_a(src, 0, 0);
    issue_s(src, 0);
    issue_w(src, 0);
    while (true) {
        const int steps = src.G >> 3;
        const bool active = src.active;
        bool more = false;
        RowsBundle nxt = cur;
        int drawn = 0;
        uint2v q[8];   // the two row tiles' weights of a step
        uint4v sc[R];  // and their scales
        // The start of step c: its operands have arrived; everyone has left the other buffer.
        auto begin = [&](int c) {
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
            if (c == 1 && w == 0 && lane == 0) ticket_word = drawn;
            __syncthreads();
            if (c == 0 && w == 0 && lane == 0)  // read at the next step's barrier
                drawn = (int)__hip_atomic_fetch_add(&tickets[part], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (c + 1 < steps) {
                issue_a(src, c + 1, buf ^ 1);
            } else {
                t = part_wgs + __builtin_amdgcn_readfirstlane(ticket_word);
                nxt = rows_bundle(tab, P, cur, t);
                more = nxt.count > 0;
                if (more) {
                    src = source(nxt);  // from here on the next bundle's
                    issue_a(src, 0, buf ^ 1);
                }
            }
            const uint32_t l = fresh_lane(), n = l & 15, kb = l >> 4;
            const uint32_t wpos = at + n * 128 + 16 * ((n >> 1) & 7) + 4 * kb, spos = at + kRowsW + 32 * n + 16 * (c & 1);
#pragma unroll
            for (int i = 0; i < 8; ++i) NVQ_RD2(q[i], wpos ^ (16 * i));
#pragma unroll
            for (int r = 0; r < R; ++r) NVQ_RD128(sc[r], spos, r * 512);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(q[i]));
#pragma unroll
            for (int r = 0; r < R; ++r) asm volatile("" : "+v"(sc[r]));
            if (c + 1 < steps || more) {
                const int next = c + 1 < steps ? c + 1 : 0;
                if (c & 1) issue_s(src, next);
                issue_w(src, next);
            }
        };
        auto bundle = [&](auto prec) {
            constexpr int PREC = decltype(prec)::value;
            // groups in a block of activations (whose places are the same but for a constant)
            constexpr int kGroups = PREC == NVQ_W4A8 ? 4 : 2;
            typedef Act<PREC> A;
            constexpr int kMatrix = 0x8, kVector = 0x2;
            uint32_t pos[4];
            uint2v a2[2][PREC == NVQ_W4A8 ? 1 : MT][2];
            uint32_t a1[2][PREC == NVQ_W4A8 ? MT : 1][2];
            typename A::operand wt[2];
            typename A::offset_t off[MT], p[2][MT];
            auto places = [&]() {
                const uint32_t l = fresh_lane(), n = l & 15, kb = l >> 4;
                const uint32_t p0 = abase + buf * kRowsA + n * 64 +
                                    (PREC == NVQ_W4A8 ? 16 * (n >> 2) + 4 * kb : 16 * ((kb >> 1) ^ (n >> 2)) + 8 * (kb & 1));
#pragma unroll
                for (int i = 0; i < 4; ++i) pos[i] = p0 ^ (uint32_t)(PREC == NVQ_W4A8 ? 16 * i : 32 * (i & 1));
            };
            auto read = [&](int i) {  // the activations of group i
                const int g = i % kGroups, block = i / kGroups * kRowsBlock;
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int mt = 0; mt < MT; ++mt) {
                        if (PREC == NVQ_W4A8)
                            NVQ_RD32(a1[i & 1][mt][h], pos[2 * (g & 1) + h], block + mt * 2048 + (g >> 1) * 1024);
                        else
                            NVQ_RD64(a2[i & 1][mt][h], pos[h], block + mt * 2048 + g * 1024);
                    }
            };
            auto arrived = [&](int i) {
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    if (PREC == NVQ_W4A8)
                        asm volatile("" : "+v"(a1[i & 1][mt][0]), "+v"(a1[i & 1][mt][1]));
                    else
                        asm volatile("" : "+v"(a2[i & 1][mt][0]), "+v"(a2[i & 1][mt][1]));
                }
            };
            auto activation = [&](int i, int mt) {
                if constexpr (PREC == NVQ_W4A8) {
                    return (long)((uint64_t)a1[i & 1][mt][0] | ((uint64_t)a1[i & 1][mt][1] << 32));
                } else {
                    const uint4v v = {a2[i & 1][mt][0].x, a2[i & 1][mt][0].y, a2[i & 1][mt][1].x, a2[i & 1][mt][1].y};
                    return __builtin_bit_cast(bf16x8, v);
                }
            };
            // W4A8: no correction, the weights enter as 16 (n - 8): the nibble in the high half of
            // its byte, its top bit flipped (the factor leaves with the result)
            auto unpack = [&](int u) {
                const uint32_t v = q[u >> 1][u & 1];
                if constexpr (PREC == NVQ_W4A8) {
                    const uint32_t lo = ((v << 4) & 0xf0f0f0f0u) ^ 0x80808080u, hi = (v & 0xf0f0f0f0u) ^ 0x80808080u;
                    wt[u & 1] = (long)((uint64_t)lo | ((uint64_t)hi << 32));
                } else {
                    wt[u & 1] = A::weights(v);
                }
            };
            auto multiply = [&](int u) {
                const int i = u >> 1;
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    if (PREC == NVQ_W4A8)
                        off[mt] = typename A::offset_t{0, 0, 0, 0};
                    else if ((u & 1) == 0)
                        off[mt] = A::offset(activation(i, mt));
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) p[u & 1][mt] = A::multiply(activation(i, mt), wt[u & 1], off[mt]);
            };
            auto scale_add = [&](int u) {
                const int i = u >> 1, r = u & 1;
                const float sw = half_bits_to_float((uint16_t)(sc[r][i >> 1] >> (16 * (i & 1))));
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    const float4v v = A::value(p[u & 1][mt]);
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj)
                        sums[r][mt][jj] = i > 0 ? fmaf(sw, v[jj], sums[r][mt][jj]) : sw * v[jj];
                }
            };
            // Unit u of a step is row tile u % 2 of group u / 2.  While the matrix core works on it, the one before
            // is scaled and added and the next one's weights are unpacked, a few instructions behind
            // every product: the wave waits neither for a product nor for the matrix core.
            auto units = [&]() {
#pragma unroll
                for (int u = 0; u < 16; ++u) {
                    const int i = u >> 1;
                    if ((u & 1) == 0) {
                        __builtin_amdgcn_sched_barrier(0);
                        arrived(i);
                        if (i < 7) read(i + 1);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    multiply(u);
                    if (u > 0) scale_add(u - 1);
                    if (u < 15) unpack(u + 1);
                    if (PREC == NVQ_W4A16 && (u & 1) == 0) {
#pragma unroll
                        for (int k = 0; k < 4; ++k) {
                            __builtin_amdgcn_sched_group_barrier(kMatrix, 1, 0);
                            __builtin_amdgcn_sched_group_barrier(kVector, 4, 0);
                        }
                    } else {
#pragma unroll
                        for (int k = 0; k < 2; ++k) {
                            __builtin_amdgcn_sched_group_barrier(kMatrix, 1, 0);
                            __builtin_amdgcn_sched_group_barrier(kVector, PREC == NVQ_W4A16 ? 7 : 9, 0);
                        }
                    }
                    __builtin_amdgcn_sched_barrier(0);
                }
            };
            for (int c = 0; c < steps; ++c) {
                // (ahead of the waves that multiply: what it asks for takes longest)
                __builtin_amdgcn_s_setprio(2);
                begin(c);
                __builtin_amdgcn_s_setprio(0);
                if (active) {
                    places();
                    read(0);
                    unpack(0);
                    units();
                    scale_add(15);
                    add(f, sums);
                    if ((c & 7) == 7) {
                        add(total, f);
                        clear(f);
                    }
                }
                buf ^= 1;
            }
        };
        clear(f);
        clear(total);
        const bool codes = src.precision == NVQ_W4A8;
        if (codes)
            bundle(std::integral_constant<int, NVQ_W4A8>());
        else
            bundle(std::integral_constant<int, NVQ_W4A16>());
        add(total, f);
        if (active) {
            CGroup &P = tab[cur.p];
            // (opaque: what follows from them would be kept in registers across the whole loop, and
            // others spilled; a spill's reload waits for every load in flight)
            int kb = lane >> 4, n = lane & 15;
            asm volatile("" : "+v"(kb), "+v"(n));
            float xs[MT][4];  // per-token activation scale of the lane's results (W4A8)
            const float unit = codes ? 0.0625f : 1.0f;  // (on the sum: scales may be as small as they like)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const int m = mt * 16 + kb * 4 + jj;
                    xs[mt][jj] = codes && m < M ? as_global<float>(P.xscale)[m] : 1.0f;
                }
            // (all of them before the first store: a load is waited for together with what was issued before it)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) asm volatile("" : "+v"(xs[mt][jj]));
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const RowRef o = locate_row(P.segs, ((cur.unit + w) * R + r) * 16 + n, 0);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) {
                        const int m = mt * 16 + kb * 4 + jj;
                        if (o.valid && m < M)
                            store_global(o.y, o.y_dtype, (int64_t)m * o.N + o.n, (unit * total[r][mt][jj]) * xs[mt][jj]);
                    }
            }
        }
        if (!more) break;
        cur = nxt;
    }
#undef NVQ_RD2
#undef NVQ_RD128
#undef NVQ_RD32
#undef NVQ_RD64
}

}  // namespace

int rows_resident(int M) { return rows_per_cu(M > 16 ? 2 : 1) * device_cu_count(); }

// A workgroup for every group of the part that has the most (the others' spare ones end at once), at most
// what is resident: a group that waits for another's workgroup takes as long again.  Counted from the units alone,
// as if groups went on across phases, the grid was too small for lists of small phases and for uneven parts: 17 tokens,
// 64 phases of 160 x 2048 36 us, so 23, of 544 x 4096 65 and 47.
int rows_grid(int groups, int nparts, int M) {
    const int64_t want = (int64_t)groups * nparts, cap = rows_resident(M);
    return (int)(want < cap ? want : cap);
}

int rows_groups(int units) { return (units + kRowsWaves - 1) / kRowsWaves; }

int launch_gemv_rows(const GroupPhase *tab, const uint32_t *part_tab, int nparts, const uint32_t *order, int grid,
                     int M, uint32_t *tickets, hipStream_t st) {
    if (nparts <= 0 || grid <= 0) return NVQ_OK;
    if (M > 16)
        hipLaunchKernelGGL(gemv_rows_kernel<2>, dim3(grid), dim3(kRowsWaves * 64), 0, st, tab, part_tab, nparts, order,
                           M, tickets);
    else
        hipLaunchKernelGGL(gemv_rows_kernel<1>, dim3(grid), dim3(kRowsWaves * 64), 0, st, tab, part_tab, nparts, order,
                           M, tickets);
    NVQ_HIP_TRY(hipGetLastError());
    return NVQ_OK;
}

}  // namespace nvq

// Small batches of 17 to 32 tokens through many independent phases as one persistent
// grid (plans whose K are all multiples of 512).  Paper: the W4A8 / W4A16 kernel
// descriptions; the arithmetic is that of mfma_act.h.
//
// With two token tiles 32 weight rows need 3.6 times their own bytes of bf16 activations,
// and the L2 caches deliver about 10 TB/s to all compute units together: a kernel whose
// waves each fetch their own (the ring kernel, which serves up to 16 tokens and shorter lists)
// stands at 3 TB/s of weights.  So a workgroup takes 128 rows at a time: four waves, each with 32 rows
// of its own (two 16-row tiles, a unit of the batch) and all of K, share the activations
// through LDS, and no sums cross the waves.  K advances by 256 inputs (a whole 128-byte
// line of a row); per step a wave asks for its quarter of the next step's activations (two
// buffers) and, once the current step's weights and scales are in registers, for its next
// weights, all straight from global memory into LDS; one barrier per step says that the
// activations have arrived and that the other buffer is free.  Three workgroups share a
// compute unit.
//
// The batch is cut into parts, one per XCD (the compute units of an XCD advance through
// the phases together, so that the activations they all read stay in their L2); the
// workgroups of a part take its groups of four units first come first served from a
// counter, which the quantisation launch in front has cleared.
//
// What bounds it: 8B layers at 32 tokens take 1,133 us (3.9 TB/s; 1,124 with the sums of a
// result in one chain, 1,480 with the ring kernel); without the loads 820-870, without the products 1,030, so either alone comes
// close and the two overlap by half.  Eight waves and 256 rows per workgroup are as fast
// on long lists and 15 % slower on short ones; 64 rows per wave 4 % slower, two steps of
// weights in flight with two thirds of the waves 15 %.
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
constexpr int kRowsWgPerCu = 3;
constexpr int kRowsW = 2 * 2048;   // a wave's weights of a step: 32 rows x 128 bytes
constexpr int kRowsSlot = kRowsW + 512;  // and its scales, 16 bytes per row

// A bundle: up to four consecutive units of one phase.
struct RowsBundle {
    int p;            // phase
    int unit, count;  // first unit (of the phase) and how many
    int next;         // unit of the batch after the bundle
    int end;          // end of the group of units it belongs to
};

__device__ __forceinline__ RowsBundle rows_bundle(CGroup *tab, int p, int u, int end) {
    RowsBundle b;
    while (u >= tab[p].unit_begin + tab[p].unit_count) ++p;  // phases have units
    const int phase_end = tab[p].unit_begin + tab[p].unit_count;
    b.p = p;
    b.unit = u - tab[p].unit_begin;
    b.next = end < phase_end ? end : phase_end;
    b.count = b.next - u;
    b.end = end;
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

__global__ __launch_bounds__(kRowsWaves * 64) __attribute__((amdgpu_waves_per_eu(3))) void
gemv_rows_kernel(const GroupPhase *__restrict__ tab_, const uint32_t *__restrict__ part_tab_, int nparts,
                 int M, uint32_t *__restrict__ tickets) {
    constexpr int MT = 2, R = 2;   // token tiles, row tiles of a wave
    constexpr int kA = 32 * 512;  // an activation buffer (bf16; codes fill half of it)
    constexpr int kASlice = 16 / kRowsWaves;  // loads of a wave and step, bf16 (codes: half)
    __shared__ __attribute__((aligned(1024))) unsigned char lds[2 * kA + kRowsWaves * kRowsSlot];
    __shared__ int ticket_word;
    CGroup *tab = (CGroup *)tab_;
    CWord *part_tab = (CWord *)part_tab_;
    const int lane = threadIdx.x & 63;
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int n = lane & 15, kb = lane >> 4;
    unsigned char *const slot = lds + 2 * kA + w * kRowsSlot;

    const int part = (int)blockIdx.x % nparts;
    const int part_end = (int)part_tab[part + 1];
    const int part_wgs = ((int)gridDim.x - 1 - part) / nparts + 1;
    const int part_begin = (int)part_tab[part];
    // the group of ticket t: units part_begin + 4 t .. + 3
    int t = (int)blockIdx.x / nparts;
    if (part_begin + t * kRowsWaves >= part_end) return;
    auto group_end = [&](int first) { return first + kRowsWaves < part_end ? first + kRowsWaves : part_end; };

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
    // the wave's share of step c's activations: whole lines of 2 (bf16) or 4 (codes) tokens
    // per load, a token's pieces permuted by its number
    auto issue_a = [&](const RowsSource &s, int c, int buf) {
        const bool codes = s.precision == NVQ_W4A8;
        unsigned char *const dst = lds + buf * kA;
#pragma unroll
        for (int j = 0; j < kASlice; ++j) {
            if (codes && j >= kASlice / 2) continue;
            const int i = (codes ? kASlice / 2 : kASlice) * w + j;
            const int m = codes ? 4 * i + (lane >> 4) : 2 * i + (lane >> 5);
            const int p = codes ? (lane & 15) ^ (m & 15) : (lane & 31) ^ (m & 15);
            const uint32_t row = (uint32_t)(s.G * (codes ? 32 : 64));
            const char *src = s.a + (size_t)c * (codes ? 256 : 512) +
                              ((uint32_t)(m < M ? m : M - 1) * row + 16u * (uint32_t)p);
            __builtin_amdgcn_global_load_lds((const void *)src, (rows_lds_ptr)(dst + i * 1024), 16, 0, 0);
        }
    };
    // Weights, load j: rows 8 j .. + 7 of the wave's 32, lane l piece (l % 8) ^ (row / 2 % 8)
    // of row l / 8; scales: 16 bytes of row l.
    auto issue_w = [&](const RowsSource &s, int c) {
        if (!s.active) return;
        int lane = threadIdx.x & 63;  // (opaque, see the result store)
        asm volatile("" : "+v"(lane));
        const int wrow = lane >> 3;
        const uint32_t row_bytes = (uint32_t)s.G * 16;  // a multiple of 256
        const uint32_t lo = (uint32_t)wrow * row_bytes + 16u * (uint32_t)((lane & 7) ^ (wrow >> 1));
        if (s.whole) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                __builtin_amdgcn_global_load_lds(
                    (const void *)(s.w + ((size_t)c * 128 + (size_t)(8 * j) * row_bytes) + ((j & 1) ? lo ^ 64u : lo)),
                    (rows_lds_ptr)(slot + j * 1024), 16, 0, 2);
            if (lane < 32)
                __builtin_amdgcn_global_load_lds((const void *)(s.s + (size_t)c * 16 + (uint32_t)lane * (uint32_t)s.G * 2u),
                                                 (rows_lds_ptr)(slot + kRowsW), 16, 0, 0);
            return;
        }
        CGroup &P = tab[s.p];
        for (int j = 0; j < 4; ++j) {
            const char *row = reinterpret_cast<const char *>(locate_row(P.segs, s.row0 + 8 * j + wrow, s.G).qw);
            const int pc = (lane & 7) ^ ((4 * j + (wrow >> 1)) & 7);
            __builtin_amdgcn_global_load_lds((const void *)(row + (size_t)c * 128 + 16 * pc),
                                             (rows_lds_ptr)(slot + j * 1024), 16, 0, 2);
        }
        const char *srow = reinterpret_cast<const char *>(locate_row(P.segs, s.row0 + (lane & 31), s.G).sc);
        if (lane < 32)
            __builtin_amdgcn_global_load_lds((const void *)(srow + (size_t)c * 16), (rows_lds_ptr)(slot + kRowsW), 16,
                                             0, 0);
    };

    // The lane's places.  Weights: dword kb of piece i of row n, piece i at position i ^ (n / 2
    // % 8); activations: W4A16 half a piece twice (pieces 4 i + 2 h + kb / 2 of half a step), W4A8
    // a dword twice (pieces 2 i + h), piece p at position p ^ n.  The permutations leave the
    // rest of an address alone: another piece is one xor away.
    const uint32_t at = (uint32_t)(uintptr_t)slot, abase = (uint32_t)(uintptr_t)lds;
    const uint32_t wpos = at + n * 128 + 16 * ((n >> 1) & 7) + 4 * kb;
    const uint32_t spos = at + kRowsW + 16 * n;
    const uint32_t apos16 = abase + n * 512 + 16 * ((kb >> 1) ^ n) + 8 * (kb & 1);
    const uint32_t apos8 = abase + n * 256 + 16 * n + 4 * kb;

    // A result's sum in three levels: the eight groups of a step, eight steps, all of K.  (One
    // chain over all of K had up to twice the error of the four that the kernel for up to 16 tokens
    // adds, registers for four would be 64; this is closer than those, at any K, for 2 % more
    // vector instructions.)
    float f[R][MT][4], total[R][MT][4];
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

#define NVQ_RD32(dst_, addr_, off_) asm volatile("ds_read_b32 %0, %1 offset:%2" : "=v"(dst_) : "v"(addr_), "n"(off_))
#define NVQ_RD64(dst_, addr_, off_) asm volatile("ds_read_b64 %0, %1 offset:%2" : "=v"(dst_) : "v"(addr_), "n"(off_))
    // The products of a step, group by group; the activations of a group are read from LDS
    // while the one before it is multiplied.
    auto products = [&](auto prec, uint32_t abuf, const uint32_t (&q)[R][8], const uint32_t (&sc)[R][4]) {
        constexpr int PREC = decltype(prec)::value;
        typedef Act<PREC> A;
        float part[R][MT][4];
        uint2v a2[2][PREC == NVQ_W4A8 ? 1 : MT][2];
        uint32_t a1[2][PREC == NVQ_W4A8 ? MT : 1][2];
        auto read = [&](int g) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint32_t pos = abuf ^ (uint32_t)(PREC == NVQ_W4A8 ? 16 * (2 * g + h) : 16 * (4 * g + 2 * h));
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    if (PREC == NVQ_W4A8)
                        NVQ_RD32(a1[g & 1][mt][h], pos, mt * 16 * 256);
                    else
                        NVQ_RD64(a2[g & 1][mt][h], pos, mt * 16 * 512);
                }
            }
        };
        read(0);
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            __builtin_amdgcn_sched_barrier(0);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if (PREC == NVQ_W4A8)
                    asm volatile("" : "+v"(a1[g & 1][mt][0]), "+v"(a1[g & 1][mt][1]));
                else
                    asm volatile("" : "+v"(a2[g & 1][mt][0]), "+v"(a2[g & 1][mt][1]));
            }
            if (g < 7) read(g + 1);
            __builtin_amdgcn_sched_barrier(0);
            typename A::operand act[MT];
            typename A::offset_t off[MT];
#pragma unroll
            for (int mt = 0; mt < MT; ++mt) {
                if constexpr (PREC == NVQ_W4A8) {
                    act[mt] = (long)((uint64_t)a1[g & 1][mt][0] | ((uint64_t)a1[g & 1][mt][1] << 32));
                } else {
                    const uint4v v = {a2[g & 1][mt][0].x, a2[g & 1][mt][0].y, a2[g & 1][mt][1].x, a2[g & 1][mt][1].y};
                    act[mt] = __builtin_bit_cast(bf16x8, v);
                }
                if (PREC == NVQ_W4A16) off[mt] = A::offset(act[mt]);
            }
            // W4A8: no correction, the weights enter as 16 (n - 8): the nibble in the high half of
            // its byte, its top bit flipped (the factor leaves with the activation scale)
            if constexpr (PREC == NVQ_W4A8) off[0] = off[MT - 1] = int4v{0, 0, 0, 0};
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float sw = half_bits_to_float((uint16_t)(sc[r][g >> 1] >> (16 * (g & 1))));
                typename A::operand wt;
                if constexpr (PREC == NVQ_W4A8) {
                    const uint32_t v = q[r][g] ^ 0x88888888u;
                    wt = (long)((uint64_t)((v << 4) & 0xf0f0f0f0u) | ((uint64_t)(v & 0xf0f0f0f0u) << 32));
                } else {
                    wt = A::weights(q[r][g]);
                }
#pragma unroll
                for (int mt = 0; mt < MT; ++mt) {
                    int4v raw;
                    const float4v p = A::product(act[mt], wt, off[mt], raw);
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj)
                        part[r][mt][jj] = g > 0 ? fmaf(sw, p[jj], part[r][mt][jj]) : sw * p[jj];
                    // (here and now: the compiler would gather the additions of a step at its end and keep
                    // the products until then)
                    asm volatile("" : "+v"(part[r][mt][0]), "+v"(part[r][mt][1]), "+v"(part[r][mt][2]),
                                 "+v"(part[r][mt][3]));
                }
            }
        }
        add(f, part);
    };

    const int first = part_begin + t * kRowsWaves;
    RowsBundle cur = rows_bundle(tab, (int)part_tab[nparts + 1 + part], first, group_end(first));
    RowsSource src = source(cur);
    int buf = 0;
    issue_a(src, 0, 0);
    issue_w(src, 0);
    while (true) {
        const int G = src.G, steps = G >> 3;
        const bool active = src.active, codes = src.precision == NVQ_W4A8;
        const bool last_of_group = cur.next >= cur.end;
        bool more = false;
        RowsBundle nxt = cur;
        int drawn = 0;
        clear(f);
        clear(total);
        for (int c = 0; c < steps; ++c) {
            // this step's operands have arrived; everyone has left the other buffer
            __builtin_amdgcn_s_waitcnt(0x0f70);  // vmcnt(0)
            if (c == 1 && last_of_group && w == 0 && lane == 0) ticket_word = drawn;
            __syncthreads();
            if (c == 0 && last_of_group && w == 0 && lane == 0)  // read at the next step's barrier
                drawn = (int)__hip_atomic_fetch_add(&tickets[part], 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (c + 1 < steps) {
                issue_a(src, c + 1, buf ^ 1);
            } else {
                // the bundle after this one: the rest of the group, or the next ticket's
                int u = cur.next, e = cur.end;
                if (last_of_group) {
                    t = part_wgs + __builtin_amdgcn_readfirstlane(ticket_word);
                    u = part_begin + t * kRowsWaves;
                    e = group_end(u);
                }
                more = u < part_end;
                if (more) {
                    nxt = rows_bundle(tab, cur.p, u, e);
                    src = source(nxt);  // from here on the next bundle's
                    issue_a(src, 0, buf ^ 1);
                }
            }
            uint32_t q[R][8], sc[R][4];
#pragma unroll
            for (int i = 0; i < 8; ++i)
#pragma unroll
                for (int r = 0; r < R; ++r) NVQ_RD32(q[r][i], wpos ^ (16 * i), r * 2048);
#pragma unroll
            for (int r = 0; r < R; ++r)
#pragma unroll
                for (int k = 0; k < 4; ++k) NVQ_RD32(sc[r][k], spos, r * 256 + 4 * k);
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
            for (int r = 0; r < R; ++r) {
#pragma unroll
                for (int i = 0; i < 8; ++i) asm volatile("" : "+v"(q[r][i]));
#pragma unroll
                for (int k = 0; k < 4; ++k) asm volatile("" : "+v"(sc[r][k]));
            }
            if (c + 1 < steps || more) issue_w(src, c + 1 < steps ? c + 1 : 0);
            if (active) {
                if (codes)
                    products(std::integral_constant<int, NVQ_W4A8>(), apos8 + buf * kA, q, sc);
                else
                    products(std::integral_constant<int, NVQ_W4A16>(), apos16 + buf * kA, q, sc);
            }
            if ((c & 7) == 7) {
                add(total, f);
                clear(f);
            }
            buf ^= 1;
        }
        add(total, f);
        if (active) {
            CGroup &P = tab[cur.p];
            // (opaque: what follows from them would be kept in registers across the whole loop, and
            // others spilled; a spill's reload waits for every load in flight)
            int kb = lane >> 4, n = lane & 15;
            asm volatile("" : "+v"(kb), "+v"(n));
            float xs[MT][4];  // per-token activation scale of the lane's results (W4A8)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const int m = mt * 16 + kb * 4 + jj;
                    xs[mt][jj] = codes && m < M ? 0.0625f * as_global<float>(P.xscale)[m] : 1.0f;
                }
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const RowRef o = locate_row(P.segs, ((cur.unit + w) * R + r) * 16 + n, G);
#pragma unroll
                for (int mt = 0; mt < MT; ++mt)
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj) {
                        const int m = mt * 16 + kb * 4 + jj;
                        if (o.valid && m < M)
                            store_global(o.y, o.y_dtype, (int64_t)m * o.N + o.n, total[r][mt][jj] * xs[mt][jj]);
                    }
            }
        }
        if (!more) break;
        cur = nxt;
    }
#undef NVQ_RD32
#undef NVQ_RD64
}

}  // namespace

// A workgroup per group of units (every part may end with a smaller one), at most what is resident.
int rows_grid(int nunits, int nparts) {
    const int groups = (nunits + kRowsWaves - 1) / kRowsWaves + nparts, cap = kRowsWgPerCu * device_cu_count();
    return groups < cap ? groups : cap;
}

int launch_gemv_rows(const GroupPhase *tab, const uint32_t *part_tab, int nparts, int grid, int M,
                     uint32_t *tickets, hipStream_t st) {
    if (nparts <= 0 || grid <= 0) return NVQ_OK;
    hipLaunchKernelGGL(gemv_rows_kernel, dim3(grid), dim3(kRowsWaves * 64), 0, st, tab, part_tab, nparts, M,
                       tickets);
    NVQ_HIP_TRY(hipGetLastError());
    return NVQ_OK;
}

}  // namespace nvq

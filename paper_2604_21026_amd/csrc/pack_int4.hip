// nvq_pack_int4: fp32 weights -> planar int4 codes + fp16 group scales.
// Block format after the paper's W4A8 section (32 weights, one fp16 scale,
// nibbles centred at 8); scale rule absmax / 7, round-half-to-even, IEEE
// division so that a CPU implementation of the same rule gives the same bytes.
//
// Eight lanes own one group of 32 weights (one float4 each), so a wave reads
// 1 KiB of consecutive weights per load, two or four loads in flight.  Lanes 0-3 of a
// team hold the low nibbles of the 16 output bytes, lanes 4-7 the high nibbles;
// the lanes exchange through the data-parallel moves of the vector ALU, and
// lanes 0-3 store one dword each.  (Four lanes per group, which need no exchange of nibbles, read
// half lines per load: 50 us against 44.)
//
// The codes are those of an IEEE division, without dividing: v * rcp(s) differs from v / s by less
// than 2^-18 (three roundings; |v / s| < 16: the fp16 scale is at least half of absmax / 7), so the two
// round to the same integer unless the product lies within 2^-16 of a tie, where the division
// decides.  Rounding (half to even) is an addition: the sum with 1.5 * 2^23 + 8 holds the code in its
// low bits; clamping first gives the same, the bounds being integers.  The memory's mix of reads and
// writes and the vector ALU bound it about equally: 14336 x 4096 46.3 us with two loads in flight, a full
// reciprocal and conversions to integers, 43.6 with four and neither, 42.1 (6.4 TB/s) in runs as below.
#include "nvq_internal.h"

namespace nvq {

typedef float pack_f32x4 __attribute__((ext_vector_type(4)));
constexpr int kPackXcds = 8;

// First group of a workgroup's i-th load of U.  Workgroups b and b + 8 run on one XCD; a workgroup takes a
// run of 64 groups, or with four loads two that lie eight apart, so that run r is written by XCD r mod 8:
// the one whose workgroup of nvq_dequant_bf16 (64 groups each) reads it next, from its own L2.  (With 128
// groups in a row 4096 x 4096 packed and unpacked took 22.6 us, with two loads in flight, 64 in a row, 20.2: passes
// repeated over the same buffers; a first pass over new ones gains nothing.  That workgroups go to XCDs in
// turn is what was observed: where they do not, the bytes are the same and the gain is gone.)
template <int U>
__device__ __forceinline__ int64_t pack_first(int64_t b, int i) {
    static_assert(U == 2 || U == 4, "one or two runs of 64 groups");
    if (U == 2) return b * 64 + i * 32;
    const int64_t run = b / kPackXcds * (2 * kPackXcds) + b % kPackXcds + (i >> 1) * kPackXcds;
    return run * 64 + (i & 1) * 32;
}

// The value of lane i ^ 1, i ^ 2, or 7 - i (within eight lanes).
template <int CTRL>
__device__ __forceinline__ uint32_t pack_dpp(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, 0xf, 0xf, false);
}
constexpr int kDppXor1 = 0xb1, kDppXor2 = 0x4e, kDppXor3 = 0x1b, kDppMirror8 = 0x141;

template <int U>
__global__ __launch_bounds__(256) void pack_int4_kernel(const float4 *__restrict__ W,
                                                        int64_t total_groups,
                                                        uint32_t *__restrict__ qw,
                                                        uint16_t *__restrict__ scales) {
    const int sub = threadIdx.x & 7;
    int64_t gid[U];
    bool valid[U];
    pack_f32x4 w[U];
#pragma unroll
    for (int i = 0; i < U; ++i) {
        gid[i] = pack_first<U>(blockIdx.x, i) + (threadIdx.x >> 3);
        valid[i] = gid[i] < total_groups;
        if (!valid[i]) gid[i] = total_groups - 1;  // keep the whole team in the exchange below
        w[i] = __builtin_nontemporal_load(reinterpret_cast<const pack_f32x4 *>(W) + gid[i] * 8 + sub);
    }
#pragma unroll
    for (int i = 0; i < U; ++i) {
        float amax = fmaxf(fmaxf(fabsf(w[i].x), fabsf(w[i].y)), fmaxf(fabsf(w[i].z), fabsf(w[i].w)));
        amax = fmaxf(amax, __uint_as_float(pack_dpp<kDppXor1>(__float_as_uint(amax))));
        amax = fmaxf(amax, __uint_as_float(pack_dpp<kDppXor2>(__float_as_uint(amax))));
        amax = fmaxf(amax, __uint_as_float(pack_dpp<kDppMirror8>(__float_as_uint(amax))));

        const float s32 = amax / 7.0f;
        const _Float16 sh = (_Float16)s32;  // round to nearest even
        const float s = (float)sh;
        const bool live = (s != 0.0f) && !__builtin_isinf(s);
        const float inv = __builtin_amdgcn_rcpf(s);

        constexpr float kCode = 12582912.0f + 8.0f;  // 1.5 * 2^23 + 8
        float t[4], off = 0.0f;  // off: the largest distance from an integer
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const float c = fminf(fmaxf(w[i][k] * inv, -8.0f), 7.0f);
            t[k] = c + kCode;
            off = fmaxf(off, fabsf(c - (t[k] - kCode)));
        }
        if (off > 0.5f - 0x1p-16f) {
#pragma unroll
            for (int k = 0; k < 4; ++k) t[k] = fminf(fmaxf(w[i][k] / s, -8.0f), 7.0f) + kCode;
        }
        // the lowest bytes of the four words
        uint32_t mine = __builtin_amdgcn_perm(__float_as_uint(t[1]), __float_as_uint(t[0]), 0x0c0c0400u) |
                        __builtin_amdgcn_perm(__float_as_uint(t[3]), __float_as_uint(t[2]), 0x04000c0cu);
        if (!live) mine = 0x08080808u;
        const uint32_t other = pack_dpp<kDppXor3>(pack_dpp<kDppMirror8>(mine));  // of lane i ^ 4
        if (valid[i]) {
            if (sub < 4) qw[gid[i] * 4 + sub] = mine | (other << 4);
            if (sub == 0) scales[gid[i]] = __builtin_bit_cast(uint16_t, sh);
        }
    }
}

}  // namespace nvq

extern "C" int nvq_pack_int4(const float *W, int64_t N, int64_t K, int group, uint8_t *qweight,
                             uint16_t *scales, void *stream) {
    if (!W || !qweight || !scales) return NVQ_ERR_INVALID_ARG;
    if (group != 32) return NVQ_ERR_UNSUPPORTED;
    if (N <= 0 || K <= 0 || (K % 32) != 0 || K > NVQ_MAX_K) return NVQ_ERR_SHAPE;
    if (!nvq::aligned(W, 16) || !nvq::aligned(qweight, 16) || !nvq::aligned(scales, 2))
        return NVQ_ERR_ALIGN;
    const int64_t groups = N * (K / 32);
    const float4 *const w = reinterpret_cast<const float4 *>(W);
    uint32_t *const q = reinterpret_cast<uint32_t *>(qweight);
    // Two loads in flight while workgroups of 64 groups are all resident, eight per compute unit: one
    // trip to memory by twice the waves.  32 groups 2.0 us against 2.3 with four, 4096 2.35 and 2.94, 65536
    // 2.95 and 3.23, 131072 (the line) 4.27 and 4.44, 196608 6.3 and 6.0, 524288 13.05 and 12.25.
    if (groups <= (int64_t)64 * 8 * nvq::device_cu_count()) {
        hipLaunchKernelGGL(nvq::pack_int4_kernel<2>, dim3((unsigned)((groups + 63) / 64)), dim3(256), 0,
                           (hipStream_t)stream, w, groups, q, scales);
    } else {
        constexpr int64_t kSpan = 128 * nvq::kPackXcds;  // groups of eight workgroups
        const int64_t blocks = (groups + kSpan - 1) / kSpan * nvq::kPackXcds;
        if (blocks > 0x7fffffffLL) return NVQ_ERR_SHAPE;
        hipLaunchKernelGGL(nvq::pack_int4_kernel<4>, dim3((unsigned)blocks), dim3(256), 0, (hipStream_t)stream, w,
                           groups, q, scales);
    }
    NVQ_HIP_TRY(hipGetLastError());
    return NVQ_OK;
}

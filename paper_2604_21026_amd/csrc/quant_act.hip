// nvq_quant_act_i8: bf16 activations -> int8 codes, fp32 scale(s) and the
// per-32 code sums that the W4A8 GEMV's deferred correction needs.
// Paper, appendix "F16 -> Q8 Activation Quantization": s = amax / 127,
// q = round(x / s), clamp to [-127, 127].  Rounding is half-to-even and the
// division is IEEE binary32, so a CPU run of the same rule gives equal codes.
//
// One workgroup per token.  A thread handles chunks of 8 consecutive values
// (one 128-bit load); four neighbouring lanes therefore cover one group of 32
// and reduce its code sum (and, for per-group scales, its absmax) with two
// cross-lane exchanges.  Pass 1 finds the token's absmax, pass 2 re-reads the
// (cache-resident) row and quantises.
#include "mfma_act.h"
#include "transform.h"

namespace nvq {

constexpr int kQuantThreads = 256;

struct MaxOp {
    __device__ float operator()(float a, float b) const { return fmaxf(a, b); }
};
// Over the lanes of a wave, in every lane; in the order 32, 16, .. 1 apart.
template <typename OP>
__device__ __forceinline__ float over_wave(float a, OP op) {
    a = with_lane_xor<32>(a, op);
    a = with_lane_xor<16>(a, op);
    a = with_lane_xor<8>(a, op);
    a = with_lane_xor<4>(a, op);
    a = with_lane_xor<2>(a, op);
    return with_lane_xor<1>(a, op);
}
// Over the four lanes of a group.
template <typename T, typename OP>
__device__ __forceinline__ T over_group(T a, OP op) {
    return with_lane_xor<2>(with_lane_xor<1>(a, op), op);
}

__device__ __forceinline__ float chunk_absmax(const uint4 &v) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    float a = 0.0f;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        a = fmaxf(a, fabsf(bf16_bits_to_float(w[i] & 0xffffu)));
        a = fmaxf(a, fabsf(bf16_bits_to_float(w[i] >> 16)));
    }
    return a;
}

// The codes of eight values with scale s, packed, and their sum.  One division per scale instead
// of one per value (some ten instructions each): t = x * fl(1 / s), corrected once by its exact remainder,
// is the quotient fl(x / s) to the bit for every bf16 x of at most the maximum that s = fl(amax / 127)
// comes from (all 128 significands of amax with all 128 of x; tests/test_quant_by_reciprocal.py).
// Without a branch: x / s lies on a tie for every x = amax / 2, so that nearly every wave had some lane
// that divided where only values near a tie were divided (a scale per group, 8 x 2048: 2.5 us, with a
// division per value 2.1, now 1.9; a list of ten phases through the rings, 3 tokens: 52.8, 48.1, now 47.1).
// Where the scale is too small for that, zero or infinite, the lane divides.
__device__ __forceinline__ uint2 quant8(const uint4 &v, float s, int *sum) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
    const bool by_reciprocal = s >= 0x1p-90f && s < 0x1p127f;
    const float inv_s = by_reciprocal ? 1.0f / s : 0.0f;
    float x[8], r[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[2 * i] = bf16_bits_to_float(w[i] & 0xffffu);
        x[2 * i + 1] = bf16_bits_to_float(w[i] >> 16);
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const float t = x[i] * inv_s;
        r[i] = rintf(fmaf(fmaf(-t, s, x[i]), inv_s, t));
    }
    if (!by_reciprocal) {
#pragma unroll
        for (int i = 0; i < 8; ++i) r[i] = s != 0.0f ? rintf(x[i] / s) : 0.0f;
    }
    int q[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) q[i] = (int)fminf(fmaxf(r[i], -127.0f), 127.0f);
    *sum = ((q[0] + q[1]) + (q[2] + q[3])) + ((q[4] + q[5]) + (q[6] + q[7]));
    uint2 out;
    out.x = (uint32_t)(q[0] & 0xff) | ((uint32_t)(q[1] & 0xff) << 8) |
            ((uint32_t)(q[2] & 0xff) << 16) | ((uint32_t)(q[3] & 0xff) << 24);
    out.y = (uint32_t)(q[4] & 0xff) | ((uint32_t)(q[5] & 0xff) << 8) |
            ((uint32_t)(q[6] & 0xff) << 16) | ((uint32_t)(q[7] & 0xff) << 24);
    return out;
}

// Codes and code sum of chunk c (eight values, a quarter of a group) of a token.
__device__ __forceinline__ void quant_chunk(const uint4 &v, float s, int c, uint2 *__restrict__ qr,
                                            int32_t *__restrict__ gs) {
    int sum;
    qr[c] = quant8(v, s, &sum);
    if (!gs) return;  // (uniform)
    sum = over_group(sum, AddOp());
    if ((c & 3) == 0) gs[c >> 2] = sum;
}

// Token m of one [M][K] input, by one workgroup.
template <bool PER_GROUP>
__device__ __forceinline__ void quant_token(const uint4 *__restrict__ x, int K, int m,
                                            int8_t *__restrict__ xq, float *__restrict__ xscale,
                                            int32_t *__restrict__ xgsum) {
    const int chunks = K / 8;  // multiple of 4
    const int G = K / 32;
    const uint4 *xr = x + (int64_t)m * chunks;
    uint2 *qr = reinterpret_cast<uint2 *>(xq + (int64_t)m * K);
    int32_t *gs = xgsum ? xgsum + (int64_t)m * G : nullptr;

    float s_tok = 0.0f;
    if (!PER_GROUP) {
        __shared__ float red[kQuantThreads / 64];
        float a = 0.0f;
        for (int c = threadIdx.x; c < chunks; c += kQuantThreads) a = fmaxf(a, chunk_absmax(xr[c]));
        a = over_wave(a, MaxOp());
        if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
        __syncthreads();
        a = red[0];
#pragma unroll
        for (int i = 1; i < kQuantThreads / 64; ++i) a = fmaxf(a, red[i]);
        s_tok = a / 127.0f;
        if (threadIdx.x == 0) xscale[m] = s_tok;
    }

    // chunks is a multiple of 4 and the stride a multiple of 4, so the four
    // lanes of a team are valid or invalid together.
    for (int c = threadIdx.x; c < chunks; c += kQuantThreads) {
        const uint4 v = xr[c];
        float s = s_tok;
        if (PER_GROUP) {
            s = over_group(chunk_absmax(v), MaxOp()) / 127.0f;
            if ((c & 3) == 0) xscale[(int64_t)m * G + (c >> 2)] = s;
        }
        quant_chunk(v, s, c, qr, gs);
    }
}

// Input transform (transform.h) and quantisation of a token in one pass, K <= 16384: a
// thread keeps its one or two chunks of eight values in registers from the load to the
// codes.  The grid is a handful of workgroups, so what it costs is its launch (1.7 us) and a
// chain of memory, exchange and barrier latencies: one trip to memory (the norm's weights are
// asked for with the input), lane exchanges that do not pass through LDS, and one division per
// scale.  By the trace 3.7 us for norm and quantisation of 8 x 4096 and 4.4 for SiLU and
// quantisation of 8 x 14336 (4.3 and 6.2 with two trips, exchanges through LDS and a division
// per value).
// Q: 0 = the transformed bf16 values (xt), 1 = codes with a scale per token, 2 = codes with a
// scale per group.
constexpr int kPrepMaxK = 16384, kPrepThreads = 1024;

// Maximum over the workgroup; red: sixteen words (waves that are not there count as zero).
__device__ __forceinline__ float block_max(float a, float *red) {
    const int waves = (int)blockDim.x >> 6, lane = (int)threadIdx.x & 63;
    a = over_wave(a, MaxOp());
    if (lane == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    a = (lane & 15) < waves ? red[lane & 15] : 0.0f;
    a = with_lane_xor<8>(a, MaxOp());
    a = with_lane_xor<4>(a, MaxOp());
    return over_group(a, MaxOp());
}

// The sum of the chunks' sums in the order of the norm kernel (transform.hip), so that a layer
// prepared here reads the same bf16 values, and gets the same codes, as one prepared by that
// call: thread t of 256 adds chunks t, t + 256, ... one after the other, then the lanes of a
// wave and the waves.  (With the chunks added as the threads here hold them, one value in some
// ten thousand rounded the other way, and every layer behind it saw that.)  Chunks and waves that
// are not there add zero.
constexpr int kNormThreads = 256;
template <int N>  // chunks that part has room for
__device__ __forceinline__ float chunk_sums_in_norm_order(const float (&part)[N], int chunks, float *red) {
    const int t = (int)threadIdx.x;
    if (t < kNormThreads) {
        float v[N / kNormThreads], ss = 0.0f;
#pragma unroll
        for (int i = 0; i < N / kNormThreads; ++i)
            v[i] = t + i * kNormThreads < chunks ? part[t + i * kNormThreads] : 0.0f;
#pragma unroll
        for (int i = 0; i < N / kNormThreads; ++i) ss += v[i];
        ss = over_wave(ss, AddOp());
        if ((t & 63) == 0) red[t >> 6] = ss;
    }
    __syncthreads();
    const int waves = (int)blockDim.x >> 6;
    float ss = red[0];
#pragma unroll
    for (int i = 1; i < kNormThreads / 64; ++i) ss += i < waves ? red[i] : 0.0f;
    return ss;
}

struct PrepJob {
    const void *x, *x2, *gamma;
    void *xt, *h_out;
    int8_t *xq;
    float *xscale;
    int32_t *xgsum;  // null: no code sums
    float eps;
    int op;  // nvq_linear.in_op
};
template <int NP>
struct PrepArgs {
    int K, M;
    PrepJob job[NP];  // workgroups 0 .. M - 1 the first
};

// (the pointers come out of memory: see as_global)
__device__ __forceinline__ uint4 load16(const void *p, int64_t i) {
    const uint4v v = as_global<uint4v>(p)[i];
    return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ __forceinline__ void store16(void *p, int64_t i, const uint4 &v) {
    const uint4v o = {v.x, v.y, v.z, v.w};
    ((__attribute__((address_space(1))) uint4v *)p)[i] = o;
}
template <typename T>
__device__ __forceinline__ void store_word(void *p, int64_t i, T v) {
    ((__attribute__((address_space(1))) T *)p)[i] = v;
}

// Token m of a job.
template <int OP, int Q, int NCH, class JOB>
__device__ __forceinline__ void prep_token(const JOB &J, int K, int m, float (&red)[2][16],
                                           float (&part)[kPrepThreads * NCH]) {
    const int chunks = K / 8, G = K / 32;
    const int64_t row = (int64_t)m * chunks;
    const void *const x2 = J.x2, *const h_out = J.h_out;
    uint4 v[NCH], gm[NCH];
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = (int)threadIdx.x + i * (int)blockDim.x;
        v[i] = make_uint4(0u, 0u, 0u, 0u);
        if (c < chunks) {
            v[i] = load16(J.x, row + c);
            if (OP == NVQ_IN_RMSNORM) {
                gm[i] = load16(J.gamma, c);  // (asked for here: one trip to memory less)
                if (x2) v[i] = add_bf16x8(v[i], load16(x2, row + c));
                if (h_out) store16(J.h_out, row + c, v[i]);
                part[c] = sumsq_bf16x8(v[i]);
            } else if (OP == NVQ_IN_SILU_MUL) {
                v[i] = silu_mul_bf16x8(v[i], load16(x2, row + c));
            }
        }
    }
    if constexpr (OP == NVQ_IN_RMSNORM) {
        __syncthreads();
        const float r = rms_scale(chunk_sums_in_norm_order(part, chunks, red[0]), K, J.eps);
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int c = (int)threadIdx.x + i * (int)blockDim.x;
            if (c < chunks) v[i] = scale_bf16x8(v[i], r, gm[i]);
        }
    }
    if (Q == 0) {
#pragma unroll
        for (int i = 0; i < NCH; ++i) {
            const int c = (int)threadIdx.x + i * (int)blockDim.x;
            if (c < chunks) store16(J.xt, row + c, v[i]);
        }
        return;
    }
    float s = 0.0f;
    if (Q == 1) {
        float a = 0.0f;
#pragma unroll
        for (int i = 0; i < NCH; ++i) a = fmaxf(a, chunk_absmax(v[i]));
        s = block_max(a, red[1]) / 127.0f;
        if (threadIdx.x == 0) store_word(J.xscale, m, s);
    }
    // four neighbouring lanes hold a group: chunks and blockDim.x are multiples of four
#pragma unroll
    for (int i = 0; i < NCH; ++i) {
        const int c = (int)threadIdx.x + i * (int)blockDim.x;
        if (c >= chunks) continue;
        if (Q == 2) {
            s = over_group(chunk_absmax(v[i]), MaxOp()) / 127.0f;
            if ((c & 3) == 0) store_word(J.xscale, (int64_t)m * G + (c >> 2), s);
        }
        int sum;
        const uint2 q = quant8(v[i], s, &sum);
        store_word(J.xq, row + c, (uint64_t)q.x | ((uint64_t)q.y << 32));
        if (J.xgsum) {
            sum = over_group(sum, AddOp());
            if ((c & 3) == 0) store_word(J.xgsum, (int64_t)m * G + (c >> 2), sum);
        }
    }
}

template <int Q, int NCH, int NP>
__global__ __launch_bounds__(kPrepThreads) void prep_token_kernel(PrepArgs<NP>) {
    __shared__ float red[2][16];
    __shared__ float part[kPrepThreads * NCH];
    // (through the segment's pointer: indexed as a parameter the struct would be copied to scratch; it is
    // the kernel's only parameter, so the segment begins with it)
    const __attribute__((address_space(4))) PrepArgs<NP> &A =
        *(const __attribute__((address_space(4))) PrepArgs<NP> *)__builtin_amdgcn_kernarg_segment_ptr();
    const int second = NP > 1 && (int)blockIdx.x >= A.M ? 1 : 0, m = (int)blockIdx.x - (second ? A.M : 0);
    const __attribute__((address_space(4))) PrepJob &J = A.job[second];
    if (J.op == NVQ_IN_RMSNORM)
        prep_token<NVQ_IN_RMSNORM, Q, NCH>(J, A.K, m, red, part);
    else if (J.op == NVQ_IN_SILU_MUL)
        prep_token<NVQ_IN_SILU_MUL, Q, NCH>(J, A.K, m, red, part);
    else
        prep_token<NVQ_IN_PLAIN, Q, NCH>(J, A.K, m, red, part);
}

template <bool PER_GROUP>
__global__ __launch_bounds__(kQuantThreads) void quant_act_kernel(
    const uint4 *__restrict__ x, int K, int8_t *__restrict__ xq, float *__restrict__ xscale,
    int32_t *__restrict__ xgsum) {
    quant_token<PER_GROUP>(x, K, blockIdx.x, xq, xscale, xgsum);
}

// Per-token scales, the inputs of many phases in one grid.
__global__ __launch_bounds__(kQuantThreads) void quant_act_group_kernel(
    const GroupPhase *__restrict__ tab, const uint16_t *__restrict__ jobs, int njobs, int M,
    uint32_t *__restrict__ clear) {
    if (clear && blockIdx.x == 0 && threadIdx.x < 8) clear[threadIdx.x] = 0u;
    const int job = blockIdx.x / M, m = blockIdx.x - job * M;
    if (job >= njobs) return;
    const GroupPhase &P = tab[jobs[job]];
    quant_token<false>(reinterpret_cast<const uint4 *>(P.x_bf16), P.G * 32, m, P.xq, P.xscale,
                       P.xgsum);
}

// ---- operand images of the persistent small-batch kernel ---------------------
// Per tile of 16 tokens, 128-input column c and piece i one KiB whose 16 bytes
// number 16 * kb + n are, for token n of the tile, the int8 codes 32 * kb +
// 16 * i .. + 15 of the column (W4A8, two pieces) or the bf16 inputs 32 * i +
// 8 * kb .. + 7 of the column (W4A16, four pieces): the order in which a wave
// of the matrix-core kernel loads its activation operands.  Two grids: the
// per-token scales of the W4A8 phases first, then the images, a wave writing
// whole KiB pieces (one workgroup per token, as for the [M][K] codes, would
// write 8 or 16 bytes here and there into lines shared with 15 other
// workgroups).

// Per-token scale of token m of every W4A8 job (the other jobs' workgroups leave).
__global__ __launch_bounds__(kQuantThreads) void token_scale_group_kernel(
    const GroupPhase *__restrict__ tab, const uint16_t *__restrict__ jobs, int M) {
    const int job = blockIdx.x / M, m = blockIdx.x - job * M;
    const GroupPhase &P = tab[jobs[job]];
    if (P.precision != NVQ_W4A8) return;
    __shared__ float red[kQuantThreads / 64];
    const int chunks = P.G * 4;
    const uint4 *xr = reinterpret_cast<const uint4 *>(P.x_bf16) + (int64_t)m * chunks;
    float a = 0.0f;
    for (int c = threadIdx.x; c < chunks; c += kQuantThreads) a = fmaxf(a, chunk_absmax(xr[c]));
    a = over_wave(a, MaxOp());
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = a;
    __syncthreads();
    if (threadIdx.x == 0) {
        a = red[0];
#pragma unroll
        for (int i = 1; i < kQuantThreads / 64; ++i) a = fmaxf(a, red[i]);
        P.xscale[m] = a / 127.0f;
    }
}

constexpr int kImageColumns = 8;  // columns of 128 inputs per workgroup (two per wave)

// img_units[u] names the phase of grid unit u; a unit is a token tile times
// kImageColumns columns of that phase.  Token slots past M are left as they are.
__global__ __launch_bounds__(kQuantThreads) void operand_image_group_kernel(
    const GroupPhase *__restrict__ tab, const uint16_t *__restrict__ img_units, int M) {
    const GroupPhase &P = tab[img_units[blockIdx.x]];
    const int local = blockIdx.x - P.img_begin;
    const int C4 = P.G >> 2, cblocks = (C4 + kImageColumns - 1) / kImageColumns;
    const int mt = local / cblocks, cb = local - mt * cblocks;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int n = lane & 15, kb = lane >> 4;
    const int m = mt * 16 + n;
    if (m >= M) return;
    const uint16_t *xr = P.x_bf16 + (int64_t)m * (P.G * 32);
    if (P.precision == NVQ_W4A8) {
        const float s = P.xscale[m];
        for (int c = cb * kImageColumns + wave; c < C4 && c < (cb + 1) * kImageColumns; c += 4) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const uint4 *src = reinterpret_cast<const uint4 *>(xr + c * 128 + 32 * kb + 16 * i);
                const uint4 v0 = src[0], v1 = src[1];
                int sum;
                const uint2 q0 = quant8(v0, s, &sum), q1 = quant8(v1, s, &sum);
                *reinterpret_cast<uint4 *>(P.xa + ((size_t)(mt * C4 + c) * 2 + i) * 1024 +
                                           lane * 16) = make_uint4(q0.x, q0.y, q1.x, q1.y);
            }
        }
    } else {
        for (int c = cb * kImageColumns + wave; c < C4 && c < (cb + 1) * kImageColumns; c += 4) {
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<uint4 *>(P.xa + ((size_t)(mt * C4 + c) * 4 + i) * 1024 +
                                           lane * 16) =
                    *reinterpret_cast<const uint4 *>(xr + c * 128 + 32 * i + 8 * kb);
        }
    }
}

int image_units(int M, int K) { return ((M + 15) / 16) * ((K / 128 + kImageColumns - 1) / kImageColumns); }

int launch_operand_images(const GroupPhase *tab, const uint16_t *jobs, int njobs,
                          const uint16_t *img_units, int nimg, int M, hipStream_t st) {
    if (njobs <= 0 || nimg <= 0) return NVQ_OK;
    hipLaunchKernelGGL(token_scale_group_kernel, dim3(njobs * M), dim3(kQuantThreads), 0, st, tab,
                       jobs, M);
    NVQ_HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(operand_image_group_kernel, dim3(nimg), dim3(kQuantThreads), 0, st, tab,
                       img_units, M);
    NVQ_HIP_TRY(hipGetLastError());
    return NVQ_OK;
}

int launch_quant_act_group(const GroupPhase *tab, const uint16_t *jobs, int njobs, int M,
                           uint32_t *clear, hipStream_t st) {
    if (njobs <= 0 && !clear) return NVQ_OK;
    hipLaunchKernelGGL(quant_act_group_kernel, dim3(njobs > 0 ? njobs * M : 1), dim3(kQuantThreads), 0, st, tab,
                       jobs, njobs, M, clear);
    NVQ_HIP_TRY(hipGetLastError());
    return NVQ_OK;
}

namespace {

template <int Q, int NP>
int prep_go(const PrepArgs<kMaxMerge> &all, hipStream_t st) {
    PrepArgs<NP> a;
    a.K = all.K;
    a.M = all.M;
    for (int i = 0; i < NP; ++i) a.job[i] = all.job[i];
    const int chunks = a.K / 8;
    const int nch = chunks <= kPrepThreads ? 1 : 2, per = (chunks + nch - 1) / nch;
    const dim3 grid(NP * a.M), block((per + 63) / 64 * 64);
    if (nch == 1)
        hipLaunchKernelGGL((prep_token_kernel<Q, 1, NP>), grid, block, 0, st, a);
    else
        hipLaunchKernelGGL((prep_token_kernel<Q, 2, NP>), grid, block, 0, st, a);
    NVQ_HIP_TRY(hipGetLastError());
    return NVQ_OK;
}

template <int Q>
int prep_jobs(const PrepArgs<kMaxMerge> &a, int jobs, hipStream_t st) {
    return jobs == 2 ? prep_go<Q, 2>(a, st) : prep_go<Q, 1>(a, st);
}

}  // namespace

int launch_quant_act(const uint16_t *x, int M, int K, int act_group, int8_t *xq, float *xscale,
                     int32_t *xgsum, hipStream_t st) {
    if (K <= kPrepMaxK) {
        nvq_linear e = {};
        e.x_bf16 = x;
        e.K = K;
        const nvq_linear *const layer = &e;
        const PrepTarget to = {nullptr, xq, xscale, xgsum};
        return launch_prep(&layer, &to, 1, M, act_group, true, st);
    }
    if (act_group == 0)
        hipLaunchKernelGGL(quant_act_kernel<false>, dim3(M), dim3(kQuantThreads), 0, st,
                           reinterpret_cast<const uint4 *>(x), K, xq, xscale, xgsum);
    else
        hipLaunchKernelGGL(quant_act_kernel<true>, dim3(M), dim3(kQuantThreads), 0, st,
                           reinterpret_cast<const uint4 *>(x), K, xq, xscale, xgsum);
    NVQ_HIP_TRY(hipGetLastError());
    return NVQ_OK;
}

// A layer whose K is beyond what one pass takes: step by step.
static int prep_long(const nvq_linear &e, const PrepTarget &to, int M, int act_group, bool quant, hipStream_t st) {
    const uint16_t *x = e.x_bf16;
    if (e.in_op != NVQ_IN_PLAIN) {
        const int t = e.in_op == NVQ_IN_RMSNORM
                          ? launch_rms_norm(e.x_bf16, e.x2_bf16, e.gamma_bf16, e.eps, M, e.K, to.xt,
                                            e.h_out_bf16, st)
                          : launch_silu_mul(e.x_bf16, e.x2_bf16, M, e.K, to.xt, st);
        if (t != NVQ_OK) return t;
        x = to.xt;
    }
    return quant ? launch_quant_act(x, M, e.K, act_group, to.xq, to.xscale, to.xgsum, st) : NVQ_OK;
}

int launch_prep(const nvq_linear *const *e, const PrepTarget *to, int n, int M, int act_group, bool quant,
                hipStream_t st) {
    PrepArgs<kMaxMerge> a = {};
    a.K = e[0]->K;
    a.M = M;
    int jobs = 0;
    for (int i = 0; i < n; ++i) {
        const nvq_linear &l = *e[i];
        if (l.K > kPrepMaxK) {
            const int t = prep_long(l, to[i], M, act_group, quant, st);
            if (t != NVQ_OK) return t;
            continue;
        }
        if (!quant && l.in_op == NVQ_IN_PLAIN) continue;
        PrepJob &j = a.job[jobs++];
        j.x = l.x_bf16;
        j.x2 = l.in_op == NVQ_IN_PLAIN ? nullptr : l.x2_bf16;
        j.gamma = l.gamma_bf16;
        j.xt = to[i].xt;
        j.h_out = l.in_op == NVQ_IN_RMSNORM ? l.h_out_bf16 : nullptr;
        j.xq = to[i].xq;
        j.xscale = to[i].xscale;
        j.xgsum = to[i].xgsum;
        j.eps = l.eps;
        j.op = l.in_op;
    }
    if (jobs == 0) return NVQ_OK;
    // without the codes nothing of a SiLU spans a token: one workgroup per 256 chunks instead
    if (!quant && jobs == 1 && a.job[0].op == NVQ_IN_SILU_MUL)
        return launch_silu_mul(static_cast<const uint16_t *>(a.job[0].x), static_cast<const uint16_t *>(a.job[0].x2), M,
                               a.K, static_cast<uint16_t *>(a.job[0].xt), st);
    if (!quant) return prep_jobs<0>(a, jobs, st);
    return act_group == 0 ? prep_jobs<1>(a, jobs, st) : prep_jobs<2>(a, jobs, st);
}

}  // namespace nvq

extern "C" int nvq_quant_act_i8(const uint16_t *x_bf16, int M, int K, int act_group, int8_t *xq,
                                float *xscale, int32_t *xgsum, void *stream) {
    if (!x_bf16 || !xq || !xscale || !xgsum) return NVQ_ERR_INVALID_ARG;
    if (act_group != 0 && act_group != 32) return NVQ_ERR_INVALID_ARG;
    if (M <= 0 || M > NVQ_MAX_M || K <= 0 || (K % 32) != 0 || K > NVQ_MAX_K) return NVQ_ERR_SHAPE;
    if (!nvq::aligned(x_bf16, 16) || !nvq::aligned(xq, 16) || !nvq::aligned(xscale, 4) ||
        !nvq::aligned(xgsum, 4))
        return NVQ_ERR_ALIGN;
    return nvq::launch_quant_act(x_bf16, M, K, act_group, xq, xscale, xgsum, (hipStream_t)stream);
}

"""GPU parity: every entry point of libnvq, called through the C ABI, against
the CPU oracle on the same seeded inputs.

Bars: packed int4 bytes, fp16 scale bits, int8 activation codes, activation
scales, block sums and W4A8 int32 accumulators are bit-exact; floating-point
outputs are within 1e-3 relative L2 of the float64 oracle (fp32 accumulation;
the observed error is around 1e-6)."""
import numpy as np
import pytest
import torch

import oracle
from paper_2604_21026_amd import nvq, synth
from tests import np_ref

pytestmark = pytest.mark.gpu

TOL = 1e-3
DEV = "cuda"


def say(*a):
    print(*a, flush=True)


def u16(t):
    return t.cpu().view(torch.int16).numpy().view(np.uint16)


def packed(seed, N, K):
    W = synth.make_weight(seed, N, K)
    q, s = oracle.pack_int4(W.numpy())
    return W, q, s


def to_dev_packed(q, s):
    return (torch.from_numpy(q).to(DEV), torch.from_numpy(s.view(np.int16)).to(DEV))


def act(seed, M, K, outliers=True):
    return synth.make_activation(seed, M, K, outliers)


def test_calls_go_to_the_current_stream():
    """The stream the binding passes is torch's current one, inside a stream context and outside."""
    assert nvq._stream() == torch.cuda.current_stream().cuda_stream
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert nvq._stream() == side.cuda_stream == torch.cuda.current_stream().cuda_stream
    assert nvq._stream() == torch.cuda.current_stream().cuda_stream


# ---- a1 pack -----------------------------------------------------------------
@pytest.mark.parametrize("N,K", [(5, 32), (64, 2048), (33, 3072), (257, 4096), (7, 14336),
                                 (1, 64), (1031, 1024)])
def test_pack_int4_bit_exact(N, K):
    say("pack", N, K)
    W, q_ref, s_ref = packed(1000 + N, N, K)
    q, s = nvq.pack_int4(W.to(DEV))
    torch.cuda.synchronize()
    assert np.array_equal(q.cpu().numpy(), q_ref)
    assert np.array_equal(u16(s), s_ref)


@pytest.mark.parametrize("exp", [-26, -18, -6, 12])
def test_pack_int4_near_ties(exp):
    """Weights at most four units of last place from a tie between two codes (the kernel divides
    only there), at scales from subnormal fp16 numbers to large ones; a group count that is no
    multiple of what a workgroup takes."""
    say("pack ties", exp)
    rng = np.random.default_rng(700 + exp)
    N, K = 67, 1056
    top = np.ldexp(1 + rng.random((N, K // 32, 1)), exp).astype(np.float32)
    s = (top / np.float32(7)).astype(np.float16).astype(np.float32)
    W = ((rng.integers(-7, 7, (N, K // 32, 32)) + 0.5).astype(np.float32) * s).astype(np.float32)
    W = (W.view(np.int32) + rng.integers(-4, 5, W.shape).astype(np.int32)).view(np.float32)
    W = np.where(np.abs(W) <= top, W, 0.5 * top).astype(np.float32)
    W[:, :, :1] = top
    W = W.reshape(N, K)
    q_ref, s_ref = oracle.pack_int4(W)
    q, sc = nvq.pack_int4(torch.from_numpy(W).to(DEV))
    torch.cuda.synchronize()
    assert np.array_equal(q.cpu().numpy(), q_ref)
    assert np.array_equal(sc.cpu().numpy().view(np.uint16), s_ref)


def test_pack_int4_edge_values():
    say("pack edge")
    W = torch.zeros(4, 64)
    S7 = 2.0 ** -7
    W[0, :12] = torch.tensor([7, 2.5, 3.5, -0.5, 0.5, 1.5, -2.5, -3.5, 6.5, -6.5, 4.5, 5.5]) * S7
    W[1, 40] = 0.5                      # one zero group, one single-spike group
    W[2, :32] = 1e-7                    # scale in the fp16 subnormal range
    W[2, 32:] = -3e-6
    W[3, 5] = 7 * 65504.0               # largest finite fp16 scale
    q_ref, s_ref = oracle.pack_int4(W.numpy())
    q, s = nvq.pack_int4(W.to(DEV))
    torch.cuda.synchronize()
    assert np.array_equal(q.cpu().numpy(), q_ref)
    assert np.array_equal(u16(s), s_ref)
    assert np_ref.unpack_codes(q.cpu().numpy())[0, :12].tolist() == [7, 2, 4, 0, 0, 2, -2, -4, 6, -6, 4, 6]


# Small matrices (a run of 64 groups per workgroup): ends inside a run or at its edge, one and many
# workgroups; nothing past the end.
@pytest.mark.parametrize("G", [1, 63, 64, 65, 511, 512, 513, 577, 1023, 1024, 1025, 1537])
def test_pack_runs_of_groups(G):
    say("pack runs", G)
    W, q_ref, s_ref = packed(3100 + G, G, 32)
    Wd = W.to(DEV)
    q = torch.full(((G + 2048) * 16,), 0xa5, dtype=torch.uint8, device=DEV)
    s = torch.full((G + 2048,), 0x5a5a, dtype=torch.int16, device=DEV)
    assert nvq.lib().nvq_pack_int4(Wd.data_ptr(), G, 32, 32, q.data_ptr(), s.data_ptr(), nvq._stream()) == 0
    torch.cuda.synchronize()
    assert np.array_equal(q[:G * 16].cpu().numpy().reshape(G, 16), q_ref)
    assert np.array_equal(u16(s[:G]).reshape(s_ref.shape), s_ref)
    assert bool((q[G * 16:] == 0xa5).all()) and bool((s[G:] == 0x5a5a).all())


# ---- prefill path: dense bf16 weights ------------------------------------------
@pytest.mark.parametrize("N,K", [(3, 32), (70, 2048), (257, 4096), (5, 14336), (1031, 1024)])
def test_dequant_bf16_bit_exact(N, K):
    say("dequant", N, K)
    _, q, s = packed(1500 + N, N, K)
    qd, sd = to_dev_packed(q, s)
    out = nvq.dequant_bf16(qd, sd)
    torch.cuda.synchronize()
    assert np.array_equal(u16(out), oracle.dequant_bf16(q, s))


def test_dequant_bf16_every_nibble_and_extreme_scales():
    say("dequant extremes")
    rng = np.random.default_rng(19)
    N, K = 33, 1024
    q = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)      # includes nibble 0 = code -8
    s = rng.integers(0x0000, 0x7c00, (N, K // 32)).astype(np.uint16)   # subnormal .. 65504
    s[0, :4] = [0x0000, 0x0001, 0x7bff, 0x3c04]
    qd, sd = to_dev_packed(q, s)
    out = nvq.dequant_bf16(qd, sd)
    torch.cuda.synchronize()
    assert np.array_equal(u16(out), oracle.dequant_bf16(q, s))


# Up to eight workgroups of 64 groups per compute unit pack with two loads in flight, beyond that with
# four, in spans of 1024 groups: the line (of a device with 256 compute units), and ends inside the first
# and the second run of a workgroup and at the edges of both.  Ties and their neighbours among the groups.
@pytest.mark.parametrize("over", [0, 1, 63, 64, 511, 513, 577, 1024, 1025])
def test_pack_with_two_and_four_loads(over):
    G = 64 * 8 * torch.cuda.get_device_properties(0).multi_processor_count + over
    say("pack two and four loads", G)
    rng = np.random.default_rng(3200)
    W = rng.normal(0, 0.02, (997, 32)).astype(np.float32)
    s = (2.0 ** rng.integers(-14, 6, 997) * (1 + rng.integers(0, 1024, 997) / 1024)).astype(np.float16).astype(np.float32)
    half = rng.integers(-15, 14, (997, 32)).astype(np.float32) * np.float32(0.5) * s[:, None]
    beside = half * (1 + rng.integers(-3, 4, half.shape).astype(np.float32) * np.float32(2.0 ** -22))
    kind = np.arange(997) % 4
    W[kind == 1], W[kind == 2] = half[kind == 1], beside[kind == 2]
    W[kind % 3 != 0, 0] = (7 * s)[kind % 3 != 0]
    q_ref, s_ref = oracle.pack_int4(W)
    at = np.arange(G) % 997
    q = torch.full(((G + 2048) * 16,), 0xa5, dtype=torch.uint8, device=DEV)
    sc = torch.full((G + 2048,), 0x5a5a, dtype=torch.int16, device=DEV)
    Wd = torch.from_numpy(W).to(DEV)[torch.from_numpy(at).to(DEV)].contiguous()
    assert nvq.lib().nvq_pack_int4(Wd.data_ptr(), G, 32, 32, q.data_ptr(), sc.data_ptr(), nvq._stream()) == 0
    torch.cuda.synchronize()
    assert np.array_equal(q[:G * 16].cpu().numpy().reshape(G, 16), q_ref.reshape(997, 16)[at])
    assert np.array_equal(u16(sc[:G]).reshape(G), s_ref.reshape(997)[at])
    assert bool((q[G * 16:] == 0xa5).all()) and bool((sc[G:] == 0x5a5a).all())


# Packing: groups whose quotients are exact ties, lie a few units beside one, or reach the bounds,
# scales from subnormal halves on, groups of zeros, the last group of a workgroup and of the matrix
# (64 groups per workgroup): the oracle's bytes.
@pytest.mark.parametrize("N,K", [(1, 32), (4, 1024), (43, 96), (65, 2048)])
def test_pack_rounds_like_the_division(N, K):
    rng = np.random.default_rng(2900 + N)
    G = N * K // 32
    W = rng.normal(0, 0.02, (G, 32)).astype(np.float32)
    kind = np.arange(G) % 7
    for g in range(G):
        s = np.float32(np.float16(2.0 ** rng.integers(-14, 6) * (1 + rng.integers(0, 1024) / 1024)))
        half = rng.integers(-15, 14, 32).astype(np.float32) * np.float32(0.5)
        if kind[g] in (1, 2, 3):
            W[g] = half * s
            W[g, 0] = 7 * s                              # the scale comes out as s
        if kind[g] == 2:
            W[g] = np.nextafter(W[g], np.float32(np.inf))
            W[g, 0] = 7 * s
        if kind[g] == 3:
            W[g] = W[g] * (1 + rng.integers(-3, 4, 32).astype(np.float32) * np.float32(2.0 ** -22))
            W[g, 0] = 7 * s
        if kind[g] == 4:
            W[g] *= np.float32(10.0 ** rng.integers(-8, -3))
        if kind[g] == 5:
            W[g] *= np.float32(10.0 ** rng.integers(4, 7))
        if kind[g] == 6:
            W[g] = 0
    W = W.reshape(N, K)
    q_ref, s_ref = oracle.pack_int4(W)
    q, s = nvq.pack_int4(torch.from_numpy(W).to(DEV))
    torch.cuda.synchronize()
    assert np.array_equal(s.cpu().numpy().view(np.uint16), s_ref)
    assert np.array_equal(q.cpu().numpy(), q_ref)


# ---- a2 activation quantisation ----------------------------------------------
@pytest.mark.parametrize("M,K,group", [(1, 32, 0), (1, 2048, 0), (3, 3072, 0), (1, 4096, 0),
                                       (2, 8192, 0), (1, 14336, 0), (32, 4096, 0),
                                       (1, 4096, 32), (4, 14336, 32), (2, 96, 32)])
def test_quant_act_bit_exact(M, K, group):
    say("quant", M, K, group)
    x = act(2000 + K + M, M, K)
    xq_r, xs_r, gs_r = oracle.quant_act_i8(u16(x), group)
    xq, xs, gs = nvq.quant_act_i8(x.to(DEV), group)
    torch.cuda.synchronize()
    assert np.array_equal(xq.cpu().numpy(), xq_r)
    assert np.array_equal(xs.cpu().numpy().view(np.uint32), xs_r.view(np.uint32))
    assert np.array_equal(gs.cpu().numpy(), gs_r)


# The kernels multiply by the scale's reciprocal and divide where that lies near a tie: rows full of
# ties and their neighbours, scales from the smallest to the largest, infinities and NaN (which the
# clamp turns into -127); one and two chunks per thread, and K beyond what one pass takes.
@pytest.mark.parametrize("group", [0, 32])
@pytest.mark.parametrize("K", [64, 8192, 8224, 16416])
def test_quant_act_codes_are_those_of_the_division(K, group):
    say("quant by reciprocal", K, group)
    rng = np.random.default_rng(K)
    amax = np.array([127.0, 254.0, 1.0, 3.0, 2.0 ** -90, 2.0 ** -99, 2.0 ** -110, 2.0 ** -130, 3e38, 5.1, 77.0, 0.3,
                     127.0, 127.0, 9.0, 0.0], dtype=np.float32)
    half = (rng.integers(-254, 255, (16, K)) / 2).astype(np.float32)  # in units of the scale
    x = half * (amax / np.float32(127.0))[:, None]
    x[:, ::32] = amax[:, None]
    xb = torch.from_numpy(x).to(torch.bfloat16)
    xb[12, 5::64] = float("inf")
    xb[13, 7::64] = float("-inf")
    xb[14, 9::64] = float("nan")
    f = xb.float().numpy().reshape(16, -1, 32 if group else K)
    with np.errstate(all="ignore"):
        s = np.fmax.reduce(np.abs(f), axis=2) / np.float32(127.0)
        q = np.fmin(np.fmax(np.rint(f / s[:, :, None]), np.float32(-127)), np.float32(127))
    q[s == 0] = 0
    q = q.reshape(16, K).astype(np.int8)
    xq, xs, gs = nvq.quant_act_i8(xb.to(DEV), group)
    torch.cuda.synchronize()
    assert np.array_equal(xs.cpu().numpy().reshape(s.shape).view(np.uint32), s.view(np.uint32))
    assert np.array_equal(xq.cpu().numpy(), q)
    assert np.array_equal(gs.cpu().numpy(), q.reshape(16, K // 32, 32).sum(2, dtype=np.int32))


def test_quant_act_edge_values():
    say("quant edge")
    x = torch.zeros(3, 64)
    x[1, :11] = torch.tensor([127.0, 0.5, 1.5, 2.5, -127.0, 3.5, -0.5, -1.5, -2.5, 126.5, 125.5])
    x[2, 40] = -3.0
    xb = x.to(torch.bfloat16)
    for group in (0, 32):
        xq_r, xs_r, gs_r = oracle.quant_act_i8(u16(xb), group)
        xq, xs, gs = nvq.quant_act_i8(xb.to(DEV), group)
        torch.cuda.synchronize()
        assert np.array_equal(xq.cpu().numpy(), xq_r)
        assert np.array_equal(xs.cpu().numpy(), xs_r)
        assert np.array_equal(gs.cpu().numpy(), gs_r)
    assert xq_r[1, :11].tolist() == [127, 0, 2, 2, -127, 4, 0, -2, -2, 126, 126]


# ---- a3 W4A8 -------------------------------------------------------------------
W4A8_CASES = [
    # N, K, M, act_group: every lane/row decomposition of the batch-1 kernel, ragged row
    # tails, more rows than one grid pass, and a wave per row (one token and K > 16384; two or
    # three tokens and few rows)
    (3, 32, 1, 0), (37, 1024, 1, 0), (70, 2048, 1, 0), (45, 2080, 1, 0), (29, 3072, 1, 0),
    (61, 4096, 1, 0), (19, 6144, 1, 0), (23, 8192, 1, 0), (11, 10240, 1, 0), (9, 12288, 1, 0),
    (13, 14336, 1, 0), (7, 16384, 1, 0), (5, 16416, 1, 0),
    (20011, 2048, 1, 0), (9003, 4096, 1, 0), (2501, 14336, 1, 0), (3000, 3072, 1, 0),
    (33, 4096, 1, 32), (21, 14336, 1, 32), (18, 3072, 1, 32),
    (40, 4096, 2, 0), (40, 4096, 4, 0), (17, 3072, 5, 0), (24, 14336, 8, 0), (12, 2048, 32, 0),
    (20, 4096, 3, 32),
    # matrix-core kernel (2 <= M <= 32, K % 128 == 0): one and two token tiles, ragged row
    # and token tails, fewer K columns than waves, 1 / 2 / 4 row tiles per workgroup
    (5, 128, 2, 0), (100, 4096, 16, 0), (70, 3072, 17, 0), (33, 14336, 32, 0), (16, 512, 9, 0),
    (16400, 2048, 8, 0), (33000, 1024, 24, 0),
]


@pytest.mark.parametrize("N,K,M,group", W4A8_CASES)
def test_gemv_w4a8_acc_bit_exact_and_output(N, K, M, group):
    say("w4a8", N, K, M, group)
    _, q, s = packed(3000 + N, N, K)
    x = act(3100 + K, M, K)
    xq_r, xs_r, gs_r = oracle.quant_act_i8(u16(x), group)
    y_r, acc_r = oracle.gemv_w4a8(q, s, xq_r, xs_r, group, want_acc=True)
    qd, sd = to_dev_packed(q, s)
    xq, xs, gs = nvq.quant_act_i8(x.to(DEV), group)
    y, acc = nvq.gemv_w4a8(qd, sd, xq, xs, gs, group, want_acc=True)
    y2 = nvq.gemv_w4a8(qd, sd, xq, xs, gs, group)            # the non-debug kernel
    torch.cuda.synchronize()
    assert np.array_equal(acc.cpu().numpy(), acc_r)
    assert np_ref.rel_l2(y.cpu().numpy(), y_r) < TOL
    assert torch.equal(y, y2)
    assert np_ref.rel_l2(y.cpu().numpy(), y_r) < 1e-5        # what fp32 accumulation gives


# Every significand of a value under every significand of the maximum, down to quotients that round to
# zero: the codes of the division.
@pytest.mark.parametrize("group", [0, 32])
@pytest.mark.parametrize("first", [0, 32, 64, 96])
def test_quant_act_every_pair_of_significands(first, group):
    say("quant significands", first, group)
    sig = (1 + np.arange(128, dtype=np.float32) / 128)
    x = np.zeros((32, 128 * 10 // 31 + 1, 32), np.float32)
    vals = np.concatenate([sig * np.float32(2.0 ** -e) for e in range(10)])
    vals = np.resize(vals, x.shape[1] * 31).reshape(x.shape[1], 31)
    x[:, :, 1:] = vals * np.where(np.arange(31) % 2, -1, 1).astype(np.float32)
    amax = sig[first:first + 32, None] * np.float32(2)  # above every value
    x[:, :, 0] = amax
    s = amax / np.float32(127)
    want = np.rint(x / s[:, :, None]).astype(np.int8).reshape(32, -1)
    xb = torch.from_numpy(x.reshape(32, -1)).to(torch.bfloat16)
    assert np.array_equal(xb.float().numpy(), x.reshape(32, -1))
    xq, xs, gs = nvq.quant_act_i8(xb.to(DEV), group)
    torch.cuda.synchronize()
    assert np.array_equal(xq.cpu().numpy(), want)
    assert bool((xs.cpu().reshape(32, -1) == torch.from_numpy(s)).all())
    assert np.array_equal(gs.cpu().numpy(), want.reshape(32, -1, 32).sum(2, dtype=np.int32))


# The calls with an output given go through csrc/binding.cpp where everything is as expected: the same
# bits as through ctypes, the same stream, and the same errors for what is not.
def test_calls_without_ctypes_equal_those_through_it(monkeypatch):
    M, N, K = 3, 70, 256
    _, q, s = packed(3050, N, K)
    qd, sd = to_dev_packed(q, s)
    x = act(3051, M, K).to(DEV)
    codes = [torch.empty_like(t) for t in nvq.quant_act_i8(x)]
    fast, served = nvq._calls, []

    class Counting:
        def __getattr__(self, name):
            def call(*args):
                status = getattr(fast, name)(*args)
                served.append((name, status))
                return status
            return call

    def outputs():
        ys = [torch.zeros((M, N), dtype=d, device=DEV) for d in (torch.float32, torch.bfloat16) for _ in range(3)]
        xq, xs, gs = nvq.quant_act_i8(x, 0, out=[t.zero_() for t in codes])
        for i in (0, 3):
            assert nvq.gemv_w4a16(qd, sd, x, out=ys[i]) is ys[i]
            assert nvq.gemv_w4a8(qd, sd, xq, xs, gs, out=ys[i + 1]) is ys[i + 1]
            assert nvq.gemm_w4a16(qd, sd, x, out=ys[i + 2]) is ys[i + 2]
        torch.cuda.synchronize()
        return [t.clone() for t in codes] + ys

    monkeypatch.setattr(nvq, "_calls", Counting())
    a = outputs()
    assert len(served) == 7 and all(status == 0 for _, status in served)
    monkeypatch.setattr(nvq, "_calls", None)
    b = outputs()
    assert all(torch.equal(u, v) for u, v in zip(a, b))
    # refused alike: types, strides, shapes, devices, what the library refuses, other numbers of tokens
    y = torch.zeros((M, N), device=DEV)
    xq, xs, gs = codes
    wrong = [lambda: nvq.gemv_w4a16(qd, sd, x.float(), out=y), lambda: nvq.gemv_w4a16(qd, sd, x[:, :128], out=y),
             lambda: nvq.gemv_w4a16(qd.cpu(), sd, x, out=y), lambda: nvq.gemv_w4a16(qd, sd[:, :4], x, out=y),
             lambda: nvq.gemv_w4a16(qd, sd, x, out=y.to(torch.float16)), lambda: nvq.gemm_w4a16(qd, sd, x, out=y.t()),
             lambda: nvq.gemv_w4a8(qd, sd, xq, xs, gs, 16, out=y), lambda: nvq.gemv_w4a8(qd, sd, xq.float(), xs, gs, out=y),
             lambda: nvq.quant_act_i8(x, 7, out=codes), lambda: nvq.quant_act_i8(x[0], 0, out=codes),
             lambda: nvq.gemv_w4a16(qd, sd, x.repeat(11, 1), out=torch.zeros((33, N), device=DEV))]
    for i, call in enumerate(wrong):
        said = []
        for calls in (fast, None):
            monkeypatch.setattr(nvq, "_calls", calls)
            with pytest.raises((ValueError, nvq.NvqError)) as e:
                call()
            said.append((type(e.value), str(e.value)))
        assert said[0] == said[1], i
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        assert fast.stream_handle() == side.cuda_stream == nvq._stream()
    assert fast.stream_handle() == nvq._stream()


# Outputs and scales that are too small are refused both ways, and nothing is written; larger ones, and
# code sums that more than three tokens do not read, are taken.
def test_calls_look_at_the_sizes_of_outputs_and_scales(monkeypatch):
    M, N, K = 4, 70, 256
    _, q, s = packed(3060, N, K)
    qd, sd = to_dev_packed(q, s)
    x = act(3061, M, K).to(DEV)
    codes = {g: nvq.quant_act_i8(x, g) for g in (0, 32)}
    y = torch.full((M * N + 64,), 7.0, device=DEV)
    few = y[:M * N - 1]
    fast = nvq._calls
    xq, xs, gs = codes[32]
    kept = [torch.full_like(t, 3) for t in (xq, xs, gs)]
    wrong = [lambda: nvq.gemv_w4a16(qd, sd, x, out=few), lambda: nvq.gemm_w4a16(qd, sd, x, out=few),
             lambda: nvq.gemv_w4a8(qd, sd, xq, xs, gs, 32, out=few),
             lambda: nvq.gemv_w4a8(qd, sd, xq, codes[0][1], gs, 32, out=y),
             lambda: nvq.gemv_w4a8(qd, sd, xq[:1], xs[:1], gs[:1, :7].contiguous(), 32, out=y),
             lambda: nvq.quant_act_i8(x, 32, out=[kept[0][1:], kept[1], kept[2]]),
             lambda: nvq.quant_act_i8(x, 32, out=[kept[0], kept[1][1:], kept[2]]),
             lambda: nvq.quant_act_i8(x, 0, out=[kept[0], kept[1], kept[2][1:]]),
             lambda: nvq.quant_act_i8(x, 0, out=[kept[0].t(), kept[1], kept[2]])]
    for i, call in enumerate(wrong):
        for calls in (fast, None):
            monkeypatch.setattr(nvq, "_calls", calls)
            with pytest.raises(ValueError):
                call()
    torch.cuda.synchronize()
    assert bool((y == 7).all()) and all(bool((t == 3).all()) for t in kept)
    want = nvq.gemv_w4a8(qd, sd, xq, xs, gs, 32)
    for calls in (fast, None):
        monkeypatch.setattr(nvq, "_calls", calls)
        y.fill_(7.0)
        assert nvq.gemv_w4a8(qd, sd, xq, xs, gs[:1], 32, out=y) is y
        torch.cuda.synchronize()
        assert torch.equal(y[:M * N].view(M, N), want) and bool((y[M * N:] == 7).all())


# One token: rows per tile go with the rows of the call (one, two, and four and eight with a single
# group per lane; teams of 64 and of 32 lanes, which a device of 256 compute units has 3072 and 6144
# of).  A row's bits are those of a short call, on both sides of every step and past the last one;
# tolerance against the oracle as above.
@pytest.mark.parametrize("N,K", [(3072, 64), (3073, 2048), (6145, 160), (12289, 96), (24581, 64), (6145, 1024),
                                 (24577, 1024), (49160, 1024), (3073, 4096), (7001, 2080), (6145, 3072),
                                 (3075, 6176), (3073, 8192), (3100, 10240)])
def test_one_token_rows_do_not_depend_on_the_tile(N, K):
    say("one token, rows per tile", N, K)
    rng = np.random.default_rng(3500 + N + K)
    q = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)
    s = rng.integers(0x1400, 0x2c00, (N, K // 32)).astype(np.uint16)
    pick = np.unique(np.concatenate([[0, 1, 7, 8, 3071, N - 9, N - 2, N - 1], rng.integers(0, N, 24)]))
    pick = pick[pick < N]
    xh = act(3600 + K, 1, K)
    (qd, sd), (qs, ss) = to_dev_packed(q, s), to_dev_packed(q[pick], s[pick])
    y = nvq.gemv_w4a16(qd, sd, xh.to(DEV))[:, pick]
    few = nvq.gemv_w4a16(qs, ss, xh.to(DEV))
    torch.cuda.synchronize()
    assert torch.equal(y, few)
    assert np_ref.rel_l2(y.cpu().numpy(), oracle.gemv_w4a16(q[pick], s[pick], u16(xh))) < 1e-5
    for group in (0, 32):
        xq, xs, gs = oracle.quant_act_i8(u16(xh), group)
        xqd, xsd, gsd = nvq.quant_act_i8(xh.to(DEV), group)
        y, acc = nvq.gemv_w4a8(qd, sd, xqd, xsd, gsd, group, want_acc=True)
        few = nvq.gemv_w4a8(qs, ss, xqd, xsd, gsd, group)
        again = nvq.gemv_w4a8(qd, sd, xqd, xsd, gsd, group)
        torch.cuda.synchronize()
        want, acc_ref = oracle.gemv_w4a8(q[pick], s[pick], xq, xs, group, want_acc=True)
        assert torch.equal(y[:, pick], few) and torch.equal(y, again)
        assert np.array_equal(acc[:, pick].cpu().numpy(), acc_ref)
        assert np_ref.rel_l2(few.cpu().numpy(), want) < 1e-5


# The small-batch kernel behind the single calls: tokens at the edges of its three sizes, rows at
# the edges of its tiles (16 rows; 32 from 12,288 rows on), K from one group on (fewer blocks of
# eight groups than waves, blocks that end early by one to seven groups, odd numbers of groups),
# scales aligned to 16, 4 and 2 bytes, K beyond 16384 with one token.  Tolerance: fp32 sums of
# products that are exact or, with a scale per group, rounded twice.
@pytest.mark.parametrize("M,N,K,off", [(2, 1, 32, 0), (8, 17, 256, 0), (9, 33, 288, 0), (16, 15, 448, 2),
                                       (17, 48, 2112, 0), (32, 100, 4096, 1), (5, 12301, 512, 0),
                                       (20, 12289, 352, 0), (32, 12320, 256, 2), (3, 70, 2720, 0),
                                       (1, 40, 16416, 0)])
def test_small_batch_kernel_edges(M, N, K, off):
    say("slice", M, N, K, off)
    _, q, s = packed(3300 + N, N, K)
    xh = act(3400 + K, M, K)
    qd, sd = to_dev_packed(q, s)
    if off:
        buf = torch.zeros(sd.numel() + off, dtype=sd.dtype, device=DEV)
        buf[off:] = sd.flatten()
        sd = buf[off:].view(sd.shape)
    y = nvq.gemv_w4a16(qd, sd, xh.to(DEV))
    yb = nvq.gemv_w4a16(qd, sd, xh.to(DEV), out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    assert np_ref.rel_l2(y.cpu().numpy(), oracle.gemv_w4a16(q, s, u16(xh))) < 1e-5
    assert torch.equal(yb, y.to(torch.bfloat16))
    for group in (0, 32):
        xq, xs, gs = oracle.quant_act_i8(u16(xh), group)
        want = oracle.gemv_w4a8(q, s, xq, xs, group)
        xqd, xsd, gsd = nvq.quant_act_i8(xh.to(DEV), group)
        y = nvq.gemv_w4a8(qd, sd, xqd, xsd, gsd, group)
        torch.cuda.synchronize()
        err = np_ref.rel_l2(y.cpu().numpy(), want)
        say("  rel l2", group, err)
        assert err < 1e-5


# The order of the additions, which decides the last bits, is that of the call and not of the
# kernel's tiling: eight or sixteen chains of columns (K % 128 == 0, scales aligned to 8 bytes, a
# scale per token), or sixty-four of groups.  Rows and tokens that reach each tiling (16 and 32
# rows per workgroup, up to 8, 16 and 32 tokens, more and fewer row tiles than compute units), K
# whose last block of eight groups ends early, K beyond 16384, and the calls of up to three tokens
# that take a wave per row, with their neighbours.
@pytest.mark.parametrize("M,N,K,off", [(3, 48, 4096, 0), (12, 33, 14336, 0), (20, 48, 8320, 0), (9, 4200, 4096, 0),
                                       (32, 4200, 4224, 0), (8, 40, 3072, 0), (16, 40, 2176, 0), (17, 40, 3072, 0),
                                       (2, 8300, 4096, 0), (5, 16400, 1024, 0), (16, 16400, 640, 0),
                                       (24, 16400, 512, 0), (6, 40, 4096, 1), (16, 40, 2720, 0), (25, 40, 2720, 0),
                                       (4, 16400, 352, 0), (1, 40, 16416, 0), (30, 17, 65536, 0),
                                       (1, 4097, 16416, 0), (1, 8300, 16416, 0), (2, 1024, 2720, 0), (2, 1025, 2720, 0), (2, 2049, 2720, 0),
                                       (2, 6144, 1056, 0), (2, 6145, 1056, 0), (2, 2049, 8224, 1), (2, 2049, 16416, 0),
                                       (3, 682, 1056, 1), (9, 2000, 2016, 0), (16, 2000, 65504, 0)])
def test_multi_token_sums_are_added_in_the_stated_order(M, N, K, off):
    """Bit for bit against the same additions on the CPU.  W4A8: the block sums are integers.  W4A16
    on small whole inputs: a group's products and their sums are exact whatever their order."""
    say("order of sums", M, N, K, off)
    rng = np.random.default_rng(N + K)
    q = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)
    s = rng.integers(0x1400, 0x2c00, (N, K // 32)).astype(np.uint16)
    qd, sd = to_dev_packed(q, s)
    if off:
        buf = torch.zeros(sd.numel() + off, dtype=sd.dtype, device=DEV)
        buf[off:] = sd.flatten()
        sd = buf[off:].view(sd.shape)
    x = act(3600 + K, M, K)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    chains = 64
    if M > 1 and K % 128 == 0 and not off:
        chains = 16 if K >= 4096 and (N + 15) // 16 <= 2 * cus else 8
    rows = np.unique(np.concatenate([np.arange(min(N, 17)), [N - 1], rng.integers(0, N, 16)]))
    sw = np_ref.half_bits_to_f64(s[rows])

    def check(y, want, what):
        got = y.cpu().numpy()[:, rows]
        assert np.array_equal(got, want), (what, int((got != want).sum()), np_ref.rel_l2(got, want))

    for group in (0, 32):
        xq, xs, gs = nvq.quant_act_i8(x.to(DEV), group)
        y, dump = nvq.gemv_w4a8(qd, sd, xq, xs, gs, group, want_acc=True)
        y2 = nvq.gemv_w4a8(qd, sd, xq, xs, gs, group)
        torch.cuda.synchronize()
        _, acc = oracle.gemv_w4a8(q[rows], s[rows], xq.cpu().numpy(), xs.cpu().numpy(), group, want_acc=True)
        assert np.array_equal(dump.cpu().numpy()[:, rows], acc)
        want = np_ref.sums_in_order(acc, sw, 64 if group else chains, xs.cpu().numpy(), group == 32)
        check(y2, want, ("w4a8", group))
        check(y, want, ("w4a8 with the accumulators", group))
    xi = rng.integers(-99, 100, (M, K)).astype(np.int8)
    _, acc = oracle.gemv_w4a8(q[rows], s[rows], xi, np.ones(M, np.float32), 0, want_acc=True)
    y = nvq.gemv_w4a16(qd, sd, torch.from_numpy(xi).to(torch.bfloat16).to(DEV))
    torch.cuda.synchronize()
    check(y, np_ref.sums_in_order(acc, sw, chains), "w4a16")


# A walk whose last block ends after one to seven groups, in the first and in the second of the two
# blocks that are in flight, with up to 8, 16 and 32 tokens: a product used behind the branch that
# ends the block must have been written (with three groups of four it was not, in most runs).
@pytest.mark.parametrize("M", [8, 16, 32])
@pytest.mark.parametrize("groups", [63, 127, 57, 122, 59, 124, 61])
def test_a_last_block_that_ends_early_gives_the_same_bits_every_time(M, groups):
    say("early end", M, groups)
    N, K = 2000, 32 * groups
    _, q, s = packed(3700 + groups, N, K)
    qd, sd = to_dev_packed(q, s)
    x = act(3800 + K, M, K).to(DEV)
    a8, a8g = nvq.quant_act_i8(x, 0), nvq.quant_act_i8(x, 32)
    for what, call in (("w4a16", lambda out: nvq.gemv_w4a16(qd, sd, x, out=out)),
                       ("w4a8", lambda out: nvq.gemv_w4a8(qd, sd, *a8, 0, out=out)),
                       ("w4a8 per group", lambda out: nvq.gemv_w4a8(qd, sd, *a8g, 32, out=out))):
        ys = torch.zeros((40, M, N), device=DEV)
        for y in ys:
            call(y)
        torch.cuda.synchronize()
        assert int((ys != ys[0]).sum()) == 0, what


@pytest.mark.parametrize("M", [1, 20])
def test_gemv_w4a8_accepts_every_nibble_and_extreme_codes(M):
    say("w4a8 extremes", M)
    rng = np.random.default_rng(17)
    N, K = 50, 4096
    q = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)      # includes nibble 0 = code -8
    q[0, :] = 0x00
    q[1, :] = 0xFF
    s = rng.integers(0x1400, 0x2c00, (N, K // 32)).astype(np.uint16)
    xq = rng.integers(-127, 128, (M, K)).astype(np.int8)
    xq[0, :64] = -127
    xq[M - 1, 64:128] = 127
    xs = np.linspace(0.03125, 0.0625, M).astype(np.float32)
    gs = xq.astype(np.int32).reshape(M, K // 32, 32).sum(axis=2).astype(np.int32)
    y_r, acc_r = oracle.gemv_w4a8(q, s, xq, xs, want_acc=True)
    assert acc_r.max() == 32512
    qd, sd = to_dev_packed(q, s)
    y, acc = nvq.gemv_w4a8(qd, sd, torch.from_numpy(xq).to(DEV), torch.from_numpy(xs).to(DEV),
                           torch.from_numpy(gs).to(DEV), want_acc=True)
    torch.cuda.synchronize()
    assert np.array_equal(acc.cpu().numpy(), acc_r)
    assert np_ref.rel_l2(y.cpu().numpy(), y_r) < TOL


def test_batched_w4a8_rows_equal_the_single_token_results():
    say("w4a8 batch rows")
    # the matrix-core kernel and the batch-1 kernel compute the same int32 accumulators
    N, K, M = 48, 4096, 19
    _, q, s = packed(3500, N, K)
    x = act(3501, M, K).to(DEV)
    qd, sd = to_dev_packed(q, s)
    xq, xs, gs = nvq.quant_act_i8(x, 0)
    y, acc = nvq.gemv_w4a8(qd, sd, xq, xs, gs, 0, want_acc=True)
    for m in (0, 7, 16, 18):
        y1, acc1 = nvq.gemv_w4a8(qd, sd, xq[m:m + 1].contiguous(), xs[m:m + 1].contiguous(),
                                 gs[m:m + 1].contiguous(), 0, want_acc=True)
        torch.cuda.synchronize()
        assert torch.equal(acc[m], acc1[0])
        assert np_ref.rel_l2(y[m].cpu().numpy(), y1[0].cpu().numpy()) < 1e-5


# ---- a4 W4A16 ------------------------------------------------------------------
W4A16_CASES = [(n, k, m) for (n, k, m, g) in W4A8_CASES if g == 0]


@pytest.mark.parametrize("N,K,M", W4A16_CASES)
def test_gemv_w4a16_output(N, K, M):
    say("w4a16", N, K, M)
    _, q, s = packed(4000 + N, N, K)
    x = act(4100 + K, M, K)
    y_r = oracle.gemv_w4a16(q, s, u16(x))
    qd, sd = to_dev_packed(q, s)
    y = nvq.gemv_w4a16(qd, sd, x.to(DEV))
    torch.cuda.synchronize()
    err = np_ref.rel_l2(y.cpu().numpy(), y_r)
    say("  rel_l2", err)
    assert err < TOL and err < 1e-5
    # per output (a norm over the whole output would let one row lose a whole group
    # unnoticed): every product code * scale * x is exact in fp32, so the GPU differs from
    # the float64 sum only by the roundings of its partial sums.  The kernel adds 136 to
    # every code and takes 136 * sum(x) away again, so a partial sum inside a group is at
    # most 279 * sum_j |x_j|; a few roundings of 2^-24 of that per group:
    sw = np_ref.half_bits_to_f64(s)                                               # [N][G]
    xa = np.abs(np_ref.bf16_bits_to_f64(u16(x))).reshape(M, K // 32, 32).sum(axis=2)   # [M][G]
    bound = 4 * 279 * 2.0 ** -24 * (xa @ sw.T)                                    # [M][N]
    diff = np.abs(y.cpu().numpy().astype(np.float64) - y_r)
    assert (diff <= bound + 1e-30).all(), float((diff / (bound + 1e-30)).max())


@pytest.mark.parametrize("M", [1, 20])
def test_gemv_w4a16_accepts_every_nibble(M):
    say("w4a16 nibbles", M)
    rng = np.random.default_rng(18)
    N, K = 40, 3072
    q = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)
    s = rng.integers(0x1400, 0x2c00, (N, K // 32)).astype(np.uint16)
    x = act(77, M, K)
    y_r = oracle.gemv_w4a16(q, s, u16(x))
    qd, sd = to_dev_packed(q, s)
    y = nvq.gemv_w4a16(qd, sd, x.to(DEV))
    torch.cuda.synchronize()
    assert np_ref.rel_l2(y.cpu().numpy(), y_r) < TOL


@pytest.mark.parametrize("prec", [nvq.W4A8, nvq.W4A16])
def test_bf16_output_is_the_rounded_fp32_output(prec):
    say("bf16 out", prec)
    N, K = 100, 4096
    _, q, s = packed(5000, N, K)
    x = act(5001, 1, K).to(DEV)
    qd, sd = to_dev_packed(q, s)
    if prec == nvq.W4A16:
        y32 = nvq.gemv_w4a16(qd, sd, x)
        y16 = nvq.gemv_w4a16(qd, sd, x, out_dtype=torch.bfloat16)
    else:
        xq, xs, gs = nvq.quant_act_i8(x)
        y32 = nvq.gemv_w4a8(qd, sd, xq, xs, gs)
        y16 = nvq.gemv_w4a8(qd, sd, xq, xs, gs, out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    assert torch.equal(y16, y32.to(torch.bfloat16))


# ---- a5 walker -------------------------------------------------------------------
def tiny_model_entries(M, seed=6000, hidden=256, kv=64, ffn=704, blocks=3, bits=(0, 1, 0)):
    """Three transformer-block-shaped groups of seven linears; K = 256 and 704
    (22 groups: a ragged lane tail)."""
    entries, host = [], []
    for b in range(blocks):
        xs = [act(seed + 10 * b + p, M, k, True) for p, k in enumerate([hidden, hidden, hidden, ffn])]
        shapes = [(hidden, hidden, 0), (kv, hidden, 0), (kv, hidden, 0), (hidden, hidden, 1),
                  (ffn, hidden, 2), (ffn, hidden, 2), (hidden, ffn, 3)]
        for slot, (N, K, p) in enumerate(shapes):
            _, q, s = packed(seed + 100 * b + slot, N, K)
            host.append(dict(qweight=q, scales=s, x=u16(xs[p]), precision=bits[b]))
            qd, sd = to_dev_packed(q, s)
            entries.append(dict(qweight=qd, scales=sd, x=None, xkey=(b, p), xhost=xs[p],
                                y=torch.zeros((M, N), dtype=torch.float32, device=DEV),
                                precision=bits[b]))
    # entries of one phase must share one device buffer (the walker keys on the pointer)
    bufs = {}
    for e in entries:
        if e["xkey"] not in bufs:
            bufs[e["xkey"]] = e["xhost"].to(DEV)
        e["x"] = bufs[e["xkey"]]
    return entries, host


@pytest.mark.parametrize("M,group", [(1, 0), (1, 32), (3, 0)])
def test_decode_linears_matches_oracle_walker_and_standalone_calls(M, group):
    say("walker", M, group)
    entries, host = tiny_model_entries(M)
    ys_ref = oracle.decode_linears(host, M, group)
    nvq.decode_linears(entries, M, group)
    torch.cuda.synchronize()
    for e, h, y_r in zip(entries, host, ys_ref):
        got = e["y"].cpu().numpy()
        assert np_ref.rel_l2(got, y_r) < TOL
        # same result (up to fp32 summation order) as the standalone entry point
        if e["precision"] == nvq.W4A16:
            alone = nvq.gemv_w4a16(e["qweight"], e["scales"], e["x"])
            other = None
        else:
            xq, xs, gs = nvq.quant_act_i8(e["x"], group)
            alone = nvq.gemv_w4a8(e["qweight"], e["scales"], xq, xs, gs, group)
            other = nvq.gemv_w4a16(e["qweight"], e["scales"], e["x"])
        assert np_ref.rel_l2(e["y"].cpu().numpy(), alone.cpu().numpy()) < 1e-5
        if other is not None:                      # the precision bit was respected
            assert np_ref.rel_l2(e["y"].cpu().numpy(), other.cpu().numpy()) > 1e-4


def test_decode_linears_runs_in_order_on_chained_buffers():
    say("walker chain")
    # entry 1 reads what entry 0 wrote (bf16 output feeding the next input)
    M, K0, N0, N1 = 1, 2048, 4096, 512
    _, q0, s0 = packed(7000, N0, K0)
    W1 = synth.make_weight(7001, N1, N0)
    q1, s1 = oracle.pack_int4(W1.numpy())
    x0 = act(7002, M, K0)
    q0d, s0d = to_dev_packed(q0, s0)
    q1d, s1d = to_dev_packed(q1, s1)
    mid = torch.zeros((M, N0), dtype=torch.bfloat16, device=DEV)
    out = torch.zeros((M, N1), dtype=torch.float32, device=DEV)
    for p0, p1 in [(1, 0), (0, 1)]:
        mid.zero_(); out.zero_()
        nvq.decode_linears([dict(qweight=q0d, scales=s0d, x=x0.to(DEV), y=mid, precision=p0),
                            dict(qweight=q1d, scales=s1d, x=mid, y=out, precision=p1)], M)
        torch.cuda.synchronize()
        # oracle on the GPU's own intermediate (bf16 rounding of entry 0 is checked above)
        mid_h = u16(mid)
        ys = oracle.decode_linears([dict(qweight=q1, scales=s1, x=mid_h, precision=p1)], M)
        assert np_ref.rel_l2(out.cpu().numpy(), ys[0]) < TOL
        y0 = oracle.decode_linears([dict(qweight=q0, scales=s0, x=u16(x0), precision=p0)], M)[0]
        assert np_ref.rel_l2(mid.float().cpu().numpy(), y0) < 4e-3   # bf16 output rounding


def test_measurement_helpers():
    say("stream helpers")
    src = torch.randint(0, 255, (1 << 20,), dtype=torch.uint8, device=DEV)
    dst = torch.zeros_like(src)
    sink = torch.zeros(1, dtype=torch.int64, device=DEV)
    nvq.stream_copy(dst, src)
    nvq.stream_read(src, sink)
    torch.cuda.synchronize()
    assert torch.equal(dst, src)
    w = src.cpu().numpy().view(np.uint32).reshape(-1, 4)
    want = int((w[:, 0] ^ w[:, 1] ^ w[:, 2] ^ w[:, 3]).astype(np.uint64).sum())
    # per-lane sums wrap at 32 bits before the 64-bit atomic; compare modulo 2^32
    assert int(sink.item()) % (1 << 32) == want % (1 << 32)


# ---- persistent streaming walker (batch 1) ------------------------------------------
def model_entries(shapes_per_block, bits, M=1, seed=8000):
    """shapes_per_block: list of (N, K, phase-in-block); one x buffer per (block, phase)."""
    entries, host = [], []
    for b, bit in enumerate(bits):
        bufs = {}
        for slot, (N, K, p) in enumerate(shapes_per_block):
            if p not in bufs:
                xh = act(seed + 50 * b + p, M, K)
                bufs[p] = (xh, xh.to(DEV))
            _, q, s = packed(seed + 100 * b + slot, N, K)
            qd, sd = to_dev_packed(q, s)
            entries.append(dict(qweight=qd, scales=sd, x=bufs[p][1], precision=bit,
                                y=torch.zeros((M, N), dtype=torch.float32, device=DEV)))
            host.append(dict(qweight=q, scales=s, x=u16(bufs[p][0]), precision=bit))
    return entries, host


STREAM_MODELS = {
    # llama-1b block shapes, two blocks, one of each precision
    "1b": ([(2048, 2048, 0), (512, 2048, 0), (512, 2048, 0), (2048, 2048, 1),
            (8192, 2048, 2), (8192, 2048, 2), (2048, 8192, 3)], (0, 1)),
    # ragged: rows that do not divide over the waves, K with a partial last chunk (G = 66, 98)
    "ragged": ([(1000, 2112, 0), (37, 2112, 0), (3, 2112, 1), (2500, 3136, 2), (777, 3136, 2),
                (64, 14336, 3)], (1, 0, 0)),
    # 8b block shapes, one W4A8 block
    "8b": ([(4096, 4096, 0), (1024, 4096, 0), (1024, 4096, 0), (4096, 4096, 1),
            (14336, 4096, 2), (14336, 4096, 2), (4096, 14336, 3)], (0,)),
    "8b twice": ([(4096, 4096, 0), (1024, 4096, 0), (1024, 4096, 0), (4096, 4096, 1),
                  (14336, 4096, 2), (14336, 4096, 2), (4096, 14336, 3)], (0, 1)),
    # llama-3b block shapes (rows of 96 groups go to the waves in pairs), one block of
    # each precision; in the third, layers with an odd number of rows (no pairs there)
    "3b": ([(3072, 3072, 0), (1024, 3072, 0), (1024, 3072, 0), (3072, 3072, 1),
            (8192, 3072, 2), (8192, 3072, 2), (3072, 8192, 3)], (0, 1)),
    "3b odd": ([(3071, 3072, 0), (1024, 3072, 0), (8190, 3072, 1), (12294, 3072, 1),
                (2, 3072, 2)], (1, 0)),
}


@pytest.mark.parametrize("name,group,ordered", [("1b", 0, False), ("1b", 0, True),
                                                ("ragged", 0, False), ("ragged", 32, True),
                                                ("8b", 0, False), ("8b", 32, False),
                                                ("8b", 0, True),
                                                ("3b", 0, False), ("3b", 0, True),
                                                ("3b", 32, False), ("3b odd", 0, False)])
def test_streaming_plan_matches_oracle_on_repeated_runs(name, group, ordered):
    say("stream plan", name, group, ordered)
    shapes, bits = STREAM_MODELS[name]
    entries, host = model_entries(shapes, bits)
    ys_ref = oracle.decode_linears(host, 1, group)
    dl = nvq.DecodeList(entries, 1, group, ordered=ordered)
    info = dl.plan_info()
    say("  plan", info)
    assert info["streaming"], "batch-1 walk should use the persistent kernel"
    # independent buffers: no phase has to wait unless ordering is forced
    assert info["waits"] == (info["phases"] - 1 if ordered else 0)
    for rep in range(3):
        for e in entries:
            e["y"].zero_()
        dl.run_plan()
        assert not dl.plan_timed_out()
        for e, y_r in zip(entries, ys_ref):
            err = np_ref.rel_l2(e["y"].cpu().numpy(), y_r)
            assert err < TOL, (rep, err)
            assert err < 1e-5, (rep, err)
    dl.close()


@pytest.mark.parametrize("seed", range(4))
def test_streaming_plan_of_random_lists_matches_oracle(seed):
    """Random phases (1 to 3 layers on one input; rows from 1 to 9000; K with whole, ragged and
    one-and-a-half-chunk rows), both precisions, with and without forced ordering."""
    rng = np.random.default_rng(7300 + seed)
    entries, host = [], []
    for ph in range(int(rng.integers(4, 14))):
        K = int(rng.choice([96, 1024, 2048, 2112, 3072, 4096, 8192]))
        xh = act(7400 + 100 * seed + ph, 1, K)
        xd = xh.to(DEV)
        bit = int(rng.integers(0, 2))
        for k in range(int(rng.integers(1, 4))):
            N = int(rng.choice([1, 2, 7, 40, 96, 511, 1024, 3072, 4097, 9000]))
            _, q, s = packed(7500 + 1000 * seed + 10 * ph + k, N, K)
            qd, sd = to_dev_packed(q, s)
            entries.append(dict(qweight=qd, scales=sd, x=xd, precision=bit,
                                y=torch.zeros((1, N), dtype=torch.float32, device=DEV)))
            host.append(dict(qweight=q, scales=s, x=u16(xh), precision=bit))
    ordered = bool(seed & 1)
    say("stream plan, random list", seed, len(entries), "layers, ordered", ordered)
    ys_ref = oracle.decode_linears(host, 1, 0)
    dl = nvq.DecodeList(entries, 1, 0, ordered=ordered)
    assert dl.plan_info()["streaming"]
    for rep in range(2):
        for e in entries:
            e["y"].zero_()
        dl.run_plan()
        assert not dl.plan_timed_out()
        for i, (e, y_r) in enumerate(zip(entries, ys_ref)):
            err = np_ref.rel_l2(e["y"].cpu().numpy(), y_r)
            # (a handful of outputs can be small against their terms: the bar only)
            assert err < (1e-5 if y_r.size >= 96 else TOL), (rep, i, err)
    dl.close()


def test_streaming_plan_of_many_tiny_phases():
    """300 independent layers of 40 rows: nearly every wave has no rows in more than 255 phases
    in a row (the skip table's cap), a few work in one phase in a hundred."""
    say("stream plan, 300 tiny phases")
    entries, host = [], []
    for i in range(300):
        N, K = 40, 2048
        xh = act(9100 + i, 1, K)
        _, q, s = packed(9500 + i, N, K)
        qd, sd = to_dev_packed(q, s)
        entries.append(dict(qweight=qd, scales=sd, x=xh.to(DEV), precision=i % 2,
                            y=torch.zeros((1, N), dtype=torch.float32, device=DEV)))
        host.append(dict(qweight=q, scales=s, x=u16(xh), precision=i % 2))
    ys_ref = oracle.decode_linears(host, 1, 0)
    dl = nvq.DecodeList(entries, 1, 0)
    info = dl.plan_info()
    assert info["streaming"] and info["phases"] == 300 and info["waits"] == 0
    skips = nvq.plan_describe_skips([dl.arr[i] for i in range(dl.n)], 1,
                                    workgroups=torch.cuda.get_device_properties(0).multi_processor_count)
    assert skips.max() == 255 and skips.shape[0] % 13 == 0
    for rep in range(2):
        for e in entries:
            e["y"].zero_()
        dl.run_plan()
        assert not dl.plan_timed_out()
        for e, y_r in zip(entries, ys_ref):
            assert np_ref.rel_l2(e["y"].cpu().numpy(), y_r) < 1e-5
    dl.close()


def test_streaming_plan_orders_dependent_phases():
    say("stream chain")
    # four phases, each reading the bf16 output of the one before it
    dims = [2048, 4096, 1024, 6144, 512]
    hostW = [oracle.pack_int4(synth.make_weight(8800 + i, dims[i + 1], dims[i]).numpy())
             for i in range(4)]
    x0 = act(8899, 1, dims[0])
    bufs = [x0.to(DEV)] + [torch.zeros((1, d), dtype=torch.bfloat16, device=DEV) for d in dims[1:]]
    entries = []
    for i, (q, s) in enumerate(hostW):
        qd, sd = to_dev_packed(q, s)
        entries.append(dict(qweight=qd, scales=sd, x=bufs[i], y=bufs[i + 1], precision=i % 2))
    dl = nvq.DecodeList(entries, 1)
    info = dl.plan_info()
    assert info["streaming"] and info["waits"] == 3      # the analysis found the chain
    for rep in range(3):
        for b in bufs[1:]:
            b.zero_()
        dl.run_plan()
        assert not dl.plan_timed_out()
        # each stage against the oracle applied to the GPU's own previous stage
        for i, (q, s) in enumerate(hostW):
            y_r = oracle.decode_linears([dict(qweight=q, scales=s, x=u16(bufs[i]),
                                              precision=i % 2)], 1)[0]
            assert np_ref.rel_l2(bufs[i + 1].float().cpu().numpy(), y_r) < 4e-3, (rep, i)
    dl.close()


# Activation scales of the smallest and largest normal numbers: the results are those of ordinary scales times
# a power of two, to the bit (chains of columns, 16 and 8, and of groups; a scale per token and per group).  The
# weights' scales are large, so that sums at the lower end are far from the numbers with fewer bits.
@pytest.mark.parametrize("M", [2, 8, 13, 29])
@pytest.mark.parametrize("group", [0, 32])
@pytest.mark.parametrize("N,K", [(160, 4096), (20000, 1024), (100, 1312), (96, 2752)])
def test_w4a8_scales_of_any_size(M, group, N, K):
    say("w4a8, scales of any size", M, group, N, K)
    rng = np.random.default_rng(8900 + M + K)
    q = torch.from_numpy(rng.integers(0, 256, (N, K // 2), dtype=np.uint8)).to(DEV)
    s = torch.from_numpy(rng.integers(0x5400, 0x6c00, (N, K // 32)).astype(np.int16)).to(DEV)
    xq, xs, gs = nvq.quant_act_i8(act(8950 + M, M, K).to(DEV), group)
    xs = 1.0 + torch.rand(xs.shape, device=DEV, generator=torch.Generator(device=DEV).manual_seed(M))
    y = nvq.gemv_w4a8(q, s, xq, xs, gs, group)
    top = 126 - int(np.ceil(np.log2(y.abs().max().item())))
    for power in (-124, top):
        got = nvq.gemv_w4a8(q, s, xq, xs * 2.0 ** power, gs, group)
        assert got.isfinite().all() and torch.equal(got.double(), y.double() * 2.0 ** power), power


# ---- grouped small-batch walker (2..32 tokens on the matrix cores) -------------------
def kernels_of(dl, ordered=False):
    """Per batch of a plan that is issued in batches: what it runs on."""
    return nvq.plan_describe_kernels([dl.arr[i] for i in range(dl.n)], dl.M, ordered)


def bulk_layer(M, mbytes, K=2048, seed=8990):
    """A layer of that many MB with random codes, made on the device: what a list needs besides the
    layers under test to be worth the grid for 17 tokens and more.  (entry, rows to look at, host
    layer of those rows)"""
    N = int(mbytes * 1e6 / (0.5625 * K))
    g = torch.Generator(device=DEV).manual_seed(seed)
    q = torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device=DEV, generator=g)
    s = torch.randint(0x1400, 0x2c00, (N, K // 32), dtype=torch.int16, device=DEV, generator=g)
    x = act(seed, M, K)
    rows = torch.tensor([0, 31, 32, 127, 128, N // 3, N // 2, N - 33, N - 1])
    entry = dict(qweight=q, scales=s, x=x.to(DEV), precision=nvq.W4A8,
                 y=torch.zeros((M, N), dtype=torch.float32, device=DEV))
    host = dict(qweight=q[rows.to(DEV)].cpu().numpy(), scales=u16(s[rows.to(DEV)]), x=u16(x), precision=nvq.W4A8)
    return entry, rows, host


def check_bulk(bulk, M):
    entry, rows, host = bulk
    want = oracle.decode_linears([host], M, 0)[0]
    assert np_ref.rel_l2(entry["y"][:, rows.to(DEV)].cpu().numpy(), want) < 1e-5


# grid: whether the product runs as a persistent grid (every K of these models is a multiple of
# 512; from 17 tokens on the work has to be enough, otherwise it goes phase by phase)
@pytest.mark.parametrize("name,M,ordered,grid", [("1b", 5, False, True), ("1b", 20, True, False),
                                                 ("8b", 16, False, True), ("8b", 32, False, False),
                                                 ("8b twice", 32, False, True)])
def test_grouped_plan_matches_oracle_on_repeated_runs(name, M, ordered, grid):
    say("grouped plan", name, M, ordered)
    shapes, bits = STREAM_MODELS[name]
    entries, host = model_entries(shapes, bits, M=M, seed=8300)
    ys_ref = oracle.decode_linears(host, M, 0)
    dl = nvq.DecodeList(entries, M, 0, ordered=ordered)
    info = dl.plan_info()
    say("  plan", info)
    assert not info["streaming"]
    assert info["persistent_grouped"] == grid
    # "waits" counts the batch boundaries: independent buffers make one batch of all phases
    assert info["waits"] == (info["phases"] - 1 if ordered else 0)
    for rep in range(3):
        for e in entries:
            e["y"].zero_()
        dl.run_plan()
        torch.cuda.synchronize()
        assert not dl.plan_timed_out()
        for e, y_r in zip(entries, ys_ref):
            err = np_ref.rel_l2(e["y"].cpu().numpy(), y_r)
            assert err < TOL, (rep, err)
            assert err < 1e-5, (rep, err)
    # the one-call entry point takes the same path
    for e in entries:
        e["y"].zero_()
    nvq.decode_linears(entries, M, 0)
    torch.cuda.synchronize()
    for e, y_r in zip(entries, ys_ref):
        assert np_ref.rel_l2(e["y"].cpu().numpy(), y_r) < 1e-5
    dl.close()


# The persistent small-batch kernels (loader wave and LDS rings; shared activations and tickets) serve
# lists with every K a multiple of 512; these shapes exercise what
# their bookkeeping has to get right: row counts that end inside a unit of 32 rows and inside a
# 16-row tile, phases of several matrices whose boundaries fall inside a unit, a phase with fewer
# units than teams next to long ones (groups of units that cross phases of other K and precision),
# K from one step (512) to 28 steps, both precisions, and token counts from 2 to 32 (one or two
# token tiles).  The kernel with shared activations takes long lists only: with a large layer in
# the middle.
RING_SHAPES = [(1000, 1536, 0), (37, 1536, 0), (3, 1536, 1), (2500, 3072, 2), (777, 3072, 2),
               (64, 14336, 3), (48, 512, 4), (4100, 512, 4), (16, 1024, 5)]


@pytest.mark.parametrize("M,bits,kernel", [(2, (0, 1), "rings"), (7, (1, 0), "rings"), (16, (0, 1, 1), "rings"),
                                           (17, (0, 1), "rings"), (32, (1, 0), "rings"), (17, (0, 1), "rows"),
                                           (32, (1, 0), "rows")])
def test_ring_plan_matches_oracle(M, bits, kernel):
    say("ring plan", M, bits, kernel)
    entries, host = model_entries(RING_SHAPES, bits, M=M, seed=8600)
    ys_ref = oracle.decode_linears(host, M, 0)
    bulk = bulk_layer(M, 640) if kernel == "rows" else None
    dl = nvq.DecodeList(entries[:7] + [bulk[0]] + entries[7:] if bulk else entries, M, 0)
    info = dl.plan_info()
    say("  plan", info)
    assert info["grouped"] and info["persistent_grouped"] and kernels_of(dl) == [kernel]
    for rep in range(3):
        for e in entries:
            e["y"].zero_()
        dl.run_plan()
        torch.cuda.synchronize()
        assert not dl.plan_timed_out()
        for e, y_r in zip(entries, ys_ref):
            assert np_ref.rel_l2(e["y"].cpu().numpy(), y_r) < 1e-5, rep
        if bulk:
            check_bulk(bulk, M)
    dl.close()


def test_rows_plan_draws_tickets_and_replays():
    """More groups of units than workgroups fit the device, so that groups are drawn from the
    counters; captured in a graph and replayed with eager work in between, every replay equal to
    the eager run (bit for bit: a row's sums do not depend on who takes it)."""
    say("rows plan, tickets")
    M = 20
    entries, host = model_entries([(120001, 512, 0), (900, 512, 0), (33, 1536, 1), (70000, 512, 2)], (0, 1),
                                  M=M, seed=8650)
    rows = np.unique(np.concatenate([[0, 31, 32, 127, 128], np.random.default_rng(1).integers(0, 33, 8)]))
    dl = nvq.DecodeList(entries, M, 0)
    assert kernels_of(dl) == ["rows"]
    dl.run_plan()
    torch.cuda.synchronize()
    eager = [e["y"].clone() for e in entries]
    for e, h in zip(entries, host):
        N = e["y"].shape[1]
        pick = np.unique(np.concatenate([rows[rows < N], [N - 1, N // 2, N // 3]]))
        sub = dict(h, qweight=h["qweight"][pick], scales=h["scales"][pick])
        want = oracle.decode_linears([sub], M, 0)[0]
        assert np_ref.rel_l2(e["y"].cpu().numpy()[:, pick], want) < 1e-5
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        dl.run_plan()
    for rep in range(3):
        for e in entries:
            e["y"].zero_()
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(e["y"], w) for e, w in zip(entries, eager)), rep
    del g
    dl.close()


# The workgroups of a part take its phases by their K: one and two phases (as they stand), and several of
# rising K, divided by the cuts or smaller than a group of units.
@pytest.mark.parametrize("shapes,mbytes", [([], 300), ([(4999, 3072, 1)], 150),
                                           ([(40000, 512, 0), (30, 1024, 1), (129, 1536, 2), (7000, 2048, 3),
                                             (3, 2560, 4), (2500, 4096, 5)], 60)])
def test_rows_plan_results_do_not_depend_on_the_order_of_the_phases(shapes, mbytes):
    say("rows plan, order of the phases", shapes)
    M = 29
    bulk = bulk_layer(M, mbytes)
    entries, host = model_entries(shapes, (1, 0)[:max(1, len(shapes) // 3)], M=M, seed=8655)
    ran = []
    for turn in (1, -1):
        dl = nvq.DecodeList((entries[:3] + [bulk[0]] + entries[3:])[::turn], M, 0)
        assert kernels_of(dl) == ["rows"]
        dl.run_plan()
        torch.cuda.synchronize()
        check_bulk(bulk, M)
        ran.append([e["y"].clone() for e in entries + [bulk[0]]])
        dl.close()
        for e in entries:
            e["y"].zero_()
    assert all(torch.equal(a, b) for a, b in zip(*ran))
    rng = np.random.default_rng(3)
    for y, h in zip(ran[0], host):
        N = y.shape[1]
        pick = np.unique(np.concatenate([[0, N - 1, N // 2], rng.integers(0, N, 24)]))
        sub = dict(h, qweight=h["qweight"][pick], scales=h["scales"][pick])
        assert np_ref.rel_l2(y.cpu().numpy()[:, pick], oracle.decode_linears([sub], M, 0)[0]) < 1e-5


# Inputs whose scales are among the smallest normal numbers: results of ordinary inputs times a power of two.
@pytest.mark.parametrize("M", [9, 30])
def test_rows_plan_with_inputs_of_any_size(M):
    say("rows plan, inputs of any size", M)
    bulk = bulk_layer(M, 100)
    entries, _ = model_entries([(300, 512, 0), (129, 1536, 1), (2500, 2048, 2)], (0, 0), M=M, seed=8790)
    for e in entries + [bulk[0]]:
        e["x"][:, 0] = 64.0                                  # (every scale at least half of 1)
    ran = []
    for power in (0, -124):
        for e in entries + [bulk[0]]:
            e["x"].mul_(2.0 ** power)
        dl = nvq.DecodeList(entries + [bulk[0]], M, 0)
        assert kernels_of(dl) == ["rows"]
        dl.run_plan()
        torch.cuda.synchronize()
        ran.append([e["y"].clone() for e in entries + [bulk[0]]])
        dl.close()
    for y, tiny in zip(*ran):
        want = y.double() * 2.0 ** -124
        big = want.abs() >= 2.0 ** -126
        assert torch.equal(tiny.double()[big], want[big])


@pytest.mark.parametrize("M,kernel", [(2, "rings"), (16, "rings"), (17, "rings"), (32, "rings"), (17, "rows"),
                                      (32, "rows")])
def test_grid_sums_are_added_in_the_stated_order(M, kernel):
    """Bit for bit against the same additions on the CPU (see the test of the single calls): K of one
    step pair, of whole eights of steps, and beyond; inputs of W4A16 layers small and whole."""
    say("grid plan, order of sums", M, kernel)
    rng = np.random.default_rng(8670 + M)
    entries, refs = [], []
    for i, K in enumerate([512, 1536, 2048, 2560, 4096, 4608, 6144, 1024] * 4):
        N, prec = int(rng.integers(20, 300)), i % 2
        q = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)
        s = rng.integers(0x1400, 0x2c00, (N, K // 32)).astype(np.uint16)
        qd, sd = to_dev_packed(q, s)
        if prec == nvq.W4A16:
            xq, xs = rng.integers(-99, 100, (M, K)).astype(np.int8), None
            x = torch.from_numpy(xq).to(torch.bfloat16)
        else:
            x = act(8680 + i, M, K)
            xq, xs, _ = oracle.quant_act_i8(u16(x), 0)
        _, acc = oracle.gemv_w4a8(q, s, xq, np.ones(M, np.float32), 0, want_acc=True)
        sw = np_ref.half_bits_to_f64(s)
        refs.append(np_ref.sums_in_steps(acc, sw, xs) if kernel == "rows" else np_ref.sums_in_order(acc, sw, 4, xs))
        entries.append(dict(qweight=qd, scales=sd, x=x.to(DEV), precision=prec,
                            y=torch.zeros((M, N), dtype=torch.float32, device=DEV)))
    bulk = [bulk_layer(M, 300)[0]] if kernel == "rows" else []
    dl = nvq.DecodeList(entries[:9] + bulk + entries[9:], M, 0)
    assert kernels_of(dl) == [kernel]
    dl.run_plan()
    torch.cuda.synchronize()
    for i, (e, want) in enumerate(zip(entries, refs)):
        got = e["y"].cpu().numpy()
        assert np.array_equal(got, want), (i, int((got != want).sum()), np_ref.rel_l2(got, want))
    dl.close()


# The same up to 16 tokens, one token tile: one and several tokens, every token there is room for; phases of
# several matrices whose boundaries fall inside a unit, fewer rows than a unit (tolerance as with the rings), and
# the order of the sums.
@pytest.mark.parametrize("M,bits,mbytes", [(2, (0, 1), 300), (7, (1, 0), 300), (16, (0, 1, 1), 120)])
def test_rows_plan_up_to_16_tokens(M, bits, mbytes):
    say("rows plan up to 16 tokens", M, bits)
    entries, host = model_entries([s for s in RING_SHAPES if s[1] != 14336], bits, M=M, seed=8600)
    ys_ref = oracle.decode_linears(host, M, 0)
    bulk = bulk_layer(M, mbytes)
    dl = nvq.DecodeList(entries[:5] + [bulk[0]] + entries[5:], M, 0)
    assert dl.plan_info()["persistent_grouped"] and kernels_of(dl) == ["rows"]
    for rep in range(3):
        for e in entries:
            e["y"].zero_()
        dl.run_plan()
        torch.cuda.synchronize()
        for e, y_r in zip(entries, ys_ref):
            assert np_ref.rel_l2(e["y"].cpu().numpy(), y_r) < 1e-5, rep
        check_bulk(bulk, M)
    dl.close()
    test_grid_sums_are_added_in_the_stated_order(M, "rows")


# The shortest lists that take the grid with shared activations: from 17 tokens on fewer groups than compute units,
# parts of a few groups; phases of three units, of one unit, of one row.
@pytest.mark.parametrize("M,phases,rows,K", [(17, 30, 340, 1024), (32, 24, 420, 1024), (20, 16, 700, 1024),
                                             (17, 40, 220, 1024), (16, 40, 1900, 1024)])
def test_rows_plan_of_short_lists(M, phases, rows, K):
    say("rows plan, short list", M, phases, rows, K)
    shapes = [(rows + 37 * (p % 5), K, p) for p in range(phases)] + [(1, 512, phases), (33, 1024, phases + 1)]
    entries, host = model_entries(shapes, (0,), M=M, seed=8660)
    for i, (e, h) in enumerate(zip(entries, host)):
        e["precision"] = h["precision"] = i % 2
    ys_ref = oracle.decode_linears(host, M, 0)
    dl = nvq.DecodeList(entries, M, 0)
    assert kernels_of(dl) == ["rows"]
    for rep in range(2):
        for e in entries:
            e["y"].fill_(9.0)
        dl.run_plan()
        torch.cuda.synchronize()
        for i, (e, y_r) in enumerate(zip(entries, ys_ref)):
            assert np_ref.rel_l2(e["y"].cpu().numpy(), y_r) < 1e-5, (rep, i)
    dl.close()


@pytest.mark.parametrize("M", [17, 32])
def test_rows_plan_short_batches_run_phase_by_phase(M):
    """Forced order: every phase is a batch of its own, too small for the persistent grid."""
    say("rows plan, single phases", M)
    entries, host = model_entries([(300, 1536, 0), (45, 1536, 0), (512, 1024, 1), (64, 14336, 2)], (0, 1), M=M,
                                  seed=8660)
    ys_ref = oracle.decode_linears(host, M, 0)
    dl = nvq.DecodeList(entries, M, 0, ordered=True)
    info = dl.plan_info()
    assert not info["grouped"] and info["waits"] == info["phases"] - 1
    assert kernels_of(dl, ordered=True) == ["phases"] * info["phases"]
    for rep in range(2):
        for e in entries:
            e["y"].zero_()
        dl.run_plan()
        torch.cuda.synchronize()
        for e, y_r in zip(entries, ys_ref):
            assert np_ref.rel_l2(e["y"].cpu().numpy(), y_r) < 1e-5, rep
    dl.close()


@pytest.mark.parametrize("M", [2, 9, 16])
def test_short_lists_of_the_rings_kind_run_as_the_per_tile_grid(M):
    """Every K a multiple of 512, but too little work for the persistent grid: the same bits (four
    chains of columns, see above), eager and replayed with eager work in between; one more, wider
    phase takes the list back to the rings."""
    say("per-tile grid, whole 512s", M)
    rng = np.random.default_rng(8720 + M)
    entries, refs = [], []
    for i, K in enumerate([512, 1024, 2048, 4608, 1536, 5632] * 2):
        N, prec = int(rng.integers(200, 500)), (i // 2) % 2
        q = rng.integers(0, 256, (N, K // 2), dtype=np.uint8)
        s = rng.integers(0x1400, 0x2c00, (N, K // 32)).astype(np.uint16)
        qd, sd = to_dev_packed(q, s)
        if prec == nvq.W4A16:
            xq, xs = rng.integers(-99, 100, (M, K)).astype(np.int8), None
            x = torch.from_numpy(xq).to(torch.bfloat16)
        else:
            x = act(8730 + i, M, K)
            xq, xs, _ = oracle.quant_act_i8(u16(x), 0)
        _, acc = oracle.gemv_w4a8(q, s, xq, np.ones(M, np.float32), 0, want_acc=True)
        refs.append(np_ref.sums_in_order(acc, np_ref.half_bits_to_f64(s), 4, xs))
        entries.append(dict(qweight=qd, scales=sd, x=x.to(DEV), precision=prec,
                            y=torch.zeros((M, N), dtype=torch.float32, device=DEV)))
    dl = nvq.DecodeList(entries, M, 0)
    info = dl.plan_info()
    assert info["grouped"] and not info["persistent_grouped"] and kernels_of(dl) == ["tiles"]
    assert not dl.plan_timed_out()
    g = torch.cuda.CUDAGraph()
    for rep in range(4):
        for e in entries:
            e["y"].zero_()
        if rep == 1:
            with torch.cuda.graph(g):
                dl.run_plan()
        if rep == 0:
            dl.run_plan()
        else:
            g.replay()
        torch.cuda.synchronize()
        for i, (e, want) in enumerate(zip(entries, refs)):
            assert np.array_equal(e["y"].cpu().numpy(), want), (rep, i)
    del g
    dl.close()
    wide, _ = model_entries([(32, 14336, 0)], (0,), M=M, seed=8740)
    dl = nvq.DecodeList(entries + wide, M, 0)
    assert dl.plan_info()["persistent_grouped"] and kernels_of(dl) == ["rings"]
    dl.run_plan()
    torch.cuda.synchronize()
    assert all(np.array_equal(e["y"].cpu().numpy(), want) for e, want in zip(entries, refs))
    dl.close()


def test_ring_plan_needs_k_multiple_of_512():
    say("ring plan fallback")
    M = 4
    entries, host = model_entries([(96, 1536, 0), (200, 640, 1)], (0, 1), M=M, seed=8700)
    ys_ref = oracle.decode_linears(host, M, 0)
    dl = nvq.DecodeList(entries, M, 0)
    info = dl.plan_info()
    assert info["grouped"] and not info["persistent_grouped"]   # K = 640: the per-tile grid
    dl.run_plan()
    torch.cuda.synchronize()
    for e, y_r in zip(entries, ys_ref):
        assert np_ref.rel_l2(e["y"].cpu().numpy(), y_r) < 1e-5
    dl.close()


def test_grouped_plan_orders_dependent_phases():
    say("grouped chain")
    # four phases, each reading the bf16 output of the one before it: four batches
    M = 6
    dims = [2048, 4096, 1024, 6144, 512]
    hostW = [oracle.pack_int4(synth.make_weight(8900 + i, dims[i + 1], dims[i]).numpy())
             for i in range(4)]
    x0 = act(8999, M, dims[0])
    bufs = [x0.to(DEV)] + [torch.zeros((M, d), dtype=torch.bfloat16, device=DEV) for d in dims[1:]]
    entries = []
    for i, (q, s) in enumerate(hostW):
        qd, sd = to_dev_packed(q, s)
        entries.append(dict(qweight=qd, scales=sd, x=bufs[i], y=bufs[i + 1], precision=i % 2))
    dl = nvq.DecodeList(entries, M)
    info = dl.plan_info()
    assert not info["streaming"] and info["waits"] == 3      # the analysis found the chain
    for rep in range(2):
        for b in bufs[1:]:
            b.zero_()
        dl.run_plan()
        torch.cuda.synchronize()
        for i, (q, s) in enumerate(hostW):
            y_r = oracle.decode_linears([dict(qweight=q, scales=s, x=u16(bufs[i]),
                                              precision=i % 2)], M)[0]
            assert np_ref.rel_l2(bufs[i + 1].float().cpu().numpy(), y_r) < 4e-3, (rep, i)
    dl.close()


# ---- input transforms: RMSNorm (+ residual) and SiLU-multiply ------------------------
def ulp_report(got_u16, want_u16):
    """(fraction of differing elements, largest difference in bf16 units of last place)."""
    a = got_u16.astype(np.int32)
    b = want_u16.astype(np.int32)
    # order-preserving integer view of the sign-magnitude patterns
    a = np.where(a & 0x8000, -(a & 0x7fff), a)
    b = np.where(b & 0x8000, -(b & 0x7fff), b)
    d = np.abs(a - b)
    return float((d != 0).mean()), int(d.max())


@pytest.mark.parametrize("M,K,with_res", [(1, 4096, False), (1, 4096, True), (3, 2048, True),
                                          (16, 14336, True), (2, 96, False), (32, 8192, False)])
def test_rms_norm_matches_oracle(M, K, with_res):
    say("rms_norm", M, K, with_res)
    x = act(9100 + K, M, K)
    r = act(9200 + K, M, K) if with_res else None
    gamma = (1.0 + 0.1 * torch.randn(K, generator=torch.Generator().manual_seed(K))).to(torch.bfloat16)
    out_r, h_r = oracle.rms_norm(u16(x), u16(gamma), 1e-5, res_bf16=u16(r) if with_res else None)
    out, h = nvq.rms_norm(x.to(DEV), gamma.to(DEV), 1e-5, r.to(DEV) if with_res else None)
    torch.cuda.synchronize()
    if with_res:
        assert np.array_equal(u16(h), h_r)            # the bf16 addition is exact-rounded
    frac, worst = ulp_report(u16(out), out_r)
    say("  differing %.2e, worst %d ulp" % (frac, worst))
    assert worst <= 1 and frac < 2e-3


@pytest.mark.parametrize("M,K", [(1, 14336), (5, 8192), (32, 4096), (2, 64)])
def test_silu_mul_matches_oracle(M, K):
    say("silu_mul", M, K)
    g = act(9300 + K, M, K)
    u = act(9400 + K, M, K)
    want = oracle.silu_mul(u16(g), u16(u))
    out = nvq.silu_mul(g.to(DEV), u.to(DEV))
    torch.cuda.synchronize()
    frac, worst = ulp_report(u16(out), want)
    say("  differing %.2e, worst %d ulp" % (frac, worst))
    assert worst <= 1 and frac < 2e-3


def block_with_transforms(M, hidden, kv, ffn, seed, bits):
    """One transformer block's linears with their neighbours fused in: RMSNorm in front of
    q/k/v, the attention output (its own buffer) into o, residual add + RMSNorm in front of
    gate/up, SiLU-multiply in front of down.  Returns (entries, buffers, host weights)."""
    g1 = (1.0 + 0.1 * torch.randn(hidden, generator=torch.Generator().manual_seed(seed))).to(torch.bfloat16)
    g2 = (1.0 + 0.1 * torch.randn(hidden, generator=torch.Generator().manual_seed(seed + 1))).to(torch.bfloat16)
    B = dict(h0=act(seed + 2, M, hidden).to(DEV), attn=act(seed + 3, M, hidden).to(DEV),
             g1=g1.to(DEV), g2=g2.to(DEV),
             o=torch.zeros((M, hidden), dtype=torch.bfloat16, device=DEV),
             h1=torch.zeros((M, hidden), dtype=torch.bfloat16, device=DEV),
             gate=torch.zeros((M, ffn), dtype=torch.bfloat16, device=DEV),
             up=torch.zeros((M, ffn), dtype=torch.bfloat16, device=DEV))
    shapes = [("q", hidden, hidden), ("k", kv, hidden), ("v", kv, hidden), ("o", hidden, hidden),
              ("gate", ffn, hidden), ("up", ffn, hidden), ("down", hidden, ffn)]
    W, entries = {}, []
    for i, (name, N, K) in enumerate(shapes):
        _, q, s = packed(seed + 10 + i, N, K)
        W[name] = (q, s)
        qd, sd = to_dev_packed(q, s)
        e = dict(qweight=qd, scales=sd, precision=bits[0] if i < 4 else bits[1])
        if name in ("q", "k", "v"):
            e.update(x=B["h0"], in_op=nvq.IN_RMSNORM, gamma=B["g1"], eps=1e-5,
                     y=torch.zeros((M, N), dtype=torch.float32, device=DEV))
        elif name == "o":
            e.update(x=B["attn"], y=B["o"])
        elif name in ("gate", "up"):
            e.update(x=B["h0"], x2=B["o"], in_op=nvq.IN_RMSNORM, gamma=B["g2"], eps=1e-5,
                     h_out=B["h1"], y=B[name])
        else:
            e.update(x=B["gate"], x2=B["up"], in_op=nvq.IN_SILU_MUL,
                     y=torch.zeros((M, N), dtype=torch.float32, device=DEV))
        entries.append(e)
    return entries, B, W


def check_block_against_oracle(entries, B, W, M):
    """Every stage against the oracle applied to the GPU's own inputs of that stage."""
    names = ["q", "k", "v", "o", "gate", "up", "down"]
    for e, name in zip(entries, names):
        q, s = W[name]
        h = dict(qweight=q, scales=s, x=u16(e["x"]), precision=e["precision"],
                 in_op=e.get("in_op", 0))
        if e.get("x2") is not None:
            h["x2"] = u16(e["x2"])
        if e.get("gamma") is not None:
            h["gamma"], h["eps"] = u16(e["gamma"]), e["eps"]
        y_r = oracle.decode_linears([h], M)[0]
        got = e["y"].float().cpu().numpy()
        err = np_ref.rel_l2(got, y_r)
        # fp32 outputs: the bar (rare one-ulp differences of a transformed bf16 input move them
        # by ~1e-4); bf16 outputs add their own rounding, 2^-9 relative per value at most
        assert err < (TOL if e["y"].dtype == torch.float32 else 4e-3), (name, err)
        if name == "gate":
            assert np.array_equal(u16(B["h1"]), h["h"])       # the updated residual stream


@pytest.mark.parametrize("M", [1, 3])
@pytest.mark.parametrize("bits", [(0, 1), (1, 0)])
def test_decode_linears_with_input_transforms(M, bits):
    say("walker with transforms", M, bits)
    entries, B, W = block_with_transforms(M, 2048, 512, 8192, 9500, bits)
    dl = nvq.DecodeList(entries, M, 0)
    info = dl.plan_info()
    say("  plan", info)
    if M == 1:
        # one launch; gate/up wait for o (their residual operand), down waits for gate/up
        assert info["streaming"] and info["phases"] == 4 and info["waits"] == 2
    for rep in range(2):
        for k in ("o", "h1", "gate", "up"):
            B[k].zero_()
        dl.run_plan()
        torch.cuda.synchronize()
        assert not dl.plan_timed_out()
        check_block_against_oracle(entries, B, W, M)
    dl.close()


# Several tokens: the walk prepares a layer's input in one launch (transform and quantisation
# together).  K with one and with two chunks of eight values per thread, the second round filled in
# part (8224: 1028 chunks) and nearly in full; K beyond 16384, which is prepared step by step; fewer
# values than one wave takes.
@pytest.mark.parametrize("M,group", [(2, 0), (8, 32), (32, 0), (32, 32)])
@pytest.mark.parametrize("K", [96, 4096, 8224, 14336, 16416])
def test_prepared_inputs_equal_the_standalone_calls(M, group, K):
    """A norm (with and without a residual), a SiLU-multiply and a plain input in front of W4A8 and
    W4A16 layers: bit for bit what the entry points give one after the other, so the norm's sum,
    the bf16 values, the codes and their scales are the same; and the oracle's product of them."""
    say("prepared inputs", M, group, K)
    N = 40
    a, b = act(9720 + K, M, K), act(9730 + K, M, K)
    gamma = (1.0 + 0.1 * torch.randn(K, generator=torch.Generator().manual_seed(K))).to(torch.bfloat16)
    ad, bd, gd = a.to(DEV), b.to(DEV), gamma.to(DEV)
    _, q, s = packed(9740 + K, N, K)
    qd, sd = to_dev_packed(q, s)
    ops = [dict(x=ad), dict(x=ad, x2=bd, in_op=nvq.IN_SILU_MUL),
           dict(x=ad, in_op=nvq.IN_RMSNORM, gamma=gd, eps=1e-5),
           dict(x=ad, x2=bd, in_op=nvq.IN_RMSNORM, gamma=gd, eps=1e-5, h_out=torch.zeros_like(ad))]
    entries = [dict(op, qweight=qd, scales=sd, precision=p,
                    y=torch.zeros((M, N), dtype=torch.float32, device=DEV))
               for op in ops for p in (nvq.W4A8, nvq.W4A16)]
    for e in entries:
        if "h_out" in e:
            e["h_out"] = torch.zeros_like(ad)
    dl = nvq.DecodeList(entries, M, group)
    dl.run_plan()
    torch.cuda.synchronize()
    for e in entries:
        x = e["x"]
        if e.get("in_op") == nvq.IN_RMSNORM:
            x, h = nvq.rms_norm(ad, gd, 1e-5, e.get("x2"))
            if "h_out" in e:
                assert torch.equal(e["h_out"], h)
        elif e.get("in_op") == nvq.IN_SILU_MUL:
            x = nvq.silu_mul(ad, bd)
        if e["precision"] == nvq.W4A16:
            want = nvq.gemv_w4a16(qd, sd, x)
        else:
            xq, xs, gs = nvq.quant_act_i8(x, group)
            want = nvq.gemv_w4a8(qd, sd, xq, xs, gs, group)
        torch.cuda.synchronize()
        what = (e.get("in_op", 0), "x2" in e, e["precision"])
        assert torch.equal(e["y"], want), (what, int((e["y"] != want).sum()))
        # the oracle on the transformed values themselves (an input that the two transforms round
        # differently can move a token's scale, and with it every one of its codes)
        h = dict(qweight=q, scales=s, x=u16(x), precision=e["precision"])
        assert np_ref.rel_l2(e["y"].cpu().numpy(), oracle.decode_linears([h], M, group)[0]) < 1e-5, what
    dl.close()


# Walk in launches per phase, two matrices whose row tiles go out two by two: what is left over gets
# workgroups of one tile each (a compute unit's worth or less: 2, 256, and with ragged matrices), so the rows
# of a matrix lie in two places of the launch.  As one matrix the same rows are one piece.
@pytest.mark.parametrize("prec", [nvq.W4A8, nvq.W4A16])
@pytest.mark.parametrize("M,Na,Nb", [(8, 8224, 8192), (5, 10240, 10240), (3, 9985, 10480), (20, 16400, 21)])
def test_walk_rows_in_two_matrices_equal_those_of_one(prec, M, Na, Nb):
    say("walk, two matrices or one", prec, M, Na, Nb)
    K = 512
    q = torch.randint(0, 256, (Na + Nb, K // 2), dtype=torch.uint8, device=DEV,
                      generator=torch.Generator(device=DEV).manual_seed(31 + M))
    s = torch.randint(0x1400, 0x2c00, (Na + Nb, K // 32), dtype=torch.int16, device=DEV,
                      generator=torch.Generator(device=DEV).manual_seed(32 + M))
    x = act(33 + M, M, K).to(DEV)
    norm = dict(x=x, in_op=nvq.IN_RMSNORM, gamma=torch.ones(K, dtype=torch.bfloat16, device=DEV), eps=1e-5,
                precision=prec)
    ys = [torch.full((M, n), 9.0, dtype=torch.float32, device=DEV) for n in (Na, Nb, Na + Nb)]
    parts = [dict(norm, qweight=q[:Na], scales=s[:Na], y=ys[0]), dict(norm, qweight=q[Na:], scales=s[Na:], y=ys[1])]
    nvq.decode_linears(parts, M, 0)
    nvq.decode_linears([dict(norm, qweight=q, scales=s, y=ys[2])], M, 0)
    torch.cuda.synchronize()
    assert torch.equal(torch.cat(ys[:2], 1), ys[2])
    h = nvq.rms_norm(x, norm["gamma"], 1e-5)[0]
    rows = torch.tensor([0, 15, 16, Na - 1, Na, Na + Nb - 1])
    host = dict(qweight=q[rows.to(DEV)].cpu().numpy(), scales=u16(s[rows.to(DEV)]), x=u16(h), precision=prec)
    want = oracle.decode_linears([host], M, 0)[0]
    assert np_ref.rel_l2(ys[2][:, rows.to(DEV)].cpu().numpy(), want) < 1e-5


# Two phases that follow each other and do not depend on each other share their launches.  q (two
# matrices) and o: independent; o and r: r reads what o wrote; r and w: w overwrites what r read;
# five matrices on one input (two phases, one preparation) and one more phase; another K.  Sizes:
# chains by columns and by groups, one and two row tiles per workgroup, ragged rows and K.  (Three
# tokens and few rows go to a kernel that takes one phase at a time.)
@pytest.mark.parametrize("M,group,K,N", [(2, 0, 256, 40), (3, 32, 96, 33), (8, 0, 4096, 512), (8, 32, 1056, 4100),
                                         (17, 0, 512, 9000), (32, 32, 288, 70), (5, 0, 16416, 24)])
@pytest.mark.parametrize("prec", [nvq.W4A8, nvq.W4A16])
def test_phases_that_share_a_launch_equal_single_calls(M, group, K, N, prec):
    say("shared launches", M, group, K, N, prec)
    dev = lambda t: t.to(DEV)
    a, b = dev(act(9900 + K, M, K)), dev(act(9910 + K, M, K))
    gamma = dev((1.0 + 0.1 * torch.randn(K, generator=torch.Generator().manual_seed(K))).to(torch.bfloat16))
    w = {}

    def layer(name, rows, k=K):
        _, q, sc = packed(9920 + len(w) + k, rows, k)
        w[name] = to_dev_packed(q, sc)
        return dict(qweight=w[name][0], scales=w[name][1], precision=prec)

    def out(rows, dt=torch.float32):
        return torch.zeros((M, rows), dtype=dt, device=DEV)

    c, over = a.clone(), b.clone()
    K2 = K + 32
    d = dev(act(9930 + K, M, K2))
    h = torch.zeros_like(a)
    norm = dict(x=a, x2=b, in_op=nvq.IN_RMSNORM, gamma=gamma, eps=1e-5, h_out=h)
    entries = [dict(layer("q0", N), **norm, y=out(N)), dict(layer("q1", 16), **norm, y=out(16)),
               dict(layer("o", K), x=c, y=out(K, torch.bfloat16))]
    r_in = entries[2]["y"]
    entries += [dict(layer("r", N), x=r_in, y=out(N)),
                # (overwrites the input of the phase before it)
                dict(layer("w", K), x=over, x2=a, in_op=nvq.IN_SILU_MUL, y=r_in),
                dict(layer("k2", 48, K2), x=d, y=out(48))]
    entries += [dict(layer("m%d" % i, N), x=b, y=out(N)) for i in range(5)]
    entries += [dict(layer("last", N), x=c, x2=b, in_op=nvq.IN_SILU_MUL, y=out(N))]

    def one(name, x):
        if prec == nvq.W4A16:
            return nvq.gemv_w4a16(*w[name], x)
        xq, xs, gs = nvq.quant_act_i8(x, group)
        return nvq.gemv_w4a8(*w[name], xq, xs, gs, group)

    xn, hn = nvq.rms_norm(a, gamma, 1e-5, b)
    o = one("o", c).to(torch.bfloat16)
    want = [one("q0", xn), one("q1", xn), None, one("r", o),
            one("w", nvq.silu_mul(over, a)).to(torch.bfloat16), one("k2", d)]
    want += [one("m%d" % i, b) for i in range(5)] + [one("last", nvq.silu_mul(c, b))]
    torch.cuda.synchronize()

    def check(what):
        torch.cuda.synchronize()
        assert torch.equal(h, hn), what
        for i, (e, y) in enumerate(zip(entries, want)):
            if y is not None:
                assert torch.equal(e["y"], y), (what, i, int((e["y"] != y).sum()))

    dl = nvq.DecodeList(entries, M, group)
    steps = nvq.plan_describe_steps([dl.arr[i] for i in range(dl.n)], M, group)
    assert [first for first, count in steps if count == 2] == ([] if M == 3 else [0, 5])
    assert dl.plan_info() == dict(streaming=False, grouped=False, persistent_grouped=False, phases=8, waits=0)
    for rep in range(2):
        dl.run_plan()
        check("plan")
    for e in entries:
        e["y"].zero_()
    dl.run_static()
    check("static")
    dl.close()


# Launches per phase store h_out without x2 as well: the phase behind reads it, or its input is what
# the next one stores, so neither pair shares a launch.
@pytest.mark.parametrize("prec", [nvq.W4A8, nvq.W4A16])
@pytest.mark.parametrize("M", [2, 8, 32])
def test_residual_outputs_without_a_second_input_are_ordered(M, prec):
    say("h_out without x2", M, prec)
    K, N = 1056, 80
    (_, q0, s0), (_, q1, s1) = packed(9970, N, K), packed(9971, N, K)
    w = [to_dev_packed(q0, s0), to_dev_packed(q1, s1)]
    x, old = act(9972, M, K).to(DEV), act(9973, M, K).to(DEV)
    gamma = torch.ones(K, dtype=torch.bfloat16, device=DEV)
    h, y = torch.empty_like(x), [torch.zeros((M, N), device=DEV) for _ in range(2)]
    norm = dict(qweight=w[0][0], scales=w[0][1], x=x, in_op=nvq.IN_RMSNORM, gamma=gamma, eps=1e-5, h_out=h, y=y[0],
                precision=prec)
    plain = dict(qweight=w[1][0], scales=w[1][1], x=h, y=y[1], precision=prec)

    def one(i, v):
        if prec == nvq.W4A16:
            return nvq.gemv_w4a16(*w[i], v)
        xq, xs, gs = nvq.quant_act_i8(v, 32)
        return nvq.gemv_w4a8(*w[i], xq, xs, gs, 32)

    normed = one(0, nvq.rms_norm(x, gamma, 1e-5)[0])
    for entries, read in (([norm, plain], x), ([plain, norm], old)):
        dl = nvq.DecodeList(entries, M, 32)
        for run in (dl.run_plan, dl.run_static):
            h.copy_(old)
            run()
            torch.cuda.synchronize()
            assert torch.equal(h, x) and torch.equal(y[0], normed) and torch.equal(y[1], one(1, read))
        dl.close()


# Which phases share launches depends on the operands and on M, and the second input that these need
# lies at the workspace's end: a workspace sized for the same shapes with the second phase behind the
# first serves the independent list too, in launches of its own, with the same bits; a byte less than
# that is refused.
@pytest.mark.parametrize("prec", [nvq.W4A8, nvq.W4A16])
def test_phases_that_could_share_a_launch_run_in_the_workspace_of_dependent_ones(prec):
    say("workspace of dependent phases", prec)
    M, K, N = 8, 1056, 80
    a, b = act(9960, M, K).to(DEV), act(9961, M, K).to(DEV)
    (_, q0, s0), (_, q1, s1) = packed(9962, K, K), packed(9963, N, K)
    w = [to_dev_packed(q0, s0), to_dev_packed(q1, s1)]
    y0, y1 = torch.zeros((M, K), dtype=torch.bfloat16, device=DEV), torch.zeros((M, N), device=DEV)

    def entries(x1):
        return [dict(qweight=w[0][0], scales=w[0][1], x=a, y=y0, precision=prec),
                dict(qweight=w[1][0], scales=w[1][1], x=x1, y=y1, precision=prec)]

    dl, behind = nvq.DecodeList(entries(b), M, 32), nvq.DecodeList(entries(y0), M, 32)
    assert behind.workspace.numel() < dl.workspace.numel()
    dl.run()
    want = y0.clone(), y1.clone()
    y0.zero_(), y1.zero_()
    dl.workspace = guarded = torch.full_like(dl.workspace, 0x5a)
    dl.workspace = guarded[:behind.workspace.numel()]
    dl.run()
    assert torch.equal(y0, want[0]) and torch.equal(y1, want[1])
    assert bool((guarded[behind.workspace.numel():] == 0x5a).all())
    dl.workspace = guarded[:behind.workspace.numel() - 1]
    with pytest.raises(nvq.NvqError):
        dl.run()
    dl.close()
    behind.close()


def test_chain_of_blocks_with_transforms_in_one_launch():
    say("block chain with transforms")
    # two blocks at the 1B shapes, the second fed by the first (the residual add of the first
    # block's down projection happens in front of the second block's q/k/v), W4A8 then W4A16
    M, hidden, kv, ffn = 1, 2048, 512, 8192
    e0, B0, W0 = block_with_transforms(M, hidden, kv, ffn, 9600, (0, 0))
    e1, B1, W1 = block_with_transforms(M, hidden, kv, ffn, 9700, (1, 1))
    down0 = torch.zeros((M, hidden), dtype=torch.bfloat16, device=DEV)
    e0[6]["y"] = down0
    h2 = torch.zeros((M, hidden), dtype=torch.bfloat16, device=DEV)
    for e in e1[:3]:                      # q/k/v of block 1: RMSNorm(h1 + down0), sum -> h2
        e.update(x=B0["h1"], x2=down0, h_out=h2)
    for e in e1[4:6]:                     # gate/up of block 1: RMSNorm(h2 + o1), sum -> h1'
        e.update(x=h2)
    entries = e0 + e1
    dl = nvq.DecodeList(entries, M, 0)
    info = dl.plan_info()
    say("  plan", info)
    assert info["streaming"] and info["phases"] == 8 and info["waits"] == 5
    for rep in range(3):
        for t in (B0["o"], B0["h1"], B0["gate"], B0["up"], down0, h2, B1["o"], B1["h1"],
                  B1["gate"], B1["up"]):
            t.zero_()
        dl.run_plan()
        torch.cuda.synchronize()
        assert not dl.plan_timed_out(), (rep, hex(dl.status_code))
        check_block_against_oracle(e0, B0, W0, M)
        check_block_against_oracle(e1, B1, W1, M)
        # the residual stream entering block 1 is the exact bf16 sum
        assert torch.equal(h2, B0["h1"] + down0)
    dl.close()


# ---- exact sums: int32 accumulators and fused int8 codes of the kernels that are timed ----
def exact_layer(rng, N, K, M, per_group):
    """Weights c * 2^-7 with integer codes c in [-7, 7] (a 7 in every group: the scale is
    2^-7 exactly) and activations q * 2^e with integer q in [-127, 127] (a 127 in every token,
    or in every group of 32: the activation scale is 2^e exactly and the codes are q).  Then
    every int32 accumulator is the plain integer sum, every fp32 partial sum of the output
    is an integer multiple of a power of two below 2^24 of it, hence exact in any order:
    the fp32 output of a correct kernel equals the float64 oracle's to the bit, and a single
    wrong code or accumulator shows."""
    c = rng.integers(-7, 8, (N, K)).astype(np.float32)
    pos = rng.integers(0, 32, (N, K // 32))
    c.reshape(N, K // 32, 32)[np.arange(N)[:, None], np.arange(K // 32)[None, :], pos] = \
        rng.choice([-7.0, 7.0], (N, K // 32))
    W = c * np.float32(2.0 ** -7)
    q = rng.integers(-127, 128, (M, K)).astype(np.float32)
    if per_group:
        pos = rng.integers(0, 32, (M, K // 32))
        q.reshape(M, K // 32, 32)[np.arange(M)[:, None], np.arange(K // 32)[None, :], pos] = \
            rng.choice([-127.0, 127.0], (M, K // 32))
        e = rng.integers(-2, 3, (M, K // 32)).astype(np.float32)
        x = (q.reshape(M, K // 32, 32) * (2.0 ** e)[:, :, None]).reshape(M, K)
    else:
        q[np.arange(M), rng.integers(0, K, M)] = rng.choice([-127.0, 127.0], M)
        x = q * (2.0 ** rng.integers(-3, 4, (M, 1)).astype(np.float32))
    xb = torch.from_numpy(x.astype(np.float32)).to(torch.bfloat16)
    assert torch.equal(xb.float(), torch.from_numpy(x.astype(np.float32)))      # exact in bf16
    qw, sc = oracle.pack_int4(W)
    assert (sc == 0x2000).all()                                               # fp16 2^-7
    return qw, sc, xb


def exact_list(seed, shapes, M, per_group):
    """shapes: (N, K, phase); one input per phase; precisions alternate by phase."""
    rng = np.random.default_rng(seed)
    entries, host, xs = [], [], {}
    for N, K, ph in shapes:
        qw, sc, xb = exact_layer(rng, N, K, M, per_group)
        if ph not in xs:
            xs[ph] = xb
        qd, sd = to_dev_packed(qw, sc)
        prec = ph % 2
        entries.append(dict(qweight=qd, scales=sd, x=xs[ph].to(DEV), precision=prec,
                            y=torch.zeros((M, N), dtype=torch.float32, device=DEV)))
        host.append(dict(qweight=qw, scales=sc, x=u16(xs[ph]), precision=prec))
    # (entries of a phase must share the device buffer to be grouped)
    by_phase = {}
    for e, (_, _, ph) in zip(entries, shapes):
        e["x"] = by_phase.setdefault(ph, e["x"])
    return entries, host


EXACT_SHAPES = [(4096, 4096, 0), (1024, 4096, 0), (1031, 4096, 1), (640, 14336, 2), (96, 14336, 2),
                (2500, 2048, 3), (77, 8192, 4), (3000, 1024, 5)]


@pytest.mark.parametrize("M,group,ordered,kernel", [
    (1, 0, False, None), (1, 0, True, None), (1, 32, False, None), (1, 32, True, None),
    (2, 0, False, "rings"), (5, 0, False, "rings"), (16, 0, False, "rings"), (17, 0, False, "phases"),
    (32, 0, False, "phases"), (17, 0, False, "rings"), (32, 0, False, "rings"), (17, 0, False, "rows"),
    (32, 0, False, "rows"), (3, 32, False, None)])
def test_exact_sums_are_bit_equal_on_the_timed_kernels(M, group, ordered, kernel):
    """Batch 1: the persistent streaming kernel with its fused quantiser, images prepared in
    the prologue (independent phases) and built after a wait (forced ordering).  2 to 32
    tokens: the persistent matrix-core kernels (every K a multiple of 512); from 17 tokens on
    the shapes alone go phase by phase, three times over through the LDS rings, and with a large
    layer among them through the grid with shared activations.  A scale per 32 activations at
    several tokens: launches per phase."""
    say("exact sums", M, group, ordered, kernel)
    times = 3 if M > 16 and kernel == "rings" else 1
    shapes = [(N, K, ph + 6 * i) for i in range(times) for N, K, ph in EXACT_SHAPES]
    entries, host = exact_list(9000 + M + group, shapes, M, group == 32)
    ys_ref = oracle.decode_linears(host, M, group)
    bulk = [bulk_layer(M, 640)[0]] if kernel == "rows" else []
    dl = nvq.DecodeList(entries[:3] + bulk + entries[3:], M, group, ordered=ordered)
    info = dl.plan_info()
    say("  plan", info)
    assert info["streaming"] == (M == 1)
    assert info["persistent_grouped"] == (kernel in ("rings", "rows"))
    assert kernel is None or kernels_of(dl) == [kernel]
    for rep in range(2):
        for e in entries:
            e["y"].zero_()
        dl.run_plan()
        assert not dl.plan_timed_out()
        for i, (e, y_r) in enumerate(zip(entries, ys_ref)):
            want = y_r.astype(np.float32)
            assert np.array_equal(want.astype(np.float64), y_r)        # the oracle's sum is exact
            got = e["y"].cpu().numpy()
            assert np.array_equal(got, want), (rep, i, int((got != want).sum()))
    dl.close()


def test_exact_sums_are_bit_equal_on_the_per_tile_matrix_core_kernel():
    """K = 640 (no multiple of 512): the grouped per-tile grid with its own quantiser."""
    say("exact sums, per-tile grid")
    M = 7
    entries, host = exact_list(9100, [(200, 640, 0), (96, 1536, 1), (333, 640, 2)], M, False)
    ys_ref = oracle.decode_linears(host, M, 0)
    dl = nvq.DecodeList(entries, M, 0)
    info = dl.plan_info()
    assert info["grouped"] and not info["persistent_grouped"]
    dl.run_plan()
    torch.cuda.synchronize()
    for e, y_r in zip(entries, ys_ref):
        assert np.array_equal(e["y"].cpu().numpy(), y_r.astype(np.float32))
    dl.close()


# ---- mail: an operand that is exactly an earlier layer's bf16 output ---------------------
def stage_reference(e, q, s, M=1):
    """The oracle on the GPU's own inputs of one layer."""
    h = dict(qweight=q, scales=s, x=u16(e["x"]), precision=e["precision"], in_op=e.get("in_op", 0))
    if e.get("x2") is not None:
        h["x2"] = u16(e["x2"])
    if e.get("gamma") is not None:
        h["gamma"], h["eps"] = u16(e["gamma"]), e["eps"]
    return oracle.decode_linears([h], M)[0]


@pytest.mark.parametrize("widths,group", [
    ((2048, 96, 2112, 4096, 64), 0),            # one ragged piece, a part of a piece, whole pieces
    ((4096, 14336, 3072, 1024, 8192, 32), 0),   # the widest input; rows streamed in pairs
    ((1024, 3136, 2048, 512), 32),              # a scale per 32 activations
])
def test_mail_chain_of_plain_layers(widths, group):
    """x0 -> L0 -> L1 -> ...: every layer reads the bf16 output of the one before it, so every
    operand but the first arrives by mail; precisions alternate; several walks (one tag each)."""
    say("mail chain", widths, group)
    entries, W = [], []
    x = act(9900 + widths[0], 1, widths[0]).to(DEV)
    for i in range(len(widths) - 1):
        K, N = widths[i], widths[i + 1]
        _, q, s = packed(9910 + 7 * i + N, N, K)
        qd, sd = to_dev_packed(q, s)
        y = torch.zeros((1, N), dtype=torch.bfloat16, device=DEV)
        entries.append(dict(qweight=qd, scales=sd, x=x, y=y, precision=(i + group // 32) % 2))
        W.append((q, s))
        x = y
    dl = nvq.DecodeList(entries, 1, group)
    info = dl.plan_info()
    _, phases = nvq.plan_describe([dl.arr[i] for i in range(dl.n)], 1, group)
    say("  plan", info, [ph["mail"] for ph in phases])
    assert info["streaming"] and info["waits"] == len(entries) - 1
    assert [ph["mail"] & 3 for ph in phases] == [0] + [1] * (len(entries) - 1)
    assert all(ph["wait"] < 0 for ph in phases)          # nobody waits for flags
    for rep in range(4):
        for e in entries:
            e["y"].zero_()
        if rep == 2:                                      # new data under the next tag
            entries[0]["x"].copy_(act(9950, 1, widths[0]).to(DEV))
        dl.run_plan()
        assert not dl.plan_timed_out()
        for e, (q, s) in zip(entries, W):
            y_r = oracle.decode_linears([dict(qweight=q, scales=s, x=u16(e["x"]),
                                              precision=e["precision"])], 1, group)[0]
            err = np_ref.rel_l2(e["y"].float().cpu().numpy(), y_r)
            assert err < 4e-3, (rep, err)                 # bf16 outputs
            # to the bit once the oracle's value is rounded to bf16 as well, but for sums that
            # fall next to a rounding boundary
            want = torch.from_numpy(y_r.astype(np.float32)).to(torch.bfloat16)
            differing = int((e["y"].cpu() != want).sum())
            assert differing <= max(1, int(5e-3 * want.numel())), (rep, differing)
    dl.close()


def test_mail_and_flags_in_one_list():
    """A buffer that is written twice and read in between: the reader takes the first
    writer's mail, the second writer waits for the first through the flags (it overwrites its
    bytes), and a last layer reads the second writer's mail."""
    say("mail and flags")
    K = 2048
    x0, x1 = act(9960, 1, K).to(DEV), act(9961, 1, K).to(DEV)
    y = torch.zeros((1, K), dtype=torch.bfloat16, device=DEV)
    outs = [torch.zeros((1, 640), dtype=torch.float32, device=DEV) for _ in range(2)]
    Ws = [packed(9970 + i, n, K) for i, n in enumerate((K, 640, K, 640))]
    dev = [to_dev_packed(q, s) for _, q, s in Ws]
    mk = lambda i, x, yy, prec: dict(qweight=dev[i][0], scales=dev[i][1], x=x, y=yy, precision=prec)
    entries = [mk(0, x0, y, 0), mk(1, y, outs[0], 1), mk(2, x1, y, 1), mk(3, y, outs[1], 0)]
    dl = nvq.DecodeList(entries, 1, 0)
    _, phases = nvq.plan_describe([dl.arr[i] for i in range(dl.n)], 1, 0)
    assert [ph["wait"] for ph in phases] == [-1, -1, 0, -1]
    assert [ph["mail"] & 3 for ph in phases] == [0, 1, 0, 1]
    for rep in range(3):
        for t in [y] + outs:
            t.zero_()
        dl.run_plan()
        assert not dl.plan_timed_out()
        # y holds the second writer's result; the first reader saw the first writer's
        y1 = oracle.decode_linears([dict(qweight=Ws[0][1], scales=Ws[0][2], x=u16(x0), precision=0)], 1)[0]
        y1b = torch.from_numpy(y1.astype(np.float32)).to(torch.bfloat16)
        r0 = oracle.decode_linears([dict(qweight=Ws[1][1], scales=Ws[1][2], x=u16(y1b), precision=1)], 1)[0]
        assert np_ref.rel_l2(outs[0].cpu().numpy(), r0) < 5e-3     # (y1b may differ by an ulp here and there)
        r2 = stage_reference(entries[2], Ws[2][1], Ws[2][2])
        assert np_ref.rel_l2(y.float().cpu().numpy(), r2) < 4e-3
        r3 = stage_reference(entries[3], Ws[3][1], Ws[3][2])
        assert np_ref.rel_l2(outs[1].cpu().numpy(), r3) < 1e-5
    dl.close()


def test_mail_tags_wrap_around():
    """A tag has 16 bits: 65535 walks later the same tag comes round again.  Between walks the
    input changes, so a consumer that took an old word for a new one would show."""
    say("mail tag wrap")
    K = 512
    _, q0, s0 = packed(9980, K, K)
    _, q1, s1 = packed(9981, 96, K)
    d0, d1 = to_dev_packed(q0, s0), to_dev_packed(q1, s1)
    x = act(9982, 1, K).to(DEV)
    mid = torch.zeros((1, K), dtype=torch.bfloat16, device=DEV)
    out = torch.zeros((1, 96), dtype=torch.float32, device=DEV)
    entries = [dict(qweight=d0[0], scales=d0[1], x=x, y=mid, precision=1),
               dict(qweight=d1[0], scales=d1[1], x=mid, y=out, precision=0)]
    dl = nvq.DecodeList(entries, 1, 0)
    dl.plan()
    xs = [act(9983 + i, 1, K).to(DEV) for i in range(3)]
    total = 65535 + 6
    for run in range(total):
        check = run < 3 or run >= 65535 - 3
        if check:
            x.copy_(xs[run % 3])
        dl.run_plan()
        if check:
            assert not dl.plan_timed_out()
            r = stage_reference(entries[1], q1, s1)
            assert np_ref.rel_l2(out.cpu().numpy(), r) < 1e-5, run
            m = oracle.decode_linears([dict(qweight=q0, scales=s0, x=u16(x), precision=1)], 1)[0]
            assert np_ref.rel_l2(mid.float().cpu().numpy(), m) < 4e-3, run
        elif run % 8192 == 0:
            torch.cuda.synchronize()
    assert not dl.plan_timed_out()
    dl.close()


# ---- prefill / large-batch product on the matrix cores --------------------------------
# Shapes: one tile, ragged tokens and rows inside a 256 x 128 workgroup tile and inside the
# 32 x 32 MFMA tiles, several workgroups in both directions, K from one group to many.
# The last two: many workgroups in both directions, ragged at both ends.
@pytest.mark.parametrize("M,N,K", [(32, 32, 32), (256, 128, 64), (77, 45, 96), (300, 200, 256),
                                   (513, 257, 2048), (1, 1, 32), (1024, 384, 4096),
                                   (4096, 4096, 64), (4000, 4300, 96)])
def test_gemm_w4a16_matches_oracle(M, N, K):
    say("gemm", M, N, K)
    _, q, s = packed(9100 + M + N, N, K)
    xh = act(9200 + K, M, K)
    want = oracle.gemm_w4a16_dense(q, s, u16(xh))
    qd, sd = to_dev_packed(q, s)
    y = nvq.gemm_w4a16(qd, sd, xh.to(DEV))
    torch.cuda.synchronize()
    err = np_ref.rel_l2(y.cpu().numpy(), want)
    say("  rel l2", err)
    assert err < 1e-5
    yb = nvq.gemm_w4a16(qd, sd, xh.to(DEV), out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    assert np_ref.rel_l2(yb.float().cpu().numpy(), want) < 4e-3


# The kernel with 256 x 256 tiles (K % 256 == 0; chosen by size, forced here so that small shapes
# reach it): one tile, ragged tokens and rows inside a tile and inside the
# MFMA tiles, a single row and token, several tiles in both directions, K from one block of four
# pairs of groups (no steady state in the loop) to many, K with an odd number of such blocks.
@pytest.mark.parametrize("M,N,K", [(256, 256, 256), (300, 200, 512), (1, 1, 256), (33, 70, 1280),
                                   (513, 257, 2048), (1024, 384, 4096), (700, 1000, 2304)])
def test_gemm_w4a16_wide_tiles_match_oracle(M, N, K, monkeypatch):
    say("gemm wide", M, N, K)
    monkeypatch.setenv("NVQ_GEMM_TILE", "wide")
    _, q, s = packed(9150 + M + N, N, K)
    xh = act(9250 + K, M, K)
    want = oracle.gemm_w4a16_dense(q, s, u16(xh))
    qd, sd = to_dev_packed(q, s)
    y = nvq.gemm_w4a16(qd, sd, xh.to(DEV))
    torch.cuda.synchronize()
    err = np_ref.rel_l2(y.cpu().numpy(), want)
    say("  rel l2", err)
    assert err < 1e-5
    yb = nvq.gemm_w4a16(qd, sd, xh.to(DEV), out_dtype=torch.bfloat16)
    torch.cuda.synchronize()
    assert np_ref.rel_l2(yb.float().cpu().numpy(), want) < 4e-3
    # both kernels add the same products in the same order
    monkeypatch.setenv("NVQ_GEMM_TILE", "narrow")
    yn = nvq.gemm_w4a16(qd, sd, xh.to(DEV))
    torch.cuda.synchronize()
    assert torch.equal(y, yn)


# The smaller tiles, each kind forced (the library chooses by size): one row and token, edges of
# the 32 x 32 MFMA tiles and of the workgroup tiles, K from one group on (fewer blocks of four
# groups than slices, and numbers that the slices cannot share evenly), K that ends inside a block,
# rows no multiple of 8 (results stored one by one), scales and results off their usual alignment.
# Tolerance: fp32 sums of exact products, up to 2048 terms in any order.
@pytest.mark.parametrize("tile", ["128x256", "128x128", "128x64", "64x64", "64x32"])
@pytest.mark.parametrize("M,N,K,off", [(1, 1, 32, 0), (65, 33, 96, 0), (64, 64, 128, 0),
                                       (63, 257, 640, 0), (129, 130, 416, 1), (200, 520, 2048, 0),
                                       (33, 72, 1152, 1)])
def test_gemm_w4a16_small_tiles_match_oracle(tile, M, N, K, off, monkeypatch):
    say("gemm tile", tile, M, N, K, off)
    monkeypatch.setenv("NVQ_GEMM_TILE", tile)
    _, q, s = packed(9170 + M + N, N, K)
    xh = act(9270 + K, M, K)
    want = oracle.gemm_w4a16_dense(q, s, u16(xh))
    qd, sd = to_dev_packed(q, s)
    if off:  # scales aligned to their two bytes only
        buf = torch.zeros(sd.numel() + off, dtype=sd.dtype, device=DEV)
        buf[off:] = sd.flatten()
        sd = buf[off:].view(sd.shape)
    y = nvq.gemm_w4a16(qd, sd, xh.to(DEV))
    yb = torch.empty(M * N + off, dtype=torch.bfloat16, device=DEV)[off:].view(M, N)
    nvq.gemm_w4a16(qd, sd, xh.to(DEV), out=yb)
    torch.cuda.synchronize()
    err = np_ref.rel_l2(y.cpu().numpy(), want)
    say("  rel l2", err)
    assert err < 1e-5
    # the bf16 results are the fp32 ones rounded
    assert torch.equal(yb, y.to(torch.bfloat16))


# The order of the additions is the tile's alone: with a tile chosen, a prompt in two pieces gives
# every token the bits it gets in one.  The wide tile and 128x256 agree, and so do the tiles with
# as many pieces of K.
def test_gemm_w4a16_bits_with_a_tile_chosen_do_not_depend_on_the_batch(monkeypatch):
    say("gemm, prompt in pieces")
    M, N, K = 200, 300, 2304
    _, q, s = packed(9185, N, K)
    xd = act(9285, M, K).to(DEV)
    qd, sd = to_dev_packed(q, s)
    whole = {}
    for tile in ("wide", "128x256", "128x128", "128x64", "64x64", "64x32"):
        monkeypatch.setenv("NVQ_GEMM_TILE", tile)
        whole[tile] = nvq.gemm_w4a16(qd, sd, xd)
        parts = torch.cat([nvq.gemm_w4a16(qd, sd, xd[a:b].contiguous()) for a, b in ((0, 1), (1, 70), (70, M))])
        torch.cuda.synchronize()
        assert torch.equal(whole[tile], parts), tile
    assert torch.equal(whole["wide"], whole["128x256"])
    assert torch.equal(whole["128x128"], whole["128x64"])
    assert torch.equal(whole["64x64"], whole["64x32"])


# The tiles of eight waves.  32x32: K in eight slices (fewer blocks than slices, numbers that eight
# cannot share evenly), half of the waves hand all of their sums over.  128x256 and 128x128 where K
# is no whole number of blocks or the scales lie off their words: the same bits as the four waves of
# the other case give, from the same weights at aligned addresses.
@pytest.mark.parametrize("tile", ["32x32", "128x256", "128x128"])
@pytest.mark.parametrize("M,N,K,off", [(1, 1, 32, 0), (33, 31, 96, 0), (32, 32, 1024, 1), (31, 33, 1152, 0),
                                       (65, 129, 1056, 1), (48, 264, 2048, 1), (129, 270, 4160, 0)])
def test_gemm_w4a16_tiles_of_eight_waves(tile, M, N, K, off, monkeypatch):
    test_gemm_w4a16_small_tiles_match_oracle(tile, M, N, K, off, monkeypatch)
    if K % 64 == 0:
        test_gemm_w4a16_small_tiles_infinite_input(tile, K, monkeypatch)
    _, q, s = packed(9186, N, K)
    xd = act(9286, M, K).to(DEV)
    qd, sd = to_dev_packed(q, s)
    monkeypatch.setenv("NVQ_GEMM_TILE", tile)
    whole = nvq.gemm_w4a16(qd, sd, xd)
    last = nvq.gemm_w4a16(qd, sd, xd[M // 2:].contiguous())
    buf = torch.zeros(sd.numel() + 1, dtype=sd.dtype, device=DEV)
    buf[1:] = sd.flatten()
    shifted = nvq.gemm_w4a16(qd, buf[1:].view(sd.shape), xd)
    torch.cuda.synchronize()
    assert torch.equal(whole[M // 2:], last) and torch.equal(whole, shifted)


# Token tiles go in bands of four where there are more than eight: one band of four or five, three of which the last
# has three; every result once, several row tiles.  Tolerance as above.
@pytest.mark.parametrize("tile", ["128x256", "128x128", "128x64", "64x64", "64x32", "32x32"])
@pytest.mark.parametrize("tiles", [4, 5, 11])
def test_gemm_w4a16_bands_of_token_tiles(tile, tiles, monkeypatch):
    tokens, rows = (int(v) for v in tile.split("x"))
    test_gemm_w4a16_small_tiles_match_oracle(tile, (tiles - 1) * tokens + 1, 2 * rows + 8, 160, 0, monkeypatch)


# Eight token tiles are one band, nine three.
@pytest.mark.parametrize("tile", ["128x256", "128x64", "64x32", "32x32"])
@pytest.mark.parametrize("tiles", [8, 9])
def test_gemm_w4a16_first_band_of_token_tiles(tile, tiles, monkeypatch):
    tokens, rows = (int(v) for v in tile.split("x"))
    test_gemm_w4a16_small_tiles_match_oracle(tile, (tiles - 1) * tokens + 1, 2 * rows + 8, 160, 0, monkeypatch)


# Products that end a little past a whole round of all compute units go in two launches, split by
# rows or by tokens (what is asked for at 256 units): rows no multiple of 8, K that ends inside a block,
# scales off their alignment, the two parts of different kinds.  Nothing outside of the result is
# written.  Tolerance as above.
@pytest.mark.parametrize("M,N,K,off,by", [(2049, 4104, 800, 0, "rows"), (2049, 4133, 800, 1, "rows"),
                                          (2049, 2056, 2048, 0, "rows"), (1300, 3079, 2080, 0, "tokens"),
                                          (1281, 3079, 2048, 0, "tokens"), (2049, 2117, 2048, 1, "tokens")])
def test_gemm_w4a16_in_two_launches(M, N, K, off, by):
    say("gemm in two launches", M, N, K, off, by)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        a, b = nvq.gemm_describe(M, N, K, scales_at=2 * off)
        assert (b["first_row"] > 0, b["first_token"] > 0) == (by == "rows", by == "tokens")
        assert (a["tile_tokens"], a["tile_rows"]) != (b["tile_tokens"], b["tile_rows"])
    _, q, s = packed(9300 + N, N, K)
    xh = act(9400 + K, M, K)
    want = oracle.gemm_w4a16_dense(q, s, u16(xh))
    qd, sd = to_dev_packed(q, s)
    buf = torch.zeros(sd.numel() + off, dtype=sd.dtype, device=DEV)
    buf[off:] = sd.flatten()
    sd = buf[off:].view(sd.shape)
    y = {}
    for dt in (torch.float32, torch.bfloat16):
        out = torch.full((M + 2, N), float("nan"), dtype=dt, device=DEV)
        nvq.gemm_w4a16(qd, sd, xh.to(DEV), out=out[1:-1])
        torch.cuda.synchronize()
        assert out[0].isnan().all() and out[-1].isnan().all()
        y[dt] = out[1:-1]
    err = np_ref.rel_l2(y[torch.float32].cpu().numpy(), want)
    say("  rel l2", err)
    assert err < 1e-5
    assert torch.equal(y[torch.bfloat16], y[torch.float32].to(torch.bfloat16))


# Cut by rows, the result itself begins at a whole 16 bytes but its rows are 2 and 8 bytes off: the same bits as the
# fp32 results rounded, nothing outside.
@pytest.mark.parametrize("M,N,K", [(2049, 4133, 800), (227, 4196, 11040)])
def test_gemm_w4a16_in_two_launches_rows_no_whole_16_bytes(M, N, K):
    say("gemm in two launches, ragged rows", M, N, K)
    ws = (torch.randint(0, 256, (N, K // 2), dtype=torch.uint8, device=DEV,
                        generator=torch.Generator(device=DEV).manual_seed(9500 + N)),
          torch.randint(0x1400, 0x2c00, (N, K // 32), dtype=torch.int16, device=DEV,
                        generator=torch.Generator(device=DEV).manual_seed(9600 + N)))
    x = act(9700 + K, M, K).to(DEV)
    if torch.cuda.get_device_properties(0).multi_processor_count == 256:
        parts = nvq.gemm_describe(M, N, K, dtype=torch.bfloat16)
        assert len(parts) == 2 and parts[1]["first_row"] > 0 and {p["store_bytes"] for p in parts} == {2}
    want = nvq.gemm_w4a16(*ws, x, out=torch.empty((M, N), dtype=torch.float32, device=DEV)).to(torch.bfloat16)
    flat = torch.full((M * N + 16,), float("nan"), dtype=torch.bfloat16, device=DEV)
    y = flat[8:8 + M * N].view(M, N)
    assert y.data_ptr() % 16 == 0
    nvq.gemm_w4a16(*ws, x, out=y)
    torch.cuda.synchronize()
    assert torch.equal(y, want) and flat[:8].isnan().all() and flat[-8:].isnan().all()


# An infinite activation in the last group of K: infinite results, NaN only where the weight is
# zero (K that ends inside a block, an odd number of blocks, a single one).
@pytest.mark.parametrize("tile", ["128x256", "128x128", "128x64", "64x64", "64x32"])
@pytest.mark.parametrize("K", [64, 192, 384])
def test_gemm_w4a16_small_tiles_infinite_input(tile, K, monkeypatch):
    monkeypatch.setenv("NVQ_GEMM_TILE", tile)
    M, N = 3, 40
    _, q, s = packed(9180, N, K)
    xh = act(9280, M, K)
    xh[1, K - 1] = float("inf")
    with np.errstate(invalid="ignore"):
        want = oracle.gemm_w4a16_dense(q, s, u16(xh))
    qd, sd = to_dev_packed(q, s)
    y = nvq.gemm_w4a16(qd, sd, xh.to(DEV)).cpu().numpy()
    assert np.array_equal(np.isnan(y), np.isnan(want))
    assert np.array_equal(np.isinf(y), np.isinf(want)) and np.isinf(y[1]).any()
    assert np.array_equal(np.sign(y[1]), np.sign(want[1]), equal_nan=True)


def test_gemm_w4a16_full_size_sampled():
    """A projection of the 8B block at 4096 tokens, as the benchmark launches it (the kernel with
    wide tiles, chosen by the library): sampled tokens and rows against the oracle."""
    say("gemm full size")
    M, N, K = 4096, 4096, 4096
    _, q, s = packed(9160, N, K)
    xh = act(9260, M, K)
    qd, sd = to_dev_packed(q, s)
    y = nvq.gemm_w4a16(qd, sd, xh.to(DEV))
    torch.cuda.synchronize()
    rng = np.random.default_rng(9161)
    toks = np.unique(np.concatenate([[0, 255, 256, M - 1], rng.integers(0, M, 28)]))
    rows = np.unique(np.concatenate([[0, 31, 32, 63, 64, 255, 256, N - 1], rng.integers(0, N, 56)]))
    want = oracle.gemm_w4a16_dense(q[rows], s[rows], u16(xh)[toks])
    got = y.cpu().numpy()[np.ix_(toks, rows)]
    err = np_ref.rel_l2(got, want)
    say("  rel l2", err)
    assert err < 1e-5


def test_gemm_w4a16_takes_every_code(monkeypatch):
    say("gemm codes")
    rng = np.random.default_rng(9300)
    M, N, K = 96, 64, 128
    q = rng.integers(0, 256, (N, K // 2)).astype(np.uint8)          # code -8 included
    s = (rng.random((N, K // 32)).astype(np.float32) * 0.1 + 0.01).astype(np.float16).view(np.uint16)
    xh = act(9301, M, K)
    want = oracle.gemm_w4a16_dense(q, s, u16(xh))
    qd, sd = to_dev_packed(q, s)
    y = nvq.gemm_w4a16(qd, sd, xh.to(DEV))
    torch.cuda.synchronize()
    assert np_ref.rel_l2(y.cpu().numpy(), want) < 1e-5
    # and with the wide tiles
    K = 256
    q = rng.integers(0, 256, (N, K // 2)).astype(np.uint8)
    s = (rng.random((N, K // 32)).astype(np.float32) * 0.1 + 0.01).astype(np.float16).view(np.uint16)
    xh = act(9302, M, K)
    want = oracle.gemm_w4a16_dense(q, s, u16(xh))
    qd, sd = to_dev_packed(q, s)
    monkeypatch.setenv("NVQ_GEMM_TILE", "wide")
    y = nvq.gemm_w4a16(qd, sd, xh.to(DEV))
    torch.cuda.synchronize()
    assert np_ref.rel_l2(y.cpu().numpy(), want) < 1e-5


# ---- calibration statistics (Algorithm 1) ----------------------------------------------
@pytest.mark.parametrize("M,Na,Nb,bf16", [(1, 5, 0, False), (7, 4096, 1024, False),
                                          (33, 4096, 0, True), (3, 1000, 37, True)])
def test_token_norms_match_oracle(M, Na, Nb, bf16):
    say("token norms", M, Na, Nb, bf16)
    g = torch.Generator().manual_seed(9400 + M)
    a = torch.randn((M, Na), generator=g) * 3
    b = torch.randn((M, Nb), generator=g) if Nb else None
    if bf16:
        a = a.to(torch.bfloat16)
        b = b.to(torch.bfloat16) if b is not None else None
        want = oracle.token_norms(u16(a), u16(b) if b is not None else None)
    else:
        want = oracle.token_norms(a.numpy(), b.numpy() if b is not None else None)
    got = nvq.token_norms(a.to(DEV), b.to(DEV) if b is not None else None)
    torch.cuda.synchronize()
    assert np.allclose(got.cpu().numpy(), want, rtol=2e-6, atol=0)

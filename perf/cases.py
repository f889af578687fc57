"""The workloads whose speed this library is judged by, each through its public entry points.

Four kinds of work that a program using the library does, over the sizes it meets:

  step     one decode step of a Llama-shaped model through a prepared plan (`DecodeList.plan`):
           independent layers, each on an input buffer of its own, or the layers wired up as a
           transformer wires them (norms, residual adds and SiLU-multiply in front of the layers
           that read them; attention runs elsewhere); 1 to 32 tokens, activation scales per
           token or per 32 inputs, mixed precision map
  linear   one layer called by itself (quantise and multiply for W4A8, multiply for W4A16)
  prefill  a block's projections over a prompt (`gemm_w4a16`): q+k+v, o, gate+up, down
  load     a weight matrix quantised and packed, and unpacked to bf16, as a loader does

`listed` are the fixed cases, `draw` gives others of the same ranges.  Shapes are those of the
models in `synth.MODELS` or generic.  All inputs come from the seed with torch alone: weights
N(0, 0.02) as 4-bit codes in groups of 32, activations N(0, 1) with one channel in a hundred
twenty times as large.
"""
import torch

from paper_2604_21026_amd import nvq

DEV = "cuda:0"
GROUP = 32
EPS = 1e-5

SHAPES = {  # hidden, kv, ffn, vocabulary rows
    "1b": (2048, 512, 8192, 0),
    "3b": (3072, 1024, 8192, 0),
    "8b": (4096, 1024, 14336, 128256),
}


def _step(name, shape, blocks, tokens, chain, act_group=0, share=0.5, head=False):
    hidden, kv, ffn, vocab = SHAPES[shape]
    return dict(name=name, kind="step", hidden=hidden, kv=kv, ffn=ffn, vocab=vocab if head else 0,
                blocks=blocks, tokens=tokens, chain=chain, act_group=act_group, w4a16_share=share)


def _prefill(name, shape, tokens):
    hidden, kv, ffn, _ = SHAPES[shape]
    return dict(name=name, kind="prefill", hidden=hidden, kv=kv, ffn=ffn, tokens=tokens)


def _linear(name, N, K, tokens, precision, act_group=0, out="float32"):
    return dict(name=name, kind="linear", N=N, K=K, tokens=tokens, precision=precision,
                act_group=act_group, out=out)


def listed():
    return [
        # The step the library's headline figure is quoted on: every layer of an 8B model and its
        # vocabulary projection for one token, half of the blocks W4A16, inputs ready beforehand.
        _step("step_8b_b1", "8b", 32, 1, chain=False, head=True),
        # The same layers as one sequence decodes them, each waiting for the one before it (eight
        # blocks: the rounding of one layer travels through all that follow, and in 32 blocks two
        # correct results end up 4 % apart).
        _step("chain_8b_b1", "8b", 8, 1, chain=True, head=True),
        # A server that decodes 32 sequences at once, the largest batch of the small-batch path.
        _step("step_8b_b32", "8b", 32, 32, chain=False, head=True),
        # Eight sequences through real blocks (four of them: the others repeat the same shapes).
        _step("chain_8b_b8", "8b", 4, 8, chain=True),
        # Four sequences with one activation scale per 32 inputs, the paper's own granularity;
        # three quarters of the blocks W4A8.
        _step("chain_3b_b4_group32", "3b", 4, 4, chain=True, act_group=32, share=0.25),
        # The smallest call: one 2048 x 2048 layer, one token (launch and latency count).
        _linear("linear_2048_w4a16_b1", 2048, 2048, 1, "w4a16"),
        # One layer by itself for a batch: the 3B down projection with its quantisation.
        _linear("linear_3b_down_w4a8_b16", 3072, 8192, 16, "w4a8", out="bfloat16"),
        # Odd sizes: rows and inputs that fill no tile, five tokens.
        _linear("linear_ragged_w4a16_b5", 4099, 2720, 5, "w4a16"),
        # A long prompt through an 8B block, the largest work here.
        _prefill("prefill_8b_4096", "8b", 4096),
        # A prompt of an ordinary length that fills no tile, 3B.
        _prefill("prefill_3b_333", "3b", 333),
        # A short question to the smallest model.
        _prefill("prefill_1b_48", "1b", 48),
        # Loading: the 8B gate projection from fp32 to packed codes, and to bf16 from those.
        dict(name="load_8b_gate", kind="load", N=14336, K=4096),
    ]


def _log(rng, lo, hi):
    return int(round(lo * (hi / lo) ** rng.random()))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "linear", "linear", "prefill", "prefill", "load"])
    if kind == "step":
        if rng.random() < 0.5:
            hidden, kv, ffn, _ = SHAPES[rng.choice(["1b", "3b", "8b"])]
        else:
            # a step's widths: whole 128s as models have them, now and then only whole 32s
            unit = rng.choice([128, 128, 32])
            hidden = unit * max(1, round(_log(rng, 512, 4096) / unit))
            kv = max(32, hidden // 4 // 32 * 32)
            ffn = unit * max(1, round(hidden * rng.uniform(2.5, 3.5) / unit))
        return dict(kind="step", hidden=hidden, kv=kv, ffn=ffn,
                    vocab=rng.choice([0, 0, _log(rng, 8000, 64000)]), blocks=rng.randint(2, 6),
                    tokens=rng.choice([1, 1, _log(rng, 2, 32), _log(rng, 2, 32), rng.randint(2, 32)]),
                    chain=rng.random() < 0.6, act_group=rng.choice([0, 0, 0, 32]),
                    w4a16_share=rng.choice([0.0, 0.25, 0.5, 1.0]))
    if kind == "linear":
        return dict(kind="linear", N=_log(rng, 256, 32768), K=GROUP * _log(rng, 16, 448),
                    tokens=rng.choice([1, _log(rng, 2, 32), rng.randint(2, 32)]),
                    precision=rng.choice(["w4a8", "w4a16"]), act_group=rng.choice([0, 0, 0, 32]),
                    out=rng.choice(["float32", "bfloat16"]))
    if kind == "prefill":
        hidden, kv, ffn, _ = SHAPES[rng.choice(["1b", "3b", "8b"])]
        if rng.random() < 0.4:
            hidden = 64 * _log(rng, 12, 64)
            kv, ffn = max(32, hidden // 4 // 32 * 32), GROUP * round(hidden * rng.uniform(2.5, 3.5) / GROUP)
        return dict(kind="prefill", hidden=hidden, kv=kv, ffn=ffn, tokens=_log(rng, 33, 4096))
    return dict(kind="load", N=_log(rng, 256, 16384), K=GROUP * _log(rng, 32, 448))


# ---- inputs -------------------------------------------------------------------
def _gen(*key):
    seed = 0
    for k in key:
        seed = (seed * 1000003 + int(k) + 12345) % (1 << 62)
    return torch.Generator(device=DEV).manual_seed(seed)


def _dense(gen, N, K):
    return torch.randn((N, K), generator=gen, device=DEV, dtype=torch.float32).mul_(0.02)


def _codes(gen, N, K):
    """A weight matrix as signed 4-bit codes (int8 [N, K/32, 32]) and fp16 scales [N, K/32]."""
    w = _dense(gen, N, K).view(N, K // GROUP, GROUP)
    s = (w.abs().amax(2) / 7.0).to(torch.float16)
    c = w.div_(s.float().unsqueeze(2)).round_().clamp_(-8, 7).to(torch.int8)
    return c, s


def _packed(gen, N, K):
    """The same in the library's layout: a byte holds input j of its group (low half) and j + 16."""
    c, s = _codes(gen, N, K)
    b = (c + 8).view(torch.uint8)
    q = b[:, :, :16] | (b[:, :, 16:] << 4)
    return q.reshape(N, K // 2), s.view(torch.int16)


def _activation(gen, M, K):
    x = torch.randn((M, K), generator=gen, device=DEV, dtype=torch.float32)
    loud = torch.randperm(K, generator=gen, device=DEV)[:K // 100]
    x[:, loud] *= 20.0
    return x.to(torch.bfloat16)


def _gamma(gen, K):
    return (1.0 + 0.1 * torch.randn(K, generator=gen, device=DEV)).to(torch.bfloat16)


def _map(case, seed):
    """Per block: True = W4A16."""
    n = case["blocks"]
    order = torch.randperm(n, generator=torch.Generator().manual_seed(seed + 77)).tolist()
    wide = set(order[:round(case["w4a16_share"] * n)])
    return [b in wide for b in range(n)]


def _block_shapes(case):
    """(N, K) of q, k, v, o, gate, up, down."""
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    return [(h, h), (kv, h), (kv, h), (h, h), (f, h), (f, h), (h, f)]


_PHASE = (0, 0, 0, 1, 2, 2, 3)  # layers of a block that read the same input


def _weight_seed(case, seed, block, slot):
    return _gen(seed, 1, block, slot)


def _step_layers(case, seed):
    """The layers of a step: (block, slot, N, K, W4A16?); block = blocks is the vocabulary
    projection."""
    wide = _map(case, seed)
    out = [(b, i, N, K, wide[b]) for b in range(case["blocks"])
           for i, (N, K) in enumerate(_block_shapes(case))]
    if case["vocab"]:
        out.append((case["blocks"], 0, case["vocab"], case["hidden"], True))
    return out


def _step_inputs(case, seed):
    """What a step reads besides weights: x[block, phase] (independent), or the residual stream,
    the attention results and the norm weights (chain)."""
    M, h = case["tokens"], case["hidden"]
    widths = (h, h, h, case["ffn"])
    if not case["chain"]:
        x = {(b, p): _activation(_gen(seed, 2, b, p), M, widths[p])
             for b in range(case["blocks"]) for p in range(4)}
        if case["vocab"]:
            x[case["blocks"], 0] = _activation(_gen(seed, 2, case["blocks"], 0), M, h)
        return dict(x=x)
    n = case["blocks"]
    return dict(h=_activation(_gen(seed, 3), M, h),
                attn=[_activation(_gen(seed, 4, b), M, h) for b in range(n)],
                gamma=[(_gamma(_gen(seed, 5, b, 0), h), _gamma(_gen(seed, 5, b, 1), h))
                       for b in range(n)],
                gamma_head=_gamma(_gen(seed, 5, n), h))


def _prepare_step(case, seed):
    M, n = case["tokens"], case["blocks"]
    inp = _step_inputs(case, seed)
    entries = []
    # results: one tensor per projection, [block, token, row]; the residual sums; the logits
    dt = torch.bfloat16 if case["chain"] else torch.float32
    ys = [torch.zeros((n, M, N), dtype=dt, device=DEV) for N, _ in _block_shapes(case)]
    logits = torch.zeros((M, case["vocab"]), dtype=torch.float32, device=DEV)
    sums = torch.zeros((2 * n, M, case["hidden"]), dtype=torch.bfloat16, device=DEV)
    nsums = 0
    cur, down = inp.get("h"), None
    norm = None  # the entry fields that q, k, v (or gate, up) of a block share
    for b, i, N, K, wide in _step_layers(case, seed):
        q, s = _packed(_weight_seed(case, seed, b, i), N, K)
        e = dict(qweight=q, scales=s, precision=nvq.W4A16 if wide else nvq.W4A8,
                 y=ys[i][b] if b < n else logits)
        if not case["chain"]:
            e.update(x=inp["x"][b, _PHASE[i] if b < n else 0])
        elif b == n or i in (0, 4):  # a norm comes first: it also adds what the last layer gave
            g = inp["gamma_head"] if b == n else inp["gamma"][b][0 if i == 0 else 1]
            norm = dict(x=cur, in_op=nvq.IN_RMSNORM, gamma=g, eps=EPS)
            add = ys[3][b] if b < n and i == 4 else down
            if add is not None:
                cur = sums[nsums]
                nsums += 1
                norm.update(x2=add, h_out=cur)
            e.update(norm)
        elif i in (1, 2, 5):
            e.update(norm)
        elif i == 3:
            e.update(x=inp["attn"][b])
        else:
            down = ys[6][b]
            e.update(x=ys[4][b], x2=ys[5][b], in_op=nvq.IN_SILU_MUL)
        entries.append(e)
    dl = nvq.DecodeList(entries, M, case["act_group"])
    dl.plan()
    out = ys + ([logits] if case["vocab"] else []) + ([sums[:nsums]] if nsums else [])
    return dict(case=case, list=dl, out=out)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "step":
        return _prepare_step(case, seed)
    if kind == "linear":
        M, N, K = case["tokens"], case["N"], case["K"]
        q, s = _packed(_gen(seed, 1), N, K)
        x = _activation(_gen(seed, 2), M, K)
        y = torch.empty((M, N), dtype=getattr(torch, case["out"]), device=DEV)
        st = dict(case=case, q=q, s=s, x=x, y=y)
        if case["precision"] == "w4a8":
            G = K // GROUP
            st["codes"] = (torch.empty((M, K), dtype=torch.int8, device=DEV),
                           torch.empty((M,) if case["act_group"] == 0 else (M, G),
                                       dtype=torch.float32, device=DEV),
                           torch.empty((M, G), dtype=torch.int32, device=DEV))
        return st
    if kind == "prefill":
        T = case["tokens"]
        mats = []
        for p, (N, K) in enumerate(_prefill_shapes(case)):
            q, s = _packed(_gen(seed, 1, p), N, K)
            mats.append((q, s, _activation(_gen(seed, 2, p), T, K),
                         torch.empty((T, N), dtype=torch.bfloat16, device=DEV)))
        return dict(case=case, mats=mats)
    N, K = case["N"], case["K"]
    return dict(case=case, W=_dense(_gen(seed, 1), N, K),
                bf16=torch.empty((N, K), dtype=torch.bfloat16, device=DEV))


def _prefill_shapes(case):
    """(N, K) of q+k+v, o, gate+up, down."""
    h, kv, f = case["hidden"], case["kv"], case["ffn"]
    return [(h + 2 * kv, h), (h, h), (2 * f, h), (h, f)]


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "step":
        state["list"].run_plan()
        return state["out"]
    if kind == "linear":
        if case["precision"] == "w4a16":
            return [nvq.gemv_w4a16(state["q"], state["s"], state["x"], out=state["y"])]
        xq, xs, gs = nvq.quant_act_i8(state["x"], case["act_group"], out=state["codes"])
        y = nvq.gemv_w4a8(state["q"], state["s"], xq, xs, gs, case["act_group"], out=state["y"])
        return [y, xq, xs, gs]
    if kind == "prefill":
        return [nvq.gemm_w4a16(q, s, x, out=y) for q, s, x, y in state["mats"]]
    q, s = nvq.pack_int4(state["W"])
    return [q, s, nvq.dequant_bf16_into(q, s, state["bf16"])]


# ---- what a pass cannot do without ---------------------------------------------
def _weight_bytes(N, K):
    return N * K // 2 + N * (K // GROUP) * 2


def work(case):
    kind = case["kind"]
    if kind == "step":
        M = case["tokens"]
        layers = _step_layers(case, 0)
        b = sum(_weight_bytes(N, K) for _, _, N, K, _ in layers)
        f = sum(2 * M * N * K for _, _, N, K, _ in layers)
        h, ffn, n = case["hidden"], case["ffn"], case["blocks"]
        if case["chain"]:
            # inputs from outside, every output once, the residual sums
            b += 2 * M * (h + n * h) + 2 * h * (2 * n + 1)
            b += sum(2 * M * N for blk, _, N, _, _ in layers if blk < n) + 2 * M * h * (2 * n - 1)
            b += 4 * M * case["vocab"] + (2 * M * h if case["vocab"] else 0)
        else:
            b += 2 * M * (n * (3 * h + ffn) + (h if case["vocab"] else 0))
            b += sum(4 * M * N for _, _, N, _, _ in layers)
        return dict(bytes=b, flops=f)
    if kind == "linear":
        M, N, K = case["tokens"], case["N"], case["K"]
        b = _weight_bytes(N, K) + 2 * M * K + M * N * (4 if case["out"] == "float32" else 2)
        if case["precision"] == "w4a8":  # the codes are results too
            b += M * K + 4 * M * (K // GROUP) + 4 * M * (1 if case["act_group"] == 0 else K // GROUP)
        return dict(bytes=b, flops=2 * M * N * K)
    if kind == "prefill":
        T = case["tokens"]
        sh = _prefill_shapes(case)
        return dict(bytes=sum(_weight_bytes(N, K) + 2 * T * K + 2 * T * N for N, K in sh),
                    flops=sum(2 * T * N * K for N, K in sh))
    N, K = case["N"], case["K"]
    return dict(bytes=4 * N * K + _weight_bytes(N, K) + 2 * N * K, flops=2 * N * K)


def tolerance(case):
    kind = case["kind"]
    if kind == "load":
        return "exact"
    if kind == "prefill":
        return {"rel": 4e-3, "max": 2e-2}  # bf16 results
    if kind == "linear":
        if case["out"] == "bfloat16":
            return {"rel": 4e-3, "max": 2e-2}
        return {"rel": 1e-5, "max": 1e-3}
    if case["chain"]:
        return {"rel": 3e-2, "max": 0.9}  # bf16 from layer to layer, int8 codes that flip with it
    return {"rel": 1e-5, "max": 1e-3}


# ---- the same in 64 bits ---------------------------------------------------------
def _quantised(x, act_group):
    """The int8 quantisation of bf16 activations as it is defined (binary32 division, half to
    even), on the CPU: codes, scales, code sums per 32."""
    f = x.cpu().float()
    M, K = f.shape
    rows = f.view(M, K // GROUP, GROUP) if act_group else f.view(M, 1, K)
    s = rows.abs().amax(2) / 127.0
    d = torch.where(s > 0, s, torch.ones_like(s)).unsqueeze(2)
    q = (rows / d).round().clamp(-127, 127) * (s > 0).unsqueeze(2)
    q = q.view(M, K).to(torch.int8)
    return q, s.view(M) if act_group == 0 else s, q.view(M, K // GROUP, GROUP).to(torch.int32).sum(2, dtype=torch.int32)


def _product(x64, codes, scales, bf16_weights=False):
    """x64 [M, K] times the dequantised weights, in float64, some rows at a time."""
    N, G = scales.shape
    out = []
    rows = max(1, (1 << 27) // (G * GROUP))
    for r in range(0, N, rows):
        w = codes[r:r + rows].double() * scales[r:r + rows].double().unsqueeze(2)
        if bf16_weights:
            w = w.float().to(torch.bfloat16).double()
        out.append(x64 @ w.view(-1, G * GROUP).t())
    return torch.cat(out, 1)


def _layer(x, c, s, wide, act_group):
    """One layer in float64 from bf16 activations."""
    if wide:
        return _product(x.double(), c, s)
    q, xs, _ = _quantised(x, act_group)
    M, K = q.shape
    xs = xs.double().view(M, -1, 1)
    return _product((q.double().view(M, xs.shape[1], -1) * xs).view(M, K).to(DEV), c, s)


def _norm(x, add, gamma):
    h = x if add is None else (x.double() + add.double()).to(torch.bfloat16)
    d = h.double()
    r = 1.0 / torch.sqrt((d * d).mean(1, keepdim=True) + EPS)
    return h, (d * r * gamma.double()).to(torch.bfloat16)


def _exact_step(case, seed):
    n, ag = case["blocks"], case["act_group"]
    inp = _step_inputs(case, seed)
    ys, logits, hs = [[] for _ in range(7)], [], []
    cur, down, o_out, gate, x = inp.get("h"), None, None, None, None
    for b, i, N, K, wide in _step_layers(case, seed):
        c, s = _codes(_weight_seed(case, seed, b, i), N, K)
        if not case["chain"]:
            y64 = _layer(inp["x"][b, _PHASE[i] if b < n else 0], c, s, wide, ag)
            (ys[i] if b < n else logits).append(y64)
            continue
        if b == n or i in (0, 4):
            g = inp["gamma_head"] if b == n else inp["gamma"][b][0 if i == 0 else 1]
            add = o_out if b < n and i == 4 else down
            cur, x = _norm(cur, add, g)
            if add is not None:
                hs.append(cur.double())
        elif i == 3:
            x = inp["attn"][b]
        elif i == 6:
            g64 = gate.double()
            x = (g64 / (1.0 + torch.exp(-g64)) * y.double()).to(torch.bfloat16)
        y64 = _layer(x, c, s, wide, ag)
        y = y64.to(torch.bfloat16)
        if i == 3:
            o_out = y
        elif i == 4:
            gate = y
        elif i == 6:
            down = y
        (ys[i] if b < n else logits).append(y64)
    return [torch.stack(y) for y in ys] + logits + ([torch.stack(hs)] if hs else [])


def exact(case, seed):
    kind = case["kind"]
    if kind == "step":
        return _exact_step(case, seed)
    if kind == "linear":
        N, K, M = case["N"], case["K"], case["tokens"]
        c, s = _codes(_gen(seed, 1), N, K)
        x = _activation(_gen(seed, 2), M, K)
        if case["precision"] == "w4a16":
            return [_layer(x, c, s, True, 0)]
        q, xs, gs = _quantised(x, case["act_group"])
        return [_layer(x, c, s, False, case["act_group"]), q, xs.double(), gs]
    if kind == "prefill":
        out = []
        for p, (N, K) in enumerate(_prefill_shapes(case)):
            c, s = _codes(_gen(seed, 1, p), N, K)
            x = _activation(_gen(seed, 2, p), case["tokens"], K)
            out.append(_product(x.double(), c, s, bf16_weights=True))
        return out
    N, K = case["N"], case["K"]
    c, s = _codes(_gen(seed, 1), N, K)
    q, _ = _packed(_gen(seed, 1), N, K)
    w = (c.double() * s.double().unsqueeze(2)).view(N, K)
    return [q, s.view(torch.int16), w]

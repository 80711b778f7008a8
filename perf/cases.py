"""Performance cases of the W4/W2-GateUp MLP library: what a serving program
has it do, through the package's entry points.

The kinds of work, and who does them:

* ``forward``  -- one block per call, binary16, 1 to 16 tokens (an engine that
  runs its own attention between the MLPs), and bfloat16 prompt chunks of a
  multiple of 128 tokens (prefill);
* ``layers``   -- a batch of independent blocks in one call, 1 to 16 tokens;
* ``stack``    -- the blocks of a decoder on a residual stream;
* ``moe``      -- one mixture-of-experts layer, routing on the device;
* ``linear``   -- the other quantized linears (attention projections, LM head);
* ``pack``     -- quantizing a block's fp32 weights when a model is loaded.

The code widths are those the library takes in earnest: 2-bit gate/up with a
4-bit down (groups 64 and 128, and 2-bit group 32, the grouping of the
method's paper), the 3-bit gate/up variant and uniform 4 and 2 bits.
Weights are N(0, 0.02), adapters A ~ N(0, 0.02) and B ~ N(0, 0.002),
activations N(0, 1), as in the benchmark's workloads.
"""
import math

import torch

import paper_2606_04238_amd as q

DEV = "cuda"


def _case(kind, name=None, M=1, d=2560, f=9728, L=1, r=16, gb=2, gg=128, db=4, dg=128, bf16=False,
          E=0, k=0):
    c = dict(kind=kind, M=M, d=d, f=f, L=L, r=r, gb=gb, gg=gg, db=db, dg=dg, bf16=bf16, E=E, k=k)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the smallest block of the test workloads, one token: launch and hand-off latency
        _case("forward", "block_tiny_m1", M=1, d=512, f=1536, r=8, gg=64, dg=64),
        # one Qwen3-4B-shaped block per call, one token: an engine's MLP step at batch 1
        _case("forward", "block_4b_m1"),
        # one Qwen3-8B-shaped block per call, eight sequences decoding together
        _case("forward", "block_8b_m8", M=8, d=4096, f=12288, r=32),
        # the benchmark's headline: 36 Qwen3-4B-shaped blocks in one call, one token
        _case("layers", "layers_4b_m1", L=36),
        # the same at Qwen3-8B shape and a full decode batch of 16 tokens
        _case("layers", "layers_8b_m16", M=16, d=4096, f=12288, L=36, r=32),
        # the paper's own INT2 grouping (32) at an odd small batch
        _case("layers", "layers_4b_g32_m5", M=5, L=36, gg=32),
        # the dependent form: 36 blocks on a residual stream, one token
        _case("stack", "stack_4b_m1", L=36),
        # the benchmark's prompt chunk: 512 tokens of the 20B-class block, bfloat16
        _case("forward", "prefill_20b_m512", M=512, d=6144, f=16384, r=32, bf16=True),
        # a short prompt chunk on the 4B shape
        _case("forward", "prefill_4b_m256", M=256, bf16=True),
        # one GPT-OSS-20B-class MoE layer, top-4 of 32 experts, eight tokens
        # (hidden and expert width 2880: no multiple of 128)
        _case("moe", "moe_20b_m8", M=8, d=2880, f=2880, gg=64, dg=64, E=32, k=4),
        # the Qwen3-4B LM head at four tokens
        _case("linear", "lm_head_4b_m4", M=4, d=2560, f=151936, r=0),
        # loading: one Qwen3-8B block's gate, up (2 bits) and down (4 bits) from fp32
        _case("pack", "pack_8b", d=4096, f=12288, r=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _size(rng, lo, hi, mult):
    return max(lo // mult, min(hi // mult, _log_int(rng, lo, hi) // mult)) * mult


def draw(rng):
    kind = rng.choice(["forward", "layers", "stack", "moe", "linear", "pack", "prefill"])
    # code widths: mostly the W4/W2-GateUp block, else one of the others
    gb, gg, db, dg = rng.choice([(2, 128, 4, 128), (2, 64, 4, 64), (2, 64, 4, 128), (2, 32, 4, 128),
                                 (3, 32, 4, 128), (4, 128, 4, 128), (2, 128, 2, 128), (4, 32, 4, 32)])
    r = rng.choice([0, 8, 16, 32])
    M = rng.choice([1, 1, 2, 3, 4, 6, 7, 8, 11, 13, 16])
    # half of the widths are multiples of 512 (as most models'), half any that the groups divide
    step = 512 if rng.random() < 0.5 else 128 if 128 in (gg, dg) or gb == 3 else 64
    d, f = _size(rng, 512, 5120, step), _size(rng, 1024, 17408, step)
    if kind == "prefill":
        gb, gg, db, dg = rng.choice([(2, 128, 4, 128), (2, 64, 4, 64)])
        d, f = _size(rng, 1024, 6144, 128), _size(rng, 2048, 16384, 128)
        M = min(_size(rng, 128, 2048, 128), max(128, 512 * 6144 * 16384 // (d * f) // 128 * 128))
        return _case("forward", M=M, d=d, f=f, r=r, gb=gb, gg=gg, db=db, dg=dg, bf16=True)
    if kind in ("layers", "stack"):
        L = min(_log_int(rng, 2, 40), max(1, 36 * 4096 * 12288 // (d * f)))
        return _case(kind, M=M, d=d, f=f, L=L, r=r, gb=gb, gg=gg, db=db, dg=dg)
    if kind == "moe":
        E = rng.choice([8, 16, 32, 40])
        k = rng.choice([1, 2, 4, 4, 6])
        d, f = _size(rng, 512, 4096, step), _size(rng, 512, 4096, step)
        return _case("moe", M=min(16, max(1, _log_int(rng, 1, 40 // k))), d=d, f=f, r=r, gb=gb, gg=gg, db=db,
                     dg=dg, E=E, k=k)
    if kind == "linear":
        L = rng.choice([1, 1, 4, 36])
        f = _size(rng, 1024, 151936 if L == 1 else 8192, 128)
        return _case("linear", M=M, d=d, f=f, L=L, r=0, db=db, dg=dg)
    return _case(kind, M=M, d=d, f=f, r=r if kind == "forward" else 0, gb=gb, gg=gg, db=db, dg=dg)


# ---------------------------------------------------------------- inputs, from the seed alone

def _gen(seed, *ids):
    s = seed
    for i in ids:
        s = (s * 1000003 + i + 1) % (1 << 62)
    return torch.Generator(device=DEV).manual_seed(s)


def _act(c):
    return torch.bfloat16 if c["bf16"] else torch.float16


def _weights(c, seed, l):
    """fp32 W_gate [f][d], W_up [f][d], W_down [d][f] of block l."""
    g = _gen(seed, l)
    return tuple(0.02 * torch.randn(s, generator=g, device=DEV)
                 for s in ((c["f"], c["d"]), (c["f"], c["d"]), (c["d"], c["f"])))


def _adapters(c, seed, l):
    """A_gate, B_gate, A_up, B_up of block l in the activation type."""
    if c["r"] == 0:
        return (None,) * 4
    g = _gen(seed, l, 1)
    return tuple((sd * torch.randn(s, generator=g, device=DEV)).to(_act(c))
                 for s, sd in (((c["r"], c["d"]), 0.02), ((c["f"], c["r"]), 0.002)) * 2)


def _x(c, seed, *shape):
    return torch.randn(shape, generator=_gen(seed, -7), device=DEV).to(_act(c))


def _routing(c, seed):
    g = _gen(seed, -9)
    order = torch.rand((c["M"], c["E"]), generator=g, device=DEV).argsort(1)
    w = torch.softmax(torch.randn((c["M"], c["k"]), generator=g, device=DEV), 1)
    return order[:, :c["k"]].to(torch.int32).contiguous(), w


def _linear_weight(c, seed, l):
    return 0.02 * torch.randn((c["f"], c["d"]), generator=_gen(seed, l), device=DEV)


_PACK = {2: "pack_w2", 3: "pack_w3", 4: "pack_w4"}


def _pack(bits, W, group):
    return getattr(q, _PACK[bits])(W, group)


def _mlp(c, seed, l):
    Wg, Wu, Wd = _weights(c, seed, l)
    return q.MLP(_pack(c["gb"], Wg, c["gg"]), _pack(c["gb"], Wu, c["gg"]), _pack(c["db"], Wd, c["dg"]),
                 *_adapters(c, seed, l))


def prepare(case, seed):
    c, kind = case, case["kind"]
    M, d, L, t = c["M"], c["d"], c["L"], _act(case)
    if kind == "pack":
        return dict(c=c, W=_weights(c, seed, 0))
    if kind == "linear":
        return dict(c=c, w=[_pack(c["db"], _linear_weight(c, seed, l), c["dg"]) for l in range(L)],
                    x=_x(c, seed, L, M, d), y=torch.empty((L, M, c["f"]), dtype=t, device=DEV))
    if kind == "forward":
        m = _mlp(c, seed, 0)
        return dict(c=c, m=m, x=_x(c, seed, M, d), y=torch.empty((M, d), dtype=t, device=DEV),
                    ws=q.workspace(m, M, t))
    blocks = [_mlp(c, seed, l) for l in range(c["E"] if kind == "moe" else L)]
    if kind == "moe":
        m = q.Layers(blocks)
        idx, w = _routing(c, seed)
        return dict(c=c, m=m, x=_x(c, seed, M, d), idx=idx, w=w, y=torch.empty((M, d), dtype=t, device=DEV),
                    ws=torch.zeros(q.moe_workspace_bytes(m, M, c["k"]), dtype=torch.uint8, device=DEV))
    y = torch.empty((L, M, d), dtype=t, device=DEV)
    if kind == "stack":
        m = q.Stack(blocks)
        return dict(c=c, m=m, x=_x(c, seed, M, d), y=y, x_out=torch.empty((M, d), dtype=t, device=DEV),
                    ws=q.stack_workspace(m, M))
    m = q.Layers(blocks)
    return dict(c=c, m=m, x=_x(c, seed, L, M, d), y=y, ws=q.layers_workspace(m, M))


def run(state):
    s, c = state, state["c"]
    kind = c["kind"]
    if kind == "forward":
        return q.forward(s["m"], s["x"], s["y"], s["ws"])
    if kind == "layers":
        return q.forward_layers(s["m"], s["x"], s["y"], s["ws"])
    if kind == "stack":
        return q.forward_stack(s["m"], s["x"], s["y"], s["ws"], s["x_out"]), s["x_out"]
    if kind == "moe":
        return q.forward_moe(s["m"], s["x"], s["idx"], s["w"], s["y"], s["ws"])
    if kind == "linear":
        return q.linear_batch(s["w"], s["x"], s["y"])
    Wg, Wu, Wd = s["W"]
    out = [_pack(c["gb"], Wg, c["gg"]), _pack(c["gb"], Wu, c["gg"]), _pack(c["db"], Wd, c["dg"])]
    return [t for w in out for t in (w.codes, w.meta)]


# ---------------------------------------------------------------- what a pass cannot do without

def _wbytes(n, k, bits, g):
    return n * k * bits // 8 + n * (k // g) * 4


def work(case):
    c = case
    M, d, f, L, r = c["M"], c["d"], c["f"], c["L"], c["r"]
    if c["kind"] == "pack":
        out = 2 * _wbytes(f, d, c["gb"], c["gg"]) + _wbytes(d, f, c["db"], c["dg"])
        return {"bytes": 3 * 4 * f * d + out, "flops": 0}
    if c["kind"] == "linear":
        return {"bytes": L * (_wbytes(f, d, c["db"], c["dg"]) + 2 * M * (d + f)), "flops": 2 * L * M * f * d}
    block = 2 * _wbytes(f, d, c["gb"], c["gg"]) + _wbytes(d, f, c["db"], c["dg"]) + 4 * r * (d + f)
    flops = 6 * M * f * d + 4 * M * r * (d + f)
    if c["kind"] == "moe":
        # every token's k experts; experts that several tokens choose are read once (expected number
        # of distinct experts under the uniform routing of the inputs)
        n = c["E"] * (1.0 - (1.0 - c["k"] / c["E"]) ** M)
        return {"bytes": int(n * block) + 4 * M * d + 8 * M * c["k"], "flops": c["k"] * flops}
    io = 4 * M * d if c["kind"] != "stack" else 2 * M * d
    return {"bytes": L * (block + io) + (4 * M * d if c["kind"] == "stack" else 0), "flops": L * flops}


def tolerance(case):
    if case["kind"] == "pack":
        return "exact"
    # about four times the error measured against 64 bits: 3.0e-4 in binary16 (h and y are rounded to it, sums
    # are 32 bits), 4.0e-3 for the bfloat16 chunks; a stack carries one block's rounding through those that
    # follow (36 Qwen3-4B-shaped blocks: 2.8e-3, largest difference 1.6e-2)
    if case["bf16"]:
        return {"rel": 1.6e-2, "max": 0.08}
    if case["kind"] == "stack":
        return {"rel": 1.1e-2, "max": 0.065}
    return {"rel": 1.2e-3, "max": 5e-3}


# ---------------------------------------------------------------- the same in 64 bits, plain torch

def _half(s):
    """Positive fp64 -> binary16, one rounding to nearest even (through fp32 rounded to odd)."""
    t = s.float()
    b = t.view(torch.int32)
    b = torch.where(t.double() > s, b - 1, b)
    b = torch.where(b.view(torch.float32).double() != s, b | 1, b)
    return b.view(torch.float32).half()


def _qdq(W, bits, g):
    """W quantized (round to nearest, min-max per group with 0 included) and back, fp64."""
    top = float((1 << bits) - 1)
    v = W.double().view(W.shape[0], -1, g)
    lo, hi = v.amin(2, keepdim=True).clamp(max=0), v.amax(2, keepdim=True).clamp(min=0)
    s = _half((hi - lo) / top).double()
    s = torch.where(s == 0, torch.ones_like(s), s)
    z = torch.round(-lo / s).clamp(0, top)
    return ((torch.round(v / s) + z).clamp(0, top) - z).mul_(s).view(W.shape)


def _block(c, seed, l, x):
    """y of block l for x [.][d], fp64."""
    Wg, Wu, Wd = _weights(c, seed, l)
    G, U = x @ _qdq(Wg, c["gb"], c["gg"]).T, x @ _qdq(Wu, c["gb"], c["gg"]).T
    Ag, Bg, Au, Bu = _adapters(c, seed, l)
    if Ag is not None:
        G += (x @ Ag.double().T) @ Bg.double().T
        U += (x @ Au.double().T) @ Bu.double().T
    return (G * torch.sigmoid(G) * U) @ _qdq(Wd, c["db"], c["dg"]).T


def exact(case, seed):
    c, kind = case, case["kind"]
    if kind == "pack":
        return None                                       # whole numbers
    if kind == "linear":
        x = _x(c, seed, c["L"], c["M"], c["d"]).double()
        return torch.stack([x[l] @ _qdq(_linear_weight(c, seed, l), c["db"], c["dg"]).T for l in range(c["L"])])
    if kind == "layers":
        x = _x(c, seed, c["L"], c["M"], c["d"]).double()
        return torch.stack([_block(c, seed, l, x[l]) for l in range(c["L"])])
    x = _x(c, seed, c["M"], c["d"]).double()
    if kind == "forward":
        return _block(c, seed, 0, x)
    if kind == "moe":
        idx, w = _routing(c, seed)
        y = torch.zeros_like(x)
        for e in idx.unique().tolist():
            m, j = (idx == e).nonzero(as_tuple=True)
            y[m] += w[m, j].double()[:, None] * _block(c, seed, e, x[m])
        return y
    ys = []
    for l in range(c["L"]):
        u = x / (x.square().mean(1, keepdim=True) + 1e-6).sqrt()
        ys.append(_block(c, seed, l, u))
        x = x + ys[-1]
    return torch.stack(ys), x

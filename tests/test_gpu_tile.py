"""The matrix-core tile kernels at several tokens, against the oracle: every
group and width they take, rows that are no whole number of steps, K slices,
tiles side by side, batches whose ranges straddle blocks, and each adapter
rank.  Bars as for the other decode paths: y and h are binary16, sums fp32."""
import numpy as np
import pytest
import torch

import oracle as orc
import workloads as wl
from qmlp_testutil import act_tensor, values_of

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def q():
    import paper_2606_04238_amd as q
    return q


def _pack(q, W, bits, g):
    return {2: q.pack_w2, 3: q.pack_w3, 4: q.pack_w4}[bits](torch.from_numpy(W).cuda(), g)


def _block(q, cfg, l, gb, gg, db, dg):
    L = wl.layer(cfg, l)
    lo = (L.A_gate, L.B_gate, L.A_up, L.B_up) if cfg.r else (None,) * 4
    m = q.MLP(_pack(q, L.W_gate, gb, gg), _pack(q, L.W_up, gb, gg), _pack(q, L.W_down, db, dg),
              *(act_tensor(t) if t is not None else None for t in lo), lora_scale=0.75)

    def ref(x):
        return orc.forward(orc.quantize(L.W_gate, gb, gg), orc.quantize(L.W_up, gb, gg),
                           orc.quantize(L.W_down, db, dg), *lo, x, lora_scale=0.75)
    return m, L.x, ref


SHAPES = [  # d, f, gate bits, group, down bits, group, rank
    (512, 1024, 2, 64, 4, 64, 8),          # one step per row: tiles side by side
    (2880, 2880, 2, 64, 4, 64, 16),        # ragged last steps (d and f)
    (2560, 1280, 2, 32, 4, 128, 16),       # 2-bit group 32
    (1344, 448, 2, 32, 4, 32, 32),         # ragged, 4-bit group 32
    (4160, 640, 2, 64, 4, 128, 32),        # nine steps: gate and up in turn
    (2304, 6656, 4, 128, 4, 128, 0),       # uniform 4 bits, two K slices, no adapters
    (1152, 7040, 4, 32, 2, 128, 16),       # 4-bit group 32 gate/up, 2-bit down in two slices
    (640, 13312, 2, 128, 2, 64, 8),        # three K slices at 2 bits
    (1280, 3200, 3, 32, 4, 64, 8),         # 3-bit gate/up (stand-alone) with a tile down
    (1024, 4608, 2, 32, 4, 128, 16),       # gate/up stand-alone at two tokens only; packed down
    (512, 4672, 2, 64, 4, 64, 0),          # ragged packed down of nineteen steps, no adapters
    (2048, 448, 2, 64, 2, 64, 8),          # one-step down: stand-alone at two tokens only
]


@pytest.mark.parametrize("M", [2, 3, 5, 8, 16])
@pytest.mark.parametrize("shape", SHAPES)
def test_forward_matches_oracle(q, shape, M):
    d, f, gb, gg, db, dg, r = shape
    print("tile forward", shape, "M", M, flush=True)
    cfg = wl.Config("tile", M=M, d=d, f=f, g=gg, r=r, L=1)
    m, xb, ref = _block(q, cfg, 0, gb, gg, db, dg)
    x = act_tensor(xb)
    ws = q.workspace(m, M)
    y = q.forward(m, x, ws=ws)
    want = ref(xb)
    torch.cuda.synchronize()
    assert orc.max_rel_err(values_of(y), want) <= 1e-2
    assert float(np.linalg.norm(values_of(y) - want) / np.linalg.norm(want)) <= 1.2e-3
    again = q.forward(m, x, ws=ws)
    torch.cuda.synchronize()
    assert torch.equal(again, y)


@pytest.mark.parametrize("L", [2, 7, 43])
@pytest.mark.parametrize("shape", [SHAPES[1], SHAPES[3], SHAPES[7]])
def test_layers_match_blocks(q, shape, L):
    """A batch (ranges that straddle blocks, two batches at 43) against the
    oracle on sampled blocks and each block's own call on all of them."""
    d, f, gb, gg, db, dg, r = shape
    M = 6
    print("tile layers", shape, "L", L, flush=True)
    cfg = wl.Config("tile", M=M, d=d, f=f, g=gg, r=r, L=L)
    blocks = [_block(q, cfg, l, gb, gg, db, dg) for l in range(min(L, 3))]
    layers = q.Layers([blocks[l % len(blocks)][0] for l in range(L)])
    rng = np.random.default_rng(3)
    xb = rng.standard_normal((L, M, d)).astype(np.float16)
    x = torch.from_numpy(xb).cuda()
    ws = q.layers_workspace(layers, M)
    y = q.forward_layers(layers, x, ws=ws)
    torch.cuda.synchronize()
    for l in sorted({0, L // 2, L - 1}):
        want = blocks[l % len(blocks)][2](xb[l].view(np.uint16))
        assert orc.max_rel_err(values_of(y[l]), want) <= 1e-2
    for l in range(L):
        one = q.forward(layers.mlps[l], x[l])
        assert orc.max_rel_err(values_of(y[l]), values_of(one)) <= 2e-3
    assert torch.equal(q.forward_layers(layers, x, ws=ws), y)


@pytest.mark.parametrize("L,shape", [
    (12, (2048, 6144, 4, 128, 2, 64, 16)),    # whole steps, one K slice
    (9, (2880, 6272, 2, 64, 4, 64, 8)),       # ragged rows, two K slices
    (12, (2112, 6272, 4, 64, 2, 128, 0)),     # ragged rows, no adapters
])
def test_one_token_batches_match_blocks(q, L, shape):
    """Large one-token batches (1.5e8 weights per matrix and more) take the
    tile kernels, a block alone and a batch one block short do not."""
    d, f, gb, gg, db, dg, r = shape
    print("tile one token", shape, "L", L, flush=True)
    assert L * d * f >= 150000000 > (L - 1) * d * f
    cfg = wl.Config("tile", M=1, d=d, f=f, g=gg, r=r, L=2)
    blocks = [_block(q, cfg, l, gb, gg, db, dg) for l in range(2)]
    x = torch.from_numpy(np.random.default_rng(4).standard_normal((L, 1, d)).astype(np.float16)).cuda()
    layers = q.Layers([blocks[l % 2][0] for l in range(L)])
    ws = q.layers_workspace(layers, 1)
    y = q.forward_layers(layers, x, ws=ws)
    for l in (0, L - 1):
        want = blocks[l % 2][2](x[l].cpu().numpy().view(np.uint16))
        assert orc.max_rel_err(values_of(y[l]), want) <= 1e-2
    short = q.forward_layers(q.Layers([blocks[l % 2][0] for l in range(L - 1)]), x[:L - 1].contiguous())
    for l in range(L - 1):
        assert orc.max_rel_err(values_of(y[l]), values_of(short[l])) <= 2e-3
    assert torch.equal(q.forward_layers(layers, x, ws=ws), y)


@pytest.mark.parametrize("M", [2, 8, 9, 16])
@pytest.mark.parametrize("n,k,bits,g,L", [(64, 64, 4, 64, 1), (192, 320, 4, 32, 3), (1088, 2560, 4, 128, 5),
                                          (320, 4096, 2, 64, 2), (17408, 1024, 4, 128, 1), (128, 6144, 4, 64, 40),
                                          (192, 5888, 4, 128, 2), (4096, 4160, 4, 64, 1), (4160, 4160, 4, 64, 1),
                                          (1024, 512, 2, 128, 1), (1024, 512, 2, 64, 12)])
def test_linear_matches_oracle(q, n, k, bits, g, L, M):
    print("tile linear", n, k, bits, g, "L", L, "M", M, flush=True)
    rng = np.random.default_rng([n, k, M])
    Ws = [(0.02 * rng.standard_normal((n, k))).astype(np.float32) for _ in range(min(L, 2))]
    xb = rng.standard_normal((L, M, k)).astype(np.float16)
    qs = [_pack(q, W, bits, g) for W in Ws]
    y = q.linear_batch([qs[l % len(qs)] for l in range(L)], torch.from_numpy(xb).cuda())
    torch.cuda.synchronize()
    for l in sorted({0, L // 2, L - 1}):
        want = orc.down(orc.quantize(Ws[l % len(Ws)], bits, g), xb[l].astype(np.float64))
        assert orc.max_rel_err(values_of(y[l]), want) <= 2e-3


@pytest.mark.parametrize("M", [2, 3, 16])
@pytest.mark.parametrize("d,f,g,r", [(1024, 4608, 32, 16), (2048, 4224, 64, 8), (1344, 448, 32, 32)])
def test_gateup_alone_matches_oracle(q, d, f, g, r, M):
    """The half by itself: LoRA-A's slices lie where the workspace has its own
    h (the last shape's is too small for them: one slice), behind which it
    stays zero; more tiles than compute units go stand-alone at two tokens."""
    cfg = wl.Config("tile_gu", M=M, d=d, f=f, g=g, r=r, L=1)
    print("tile gateup alone", d, f, g, r, "M", M, flush=True)
    L = wl.layer(cfg, 0)
    m, xb, _ = _block(q, cfg, 0, 2, g, 4, 64)
    ws = q.workspace(m, M)
    h = q.gateup_w2_lora(m, act_tensor(xb), ws=ws)
    want = orc.gateup(orc.quantize(L.W_gate, 2, g), orc.quantize(L.W_up, 2, g), L.A_gate, L.B_gate, L.A_up, L.B_up,
                      xb, lora_scale=0.75)
    torch.cuda.synchronize()
    assert orc.max_rel_err(values_of(h), want) <= 2e-3
    r256 = lambda v: (v + 255) // 256 * 256
    assert not bool(ws[1024 + r256(M * 2 * r * 4) + r256(M * f * 2):].any())
    assert torch.equal(q.gateup_w2_lora(m, act_tensor(xb), ws=ws), h)


@pytest.mark.parametrize("M", [9, 16])
def test_slices_leave_the_workspace_clean(q, M):
    """Two slices of f: past t and h the workspace is zero after a call, so a
    workspace that serves other token counts (the one-kernel layer's hand-off
    words) never meets stale partial sums; and it does serve them."""
    cfg = wl.Config("tile_ws", M=M, d=1024, f=6656, g=128, r=16, L=1)
    print("tile workspace", M, flush=True)
    m, xb, ref = _block(q, cfg, 0, 2, 128, 4, 128)
    ws = q.workspace(m, M)
    want = ref(xb)
    r256 = lambda v: (v + 255) // 256 * 256
    head = 1024 + r256(M * 2 * cfg.r * 4) + r256(M * cfg.f * 2)
    for _ in range(2):
        y = q.forward(m, act_tensor(xb), ws=ws)
        torch.cuda.synchronize()
        assert orc.max_rel_err(values_of(y), want) <= 1e-2
        assert not bool(ws[head:].any())
    for k in (1, M, 4, 2, M):
        y = q.forward(m, act_tensor(xb[:k]), ws=ws)
        torch.cuda.synchronize()
        assert q.workspace_errors(ws) == 0
        assert orc.max_rel_err(values_of(y), want[:k]) <= 1e-2


@pytest.mark.parametrize("M", [8, 13, 16])
def test_partial_sums_get_their_workspace(q, M):
    """Three slices of f (12 steps of 256 codes a slice) of a wide block: their
    partials pass the hand-off words' bytes at 16 tokens, and the workspace
    has room for them.  The smaller one of the no-allocation entry point
    serves as well, on the stand-alone down kernel where they do not fit."""
    d, f, r = 4096, 9216, 16
    print("tile partials", M, flush=True)
    cfg = wl.Config("tile_parts", M=M, d=d, f=f, g=64, r=r, L=1)
    m, xb, ref = _block(q, cfg, 0, 2, 64, 4, 32)
    r256 = lambda v: (v + 255) // 256 * 256
    head = 1024 + r256(M * 2 * r * 4) + r256(M * f * 2)
    assert q.workspace_bytes(m, M) >= head + r256(4 * M * 2 * r * 4) + 1024 + (2 if M <= 8 else 3) * M * d * 4
    x = act_tensor(xb)
    ws = q.workspace(m, M)
    y = q.forward(m, x, ws=ws)
    want = ref(xb)
    torch.cuda.synchronize()
    assert orc.max_rel_err(values_of(y), want) <= 1e-2
    assert torch.equal(q.forward(m, x, ws=ws), y) and not bool(ws[head:].any())
    assert orc.max_rel_err(values_of(q.forward_noalloc(m, x)), want) <= 1e-2
    # what sufficed without them still does, for a block, its gate/up half and a stack
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    least = head + cus * 256 * 8 + r256(4 * f * 4)
    small = torch.zeros(least, dtype=torch.uint8, device="cuda")
    assert orc.max_rel_err(values_of(q.forward(m, x, ws=small)), want) <= 1e-2
    q.gateup_w2_lora(m, x, ws=small)
    with pytest.raises(q.QmlpError):
        q.forward(m, x, ws=small[:-256])
    st, more = q.Stack([m, m]), 3 * r256(M * d * 2)
    ref_y = q.forward_stack(st, x, ws=q.stack_workspace(st, M))
    some_y = q.forward_stack(st, x, ws=torch.zeros(least + more, dtype=torch.uint8, device="cuda"))
    assert orc.max_rel_err(values_of(some_y), values_of(ref_y)) <= 2e-3
    with pytest.raises(q.QmlpError):
        q.forward_stack(st, x, ws=torch.zeros(least + more - 256, dtype=torch.uint8, device="cuda"))


@pytest.mark.parametrize("d,f,gb,g,db,r,E,k,M,same", [
    (2048, 1600, 2, 64, 4, 16, 4, 4, 10, False),       # every expert shared by all tokens
    (1600, 2048, 2, 64, 4, 32, 5, 4, 10, True),        # all forty instances on one expert: three operands of rows
    (512, 6656, 2, 128, 4, 8, 6, 6, 6, False),         # two slices of f
    (2560, 1024, 4, 128, 4, 0, 4, 2, 16, False),       # uniform 4 bits, no adapters
])
def test_shared_experts_match_oracle(q, d, f, gb, g, db, r, E, k, M, same):
    """Routed layers whose experts are shared by enough tokens to run on the
    tile kernels (each expert in use read once)."""
    print("tile moe", d, f, E, k, M, flush=True)
    cfg = wl.Config("tile_moe", M=1, d=d, f=f, g=g, r=r, L=1)
    lays = [wl.layer(cfg, e) for e in range(E)]
    mlps = [_block(q, cfg, e, gb, g, db, g)[0] for e in range(E)]
    experts = q.Layers(mlps)
    x = wl.activations(cfg, 9, 0, M=M)
    idx, w = wl.routing(M, E, k, 1)
    if same:
        idx[:] = E - 2
    ws = torch.zeros(q.moe_workspace_bytes(experts, M, k), dtype=torch.uint8, device="cuda")
    # the tile kernels run: fp32 outputs of every slice of f (otherwise binary16 ones)
    n, sk, r256 = M * k, 2 if f > 6144 else 1, lambda v: (v + 255) // 256 * 256
    assert ws.numel() == 1024 + r256(2 * n * 2 * r * 4) + r256(n * f * 2) + r256(n * d * 4 * sk)
    ys = [q.forward_moe(experts, act_tensor(x), torch.from_numpy(idx).cuda(), torch.from_numpy(w).cuda(), ws=ws)
          for _ in range(2)]
    torch.cuda.synchronize()
    oq = [(orc.quantize(l.W_gate, gb, g), orc.quantize(l.W_up, gb, g), orc.quantize(l.W_down, db, g)) +
          ((l.A_gate, l.B_gate, l.A_up, l.B_up) if r else (None,) * 4) for l in lays]
    want = orc.moe_forward(oq, idx, w, x, lora_scale=0.75)
    assert orc.max_rel_err(values_of(ys[0]), want) <= 1e-2
    assert torch.equal(ys[0], ys[1])
    assert q.workspace_errors(ws) == 0 and int(ws[0:4].view(torch.int32).item()) == 2


# Small activations: the tile kernels scale an activation by up to 2^-s before
# it is rounded to binary16 (s = 2 for 4-bit codes, 4 for 2-bit ones), so below
# binary16's normal range it is off by at most 2^(s - 25), 2^(s - 25) /
# sqrt(3) in the mean; the weights, the sums and the zero-point term add
# nothing that counts, and the output is rounded to binary16 once (2^-11 /
# sqrt(3) in the mean).  At rms 2^-11 that is 1.4e-4 and 5.6e-4 of the
# activations (scaled by 2^-6 and 2^-8 they would be off by four and sixteen times as much).
SMALL = 2.0 ** -11


def _small_bar(bits, factor=1.0):
    return float(np.hypot(2.0 ** -11, factor * 2.0 ** ((2 if bits == 4 else 4) - 25) / SMALL) / np.sqrt(3.0))


@pytest.mark.parametrize("bits,g", [(4, 128), (4, 64), (4, 32), (2, 128), (2, 64)])
@pytest.mark.parametrize("packed,M", [(False, 2), (False, 9), (True, 8)])
def test_linear_small_activations(q, bits, g, packed, M):
    """One step per operand and two (rows past twelve waves' steps at up to
    eight tokens: two steps share an operand; 4-bit groups of 32 hold half
    as long a row, and longer ones run the stand-alone kernel)."""
    n, k = 256, (2560 if not packed else 5120 if (bits, g) == (4, 32) else 9216)
    print("tile small linear", n, k, bits, g, "M", M, flush=True)
    rng = np.random.default_rng([k, bits, g])
    W = (4.0 * rng.standard_normal((n, k))).astype(np.float32)      # outputs well inside binary16
    x = (SMALL * rng.standard_normal((1, M, k))).astype(np.float16)
    y = values_of(q.linear_batch([_pack(q, W, bits, g)], torch.from_numpy(x).cuda())[0])
    want = orc.down(orc.quantize(W, bits, g), x[0].astype(np.float64))
    assert np.linalg.norm(y - want) / np.linalg.norm(want) <= _small_bar(bits)


@pytest.mark.parametrize("bits,g", [(2, 128), (2, 64), (2, 32), (4, 128), (4, 64), (4, 32)])
@pytest.mark.parametrize("M", [5, 16])
def test_gateup_small_activations(q, bits, g, M):
    """G and U of rms about 1/2, so h is about G U / 2 and takes each sum's
    error once (in the mean sqrt(2) of it; 2 in the bar); the down weights pass h on as it is."""
    d, f = 2560, 512
    print("tile small gateup", bits, g, "M", M, flush=True)
    rng = np.random.default_rng([M, bits, g])
    Wg, Wu = ((20.0 * rng.standard_normal((f, d))).astype(np.float32) for _ in range(2))
    Wd = np.zeros((d, f), np.float32)                               # y[:f] = h: scale 1/15, code 15
    Wd[np.arange(f), np.arange(f)] = 1.0
    x = (SMALL * rng.standard_normal((M, d))).astype(np.float16)
    m = q.MLP(_pack(q, Wg, bits, g), _pack(q, Wu, bits, g), _pack(q, Wd, 4, 128), None, None, None, None)
    y = values_of(q.forward(m, torch.from_numpy(x).cuda()))
    want = orc.forward(orc.quantize(Wg, bits, g), orc.quantize(Wu, bits, g), orc.quantize(Wd, 4, 128),
                       None, None, None, None, x.view(np.uint16))
    # h is rounded to binary16 and its diagonal weight 15 s to the scale's: the oracle holds the same weight
    bar = float(np.hypot(2.0 ** -11 / np.sqrt(3.0), _small_bar(bits, 2.0)))
    assert np.linalg.norm(y - want) / np.linalg.norm(want) <= bar

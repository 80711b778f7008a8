"""The packer's fp32 quotient rounding and its wave-wide layout.

* CPU: rint(w / scale) as the packing kernel forms it in fp32 (a reciprocal,
  a remainder and a correction) against IEEE fp64 division and rint, on random
  quotients, exact ties and the neighbours of ties, over normal and subnormal
  binary16 scales.
* GPU: codes and metadata against the oracle where a wave's 1024 weights hold
  part of a group row, end past the matrix, or span many short rows."""
import numpy as np
import pytest
import torch

import oracle as orc


def div_rint_f32(w, sd):
    """The kernel's div_rint in numpy fp32 (every step but the fused
    remainder, which fp64 holds exactly)."""
    w, sd = w.astype(np.float32), sd.astype(np.float32)
    c = np.rint(w * (np.float32(1.0) / sd)).astype(np.float32)
    rem64 = w.astype(np.float64) - c.astype(np.float64) * sd.astype(np.float64)
    rem = rem64.astype(np.float32)
    assert np.array_equal(rem.astype(np.float64), rem64)       # exact: one fma gives it
    twice = np.float32(2.0) * np.abs(rem)
    nxt = c + np.copysign(np.float32(1.0), rem)
    odd = (c.astype(np.int64) & 1) != 0
    return np.where((twice > sd) | ((twice == sd) & odd), nxt, c)


def test_div_rint_is_fp64_division():
    rng = np.random.default_rng(5)
    h = np.concatenate([np.arange(1, 0x7C00, 7), [1, 2, 3, 0x3FF, 0x400, 0x7BFF]]).astype(np.uint16)
    sd = h.view(np.float16).astype(np.float32)
    for _ in range(40):
        s = rng.permutation(sd)
        half = np.float32(0.5) * rng.integers(-45, 46, s.size).astype(np.float32)
        tie = (half * s).astype(np.float32)                    # exact: 11 + 6 bits
        for w in (tie, np.nextafter(tie, np.float32(np.inf)), np.nextafter(tie, np.float32(-np.inf)),
                  (rng.uniform(-22, 22, s.size) * s).astype(np.float32)):
            ref = np.rint(w.astype(np.float64) / s.astype(np.float64))
            assert np.array_equal(div_rint_f32(w, s).astype(np.float64), ref)


@pytest.mark.gpu
@pytest.mark.parametrize("bits", [2, 3, 4])
@pytest.mark.parametrize("group", [32, 64, 128])
@pytest.mark.parametrize("n,kg", [(1, 1), (3, 5), (37, 9), (130, 4), (5, 33)])
def test_pack_tiles_bit_exact(bits, group, n, kg):
    import paper_2606_04238_amd as q
    k = kg * group
    if bits == 3:
        k = (k + 127) // 128 * 128
    print("pack tiles", bits, group, n, k, flush=True)
    rng = np.random.default_rng([bits, group, n, kg])
    W = (0.02 * rng.standard_normal((n, k))).astype(np.float32)
    flat = W.reshape(-1, group)
    for i in range(0, flat.shape[0], 3):                       # every third group on half steps: ties
        flat[i] = rng.integers(-3, 4, group).astype(np.float32) * np.float32(0.5)
    flat[-1, -1] = -0.0
    if flat.shape[0] > 4:
        flat[1] = -np.abs(flat[1])
        flat[2] = np.abs(flat[2])
        flat[3] = 0.0
        flat[4, 7] = np.nan
        flat[-2, 3] = np.float32(1e-40)                        # fp32 subnormal
    ref = orc.quantize(W, bits, group)
    fn = {2: q.pack_w2, 3: q.pack_w3, 4: q.pack_w4}[bits]
    w = fn(torch.from_numpy(W).cuda(), group)
    got = w.codes.cpu().numpy().view(np.uint32).reshape(n, -1)
    assert np.array_equal(got, ref.packed())
    assert np.array_equal(w.meta.cpu().numpy().view(np.uint16).reshape(ref.scale.shape + (2,)), ref.meta())
    assert w.invalid_groups() == (ref.bad > 0)

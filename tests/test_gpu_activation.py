"""The activation between the FFN halves, silu(g) * u, at single elements: g is built exactly from three bf16 weights, u is 1 and
W2 the identity, so a layer's output is the activation itself, rounded to fp16."""
import dataclasses

import numpy as np
import pytest
import torch

from paper_2510_26730_amd import binding as ef
from paper_2510_26730_amd import synth

from helpers import LayerStack, dev_u16

pytestmark = pytest.mark.gpu

D = F = 256
COLS = 64      # a token selects one of this many sets of gate values


def bf16_bits(x):
    """Nearest bf16 bit pattern of float32 values (ties to even)."""
    b = np.ascontiguousarray(x, np.float32).view(np.uint32)
    return ((b + 0x7FFF + ((b >> 16) & 1)) >> 16).astype(np.uint16)


def bf16_value(bits):
    return (bits.astype(np.uint32) << 16).view(np.float32)


def denominator(g, scale=1.0):
    """1 + exp(-g) as 32-bit arithmetic gives it, with the exponential off by a factor."""
    return (1 + (np.exp(-g.astype(np.float64)) * scale).astype(np.float32)).astype(np.float32)


def critical_gates():
    """Gate values in 8..16 whose activation, with 1 + exp(-g) and the quotient rounded to 32 bits once each, lies next to the
    middle between two fp16 numbers: one unit in the last place of the quotient decides its fp16 value.  Left out: those for
    which an error of 2^-18 in the exponential decides the sum's last bit.  -> g, activation in fp16."""
    mid = np.arange(8 + 2.0 ** -8, 16, 2.0 ** -7)
    g = (mid * (1 + np.exp(-mid))).astype(np.float32)
    g = (g.view(np.int32)[:, None] + np.arange(-8, 9, dtype=np.int32)).reshape(-1).view(np.float32)
    x = denominator(g)
    q = g / x
    ends = [np.nextafter(q, np.float32(s * np.inf)).astype(np.float16) for s in (-1, 1)]
    use = (x > 1) & (denominator(g, 1 + 2.0 ** -18) == x) & (denominator(g, 1 - 2.0 ** -18) == x) & (ends[0] != ends[1])
    return g[use], q[use].astype(np.float16)


@pytest.mark.parametrize("T,form", [(64, "streamed"), (160, "shared"), (640, "tiled")])
def test_quotient_of_the_activation_is_rounded_once(T, form):
    """Streamed kernels, those that share fragments in LDS, tiled ones: the quotient as an IEEE division gives it."""
    values, act = critical_gates()
    assert values.size > 1000
    ends = np.array([-3e38, -100, -88.5, -87.5, -87, 0, 1e-30, 60000], np.float32)     # no infinities: W2 has zeros
    values, act = np.append(values, ends), np.append(act, np.array([0, 0, 0, 0, 0, 0, 0, 60000], np.float16))
    rng = np.random.default_rng(5)
    pick = rng.integers(0, values.size, (F, COLS))
    g = values[pick]
    hi = bf16_bits(g)
    mid = bf16_bits(g - bf16_value(hi))
    lo = bf16_bits(g - bf16_value(hi) - bf16_value(mid))
    assert np.array_equal(bf16_value(hi) + bf16_value(mid) + bf16_value(lo), g)
    one = bf16_bits(np.float32(1))
    W1, W3, W2 = (np.zeros(s, np.uint16) for s in ((F, D), (F, D), (D, F)))
    W1[:, :COLS], W1[:, COLS:2 * COLS], W1[:, 2 * COLS:3 * COLS] = hi, mid, lo
    W3[:, 3 * COLS:] = one
    W2[np.arange(F), np.arange(F)] = one
    h = np.zeros((T, D), np.uint16)
    for block in range(4):
        h[np.arange(T), block * COLS + np.arange(T) % COLS] = one
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="activation", d=D, F=F, F_shared=0, E=2, k=1)
    st = LayerStack(cfg, 1, slots_total=2, max_tokens=T, flags=ef.EF_FLAG_PROFILE)
    try:
        store = st._keep[2].numpy()
        for e in range(2):
            ef.ef_pack_expert(W1, W3, W2, blob=store[e * st.es:(e + 1) * st.es])
            ef.ef_cache_swap_in(st.ctx, 0, e, 0, 0)
        ef.ef_get_stats(st.ctx)
        i32 = lambda a: torch.from_numpy(np.asarray(a, np.int32)).cuda()
        order = np.arange(T)
        out = torch.full((T, D), float("nan"), dtype=torch.float32, device="cuda")
        ef.ef_moe_ffn(st.ctx, 0, dev_u16(h), T, i32(np.zeros((T, 1))), torch.ones(T, 1, device="cuda"), np.array([T, 0], np.int32),
                      i32([0, T, T]), i32(order), i32(order), out, torch.cuda.current_stream())
        torch.cuda.synchronize()
        launches = dict(zip(ef.EF_KERNELS, ef.ef_get_stats(st.ctx)["kernel_launches"]))
        assert launches["ffn_up_tiled"] == int(form == "tiled") and launches["ffn_up"] == int(form != "tiled")
        got = out.cpu().numpy()
        want = act[pick].T[np.arange(T) % COLS].astype(np.float32)
        print(f"{form}: {int((got != want).sum())} of {got.size} differ", flush=True)
        assert np.array_equal(got, want)
    finally:
        st.close()

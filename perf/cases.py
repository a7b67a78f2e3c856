"""What a program that uses this library has it do, as cases that can be timed and compared.

Three kinds of work, each through the public entry points of ``paper_2510_26730_amd.binding``:

``layer``  one step through a stack of two MoE layers with ``ef_layer_step`` (look-ahead, routing, grouping, swap-in,
           expert FFN, un-permute): what a serving loop does for every batch.  Decode batches of one token to a few
           dozen, chunked prefill mixed with decode, whole prompts; 16-bit and 4-bit experts; with the residency quota
           and bias of a small expert cache, with every expert resident, and with experts that must come over the link.
``route``  routing and grouping alone (``ef_route`` or ``ef_route_predict``): a program that runs its own FFN.
``dist``   the intra-batch diversity signal ``ef_token_dist`` of one iteration's tokens.

A cache with a quota and no residency bias keeps changing, and with it the experts that are copied, but not the results;
a bias together with misses would make the results depend on what earlier passes left in the cache, so no case has both.
"""
import functools
import math

import numpy as np
import torch

from paper_2510_26730_amd import binding as ef
from paper_2510_26730_amd import synth

LAYERS = 2        # layers of a stack: the first one looks ahead to the second
TIE = 5e-5        # tokens whose k-th and (k+1)-th best scores are closer than this are drawn again: either choice is right


def _layer(name, shape, bits, T, slots, beta):
    return {"name": name, "op": "layer", "shape": shape, "bits": bits, "T": T, "slots": slots, "beta": beta}


def listed():
    return [
        # one sequence being decoded, every expert in the cache: the smallest call there is
        _layer("mixtral_decode_1", "mixtral_decode", 16, 1, 8, 0.0),
        # the benchmark's headline: a decode batch with two of eight experts in the cache and routing kept on them
        _layer("mixtral_decode_64", "mixtral_decode", 16, 64, 2, 16.0),
        # a chunk of a prompt beside some decoding sequences: every expert gets a few token tiles, ragged
        _layer("mixtral_chunk_300", "mixtral_decode", 16, 300, 8, 0.0),
        # four prompts of 2048 tokens at once, half of the experts in the cache
        _layer("mixtral_prefill_8192", "mixtral_prefill", 16, 8192, 4, 16.0),
        # decode with 64 small experts and a shared FFN, a quarter of the experts in the cache
        _layer("deepseek_decode_32", "deepseek_v2_lite", 16, 32, 16, 6.0),
        # the same without the bias: most of the experts a layer needs are copied in from the host
        _layer("deepseek_swap_32", "deepseek_v2_lite", 16, 32, 16, 0.0),
        # a prompt of 1024 tokens together with 32 decode tokens, over all 64 experts
        _layer("deepseek_mixed_1056", "deepseek_v2_lite", 16, 1056, 64, 0.0),
        # 512 prompt and 128 decode tokens, a fifth of the experts in the cache, a wide shared FFN
        _layer("qwen_mixed_640", "qwen15_moe", 16, 640, 12, 8.0),
        # 4-bit experts make the whole layer fit: a decode batch over all eight of them
        _layer("mixtral_int4_decode_64", "mixtral_decode", 4, 64, 8, 0.0),
        # 4-bit experts and 4-bit shared FFN, prompt and decode tokens mixed
        _layer("qwen_int4_mixed_640", "qwen15_moe", 4, 640, 60, 0.0),
        # routing of many prompts at once with one look-ahead layer: bound by reading the hidden states
        {"name": "route_32768", "op": "route", "shape": "mixtral_prefill", "T": 32768, "H": 1, "delta": False},
        # diversity of one mixed batch
        {"name": "dist_1056", "op": "dist", "shape": "deepseek_v2_lite", "T": 1056},
    ]


def _log_int(rng, lo, hi):
    return min(hi, max(lo, round(math.exp(rng.uniform(math.log(lo), math.log(hi + 1))))))


def draw(rng):
    op = rng.choices(["layer", "route", "dist"], weights=[8, 2, 2])[0]
    if op == "dist":
        return {"op": "dist", "shape": rng.choice(["mixtral_prefill", "deepseek_v2_lite"]), "T": _log_int(rng, 2, 8192)}
    if op == "route":
        H = rng.randint(0, 4)
        return {"op": "route", "shape": rng.choice(["mixtral_prefill", "deepseek_v2_lite", "qwen15_moe"]),
                "T": _log_int(rng, 1, 32768 // max(1, H)), "H": H, "delta": H > 0 and rng.random() < 0.5}
    shape = rng.choice(["mixtral_decode", "deepseek_v2_lite", "qwen15_moe", "deepseek_v2_lite", "qwen15_moe", "tiny"])
    bits = rng.choice([16, 16, 4])
    cfg = synth.CONFIGS[shape]
    mode = rng.choice(["all", "all", "quota", "quota", "swap"])
    if mode == "swap" and (shape != "deepseek_v2_lite" or bits != 16):
        mode = "quota"
    T = _log_int(rng, 1, {"all": 4096, "quota": 4096, "swap": 32}[mode])
    return {"op": "layer", "shape": shape, "bits": bits, "T": T, "slots": cfg.E if mode == "all" else cfg.slots_per_layer,
            "beta": 16.0 if mode == "quota" else 0.0}


# ---- inputs -----------------------------------------------------------------------------------------------------

def _generator(seed, *key):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(np.random.SeedSequence([seed, *key]).generate_state(1, np.uint64)[0] >> np.uint64(1)))
    return g


def _normal(g, *shape, std=1.0):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float32).mul_(std)


def _ranks(case, seed, layer):
    cfg = synth.CONFIGS[case["shape"]]
    return np.random.default_rng([seed, 1, layer]).permutation(cfg.E) + 1


def _gate(case, seed, layer):
    """Gate matrix [E, d] bf16 and bias [E] f32: the logarithm of a Zipf popularity of the experts."""
    cfg = synth.CONFIGS[case["shape"]]
    w = _normal(_generator(seed, 2, layer), cfg.E, cfg.d, std=cfg.w_std).to(torch.bfloat16)
    b = torch.from_numpy((-cfg.zipf_s * np.log(_ranks(case, seed, layer))).astype(np.float32)).cuda()
    return w, b


def _residents(case, seed, layer):
    """The experts that the cache holds before the first pass: the most popular ones."""
    return np.argsort(_ranks(case, seed, layer), kind="stable")[:case["slots"]]


def _score(h, gate, beta=0.0, residents=(), delta=None):
    z = h.double() @ gate[0].double().T + gate[1].double()
    s = z.clone()
    if len(residents):
        s[:, torch.as_tensor(np.asarray(residents), device="cuda")] += beta
    if delta is not None:
        s += delta.double()
    return z, s


def _near_tie(s, k):
    top = s.topk(min(k + 1, s.shape[1]), dim=1).values
    return top[:, k - 1] - top[:, k] < TIE if s.shape[1] > k else torch.zeros(s.shape[0], dtype=torch.bool, device="cuda")


def _draw_tokens(make, tied):
    """make() gives [T, d] bf16; tokens for which tied(h) holds are taken from another draw."""
    h = make()
    for _ in range(8):
        bad = tied(h)
        if not bool(bad.any()):
            break
        h[bad] = make()[bad]
    return h


def _hidden_stack(case, seed):
    """Hidden states of the layers of a step: each layer's are the previous ones with some noise."""
    cfg, T = synth.CONFIGS[case["shape"]], case["T"]
    hs, g = [], _generator(seed, 3)
    for l in range(LAYERS):
        gate, res = _gate(case, seed, l), _residents(case, seed, l)

        def make():
            if not hs:
                return _normal(g, T, cfg.d).to(torch.bfloat16)
            return (hs[-1].float() + _normal(g, T, cfg.d, std=cfg.noise)).to(torch.bfloat16)

        hs.append(_draw_tokens(make, lambda h: _near_tie(_score(h, gate, case["beta"], res)[1], cfg.k)))
    return hs


def _expert16(cfg, F, seed, *key):
    """W1 [F, d], W3 [F, d], W2 [d, F] in bf16."""
    g = _generator(seed, 4, *key)
    return [_normal(g, *s, std=cfg.w_std).to(torch.bfloat16) for s in ((F, cfg.d), (F, cfg.d), (cfg.d, F))]


def _expert4(cfg, F, seed, *key):
    """Codes (0..15) and bf16 scales of W1, W3, W2."""
    g = _generator(seed, 5, *key)
    out = []
    for r, c in ((F, cfg.d), (F, cfg.d), (cfg.d, F)):
        q = _normal(g, r, c, std=2.5).round_().add_(8).clamp_(0, 15).to(torch.uint8)
        s = _normal(g, r, c // 128).clamp_(-3, 3).mul_(0.1).add_(1).mul_(cfg.w_std / 2.5).to(torch.bfloat16)
        out.append((q, s))
    return out


def _fragments(w):
    """[r, c] -> [r/32, c/16, 512]: the operand order of a packed blob's first section."""
    r, c = w.shape
    return w.view(r // 32, 32, c // 16, 2, 8).permute(0, 2, 3, 1, 4).reshape(r // 32, c // 16, 512)


def _pack16(w1, w3, w2, blob):
    """Row-major weights into a packed blob (int16 on the device), as ef_pack_expert lays it out."""
    F, d = w1.shape
    a = blob[:2 * d * F].view(F // 32, 2, d // 16, 512)
    a[:, 0], a[:, 1] = _fragments(w1).view(torch.int16), _fragments(w3).view(torch.int16)
    b = w2.to(torch.float16).view(torch.int16).view(d // 32, 32, F // 16, 2, 2, 4).permute(0, 2, 4, 1, 3, 5)
    blob[2 * d * F:] = b.reshape(-1)


def _quads(q, paired):
    """Codes [r, c] -> [r/32, c/64, 1024] bytes."""
    r, c = q.shape
    if paired:
        f = q.view(r // 32, 32, c // 64, 4, 2, 2, 4).permute(0, 2, 5, 1, 3, 4, 6)
    else:
        f = q.view(r // 32, 32, c // 64, 4, 2, 8).permute(0, 2, 4, 1, 3, 5)
    f = f.reshape(r // 32, c // 64, 256, 8)
    return (f[..., [0, 4, 1, 5]] | (f[..., [2, 6, 3, 7]] << 4)).reshape(r // 32, c // 64, 1024)


def _pack4(m1, m3, m2, blob):
    """Codes and scales into a packed 4-bit blob (uint8 on the device), as ef_pack_expert_q4 lays it out."""
    (q1, s1), (q3, s3), (q2, s2) = m1, m3, m2
    F, d = q1.shape
    n = d * F // 2
    a = blob[:2 * n].view(F // 32, d // 64, 2, 1024)
    a[:, :, 0], a[:, :, 1] = _quads(q1, False), _quads(q3, False)
    blob[2 * n:3 * n] = _quads(q2, True).reshape(-1)
    s13 = torch.stack([s.view(F // 32, 32, d // 128).permute(0, 2, 1) for s in (s1, s3)], dim=2).reshape(-1)
    blob[3 * n:3 * n + 2 * s13.numel()] = s13.view(torch.uint8)
    blob[3 * n + 2 * s13.numel():] = s2.view(d // 32, 32, F // 128).permute(0, 2, 1).reshape(-1).view(torch.uint8)


def _blob(cfg, F, bits, seed, *key):
    if bits == 4:
        blob = torch.empty(ef.ef_expert_bytes_q4(cfg.d, F), dtype=torch.uint8, device="cuda")
        _pack4(*_expert4(cfg, F, seed, *key), blob)
    else:
        blob = torch.empty(ef.ef_expert_bytes(cfg.d, F) // 2, dtype=torch.int16, device="cuda")
        _pack16(*_expert16(cfg, F, seed, *key), blob)
    return blob


# ---- states -----------------------------------------------------------------------------------------------------

class _State:
    """A context and what it refers to; the context goes before the buffers do."""

    def __init__(self, case):
        self.case, self.ctx = case, None

    def __del__(self):
        if self.ctx is not None:
            torch.cuda.synchronize()
            ef.ef_destroy(self.ctx)


def _prepare_layer(case, seed):
    cfg, T = synth.CONFIGS[case["shape"]], case["T"]
    st = _State(case)
    st.ctx = ef.ef_create(n_layers=LAYERS, d_model=cfg.d, n_experts=cfg.E, top_k=cfg.k, d_ff=cfg.F, d_ff_shared=cfg.F_shared,
                          slots_total=LAYERS * case["slots"], slots_per_layer_max=case["slots"], max_tokens=T,
                          renorm_topk=int(cfg.renorm), weight_bits=case["bits"])
    first = _blob(cfg, cfg.F, case["bits"], seed, 0)
    st.store = torch.empty(cfg.E, first.numel(), dtype=first.dtype, pin_memory=True)   # shared by the layers
    for e in range(cfg.E):
        st.store[e].copy_(first if e == 0 else _blob(cfg, cfg.F, case["bits"], seed, e))
    st.shared = _blob(cfg, cfg.F_shared, case["bits"], seed, cfg.E) if cfg.F_shared else None
    st.gates = [_gate(case, seed, l) for l in range(LAYERS)]
    st.hidden = _hidden_stack(case, seed)
    st.out = [torch.empty(T, cfg.d, dtype=torch.float32, device="cuda") for _ in range(LAYERS)]
    st.counts = [np.zeros(cfg.E, dtype=np.int32) for _ in range(LAYERS)]
    torch.cuda.synchronize()
    for l in range(LAYERS):
        ef.ef_register_layer(st.ctx, l, st.gates[l][0], st.gates[l][1], st.store, st.shared)
        for e in _residents(case, seed, l):
            ef.ef_cache_swap_in(st.ctx, l, int(e), 0, 0)
    ef.ef_get_stats(st.ctx)      # waits until the copies are done
    st.stream = torch.cuda.current_stream()
    return st


def _delta(case, seed):
    """Deviation of each request's look-ahead [R, H, E], and the request of each token."""
    if not case["delta"]:
        return None, None
    cfg, T, R = synth.CONFIGS[case["shape"]], case["T"], min(case["T"], 32)
    d = _normal(_generator(seed, 6), R, case["H"], cfg.E, std=0.5)
    return d, torch.arange(T, device="cuda", dtype=torch.int32).mul_(R).div_(T, rounding_mode="floor").to(torch.int32)


def _route_tokens(case, seed, delta, tok2req):
    cfg, T = synth.CONFIGS[case["shape"]], case["T"]
    gates = [_gate(case, seed, l) for l in range(case["H"] + 1)]
    g = _generator(seed, 3)

    def tied(h):
        bad = torch.zeros(T, dtype=torch.bool, device="cuda")
        for l, gate in enumerate(gates):
            bad |= _near_tie(_score(h, gate, delta=None if l == 0 or delta is None else delta[tok2req.long(), l - 1])[1], cfg.k)
        return bad

    return gates, _draw_tokens(lambda: _normal(g, T, cfg.d).to(torch.bfloat16), tied)


def _prepare_route(case, seed):
    cfg, T, H = synth.CONFIGS[case["shape"]], case["T"], case["H"]
    st = _State(case)
    # experts of the smallest size: none of them runs
    st.ctx = ef.ef_create(n_layers=H + 1, d_model=cfg.d, n_experts=cfg.E, top_k=cfg.k, d_ff=32, slots_total=1, max_tokens=T,
                          renorm_topk=int(cfg.renorm))
    st.store = torch.zeros(cfg.E * ef.ef_expert_bytes(cfg.d, 32), dtype=torch.uint8, pin_memory=True)
    st.delta, st.tok2req = _delta(case, seed)
    st.gates, st.hidden = _route_tokens(case, seed, st.delta, st.tok2req)
    for l, (w, b) in enumerate(st.gates):
        ef.ef_register_layer(st.ctx, l, w, b, st.store, None)
    i32 = dict(dtype=torch.int32, device="cuda")
    st.o = {"ids": torch.empty(T, cfg.k, **i32), "w": torch.empty(T, cfg.k, dtype=torch.float32, device="cuda"),
            "counts": torch.empty(cfg.E, **i32), "offsets": torch.empty(cfg.E + 1, **i32), "perm": torch.empty(T * cfg.k, **i32),
            "inv_perm": torch.empty(T * cfg.k, **i32)}
    if H:
        st.o.update(pred_ids=torch.empty(H, T, cfg.k, **i32), pred_hist=torch.empty(H, cfg.E, **i32))
    st.stream = torch.cuda.current_stream()
    return st


def _prepare_dist(case, seed):
    cfg, T = synth.CONFIGS[case["shape"]], case["T"]
    st = _State(case)
    st.ctx = ef.ef_create(n_layers=1, d_model=cfg.d, n_experts=cfg.E, top_k=cfg.k, d_ff=32, slots_total=1, max_tokens=T,
                          renorm_topk=int(cfg.renorm))
    st.hidden = _normal(_generator(seed, 3), T, cfg.d).to(torch.bfloat16)
    st.o = {"tok_dist": torch.empty(T, dtype=torch.float32, device="cuda"), "dist": torch.empty(1, dtype=torch.float64, device="cuda")}
    st.stream = torch.cuda.current_stream()
    return st


def prepare(case, seed):
    return {"layer": _prepare_layer, "route": _prepare_route, "dist": _prepare_dist}[case["op"]](case, seed)


def run(st):
    case = st.case
    if case["op"] == "layer":
        for l in range(LAYERS):
            ef.ef_layer_step(st.ctx, l, st.hidden[l], case["T"], case["beta"], -1, None, None, st.out[l], st.counts[l], st.stream)
        return {"out": st.out, "counts": st.counts}
    o = st.o
    if case["op"] == "dist":
        ef.ef_token_dist(st.ctx, st.hidden, case["T"], o["tok_dist"], o["dist"], st.stream)
    elif case["H"]:
        ef.ef_route_predict(st.ctx, 0, st.hidden, case["T"], 0.0, case["H"], st.delta, st.tok2req, o["ids"], o["w"], o["counts"],
                            o["offsets"], o["perm"], o["inv_perm"], o["pred_ids"], o["pred_hist"], st.stream)
    else:
        ef.ef_route(st.ctx, 0, st.hidden, case["T"], 0.0, o["ids"], o["w"], o["counts"], o["offsets"], o["perm"], o["inv_perm"],
                    st.stream)
    return o


# ---- work, tolerance, values in 64 bits -----------------------------------------------------------------------------

@functools.lru_cache(maxsize=None)
def _experts_used(shape, T, slots, beta):
    """Mean number of experts that T tokens use, with logits as the gates give them."""
    cfg, rng, n = synth.CONFIGS[shape], np.random.default_rng(0), 0
    bias = -cfg.zipf_s * np.log(np.arange(1, cfg.E + 1)) + np.where(np.arange(cfg.E) < slots, beta, 0.0)
    for _ in range(8):
        z = rng.standard_normal((T, cfg.E), dtype=np.float32) * (cfg.w_std * math.sqrt(cfg.d)) + bias
        n += len(np.unique(np.argpartition(-z, cfg.k - 1, axis=1)[:, :cfg.k]))
    return n / 8


def work(case):
    cfg, T = synth.CONFIGS[case["shape"]], case["T"]
    d, E, k = cfg.d, cfg.E, cfg.k
    if case["op"] == "dist":
        return {"bytes": 2 * T * d + 4 * T + 8, "flops": T * (T - 1) * d}
    gate = 2 * E * d + 4 * E
    if case["op"] == "route":
        G = case["H"] + 1
        return {"bytes": 2 * T * d + G * gate + 4 * T * k * (G + 3) + 4 * (G + 1) * E, "flops": 2 * G * T * E * d}
    size = ef.ef_expert_bytes if case["bits"] == 16 else ef.ef_expert_bytes_q4
    weights = _experts_used(case["shape"], T, case["slots"], case["beta"]) * size(d, cfg.F)
    if cfg.F_shared:
        weights += size(d, cfg.F_shared)
    return {"bytes": LAYERS * (weights + gate + 6 * T * d),
            "flops": LAYERS * (6 * T * d * (k * cfg.F + cfg.F_shared) + 2 * T * E * d) + 2 * T * E * d}


def tolerance(case):
    if case["op"] == "layer":
        # products of 16-bit numbers summed in 32 bits; the activation between the FFN halves is rounded to 16 bits
        return {"rel": 8e-4, "max": 6e-3, "differ": 0.0}
    if case["op"] == "route":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}      # softmax of 32-bit sums; ids are whole values
    return {"rel": 1e-6, "max": 1e-5}                          # 32-bit squared distances, sums in 64 bits


def _topk(s, k):
    return s.topk(k, dim=1).indices.sort(dim=1).values


def _combine_weights(z, ids, renorm):
    w = torch.softmax(z, dim=1).gather(1, ids)
    return w / w.sum(dim=1, keepdim=True) if renorm else w


def _matrices(cfg, F, bits, seed, *key):
    if bits == 16:
        return [w.double() for w in _expert16(cfg, F, seed, *key)]
    return [(q.double() - 8) * s.double().repeat_interleave(128, dim=1) for q, s in _expert4(cfg, F, seed, *key)]


def _swiglu(x, w1, w3, w2):
    return (torch.nn.functional.silu(x @ w1.T) * (x @ w3.T)) @ w2.T


def _exact_layer(case, seed):
    cfg = synth.CONFIGS[case["shape"]]
    hs = _hidden_stack(case, seed)
    plan, out, counts = [], [], []
    for l in range(LAYERS):
        z, s = _score(hs[l], _gate(case, seed, l), case["beta"], _residents(case, seed, l))
        ids = _topk(s, cfg.k)
        plan.append((hs[l].double(), ids, _combine_weights(z, ids, cfg.renorm)))
        out.append(torch.zeros(case["T"], cfg.d, dtype=torch.float64, device="cuda"))
        counts.append(torch.bincount(ids.reshape(-1), minlength=cfg.E).to(torch.int32))
    for e in range(cfg.E):
        if not any(int(c[e]) for c in counts):
            continue
        m = _matrices(cfg, cfg.F, case["bits"], seed, e)
        for l, (x, ids, w) in enumerate(plan):
            t, j = torch.nonzero(ids == e, as_tuple=True)
            if t.numel():
                out[l].index_add_(0, t, _swiglu(x[t], *m) * w[t, j].unsqueeze(1))
    if cfg.F_shared:
        m = _matrices(cfg, cfg.F_shared, case["bits"], seed, cfg.E)
        for l, (x, _, _) in enumerate(plan):
            out[l] += _swiglu(x, *m)
    return {"out": out, "counts": counts}


def _exact_route(case, seed):
    cfg = synth.CONFIGS[case["shape"]]
    delta, tok2req = _delta(case, seed)
    gates, h = _route_tokens(case, seed, delta, tok2req)
    z, s = _score(h, gates[0])
    ids = _topk(s, cfg.k)
    flat = ids.reshape(-1)
    counts = torch.bincount(flat, minlength=cfg.E)
    perm = torch.sort(flat, stable=True).indices
    inv = torch.empty_like(perm)
    inv[perm] = torch.arange(perm.numel(), device="cuda")
    i32 = torch.int32
    o = {"ids": ids.to(i32), "w": _combine_weights(z, ids, cfg.renorm), "counts": counts.to(i32),
         "offsets": torch.cat([counts.new_zeros(1), counts.cumsum(0)]).to(i32), "perm": perm.to(i32), "inv_perm": inv.to(i32)}
    if case["H"]:
        p = [_topk(_score(h, gates[j], delta=None if delta is None else delta[tok2req.long(), j - 1])[1], cfg.k)
             for j in range(1, case["H"] + 1)]
        o["pred_ids"] = torch.stack(p).to(i32)
        o["pred_hist"] = torch.stack([torch.bincount(x.reshape(-1), minlength=cfg.E) for x in p]).to(i32)
    return o


def _exact_dist(case, seed):
    cfg, T = synth.CONFIGS[case["shape"]], case["T"]
    h = _normal(_generator(seed, 3), T, cfg.d).to(torch.bfloat16).double()
    n = h.square().sum(dim=1)
    per = (n[:, None] + n[None, :] - 2.0 * (h @ h.T)).clamp_min_(0).sqrt_().triu_(1).sum(dim=0)
    return {"tok_dist": per, "dist": per.sum().reshape(1)}


def exact(case, seed):
    return {"layer": _exact_layer, "route": _exact_route, "dist": _exact_dist}[case["op"]](case, seed)

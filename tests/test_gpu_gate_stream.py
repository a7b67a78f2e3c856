"""Routing and look-ahead of batches with many token tiles (the gate kernel that streams the hidden states
through LDS) against the CPU oracle: ids bit-exact outside near-ties and valid inside, histograms, counts,
offsets and permutation teacher-forced, weights to 1e-5; and against the other form of the kernel."""
import dataclasses
import sys

import numpy as np
import pytest
import torch

from paper_2510_26730_amd import binding as ef
from paper_2510_26730_amd import synth

import helpers
from helpers import LayerStack, check_ids_valid, check_route, dev_u16, to_np

pytestmark = pytest.mark.gpu


def say(msg):
    print(msg, flush=True)
    sys.stdout.flush()


def shape(base, **kw):
    return dataclasses.replace(synth.CONFIGS[base], **kw)


CASES = [
    # name, shape (experts of the smallest legal size: routing only), tokens, look-ahead H
    ("e8_route_only", shape("mixtral_prefill", name="gs_e8", d=512, F=32), 6144, 0),
    ("e8_ragged_h1", shape("mixtral_prefill", name="gs_e8b", d=768, F=32), 6500, 1),
    ("e8_h3_32cols", shape("mixtral_prefill", name="gs_e8c", d=256, F=32), 7000, 3),
    ("e8_h4_40cols", shape("mixtral_prefill", name="gs_e8d", d=512, F=32), 6200, 4),
    ("e3_k2", shape("mixtral_prefill", name="gs_e3", d=1280, E=3, k=2, F=32), 6145, 0),
    ("e64_k6", shape("deepseek_v2_lite", name="gs_e64", d=1024, F=32, F_shared=0), 6300, 0),
    ("e60_k4_h1", shape("qwen15_moe", name="gs_e60", d=512, F=32, F_shared=0), 6150, 1),
]


@pytest.mark.parametrize("name,cfg,T,H", CASES, ids=[c[0] for c in CASES])
def test_streaming_gate_against_oracle(oracle_mod, name, cfg, T, H):
    say(f"streaming gate {name}: E={cfg.E} k={cfg.k} d={cfg.d} T={T} H={H}")
    L = H + 1
    results = []
    for stream_form in (1, 0):
        st = LayerStack(cfg, L, slots_total=cfg.E, max_tokens=T, expert_layers=[0], h_max=max(1, min(H, 7)))
        try:
            ef.ef_set_tuning(st.ctx, gate_stream=stream_form)
            for l in range(L):
                for e in np.nonzero(synth.residency(cfg, l, n_resident=max(1, cfg.E // 4), most_popular=False))[0]:
                    ef.ef_cache_swap_in(st.ctx, l, int(e), 0, l)
            res = [ef.ef_cache_query(st.ctx, l, cfg.E) for l in range(L)]
            h = synth.hidden(cfg, 11, T)
            hd = dev_u16(h)
            beta = 0.6
            o = st.route(0, hd, T, 0.0)     # fresh buffers, overwritten by the fused call
            n = T * cfg.k
            pids = torch.full((max(1, H * n),), -1, dtype=torch.int32, device="cuda")
            phist = torch.full((max(1, H * cfg.E),), -1, dtype=torch.int32, device="cuda")
            he = ef.ef_route_predict(st.ctx, 0, hd, T, beta, H, None, None, o["ids"], o["w"], o["counts"], o["offsets"],
                                     o["perm"], o["inv_perm"], pids, phist, torch.cuda.current_stream())
            assert he == H
            got = to_np(o, T, cfg.k)
            got["pred_ids"] = pids.cpu().numpy()[:H * n].reshape(H, T, cfg.k)
            got["pred_hist"] = phist.cpu().numpy()[:H * cfg.E].reshape(H, cfg.E)
            results.append(got)
            ora = oracle_mod.route(h, st.gates[0], st.biases[0], cfg.k, beta, res[0], renorm=cfg.renorm)
            _, nties = check_route(got, ora, cfg.E, cfg.k, cfg.renorm, oracle_mod=oracle_mod)
            if H:
                oids, ohist, ogap, osc = oracle_mod.predict(h, st.gates[1:L], st.biases[1:L], cfg.k, beta, res[1:L],
                                                            return_scores=True)
                tie = ogap < helpers.TIE_GAP
                assert np.array_equal(got["pred_ids"][~tie], oids[~tie])
                for j in range(H):
                    check_ids_valid(got["pred_ids"][j], osc[j], ogap[j], cfg.k)
                    assert np.array_equal(got["pred_hist"][j], oracle_mod.histogram(got["pred_ids"][j], cfg.E))
                nties += int(tie.sum())
            say(f"  streaming form {stream_form}: near-ties {nties}")
        finally:
            st.close()
    # the two forms add the K range up in different orders: same ids wherever the oracle sees no near-tie was
    # checked above; weights agree to rounding
    assert np.max(np.abs(results[0]["w"] - results[1]["w"])) < 1e-5


@pytest.mark.parametrize("E,H", [(2, 0), (8, 0), (9, 0), (5, 1), (8, 1), (17, 0), (11, 2)],
                         ids=lambda v: str(v))
def test_gate_row_blocks_at_their_column_limits(oracle_mod, E, H):
    """Up to 8, 16 and 32 logit columns a stage holds 4, 8 and 16 blocks of gate rows: both sides of each limit."""
    cfg = shape("mixtral_prefill", name=f"gs_cols_{E}_{H}", d=768, E=E, k=min(2, E), F=32)
    test_streaming_gate_against_oracle(oracle_mod, cfg.name, cfg, 6177, H)


@pytest.mark.parametrize("T,H", [(2049, 2), (2080, 7), (6145, 1), (32800, 2)], ids=lambda v: str(v))
def test_histograms_from_per_tile_counts_at_their_limits(oracle_mod, T, H):
    """From 65 token tiles on the grouping adds the look-ahead histograms up from per-tile counts: first such batch,
    an odd last tile, the widest look-ahead, more than one chunk of 64 tiles per wave (over 1024 tiles)."""
    cfg = shape("mixtral_prefill", name=f"gs_hist_{T}_{H}", d=256, F=32)
    test_streaming_gate_against_oracle(oracle_mod, cfg.name, cfg, T, H)


@pytest.mark.parametrize("E,k,T,H", [(8, 2, 129, 1), (3, 1, 2049, 0), (60, 8, 1024, 1), (64, 6, 8192, 1), (64, 6, 8193, 1)],
                         ids=lambda v: str(v))
def test_grouping_by_sums_at_its_limits(oracle_mod, E, k, T, H):
    """From five token tiles to 16384 per-tile counts one launch groups the tokens: the first such batch, an expert count that
    leaves threads over, eight ids a token, the largest number of counts, and the first batch past it."""
    cfg = shape("mixtral_prefill", name=f"gs_sums_{E}_{T}", d=256, E=E, k=k, F=32)
    test_streaming_gate_against_oracle(oracle_mod, cfg.name, cfg, T, H)

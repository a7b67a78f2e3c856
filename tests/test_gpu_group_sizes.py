"""The grouped FFN at chosen group sizes: every number of live token tiles in a pass, full and ragged last tiles, against
the CPU oracle.  The routing is the caller's (ef_moe_ffn takes ids, weights and permutation), so each expert gets exactly
the tokens the case names.  Bounds as in the other parity tests: max-abs 2e-2, relative L2 1e-2 (one fp16 rounding of the
intermediate activation; observed relative L2 2e-4)."""
import contextlib
import dataclasses
import re

import numpy as np
import pytest
import torch

from paper_2510_26730_amd import binding as ef
from paper_2510_26730_amd import synth

from helpers import LayerStack, dev_u16, float_close

pytestmark = pytest.mark.gpu

# tokens per expert (eight experts, one each)
SIZES = {
    "one tile": [1, 31, 32, 7, 0, 2, 16, 30],
    "one and two tiles": [33, 64, 1, 32, 63, 0, 31, 2],
    "up to four tiles": [97, 128, 65, 96, 33, 1, 0, 127],
    "second passes": [129, 160, 193, 224, 225, 32, 1, 161],
    "tiled beside streamed": [320, 300, 33, 1, 100, 513, 64, 0],
    "three live tiles last": [350, 449, 257, 480, 0, 97, 289, 1],
    "half live tiles": [15, 17, 33, 48, 47, 49, 34, 16],
}


def run_groups(oracle_mod, cfg, sizes, q4, tune, slots=None, expect=None, flops=None, forms=None, q4_forms=None):
    """Output of the layer; compared with the oracle if one is given.  slots: fewer cache slots than experts, all empty.
    expect: launches of kernel kinds; flops: their algorithmic flops; forms: template arguments of the LDS-shared kernels that
    ran (token tiles per pass, register ring, workgroups per compute unit), the same in both halves; q4_forms: of the 4-bit
    first halves that ran (token tiles per pass, parts of the K range, workgroups per compute unit)."""
    T, E = sum(sizes), cfg.E
    st = LayerStack(cfg, 1, slots_total=slots or E, max_tokens=T, q4=q4, flags=ef.EF_FLAG_PROFILE if expect else 0)
    try:
        if tune:
            ef.ef_set_tuning(st.ctx, **tune)
        for e in range(E if slots is None else 0):
            ef.ef_cache_swap_in(st.ctx, 0, e, 0, 0)
        ef.ef_get_stats(st.ctx)     # waits for the copies: one phase
        rng = np.random.default_rng(sum(sizes) + 1)
        ids = np.repeat(np.arange(E, dtype=np.int32), sizes)
        rng.shuffle(ids)
        w = rng.uniform(0.2, 1.0, size=(T, 1)).astype(np.float32)
        perm = np.argsort(ids, kind="stable").astype(np.int32)
        inv = np.empty(T, np.int32)
        inv[perm] = np.arange(T, dtype=np.int32)
        counts = np.bincount(ids, minlength=E).astype(np.int32)
        offsets = np.concatenate([[0], np.cumsum(counts)]).astype(np.int32)
        h = synth.hidden(cfg, 0, T)
        dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).cuda()
        out = torch.full((T, cfg.d), float("nan"), dtype=torch.float32, device="cuda")
        hd, d_ids, d_w, d_off, d_perm, d_inv = dev_u16(h), dev(ids), dev(w), dev(offsets), dev(perm), dev(inv)
        with torch.profiler.profile(activities=[torch.profiler.ProfilerActivity.CUDA]) if forms or q4_forms else contextlib.nullcontext() as prof:
            ef.ef_moe_ffn(st.ctx, 0, hd, T, d_ids, d_w, counts, d_off, d_perm, d_inv, out, torch.cuda.current_stream())
            torch.cuda.synchronize()
        if forms:
            ran = [m.groups() for m in (re.search(r"ffn_(gate_up|down)_shared_kernel<([\d, ]+)>", e.name) for e in prof.events()) if m]
            assert sorted(ran) == sorted((half, form) for half in ("down", "gate_up") for form in forms), ran
        if q4_forms:
            ran = [m.group(1) for m in (re.search(r"ffn_gate_up_q4_kernel<([\d, ]+)>", e.name) for e in prof.events()) if m]
            assert sorted(ran) == sorted(q4_forms), ran
        if expect:
            launches = dict(zip(ef.EF_KERNELS, ef.ef_get_stats(st.ctx)["kernel_launches"]))
            assert {k: launches[k] for k in expect} == expect
        if flops:
            done = dict(zip(ef.EF_KERNELS, ef.ef_get_stats(st.ctx)["kernel_flops"]))
            assert {k: done[k] for k in flops} == flops
        if oracle_mod is None:
            return out.cpu().numpy()
        ffn = oracle_mod.expert_ffn_q4 if q4 else oracle_mod.expert_ffn
        y = ffn(h, st.experts[0], ids.reshape(T, 1), perm)
        shared = None
        if cfg.F_shared:
            if q4:
                shared = oracle_mod.expert_ffn_q4(h, [st.shared[0]], np.zeros((T, 1), np.int32), np.arange(T))
            else:
                shared = oracle_mod.dense_ffn(h, *st.shared[0])
        ref = oracle_mod.combine(y, w.astype(np.float64), inv, shared)
        print(sizes, tune, float_close(out.cpu().numpy(), ref), flush=True)
        return out.cpu().numpy()
    finally:
        st.close()


@pytest.mark.parametrize("q4", [False, True], ids=["bf16", "int4"])
@pytest.mark.parametrize("d,F,F_shared", [(256, 128, 0), (512, 640, 256)])
@pytest.mark.parametrize("sizes", list(SIZES), ids=[s.replace(" ", "_") for s in SIZES])
def test_group_sizes(oracle_mod, sizes, d, F, F_shared, q4):
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="groups", d=d, F=F, F_shared=F_shared, k=1)
    run_groups(oracle_mod, cfg, SIZES[sizes], q4, {})


@pytest.mark.parametrize("F_shared", [256, 1024])
@pytest.mark.parametrize("sizes", ["tiled beside streamed", "three live tiles last"], ids=lambda s: s.replace(" ", "_"))
def test_expanded_groups_of_two_widths(oracle_mod, sizes, F_shared):
    """4-bit routed groups and the shared FFN expanded side by side (hidden sizes on both sides of each other in one staging
    area, ragged token panels), beside streamed groups."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="groups", d=512, F=640, F_shared=F_shared, k=1)
    run_groups(oracle_mod, cfg, SIZES[sizes], True, dict(q4_expand_min_units=0))


@pytest.mark.parametrize("tune", [dict(lds_shared_occupancy=2), dict(lds_shared_occupancy=1, down_k_slices=3)], ids=str)
def test_group_sizes_of_the_shared_forms(oracle_mod, tune):
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="groups", d=512, F=640, k=1)
    run_groups(oracle_mod, cfg, SIZES["second passes"], False, tune)


@pytest.mark.parametrize("F,F_shared,tune", [(128, 0, dict(down_k_slices=3)), (256, 0, dict(down_k_slices=8)),
                                             (384, 128, dict(down_k_slices=7)), (512, 256, dict(down_k_slices=8)),
                                             (128, 2048, dict(down_split_slice_counts=0))], ids=str)
def test_more_slices_than_stages(oracle_mod, F, F_shared, tune):
    """A slice count above the F / 64 stages of the second half's K range, forced or taken over from a wide tiled shared FFN:
    a group takes one slice per stage, and the forced count gives the same sums as that one."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="groups_slices", d=256, F=F, F_shared=F_shared, k=1)
    sizes = [97, 65, 31, 0, 1, 5, 0, 1] if F_shared < 1024 else [97, 128, 65, 7, 1, 0, 0, 2]
    out = run_groups(oracle_mod, cfg, sizes, False, tune)
    if not F_shared:
        assert np.array_equal(out, run_groups(None, cfg, sizes, False, dict(down_k_slices=F // 64)))


@pytest.mark.parametrize("d,F,F_shared,sizes", [
    (256, 2432, 0, SIZES["second passes"]),                       # 266 workgroups in passes of four
    (320, 4224, 0, [256, 255, 97, 64, 33, 129, 1, 0]),            # 330; an odd number of stages, waves past the last column
    (256, 2816, 0, [320, 320, 320, 320, 320, 320, 288, 161]),     # 44 beside 308 tiled
    (320, 2432, 0, [288, 345, 512, 65, 96, 31, 0, 7]),            # 228 + 57: second passes of one, three and eight tiles
    (256, 4096, 2816, [33, 40, 96, 65, 1, 7, 12, 11]),            # the shared FFN, nine tiles, streams with the experts
])
def test_passes_of_eight(oracle_mod, d, F, F_shared, sizes):
    """One to eight live tiles in passes of eight, first and second ones, full and ragged last tiles, K slices of unequal
    length; and the bits of both forms of the passes of four."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="groups_eight", d=d, F=F, F_shared=F_shared, k=1)
    out = run_groups(oracle_mod, cfg, sizes, False, {}, expect=dict(ffn_up=1), forms=["8, 3, 1"])
    same = run_groups(None, cfg, sizes, False, dict(down_k_slices=3), forms=["8, 3, 1"])
    assert np.linalg.norm(out - same) <= 1e-5 * np.linalg.norm(out)      # the order of 32-bit sums
    for occupancy, form in ((1, "4, 3, 1"), (2, "4, 2, 2")):
        four = run_groups(None, cfg, sizes, False, dict(down_k_slices=3, lds_shared_occupancy=occupancy), forms=[form])
        assert np.array_equal(same, four)


@pytest.mark.parametrize("occupancy,form", [(0, "8, 3, 1"), (1, "4, 3, 1"), (2, "4, 2, 2")])
def test_a_set_occupancy_asks_for_a_form_of_passes_of_four(occupancy, form):
    """266 workgroups in passes of four, groups of up to eight tiles: passes of eight unless a form of the others is set."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="groups_forms", d=256, F=2432, F_shared=0, k=1)
    run_groups(None, cfg, SIZES["second passes"], False, dict(lds_shared_occupancy=occupancy), forms=[form])


@pytest.mark.parametrize("large,form", [(4, "4, 3, 1"), (5, "8, 3, 1")])
def test_pass_width_beside_tiled_groups(oracle_mod, large, form):
    """Groups of 17 token tiles, 51 units of a tiled first half each on 56 workgroups (an XCD's share is rounded up): the
    streamed group of six tiles takes passes of four beside four of them (224), of eight beside five (280; 255 units)."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="groups_units", d=256, F=2176, F_shared=0, k=1)
    sizes = [513] * large + [161, 1] + [0] * (6 - large)
    run_groups(oracle_mod, cfg, sizes, False, {}, expect=dict(ffn_up=1, ffn_up_tiled=1), forms=[form])


@pytest.mark.parametrize("sizes,F", [([257, 300, 288, 320, 352, 290, 383, 289], 4864),   # 912 workgroups in passes of four
                                     ([140, 320, 160, 150, 3, 97, 33, 129], 4736)])      # 518, one group of ten tiles
def test_q4_large_groups_do_not_depend_on_phases(sizes, F):
    """4-bit groups of nine tiles and more that stream because of the whole layer's size: the same bits with every expert
    resident (one phase) and through a single cache slot (one expert per phase)."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="groups_phases", d=512, F=F, F_shared=0, k=1)
    a = run_groups(None, cfg, sizes, True, {})
    b = run_groups(None, cfg, sizes, True, {}, slots=1)
    rng = np.random.default_rng(sum(sizes) + 1)
    ids = np.repeat(np.arange(cfg.E), sizes)
    rng.shuffle(ids)
    large = np.asarray(sizes)[ids] > 8 * 32
    assert np.all(np.isfinite(a)) and np.array_equal(a[large], b[large])


MANY = [320] + [1 + 5 * i % 40 for i in range(63)]     # one group of ten tiles, 63 of one or two


@pytest.mark.parametrize("F,q4,expect", [
    (384, False, dict(ffn_up=1, ffn_up_tiled=0)),      # 6 tiled units beside 189 streamed workgroups: all streamed
    (256, False, dict(ffn_up=1, ffn_up_tiled=1)),      # 4 beside 126: fewer than half of the compute units
    (1792, True, dict(ffn_up=1, ffn_up_tiled=0)),      # 924 workgroups in passes of four: every group takes them
    (1024, True, dict(ffn_up=1, ffn_up_tiled=0)),      # 528, the large group a 22nd of them: one launch, passes of two
    (256, True, dict(ffn_up=2, ffn_up_tiled=0)),       # 132: the large group in passes of four of its own
])
def test_one_large_group_among_many_small(oracle_mod, F, q4, expect):
    """Where a group of a tiled one's size runs, by what runs beside it: each rule of the plan, by the launches it makes."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="groups_many", d=256, E=64, F=F, F_shared=0, k=1)
    run_groups(oracle_mod, cfg, MANY, q4, {}, expect=expect)


@pytest.mark.parametrize("q4", [False, True], ids=["bf16", "int4"])
@pytest.mark.parametrize("sizes", ["one tile", "up to four tiles"], ids=lambda s: s.replace(" ", "_"))
def test_wide_shared_ffn_takes_slices_of_its_own(oracle_mod, sizes, q4):
    """A streamed shared FFN eleven times as wide as the experts: more K slices than theirs (the sums round differently from
    one slice count for all), in the kernels of one and two tiles per pass and of four."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="groups_wide", d=512, F=128, F_shared=1408, k=1)
    small = [n // 4 for n in SIZES[sizes]]             # the shared FFN sees every token: seven tiles at most
    out = run_groups(oracle_mod, cfg, small, q4, {}, expect=dict(ffn_up=1, ffn_up_tiled=0))
    same = run_groups(None, cfg, small, q4, dict(down_split_slice_counts=0))
    assert not np.array_equal(out, same)


@pytest.mark.parametrize("F,F_shared,ks", [(512, 2048, 0), (1024, 2048, 0), (512, 4096, 0), (512, 2048, 2)])
def test_tiled_shared_ffn_takes_slices_of_its_own(oracle_mod, F, F_shared, ks):
    """A tiled shared FFN of two to eight times the experts' width beside tiled and streamed groups: slice counts of their
    own in the second half, and one count for all where it is forced."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="groups_own", d=256, F=F, F_shared=F_shared, k=1)
    sizes = [330, 321, 40, 33, 1, 0, 100, 31]
    out = run_groups(oracle_mod, cfg, sizes, False, dict(down_k_slices=ks), expect=dict(ffn_up=1, ffn_up_tiled=1))
    same = run_groups(None, cfg, sizes, False, dict(down_split_slice_counts=0))
    assert np.linalg.norm(out - same) <= 1e-5 * np.linalg.norm(out)      # the order of 32-bit sums


@pytest.mark.parametrize("tens,early", [(4, True), (5, False), (6, True)])
def test_nine_tiles_join_the_tiled_launch_unless_they_fill_the_chip(oracle_mod, tens, early):
    """A group of nine tiles (44 units of a first half) beside `tens` groups of ten in the tiled launch: 220 units in all, from
    220 to 264 over the 256 compute units, and from 264 to 308.  The tiled launches' flops say which groups they held."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="groups_nine", d=256, F=2816, F_shared=0, k=1)
    sizes = ([288] + [320] * tens + [40, 0, 7])[:8]
    sizes += [0] * (8 - len(sizes))
    want = 4.0 * cfg.d * cfg.F * (320 * tens + (288 if early else 0))
    run_groups(oracle_mod, cfg, sizes, False, {}, expect=dict(ffn_up=int(not early or sum(sizes) > 288 + 320 * tens), ffn_up_tiled=1),
               flops=dict(ffn_up_tiled=want))


@pytest.mark.parametrize("sizes,expanded", [([1800, 1793], True),            # 1792 units, all in groups of 57 tiles
                                            ([1800, 1792, 300], False),      # 1680, and a group of ten tiles
                                            ([1792, 1792], False)])          # 1568
def test_q4_two_large_groups_are_expanded(sizes, expanded):
    """Seven rounds of tiled workgroups are enough where every tiled group has 32 tiles and more: the launches say which
    kernels ran, and both forms agree to the rounding of the intermediate activation."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name="groups_two", d=256, E=3, F=14336, F_shared=0, k=1)
    sizes = sizes + [0] * (3 - len(sizes))
    out = run_groups(None, cfg, sizes, True, {}, expect=dict(ffn_up=int(not expanded), ffn_up_tiled=int(expanded)))
    other = run_groups(None, cfg, sizes, True, dict(q4_expand_min_units=1 << 20 if expanded else 0))
    assert np.linalg.norm(out - other) <= 1e-3 * np.linalg.norm(other)


@pytest.mark.parametrize("F,sizes", [(384, [350, 449, 320, 480, 0, 600, 1, 7]), (128, [300] * 8), (2048, [512] * 8),
                                     (2048, [512] * 7 + [600])], ids=["33 units", "16 units", "256 units", "272 units"])
def test_tiled_first_half_in_unit_order(oracle_mod, F, sizes):
    """Up to 256 units the tiled first half takes them in order, uneven shares per XCD among them; past that, and without
    tiled_xcd_rotation, an eighth of every group.  The order changes no bit."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name=f"in_order_{F}_{sum(sizes)}", d=256, E=8, k=1, F=F)
    a = run_groups(oracle_mod if F < 2048 else None, cfg, sizes, False, {})
    b = run_groups(None, cfg, sizes, False, {"tiled_xcd_rotation": 0})
    assert np.array_equal(a, b)


@pytest.mark.parametrize("d,F,sizes,form", [
    (2048, 1024, [33, 48, 49, 50, 63, 64, 57, 40], "1, 2, 1"),       # second passes re-read 16 MiB of codes: passes of one
    (2048, 1152, [33, 48, 49, 50, 63, 64, 57, 40], "2, 2, 1"),       # 18 MiB
    (2048, 1024, [97, 50, 64, 33, 49, 16, 0, 5], "2, 2, 1"),         # a group of four tiles beside
    (256, 14336, [97, 128, 65, 96, 33, 1, 64, 127], "4, 1, 2"),      # 896 workgroups in passes of four
])
def test_q4_results_do_not_depend_on_what_is_resident(oracle_mod, d, F, sizes, form):
    """Passes of four, and of two over 49 tokens and more, multiply with weights rounded to fp16, narrower ones with the codes:
    the width is the layer's, so the bits are the same with every expert resident (one phase) and through a single cache slot
    (one expert per phase)."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name=f"groups_width_{d}_{F}", d=d, F=F, F_shared=0, k=1)
    a = run_groups(oracle_mod, cfg, sizes, True, {}, q4_forms=[form])
    b = run_groups(None, cfg, sizes, True, {}, slots=1)
    assert np.array_equal(a, b)


@pytest.mark.parametrize("d", [512, 640, 768, 896, 1280])
@pytest.mark.parametrize("sizes,form", [([1, 15, 16, 17, 31, 32, 0, 30], "1, 2, 1"), ([97, 33, 47, 48, 49, 63, 64, 1], "2, 2, 1")],
                         ids=["passes of one", "passes of two"])
def test_q4_k_range_in_halves(oracle_mod, d, sizes, form):
    """A first half of few workgroups cuts its K range in two, whole and half tiles, passes of two (the largest group has four
    tiles) on both sides of 48 tokens: halves of 4, 6 and 10 stages (one turn of the register ring, a turn and a tail, two and a
    tail) and, of an odd number of 128-input blocks, 6 + 4 and 8 + 6 (full passes of two: 5 + 5 and 7 + 7)."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name=f"groups_halves_{d}", d=d, F=256, F_shared=0, k=1)
    out = run_groups(oracle_mod, cfg, sizes, True, {}, q4_forms=[form])
    same = run_groups(None, cfg, sizes, True, dict(down_k_slices=2), q4_forms=[form])
    assert np.linalg.norm(out - same) <= 1e-5 * np.linalg.norm(out)      # the order of 32-bit sums


@pytest.mark.parametrize("d,F,sizes,form", [
    (384, 256, [1, 15, 16, 17, 31, 32, 0, 30], "1, 1, 1"),           # six stages: too few for halves
    (384, 256, [97, 33, 47, 48, 49, 63, 64, 1], "2, 1, 1"),
    (384, 4736, [1, 15, 16, 17, 31, 32, 8, 30], "1, 1, 2"),          # 296 workgroups
    (640, 4736, [33, 47, 48, 49, 63, 64, 34, 40], "2, 1, 2"),        # 296, second passes would re-read 23 MiB
])
def test_q4_undivided_k_range(oracle_mod, d, F, sizes, form):
    """The other forms of the 4-bit first half, at the same sizes: a ring of six stages, one turn of it,
    and for more workgroups than compute units one of four, a turn or two and a tail."""
    cfg = dataclasses.replace(synth.CONFIGS["tiny"], name=f"groups_whole_{d}_{F}", d=d, F=F, F_shared=0, k=1)
    run_groups(oracle_mod, cfg, sizes, True, {}, q4_forms=[form])

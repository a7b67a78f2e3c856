// Launch planner: the gate / grouping launches of routing and prediction, and the grouped FFN of one layer in
// phases (experts that are ready, experts whose copy is in flight, misses that wait for a slot), each phase
// split over the streaming and the tiled kernels.  Declarations and argument contracts of the entry points are
// in include/expertflow.h.
#include "ef_ctx.h"

#include <algorithm>
#include <cmath>

namespace efi {

const ef::GroupExport kNoExport{nullptr, nullptr, 0, 0, 0};

// One pass over `hidden`: optionally the current layer's own gate (routing outputs and grouping)
// and the gates of the next He layers (prediction outputs).  Wide launches are split over the gates.
int run_gates(ef_ctx *c, int layer, const void *hidden, int T, float beta, bool do_route, int He, int H_stride,
              const float *delta, const int32_t *tok2req, int32_t *topk_ids, float *topk_w, int32_t *counts,
              int32_t *offsets, int32_t *perm, int32_t *inv_perm, int32_t *pred_ids, int32_t *pred_hist,
              const ef::GroupExport &ex, const EfRouteScratch &rs, hipStream_t s) {
    const int E = c->cfg.n_experts, k = c->cfg.top_k, d = c->cfg.d_model;
    const int ntiles = (T + ef::kTile - 1) / ef::kTile;
    const int per_launch = ef::kMaxGates;
    const int total_gates = (do_route ? 1 : 0) + He;
    bool grouped = false;
    int32_t *hist_tiles = nullptr;
    for (int g0 = 0; g0 < total_gates; g0 += per_launch) {
        ef::GateArgs a{};
        a.h = static_cast<const uint16_t *>(hidden);
        a.T = T; a.d = d; a.E = E; a.k = k;
        a.G = std::min(per_launch, total_gates - g0);
        a.beta = beta;
        a.tok2req = tok2req;
        a.delta = nullptr;
        a.delta_req_stride = H_stride * E;
        a.delta_gate_begin = 0;
        bool first_pred = true;
        for (int gi = 0; gi < a.G; ++gi) {
            const int gg = g0 + gi;                       // index over [route?] + predictions
            const bool is_route = do_route && gg == 0;
            const int j = gg - (do_route ? 1 : 0);        // prediction index (0-based) when !is_route
            const int ly = is_route ? layer : layer + 1 + j;
            const EfLayerReg &L = c->layers[(size_t)ly];
            a.Wg[gi] = L.gate_w;
            a.bias[gi] = L.gate_b;
            a.resident[gi] = resident_mask(c, ly);
            if (is_route) {
                a.ids[gi] = topk_ids;
                a.hist[gi] = nullptr;
                a.w = topk_w;
                a.blockcounts = rs.blockcounts;
                a.renorm = c->cfg.renorm_topk;
                a.routed_scale = c->cfg.routed_scale;
            } else {
                a.ids[gi] = pred_ids + (size_t)j * T * k;
                a.hist[gi] = pred_hist + (size_t)j * E;
                if (first_pred) {
                    a.delta_gate_begin = gi;
                    a.delta = delta ? delta + (size_t)j * E : nullptr;
                    first_pred = false;
                }
            }
        }
        a.gpw = ef::gate_pick_gpw(T, a.G, E);
        a.ksplit = ef::gate_pick_ksplit(T, d, a.G, E, a.gpw, rs.gate_part_floats);
        {
            const int forced = c->tune.gate_k_split;
            if (forced >= 1 && forced <= 16 &&
                (size_t)ntiles * ((a.G + a.gpw - 1) / a.gpw) * forced * ef::kTile * 128 <= rs.gate_part_floats)
                a.ksplit = forced;
        }
        a.part = rs.gate_part;
        a.tsplit = 1;
        // batches of many token tiles stream the hidden states through LDS in one kernel (no second step)
        a.stream = (c->tune.gate_stream != 0 && a.ksplit == 1 && ef::gate_stream_shape_ok(T, d, a.G, E, a.gpw)) ? 1 : 0;
        if (!a.stream) {   // the two-kernel form also pays off without a K split when the per-token part dominates
            const int ts = ef::gate_pick_tsplit(T, a.G, E, a.gpw);
            const size_t need = (size_t)ntiles * ((a.G + a.gpw - 1) / a.gpw) * a.ksplit * ef::kTile * 128;
            if (ts > 1 && need <= rs.gate_part_floats && c->tune.gate_token_split != 0) a.tsplit = ts;
        }
        a.two_step = (a.ksplit > 1 || a.tsplit > 1) ? 1 : 0;
        // histograms of the look-ahead: the library's own buffer is left zeroed by the hand-over step of the previous
        // layer; a caller's is written by the grouping, which adds per-tile counts up, from five tiles on, and cleared
        // here for the gates' atomics otherwise (a launch of 4 us)
        if (He > 0 && !ex.host_meta && g0 == 0) {
            if (do_route && total_gates <= per_launch && !a.two_step && ntiles > ef::kGroupSmallTiles)
                hist_tiles = rs.blockcounts + (size_t)ntiles * E;
            else EF_HIP(c, ef::launch_fill_i32(pred_hist, He * E, 0, s));
        }
        a.hist_tiles = hist_tiles;
        const bool has_route = do_route && g0 == 0;
        // decode-sized batches with a K-split gate and few experts: its second step and the grouping run as
        // one workgroup (with more than 16 experts a token takes a whole wave round of the epilogue, and the
        // many workgroups of the separate second step are faster: 27 against 36 us at 64 experts)
        const bool fused = has_route && total_gates <= per_launch && ntiles <= ef::kFusedMaxTiles && a.ksplit > 1 &&
                           E <= 16 &&
                           ef::gate_fused_lds_bytes(T, a.G, E, a.gpw) <= ef::kFusedMaxLds &&
                           c->tune.gate_fused_finish != 0;
        if (fused) a.tsplit = 1;
        {
            KernelTimer kt(c, s, has_route ? EF_K_ROUTE : EF_K_PREDICT,
                           (double)T * d * 2 + (double)a.G * E * d * 2 + (double)a.G * T * k * 4 +
                               (has_route ? (double)T * k * 4 + (double)ntiles * E * 4 : 0.0) +
                               (double)(a.G - (has_route ? 1 : 0)) * E * 4 +
                               (fused ? (double)(2 * E + 1) * 4 + (double)T * k * 12 : 0.0));
            if (fused) EF_HIP(c, ef::launch_gate_fused(a, counts, offsets, perm, inv_perm, ex, s));
            else EF_HIP(c, ef::launch_gate(a, s));
        }
        if (fused) grouped = true;
    }
    if (do_route && !grouped) {
        KernelTimer kt(c, s, EF_K_GROUP, (double)ntiles * E * 8 + (double)(2 * E + 1) * 4 + (double)T * k * 12);
        EF_HIP(c, ef::launch_group(rs.blockcounts, topk_ids, T, k, E, rs.blockbase, counts, offsets, perm,
                                   inv_perm, hist_tiles, hist_tiles ? He : 0, pred_hist, ex, s));
    }
    return EF_OK;
}

int check_predict_args(ef_ctx *c, int layer, int T, int H, int *He_out, const char *who) {
    if (c->fake) return fail(c, EF_ENOSYS, "%s: fake-copy context has no device", who);
    if (H < 0 || H > EF_MAX_HORIZON) return fail(c, EF_EINVAL, "%s: H must be in 0..%d", who, EF_MAX_HORIZON);
    if (T < 0 || T > c->cfg.max_tokens) return fail(c, EF_EINVAL, "%s: T=%d outside 0..max_tokens", who, T);
    int He = std::max(0, std::min(H, c->cfg.n_layers - 1 - layer));
    for (int j = 1; j <= He; ++j)
        if (!c->layers[(size_t)(layer + j)].set)
            return fail(c, EF_EINVAL, "%s: layer %d is not registered", who, layer + j);
    *He_out = He;
    return EF_OK;
}

int open_layer_timer(ef_ctx *c, hipStream_t s) {
    poll_pairs(c, false);
    if ((c->layer_calls++ % kLayerTimerEvery) != 0) return EF_OK;
    c->layer_cur = next_pair(c->layer_ring, c->layer_next, c->layer_pending);
    EF_HIP(c, hipEventRecord(c->layer_cur.a, s));
    c->layer_open = true;
    return EF_OK;
}

}  // namespace efi

using namespace efi;

namespace {

struct PhaseGroup {
    int expert;  // -1: dense shared FFN
    int slot;
};
constexpr int kNoSplit = -2;

// The tiled second half of a layer is `before` workgroups of one time unit each, dealt in order to the 256 compute
// units, then `units` more of the layer's last tiled group.  With that group cut into s K slices its workgroups
// take 1/s of a unit each: the time, in units, until the last one ends.
double tiled_tail_makespan(long long before, long long units, int s) {
    const long long q = before / 256, r = before % 256;   // r compute units are busy until q + 1, the others until q
    for (long long step = 1;; ++step) {
        const long long cap = (256 - r) * step + r * std::max<long long>(0, step - s);
        if (cap >= units * s) return (double)q + (double)step / s;
    }
}

// Whether a group of n_tiles token tiles takes the tiled kernels: every shared FFN that fits them, routed groups from
// tiled_min_tiles tiles on, and one tile earlier where passes of four would end in a pass of a single tile, a whole read of
// the weights for it (groups of 9: Mixtral-shaped 1000 tokens 2050 -> 1942 us for two layers, DeepSeek-shaped 1056 tokens
// 784 -> 776; groups of 8 stay streamed: DeepSeek-shaped 2000 tokens on 16 experts 883 against 905 us).  `early`: whether the
// layer's groups take them one tile earlier (early_tiled).
bool ends_in_one_tile(const ef_ctx *c, int n_tiles) { return n_tiles == c->tune.tiled_min_tiles - 1 && n_tiles % 4 == 1; }
bool takes_tiled(const ef_ctx *c, int F, int n_tiles, bool routed, bool early) {
    if (!ef::ffn_tiled_ok(c->cfg.d_model, F, n_tiles)) return false;
    return !routed || n_tiles >= c->tune.tiled_min_tiles || (early && ends_in_one_tile(c, n_tiles));
}

// The earlier line costs more than it saves where it takes the last free compute units: the streamed launch has fewer
// workgroups than there are units, and the groups it adds bring the tiled first half from less than a round to (nearly) all
// of one, so that the streamed workgroups wait for the tiled ones (DeepSeek-shaped on 16 experts, 660 / 680 tokens, 206 and 209
// units without them: 452 -> 426 / 468 -> 446 us for two layers; Qwen-shaped on 12 experts, 680 tokens 422 -> 413; with 198
// units in all, 580 tokens, the earlier line saves 2 %, and from 270 on 1 to 2 %).
bool early_tiled(const ef_ctx *c, const int32_t *counts_host, bool has_shared, int T) {
    if (c->q4) return true;
    bool any = false;
    for (int e = 0; e < c->cfg.n_experts; ++e) any = any || ends_in_one_tile(c, (counts_host[e] + ef::kTile - 1) / ef::kTile);
    if (!any) return true;
    long long with = 0, without = 0, streamed = 0;   // tiled units with and without those groups, streamed workgroups without
    auto add = [&](int F, int cnt, bool routed) {
        const int nt = (cnt + ef::kTile - 1) / ef::kTile, units = ef::ffn_tiled_units(F / 128, nt, 1);
        if (takes_tiled(c, F, nt, routed, true)) with += units;
        if (takes_tiled(c, F, nt, routed, false)) without += units;
        else streamed += (long long)(F / 128) * ((nt + 3) / 4);
    };
    for (int e = 0; e < c->cfg.n_experts; ++e) add(c->cfg.d_ff, counts_host[e], true);
    if (has_shared) add(c->cfg.d_ff_shared, T, false);
    return streamed > 256 || with <= 224 || without >= 240;
}

// Token tiles per pass over a streamed group's weights, for a launch whose largest group has `max_tiles` and whose first
// half would have `wgs_of_four` workgroups in passes of four, beside `tiled_wgs` of a tiled one.  16-bit: groups of three or
// more tiles (too few for the tiled kernels) take passes of four, which halves the re-reads of their weights, and where the
// largest has five or more and the chip has more workgroups than compute units, streamed or tiled, passes of eight: a group of
// up to eight tiles reads its weights once (two layers, passes of four / eight: Mixtral-shaped 300 / 350 / 700 tokens 1219 /
// 1110, 1278 / 1139, 1619 / 1480 us, two experts 200 tokens 556 / 454; DeepSeek-shaped 1056 tokens 711 / 694, on 16 experts
// with 385 tiled workgroups 551 / 524).  With fewer every workgroup has a unit to itself, and the longer ones end the launch
// (Qwen-shaped on 12 experts, 121 streamed and 231 tiled, 640 tokens 357 / 413; DeepSeek-shaped on 16, 176 and 198, 600 tokens
// 372 / 380; d = 512, 56 and 40, 700 tokens 147 / 155).  Tiled workgroups are counted as a multiple of
// eight per group: with 240 to 256 that do not exit at once the streamed ones wait for units all the same (Qwen-shaped on 12
// experts, 700 / 760 tokens 409 / 399, 434 / 420; DeepSeek-shaped on 16, 700 tokens 416 / 419).  A set lds_shared_occupancy
// asks for a form of the passes of four.  4-bit: passes of four dequantise half as often, but a pass is twice as long; they
// pay from 7/4 rounds of two workgroups per compute unit on (two layers, passes of two / four: Mixtral-shaped 200 tokens, 1008
// workgroups, 574 / 538 us; DeepSeek-shaped 1000 tokens, 1085, 564 / 515; Qwen-shaped 640 tokens, 835, 408 / 442; DeepSeek-
// shaped 300 tokens, 671, 289 / 312).
// Passes of one although some group has two tiles (4-bit): their kernels fit three workgroups per compute unit and issue less,
// while second passes re-read no more than 16 MiB of first-half codes (`wgs_second` of their workgroups; two layers, passes of
// two / one: DeepSeek-shaped 36 / 52 tokens 147.8 / 141.0, 156.5 / 152.0, on 16 experts 52 / 60 136.9 / 131.3, 139.3 / 138.1;
// Qwen-shaped 36 / 60 147.2 / 137.2, 151.9 / 147.9, on 12 experts 60 tokens 134.2 / 128.8; Mixtral-shaped, 56 MiB per second
// pass, 48 tokens on four experts 224.2 / 258.8, on eight 338.0 / 357.7).
constexpr long long kSecondPassWeights = 16ll << 20;
int tiles_per_pass(const ef_ctx *c, int max_tiles, long long wgs_of_four, long long wgs_second, long long tiled_wgs) {
    if (max_tiles >= 5 && (wgs_of_four > 256 || tiled_wgs > 256) && c->tune.passes_of_four != 0 && !c->q4 &&
        c->tune.lds_shared != 0 && c->tune.lds_shared_occupancy == 0 && c->cfg.d_ff % 128 == 0 && c->cfg.d_ff_shared % 128 == 0)
        return 8;
    if (max_tiles >= 3 && c->tune.passes_of_four != 0 && (!c->q4 || wgs_of_four >= 896)) return 4;
    if (max_tiles == 2 && c->q4 && wgs_second * c->cfg.d_model <= kSecondPassWeights / 128) return 1;
    return max_tiles >= 2 ? 2 : 1;
}

// Build the launch tables of one phase and enqueue both FFN halves.
int launch_phase(ef_ctx *c, int layer, const std::vector<PhaseGroup> &groups, const int32_t *counts_host,
                 const std::vector<int> &offs_host, const std::vector<int> &tile_start,
                 const std::vector<long long> &act_off, int shared_tile_start, long long shared_act_off, int T,
                 int tpp_layer, int ksg_stream, int ksg_shared, int ksg_tiled, int split_expert, int split_ksg,
                 ef::PlaneTable &planes, long long y_plane, bool use_tiled, bool early, bool expand, bool side_waits,
                 bool *forked, hipStream_t s) {
    // tpp_layer: token tiles per pass that the layer's streamed groups would take in one launch.
    // split_expert: the tiled group of the layer (expert id, -1 = shared FFN, kNoSplit = none) whose second half takes
    // split_ksg K slices instead of ksg_tiled; it goes last among the tiled groups of its launch.  expand: the tiled groups
    // of a 4-bit context are expanded to 16 bits first (else they run in passes of four tiles on the 4-bit blobs).
    // side_waits: the side stream already waits for what this phase needs.  *forked: whether the phase took both streams
    if (groups.empty()) return EF_OK;
    const int d = c->cfg.d_model, k = c->cfg.top_k;
    // groups with many tokens go to the tiled (matrix-core bound) kernels, the others to the
    // weight-streaming kernels; at most two launches per FFN half
    ef::GroupTable gu{}, big{};
    ef::DequantTable dq{};
    int streamed[ef::kMaxGroups];   // expert of each group of `gu`
    int n = 0, nb = 0, max_tiles = 1;
    bool large = false;   // 4-bit: a streamed group has a tiled one's size
    const bool allow_tiled = use_tiled;
    // Workgroups start in index order; groups with the most work go first so that the launch's last round holds
    // the short ones (the groups are independent: the order changes no result)
    std::vector<PhaseGroup> ordered(groups);
    if (c->tune.sort_groups != 0) {
        auto work = [&](const PhaseGroup &pg) {
            const long long cnt = pg.expert < 0 ? T : counts_host[pg.expert];
            const long long F = pg.expert < 0 ? c->cfg.d_ff_shared : c->cfg.d_ff;
            return ((cnt + ef::kTile - 1) / ef::kTile) * F;
        };
        std::stable_sort(ordered.begin(), ordered.end(),
                         [&](const PhaseGroup &a, const PhaseGroup &b) { return work(a) > work(b); });
    }
    if (split_expert != kNoSplit) {
        auto it = std::find_if(ordered.begin(), ordered.end(), [&](const PhaseGroup &pg) { return pg.expert == split_expert; });
        if (it != ordered.end()) std::rotate(it, it + 1, ordered.end());
    }
    int split_grp = -1;
    for (const PhaseGroup &pg : ordered) {
        int cnt, ts, F, ro;
        long long ao;
        const void *blob;
        if (pg.expert < 0) {
            cnt = T; ts = shared_tile_start; F = c->cfg.d_ff_shared; ro = T * k; ao = shared_act_off;
            blob = c->layers[(size_t)layer].shared_blob;
        } else {
            cnt = counts_host[pg.expert]; ts = tile_start[(size_t)pg.expert]; F = c->cfg.d_ff;
            ro = offs_host[(size_t)pg.expert]; ao = act_off[(size_t)pg.expert];
            blob = c->pool + (size_t)pg.slot * c->expert_bytes;
        }
        const int nt = (cnt + ef::kTile - 1) / ef::kTile;
        const bool tiled = allow_tiled && takes_tiled(c, F, nt, pg.expert >= 0, early) &&
                           (!c->q4 || !expand || nb < c->q4_stage_slots);
        ef::GroupTable &g = tiled ? big : gu;
        int &i = tiled ? nb : n;
        if (tiled && c->q4 && expand) {   // the tiled kernels read a 16-bit copy written just before them on the same stream
            void *copy = c->q4_stage + (size_t)nb * c->q4_stage_bytes;
            dq.F[nb] = F; dq.src[nb] = blob; dq.dst[nb] = copy;
            blob = copy;
        }
        if (!tiled) streamed[i] = pg.expert;
        const bool split = tiled && split_expert != kNoSplit && pg.expert == split_expert;
        if (split) split_grp = nb;
        (pg.expert < 0 ? planes.shared : planes.routed[pg.expert]) =
            (uint8_t)(split ? split_ksg : tiled ? ksg_tiled : pg.expert < 0 ? ksg_shared : ksg_stream);
        g.tile_start[i] = ts; g.n_tiles[i] = nt; g.row_offset[i] = ro;
        g.ksg[i] = pg.expert < 0 ? planes.shared : planes.routed[pg.expert];
        g.count[i] = cnt; g.F[i] = F; g.act_off[i] = ao; g.blob[i] = blob;
        if (!tiled) {
            max_tiles = std::max(max_tiles, nt);
            large = large || (c->q4 && c->tune.tiled != 0 && takes_tiled(c, F, nt, pg.expert >= 0, early));
        }
        ++i;
    }
    gu.n_groups = n;
    big.n_groups = nb;
    // weights: 2 bytes each, or half a byte plus one bf16 scale per 128
    const double wb = c->q4 ? 0.5 + 2.0 / 128.0 : 2.0;
    auto alg_bytes = [&](const ef::GroupTable &g, int cnt_groups, double &b_up, double &b_dn) {
        for (int i = 0; i < cnt_groups; ++i) {
            b_up += 2.0 * wb * d * g.F[i] + 2.0 * g.count[i] * d + 2.0 * g.count[i] * g.F[i];
            b_dn += wb * d * g.F[i] + 2.0 * g.count[i] * g.F[i] + 4.0 * g.count[i] * d;
        }
    };
    // A phase with both kinds of groups runs its streamed launches on the side stream, beside the tiled ones: the two touch
    // different groups (tiles of the packed tokens, activations, rows of Y), small tiled launches leave half of the compute
    // units idle, and the streamed kernels are bound by HBM, not by compute units.  Fork: the side stream waits for
    // everything enqueued so far (the token packing, the previous layer's un-permute); ef_layer_step has made it wait behind
    // the packing while the routing ran where the previous layer forked too (13-16 us of host time that the compute units
    // would otherwise idle through), else it waits for an event here.  Join: the caller's stream waits behind the last
    // side-stream launch before anything after this phase.  Both events are completion events of the launches themselves: a
    // separate record is a packet of its own (other stream 8.5 us after the forking kernel instead of 11.6, its own stream
    // 2.6 instead of 5.7, join 7 instead of 11).
    // Once `forked`, whatever path leaves this function (an error included) makes the caller's stream wait for the side
    // stream: the caller releases the phase's cache slots behind its own stream, and kernels still running on the side
    // stream read those slots.
    struct SideJoin {
        ef_ctx *c;
        hipStream_t s;
        bool forked = false;
        hipEvent_t join = nullptr;   // completion of the last side-stream launch, once that has been enqueued
        hipError_t wait() {
            if (!forked) return hipSuccess;
            hipError_t e = hipSuccess;
            if (!join) {
                join = next_fork_event(c);
                e = hipEventRecord(join, c->side_stream);
            }
            if (e == hipSuccess) e = hipStreamWaitEvent(s, join, 0);
            forked = false;
            return e;
        }
        ~SideJoin() { (void)wait(); }
    } side{c, s};
    const bool forks = n > 0 && nb > 0 && c->side_stream && c->tune.overlap_tiled != 0;
    if (forks && !side_waits) {
        hipEvent_t fork = next_fork_event(c);
        EF_HIP(c, hipEventRecord(fork, s));
        EF_HIP(c, hipStreamWaitEvent(c->side_stream, fork, 0));
    }
    side.forked = *forked = forks;
    hipStream_t gs = forks ? c->side_stream : s;   // of the streamed launches
    int tiled_up_wgs = 0, tiled_dn_wgs = 0;
    double tb_up = 0.0, tb_dn = 0.0, tf_up = 0.0, tf_dn = 0.0;
    ef::GroupTable bdn = big;
    if (nb > 0) {
        int wg_up = 0, wg_dn = 0;
        // Workgroups go to the XCDs round-robin by index and hold one of an XCD's 32 compute units for their whole
        // K loop.  An XCD takes an eighth of a group's units; the eighths differ by one unit, and each group starts on the
        // XCD that leaves the fullest XCD of the launch least full.
        int load_up[8] = {}, load_dn[8] = {};
        const int rot_on = c->tune.tiled_xcd_rotation;
        auto place = [&](int units, int (&load)[8]) {
            int best = 0, best_max = 1 << 30;
            for (int rot = 0; rot < (rot_on ? 8 : 1); ++rot) {
                int mx = 0;
                for (int x = 0; x < 8; ++x) {
                    const int part = (x - rot) & 7;
                    mx = std::max(mx, load[x] + ef::tiled_xcd_begin(units, part + 1) - ef::tiled_xcd_begin(units, part));
                }
                if (mx < best_max) { best_max = mx; best = rot; }
            }
            for (int x = 0; x < 8; ++x) {
                const int part = (x - best) & 7;
                load[x] += ef::tiled_xcd_begin(units, part + 1) - ef::tiled_xcd_begin(units, part);
            }
            return best;
        };
        int units_up = 0;
        for (int i = 0; i < nb; ++i) units_up += ef::ffn_tiled_units(big.F[i] / 128, big.n_tiles[i], 1);
        const bool in_order = rot_on && units_up <= ef::kTiledInOrderUnits;
        for (int i = 0; i < nb; ++i) {
            big.wg_start[i] = wg_up;
            bdn.wg_start[i] = wg_dn;
            if (c->q4 && !expand) {
                wg_up += ef::ffn_gate_up_q4_wgs(big.F[i], big.n_tiles[i], 4);
                wg_dn += ef::ffn_down_q4_wgs(d, big.n_tiles[i], 4, ksg_tiled);
                continue;
            }
            const int ks = i == split_grp ? split_ksg : ksg_tiled;
            const int nu = ef::ffn_tiled_units(big.F[i] / 128, big.n_tiles[i], 1);
            big.xcd_rot[i] = in_order ? ef::kTiledInOrder : place(nu, load_up);
            bdn.xcd_rot[i] = place(ef::ffn_tiled_units(d / 256, big.n_tiles[i], ks), load_dn);
            wg_up += in_order ? nu : ef::ffn_tiled_wgs(nu);
            tiled_up_wgs += ef::ffn_tiled_wgs(nu);   // what the rules below count, whatever the order
            wg_dn += ef::ffn_down_tiled_wgs(d, big.n_tiles[i], ks);
        }
        big.wg_start[nb] = wg_up;
        if (c->q4 && !expand) tiled_up_wgs = wg_up;
        bdn.wg_start[nb] = wg_dn;
        tiled_dn_wgs = wg_dn;
        alg_bytes(big, nb, tb_up, tb_dn);
        for (int i = 0; i < nb; ++i) {
            tf_up += 4.0 * big.count[i] * d * big.F[i];   // two d x F products, 2 flops per multiply-add
            tf_dn += 2.0 * big.count[i] * d * big.F[i];
        }
    }
    auto tiled_up = [&]() -> int {
        if (c->q4 && !expand) {   // passes of four on the 4-bit blobs: counted with the streamed launches
            KernelTimer kt(c, s, EF_K_FFN_UP, tb_up);
            EF_HIP(c, ef::launch_ffn_gate_up_q4(big, tiled_up_wgs, 4, false, c->xp, c->act, d, s));
            return EF_OK;
        }
        KernelTimer kt(c, s, EF_K_FFN_UP_TILED, tb_up, tf_up);   // 4-bit: the expansion is timed with the first half
        if (c->q4) {
            dq.n = nb;
            EF_HIP(c, ef::launch_dequant_q4(dq, d, s));
        }
        EF_HIP(c, ef::launch_ffn_gate_up_tiled(big, big.wg_start[nb], c->xp, c->act, d, c->q4, s));
        return EF_OK;
    };
    auto tiled_down = [&]() -> int {
        if (c->q4 && !expand) {
            KernelTimer kt(c, s, EF_K_FFN_DOWN, tb_dn);
            EF_HIP(c, ef::launch_ffn_down_q4(bdn, tiled_dn_wgs, 4, c->act, c->y, y_plane, d, nullptr, s));
            return EF_OK;
        }
        KernelTimer kt(c, s, EF_K_FFN_DOWN_TILED, tb_dn, tf_dn);
        EF_HIP(c, ef::launch_ffn_down_tiled(bdn, tiled_dn_wgs, ksg_tiled, split_grp, split_ksg, c->act, c->y, y_plane, d, s));
        return EF_OK;
    };
    // both first halves before the second ones: the stream that is served last waits for one launch call, not for two
    int rc = nb > 0 ? tiled_up() : EF_OK;
    if (rc) return rc;
    if (n == 0) return tiled_down();
    ef::GroupTable dn = gu;
    long long wgs_of_four = 0;
    for (int i = 0; i < n; ++i) wgs_of_four += (long long)(gu.F[i] / 128) * ((gu.n_tiles[i] + 3) / 4);
    // 4-bit: passes of four, and full ones of two, multiply with weights rounded to fp16, all others with the codes, so every
    // phase keeps to the layer's width whatever is resident (a width of one where a phase has no second tile is the same
    // arithmetic as two).  Groups of a tiled one's size stream because of what the whole layer holds; a phase that has one
    // does not cut the first half's K range in two either: such a group's sums do not depend on the phase it runs in
    const int tpp = !c->q4 ? tiles_per_pass(c, max_tiles, wgs_of_four, 0, tiled_up_wgs)
                           : tpp_layer == 2 && max_tiles == 1 ? 1 : tpp_layer;
    // K slices inside a workgroup of the first half: split while the launch has too few waves to
    // keep enough weight bytes in flight, as long as a slice keeps >= 16 fragments
    long long units = 0;
    for (int i = 0; i < n; ++i) units += (long long)(gu.F[i] / 32) * ((gu.n_tiles[i] + tpp - 1) / tpp);
    int ks = 1;
    const int want_waves = c->tune.up_want_waves, nkb = d / 16;
    while (ks < 4 && units * ks < want_waves && nkb / (ks * 2) >= 16) ks *= 2;
    if (c->tune.up_k_slices > 0) ks = c->tune.up_k_slices;
    // passes of four tiles and more: the kernels whose four waves share the token / activation fragments through LDS
    // (per-wave copies of them would be twice the weights' bytes from L2)
    bool shared = tpp >= 4 && !c->q4 && c->tune.lds_shared != 0;
    for (int i = 0; i < n && shared; ++i) shared = gu.F[i] % 128 == 0;
    int wg_gu = 0, wg_dn = 0;
    for (int i = 0; i < n; ++i) {
        gu.wg_start[i] = wg_gu;
        dn.wg_start[i] = wg_dn;
        if (shared) {
            if (const int ksg = ef::ffn_down_shared_slices(gu.F[i], gu.ksg[i]); ksg < gu.ksg[i]) {
                gu.ksg[i] = dn.ksg[i] = ksg;
                (streamed[i] < 0 ? planes.shared : planes.routed[streamed[i]]) = (uint8_t)ksg;
            }
            wg_gu += ef::ffn_gate_up_shared_wgs(gu.F[i], gu.n_tiles[i], tpp);
            wg_dn += ef::ffn_down_shared_wgs(d, gu.n_tiles[i], tpp, gu.ksg[i]);
            continue;
        }
        wg_gu += c->q4 ? ef::ffn_gate_up_q4_wgs(gu.F[i], gu.n_tiles[i], tpp)
                       : ef::ffn_gate_up_wgs(gu.F[i], gu.n_tiles[i], tpp, ks);
        wg_dn += c->q4 ? ef::ffn_down_q4_wgs(d, gu.n_tiles[i], tpp, gu.ksg[i])
                       : ef::ffn_down_wgs(d, gu.n_tiles[i], tpp, gu.ksg[i]);
    }
    gu.wg_start[n] = wg_gu;
    dn.wg_start[n] = wg_dn;
    double b_up = 0.0, b_dn = 0.0;
    alg_bytes(gu, n, b_up, b_dn);
    // Workgroups per compute unit of the LDS-shared kernels: two (register ring of two stages each) or one (ring of three).
    // A tiled workgroup holds its unit's LDS.  Two for a launch that has most of the chip to itself and more workgroups than
    // units (64 DeepSeek-shaped experts, 200 tokens, 440 us with two against 452 for two layers, Qwen-shaped 250 tokens 418 /
    // 424), with the long streams of a large model dimension more than two per unit (eight Mixtral-shaped experts, 130 tokens
    // 1026 / 1050; two experts, 448 workgroups, 200 tokens 560 / 520), and for one of at most a
    // workgroup per unit beside a tiled launch of more than one round: its workgroups start where a tiled one has ended and
    // are done sooner in pairs (DeepSeek-shaped on 16 experts, 700 / 1056 / 1700 tokens 472 -> 460 / 592 -> 541 / 755 -> 703
    // us, Qwen-shaped on 12, 1056 tokens 587 -> 565; 850 tokens 495 -> 500).  One otherwise: beside less than a round of
    // tiled ones there are units without any (DeepSeek-shaped 600 tokens on 16 experts 397 against 425, Qwen-shaped 640 on
    // 12 389 / 418), and a long streamed launch beside a long tiled one is better off with the deeper ring (64 experts, 1300
    // tokens 797 / 865, Qwen-shaped 3000 tokens 1192 / 1280, Mixtral-shaped 1000 tokens 2035 / 2105).
    // A few short workgroups wait for their instructions more than for anything else, and the shorter ring has a third less
    // of them (d = 512, eight experts, 130 / 230 tokens 112.1 -> 108.6 / 113.8 -> 110.1 us).
    const bool pairs = tiled_up_wgs < 128 ? wg_gu > (d > 2048 ? 512 : 256) || (wg_gu <= 128 && d <= 1024) : tiled_up_wgs > 256 && wg_gu <= 256;
    const int occ = c->tune.lds_shared_occupancy != 0 ? c->tune.lds_shared_occupancy : pairs ? 2 : 1;
    {
        KernelTimer kt(c, gs, EF_K_FFN_UP, b_up);
        if (shared) EF_HIP(c, ef::launch_ffn_gate_up_shared(gu, wg_gu, tpp, occ, c->xp, c->act, d, gs));
        else if (c->q4) EF_HIP(c, ef::launch_ffn_gate_up_q4(gu, wg_gu, tpp, !large, c->xp, c->act, d, gs));
        else EF_HIP(c, ef::launch_ffn_gate_up(gu, wg_gu, tpp, ks, c->xp, c->act, d, gs));
    }
    if (nb > 0 && (rc = tiled_down())) return rc;
    {
        KernelTimer kt(c, gs, EF_K_FFN_DOWN, b_dn);
        hipEvent_t done = forks ? next_fork_event(c) : nullptr;
        if (shared) EF_HIP(c, ef::launch_ffn_down_shared(dn, wg_dn, tpp, occ, c->act, c->y, y_plane, d, done, gs));
        else if (c->q4) EF_HIP(c, ef::launch_ffn_down_q4(dn, wg_dn, tpp, c->act, c->y, y_plane, d, done, gs));
        else EF_HIP(c, ef::launch_ffn_down(dn, wg_dn, tpp, c->act, c->y, y_plane, d, done, gs));
        side.join = done;
    }
    EF_HIP(c, side.wait());
    return EF_OK;
}

}  // namespace

extern "C" int ef_moe_ffn(ef_ctx *c, int layer, const void *hidden, int T, const int32_t *topk_ids,
                          const float *topk_w, const int32_t *counts_host, const int32_t *offsets,
                          const int32_t *perm, const int32_t *inv_perm, float *out, void *stream) {
    // set by ef_layer_step for the call it makes right afterwards; never survive this call
    const bool prepacked = c && c->prepacked, side_waits = prepacked && c->side_waits;
    if (c) c->prepacked = c->side_waits = false;
    int rc = check_ctx_layer(c, layer);
    if (rc) return rc;
    if (T < 0 || T > c->cfg.max_tokens) return fail(c, EF_EINVAL, "ef_moe_ffn: T=%d outside 0..max_tokens", T);
    if (!counts_host) return fail(c, EF_EINVAL, "ef_moe_ffn: counts_host is null");
    const int E = c->cfg.n_experts, k = c->cfg.top_k, d = c->cfg.d_model;
    long long tot = 0;
    for (int e = 0; e < E; ++e) {
        if (counts_host[e] < 0 || counts_host[e] > T)
            return fail(c, EF_EINVAL, "ef_moe_ffn: counts_host[%d]=%d outside 0..T", e, counts_host[e]);
        tot += counts_host[e];
    }
    if (tot != (long long)T * k) return fail(c, EF_EINVAL, "ef_moe_ffn: counts_host sums to %lld, not T*k", tot);
    if (!c->fake && T > 0) {
        if (!hidden || !topk_ids || !topk_w || !offsets || !perm || !inv_perm || !out)
            return fail(c, EF_EINVAL, "ef_moe_ffn: null pointer");
        if (!aligned16(hidden) || !aligned16(out)) return fail(c, EF_EINVAL, "ef_moe_ffn: hidden/out must be 16-byte aligned");
    }
    hipStream_t s = static_cast<hipStream_t>(stream);
    const bool strict = (c->cfg.flags & EF_FLAG_STRICT_RESIDENT) != 0;
    poll_all_copies(c);
    if (T > 0) {   // how much of what this layer uses had the look-ahead of j layers ago named?
        uint64_t used = 0;
        for (int e = 0; e < E; ++e)
            if (counts_host[e] > 0) used |= 1ull << e;
        for (int j = 0; j < EF_MAX_HORIZON; ++j) {
            const size_t at = (size_t)layer * EF_MAX_HORIZON + j;
            if (!c->pred_valid[at]) continue;
            c->pred_valid[at] = 0;
            c->st.pred_overlap_hits[j] += __builtin_popcountll(used & c->pred_mask[at]);
            c->st.pred_overlap_total[j] += __builtin_popcountll(used);
        }
    }

    // host copies of the group geometry
    std::vector<int> offs_host((size_t)E + 1, 0), tile_start((size_t)E, 0);
    std::vector<long long> act_off((size_t)E, 0);
    int tiles = 0;
    for (int e = 0; e < E; ++e) {
        offs_host[(size_t)e + 1] = offs_host[(size_t)e] + counts_host[e];
        tile_start[(size_t)e] = tiles;
        act_off[(size_t)e] = (long long)tiles * ef::kTile * c->cfg.d_ff / 8;   // 16-byte units
        tiles += (counts_host[e] + ef::kTile - 1) / ef::kTile;
    }
    const bool has_shared = c->cfg.d_ff_shared > 0 && T > 0;
    const int shared_tile_start = tiles;
    const long long shared_act_off = (long long)tiles * ef::kTile * c->cfg.d_ff / 8;
    if (has_shared) tiles += (T + ef::kTile - 1) / ef::kTile;
    if (!c->fake && tiles > c->max_tiles) return fail(c, EF_EINVAL, "ef_moe_ffn: scratch too small (internal)");

    // K slices of the second FFN half across workgroups (one Y plane each, summed by the un-permute):
    // split while the layer's launch would have too few workgroups, a slice keeps >= 32 fragments per
    // wave and the planes fit the scratch.  One value per call: every phase shares the planes.
    const long long y_plane = ((long long)T * k + (has_shared ? T : 0)) * d;
    // Groups of many token tiles (takes_tiled) go to the matrix-core tiled kernels, unless the rules below say otherwise.
    // The two thresholds (total workgroups of the tiled launches) exist for tuning only: on the mixed batches measured (640
    // tokens with a 2048 x 5632 shared expert, 1056 tokens over 64 experts) the tiled kernels were equal to or 8 % faster
    // than streaming the same groups in several passes, even at 150-200 workgroups.
    bool use_tiled = false;
    const bool early = early_tiled(c, counts_host, has_shared, T);
    // 4-bit contexts: the tiled groups are expanded to 16 bits and go through the 256 x 256 tiles when the groups of 32
    // tiles and more alone make eight rounds of those over the compute units; below that the expansion (a pass over 2.5
    // bytes per weight ahead of the first half) and the tiles' fixed costs outweigh them, and the groups run in passes of
    // four token tiles on the 4-bit blobs, dequantised between the matrix instructions.  Two layers, expanded / direct:
    // Mixtral-shaped 4000 tokens on two experts 4610 / 5350 us, 2000 tokens on eight 3050 / 3080; DeepSeek-shaped 4000
    // tokens 1560 / 1459, 2000 tokens on 16 experts 873 / 778; Qwen-shaped 3000 tokens 1120 / 1026.
    bool q4_expand = false;
    long long passes_of_four_dn = 0;   // workgroups of a second half of the tiled groups in passes of four
    long long tiled_up_units = 0, tiled_up_wgs = 0;   // of the tiled first half; its launch rounds up to eight per group
    long long tiled_dn_wgs = 0, tiled_rows = 0;
    int tiled_stages_min = 1 << 30;   // fewest K stages (32 columns each) among the tiled groups
    int tiled_stages_max = 0;         // ... and most
    if (T > 0 && c->tune.tiled != 0) {
        long long wg_up = 0, wg_dn = 0, wg_up_large = 0;
        auto add = [&](int F, int cnt, bool routed) {
            const int nt = (cnt + ef::kTile - 1) / ef::kTile;
            if (!takes_tiled(c, F, nt, routed, early)) return;
            wg_up += ef::ffn_tiled_units(F / 128, nt, 1);
            tiled_up_wgs += ef::ffn_gate_up_tiled_wgs(F, nt);
            if (nt >= ef::kQ4ExpandTiles) wg_up_large += ef::ffn_tiled_units(F / 128, nt, 1);
            passes_of_four_dn += ef::ffn_down_q4_wgs(d, nt, 4, 1);
            wg_dn += ef::ffn_tiled_units(d / 256, nt, 1);
            tiled_rows += cnt;
            tiled_stages_min = std::min(tiled_stages_min, F / 32);
            tiled_stages_max = std::max(tiled_stages_max, F / 32);
        };
        for (int e = 0; e < E; ++e) add(c->cfg.d_ff, counts_host[e], true);
        if (has_shared) add(c->cfg.d_ff_shared, T, false);
        use_tiled = wg_up >= c->tune.tiled_min_up_wgs && wg_dn >= c->tune.tiled_min_down_wgs;
        // Where every tiled group is that large, seven rounds do (Mixtral-shaped on two experts, 1700 / 2000 / 2300 tokens, 1568,
        // 1792 and 2016 units: direct 2360 / 2670 / 3210 us, expanded 2360 / 2540 / 2950; eight experts, 3300 tokens, smaller
        // groups beside: 4635 / 5215).
        q4_expand = c->q4_stage && wg_up_large >= ef::q4_expand_units(c->tune.q4_expand_min_units, wg_up_large == wg_up);
        // Groups that would not use what the tiled kernels offer run with the streamed ones: one launch per half instead of
        // two on two streams, whose fork and join cost about 10 us.  In passes of four token tiles:
        long long four_all = 0, four_tiled = 0;
        auto count = [&](int F, int cnt, bool routed) {
            const int nt = (cnt + ef::kTile - 1) / ef::kTile;
            const long long wgs = (long long)(F / 128) * ((nt + 3) / 4);
            four_all += wgs;
            if (takes_tiled(c, F, nt, routed, early)) four_tiled += wgs;
        };
        if (use_tiled) {   // a decode batch has none: nothing to look at (0.1 us of the host with 64 experts)
            for (int e = 0; e < E; ++e) count(c->cfg.d_ff, counts_host[e], true);
            if (has_shared) count(c->cfg.d_ff_shared, T, false);
        }
        if (c->q4 && !q4_expand) {
            // passes of four for all groups alike (tiles_per_pass), or tiled groups that are a quarter of the workgroups or
            // less (two layers: Mixtral-shaped 700 tokens 1245 -> 1188 us, DeepSeek-shaped 300 tokens 315 -> 286, 4000 tokens
            // 1560 -> 1459); a launch of their own is passes of four too
            if (c->tune.passes_of_four == 0 || tiles_per_pass(c, 4, four_all, 0, 0) == 4 ||
                (four_all >= 512 && four_tiled * 4 <= four_all))
                use_tiled = false;
        } else if (!c->q4 && wg_up < 64 && four_all - four_tiled >= 128 && c->tune.passes_of_four != 0 &&
                   c->tune.lds_shared != 0) {
            // fewer than 64 of the 256 x 256 tiles beside a streamed launch that covers half of the compute units (two
            // layers, tiled / all streamed: DeepSeek-shaped 260 tokens, 44 tiles, 526 / 479 us, on 16 experts 361 / 328;
            // Qwen-shaped 260 tokens on 12 experts, 88 tiles, 290 / 348 us)
            use_tiled = false;
        }
        tiled_up_units = wg_up;
        tiled_dn_wgs = wg_dn;
    }
    // K slices of the second half (one Y plane each, summed by the un-permute): the streamed launch and the tiled
    // launch of the layer choose separately, each for its own workgroup count
    int ksg = 1, ksg_shared = 1, ksg_tiled = 1, split_expert = kNoSplit, split_ksg = 1;
    int tpp = 1;
    if (T > 0) {
        long long base_wgs = 0;
        double streamed_w2_bytes = 0.0;   // second-half weights of the routed groups that stream (4-bit blobs)
        // token tiles per pass of the streamed launch: from the groups that stream (the tiled ones have kernels of
        // their own), with the rule that launch_phase applies to a phase's groups (16-bit; 4-bit phases take this width)
        int tmax = 1;
        long long wgs_of_four = 0, wgs_second = 0;
        auto see = [&](int F, int cnt) {
            const int nt = (cnt + ef::kTile - 1) / ef::kTile;
            tmax = std::max(tmax, nt);
            wgs_of_four += (long long)(F / 128) * ((nt + 3) / 4);
            if (nt > 1) wgs_second += F / 128;
        };
        auto streams = [&](int F, int cnt, bool routed) {
            const int nt = (cnt + ef::kTile - 1) / ef::kTile;
            return !(use_tiled && takes_tiled(c, F, nt, routed, early));
        };
        for (int e = 0; e < E; ++e)
            if (counts_host[e] > 0 && streams(c->cfg.d_ff, counts_host[e], true)) see(c->cfg.d_ff, counts_host[e]);
        if (has_shared && streams(c->cfg.d_ff_shared, T, false)) see(c->cfg.d_ff_shared, T);
        tpp = tiles_per_pass(c, tmax, wgs_of_four, wgs_second, use_tiled ? tiled_up_wgs : 0);
        double stream_work = 0.0;     // workgroups times their k-blocks
        double stream_bytes = 0.0;    // weights of the streamed groups, as often as their passes read them
        auto add_base = [&](int F, int nt) {
            const int wgs = c->q4 ? ef::ffn_down_q4_wgs(d, nt, tpp, 1)
                                  : tpp >= 4 ? ef::ffn_down_shared_wgs(d, nt, tpp, 1) : ef::ffn_down_wgs(d, nt, tpp, 1);
            base_wgs += wgs;
            stream_work += (double)wgs * (F / 16);
            stream_bytes += (c->q4 ? 1.55 : 6.0) * d * F * ((nt + tpp - 1) / tpp);
        };
        // workgroups of the streamed launch with one slice (groups that take the tiled kernels do not count)
        for (int e = 0; e < E; ++e)
            if (counts_host[e] > 0) {
                const int nt = (counts_host[e] + ef::kTile - 1) / ef::kTile;
                if (use_tiled && takes_tiled(c, c->cfg.d_ff, nt, true, early)) continue;
                streamed_w2_bytes += (0.5 + 2.0 / 128.0) * d * c->cfg.d_ff;
                add_base(c->cfg.d_ff, nt);
            }
        if (has_shared && streams(c->cfg.d_ff_shared, T, false)) add_base(c->cfg.d_ff_shared, (T + ef::kTile - 1) / ef::kTile);
        // the LDS-shared kernels run two workgroups per compute unit in passes of four, beside a tiled launch one (there
        // twice the workgroups only cost planes: DeepSeek-shaped 1056 tokens 772 -> 750 us for two layers, Mixtral-shaped 700
        // tokens 1655 -> 1625); in passes of eight they run one, but two shorter rounds are better than one (Mixtral-shaped
        // 300 / 350 tokens 1111 / 1140 us, for 256 workgroups 1133 / 1185)
        const int want = c->tune.down_want_wgs > 0 ? c->tune.down_want_wgs : (tpp >= 4 && !c->q4 && !use_tiled) ? 512 : 256;
        const int nkb_min = std::min(c->cfg.d_ff, has_shared ? c->cfg.d_ff_shared : c->cfg.d_ff) / 16;
        // a slice keeps >= 32 fragments per wave (bf16: four waves split it again), >= 6 quads (4-bit), or >= 8
        // stages of four fragments (LDS-shared kernels: a wave walks the whole slice)
        const int units = c->q4 ? nkb_min / 4 / 6 : tpp >= 4 ? nkb_min / 4 / 8 : nkb_min / 4 / 32;
        while (ksg < 8 && base_wgs * ksg < want && units / (ksg * 2) >= 1 && y_plane * (ksg * 2) <= c->y_floats)
            ksg *= 2;
        // 4-bit: two workgroups per compute unit (their waves stall at different times) while the planes this adds
        // cost little beside the weights, at most a quarter of their bytes written and read: eight Mixtral-shaped
        // experts 64 tokens 416 -> 390 us per two layers, 64 DeepSeek-shaped 100 tokens 210 -> 204 us; past that
        // the planes cost more than they gain (300 tokens, 0.4 of the weights' bytes: 385 -> 394 us).  Groups of one tile
        // each gain nothing (8 tokens 314.7 -> 318.0 us, 16 tokens 341.5 -> 349.7, 4 and 30 the same)
        if (c->q4 && tpp > 1 && c->tune.down_want_wgs == 0)
            while (ksg < 8 && base_wgs * ksg < 512 && units / (ksg * 2) >= 1 && y_plane * (ksg * 2) <= c->y_floats &&
                   8.0 * y_plane * ksg <= 0.25 * streamed_w2_bytes)
                ksg *= 2;
        // A streamed launch of a little more than one round of workgroups (two fit a compute unit: 512 at a time)
        // ends in a round that is mostly empty: 544 workgroups took 28 us where 512 took 22.5.  Twice the slices make
        // the rounds half as long; taken when that saves at least a tenth of a round and a wave keeps >= 8 fragments.
        if (!c->q4 && tpp <= 2 && c->tune.down_tail_split != 0 && c->tune.down_k_slices == 0) {
            const long long slots = 512, w = base_wgs * ksg;
            if (w > slots && ksg < 8 && nkb_min / (ksg * 2 * 4) >= 8 && y_plane * (ksg * 2) <= c->y_floats) {
                const double now = (double)((w + slots - 1) / slots);
                const double halved = (double)((2 * w + slots - 1) / slots) / 2.0;
                if (halved + 0.1 < now) ksg *= 2;
            }
        }
        if (use_tiled) {
            // the tiled second half: slices until its 256 x 256 tiles fill the chip, each slice keeping at least
            // 16 stages
            // (any count from 1 to 8: 40 tiles in 6 slices are 240 workgroups, one round over the 256 compute units
            // at a sixth of the length, where 8 slices are 320 workgroups, two rounds at an eighth; a plane more is
            // priced at what it takes to write and read)
            if (c->q4 && !q4_expand) {
                // passes of four tiles: slices by the same model; two workgroups per compute unit, a stage of 64 columns
                // about 1 us with both busy
                const int stages = tiled_stages_max / 2;
                const double plane_pen = (double)tiled_rows * d * 8.0 / 5e12 / (stages * 1e-6);
                double best = 0.0;
                for (int ks = 1; ks <= 8; ++ks) {
                    if (ks > 1 && (tiled_stages_min / 2 / ks < 6 || y_plane * ks > c->y_floats)) break;
                    const double t = (double)((passes_of_four_dn * ks + 511) / 512) / ks + (ks - 1) * plane_pen;
                    if (ks == 1 || t < best - 1e-9) { best = t; ksg_tiled = ks; }
                }
            } else if (tiled_dn_wgs < 256) {
                const int stages_ref = c->tune.down_slices_by_longest_k ? tiled_stages_max : tiled_stages_min;
                // Beside a streamed launch the tiled ones are hidden as long as both halves of them end before it does: then
                // a slice more only costs planes (Mixtral-shaped 400 tokens 1405 -> 1338 us for two layers).  The streamed
                // launches are taken at 5.5 TB/s of weights, which long ones reach; 110 workgroups of Qwen-shaped experts take
                // 92 us where this says 35, so short ones count as hiding less than they do
                const double unit_s = stages_ref * 0.77e-6;
                const double plane_s = (double)tiled_rows * d * 8.0 / 5e12, stream_s = stream_bytes / 5.5e12;
                const double up_s = (double)((tiled_up_units + 255) / 256) * (d / 32) * 0.6e-6;
                double best = 0.0;
                for (int ks = 1; ks <= 8; ++ks) {
                    if (ks > 1 && (stages_ref / ks < 16 || y_plane * ks > c->y_floats)) break;
                    const double t = std::max(up_s + (double)((tiled_dn_wgs * ks + 255) / 256) / ks * unit_s, stream_s) +
                                     (ks - 1) * plane_s;
                    if (ks == 1 || t < best - 1e-9) { best = t; ksg_tiled = ks; }
                }
                // A shared FFN beside routed groups has a K of its own: with a slice count of its own too, both kinds end at
                // about the same time (K 5632 and 1408 in three slices each are 59 and 15 stages on 240 workgroups, in four
                // and one 44 each on 152).  Within one round of workgroups, where the longest decides; a workgroup costs 10 us
                // of a compute unit whatever its length.  Two layers, one count / two: Qwen-shaped on 12 experts 400 / 560 /
                // 640 / 720 / 760 / 800 / 1000 / 1200 tokens 317 / 306, 332 / 317, 346 / 340, 402 / 396, 418 / 404, 424 / 413,
                // 495 / 457, 609 / 529, on 60 1000 tokens 654 / 596; DeepSeek-shaped on 16 300 / 400 / 600 / 700 / 760 tokens
                // 326 / 317, 344 / 332, 367 / 354, 424 / 390, 441 / 410.
                const int nt_shared = has_shared ? (T + ef::kTile - 1) / ef::kTile : 0;
                if (c->tune.down_split_slice_counts != 0 && has_shared &&
                    takes_tiled(c, c->cfg.d_ff_shared, nt_shared, false, early)) {
                    const int units_s = ef::ffn_tiled_units(d / 256, nt_shared, 1), units_r = (int)tiled_dn_wgs - units_s;
                    const int stages_s = c->cfg.d_ff_shared / 32, stages_r = c->cfg.d_ff / 32;
                    const double wg_s = 10e-6 / 256.0;
                    best += (double)tiled_dn_wgs * ksg_tiled * wg_s;
                    for (int kr = 1; kr <= 8 && units_r > 0; ++kr)
                        for (int kh = 1; kh <= 8; ++kh) {
                            if (kr == kh || units_r * kr + units_s * kh > 256 || y_plane * std::max(kr, kh) > c->y_floats ||
                                (kr > 1 && stages_r / kr < 16) || (kh > 1 && stages_s / kh < 16))
                                continue;
                            const double longest = std::max((double)stages_r / kr, (double)stages_s / kh);
                            const double planes_s = ((double)(tiled_rows - T) * (kr - 1) + (double)T * (kh - 1)) * d * 8.0 / 5e12;
                            const double t = std::max(up_s + longest * 0.77e-6, stream_s) + planes_s + (units_r * kr + units_s * kh) * wg_s;
                            if (t < best - 1e-9) { best = t; ksg_tiled = kr; split_expert = -1; split_ksg = kh; }
                        }
                }
            }
            if (c->tune.down_split_slice_counts == 0) ksg = ksg_tiled;   // one slice count for both launches
        }
        // A shared FFN that streams with the routed experts has a K of its own.  It gets more slices, down to about the routed
        // ones' length, while one of its workgroups runs half as long again as the launch's work spread over two workgroups
        // per compute unit (Qwen-shaped, K 5632 against 1408, two layers: 100 tokens on 12 experts 253 -> 207 us, 200 tokens
        // 420 -> 393, one token 150 -> 124).  The routed ones' length is what keeps its slices from getting too short; where the other groups fill that time anyway, more planes only cost
        // (DeepSeek-shaped 32 tokens on 16 experts 183.7 -> 185.8, 4-bit 1000 tokens 508 -> 518).
        ksg_shared = ksg;
        if (has_shared && c->tune.down_split_slice_counts != 0) {
            const int ratio = (c->cfg.d_ff_shared + c->cfg.d_ff / 2) / c->cfg.d_ff;
            while (ksg_shared < 8 && ksg_shared < ksg * ratio && y_plane * (ksg_shared + 1) <= c->y_floats &&
                   (double)(c->cfg.d_ff_shared / 16) / ksg_shared > 1.5 * stream_work / 512.0)
                ++ksg_shared;
        }
        int forced = c->tune.down_k_slices;
        if (forced >= 1 && forced <= 8 && y_plane * forced <= c->y_floats) {
            ksg = ksg_shared = ksg_tiled = forced;
            split_expert = kNoSplit;
        }
        // A tiled second half of more than one round of workgroups over the compute units ends in a round that is
        // partly empty (1056 workgroups: four rounds and an eighth; every compute unit holds one at a time).  The
        // layer's last tiled group (the one with the least work; the highest expert among equals) is cut into K
        // slices so that its shorter workgroups fill that round: the slice count with the least modelled time,
        // a Y plane more costing what the second half and the un-permute take to write and read it.  The choice
        // depends on the layer's token counts only, never on what is resident.
        if (use_tiled && (!c->q4 || q4_expand) && ksg_tiled == 1 && forced < 1 && tiled_dn_wgs > 256 && c->tune.tiled_tail_slices != 0) {
            long long best_work = -1, units = 0, rows = 0;
            int F_last = 0;
            auto consider = [&](int expert, int F, int cnt, bool routed) {
                const int nt = (cnt + ef::kTile - 1) / ef::kTile;
                if (!takes_tiled(c, F, nt, routed, early)) return;
                const long long work = (long long)nt * F;
                if (best_work < 0 || work <= best_work) {
                    best_work = work; split_expert = expert; units = ef::ffn_tiled_units(d / 256, nt, 1); rows = cnt; F_last = F;
                }
            };
            if (has_shared) consider(-1, c->cfg.d_ff_shared, T, false);
            for (int e = 0; e < E; ++e) consider(e, c->cfg.d_ff, counts_host[e], true);
            if (split_expert != kNoSplit) {
                const double unit_s = (F_last / 32) * 0.77e-6;                        // one workgroup: its K stages
                const double plane_units = (double)rows * d * 8.0 / 5e12 / unit_s;     // write + read of one more plane
                double best = 0.0;
                for (int sl = 1; sl <= 8; sl *= 2) {
                    if (F_last / 32 / sl < 16 || y_plane * sl > c->y_floats) break;
                    const double t = tiled_tail_makespan(tiled_dn_wgs - units, units, sl) + (sl - 1) * plane_units;
                    if (sl == 1 || t < best - 1e-9) { best = t; split_ksg = sl; }
                }
                const int want = c->tune.tiled_tail_slices;   // 1: the modelled best; 2, 4, 8: that count if it fits
                if (want > 1 && F_last / 32 / want >= 16 && y_plane * want <= c->y_floats) split_ksg = want;
                if (split_ksg == 1) split_expert = kNoSplit;
            }
        }
    }
    ef::PlaneTable planes{};

    // classify the needed experts
    std::vector<PhaseGroup> ready, loading;
    std::vector<int> missing;
    bool any_not_ready = false;
    for (int e = 0; e < E; ++e) {
        if (counts_host[e] == 0) continue;
        int slot = c->cache->lookup(layer, e);
        if (slot < 0) {
            if (strict) {
                for (const auto &g : ready) c->cache->pin(g.slot, false);
                for (const auto &g : loading) c->cache->pin(g.slot, false);
                return fail(c, EF_ENOTRESIDENT, "ef_moe_ffn: layer %d expert %d is not resident", layer, e);
            }
            missing.push_back(e);
            any_not_ready = true;
            c->st.misses += 1;
            continue;
        }
        c->st.hits += 1;
        if (c->slots[(size_t)slot].prefetched_unused) {
            c->slots[(size_t)slot].prefetched_unused = false;
            c->st.prefetch_used += 1;
        }
        c->cache->touch(slot);
        c->cache->pin(slot, true);
        if (c->slots[(size_t)slot].copy_pending) { loading.push_back({e, slot}); any_not_ready = true; }
        else ready.push_back({e, slot});
    }
    // feedback counters (paper Sec. 3.2.2): a layer that had to wait counts as a stall, a layer
    // whose experts were all loaded in time counts as an overfetch
    if (T > 0) {
        if (any_not_ready) {
            if (++c->stall_counter >= std::max(1, c->cfg.stall_thresh)) { c->stall_counter = 0; c->fb_adjust += 1; }
        } else {
            if (++c->overfetch_counter >= std::max(1, c->cfg.overfetch_thresh)) { c->overfetch_counter = 0; c->fb_adjust -= 1; }
        }
        c->fb_adjust = std::max(-(c->cfg.h_max - 1), std::min(c->cfg.h_max - 1, c->fb_adjust));
    }

    auto unpin_all = [&](const std::vector<PhaseGroup> &v) {
        for (const auto &g : v)
            if (g.expert >= 0) c->cache->pin(g.slot, false);
    };
    // start what misses can start right now (slots not needed by this layer)
    std::vector<int> deferred;
    for (int e : missing) {
        int slot = -1;
        int r = swap_in_impl(c, layer, e, 1, 0, &slot, nullptr);
        if (r == EF_EBUSY) { deferred.push_back(e); continue; }
        if (r != EF_OK) { unpin_all(ready); unpin_all(loading); return r; }
        c->cache->touch(slot);
        c->cache->pin(slot, true);
        loading.push_back({e, slot});
    }

    // A slot may be overwritten once the kernels that read it have finished: an event recorded behind them
    // is what a later swap-in waits for.  One event behind the layer's last kernel serves every slot of the
    // layer; only when misses are still waiting for a slot (phase C) must each phase's slots be released as
    // soon as that phase's kernels are enqueued.
    const bool eager_marks = !deferred.empty();
    std::vector<int> read_slots;
    // An error return between the phases must not leave the collected slots pinned, and kernels already
    // enqueued may still read them: they are released behind an event on the stream, like on the normal path.
    struct PinGuard {
        ef_ctx *c;
        hipStream_t s;
        std::vector<int> *v;
        ~PinGuard() {
            if (v->empty()) return;
            hipEvent_t ev = nullptr;
            if (!c->fake) {
                ev = c->read_ring[c->read_next];
                c->read_next = (c->read_next + 1) % c->read_ring.size();
                if (hipEventRecord(ev, s) != hipSuccess) ev = nullptr;
            }
            for (int slot : *v) {
                if (ev) c->slots[(size_t)slot].last_read = ev;
                c->cache->pin(slot, false);
            }
        }
    } pin_guard{c, s, &read_slots};
    auto mark_read = [&](const std::vector<PhaseGroup> &v) -> int {
        if (c->fake) { unpin_all(v); return EF_OK; }
        if (!eager_marks) {
            for (const auto &g : v)
                if (g.expert >= 0) read_slots.push_back(g.slot);
            return EF_OK;   // still pinned: released behind the layer's last kernel
        }
        hipEvent_t ev = c->read_ring[c->read_next];
        c->read_next = (c->read_next + 1) % c->read_ring.size();
        EF_HIP(c, hipEventRecord(ev, s));
        for (const auto &g : v)
            if (g.expert >= 0) c->slots[(size_t)g.slot].last_read = ev;
        unpin_all(v);
        return EF_OK;
    };
    auto release_read_slots = [&]() -> int {
        if (read_slots.empty()) return EF_OK;
        hipEvent_t ev = c->read_ring[c->read_next];
        c->read_next = (c->read_next + 1) % c->read_ring.size();
        hipError_t he = hipEventRecord(ev, s);
        for (int slot : read_slots) {
            c->slots[(size_t)slot].last_read = ev;
            c->cache->pin(slot, false);
        }
        read_slots.clear();
        if (he != hipSuccess) return fail(c, EF_EHIP, "hipEventRecord failed: %s", hipGetErrorString(he));
        return EF_OK;
    };
    auto wait_loaded = [&](const std::vector<PhaseGroup> &v) -> int {
        if (v.empty()) return EF_OK;
        std::vector<int> slots;
        for (const auto &g : v) slots.push_back(g.slot);
        if (c->fake) {
            const double need = fake_copy_wait(c, slots.data(), (int)slots.size());
            c->st.stall_seconds += need - c->fake_now;
            c->fake_now = need;
            for (const auto &g : v) poll_copy(c, g.slot);
            return EF_OK;
        }
        EfEventPair p = next_pair(c->stall_ring, c->stall_next, c->stall_pending);
        EF_HIP(c, hipEventRecord(p.a, s));
        // copies still (partly) in the queue become priority copies; once every chunk of them is on the copy
        // stream their ready events exist and the compute stream can wait for them
        int fr = copy_engine_flush(c, slots.data(), (int)slots.size());
        if (fr) return fr;
        for (const auto &g : v) EF_HIP(c, hipStreamWaitEvent(s, c->slots[(size_t)g.slot].ready, 0));
        EF_HIP(c, hipEventRecord(p.b, s));
        c->stall_pending.push_back(p);
        return EF_OK;
    };
    auto run_phase = [&](std::vector<PhaseGroup> &v, bool with_shared) -> int {
        std::vector<PhaseGroup> g = v;
        if (with_shared && has_shared) g.push_back({-1, -1});
        if (!c->fake) {
            bool forked = false;
            int r = launch_phase(c, layer, g, counts_host, offs_host, tile_start, act_off, shared_tile_start,
                                 shared_act_off, T, tpp, ksg, ksg_shared, ksg_tiled, split_expert, split_ksg, planes, y_plane, use_tiled,
                                 early, q4_expand, with_shared && side_waits, &forked, s);
            if (with_shared) c->forks = forked;
            if (r) {   // part of the phase may be enqueued: its slots still get their read marker
                (void)mark_read(v);
                v.clear();   // released: the caller's error path has nothing left to unpin
                return r;
            }
        }
        return mark_read(v);
    };

    if (T > 0) {
        if (!c->fake && !prepacked) {
            // token permutation into per-expert tiles (all groups of this layer in one launch)
            ef::PackTable pt{};
            int n = 0;
            for (int e = 0; e < E; ++e) {
                if (counts_host[e] == 0) continue;
                pt.tile_start[n] = tile_start[(size_t)e];
                pt.row_offset[n] = offs_host[(size_t)e];
                pt.count[n] = counts_host[e];
                ++n;
            }
            if (has_shared) {
                pt.tile_start[n] = shared_tile_start;
                pt.row_offset[n] = -1;
                pt.count[n] = T;
                ++n;
            }
            pt.tile_start[n] = tiles;
            pt.n_groups = n;
            int r = EF_OK;
            long long rows = (long long)T * k + (has_shared ? T : 0);
            KernelTimer kt(c, s, EF_K_PACK, 4.0 * rows * d + 4.0 * T * k);
            hipError_t he = ef::launch_pack_x(pt, tiles, static_cast<const uint16_t *>(hidden), d, k, perm, c->xp, c->q4, s);
            if (he != hipSuccess) r = fail(c, EF_EHIP, "pack_x launch failed: %s", hipGetErrorString(he));
            if (r) { unpin_all(ready); unpin_all(loading); return r; }
        }
        // phase A: experts that are ready (+ the dense shared FFN): tokens whose experts are resident go first
        rc = run_phase(ready, true);
        if (rc) { unpin_all(loading); return rc; }
        // phase B: experts whose copy is in flight (earlier prefetches and the misses started above)
        if (!loading.empty()) {
            rc = wait_loaded(loading);
            if (!rc) rc = run_phase(loading, false);
            if (rc) { unpin_all(loading); return rc; }
        }
        // phase C: misses that had no slot until an earlier phase released one
        size_t next = 0;
        while (next < deferred.size()) {
            std::vector<PhaseGroup> wave;
            while (next < deferred.size()) {
                int slot = -1;
                int r = swap_in_impl(c, layer, deferred[next], 1, 0, &slot, nullptr);
                if (r == EF_EBUSY) break;
                if (r != EF_OK) { unpin_all(wave); return r; }
                c->cache->touch(slot);
                c->cache->pin(slot, true);
                wave.push_back({deferred[next], slot});
                ++next;
            }
            if (wave.empty()) return fail(c, EF_EBUSY, "ef_moe_ffn: no cache slot can be freed for layer %d", layer);
            rc = wait_loaded(wave);
            if (!rc) rc = run_phase(wave, false);
            if (rc) { unpin_all(wave); return rc; }
        }
        if (!c->fake) {
            KernelTimer kt(c, s, EF_K_COMBINE, 4.0 * ((double)T * k + (has_shared ? T : 0)) * d + 4.0 * T * d +
                                                   8.0 * T * k);
            // the layer's last kernel carries the read marker of the slots collected above
            hipEvent_t done = nullptr;
            if (!read_slots.empty()) {
                done = c->read_ring[c->read_next];
                c->read_next = (c->read_next + 1) % c->read_ring.size();
            }
            EF_HIP(c, ef::launch_combine(c->y, planes, y_plane, topk_w, topk_ids, inv_perm, T, k, d,
                                         has_shared ? (long long)T * k : -1ll, out, done, s));
            if (done) {
                for (int slot : read_slots) {
                    c->slots[(size_t)slot].last_read = done;
                    c->cache->pin(slot, false);
                }
                read_slots.clear();
            }
        }
    }
    if ((rc = release_read_slots())) return rc;
    if (!c->fake && c->layer_open) {
        EF_HIP(c, hipEventRecord(c->layer_cur.b, s));
        c->layer_pending.push_back(c->layer_cur);
        c->layer_open = false;
    }
    c->st.layers_run += 1;
    c->st.tokens_run += T;
    c->cache->advance(layer);
    return EF_OK;
}


// Internal launch interface between the C-ABI layer and the gfx950 kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>

namespace ef {

constexpr int kMaxE = 64;      // experts per layer
constexpr int kMaxK = 8;       // top-k
constexpr int kMaxGates = 8;   // gate matrices per launch (look-ahead + 1)
constexpr int kTile = 32;      // tokens per tile (rows of one matrix-core operand fragment)
constexpr int kMaxGroups = kMaxE + 1;  // routed experts + the dense shared FFN
constexpr int kDownColBlocks = 2;      // 32-column blocks per wave in the second FFN half

constexpr int kGroupSmallTiles = 4;    // token tiles the single-workgroup grouping kernel handles
constexpr int kGroupSumsWords = 16384; // per-tile counts (tiles x experts) that the single-launch one adds up

// Gate / predict launch: G gate matrices applied to the same hidden states.
struct GateArgs {
    const uint16_t *h;             // [T,d] bf16
    int T, d, E, k, G;
    const uint16_t *Wg[kMaxGates]; // [E,d] bf16 each
    const float *bias[kMaxGates];  // [E] or null
    uint64_t resident[kMaxGates];  // bit e: expert e of that gate's layer is in the cache
    float beta;
    const float *delta;            // f32 or null: delta[req*delta_req_stride + (gate-delta_gate_begin)*E + e]
    int delta_req_stride;
    int delta_gate_begin;          // gates below this index take no delta (the current layer's own gate)
    const int32_t *tok2req;        // [T] or null
    int32_t *ids[kMaxGates];       // per gate: [T,k]
    float *w;                      // [T,k] combine weights of gate 0, or null
    int renorm;
    float routed_scale;
    int32_t *hist[kMaxGates];      // per gate: [E] accumulated with integer atomics, or null
    int32_t *blockcounts;          // [ntiles,E] per-tile counts of gate 0, or null
    int gpw;                       // gates per workgroup (gpw * E <= 128 logit columns)
    int ksplit;                    // workgroups that share the K range of one (tile, gate group); >= 1
    int two_step;                  // 1: gate_kernel leaves partial logits, gate_finish_kernel does the per-token part
    int tsplit;                    // two_step: workgroups that share the 32 tokens of a tile in the finish (1, 2, 4)
    float *part;                   // two_step: [tiles][groups][ksplit][32][32 * column blocks] partial logits
    int stream;                    // 1: launches that qualify (gate_stream_ok) take the streaming form of the kernel
    int32_t *hist_tiles;           // null, or [G-1][ntiles][E]: gates 1.. leave per-tile counts here and `hist` alone
                                   // (one-step launches with gate 0 = the current layer; the grouping adds them up)
};

// Grouped FFN launch: one group per active expert (+ one for the dense shared FFN).
struct GroupTable {
    int n_groups;
    int wg_start[kMaxGroups + 1];  // first workgroup of each group in this launch (cumulative)
    int tile_start[kMaxGroups];    // first 32-row tile of the group in the packed X / activation space
    int n_tiles[kMaxGroups];
    int row_offset[kMaxGroups];    // first row of the group in Y (= offsets[e]; T*k for the shared FFN)
    int count[kMaxGroups];         // rows in the group
    int F[kMaxGroups];             // FFN hidden dim of the group
    long long act_off[kMaxGroups]; // first 16-byte unit of the group's activation fragments
    const void *blob[kMaxGroups];  // packed weights (cache slot or shared blob)
    int ksg[kMaxGroups];           // streamed second half: K slices of the group (one Y plane each); a whole word comes with
                                   // the scalar loads of the other fields, a byte is a vector load of its own ahead of
                                   // everything else (4-bit Mixtral-shaped decode of one token 149.6 against 148.6 us)
    int xcd_rot[kMaxGroups];       // tiled kernels: the XCD (0..7) that takes the first eighth of the group's units, or
                                   // kTiledInOrder
};

// Optional hand-over of counts and predicted histograms to the host (host-mapped memory): every word is
// (tag << 24) | value, value < 2^24, tag = `seq` in 0..254 (the caller's sequence number modulo 255; the host
// marks words it has consumed, and the fresh buffer, with tag 255, which no call carries).
constexpr int kMetaHist = kMaxE;                          // hist starts after the E counts
constexpr int kMetaInts = kMaxE + (kMaxGates - 1) * kMaxE;
constexpr int kMetaValueBits = 24;
struct GroupExport {
    int32_t *host_meta;   // device view of the host-mapped buffer, or null
    int32_t *hist;        // [n_hist] device histograms to copy out; [n_clear] is zeroed afterwards
    int n_hist;
    int n_clear;
    int seq;
};

// Describes how rows are gathered into tiles for the X packing kernel.
struct PackTable {
    int n_groups;
    int tile_start[kMaxGroups + 1]; // cumulative over groups
    int row_offset[kMaxGroups];     // offsets[e] (index into perm); -1 = identity (shared FFN: row = token)
    int count[kMaxGroups];
};

hipError_t launch_fill_i32(int32_t *p, int n, int32_t v, hipStream_t s);
int gate_pick_gpw(int T, int G, int E);
constexpr size_t kGateSplitFloats = 960 * 1024;   // partial logits of a K-split gate launch (3.75 MiB), in any scratch
int gate_pick_ksplit(int T, int d, int G, int E, int gpw, size_t part_floats);
int gate_pick_tsplit(int T, int G, int E, int gpw);
hipError_t launch_gate(const GateArgs &a, hipStream_t s);
// batches of many token tiles: hidden states streamed through LDS by direct global -> LDS loads
bool gate_stream_ok(const GateArgs &a);
bool gate_stream_shape_ok(int T, int d, int G, int E, int gpw);
// decode-sized batches: K-split gate, then its second step and the grouping fused in one workgroup
constexpr int kFusedMaxTiles = 2;
constexpr size_t kFusedMaxLds = 48 * 1024;   // dynamic LDS of the fused kernel (logits of all pairs)
size_t gate_fused_lds_bytes(int T, int G, int E, int gpw);
hipError_t launch_gate_fused(const GateArgs &a, int32_t *counts, int32_t *offsets, int32_t *perm, int32_t *inv_perm,
                             const GroupExport &ex, hipStream_t s);
// n_hist > 0 (more than kGroupSmallTiles token tiles only): hist[j][E] = sums of the per-tile counts hist_tiles[j], j < n_hist
hipError_t launch_group(const int32_t *blockcounts, const int32_t *ids, int T, int k, int E, int32_t *blockbase,
                        int32_t *counts, int32_t *offsets, int32_t *perm, int32_t *inv_perm,
                        const int32_t *hist_tiles, int n_hist, int32_t *hist, const GroupExport &ex, hipStream_t s);
// f16: write fp16 instead of bf16 fragments (contexts with 4-bit experts).  `done` (here and below): null, or an event that
// is recorded as the launch's own completion
hipError_t launch_pack_x(const PackTable &pt, int total_tiles, const uint16_t *h, int d, int k,
                         const int32_t *perm, void *xp, bool f16, hipStream_t s);
hipError_t launch_pack_x_dev(const int32_t *counts, int E, bool has_shared, int T,
                             int max_tiles, const uint16_t *h, int d, int k, const int32_t *perm, void *xp,
                             bool f16, hipEvent_t done, hipStream_t s);
hipError_t launch_ffn_gate_up(const GroupTable &gt, int total_wgs, int tiles_per_pass, int ks, const void *xp,
                              void *act, int d, hipStream_t s);
hipError_t launch_ffn_down(const GroupTable &gt, int total_wgs, int tiles_per_pass, const void *act, float *y,
                           long long y_plane, int d, hipEvent_t done, hipStream_t s);
// K-slice planes of Y each expert's rows (and the shared FFN's) were written to: the streamed and the tiled launch
// of a layer choose their slice counts separately
struct PlaneTable {
    uint8_t routed[kMaxE];
    uint8_t shared;
};
hipError_t launch_combine(const float *y, const PlaneTable &planes, long long y_plane, const float *w,
                          const int32_t *ids, const int32_t *inv_perm, int T, int k, int d, long long shared_row0,
                          float *out, hipEvent_t done, hipStream_t s);

// 4-bit expert weights (d and F multiples of 128): a workgroup of the first half takes four 32-row
// blocks of F, one of the second half eight 32-column blocks of d and one of ksg K-slices
inline int ffn_gate_up_q4_wgs(int F, int n_tiles, int tiles_per_pass) {
    return (F / 128) * ((n_tiles + tiles_per_pass - 1) / tiles_per_pass);
}
inline int ffn_down_q4_wgs(int d, int n_tiles, int tiles_per_pass, int ksg) {
    return ((d / 32 + 7) / 8) * ((n_tiles + tiles_per_pass - 1) / tiles_per_pass) * ksg;
}
// k_halves: a launch of few workgroups may split K over two halves of a workgroup (a different order of the sums)
hipError_t launch_ffn_gate_up_q4(const GroupTable &gt, int total_wgs, int tiles_per_pass, bool k_halves, const void *xp,
                                 void *act, int d, hipStream_t s);
hipError_t launch_ffn_down_q4(const GroupTable &gt, int total_wgs, int tiles_per_pass, const void *act, float *y,
                              long long y_plane, int d, hipEvent_t done, hipStream_t s);
// Expands 4-bit expert blobs into 16-bit blobs of the bf16 layout whose elements are the fp16 numbers
// (q - 8) * s, the same values the 4-bit kernels form on the fly: large groups then run through the
// tiled matrix-core kernels, which read every weight many times.
struct DequantTable {
    int n;
    int F[kMaxGroups];
    const void *src[kMaxGroups];   // 4-bit blob (cache slot)
    void *dst[kMaxGroups];         // 3*d*F*2 bytes each
};
// A launch of large groups is expanded when those of this many token tiles and more make ef_tuning.q4_expand_min_units of
// the tiled first half's workgroups, or five sixths of that if no smaller group is tiled.
constexpr int kQ4ExpandTiles = 32;
inline int q4_expand_units(int min_units, bool only_large) { return only_large ? min_units - min_units / 6 : min_units; }
hipError_t launch_dequant_q4(const DequantTable &t, int d, hipStream_t s);

// Dist(t): scratch floats launch_token_dist needs for T tokens (norms, partials, workgroup sums)
size_t dist_scratch_floats(int T);
// Form 0 by batch size: up to kDistSmallMaxTokens tokens the squared differences (up to kDistRowMaxTokens one workgroup
// per token: fewer tokens than that share too little), up to kDistBlockMaxTokens Gram blocks
// of 32 x 32 or 64 x 64; both read the tokens as they are.  The other Gram forms read the packed copy, which the caller
// writes first.
constexpr int kDistRowMaxTokens = 64;
constexpr int kDistSmallMaxTokens = 256;
constexpr int kDistBlockMaxTokens = 3584;   // the call at T = 3500: 87 / 148 us (d = 2048 / 4096) against 106 / 156 us
                                            // through 256 x 256 blocks; from T = 4096 on those are level or ahead
inline bool dist_needs_packed(int T, int form) { return !(form == 0 && T <= kDistBlockMaxTokens); }
// 64 x 64 blocks once there are enough of them for half of the compute units, else 32 x 32 (the call with four waves for
// either, d = 2048 / 4096: T = 900 16.0 / 23.6 us with 32 x 32 against 19.5 / 30.2, T = 1200 22.7 / 33.2 against 20.4 /
// 30.5; not measured again with the eight waves that blocks of 64 x 64 take up to T = 1408)
inline bool dist_block_wide(int T) { return T > 960; }
// `form`: 0 = by batch size, 1 = register-fed 128 x 256 Gram blocks, 2 = 256 x 256 blocks through LDS (same bits)
hipError_t launch_token_dist(const uint16_t *h, int T, int d, const void *xp, float *scratch, float *tok_dist,
                             double *dist, int form, hipStream_t s);

// f16: the W1 / W3 fragments and the packed tokens hold fp16 instead of bf16 (4-bit contexts: the blobs are
// the staging copies launch_dequant_q4 wrote).  Activations and W2 fragments are fp16 in every context.
hipError_t launch_ffn_gate_up_tiled(const GroupTable &gt, int total_wgs, const void *xp, void *act, int d,
                                    bool f16, hipStream_t s);
// `split_grp` (or -1): the group of this launch whose slice count is `split_ksg` instead of `ksg`
hipError_t launch_ffn_down_tiled(const GroupTable &gt, int total_wgs, int ksg, int split_grp, int split_ksg,
                                 const void *act, float *y, long long y_plane, int d, hipStream_t s);

// The tiled (matrix-core bound) kernels take groups of at least kTiledMinTiles token tiles whose shapes
// fit their 256 x 256 workgroup tiles: F a multiple of 128 (4 row blocks), d a multiple of 256 (8 column
// blocks) and of 32 (whole k-step pairs).
constexpr int kTiledMinTiles = 8;
inline bool ffn_tiled_ok(int d, int F, int n_tiles) {
    return n_tiles >= kTiledMinTiles && F % 128 == 0 && d % 256 == 0;
}
// Workgroups are dealt to the 8 XCDs round-robin by index, and each XCD has an L2 of its own and 32 compute units that run
// one tiled workgroup each.  The units of a group (weight panel x token panel x K slice) are put in one order and every XCD
// takes an eighth of it, even to one unit, so that the 32 units an XCD runs side by side are neighbours in the order and
// share panels in its L2: K slices one after the other (units of one slice walk the same columns), strips of up to
// kTiledStrip token panels, weight panel by weight panel within a strip.  A full strip makes 32 neighbours 4 weight x 8
// token panels, 12 panels for 32 units; two weight panels x 16 token panels (the order before this one) read 18.
constexpr int kTiledStrip = 8;
struct TiledUnit { int np, mp, slice; };
inline __host__ __device__ int tiled_xcd_begin(int n_units, int xcd) { return (int)((long long)n_units * xcd / 8); }
inline __host__ __device__ TiledUnit tiled_unit(int u, int npanels, int mpanels) {
    const int tiles = npanels * mpanels, strips = (mpanels + kTiledStrip - 1) / kTiledStrip;
    const int w = (mpanels + strips - 1) / strips;
    const int slice = u / tiles, r = u - slice * tiles;
    const int strip = r / (w * npanels), rr = r - strip * w * npanels;
    const int width = mpanels - strip * w < w ? mpanels - strip * w : w;
    return TiledUnit{rr / width, strip * w + rr % width, slice};
}
inline int ffn_tiled_units(int npanels, int n_tiles, int slices) { return npanels * ((n_tiles + 7) / 8) * slices; }
// every XCD gets the same number of workgroups; those past an XCD's share of units exit at once
inline int ffn_tiled_wgs(int n_units) { return (n_units + 7) / 8 * 8; }
// A first half of at most a round of units (one per compute unit) takes them in order over all groups instead, an even share of
// the launch per XCD: that XCD's units come from one or two groups and share most of their panels, where an eighth of a small
// group is three units of a weight panel and up to three token panels each (DeepSeek-shaped 400 / 700 tokens, 110 / 220 units:
// 127 -> 78, 252 -> 142 MB past L2; Qwen-shaped 640 tokens, 231 units, 200 -> 130).  The kernel itself gains at 110 units (54 ->
// 47 us) and not from 209 on (52 -> 55, 56 -> 57); the streamed one beside it gains, which gets the compute units and the bytes.
// Two layers, eighths / in order: DeepSeek-shaped 300 / 400 / 700 tokens 463 / 456, 478 / 467, 584 / 575 us, on 16 experts 400
// tokens 327 / 317, 600 level; Qwen-shaped on 12 experts 300 / 500 / 640 tokens 289 / 286, 312 / 308, 334 / 332, on 60 level.
// Above a round the last units of an XCD's share run alone (DeepSeek-shaped on 16 experts 1700 tokens 654 -> 734), and second
// halves, whose units differ in length, lose as much as they gain.
constexpr int kTiledInOrder = -1;        // xcd_rot of every group of such a launch
constexpr int kTiledInOrderUnits = 256;
inline int ffn_gate_up_tiled_wgs(int F, int n_tiles) { return ffn_tiled_wgs(ffn_tiled_units(F / 128, n_tiles, 1)); }
inline int ffn_down_tiled_wgs(int d, int n_tiles, int slices) { return ffn_tiled_wgs(ffn_tiled_units(d / 256, n_tiles, slices)); }

// workgroups a group needs in the two FFN launches
inline int ffn_gate_up_wgs(int F, int n_tiles, int tiles_per_pass, int ks) {
    int nrb = F / 32, rbw = 4 / ks;
    return ((nrb + rbw - 1) / rbw) * ((n_tiles + tiles_per_pass - 1) / tiles_per_pass);
}
// LDS-shared streaming kernels (groups of a few token tiles, csrc/ef_ffn_shared.hip): a workgroup is four
// 32-row blocks of F (first half) or eight 32-column blocks of d (second half) for one pass of token tiles.
inline int ffn_gate_up_shared_wgs(int F, int n_tiles, int tiles_per_pass) {
    return (F / 128) * ((n_tiles + tiles_per_pass - 1) / tiles_per_pass);
}
inline int ffn_down_shared_wgs(int d, int n_tiles, int tiles_per_pass, int ksg) {
    return ((d / 32 + 7) / 8) * ((n_tiles + tiles_per_pass - 1) / tiles_per_pass) * ksg;
}
// Their K loops walk stages of 64 columns.  A K slice of the second half is the stages [begin(slice), begin(slice + 1)); a
// group takes at most one slice per stage (more would be planes of zeros).  Loads run ahead of the loop without a test: past
// the slice's end they read its last stage again, in an empty slice stage 0, so no load leaves the group's stages.
inline __host__ __device__ int shared_slice_begin(int stages, int slices, int slice) {
    return (int)((long long)slice * stages / slices);
}
inline __host__ __device__ int shared_last_stage(int end) { return end > 0 ? end - 1 : 0; }
inline __host__ __device__ unsigned shared_stage_offset(int stage, int last) {   // bytes: four fragments of 1 KiB
    return (unsigned)(stage < last ? stage : last) * 4096u;
}
inline int ffn_down_shared_slices(int F, int wanted) { return wanted < F / 64 ? wanted : F / 64; }
hipError_t launch_ffn_gate_up_shared(const GroupTable &gt, int total_wgs, int tiles_per_pass, int occ, const void *xp,
                                     void *act, int d, hipStream_t s);
hipError_t launch_ffn_down_shared(const GroupTable &gt, int total_wgs, int tiles_per_pass, int occ, const void *act, float *y,
                                  long long y_plane, int d, hipEvent_t done, hipStream_t s);
inline int ffn_down_wgs(int d, int n_tiles, int tiles_per_pass, int ksg) {
    return (d / 32 / kDownColBlocks) * ((n_tiles + tiles_per_pass - 1) / tiles_per_pass) * ksg;
}

}  // namespace ef

// Grouped SwiGLU expert FFN for launches whose largest group has a few token tiles (three or more, too many for one pass
// of the plain weight-streaming kernels; routed groups up to 9, beyond that the matrix-core tiled kernels, unless few tiled
// workgroups would run beside many streamed ones: ef_plan.hip).
//
// The plain streaming kernels give every wave its own copy of the token (or activation) fragments: with
// TT token tiles per pass a wave fetches TT KiB of them from L2 for every 2 KiB of weights, and at four
// tiles that traffic, not HBM, bounds the kernel.  Here the four waves of a workgroup work on the same
// token tiles and share those fragments through an LDS ring: each wave loads a quarter of a stage's
// fragments and every wave reads all of them from LDS, so L2 serves them once per workgroup.  Weights
// still stream straight from HBM into operand registers (1 KiB fragments, nontemporal), a register ring
// of three stages per wave, one barrier per stage of four k-blocks.
//
// Passes of four or eight tiles.  A second pass over a group's weights is read from HBM again: the two are not in step,
// and what the 64 workgroups of an XCD have in flight alone fills its L2 (numbering them so that both passes over a row block
// run on one XCD side by side changed nothing).  Eight tiles are 256 accumulator registers and 64 matrix instructions per
// stage and wave, 1 us for the 32 KiB of weights that a compute unit gets in 1.3 us at 6.3 TB/s: still bound by HBM
// (Mixtral-shaped 300 tokens, groups of up to six tiles, two layers 1219 -> 1110 us).
#include "ef_device.h"
#include "ef_kernels.h"

namespace ef {

constexpr int kShDepth = 3;   // register ring: stages in flight per wave (one workgroup per CU); the variants that
                              // fit two workgroups per CU (<= 256 registers) keep two stages (passes of eight with two and
                              // three: the same time)
constexpr int kShLds = 4;     // LDS ring of shared token / activation fragments (stages, power of two)

template <bool HALF>
__device__ __forceinline__ floatx16 shared_mfma(u32x4_t a, u32x4_t b, floatx16 c) {
    return HALF ? mfma32h(a, b, c) : mfma32v(a, b, c);
}

// K loop of either half for NTL live token tiles of a pass of TT (the same number for the whole workgroup; loads, LDS traffic
// and matrix-core work of tiles that do not exist are left out): stages [q0, q1) of four k-blocks, two weight streams per
// wave (wa: W1 or the first column block of W2, wb: W3 or the second).  src: the tiles' fragments.  Every pointer is uniform.
//
// A wave issues in order, and with one wave per SIMD nothing covers what it waits for, so each of the stage's 4 NTL pairs of
// matrix instructions (64 cycles) carries what would otherwise be a wait or a burst: the LDS read of the fragment three
// pairs on, and at most two of the global loads that refill the stage's registers as they fall free.  Against all reads just
// ahead of their use and all loads at the stage's end, two layers: Mixtral-shaped 300 / 700 / 1500 tokens 1102 / 1087, 1442 /
// 1385, 2342 / 2285 us, two experts 200 tokens 450 / 425, d = 512 130 tokens 103 / 96; DeepSeek- and Qwen-shaped the same.
template <int TT, int NTL, int D, bool HALF>
__device__ __forceinline__ void shared_stream(const char *__restrict__ wa, const char *__restrict__ wb,
                                              const char *const (&src)[TT], u32x4_t (*xs)[TT * 4][64], int q0, int q1, int wave,
                                              int lane, floatx16 (&A)[NTL], floatx16 (&B)[NTL]) {
    constexpr int N = 4 * NTL, LA = 3;
    u32x4_t fa[D][4], fb[D][4], xr[D][NTL], xb[LA + 1];
    const unsigned wo = lane * 16, xo = wave * 1024 + lane * 16;   // this wave loads k-block `wave` of each tile
    const int last = shared_last_stage(q1);
    // every load is unconditional (past the end the last stage is re-read, in bounds).  The token fragments are
    // requested before the weights: they are handed to the workgroup one stage before the weights of their
    // stage are used, and loads return in issue order, so waiting for them must not mean waiting for those weights
#define EF_SH_X(slot, u, at) xr[slot][u] = *reinterpret_cast<const u32x4_t *>(src[u] + (xo + (at)));
#define EF_SH_W(f, p, j, at) f = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>((p) + (wo + (at)) + 1024 * (j)));
    // one stage: hand the next stage's token fragments to the workgroup, compute this one while its registers are
    // refilled, barrier (the next stage's fragments are visible; this stage's LDS buffer is overwritten three stages on)
#define EF_SH_STAGE(slot, next_slot, st)                                                                 \
    {                                                                                                    \
        const unsigned at_ = shared_stage_offset((st) + D, last);                                        \
        u32x4_t(*const now_)[64] = xs[(st) & (kShLds - 1)];                                              \
        _Pragma("unroll") for (int i = 0; i < LA; ++i) xb[i] = now_[i % NTL * 4 + i / NTL][lane];        \
        _Pragma("unroll") for (int u = 0; u < NTL; ++u) xs[((st) + 1) & (kShLds - 1)][u * 4 + wave][lane] = xr[next_slot][u]; \
        __builtin_amdgcn_sched_barrier(0);                                                               \
        _Pragma("unroll") for (int i = 0; i < N; ++i) {                                                  \
            const int j = i / NTL, tt = i % NTL, n = i + LA;                                             \
            if (n < N) xb[n % (LA + 1)] = now_[n % NTL * 4 + n / NTL][lane];                             \
            A[tt] = shared_mfma<HALF>(fa[slot][j], xb[i % (LA + 1)], A[tt]);                             \
            if (j == 0) EF_SH_X(slot, tt, at_)                                                           \
            if (j > 0 && tt == 0) EF_SH_W(fa[slot][j - 1], wa, j - 1, at_)                               \
            if (j > 0 && tt == (NTL > 1 ? 1 : 0)) EF_SH_W(fb[slot][j - 1], wb, j - 1, at_)               \
            B[tt] = shared_mfma<HALF>(fb[slot][j], xb[i % (LA + 1)], B[tt]);                             \
            __builtin_amdgcn_sched_barrier(0);                                                           \
        }                                                                                                \
        EF_SH_W(fa[slot][3], wa, 3, at_)                                                                 \
        EF_SH_W(fb[slot][3], wb, 3, at_)                                                                 \
        __syncthreads();                                                                                 \
    }
#pragma unroll
    for (int r = 0; r < D; ++r) {
        const unsigned at = shared_stage_offset(q0 + r, last);
#pragma unroll
        for (int u = 0; u < NTL; ++u) EF_SH_X(r, u, at)
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            EF_SH_W(fa[r][j], wa, j, at)
            EF_SH_W(fb[r][j], wb, j, at)
        }
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int u = 0; u < NTL; ++u) xs[q0 & (kShLds - 1)][u * 4 + wave][lane] = xr[0][u];
    __syncthreads();
    int st = q0;
    for (; st + D <= q1; st += D) {
#pragma unroll
        for (int r = 0; r < D; ++r) EF_SH_STAGE(r, (r + 1) % D, st + r)
    }
#pragma unroll
    for (int r = 0; r < D - 1; ++r)
        if (st + r < q1) EF_SH_STAGE(r, r + 1, st + r)
#undef EF_SH_X
#undef EF_SH_W
#undef EF_SH_STAGE
}

// A pass with NTL live tiles or more: the loop for its number of them, and its activations (dst: those of the wave's row
// block and the pass's first tile).  The accumulators live in here: none are held, or merged, for tiles a pass does not have.
template <int TT, int NTL, int D>
__device__ __forceinline__ void shared_up_pass(const char *__restrict__ w1, const char *__restrict__ w3,
                                               const char *const (&xsrc)[TT], u32x4_t (*xs)[TT * 4][64], int nq, int wave,
                                               int lane, int ntl, uint4 *__restrict__ dst, int nkb2) {
    if constexpr (NTL < TT)
        if (ntl != NTL) return shared_up_pass<TT, NTL + 1, D>(w1, w3, xsrc, xs, nq, wave, lane, ntl, dst, nkb2);
    floatx16 G[NTL], U[NTL];
#pragma unroll
    for (int tt = 0; tt < NTL; ++tt) { zero16(G[tt]); zero16(U[tt]); }
    shared_stream<TT, NTL, D, false>(w1, w3, xsrc, xs, 0, nq, wave, lane, G, U);

    // a lane holds 16 F-values of one token: the two paired-order fragments the second half consumes
#pragma unroll
    for (int tt = 0; tt < NTL; ++tt) {
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            uint32_t pk[4];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float g0 = G[tt][8 * s + 2 * q], g1 = G[tt][8 * s + 2 * q + 1];
                const float v0 = silu_mul(g0, U[tt][8 * s + 2 * q]);
                const float v1 = silu_mul(g1, U[tt][8 * s + 2 * q + 1]);
                pk[q] = pack_act2(v0, v1);
            }
            dst[((size_t)tt * nkb2 + s) * 64] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
        }
    }
}

// ------------------------------------------------------------------------------------------
// first half: act = silu(X W1^T) * (X W3^T).  Workgroup = (group, pass of TT token tiles, four
// consecutive 32-row blocks of F), wave = one row block, whole K range in stages of four k-blocks.
// ------------------------------------------------------------------------------------------
template <int TT, int D, int OCC>
__global__ __launch_bounds__(256, OCC) void ffn_gate_up_shared_kernel(GroupTable gt, const uint4 *__restrict__ xp,
                                                                    uint4 *__restrict__ act, int d) {
    __shared__ __attribute__((aligned(16))) u32x4_t xs[kShLds][TT * 4][64];
    const int wg = blockIdx.x;
    int grp = 0;
    while (grp + 1 < gt.n_groups && gt.wg_start[grp + 1] <= wg) ++grp;
    const int local = wg - gt.wg_start[grp];
    const int F = gt.F[grp];
    const int rbw = (F >> 5) >> 2;               // workgroups per pass (F is a multiple of 128)
    const int pass = local / rbw;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int rb = (local % rbw) * 4 + wave;
    int ntl = gt.n_tiles[grp] - pass * TT;
    if (ntl > TT) ntl = TT;
    const int nkb = d >> 4, nq = d >> 6;         // d is a multiple of 64: whole stages

    const char *w1 = reinterpret_cast<const char *>(gt.blob[grp]) + (size_t)rb * 2 * nkb * 1024;
    const char *w3 = w1 + (size_t)nkb * 1024;
    // this wave's share of the token fragments of a stage: k-block `wave` of each tile (tiles past the
    // group's last one repeat it; their results are dropped)
    const char *xsrc[TT];
#pragma unroll
    for (int u = 0; u < TT; ++u)
        xsrc[u] = reinterpret_cast<const char *>(xp) + (size_t)(gt.tile_start[grp] + pass * TT + min(u, ntl - 1)) * nkb * 1024;

    uint4 *dst = act + gt.act_off[grp] + ((size_t)pass * TT * (F >> 4) + rb * 2) * 64 + lane;
    shared_up_pass<TT, 1, D>(w1, w3, xsrc, xs, nq, wave, lane, ntl, dst, F >> 4);
}

hipError_t launch_ffn_gate_up_shared(const GroupTable &gt, int total_wgs, int tiles_per_pass, int occ, const void *xp,
                                     void *act, int d, hipStream_t s) {
    if (total_wgs <= 0) return hipSuccess;
    if (d % 64 != 0) return hipErrorInvalidValue;
    for (int i = 0; i < gt.n_groups; ++i)
        if (gt.F[i] % 128 != 0 || gt.n_tiles[i] <= 0 ||
            gt.wg_start[i + 1] - gt.wg_start[i] != ffn_gate_up_shared_wgs(gt.F[i], gt.n_tiles[i], tiles_per_pass))
            return hipErrorInvalidValue;
    if (gt.wg_start[gt.n_groups] != total_wgs) return hipErrorInvalidValue;
    const uint4 *x = reinterpret_cast<const uint4 *>(xp);
    uint4 *a = reinterpret_cast<uint4 *>(act);
    if (tiles_per_pass == 4 && occ == 2)
        hipLaunchKernelGGL((ffn_gate_up_shared_kernel<4, 2, 2>), dim3(total_wgs), dim3(256), 0, s, gt, x, a, d);
    else if (tiles_per_pass == 4)
        hipLaunchKernelGGL((ffn_gate_up_shared_kernel<4, kShDepth, 1>), dim3(total_wgs), dim3(256), 0, s, gt, x, a, d);
    else if (tiles_per_pass == 8)
        hipLaunchKernelGGL((ffn_gate_up_shared_kernel<8, kShDepth, 1>), dim3(total_wgs), dim3(256), 0, s, gt, x, a, d);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// as shared_up_pass.  row: the lane's first token and column; rows: tokens from that one on that the group has (0: drop all)
template <int TT, int NTL, int D>
__device__ __forceinline__ void shared_down_pass(const char *__restrict__ w2a, const char *__restrict__ w2b,
                                                 const char *const (&asrc)[TT], u32x4_t (*as)[TT * 4][64], int q0, int q1,
                                                 int wave, int lane, int ntl,
                                                 int rows, float *__restrict__ row, int d) {
    if constexpr (NTL < TT)
        if (ntl != NTL)
            return shared_down_pass<TT, NTL + 1, D>(w2a, w2b, asrc, as, q0, q1, wave, lane, ntl, rows, row, d);
    floatx16 acc[2][NTL];
#pragma unroll
    for (int cw = 0; cw < 2; ++cw)
#pragma unroll
        for (int tt = 0; tt < NTL; ++tt) zero16(acc[cw][tt]);
    shared_stream<TT, NTL, D, true>(w2a, w2b, asrc, as, q0, q1, wave, lane, acc[0], acc[1]);
#pragma unroll
    for (int tt = 0; tt < NTL; ++tt) {
        // the product is formed transposed (W2 fragment first: the operand layouts are mirror images), so a lane
        // holds token lane % 32 and four consecutive output columns per accumulator quad: 16-byte stores
        if (tt * kTile >= rows) break;
#pragma unroll
        for (int cw = 0; cw < 2; ++cw)
#pragma unroll
            for (int q = 0; q < 4; ++q)
                *reinterpret_cast<float4 *>(row + (size_t)tt * kTile * d + cw * 32 + 8 * q) =
                    make_float4(acc[cw][tt][4 * q], acc[cw][tt][4 * q + 1], acc[cw][tt][4 * q + 2], acc[cw][tt][4 * q + 3]);
    }
}

// ------------------------------------------------------------------------------------------
// second half: Y = act W2^T.  Workgroup = (group, pass of TT token tiles, eight consecutive
// 32-column blocks of d, one of the group's K-slices), wave = two column blocks.  Activations (fp16) are operand
// A (rows = tokens), shared through LDS; W2 fragments (fp16) operand B (a lane holds one output column).
// Each K-slice writes its own partial Y plane; the un-permute sums the planes in order.
// ------------------------------------------------------------------------------------------
template <int TT, int D, int OCC>
__global__ __launch_bounds__(256, OCC) void ffn_down_shared_kernel(GroupTable gt, const uint4 *__restrict__ act,
                                                                 float *__restrict__ Y, int d,
                                                                 long long y_plane) {
    __shared__ __attribute__((aligned(16))) u32x4_t as[kShLds][TT * 4][64];
    const int wg = blockIdx.x;
    int grp = 0;
    while (grp + 1 < gt.n_groups && gt.wg_start[grp + 1] <= wg) ++grp;
    const int local = wg - gt.wg_start[grp];
    const int ncb = d >> 5, ncq = (ncb + 7) >> 3;
    const int ksg = gt.ksg[grp], kslice = local % ksg;
    const int cq = (local / ksg) % ncq, pass = (local / ksg) / ncq;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int cb0 = cq * 8 + wave * 2;
    const bool valid = cb0 < ncb;                 // d is a multiple of 64: both column blocks or none
    const int cbc = valid ? cb0 : 0;              // waves past the last column load block 0 and drop the result
    const int F = gt.F[grp];
    const int nkb = F >> 4, nq = F >> 6;          // F is a multiple of 128: whole stages
    const int q0 = shared_slice_begin(nq, ksg, kslice), q1 = shared_slice_begin(nq, ksg, kslice + 1);
    int ntl = gt.n_tiles[grp] - pass * TT;
    if (ntl > TT) ntl = TT;

    const char *w2a = reinterpret_cast<const char *>(gt.blob[grp]) + (size_t)4 * d * F + (size_t)cbc * nkb * 1024;
    const char *w2b = w2a + (size_t)nkb * 1024;
    const char *asrc[TT];
#pragma unroll
    for (int u = 0; u < TT; ++u)
        asrc[u] = reinterpret_cast<const char *>(act + gt.act_off[grp]) + (size_t)(pass * TT + min(u, ntl - 1)) * nkb * 1024;

    // this lane's part of its token's row: lane % 32 of the pass's first tile
    const int t0 = pass * TT * kTile + (lane & 31);
    float *row = Y + (size_t)kslice * y_plane + (size_t)(gt.row_offset[grp] + t0) * d + cb0 * 32 + 4 * (lane >> 5);
    shared_down_pass<TT, 1, D>(w2a, w2b, asrc, as, q0, q1, wave, lane, ntl, valid ? gt.count[grp] - t0 : 0, row, d);
}

hipError_t launch_ffn_down_shared(const GroupTable &gt, int total_wgs, int tiles_per_pass, int occ, const void *act,
                                  float *y, long long y_plane, int d, hipEvent_t done, hipStream_t s) {
    if (total_wgs <= 0) return hipSuccess;
    if (d % 64 != 0) return hipErrorInvalidValue;
    for (int i = 0; i < gt.n_groups; ++i)
        if (gt.F[i] % 128 != 0 || gt.n_tiles[i] <= 0 || gt.ksg[i] < 1 || gt.ksg[i] > gt.F[i] / 64 ||
            gt.wg_start[i + 1] - gt.wg_start[i] != ffn_down_shared_wgs(d, gt.n_tiles[i], tiles_per_pass, gt.ksg[i]))
            return hipErrorInvalidValue;
    if (gt.wg_start[gt.n_groups] != total_wgs) return hipErrorInvalidValue;
    const uint4 *a = reinterpret_cast<const uint4 *>(act);
    if (tiles_per_pass == 4 && occ == 2)
        return launch_done(ffn_down_shared_kernel<4, 2, 2>, dim3(total_wgs), dim3(256), done, s, gt, a, y, d, y_plane);
    else if (tiles_per_pass == 4)
        return launch_done(ffn_down_shared_kernel<4, kShDepth, 1>, dim3(total_wgs), dim3(256), done, s, gt, a, y, d, y_plane);
    else if (tiles_per_pass == 8)
        return launch_done(ffn_down_shared_kernel<8, kShDepth, 1>, dim3(total_wgs), dim3(256), done, s, gt, a, y, d, y_plane);
    return hipErrorInvalidValue;
}

}  // namespace ef

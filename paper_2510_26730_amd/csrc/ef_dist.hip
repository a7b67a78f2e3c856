// Intra-batch diversity Dist(t) = sum over token pairs of the Euclidean distance between their
// embeddings (paper Sec. 2.2), computed per token: s[j] = sum_{i<j} ||v_i - v_j||_2.  Three families of kernels by batch
// size: the squared differences themselves (up to kDistSmallMaxTokens), Gram blocks of 32 x 32 or 64 x 64 (up to
// kDistBlockMaxTokens), and, described here, large Gram blocks over a packed copy.
//
// ||v_i - v_j||^2 = n_i + n_j - 2 <v_i, v_j>: the inner products are one T x T Gram matrix, a dense
// contraction over d that runs on the matrix cores from the packed (operand-fragment) copy of the
// tokens; only tiles that hold a pair i < j are computed.  Three steps on one stream:
//   1. squared norms n_i in fp32 (bf16 products are exact in fp32), one wave per token;
//   2. Gram tiles: a workgroup owns 256 rows i x 256 columns j whose operands pass through LDS (dist_form 1: 128 x 256,
//      operands straight into registers); the epilogue turns inner products into distances, masks i >= j and
//      columns past T, and adds 64 rows per column: one partial per (64-row block,
//      token j), no atomics;
//   3. per token the partials of its row blocks are added in ascending order, and the per-token
//      values are added in fixed order (workgroup tree, then one workgroup over the workgroup
//      sums) into Dist(t) in fp64: the result does not depend on scheduling.
#include "ef_device.h"
#include "ef_kernels.h"
#include "ef_tiled_pipeline.h"

namespace ef {

// one wave per token: n[t] = sum_c x[t,c]^2 in fp32, lanes stride the row in 16-byte pieces
__global__ __launch_bounds__(256) void dist_norm_kernel(const uint16_t *__restrict__ h, int T, int d,
                                                        float *__restrict__ norms, int n_pad) {
    const int t = blockIdx.x * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
    if (t >= n_pad) return;
    float acc = 0.f;
    if (t < T) {
        const uint4 *row = reinterpret_cast<const uint4 *>(h + (size_t)t * d);
        for (int c = lane; c < (d >> 3); c += 64) {
            const uint4 v = row[c];
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const float lo = __builtin_bit_cast(float, w[q] << 16);
                const float hi = __builtin_bit_cast(float, w[q] & 0xFFFF0000u);
                acc += lo * lo;
                acc += hi * hi;
            }
        }
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) acc += __shfl_xor(acc, off);
    if (lane == 0) norms[t] = acc;   // rows of the padding up to whole tiles get 0
}

// Decode-sized batches (up to kDistRowMaxTokens tokens): the Gram route would be one or two workgroups walking all of
// d in sequence behind five launches.  Here workgroup j owns token j: wave w of 16 takes the rows i = w, w + 16, ...
// < j, two at a time (their loads are independent), the lanes stride the row pair in 16-byte pieces and add
// (x_i - x_j)^2 in fp32 (no norms, no cancellation), a shuffle tree adds the lanes, the root is added to the wave's
// sum in fp64 in ascending i; the waves' sums are added in order.  Everything in a fixed order: the result does not
// depend on scheduling.
constexpr int kDistRowWaves = 16;
__device__ __forceinline__ float dist_sq_piece(uint4 a, uint4 b) {
    const uint32_t wa[4] = {a.x, a.y, a.z, a.w}, wb[4] = {b.x, b.y, b.z, b.w};
    float acc = 0.f;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        const float dl = __builtin_bit_cast(float, wa[q] << 16) - __builtin_bit_cast(float, wb[q] << 16);
        const float dh = __builtin_bit_cast(float, wa[q] & 0xFFFF0000u) - __builtin_bit_cast(float, wb[q] & 0xFFFF0000u);
        acc += dl * dl;
        acc += dh * dh;
    }
    return acc;
}
__global__ __launch_bounds__(64 * kDistRowWaves) void dist_row_kernel(const uint16_t *__restrict__ h, int T, int d,
                                                                           float *__restrict__ tok_dist,
                                                                           double *__restrict__ wg_sums) {
    __shared__ double red[kDistRowWaves];
    const int j = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const uint4 *rj = reinterpret_cast<const uint4 *>(h + (size_t)j * d);
    const int nc = d >> 3;
    double s = 0.0;
    for (int i = wave; i < j; i += 2 * kDistRowWaves) {
        const int i2 = i + kDistRowWaves;
        const bool two = i2 < j;
        const uint4 *r0 = reinterpret_cast<const uint4 *>(h + (size_t)i * d);
        const uint4 *r1 = reinterpret_cast<const uint4 *>(h + (size_t)(two ? i2 : i) * d);
        float acc0 = 0.f, acc1 = 0.f;
        for (int c = lane; c < nc; c += 64) {
            const uint4 b = rj[c];
            acc0 += dist_sq_piece(r0[c], b);
            acc1 += dist_sq_piece(r1[c], b);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) {
            acc0 += __shfl_xor(acc0, off);
            acc1 += __shfl_xor(acc1, off);
        }
        s += (double)__builtin_sqrtf(acc0);
        if (two) s += (double)__builtin_sqrtf(acc1);
    }
    if (lane == 0) red[wave] = s;
    __syncthreads();
    if (threadIdx.x == 0) {
        double t = 0.0;
        for (int w = 0; w < kDistRowWaves; ++w) t += red[w];
        if (tok_dist) tok_dist[j] = (float)t;
        wg_sums[j] = t;
    }
}

// Batches up to a few hundred tokens: the squared differences themselves, no norms and no cancellation.
// Bound by vector instructions (two per pair and element, one more to unpack each bf16) and, at a few dozen tokens, by
// launch latency.  A workgroup owns 8 tokens j and a chunk of 16 rows i, one wave two of the rows: a lane holds its
// 16-byte piece of the eight tokens unpacked and meets two rows with it, so a piece is loaded and unpacked once for two
// (eight) pairs.  The lanes' sums of a wave's 16 pairs meet in a butterfly that halves the number of values per step (31
// exchanges instead of 96); the roots are added in fp64 in ascending i, one partial per (chunk, j).  Fixed order
// throughout.  d = 4096, the call, against one workgroup per token j that walks every row before it: T = 256 46 -> 23 us,
// T = 128 22.5 -> 16 us; at 64 tokens both take 14 us, below that the other form is ahead (T = 16: 7 against 13 us).
constexpr int kDistSmallCols = 8, kDistSmallRows = 16, kDistSmallWaves = 8;
__device__ __forceinline__ void dist_unpack(uint4 v, float (&f)[8]) {
    const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        f[2 * q] = __builtin_bit_cast(float, w[q] << 16);
        f[2 * q + 1] = __builtin_bit_cast(float, w[q] & 0xFFFF0000u);
    }
}
__global__ __launch_bounds__(64 * kDistSmallWaves) void dist_small_kernel(const uint16_t *__restrict__ h, int T, int d,
                                                                           double *__restrict__ part) {
    constexpr int NC = kDistSmallCols, RW = kDistSmallRows / kDistSmallWaves;   // rows per wave
    static_assert(RW * NC == 16, "the butterfly reduces 16 values");
    __shared__ float sq[kDistSmallRows][NC];
    const int i0 = blockIdx.x * kDistSmallRows, j0 = blockIdx.y * NC;
    if (i0 >= j0 + NC) return;   // every row past every token of the group
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int nc = d >> 3;
    const uint4 *rj[NC], *ri[RW];
#pragma unroll
    for (int j = 0; j < NC; ++j) rj[j] = reinterpret_cast<const uint4 *>(h + (size_t)min(j0 + j, T - 1) * d);
#pragma unroll
    for (int r = 0; r < RW; ++r) ri[r] = reinterpret_cast<const uint4 *>(h + (size_t)min(i0 + wave * RW + r, T - 1) * d);
    float acc[16];   // [row][token]
#pragma unroll
    for (int q = 0; q < 16; ++q) acc[q] = 0.f;
    for (int c = lane; c < nc; c += 64) {
        uint4 vi[RW], vj[NC];
#pragma unroll
        for (int r = 0; r < RW; ++r) vi[r] = ri[r][c];
#pragma unroll
        for (int j = 0; j < NC; ++j) vj[j] = rj[j][c];
        float fi[RW][8];
#pragma unroll
        for (int r = 0; r < RW; ++r) dist_unpack(vi[r], fi[r]);
#pragma unroll
        for (int j = 0; j < NC; ++j) {
            float fj[8];
            dist_unpack(vj[j], fj);
#pragma unroll
            for (int r = 0; r < RW; ++r) {
                // a piece's sum first: one long chain of small squares onto a growing sum loses them to rounding (d = 4096:
                // distances 5e-8 low on average, with piece sums 5e-9)
                float p = 0.f;
#pragma unroll
                for (int e = 0; e < 8; ++e) {
                    const float x = fi[r][e] - fj[e];
                    p += x * x;
                }
                acc[r * NC + j] += p;
            }
        }
    }
    // 16 values x 64 lanes: step s exchanges half of the values left between lanes that differ in bit s, so lane l ends
    // with value l % 16 summed over the lanes that agree with it in the low four bits; two plain steps add those
#pragma unroll
    for (int s = 0; s < 4; ++s) {
        const bool up = (lane >> s) & 1;
#pragma unroll
        for (int q = 0; q < (8 >> s); ++q) {
            const float keep = up ? acc[2 * q + 1] : acc[2 * q], give = up ? acc[2 * q] : acc[2 * q + 1];
            acc[q] = keep + __shfl_xor(give, 1 << s);
        }
    }
    float v = acc[0];
    v += __shfl_xor(v, 16);
    v += __shfl_xor(v, 32);
    if (lane < 16) sq[wave * RW + (lane >> 3)][lane & 7] = v;
    __syncthreads();
    if (threadIdx.x < NC) {
        const int j = j0 + threadIdx.x;
        double t = 0.0;
        for (int r = 0; r < kDistSmallRows; ++r)
            if (i0 + r < j) t += (double)__builtin_sqrtf(sq[r][threadIdx.x]);
        if (j < T) part[(size_t)blockIdx.x * T + j] = t;
    }
}

// ------------------------------------------------------------------------------------------
// Gram blocks of batches between the two sizes above and below (kDistSmallMaxTokens to kDistBlockMaxTokens): too few
// 256 x 256 (or 128 x 256) blocks to fill the chip, each walking all of d alone: 25 workgroups and 49 us at T = 1056,
// d = 2048.  Here a workgroup owns a block of 32B x 32B pairs (B = 1 or 2) and its NW = 4 or 8 waves a part of d each: their
// partial products meet in LDS in a fixed order, and every wave turns its share of them into distances.  Rows are read as
// they are, whole 128-byte lines by eight lanes each, and turned into operand fragments through a wave's own LDS buffer,
// pieces of a row rotated by an exclusive or so that neither side meets bank conflicts (read straight into operand registers, 32 lines per load, the address path bound the
// kernel: T = 1056, d = 2048 26.6 against 18.8 us for the call; T = 2048, d = 4096 119 and 66).  No packed copy; the norms
// are the diagonals of the row and column tiles' own products, formed beside the block's in the same order (one launch
// less; equal rows give a distance of exactly 0).  Products are summed stage by stage (below), which takes those two sizes
// to 19.6 and 71 us.
// ------------------------------------------------------------------------------------------
// element dv of an accumulator, dv different from lane to lane
__device__ __forceinline__ float diag_of(const floatx16 &m, int dv) {
    float r = m[0];
#pragma unroll
    for (int v = 1; v < 16; ++v) r = dv == v ? m[v] : r;
    return r;
}
// the waves' parts of a sum, `stride` floats apart, as a tree: half the roundings of a chain
template <int NW>
__device__ __forceinline__ float over_waves(const float *p, int stride) {
    const float lo = (p[0] + p[stride]) + (p[2 * stride] + p[3 * stride]);
    if constexpr (NW == 4) return lo;
    else return lo + ((p[4 * stride] + p[5 * stride]) + (p[6 * stride] + p[7 * stride]));
}
// NW = 8: one block per compute unit
template <int B, int R, int NW>
__global__ __launch_bounds__(64 * NW, NW == 4 ? 2 : 1) void dist_block_kernel(const uint16_t *__restrict__ h, int T, int d,
                                                                              float *__restrict__ part, int t_pad) {
    constexpr int U = 4;   // k-steps (16 columns each) per stage
    constexpr int TILE = 256;   // 16-byte units of a tile's stage: 32 rows x 128 bytes
    // a stage buffer per wave; the partial products take its place afterwards
    __shared__ __attribute__((aligned(16))) u32x4_t lds[NW][2 * B * TILE];
    __shared__ float nrm[NW][2 * B][32];
    __shared__ float csum[NW][32];
    static_assert(sizeof(lds[0]) >= sizeof(float) * B * B * 16 * 64, "a wave's partial products fit its stage buffer");
    // block t of the upper triangle, column by column: IB <= JB
    const int t = blockIdx.x;
    int JB = (int)((__builtin_sqrtf(8.f * (float)t + 1.f) - 1.f) * 0.5f);
    while ((JB + 1) * (JB + 2) / 2 <= t) ++JB;
    while (JB * (JB + 1) / 2 > t) --JB;
    const int IB = t - JB * (JB + 1) / 2;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int g = lane >> 5, c = lane & 31;
    const int n = (d >> 4) / NW, k0 = wave * n;   // d is a multiple of 16 NW: equal parts
    // global load u of a tile's stage: rows 8u .. 8u+7, eight lanes to a row's 128 bytes
    const int lr = lane >> 3, lc = lane & 7;
    // of row tiles, then column tiles; rows past the last token read the last one (16-byte units: T d / 8 fits 32 bits)
    const u32x4_t *const h4 = reinterpret_cast<const u32x4_t *>(h) + 2 * k0;
    const unsigned stride = d >> 3, last = (unsigned)(T - 1) * stride;
    const unsigned row0 = (unsigned)(IB * B * kTile + lr) * stride, col0 = (unsigned)(JB * B * kTile + lr) * stride;
    u32x4_t *const buf = lds[wave];
    const int put = lr * 8 + (lc ^ lr);   // + 64 u + TILE a
    // The matrix instruction's sums of like sign drift upwards as the accumulator grows (a norm from one chain of 32: 4e-8
    // of it on average, from chains of 4: 5e-9), and the norm of a token enters all of its distances.  So a stage's
    // products form a chain of their own, which is then added to the total (for the norms to the lane's diagonal element).
    floatx16 acc[B][B];
    float diag[2 * B];   // of the lanes that hold a diagonal element: row c of tile a, in the lanes with g = c / 4 % 2
#pragma unroll
    for (int a = 0; a < B; ++a)
#pragma unroll
        for (int b = 0; b < B; ++b) zero16(acc[a][b]);
#pragma unroll
    for (int a = 0; a < 2 * B; ++a) diag[a] = 0.f;
    const int dv = 4 * (c >> 3) + (c & 3);   // accumulator element of that row
    u32x4_t f[R][2 * B][U];
#define EF_DISTB_LOAD(f_, kb)                                                                             \
    {                                                                                                     \
        const unsigned ch_ = min(2 * (kb) + lc, 2 * n - 1); /* past the part's end its last piece again */ \
        _Pragma("unroll") for (int a = 0; a < 2 * B; ++a)                                                 \
            _Pragma("unroll") for (int u = 0; u < U; ++u)                                                 \
                f_[a][u] = h4[min((a < B ? row0 : col0) + (unsigned)((a % B) * kTile + 8 * u) * stride, last) + ch_]; \
    }
    // products of the stage in LDS: row tile `a` with the column tiles, its norm and that of column tile `a`
#define EF_DISTB_PRODUCTS                                                                                 \
    _Pragma("unroll") for (int a = 0; a < B; ++a) {                                                       \
        floatx16 p_[B], qr_, qc_;                                                                         \
        _Pragma("unroll") for (int b = 0; b < B; ++b) zero16(p_[b]);                                      \
        zero16(qr_);                                                                                      \
        zero16(qc_);                                                                                      \
        _Pragma("unroll") for (int u = 0; u < U; ++u) {                                                   \
            const int at_ = c * 8 + ((2 * u + g) ^ (c & 7));                                              \
            const u32x4_t x_ = buf[a * TILE + at_];                                                       \
            u32x4_t y_[B];                                                                                \
            _Pragma("unroll") for (int b = 0; b < B; ++b) y_[b] = buf[(B + b) * TILE + at_];              \
            _Pragma("unroll") for (int b = 0; b < B; ++b) p_[b] = mfma32v(x_, y_[b], p_[b]);              \
            qr_ = mfma32v(x_, x_, qr_);                                                                   \
            qc_ = mfma32v(y_[a], y_[a], qc_);                                                             \
        }                                                                                                 \
        _Pragma("unroll") for (int b = 0; b < B; ++b)                                                     \
            _Pragma("unroll") for (int v = 0; v < 16; ++v) acc[a][b][v] += p_[b][v];                      \
        diag[a] += diag_of(qr_, dv);                                                                      \
        diag[B + a] += diag_of(qc_, dv);                                                                  \
        __builtin_amdgcn_sched_barrier(0);                                                                \
    }
    // one stage: into the wave's LDS buffer, the registers refilled R stages ahead, then operand fragments from LDS.  A
    // lane reads what other lanes of its wave wrote and the next stage overwrites it: both ways the order is stated to the
    // compiler (no wait and no instruction: the hardware keeps a wave's LDS operations in order)
#define EF_DISTB_STAGE(f_, kb)                                                                            \
    {                                                                                                     \
        if ((kb) + U > n) { /* the part ends inside the stage: zeros past its end */                      \
            const bool past_ = 2 * (kb) + lc >= 2 * n;                                                    \
            _Pragma("unroll") for (int a = 0; a < 2 * B; ++a)                                             \
                _Pragma("unroll") for (int u = 0; u < U; ++u) f_[a][u] = past_ ? u32x4_t{0, 0, 0, 0} : f_[a][u]; \
        }                                                                                                 \
        _Pragma("unroll") for (int a = 0; a < 2 * B; ++a)                                                 \
            _Pragma("unroll") for (int u = 0; u < U; ++u) buf[a * TILE + 64 * u + put] = f_[a][u];        \
        wave_lds_sync();                                                                                  \
        EF_DISTB_LOAD(f_, (kb) + R * U)                                                                   \
        EF_DISTB_PRODUCTS                                                                                 \
        wave_lds_sync();                                                                                  \
    }
#pragma unroll
    for (int r = 0; r < R; ++r) EF_DISTB_LOAD(f[r], r * U)
    for (int kb = 0; kb < n; kb += R * U) {
#pragma unroll
        for (int r = 0; r < R; ++r)
            if (kb + r * U < n) EF_DISTB_STAGE(f[r], kb + r * U)
    }
#undef EF_DISTB_LOAD
#undef EF_DISTB_PRODUCTS
#undef EF_DISTB_STAGE
    float(*const red)[B * B * 16][64] = reinterpret_cast<float(*)[B * B * 16][64]>(&lds[0][0]);
    // the partials' stride is a wave's own buffer or less, so every wave has to be done with its stages first
    __syncthreads();
#pragma unroll
    for (int a = 0; a < B; ++a)
#pragma unroll
        for (int b = 0; b < B; ++b)
#pragma unroll
            for (int v = 0; v < 16; ++v) red[wave][(a * B + b) * 16 + v][lane] = acc[a][b][v];
    // accumulator lane l holds column l%32 and rows 8*(v/4) + 4*(l/32) + v%4
    if (g == ((c >> 2) & 1)) {
#pragma unroll
        for (int a = 0; a < 2 * B; ++a) nrm[wave][a][c] = diag[a];
    }
    __syncthreads();
    // every wave takes its share of the block's elements, all of one tile: VW rows of 32 columns in each lane half
    constexpr int VW = B * B * 16 / NW;
    const int tile = wave * VW >> 4, a = tile / B, b = tile % B;
    const int j = (JB * B + b) * kTile + c;
    const float nj = over_waves<NW>(&nrm[0][B + b][c], 2 * B * 32);
    float sum = 0.f;
#pragma unroll
    for (int u = 0; u < VW; ++u) {
        const int q = wave * VW + u, v = q & 15;
        const int r = 8 * (v >> 2) + 4 * g + (v & 3), i = (IB * B + a) * kTile + r;
        const float ip = over_waves<NW>(&red[0][q][lane], B * B * 16 * 64), ni = over_waves<NW>(&nrm[0][a][r], 2 * B * 32);
        if (i < j && j < T) {
            const float dd = ni + nj - 2.f * ip;
            sum += __builtin_sqrtf(fmaxf(dd, 0.f));
        }
    }
    sum += __shfl_xor(sum, 32);
    if (g == 0) csum[wave][c] = sum;
    __syncthreads();
    // one partial per block of rows: the waves' sums in ascending order
    if (threadIdx.x < B * 32) {
        const int bb = threadIdx.x >> 5;
        float total = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w)
            if ((w * VW >> 4) % B == bb) total += csum[w][c];
        const int jj = (JB * B + bb) * kTile + c;
        if (jj < t_pad) part[(size_t)IB * t_pad + jj] = total;
    }
}

// Per-token sums over the row blocks and their total, for the batches of the two kernels above: one workgroup, since a
// second launch costs as much as the sums.  Partial row block rb of token j at part[rb * stride + j], row blocks
// 0 .. j / rows of token j; added in ascending order, the tokens' sums by a fixed tree.
template <typename P>
__global__ __launch_bounds__(1024) void dist_sum_kernel(const P *__restrict__ part, int T, int stride, int rows,
                                                        float *__restrict__ tok_dist, double *__restrict__ dist) {
    __shared__ double red[1024];
    double total = 0.0;
    for (int j = threadIdx.x; j < T; j += 1024) {
        const int n = j / rows + 1;
        double s = 0.0;
        int rb = 0;
        for (; rb + 8 <= n; rb += 8) {
            P v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = part[(size_t)(rb + u) * stride + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += (double)v[u];
        }
        for (; rb < n; ++rb) s += (double)part[(size_t)rb * stride + j];
        if (tok_dist) tok_dist[j] = (float)s;
        total += s;
    }
    red[threadIdx.x] = total;
    __syncthreads();
    for (int o = 512; o >= 1; o >>= 1) {
        if (threadIdx.x < o) red[threadIdx.x] += red[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) *dist = red[0];
}

constexpr int kDistRowTiles = 4;   // token tiles (32 rows) of operand A per workgroup: 128 rows i
constexpr int kDistColTiles = 8;   // token tiles of operand B per workgroup: 256 columns j

// grid (column blocks, row blocks); xp = packed tokens [tile][d/16][1 KiB]
__global__ __launch_bounds__(256, 2) void dist_tile_kernel(const uint4 *__restrict__ xp,
                                                           const float *__restrict__ norms, int T, int d,
                                                           float *__restrict__ part, int t_pad,
                                                           int n_rowblk) {
    const int JB = blockIdx.x, IB = blockIdx.y;
    if (IB > 2 * JB + 1) return;   // every row of the block is >= every column: no pair i < j
    const int ntiles = (T + kTile - 1) / kTile;
    const int nkb = d >> 4;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int it0 = IB * kDistRowTiles + (wave >> 1) * 2;    // 2 row tiles of this wave
    const int jt0 = JB * kDistColTiles + (wave & 1) * 4;     // 4 column tiles of this wave
    const uint4 *a_src[2], *b_src[4];
#pragma unroll
    for (int a = 0; a < 2; ++a) a_src[a] = xp + (size_t)min(it0 + a, ntiles - 1) * nkb * 64 + lane;
#pragma unroll
    for (int b = 0; b < 4; ++b) b_src[b] = xp + (size_t)min(jt0 + b, ntiles - 1) * nkb * 64 + lane;

    floatx16 acc[2][4];
#pragma unroll
    for (int a = 0; a < 2; ++a)
#pragma unroll
        for (int b = 0; b < 4; ++b) zero16(acc[a][b]);

    // two register stages of two k-steps each; the prefetch is unconditional (clamped, in bounds)
    constexpr int UNR = 2;
    u32x4_t fa0[2][UNR], fb0[4][UNR], fa1[2][UNR], fb1[4][UNR];
#define EF_DIST_LOAD(fa, fb, kb)                                                                          \
    {                                                                                                     \
        _Pragma("unroll") for (int u = 0; u < UNR; ++u) {                                                 \
            const int kk_ = min((kb) + u, nkb - 1);                                                       \
            _Pragma("unroll") for (int a = 0; a < 2; ++a)                                                 \
                fa[a][u] = *reinterpret_cast<const u32x4_t *>(a_src[a] + (size_t)kk_ * 64);               \
            _Pragma("unroll") for (int b = 0; b < 4; ++b)                                                 \
                fb[b][u] = *reinterpret_cast<const u32x4_t *>(b_src[b] + (size_t)kk_ * 64);               \
        }                                                                                                 \
    }
#define EF_DIST_MMA(fa, fb, kb)                                                                           \
    {                                                                                                     \
        _Pragma("unroll") for (int u = 0; u < UNR; ++u)                                                   \
            if ((kb) + u < nkb) {                                                                         \
                _Pragma("unroll") for (int a = 0; a < 2; ++a)                                             \
                    _Pragma("unroll") for (int b = 0; b < 4; ++b)                                         \
                        acc[a][b] = mfma32v(fa[a][u], fb[b][u], acc[a][b]);                               \
            }                                                                                             \
    }
    EF_DIST_LOAD(fa0, fb0, 0)
    for (int kb = 0; kb < nkb; kb += 2 * UNR) {
        EF_DIST_LOAD(fa1, fb1, kb + UNR)
        EF_DIST_MMA(fa0, fb0, kb)
        EF_DIST_LOAD(fa0, fb0, kb + 2 * UNR)
        EF_DIST_MMA(fa1, fb1, kb + UNR)
    }
#undef EF_DIST_LOAD
#undef EF_DIST_MMA

    // accumulator lane l holds column l%32 and rows 8*(v/4) + 4*(l/32) + v%4: the sum over the
    // wave's 64 rows of one column is 32 in-lane adds and one exchange between the lane halves
    const int g = lane >> 5, c = lane & 31;
    const int rowblk = IB * 2 + (wave >> 1);   // 64-row block of the partials
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        const int j = (jt0 + b) * kTile + c;
        const float nj = j < T ? norms[j] : 0.f;
        float sum = 0.f;
#pragma unroll
        for (int a = 0; a < 2; ++a) {
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int i = (it0 + a) * kTile + 8 * (v >> 2) + 4 * g + (v & 3);
                if (i < j && j < T) {
                    const float sq = norms[i] + nj - 2.f * acc[a][b][v];
                    sum += __builtin_sqrtf(fmaxf(sq, 0.f));
                }
            }
        }
        sum += __shfl_xor(sum, 32);
        if (g == 0 && j < t_pad && rowblk < n_rowblk) part[(size_t)rowblk * t_pad + j] = sum;
    }
}

// ------------------------------------------------------------------------------------------
// Gram tiles through the LDS operand pipeline (large batches): a workgroup owns 256 rows i x 256 columns
// j, both operands are token fragments.  Same accumulation order over k, same epilogue sums and the same
// partials as dist_tile_kernel: the two forms give the same bits.
//
// Only blocks with a pair i < j exist (block row IB <= block column JB).  They are numbered in strips of
// four block rows, column by column within a strip, so that 32 consecutive blocks cover about 4 block
// rows x 8 block columns; runs of 32 go to the XCDs in turn (workgroups with the same index mod 8 share an
// XCD and run side by side on its 32 compute units), so the 64 operand panels of a run are 12 distinct ones
// and an XCD's L2 serves the rest.
// ------------------------------------------------------------------------------------------
constexpr int kGramRun = 32;     // consecutive blocks that one XCD runs side by side
constexpr int kGramStrip = 4;    // block rows per strip

// blocks in the strips before strip R (nB block rows / columns)
__host__ __device__ inline long long gram_blocks_before(int R, int nB) {
    const long long r = kGramStrip * R < nB ? kGramStrip * R : nB;   // block rows before the strip
    return r * nB - r * (r - 1) / 2;                           // row IB holds nB - IB blocks
}
inline long long gram_blocks(int nB) { return (long long)nB * (nB + 1) / 2; }

__global__ __launch_bounds__(256, 1) void dist_gram_tiled_kernel(const uint4 *__restrict__ xp,
                                                                  const float *__restrict__ norms, int T, int d,
                                                                  float *__restrict__ part, int t_pad,
                                                                  int n_rowblk, int nB, long long total_whole,
                                                                  int main_grid) {
    constexpr bool kSwapOperands = false;
    constexpr bool HALF = false;   // bf16 token fragments
    __shared__ __attribute__((aligned(16))) u32x4_t lds[kTileStages][kStageFrags][64];
    const int w = blockIdx.x;
    // workgroups [0, main_grid): whole blocks [0, total_whole) in runs over the XCDs; the workgroups after them:
    // the quarters (128 x 128) of the blocks from total_whole on
    long long t;
    int quarter = -1;
    if (w < main_grid) {
        t = ((long long)(w >> 3) / kGramRun * 8 + (w & 7)) * kGramRun + ((w >> 3) % kGramRun);
        if (t >= total_whole) return;
    } else {
        t = total_whole + ((w - main_grid) >> 2);
        quarter = (w - main_grid) & 3;
    }
    // strip R, then the block within the strip: its first h columns hold 1..h blocks (the diagonal), the
    // columns after them h blocks each
    int R = 0;
    while (gram_blocks_before(R + 1, nB) <= t) ++R;
    const int u = (int)(t - gram_blocks_before(R, nB));
    const int h = min(kGramStrip, nB - kGramStrip * R);
    int a, cidx;
    if (u < h * (h + 1) / 2) {
        cidx = 0;
        while ((cidx + 1) * (cidx + 2) / 2 <= u) ++cidx;
        a = u - cidx * (cidx + 1) / 2;
    } else {
        const int v = u - h * (h + 1) / 2;
        cidx = h + v / h;
        a = v % h;
    }
    const int IB = kGramStrip * R + a, JB = kGramStrip * R + cidx;

    const int ntiles = (T + kTile - 1) / kTile;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: LDS DMA targets go through M0
    const int wi = wave & 1, wj = wave >> 1;
    const int nkb = d >> 4;
    const int nstage = nkb / kTileKS;
    const int g = lane >> 5, c = lane & 31;
    const unsigned lds_base = (unsigned)(size_t)&lds[0][0][0];   // LDS byte offset: the low half of its flat address
    const u32x4_t *src[kStageFrags / 4];
    floatx16 acc[4][4];   // [row tile][column tile]
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) zero16(acc[i][j]);

    if (quarter < 0) {
        const int it0 = IB * 8, jt0 = JB * 8;
        // operand A slots 0..7 = row tiles it0..it0+7, operand B slots 8..15 = column tiles jt0..jt0+7
#pragma unroll
        for (int q = 0; q < kStageFrags / 4; ++q) {
            const int fi = q * 4 + wave;
            const int ks = fi >> 4, slot = fi & 15;
            const int tile = min(slot < 8 ? it0 + slot : jt0 + slot - 8, ntiles - 1);
            src[q] = reinterpret_cast<const u32x4_t *>(xp + ((size_t)tile * nkb + ks) * 64 + lane);
        }
        const int AOFF = wi * 4, BOFF = wj * 4;
        // column tiles of this wave that exist; none count when every row of the wave is past every column
        // (the lower left quarter of a diagonal block)
        const bool below = it0 + AOFF >= jt0 + BOFF + 4;
        const int live = below ? 0 : max(0, min(4, ntiles - (jt0 + BOFF)));
        EF_TILED_PIPELINE_TILES_B(0, nstage, live)

#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int j = (jt0 + BOFF + b) * kTile + c;
            const float nj = j < T ? norms[j] : 0.f;
#pragma unroll
            for (int rp = 0; rp < 2; ++rp) {   // the wave's two 64-row blocks of the partials
                const int rowblk = IB * 4 + wi * 2 + rp;
                float sum = 0.f;
#pragma unroll
                for (int aa = 0; aa < 2; ++aa) {
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int i = (it0 + AOFF + 2 * rp + aa) * kTile + 8 * (v >> 2) + 4 * g + (v & 3);
                        if (i < j && j < T) {
                            const float sq = norms[i] + nj - 2.f * acc[2 * rp + aa][b][v];
                            sum += __builtin_sqrtf(fmaxf(sq, 0.f));
                        }
                    }
                }
                sum += __shfl_xor(sum, 32);
                if (g == 0 && j < t_pad && rowblk < n_rowblk) part[(size_t)rowblk * t_pad + j] = sum;
            }
        }
    } else {
        // a quarter: 128 rows x 128 columns, a wave 64 x 64 (2 x 2 accumulators): the same loads and barriers
        // per stage for a quarter of the matrix-core work, for the few blocks that would otherwise be a round
        // of workgroups of their own over a mostly idle chip
        const int it0 = IB * 8 + (quarter >> 1) * 4, jt0 = JB * 8 + (quarter & 1) * 4;
        if (it0 >= jt0 + 4) return;   // every row past every column
        // operand A slots 0..3 = row tiles it0..it0+3, operand B slots 8..11 = column tiles jt0..jt0+3; the other
        // slots repeat them (never read from LDS)
#pragma unroll
        for (int q = 0; q < kStageFrags / 4; ++q) {
            const int fi = q * 4 + wave;
            const int ks = fi >> 4, slot = fi & 15;
            const int tile = min(slot < 8 ? it0 + (slot & 3) : jt0 + (slot & 3), ntiles - 1);
            src[q] = reinterpret_cast<const u32x4_t *>(xp + ((size_t)tile * nkb + ks) * 64 + lane);
        }
        const int AOFF = wi * 2, BOFF = wj * 2;
        EF_TILED_PIPELINE_2X2(0, nstage)

        const int rowblk = (it0 + AOFF) >> 1;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int j = (jt0 + BOFF + b) * kTile + c;
            const float nj = j < T ? norms[j] : 0.f;
            float sum = 0.f;
#pragma unroll
            for (int aa = 0; aa < 2; ++aa) {
#pragma unroll
                for (int v = 0; v < 16; ++v) {
                    const int i = (it0 + AOFF + aa) * kTile + 8 * (v >> 2) + 4 * g + (v & 3);
                    if (i < j && j < T) {
                        const float sq = norms[i] + nj - 2.f * acc[aa][b][v];
                        sum += __builtin_sqrtf(fmaxf(sq, 0.f));
                    }
                }
            }
            sum += __shfl_xor(sum, 32);
            if (g == 0 && j < t_pad && rowblk < n_rowblk) part[(size_t)rowblk * t_pad + j] = sum;
        }
    }
}

// s[j] = partials of row blocks 0 .. j/64 in ascending order; workgroup sum in fp64 by a fixed tree
__global__ __launch_bounds__(256) void dist_reduce_kernel(const float *__restrict__ part, int T, int t_pad,
                                                          float *__restrict__ tok_dist,
                                                          double *__restrict__ wg_sums) {
    __shared__ double red[256];
    const int j = blockIdx.x * 256 + threadIdx.x;
    double s = 0.0;
    if (j < T) {
        // eight loads in flight, added in ascending order of the row block
        const int n = (j >> 6) + 1;
        int rb = 0;
        for (; rb + 8 <= n; rb += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) v[u] = part[(size_t)(rb + u) * t_pad + j];
#pragma unroll
            for (int u = 0; u < 8; ++u) s += (double)v[u];
        }
        for (; rb < n; ++rb) s += (double)part[(size_t)rb * t_pad + j];
        if (tok_dist) tok_dist[j] = (float)s;
    }
    red[threadIdx.x] = s;
    __syncthreads();
    for (int off = 128; off >= 1; off >>= 1) {
        if (threadIdx.x < off) red[threadIdx.x] += red[threadIdx.x + off];
        __syncthreads();
    }
    if (threadIdx.x == 0) wg_sums[blockIdx.x] = red[0];
}

__global__ __launch_bounds__(64) void dist_final_kernel(const double *__restrict__ wg_sums, int n,
                                                        double *__restrict__ dist) {
    if (threadIdx.x != 0) return;
    double s = 0.0;
    for (int i = 0; i < n; ++i) s += wg_sums[i];
    *dist = s;
}

size_t dist_scratch_floats(int T) {
    const int ntl = (T + kTile - 1) / kTile, t_pad = ntl * kTile;
    const int n_rowblk = (T + 63) / 64;
    const int n_wg = (T + 255) / 256;
    const size_t gram = (size_t)t_pad + (size_t)n_rowblk * t_pad + 2 * (size_t)n_wg + 2;
    // the forms for fewer tokens keep partials of 16 rows in fp64 or of 32 rows: at most 2 T (T / 16 + 1) floats, less
    // than the T * 64 floats that every context has for T tokens
    if (T <= kDistSmallMaxTokens) return gram > 2 * (size_t)T * ((T + 15) / 16) ? gram : 2 * (size_t)T * ((T + 15) / 16);
    if (!dist_block_wide(T)) return gram > (size_t)t_pad * ntl ? gram : (size_t)t_pad * ntl;
    return gram;
}

hipError_t launch_token_dist(const uint16_t *h, int T, int d, const void *xp, float *scratch, float *tok_dist,
                             double *dist, int form, hipStream_t s) {
    if (T <= 0 || d % 64 != 0 || form < 0 || form > 2) return hipErrorInvalidValue;
    const int ntiles = (T + kTile - 1) / kTile;
    const int t_pad = ntiles * kTile;
    const int n_rowblk = (T + 63) / 64;
    const int n_wg = (T + 255) / 256;
    if (form == 0 && T <= kDistRowMaxTokens) {
        double *sums = reinterpret_cast<double *>(scratch);   // T doubles (8-byte aligned: the scratch is), then their sum
        hipLaunchKernelGGL(dist_row_kernel, dim3(T), dim3(64 * kDistRowWaves), 0, s, h, T, d, tok_dist, sums);
        hipLaunchKernelGGL(dist_final_kernel, dim3(1), dim3(64), 0, s, sums, T, dist);
        return hipGetLastError();
    }
    if (form == 0 && T <= kDistSmallMaxTokens) {
        double *part = reinterpret_cast<double *>(scratch);   // 8-byte aligned: the scratch is
        const int cols = (T + kDistSmallCols - 1) / kDistSmallCols, rows = (T + kDistSmallRows - 1) / kDistSmallRows;
        hipLaunchKernelGGL(dist_small_kernel, dim3(rows, cols), dim3(64 * kDistSmallWaves), 0, s, h, T, d, part);
        // the last row chunk of token j's group is that of its last token: (8 (j / 8) + 7) / 16 = j / 16
        hipLaunchKernelGGL(dist_sum_kernel<double>, dim3(1), dim3(1024), 0, s, part, T, T, kDistSmallRows, tok_dist, dist);
        return hipGetLastError();
    }
    if (!dist_needs_packed(T, form)) {
        const bool wide = dist_block_wide(T);
        const int nb = (T + (wide ? 63 : 31)) / (wide ? 64 : 32), blocks = nb * (nb + 1) / 2;
        // a block's d over eight waves while every block has a compute unit to itself: half the stages one after the other
        // (the call, four / eight waves: d = 2048, T = 700 12.6 / 12.4, 1056 20.2 / 18.0 us; d = 4096, 700 17.1 / 16.5, 1100
        // 30.7 / 26.3); with more blocks two of four waves share a unit as well and add up fewer partials (d = 2048, T = 900
        // 16.0 / 18.3, 1500 28.2 / 32.7; d = 4096 23.0 / 26.7, 43.7 / 49.3)
        const bool eight = blocks <= 256 && d % 128 == 0;
        if (wide && eight) hipLaunchKernelGGL((dist_block_kernel<2, 1, 8>), dim3(blocks), dim3(512), 0, s, h, T, d, scratch, t_pad);
        else if (wide) hipLaunchKernelGGL((dist_block_kernel<2, 1, 4>), dim3(blocks), dim3(256), 0, s, h, T, d, scratch, t_pad);
        else if (eight) hipLaunchKernelGGL((dist_block_kernel<1, 2, 8>), dim3(blocks), dim3(512), 0, s, h, T, d, scratch, t_pad);
        else hipLaunchKernelGGL((dist_block_kernel<1, 2, 4>), dim3(blocks), dim3(256), 0, s, h, T, d, scratch, t_pad);
        hipLaunchKernelGGL(dist_sum_kernel<float>, dim3(1), dim3(1024), 0, s, scratch, T, t_pad, wide ? 64 : 32, tok_dist, dist);
        return hipGetLastError();
    }
    float *norms = scratch;
    float *part = scratch + t_pad;
    // 8-byte aligned slot for the workgroup sums behind the partials
    size_t off = (size_t)t_pad + (size_t)n_rowblk * t_pad;
    off += off & 1;
    double *wg_sums = reinterpret_cast<double *>(scratch + off);
    hipLaunchKernelGGL(dist_norm_kernel, dim3((t_pad + 3) / 4), dim3(256), 0, s, h, T, d, norms, t_pad);
    const int nB = (ntiles + 7) / 8;
    const long long total = gram_blocks(nB);
    if (form != 1) {
        // One block per compute unit at a time: the blocks left over after the last full round of 256 would be a
        // round of their own.  Up to 64 of them run as quarters instead (at most 256 workgroups, each with a
        // quarter of the matrix-core work per stage).
        const long long rem = total % 256;
        const long long n_split = total > 256 && rem <= 64 ? rem : 0;
        const long long whole = total - n_split;
        const long long runs = (whole + kGramRun - 1) / kGramRun;
        const long long main_grid = (runs + 7) / 8 * 8 * kGramRun;
        const long long grid = main_grid + 4 * n_split;
        if (grid > 0x7fffffffLL) return hipErrorInvalidValue;
        hipLaunchKernelGGL(dist_gram_tiled_kernel, dim3((unsigned)grid), dim3(256), 0, s,
                           reinterpret_cast<const uint4 *>(xp), norms, T, d, part, t_pad, n_rowblk, nB, whole,
                           (int)main_grid);
    } else {
        const int nJB = (ntiles + kDistColTiles - 1) / kDistColTiles;
        const int nIB = (ntiles + kDistRowTiles - 1) / kDistRowTiles;
        hipLaunchKernelGGL(dist_tile_kernel, dim3(nJB, nIB), dim3(256), 0, s, reinterpret_cast<const uint4 *>(xp),
                           norms, T, d, part, t_pad, n_rowblk);
    }
    hipLaunchKernelGGL(dist_reduce_kernel, dim3(n_wg), dim3(256), 0, s, part, T, t_pad, tok_dist, wg_sums);
    hipLaunchKernelGGL(dist_final_kernel, dim3(1), dim3(64), 0, s, wg_sums, n_wg, dist);
    return hipGetLastError();
}

}  // namespace ef

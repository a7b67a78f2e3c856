// Grouped SwiGLU expert FFN with 4-bit expert weights (w = (q - 8) * s, one bf16 scale per matrix row
// and group of 128 inputs), for groups of any size (the largest launches expand the weights first: ef_plan.hip).
//
// With 4-bit weights a byte of weights meets four times as many token bytes as with bf16, so the
// re-reads of the token (or activation) fragments, not the weight stream, would bound a kernel in
// which every wave fetches its own copy.  Here the four waves of a workgroup work on the same
// tokens and the same K range (different weight rows / output columns): each wave fetches a quarter
// of the token fragments of a stage, the workgroup shares them through a small LDS ring, and only
// the weight stream is private to a wave.  A stage is one "quad" of weights per matrix (four
// k-steps, 64 inputs); weight quads, scales and the wave's share of token fragments sit in a
// register ring of kDepth stages filled that many stages ahead with unconditional loads (clamped
// addresses), one barrier per stage.  Dequantisation happens on the operand fragment, where a lane
// holds one matrix row (column) and therefore needs one scale per group, and in fp16: the codes
// become the fp16 numbers 1024 + q (or 64 + q) by one bit operation, a packed subtraction gives q - 8 exactly and
// a packed multiplication (q - 8) * s: three vector instructions per pair of weights where an fp32
// route costs seven, which is what keeps these kernels on the memory side of the balance.  Passes of one and
// of two token tiles with up to 48 tokens leave the scale to the sums (q4_stream16, q4_stream32).  The
// matrix cores therefore run in fp16 (fp32 accumulation): the packed tokens of a 4-bit context and
// the intermediate activations are fp16 fragments (tokens convert exactly from bf16 for
// 2^-14 <= |x| < 65504).
#include <algorithm>

#include "ef_device.h"
#include "ef_kernels.h"

namespace ef {

typedef _Float16 q4_half2 __attribute__((ext_vector_type(2)));
typedef _Float16 q4_half8 __attribute__((ext_vector_type(8)));

// dword x = eight codes of one lane for one k-step, code t at bits 4*(t/2) + 16*(t%2);
// s2 = the lane's scale in both halves.  Codes in mantissa bits 0..3 under the exponent of 1024 (unit in the
// last place 1) are the fp16 numbers 1024 + q, codes in mantissa bits 4..7 under the exponent of 64 (unit
// 1/16) are 64 + q: x & 0x000F000F | 0x64006400 is the pair t = 0, 1, x & 0x00F000F0 | 0x54005400 the pair
// t = 2, 3, and x >> 8 gives the other two pairs the same way (one shift per dword instead of three).  Minus
// 1032 (72) is q - 8 exactly; times s rounds once to fp16 (11 significant bits for a 4-bit integer times an
// 8-bit mantissa: relative error <= 2^-12).
__device__ __forceinline__ u32x4_t q4_codes(uint32_t x) {   // q - 8
    const q4_half2 off_lo = {(_Float16)-1032.f, (_Float16)-1032.f}, off_hi = {(_Float16)-72.f, (_Float16)-72.f};
    const uint32_t y = x >> 8;
    // the masks live in vector registers the compiler cannot see through: "and" and "or" then fit one
    // three-operand instruction (it takes a single literal, here the exponent pattern)
    uint32_t m_lo = 0x000F000Fu, m_hi = 0x00F000F0u;
    asm("" : "+v"(m_lo));
    asm("" : "+v"(m_hi));
    const uint32_t pr[4] = {(x & m_lo) | 0x64006400u, (x & m_hi) | 0x54005400u,
                            (y & m_lo) | 0x64006400u, (y & m_hi) | 0x54005400u};
    u32x4_t out;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const q4_half2 w = __builtin_bit_cast(q4_half2, pr[p]) + ((p & 1) ? off_hi : off_lo);
        out[p] = __builtin_bit_cast(uint32_t, w);
    }
    return out;
}
__device__ __forceinline__ u32x4_t dequant_q4(uint32_t x, q4_half2 s2) {   // (q - 8) s
    u32x4_t out = q4_codes(x);
#pragma unroll
    for (int p = 0; p < 4; ++p) {
        const uint32_t c = out[p];   // (a bit cast of the element itself reads element 0)
        out[p] = __builtin_bit_cast(uint32_t, __builtin_bit_cast(q4_half2, c) * s2);
    }
    return out;
}

// bf16 scale (exact in fp16 for 2^-14 <= |s| < 65504) in both halves of a packed pair
__device__ __forceinline__ q4_half2 q4_scale(uint16_t b) {
    const _Float16 h = (_Float16)__builtin_bit_cast(float, (uint32_t)b << 16);
    return q4_half2{h, h};
}

// beyond the largest finite fp16 an activation saturates to it, as in the 16-bit kernels; NaN stays NaN
__device__ __forceinline__ float q4_saturate(float v) {
    const float lim = 65504.f;
    v = v > lim ? lim : v;
    return v < -lim ? -lim : v;
}

// 16 rows of matrix A (weights) x 16 tokens, 32 inputs: lane l carries 8 inputs (group l / 16) of row, and of token, l % 16;
// the accumulator lane l holds token l % 16 and rows 4 (l / 16) .. + 3.
typedef float floatx4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ floatx4_t mfma16h(u32x4_t a, u32x4_t b, floatx4_t c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, b), c, 0, 0, 0);
}
// x, y: a dword per lane of two fragments (32 rows, lanes 32 g + i) -> lo: of rows 0..15, hi: of rows 16..31, lane l row
// l % 16, with the inputs of its quarter l / 16 = 2 g + f from half g of fragment f (0: x, 1: y).  For x = y: a value per row
// in the lanes of that row.
__device__ __forceinline__ void split_rows(uint32_t x, uint32_t y, uint32_t &lo, uint32_t &hi) {
    const auto r = __builtin_amdgcn_permlane16_swap(x, y, false, false);
    lo = r[0];
    hi = r[1];
}

// register ring: stages in flight per wave (four were measured slower than six with two token tiles per pass
// and one wave per SIMD)
constexpr int kQ4Depth = 6;
constexpr int kQ4Lds = 4;     // LDS ring of shared token / activation fragments (stages)

// The K loops of the first half share everything but a stage's arithmetic (COMPUTE).  A stage: hand the next stage's token
// fragments to the workgroup, compute this one, refill the register slot just used, barrier (the next stage's fragments are
// visible; this stage's LDS buffer is overwritten three stages from now).  Loads are unconditional: past the end the last
// stage is read again.
// a scale holds for two stages: where the loop starts at an even one (PAIRS) and the ring has an even length, the even slots
// hold the even stages and only those load it
#define EF_Q4U_SCALES(slot) (!PAIRS || D % 2 != 0 || (slot) % 2 == 0)
#define EF_Q4U_LOAD(slot, kq)                                                                             \
    {                                                                                                     \
        const int kc_ = k0 + min((kq), nloc - 1);                                                         \
        _Pragma("unroll") for (int u = 0; u < NTL; ++u)                                                   \
            xr[slot][u] = *reinterpret_cast<const u32x4_t *>(xsrc[u] + (size_t)(4 * kc_ + wave) * 64);    \
        __builtin_amdgcn_sched_barrier(0);                                                                \
        qa[slot] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(w13 + (size_t)kc_ * 128));       \
        qb[slot] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(w13 + (size_t)kc_ * 128 + 64));  \
        if (EF_Q4U_SCALES(slot)) {                                                                        \
            sa[slot] = sA[(size_t)(kc_ >> 1) * 64];                                                       \
            sb[slot] = sA[(size_t)(kc_ >> 1) * 64 + 32];                                                  \
        }                                                                                                 \
    }
#define EF_Q4U_SHARE(slot, st)                                                                            \
    {                                                                                                     \
        _Pragma("unroll") for (int u = 0; u < NTL; ++u) xs[(st) & (kQ4Lds - 1)][u * 4 + wave][lane] = xr[slot][u]; \
    }
#define EF_Q4U_STAGE(COMPUTE, slot, next_slot, st)                                                        \
    {                                                                                                     \
        EF_Q4U_SHARE(next_slot, (st) + 1)                                                                 \
        COMPUTE(slot, st)                                                                                 \
        EF_Q4U_LOAD(slot, (st) + D)                                                                       \
        __syncthreads();                                                                                  \
    }
#define EF_Q4U_RUN(COMPUTE)                                                                               \
    {                                                                                                     \
        _Pragma("unroll") for (int ring_ = 0; ring_ < D; ++ring_) EF_Q4U_LOAD(ring_, ring_)               \
        EF_Q4U_SHARE(0, 0)                                                                                \
        __syncthreads();                                                                                  \
        int st = 0;                                                                                       \
        for (; st + D <= nloc; st += D) {                                                                 \
            _Pragma("unroll") for (int ring_ = 0; ring_ < D; ++ring_) EF_Q4U_STAGE(COMPUTE, ring_, (ring_ + 1) % D, st + ring_) \
        }                                                                                                 \
        _Pragma("unroll") for (int ring_ = 0; ring_ < D - 1; ++ring_)                                     \
            if (st + ring_ < nloc) EF_Q4U_STAGE(COMPUTE, ring_, ring_ + 1, st + ring_)                    \
    }

// K loop of the first half for NTL live token tiles of a pass of four: stages [k0, k0 + nloc) of 64 inputs each, `xs` the
// LDS ring of the four waves that share these stages.  The number of live tiles is the same for a whole workgroup.
template <int TT, int NTL, int D, bool PAIRS>
__device__ __forceinline__ void q4_up_stream(const uint4 *__restrict__ w13, const uint16_t *__restrict__ sA,
                                             const uint4 *const (&xsrc)[TT], u32x4_t (*xs)[TT * 4][64], int k0, int nloc,
                                             int wave, int lane, floatx16 (&G)[TT], floatx16 (&U)[TT]) {
    u32x4_t qa[D], qb[D], xr[D][NTL];
    uint16_t sa[D], sb[D];
    q4_half2 f1_, f3_;
    // The MFMAs of a k-step are issued between the vector instructions that dequantise the next
    // k-step's fragments (one MFMA, then a share of the ~40 vector instructions), so the matrix
    // cores work while the wave converts: a wave issues in order and has the SIMD to itself, nothing
    // else would overlap the two.
#define EF_Q4U_COMPUTE(slot, st)                                                                          \
    {                                                                                                     \
        if (EF_Q4U_SCALES(slot)) { f1_ = q4_scale(sa[slot]); f3_ = q4_scale(sb[slot]); }                   \
        u32x4_t xb_[NTL][4];                                                                              \
        _Pragma("unroll") for (int tt = 0; tt < NTL; ++tt)                                                \
            _Pragma("unroll") for (int j = 0; j < (NTL > 2 ? 1 : 4); ++j) xb_[tt][j] = xs[(st) & (kQ4Lds - 1)][tt * 4 + j][lane]; \
        u32x4_t a1_ = dequant_q4(qa[slot][0], f1_), a3_ = dequant_q4(qb[slot][0], f3_);                   \
        _Pragma("unroll") for (int j = 0; j < 4; ++j) {                                                   \
            u32x4_t n1_ = a1_, n3_ = a3_;                                                                 \
            if (NTL > 2 && j < 3) { /* wide passes: a k-step ahead, not the whole stage (registers) */   \
                _Pragma("unroll") for (int tt = 0; tt < NTL; ++tt)                                        \
                    xb_[tt][j + 1] = xs[(st) & (kQ4Lds - 1)][tt * 4 + j + 1][lane];                       \
            }                                                                                             \
            if (j < 3) { n1_ = dequant_q4(qa[slot][j + 1], f1_); n3_ = dequant_q4(qb[slot][j + 1], f3_); } \
            _Pragma("unroll") for (int tt = 0; tt < NTL; ++tt) {                                           \
                G[tt] = mfma32h(a1_, xb_[tt][j], G[tt]);                                                  \
                U[tt] = mfma32h(a3_, xb_[tt][j], U[tt]);                                                  \
            }                                                                                             \
            if (j < 3) {                                                                                  \
                _Pragma("unroll") for (int q_ = 0; q_ < 2 * NTL; ++q_) {                                  \
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                    \
                    __builtin_amdgcn_sched_group_barrier(0x002, 40 / (2 * NTL), 0);                       \
                }                                                                                         \
            }                                                                                             \
            a1_ = n1_; a3_ = n3_;                                                                         \
        }                                                                                                 \
    }
    EF_Q4U_RUN(EF_Q4U_COMPUTE)
#undef EF_Q4U_COMPUTE
}

#undef EF_Q4U_RUN
#undef EF_Q4U_STAGE
#undef EF_Q4U_SHARE
#undef EF_Q4U_LOAD
#undef EF_Q4U_SCALES

// ------------------------------------------------------------------------------------------
// K loops of passes of one and two tiles with up to 48 tokens, either half: sum_k x_k (q_k - 8) s as s (sum_k x_k (q_k - 8))
// per block of the 128 inputs that share a scale.  The operand is q - 8 alone, nine vector instructions per eight weights
// instead of thirteen, and the weights' scales are read and converted once per block; the matrix cores sum a block from zero,
// and every second stage the block's sums join the totals with one multiply-add per accumulator element, in 32 bits and with
// the scale as it is.  The operands are swapped against the other passes (tokens are the rows), so a lane has one weight row
// and needs one scale.  Passes of 49 tokens and more, and passes of four whatever their last one holds, keep (q - 8) s as the
// operand: tiles share its cost, and a block's accumulators beside those of the totals would take the registers of the ring.
// The two round differently, so the width of a layer's passes is chosen once for all of its phases (launch_phase).
//
// Bound by the weight stream and what a wave's in-order issue leaves idle of it.  Two layers, before / after: eight
// Mixtral-shaped experts 1 / 8 / 30 / 64 tokens 145.0 / 137.8, 270.8 / 254.4, 331.0 / 314.9, 361.2 / 338.8 us (64 tokens: first
// half 103 -> 100, its loads alone 91, second half 57 -> 51); DeepSeek-shaped 4 / 32 / 100 tokens 107.3 / 101.9, 146.6 / 140.6,
// 186.1 / 181.2; Qwen-shaped 25 / 200 tokens 116.9 / 111.5, 219.0 / 214.1.  The block's sums cost registers: first halves of
// passes of one need 155 instead of 117 to 123 and fit three waves per SIMD instead of four.  Raised codes 64 + q as the
// operand (seven instructions), 72 times the sum of the inputs taken off through LDS: 257.9 and 360.7 us at 8 and 64 tokens,
// and rounding errors of its own.
// ------------------------------------------------------------------------------------------
struct Q4Streams {                 // of one wave: two weight streams (W1 and W3, or two column blocks of W2) and their scales
    const uint4 *wa, *wb;
    const uint16_t *sa, *sb;
    int wstep, sstep;              // 16-byte units per stage, scales per block of 128 inputs
};
// A stage is that of EF_Q4U_STAGE.  Even slots of the ring hold the first stage of a block, and only those load its scales:
// the loops start at an even stage.
#define EF_Q4_LOAD(slot, kq)                                                                              \
    {                                                                                                     \
        const int kc_ = min((kq), last);                                                                  \
        _Pragma("unroll") for (int u = 0; u < NTL; ++u)                                                   \
            xr[slot][u] = *reinterpret_cast<const u32x4_t *>(src[u] + (size_t)(4 * kc_ + wave) * 64);     \
        __builtin_amdgcn_sched_barrier(0);                                                                \
        qa[slot] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(w.wa + (size_t)kc_ * w.wstep)); \
        qb[slot] = __builtin_nontemporal_load(reinterpret_cast<const u32x4_t *>(w.wb + (size_t)kc_ * w.wstep)); \
        if ((slot) % 2 == 0) {                                                                            \
            sa[(slot) / 2] = w.sa[(size_t)(kc_ >> 1) * w.sstep];                                          \
            sb[(slot) / 2] = w.sb[(size_t)(kc_ >> 1) * w.sstep];                                          \
        }                                                                                                 \
    }
#define EF_Q4_SHARE(slot, st)                                                                             \
    {                                                                                                     \
        _Pragma("unroll") for (int u = 0; u < NTL; ++u) xs[(st) & (kQ4Lds - 1)][u * 4 + wave][lane] = xr[slot][u]; \
    }
#define EF_Q4_STAGE(COMPUTE, slot, next_slot, st)                                                         \
    {                                                                                                     \
        EF_Q4_SHARE(next_slot, (st) + 1)                                                                  \
        COMPUTE(slot, st)                                                                                 \
        EF_Q4_LOAD(slot, (st) + D)                                                                        \
        __syncthreads();                                                                                  \
    }
#define EF_Q4_RUN(COMPUTE)                                                                                \
    {                                                                                                     \
        static_assert(D % 2 == 0, "even slots hold the first stage of a block");                          \
        const int last = max(q1, 1) - 1;                                                                  \
        _Pragma("unroll") for (int ring_ = 0; ring_ < D; ++ring_) EF_Q4_LOAD(ring_, q0 + ring_)           \
        EF_Q4_SHARE(0, q0)                                                                                \
        __syncthreads();                                                                                  \
        int st = q0;                                                                                      \
        for (; st + D <= q1; st += D) {                                                                   \
            _Pragma("unroll") for (int ring_ = 0; ring_ < D; ++ring_) EF_Q4_STAGE(COMPUTE, ring_, (ring_ + 1) % D, st + ring_) \
        }                                                                                                 \
        _Pragma("unroll") for (int ring_ = 0; ring_ < D - 2; ++ring_)                                     \
            if (st + ring_ < q1) EF_Q4_STAGE(COMPUTE, ring_, ring_ + 1, st + ring_)                       \
    }
__device__ __forceinline__ float q4_scale_f32(uint16_t b) { return __builtin_bit_cast(float, (uint32_t)b << 16); }

// NH half tiles of 16 tokens, an odd number: a last tile that is half live takes half the matrix work (most experts of a decode
// batch have no more than 16 tokens).  The codes of two k-steps are regrouped by rows before they are converted (one lane exchange
// per pair of dwords), so the instruction of 16 rows x 16 tokens takes 32 inputs of a quad's row; the token fragments are read
// from LDS in the same order of inputs.  A, B: [row half][half tile]; a lane holds row l % 16 of the half and tokens
// 4 (l / 16) .. + 3.
template <int TT, int NH, int D>
__device__ __forceinline__ void q4_stream16(const Q4Streams &w, const uint4 *const (&src)[TT], u32x4_t (*xs)[TT * 4][64],
                                            int q0, int q1, int wave, int lane,
                                            floatx4_t (&A)[2][2 * TT - 1], floatx4_t (&B)[2][2 * TT - 1]) {
    constexpr int NTL = (NH + 1) / 2;
    u32x4_t qa[D], qb[D], xr[D][NTL];
    uint16_t sa[D / 2], sb[D / 2];
    float f_[4];                      // scales of the current block: matrix, row half
    floatx4_t bl_[4][NH];             // sums of the current block
    const floatx4_t zero = {0.f, 0.f, 0.f, 0.f};
    const int rd = ((lane >> 4) & 1) * 64 + (lane >> 5) * 32 + (lane & 15);   // inputs of quarter l / 16: fragment l / 16 % 2, half l / 32
#define EF_Q4_COMPUTE(slot, st)                                                                           \
    {                                                                                                     \
        u32x4_t xb_[NH][2];                                                                               \
        _Pragma("unroll") for (int h = 0; h < NH; ++h)                                                    \
            _Pragma("unroll") for (int p = 0; p < 2; ++p)                                                 \
                xb_[h][p] = (&xs[(st) & (kQ4Lds - 1)][(h >> 1) * 4 + 2 * p][0])[rd + 16 * (h & 1)];       \
        uint32_t cd_[8]; /* codes of operand x */                                                         \
        if ((slot) % 2 == 0) {                                                                            \
            uint32_t fl_[4];                                                                              \
            const uint32_t fa_ = (uint32_t)sa[(slot) / 2] << 16, fb_ = (uint32_t)sb[(slot) / 2] << 16;    \
            split_rows(fa_, fa_, fl_[0], fl_[1]);                                                         \
            split_rows(fb_, fb_, fl_[2], fl_[3]);                                                         \
            _Pragma("unroll") for (int i = 0; i < 4; ++i) f_[i] = __builtin_bit_cast(float, fl_[i]);      \
        }                                                                                                 \
        _Pragma("unroll") for (int p = 0; p < 2; ++p) {                                                   \
            split_rows(qa[slot][2 * p], qa[slot][2 * p + 1], cd_[4 * p], cd_[4 * p + 1]);                 \
            split_rows(qb[slot][2 * p], qb[slot][2 * p + 1], cd_[4 * p + 2], cd_[4 * p + 3]);             \
        }                                                                                                 \
        u32x4_t w_ = q4_codes(cd_[0]);                                                                   \
        _Pragma("unroll") for (int x = 0; x < 8; ++x) {                                                   \
            u32x4_t n_ = w_;                                                                              \
            if (x < 7) n_ = q4_codes(cd_[x + 1]);                                                        \
            _Pragma("unroll") for (int h = 0; h < NH; ++h)                                                \
                bl_[x & 3][h] = mfma16h(xb_[h][x >> 2], w_, (slot) % 2 == 0 && x < 4 ? zero : bl_[x & 3][h]); \
            if (x < 7) {                                                                                  \
                _Pragma("unroll") for (int q_ = 0; q_ < NH; ++q_) {                                       \
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                    \
                    __builtin_amdgcn_sched_group_barrier(0x002, (10 + NH - 1) / NH, 0);                    \
                }                                                                                         \
            }                                                                                             \
            w_ = n_;                                                                                      \
        }                                                                                                 \
        if ((slot) % 2 == 1) {                                                                            \
            _Pragma("unroll") for (int h = 0; h < NH; ++h)                                                \
                _Pragma("unroll") for (int r = 0; r < 2; ++r)                                             \
                    _Pragma("unroll") for (int v = 0; v < 4; ++v) {                                       \
                        A[r][h][v] = __builtin_fmaf(f_[r], bl_[r][h][v], A[r][h][v]);                     \
                        B[r][h][v] = __builtin_fmaf(f_[2 + r], bl_[2 + r][h][v], B[r][h][v]);             \
                    }                                                                                     \
        }                                                                                                 \
    }
    EF_Q4_RUN(EF_Q4_COMPUTE)
#undef EF_Q4_COMPUTE
}

// One whole tile of 32 tokens (as two half tiles: the same matrix time, more instructions).  A lane holds row l % 32 and, in
// element v, token 8 (v / 4) + 4 (l / 32) + v % 4.
template <int TT, int D>
__device__ __forceinline__ void q4_stream32(const Q4Streams &w, const uint4 *const (&src)[TT], u32x4_t (*xs)[TT * 4][64],
                                            int q0, int q1, int wave, int lane, floatx16 &A, floatx16 &B) {
    constexpr int NTL = 1;
    u32x4_t qa[D], qb[D], xr[D][NTL];
    uint16_t sa[D / 2], sb[D / 2];
    float fa_ = 0.f, fb_ = 0.f;
    floatx16 ba_, bb_, zero;
    zero16(zero);
    zero16(ba_);
    zero16(bb_);
#define EF_Q4_COMPUTE(slot, st)                                                                           \
    {                                                                                                     \
        u32x4_t xb_[4];                                                                                   \
        _Pragma("unroll") for (int j = 0; j < 4; ++j) xb_[j] = xs[(st) & (kQ4Lds - 1)][j][lane];          \
        if ((slot) % 2 == 0) {                                                                            \
            fa_ = q4_scale_f32(sa[(slot) / 2]);                                                           \
            fb_ = q4_scale_f32(sb[(slot) / 2]);                                                           \
        }                                                                                                 \
        u32x4_t w_ = q4_codes(qa[slot][0]);                                                              \
        _Pragma("unroll") for (int x = 0; x < 8; ++x) {                                                   \
            u32x4_t n_ = w_;                                                                              \
            if (x < 7) n_ = q4_codes(((x + 1) & 1) ? qb[slot][(x + 1) >> 1] : qa[slot][(x + 1) >> 1]);   \
            if (x & 1) bb_ = mfma32h(xb_[x >> 1], w_, (slot) % 2 == 0 && x < 2 ? zero : bb_);             \
            else ba_ = mfma32h(xb_[x >> 1], w_, (slot) % 2 == 0 && x < 2 ? zero : ba_);                   \
            if (x < 7) {                                                                                  \
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                        \
                __builtin_amdgcn_sched_group_barrier(0x002, 10, 0);                                        \
            }                                                                                             \
            w_ = n_;                                                                                      \
        }                                                                                                 \
        if ((slot) % 2 == 1) {                                                                            \
            _Pragma("unroll") for (int v = 0; v < 16; ++v) {                                              \
                A[v] = __builtin_fmaf(fa_, ba_[v], A[v]);                                                 \
                B[v] = __builtin_fmaf(fb_, bb_[v], B[v]);                                                 \
            }                                                                                             \
        }                                                                                                 \
    }
    EF_Q4_RUN(EF_Q4_COMPUTE)
#undef EF_Q4_COMPUTE
}
#undef EF_Q4_RUN
#undef EF_Q4_STAGE
#undef EF_Q4_SHARE
#undef EF_Q4_LOAD


// ------------------------------------------------------------------------------------------
// first half: act = silu(X W1^T) * (X W3^T).  Workgroup = (group, pass of TT token tiles, four
// consecutive 32-row blocks of F), wave = one row block and one of KH halves of the K range.
//
// OCC = 2: registers for two workgroups per compute unit (launches with more workgroups than compute units).
// TT = 4: launches of many workgroups, and groups of 8 token tiles and more.  Bound by the matrix cores (32 instructions
// of 32 cycles per stage and wave, the dequantisation of about 520 cycles between them); a register ring of three stages
// and two workgroups per compute unit (ring of two: 3 to 5 % slower, four with one workgroup: 10 to 18 %).  Against passes of two, two
// layers: Mixtral-shaped 700 tokens 1370 -> 1190 us, DeepSeek-shaped 1000 tokens 564 -> 515; against the expansion to 16
// bits and 256 x 256 tiles for groups of 8 tiles and more: 1600 -> 1190 and 680 -> 515 us.
// KH = 2: eight waves, two per SIMD.  A wave issues in order, so with one wave per SIMD its dequantising
// vector instructions (about 40 % of its cycles), its waits for LDS and barriers (25 %) and its issue stalls
// add up; a second wave on the SIMD fills them.  A launch rarely has enough row blocks for that (two Mixtral-
// shaped experts: 896 for 1024 SIMDs), so the second wave comes from the K range: the four waves of a half
// share their token fragments as before (a ring per half), and at the end the upper half hands its partial
// sums to the lower one through LDS (the ring's space).
// ------------------------------------------------------------------------------------------
template <int TT, int KH, int OCC>
__global__ __launch_bounds__(256 * KH, OCC) void ffn_gate_up_q4_kernel(GroupTable gt, const uint4 *__restrict__ xp,
                                                                       uint4 *__restrict__ act, int d) {
    constexpr int D = TT == 4 ? 3 : (KH == 2 || OCC == 2) ? 4 : kQ4Depth;   // 3 and 6 measured slower with two waves per SIMD
    __shared__ __attribute__((aligned(16))) u32x4_t xs[KH][kQ4Lds][TT * 4][64];
    const int wg = blockIdx.x;
    int grp = 0;
    while (grp + 1 < gt.n_groups && gt.wg_start[grp + 1] <= wg) ++grp;
    const int local = wg - gt.wg_start[grp];
    const int F = gt.F[grp];
    const int rbw = (F >> 5) >> 2;               // workgroups per pass (F is a multiple of 128)
    const int pass = local / rbw;
    const int wave = (threadIdx.x >> 6) & 3, lane = threadIdx.x & 63;
    // scalar where it bounds the K loop; undivided ranges keep vector addresses (0 spelled out: <4, 1, 2> 71.4 -> 72.3 us for
    // 20 tiles of 5632 x 2048)
    const int kh = KH == 1 ? threadIdx.x >> 8 : __builtin_amdgcn_readfirstlane(threadIdx.x >> 8);
    const int rb = (local % rbw) * 4 + wave;
    int ntl = gt.n_tiles[grp] - pass * TT;
    if (ntl > TT) ntl = TT;
    const int nkb = d >> 4, nq = d >> 6;
    const char *blob = reinterpret_cast<const char *>(gt.blob[grp]);
    const uint4 *w13 = reinterpret_cast<const uint4 *>(blob) + (size_t)rb * nq * 128 + lane;
    const uint16_t *sA = reinterpret_cast<const uint16_t *>(blob + (size_t)3 * d * F / 2) +
                         (size_t)rb * (d >> 7) * 64 + (lane & 31);
    // live half tiles of 16 tokens (passes of one or two tiles work in those; of a half live tile they read the tokens that
    // exist twice, the same cache lines)
    const int nh = min((gt.count[grp] - pass * TT * kTile + 15) >> 4, 2 * TT);
    // Stages [k0, k0 + nloc) of this wave's half.  The loops that put the scale on the sums take whole blocks of 128 inputs,
    // the lower half the odd one; the upper half then waits at as many barriers more (`even`: barriers count waves), so every
    // wave passes the same number.
    const int cut = KH == 1 ? nq : TT < 4 && nh < 4 ? ((nq >> 1) + 1) / 2 * 2 : nq / 2;
    const int k0 = kh * cut, nloc = KH == 2 && kh ? nq - cut : cut;
    auto even = [&] {
        if constexpr (KH == 2)
            for (int i = nloc; i < cut; ++i) __syncthreads();
    };
    // this wave's share of the token fragments of a stage: k-step `wave` of each tile (tiles past the
    // group's last one repeat it; their results are dropped)
    const uint4 *xsrc[TT];
#pragma unroll
    for (int u = 0; u < TT; ++u)
        xsrc[u] = xp + (size_t)(gt.tile_start[grp] + pass * TT + min(u, ntl - 1)) * nkb * 64 +
                  (TT < 4 && nh == 2 * u + 1 ? lane & ~16 : lane);

    if constexpr (TT < 4) if (nh < 4) {
        const Q4Streams w = {w13, w13 + 64, sA, sA + 32, 128, 64};
        constexpr int HT = 2 * TT - 1;   // half tiles of a pass with a half live tile
        // where a lane's row f (0 .. 31) of the row block goes: half f / 16 of the paired-order fragments, lanes of half f / 4 % 2,
        // element 4 (f / 8 % 2) + f % 4
        uint16_t *out = reinterpret_cast<uint16_t *>(act + gt.act_off[grp] + ((size_t)pass * TT * (F >> 4) + rb * 2) * 64) +
                        ((lane >> 2) & 1) * 256 + ((lane >> 3) & 1) * 4 + (lane & 3);
        const size_t tile_halves = (size_t)(F >> 4) * 512;
        auto put = [&](uint16_t *at, float g, float u) {
            *at = __builtin_bit_cast(uint16_t, (_Float16)q4_saturate(silu_mul(g, u)));
        };
        if (nh == 2) {
            floatx16 G, U;
            zero16(G);
            zero16(U);
            q4_stream32<TT, D>(w, xsrc, xs[kh], k0, k0 + nloc, wave, lane, G, U);
            even();
            if constexpr (KH == 2) {
                float4 *red = reinterpret_cast<float4 *>(&xs[0][0][0][0]) + (size_t)wave * 8 * 64 + lane;
                if (kh == 1) {
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        red[q * 64] = make_float4(G[4 * q], G[4 * q + 1], G[4 * q + 2], G[4 * q + 3]);
                        red[(4 + q) * 64] = make_float4(U[4 * q], U[4 * q + 1], U[4 * q + 2], U[4 * q + 3]);
                    }
                }
                __syncthreads();
                if (kh == 1) return;
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 g = red[q * 64], u = red[(4 + q) * 64];
                    G[4 * q] += g.x; G[4 * q + 1] += g.y; G[4 * q + 2] += g.z; G[4 * q + 3] += g.w;
                    U[4 * q] += u.x; U[4 * q + 1] += u.y; U[4 * q + 2] += u.z; U[4 * q + 3] += u.w;
                }
            }
#pragma unroll
            for (int v = 0; v < 16; ++v)
                put(out + ((lane >> 4) & 1) * 512 + (8 * (v >> 2) + 4 * (lane >> 5) + (v & 3)) * 8, G[v], U[v]);
            return;
        }
        floatx4_t G[2][HT], U[2][HT];   // [row half][half tile of 16 tokens]
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int h = 0; h < HT; ++h) G[r][h] = U[r][h] = floatx4_t{0.f, 0.f, 0.f, 0.f};
        if (TT == 1 || nh == 1) q4_stream16<TT, 1, D>(w, xsrc, xs[kh], k0, k0 + nloc, wave, lane, G, U);
        else q4_stream16<TT, 2 * TT - 1, D>(w, xsrc, xs[kh], k0, k0 + nloc, wave, lane, G, U);
        even();

        if constexpr (KH == 2) {
            // every stage ends with a barrier: the ring is no longer read.  Lower half + upper half, in this order.
            floatx4_t *red = reinterpret_cast<floatx4_t *>(&xs[0][0][0][0]) + (size_t)wave * (4 * HT) * 64 + lane;
            static_assert(sizeof(xs) >= (size_t)4 * (4 * HT) * 64 * sizeof(floatx4_t), "partial sums fit the ring's space");
            if (kh == 1) {
#pragma unroll
                for (int r = 0; r < 2; ++r)
#pragma unroll
                    for (int h = 0; h < HT; ++h) {
                        red[((r * HT + h) * 2) * 64] = G[r][h];
                        red[((r * HT + h) * 2 + 1) * 64] = U[r][h];
                    }
            }
            __syncthreads();
            if (kh == 1) return;
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int h = 0; h < HT; ++h) {
                    G[r][h] += red[((r * HT + h) * 2) * 64];
                    U[r][h] += red[((r * HT + h) * 2 + 1) * 64];
                }
        }
#pragma unroll
        for (int h = 0; h < HT; ++h) {
            if (h >= nh) break;
#pragma unroll
            for (int r = 0; r < 2; ++r)
#pragma unroll
                for (int v = 0; v < 4; ++v)
                    put(out + (h >> 1) * tile_halves + r * 512 + (16 * (h & 1) + 4 * (lane >> 4) + v) * 8, G[r][h][v], U[r][h][v]);
        }
        return;
    }

    if constexpr (TT > 1) {
        floatx16 G[TT], U[TT];
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) { zero16(G[tt]); zero16(U[tt]); }

        if (TT == 4 && ntl == 1) q4_up_stream<TT, 1, D, KH == 1>(w13, sA, xsrc, xs[kh], k0, nloc, wave, lane, G, U);
        else if (TT == 2 || ntl == 2) q4_up_stream<TT, 2, D, KH == 1>(w13, sA, xsrc, xs[kh], k0, nloc, wave, lane, G, U);
        else if (ntl == 3) q4_up_stream<TT, (TT > 2 ? 3 : TT), D, KH == 1>(w13, sA, xsrc, xs[kh], k0, nloc, wave, lane, G, U);
        else q4_up_stream<TT, TT, D, KH == 1>(w13, sA, xsrc, xs[kh], k0, nloc, wave, lane, G, U);

        if constexpr (KH == 2) {
            // every stage ends with a barrier: the ring is no longer read.  Lower half + upper half, in this order.
            float4 *red = reinterpret_cast<float4 *>(&xs[0][0][0][0]) + (size_t)wave * (2 * TT * 4) * 64 + lane;
            static_assert(sizeof(xs) >= (size_t)4 * (2 * TT * 4) * 64 * sizeof(float4), "partial sums fit the ring's space");
            if (kh == 1) {
#pragma unroll
                for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        red[((tt * 2) * 4 + q) * 64] = make_float4(G[tt][4 * q], G[tt][4 * q + 1], G[tt][4 * q + 2], G[tt][4 * q + 3]);
                        red[((tt * 2 + 1) * 4 + q) * 64] = make_float4(U[tt][4 * q], U[tt][4 * q + 1], U[tt][4 * q + 2], U[tt][4 * q + 3]);
                    }
            }
            __syncthreads();
            if (kh == 1) return;
#pragma unroll
            for (int tt = 0; tt < TT; ++tt)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float4 g = red[((tt * 2) * 4 + q) * 64], u = red[((tt * 2 + 1) * 4 + q) * 64];
                    G[tt][4 * q] += g.x; G[tt][4 * q + 1] += g.y; G[tt][4 * q + 2] += g.z; G[tt][4 * q + 3] += g.w;
                    U[tt][4 * q] += u.x; U[tt][4 * q + 1] += u.y; U[tt][4 * q + 2] += u.z; U[tt][4 * q + 3] += u.w;
                }
        }
        // a lane holds 16 F-values of one token: the two paired-order fragments (fp16) the second half consumes
        const int nkb2 = F >> 4;
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            if (tt >= ntl) break;
            uint4 *dst = act + gt.act_off[grp] + ((size_t)(pass * TT + tt) * nkb2 + rb * 2) * 64 + lane;
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                uint32_t pk[4];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const float g0 = G[tt][8 * s + 2 * q], g1 = G[tt][8 * s + 2 * q + 1];
                    const float v0 = silu_mul(g0, U[tt][8 * s + 2 * q]);
                    const float v1 = silu_mul(g1, U[tt][8 * s + 2 * q + 1]);
                    pk[q] = __builtin_bit_cast(uint32_t, q4_half2{(_Float16)q4_saturate(v0), (_Float16)q4_saturate(v1)});
                }
                dst[(size_t)s * 64] = make_uint4(pk[0], pk[1], pk[2], pk[3]);
            }
        }
    }
}

hipError_t launch_ffn_gate_up_q4(const GroupTable &gt, int total_wgs, int tiles_per_pass, bool k_halves, const void *xp,
                                 void *act, int d, hipStream_t s) {
    if (total_wgs <= 0) return hipSuccess;
    if (d % 128 != 0) return hipErrorInvalidValue;
    for (int i = 0; i < gt.n_groups; ++i)
        if (gt.F[i] % 128 != 0 || gt.n_tiles[i] <= 0 ||
            gt.wg_start[i + 1] - gt.wg_start[i] != ffn_gate_up_q4_wgs(gt.F[i], gt.n_tiles[i], tiles_per_pass))
            return hipErrorInvalidValue;
    if (gt.wg_start[gt.n_groups] != total_wgs) return hipErrorInvalidValue;
    const uint4 *x = reinterpret_cast<const uint4 *>(xp);
    uint4 *a = reinterpret_cast<uint4 *>(act);
    // two K halves per workgroup when each half keeps a few stages (d / 64 in all, an even number; whole range / halves of an odd
    // number of 128-input blocks, eight experts of F = 2048, two layers: d = 640 16 / 200 tokens 78.1 / 76.9, 100.0 / 96.9 us,
    // d = 1920 95.7 / 92.5, 135.7 / 130.7)
    const bool halves = k_halves && (d >> 6) >= 8;
    // more workgroups than compute units: two of them per unit instead (whole K range each, the short register ring);
    // their waves stall at different times, where the halves of one workgroup meet at the same barriers
    // (seven Mixtral-shaped experts: 127 against 135 us, Qwen-shaped batch 52 against 60 us)
    const bool many = total_wgs > 256;
    if (tiles_per_pass == 4) hipLaunchKernelGGL((ffn_gate_up_q4_kernel<4, 1, 2>), dim3(total_wgs), dim3(256), 0, s, gt, x, a, d);
    else if (tiles_per_pass == 1 && many) hipLaunchKernelGGL((ffn_gate_up_q4_kernel<1, 1, 2>), dim3(total_wgs), dim3(256), 0, s, gt, x, a, d);
    else if (tiles_per_pass == 2 && many) hipLaunchKernelGGL((ffn_gate_up_q4_kernel<2, 1, 2>), dim3(total_wgs), dim3(256), 0, s, gt, x, a, d);
    else if (tiles_per_pass == 1 && halves) hipLaunchKernelGGL((ffn_gate_up_q4_kernel<1, 2, 1>), dim3(total_wgs), dim3(512), 0, s, gt, x, a, d);
    else if (tiles_per_pass == 1) hipLaunchKernelGGL((ffn_gate_up_q4_kernel<1, 1, 1>), dim3(total_wgs), dim3(256), 0, s, gt, x, a, d);
    else if (tiles_per_pass == 2 && halves) hipLaunchKernelGGL((ffn_gate_up_q4_kernel<2, 2, 1>), dim3(total_wgs), dim3(512), 0, s, gt, x, a, d);
    else if (tiles_per_pass == 2) hipLaunchKernelGGL((ffn_gate_up_q4_kernel<2, 1, 1>), dim3(total_wgs), dim3(256), 0, s, gt, x, a, d);
    else return hipErrorInvalidValue;
    return hipGetLastError();
}

// The K loops of the second half, as those of the first (a scale is loaded and converted for every stage)
#define EF_Q4D_LOAD(slot, kq)                                                                             \
    {                                                                                                     \
        const int kc_ = min((kq), nq - 1);                                                                \
        _Pragma("unroll") for (int u = 0; u < NTL; ++u)                                                   \
            ar[slot][u] = *reinterpret_cast<const u32x4_t *>(asrc[u] + (size_t)(4 * kc_ + wave) * 64);    \
        __builtin_amdgcn_sched_barrier(0);                                                                \
        _Pragma("unroll") for (int cw = 0; cw < CBW; ++cw) {                                              \
            qw[slot][cw] = __builtin_nontemporal_load(                                                    \
                reinterpret_cast<const u32x4_t *>(w2q + cw * qstride + (size_t)kc_ * 64));                \
            sc[slot][cw] = sB[cw * sstride + (size_t)(kc_ >> 1) * 32];                                    \
        }                                                                                                 \
    }
#define EF_Q4D_SHARE(slot, st)                                                                            \
    {                                                                                                     \
        _Pragma("unroll") for (int u = 0; u < NTL; ++u) as[(st) & (kQ4Lds - 1)][u * 4 + wave][lane] = ar[slot][u]; \
    }
#define EF_Q4D_STAGE(COMPUTE, slot, next_slot, st)                                                        \
    {                                                                                                     \
        EF_Q4D_SHARE(next_slot, (st) + 1)                                                                 \
        COMPUTE(slot, st)                                                                                 \
        EF_Q4D_LOAD(slot, (st) + D)                                                                       \
        __syncthreads();                                                                                  \
    }
#define EF_Q4D_RUN(COMPUTE)                                                                               \
    {                                                                                                     \
        _Pragma("unroll") for (int ring_ = 0; ring_ < D; ++ring_) EF_Q4D_LOAD(ring_, q0 + ring_)          \
        EF_Q4D_SHARE(0, q0)                                                                               \
        __syncthreads();                                                                                  \
        int st = q0;                                                                                      \
        for (; st + D <= q1; st += D) {                                                                   \
            _Pragma("unroll") for (int ring_ = 0; ring_ < D; ++ring_) EF_Q4D_STAGE(COMPUTE, ring_, (ring_ + 1) % D, st + ring_) \
        }                                                                                                 \
        _Pragma("unroll") for (int ring_ = 0; ring_ < D - 1; ++ring_)                                     \
            if (st + ring_ < q1) EF_Q4D_STAGE(COMPUTE, ring_, ring_ + 1, st + ring_)                      \
    }

// K loop of the second half for passes of four token tiles, as q4_up_stream: stages [q0, q1) of the nq stages of F
template <int TT, int NTL, int D, int CBW>
__device__ __forceinline__ void q4_down_stream(const uint4 *__restrict__ w2q, size_t qstride,
                                               const uint16_t *__restrict__ sB, size_t sstride,
                                               const uint4 *const (&asrc)[TT], u32x4_t (*as)[TT * 4][64], int nq, int q0,
                                               int q1, int wave, int lane, floatx16 (&acc)[CBW][TT]) {
    u32x4_t qw[D][CBW], ar[D][NTL];
    uint16_t sc[D][CBW];
    // as in the first half: the MFMAs of one weight fragment are issued between the vector
    // instructions that dequantise the next one
#define EF_Q4D_COMPUTE(slot, st)                                                                          \
    {                                                                                                     \
        u32x4_t af_[NTL][4];                                                                              \
        _Pragma("unroll") for (int tt = 0; tt < NTL; ++tt)                                                \
            _Pragma("unroll") for (int j = 0; j < 4; ++j) af_[tt][j] = as[(st) & (kQ4Lds - 1)][tt * 4 + j][lane]; \
        q4_half2 f_[CBW];                                                                                 \
        _Pragma("unroll") for (int cw = 0; cw < CBW; ++cw) f_[cw] = q4_scale(sc[slot][cw]);               \
        u32x4_t w_ = dequant_q4(qw[slot][0][0], f_[0]);                                                   \
        _Pragma("unroll") for (int idx = 0; idx < CBW * 4; ++idx) {                                       \
            const int cw = idx >> 2, j = idx & 3;                                                         \
            u32x4_t n_ = w_;                                                                              \
            if (idx + 1 < CBW * 4) n_ = dequant_q4(qw[slot][(idx + 1) >> 2][(idx + 1) & 3], f_[(idx + 1) >> 2]); \
            _Pragma("unroll") for (int tt = 0; tt < NTL; ++tt) acc[cw][tt] = mfma32h(w_, af_[tt][j], acc[cw][tt]); \
            if (idx + 1 < CBW * 4) {                                                                      \
                _Pragma("unroll") for (int q_ = 0; q_ < NTL; ++q_) {                                      \
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                    \
                    __builtin_amdgcn_sched_group_barrier(0x002, 20 / NTL, 0);                             \
                }                                                                                         \
            }                                                                                             \
            w_ = n_;                                                                                      \
        }                                                                                                 \
    }
    EF_Q4D_RUN(EF_Q4D_COMPUTE)
#undef EF_Q4D_COMPUTE
}

#undef EF_Q4D_RUN
#undef EF_Q4D_STAGE
#undef EF_Q4D_SHARE
#undef EF_Q4D_LOAD

// ------------------------------------------------------------------------------------------
// second half: Y = act W2^T.  Workgroup = (group, pass of TT token tiles, eight consecutive
// 32-column blocks of d, one of the group's K-slices), wave = two column blocks.  Activations are operand
// A (rows = tokens), shared through LDS; W2 quads operand B (a lane holds one output column).
// Each K-slice writes its own partial Y plane; the un-permute sums the planes in order.
// ------------------------------------------------------------------------------------------
template <int TT>
__global__ __launch_bounds__(256, 2) void ffn_down_q4_kernel(GroupTable gt, const uint4 *__restrict__ act,
                                                             float *__restrict__ Y, int d,
                                                             long long y_plane) {
    // passes of one with a ring of four fit three workgroups per compute unit (six: two; DeepSeek-shaped 32 tokens 144.3 -> 141.1
    // us for two layers); passes of two with six spill registers (DeepSeek-shaped 100 tokens 190 against 185.7)
    constexpr int D = TT == 4 ? 3 : 4, CBW = 2;
    __shared__ __attribute__((aligned(16))) u32x4_t as[kQ4Lds][TT * 4][64];
    const int wg = blockIdx.x;
    int grp = 0;
    while (grp + 1 < gt.n_groups && gt.wg_start[grp + 1] <= wg) ++grp;
    const int local = wg - gt.wg_start[grp];
    const int ncb = d >> 5, ncq = (ncb + 7) >> 3;
    const int ksg = gt.ksg[grp], kslice = local % ksg;
    const int cq = (local / ksg) % ncq, pass = (local / ksg) / ncq;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int cb0 = cq * 8 + wave * CBW;
    const bool valid = cb0 < ncb;                 // d is a multiple of 64: both column blocks or none
    const int cbc = valid ? cb0 : 0;              // waves past the last column load block 0 and drop the result
    const int F = gt.F[grp];
    const int nkb = F >> 4, nq = F >> 6;
    // whole blocks of 128 inputs (two stages)
    const int q0 = (int)((long long)kslice * (nq >> 1) / ksg) * 2, q1 = (int)((long long)(kslice + 1) * (nq >> 1) / ksg) * 2;
    int ntl = gt.n_tiles[grp] - pass * TT;
    if (ntl > TT) ntl = TT;

    const char *blob = reinterpret_cast<const char *>(gt.blob[grp]);
    const size_t qstride = (size_t)nq * 64, sstride = (size_t)(F >> 7) * 32;
    const uint4 *w2q = reinterpret_cast<const uint4 *>(blob + (size_t)d * F) + (size_t)cbc * qstride + lane;
    const uint16_t *sB = reinterpret_cast<const uint16_t *>(blob + (size_t)3 * d * F / 2 + (size_t)d * F / 32) +
                         (size_t)cbc * sstride + (lane & 31);
    const int nh = min((gt.count[grp] - pass * TT * kTile + 15) >> 4, 2 * TT);   // as in the first half
    const uint4 *asrc[TT];
#pragma unroll
    for (int u = 0; u < TT; ++u)
        asrc[u] = act + gt.act_off[grp] + (size_t)(pass * TT + min(u, ntl - 1)) * nkb * 64 +
                  (TT < 4 && nh == 2 * u + 1 ? lane & ~16 : lane);

    float *Yp = Y + (size_t)kslice * y_plane;
    if constexpr (TT < 4) if (nh < 4) {
        constexpr int HT = 2 * TT - 1;
        const Q4Streams w = {w2q, w2q + qstride, sB, sB + sstride, 64, 32};
        const int t0 = pass * TT * kTile, rows = gt.count[grp] - t0;
        float *row = Yp + (size_t)(gt.row_offset[grp] + t0) * d + cb0 * 32;
        if (nh == 2) {
            floatx16 a, b;
            zero16(a);
            zero16(b);
            q4_stream32<TT, D>(w, asrc, as, q0, q1, wave, lane, a, b);
            if (!valid) return;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int t = 8 * (v >> 2) + 4 * (lane >> 5) + (v & 3);
                if (t >= rows) continue;
                row[(size_t)t * d + (lane & 31)] = a[v];
                row[(size_t)t * d + 32 + (lane & 31)] = b[v];
            }
            return;
        }
        floatx4_t a[2][HT], b[2][HT];   // [half of the block's columns][half tile of 16 tokens]
#pragma unroll
        for (int r = 0; r < 2; ++r)
#pragma unroll
            for (int h = 0; h < HT; ++h) a[r][h] = b[r][h] = floatx4_t{0.f, 0.f, 0.f, 0.f};
        if (TT == 1 || nh == 1) q4_stream16<TT, 1, D>(w, asrc, as, q0, q1, wave, lane, a, b);
        else q4_stream16<TT, 2 * TT - 1, D>(w, asrc, as, q0, q1, wave, lane, a, b);

        if (!valid) return;
#pragma unroll
        for (int h = 0; h < HT; ++h)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int t = 16 * h + 4 * (lane >> 4) + v;
                if (h >= nh || t >= rows) continue;
#pragma unroll
                for (int r = 0; r < 2; ++r) {
                    row[(size_t)t * d + 16 * r + (lane & 15)] = a[r][h][v];
                    row[(size_t)t * d + 32 + 16 * r + (lane & 15)] = b[r][h][v];
                }
            }
        return;
    }
    if constexpr (TT > 1) {
        floatx16 acc[CBW][TT];
#pragma unroll
        for (int cw = 0; cw < CBW; ++cw)
#pragma unroll
            for (int tt = 0; tt < TT; ++tt) zero16(acc[cw][tt]);

        if (TT == 4 && ntl == 1) q4_down_stream<TT, 1, D, CBW>(w2q, qstride, sB, sstride, asrc, as, nq, q0, q1, wave, lane, acc);
        else if (TT == 2 || ntl == 2) q4_down_stream<TT, 2, D, CBW>(w2q, qstride, sB, sstride, asrc, as, nq, q0, q1, wave, lane, acc);
        else if (ntl == 3) q4_down_stream<TT, (TT > 2 ? 3 : TT), D, CBW>(w2q, qstride, sB, sstride, asrc, as, nq, q0, q1, wave, lane, acc);
        else q4_down_stream<TT, TT, D, CBW>(w2q, qstride, sB, sstride, asrc, as, nq, q0, q1, wave, lane, acc);

        if (!valid) return;
        const int g = lane >> 5;
#pragma unroll
        for (int tt = 0; tt < TT; ++tt) {
            if (tt >= ntl) break;
            // the product is formed transposed (W2 fragment first: the operand layouts are mirror images), so a lane
            // holds token lane % 32 and four consecutive output columns per accumulator quad: 16-byte stores
            const int tl = (pass * TT + tt) * kTile + (lane & 31);
            if (tl >= gt.count[grp]) continue;
            float *row = Yp + (size_t)(gt.row_offset[grp] + tl) * d;
#pragma unroll
            for (int cw = 0; cw < CBW; ++cw) {
                const int col = (cb0 + cw) * 32 + 4 * g;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    *reinterpret_cast<float4 *>(row + col + 8 * q) =
                        make_float4(acc[cw][tt][4 * q], acc[cw][tt][4 * q + 1], acc[cw][tt][4 * q + 2], acc[cw][tt][4 * q + 3]);
            }
        }
    }
}

hipError_t launch_ffn_down_q4(const GroupTable &gt, int total_wgs, int tiles_per_pass, const void *act,
                              float *y, long long y_plane, int d, hipEvent_t done, hipStream_t s) {
    if (total_wgs <= 0) return hipSuccess;
    if (d % 128 != 0) return hipErrorInvalidValue;
    for (int i = 0; i < gt.n_groups; ++i)
        if (gt.F[i] % 128 != 0 || gt.n_tiles[i] <= 0 || gt.ksg[i] < 1 ||
            gt.wg_start[i + 1] - gt.wg_start[i] != ffn_down_q4_wgs(d, gt.n_tiles[i], tiles_per_pass, gt.ksg[i]))
            return hipErrorInvalidValue;
    if (gt.wg_start[gt.n_groups] != total_wgs) return hipErrorInvalidValue;
    const uint4 *a = reinterpret_cast<const uint4 *>(act);
    if (tiles_per_pass == 1)
        return launch_done(ffn_down_q4_kernel<1>, dim3(total_wgs), dim3(256), done, s, gt, a, y, d, y_plane);
    else if (tiles_per_pass == 2)
        return launch_done(ffn_down_q4_kernel<2>, dim3(total_wgs), dim3(256), done, s, gt, a, y, d, y_plane);
    else if (tiles_per_pass == 4)
        return launch_done(ffn_down_q4_kernel<4>, dim3(total_wgs), dim3(256), done, s, gt, a, y, d, y_plane);
    return hipErrorInvalidValue;
}

// ------------------------------------------------------------------------------------------
// 4-bit blob -> 16-bit blob of the bf16 layout holding the fp16 numbers (q - 8) * s.
// One wave per quad position: (rb, kq) of W1 and W3 together (two quads in, eight fragments out), then
// (cb, kq) of W2 (one quad in, four fragments out).  A quad's dword j of lane l is the fragment of k-step
// 4*kq + j of the same lane, so reads and writes are whole 1 KiB rows of 64 lanes.
// ------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void dequant_q4_kernel(DequantTable t, int d) {
    const int grp = blockIdx.y;
    const int F = t.F[grp];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int nq = d >> 6, nq2 = F >> 6, nkb = d >> 4, nkb2 = F >> 4;
    const int nA = (F >> 5) * nq, nB = (d >> 5) * nq2;
    const int u = blockIdx.x * 4 + wave;
    if (u >= nA + nB) return;
    const char *blob = reinterpret_cast<const char *>(t.src[grp]);
    uint4 *out = reinterpret_cast<uint4 *>(t.dst[grp]);
    if (u < nA) {
        const int rb = u / nq, kq = u - rb * nq;
        const uint4 *q = reinterpret_cast<const uint4 *>(blob) + ((size_t)rb * nq + kq) * 128 + lane;
        const uint16_t *sc = reinterpret_cast<const uint16_t *>(blob + (size_t)3 * d * F / 2) +
                             ((size_t)rb * (d >> 7) + (kq >> 1)) * 64 + (lane & 31);
        const uint4 q1 = q[0], q3 = q[64];
        const q4_half2 f1 = q4_scale(sc[0]), f3 = q4_scale(sc[32]);
        uint4 *o1 = out + ((size_t)rb * 2 * nkb + 4 * kq) * 64 + lane;
        uint4 *o3 = o1 + (size_t)nkb * 64;
        const uint32_t c1[4] = {q1.x, q1.y, q1.z, q1.w}, c3[4] = {q3.x, q3.y, q3.z, q3.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const u32x4_t a = dequant_q4(c1[j], f1), b = dequant_q4(c3[j], f3);
            o1[(size_t)j * 64] = make_uint4(a[0], a[1], a[2], a[3]);
            o3[(size_t)j * 64] = make_uint4(b[0], b[1], b[2], b[3]);
        }
    } else {
        const int v = u - nA;
        const int cb = v / nq2, kq = v - cb * nq2;
        const uint4 *q = reinterpret_cast<const uint4 *>(blob + (size_t)d * F) + ((size_t)cb * nq2 + kq) * 64 + lane;
        const uint16_t *sc = reinterpret_cast<const uint16_t *>(blob + (size_t)3 * d * F / 2 + (size_t)d * F / 32) +
                             ((size_t)cb * (F >> 7) + (kq >> 1)) * 32 + (lane & 31);
        const uint4 q2 = q[0];
        const q4_half2 f2 = q4_scale(sc[0]);
        uint4 *o2 = reinterpret_cast<uint4 *>(reinterpret_cast<char *>(out) + (size_t)4 * d * F) +
                    ((size_t)cb * nkb2 + 4 * kq) * 64 + lane;
        const uint32_t c2[4] = {q2.x, q2.y, q2.z, q2.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const u32x4_t a = dequant_q4(c2[j], f2);
            o2[(size_t)j * 64] = make_uint4(a[0], a[1], a[2], a[3]);
        }
    }
}

hipError_t launch_dequant_q4(const DequantTable &t, int d, hipStream_t s) {
    if (t.n <= 0) return hipSuccess;
    if (t.n > kMaxGroups || d <= 0 || d % 128 != 0) return hipErrorInvalidValue;
    int units = 0;
    for (int i = 0; i < t.n; ++i) {
        if (t.F[i] <= 0 || t.F[i] % 128 != 0 || !t.src[i] || !t.dst[i]) return hipErrorInvalidValue;
        units = std::max(units, (t.F[i] / 32) * (d / 64) + (d / 32) * (t.F[i] / 64));
    }
    hipLaunchKernelGGL(dequant_q4_kernel, dim3((units + 3) / 4, t.n), dim3(256), 0, s, t, d);
    return hipGetLastError();
}

}  // namespace ef

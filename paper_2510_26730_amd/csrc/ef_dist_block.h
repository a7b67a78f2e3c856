// Body of the two kernels of Gram blocks (ef_dist.hip): B, R and NW are constants of the kernel that includes it, h, T, d,
// part and t_pad its arguments.
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
        const unsigned ch_ = min(2 * (kb) + lc, 2 * n - 1); /* past the part's end its last piece again */  \
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
        if ((kb) + U > n) { /* the part ends inside the stage: zeros past its end */                   \
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

// The forward product Y = X W^T of few tokens, whose work is the reading of W.
//
// What bounds it is how many compute units load and how much each has under way: in 64 x 64 tiles, 64 x 4096 x 4096 keeps
// 64 units busy with 512 KB each.  Here a tile is smaller (16 TM x 16 TN), and its four waves take every fourth K step of
// 128 each, through a ring of STAGES steps in LDS that is the wave's own: no barrier, and the whole LDS is in flight.  Their
// sums meet in LDS at the end and are added in the order of the waves.  us with the weights not in the caches, 64 x 64
// tiles / this (tokens x outputs x inputs): 16 x 4096 x 4096 10.8 / 6.3, 64 x 4096 x 4096 14.4 / 8.4, 128 x 4096 x 4096
// 13.1 / 10.4, 64 x 2176 x 7936 23.3 / 12.2, 64 x 1024 x 1024 5.4 / 3.9.  (Straight to registers, without LDS, a load
// covers 64 bytes of a row instead of 128: 64 x 4096 x 4096 10.5.)
#include "f8_gemm_kernels.hpp"

namespace f8 {

template <int GRAN, int TM, int TN, int STAGES>
__global__ __launch_bounds__(256) void gemm_rows_kernel(const uint8_t* __restrict__ A, const uint8_t* __restrict__ B,
                                                        uint16_t* __restrict__ D, int M, int N, int K, int64_t lda, int64_t ldb,
                                                        int64_t ldd, const float* __restrict__ isa, const float* __restrict__ isb,
                                                        int tiles_m, int tiles_n, uint32_t* __restrict__ amax_bits /* nullable */)
{
    constexpr int NW = 4, ROWS = 16 * TM, COLS = 16 * TN, PITCH = COLS + 4, STEP = (ROWS + COLS) * kBK, LOADS = 2 * (TM + TN);
    static_assert(NW * ROWS * PITCH * 4 <= NW * STAGES * STEP && (STAGES - 1) * LOADS < 64, "the sums take the ring's place; wait count");
    __shared__ __attribute__((aligned(1024))) uint8_t ring[NW][STAGES][STEP];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int fr = lane & 15, fg = lane >> 4;
    int tm, tn;
    tile_coords((int)blockIdx.x, tiles_m, tiles_n, &tm, &tn);
    const int m0 = tm * ROWS, n0 = tn * COLS;
    const uint8_t *a_base = A + (int64_t)m0 * lda, *b_base = B + (int64_t)n0 * ldb;

    // load l of a step: 8 rows of 128 bytes, A's rows first; lane: row lane / 8 of them, one 16-byte chunk.  Past the end of
    // the matrix or of the contraction it reads zeros.
    uint32_t off[LOADS];
    const int row8 = lane >> 3;
    static_for<LOADS>([&](auto L) {
        constexpr int l = L(), r = l < 2 * TM ? 8 * l : 8 * (l - 2 * TM);
        const int row = r + row8, left = l < 2 * TM ? M - m0 : N - n0;
        off[l] = row < left ? (uint32_t)row * (uint32_t)(l < 2 * TM ? lda : ldb) + 16 * ((lane & 7) ^ swz(row)) : kPastEnd;
    });
    typedef uint32_t v4u __attribute__((ext_vector_type(4)));
    const int steps = (K + kBK - 1) / kBK;
    // the step's number i among this wave's: step wave + 4 i
    auto request = [&](int i, int stage) {
        const int kt = wave + NW * i, left = K - kt * kBK;  // may be negative
        const int64_t k = (int64_t)(kt < steps ? kt : 0) * kBK;
        const uint64_t pa = (uint64_t)(a_base + k), pb = (uint64_t)(b_base + k);
        const v4u sa = {(uint32_t)pa, (uint32_t)(pa >> 32), kRecords, 0x00020000u}, sb = {(uint32_t)pb, (uint32_t)(pb >> 32), kRecords, 0x00020000u};
        static_for<LOADS>([&](auto L) {
            constexpr int l = L();
            uint8_t* lds = ring[wave][stage] + l * 1024;
            const uint32_t l32 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint8_t*)lds;
            // the swizzle looks at bits 1 and 2 of the row only: the same chunk in every load
            const uint32_t o = 16 * ((lane & 7) ^ swz(row8)) < left ? off[l] : kPastEnd;
            const v4u src = l < 2 * TM ? sa : sb;
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" : : "s"(l32), "v"(o), "s"(src) : "memory");
        });
    };
    auto fragment = [&](const uint8_t* op) {  // 16 rows; lane: row fr, k 32 fg .. + 31 (see gemm_tile_kernel)
        const uint8_t* row = op + fr * kBK;
        const int4 lo = *reinterpret_cast<const int4*>(row + 16 * ((2 * fg) ^ swz(fr)));
        const int4 hi = *reinterpret_cast<const int4*>(row + 16 * ((2 * fg + 1) ^ swz(fr)));
        return v8i{lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
    };
    v4f acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[i][j] = v4f{0.f, 0.f, 0.f, 0.f};

    const int mine = (steps - wave + NW - 1) / NW;
    static_for<STAGES - 1>([&](auto I) { request(I(), I()); });
    constexpr int kWait = (STAGES - 2) * LOADS;
    int stage = 0;
    for (int i = 0; i < mine; ++i) {
        // the oldest step has landed; this wave's reads of the step before it are done, whose place the request takes
        asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"(kWait) : "memory");
        request(i + STAGES - 1, stage == 0 ? STAGES - 1 : stage - 1);
        v8i a[TM], b[TN];
#pragma unroll
        for (int x = 0; x < TM; ++x) a[x] = fragment(ring[wave][stage] + 16 * x * kBK);
#pragma unroll
        for (int x = 0; x < TN; ++x) b[x] = fragment(ring[wave][stage] + (ROWS + 16 * x) * kBK);
#pragma unroll
        for (int x = 0; x < TM; ++x)
#pragma unroll
            for (int y = 0; y < TN; ++y)
                acc[x][y] = __builtin_amdgcn_mfma_scale_f32_16x16x128_f8f6f4(b[y], a[x], acc[x][y], F8_E4M3, F8_E4M3, 0, 0, 0, 0);
        stage = stage + 1 == STAGES ? 0 : stage + 1;
    }
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");  // no load may still be writing the ring
    __syncthreads();
    float(*sums)[ROWS][PITCH] = reinterpret_cast<float(*)[ROWS][PITCH]>(&ring[0][0][0]);
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j) *reinterpret_cast<v4f*>(&sums[wave][16 * i + fr][16 * j + 4 * fg]) = acc[i][j];
    __syncthreads();
    uint32_t amax_acc = 0;
    for (int q = threadIdx.x; q < ROWS * COLS / 4; q += 256) {  // four neighbouring outputs
        const int r = q / (COLS / 4), c = q % (COLS / 4) * 4, m = m0 + r, n = n0 + c;
        if (m >= M || n >= N) continue;
        v4f t = *reinterpret_cast<const v4f*>(&sums[0][r][c]);
#pragma unroll
        for (int w = 1; w < NW; ++w) t += *reinterpret_cast<const v4f*>(&sums[w][r][c]);
        f2 lo, hi;
        if constexpr (GRAN == F8_TENSORWISE) {
            const float st = isa[0] * isb[0];
            lo = f2{t[0] * st, t[1] * st}, hi = f2{t[2] * st, t[3] * st};
        } else {
            const float sa = isa[m];
            const float4 sb = *reinterpret_cast<const float4*>(isb + n);
            lo = f2{(t[0] * sa) * sb.x, (t[1] * sa) * sb.y}, hi = f2{(t[2] * sa) * sb.z, (t[3] * sa) * sb.w};
        }
        uint2 o;
        o.x = __builtin_bit_cast(uint32_t, __builtin_convertvector(lo, b2));
        o.y = __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, b2));
        *reinterpret_cast<uint2*>(D + (int64_t)m * ldd + n) = o;
        amax_acc = amax_pair(amax_acc, o);
    }
    if (amax_bits) {  // uniform; every thread of the block takes part
        __syncthreads();
        amax_publish<NW>(amax_acc, amax_bits, reinterpret_cast<uint32_t*>(&ring[0][0][0]));
    }
}

namespace {

struct RowsArgs {
    int g, M, N, K;
    const uint8_t *A, *B;
    const float *isa, *isb;
    uint16_t* D;
    uint32_t* amax_bits;
};

template <int TM, int TN, int STAGES>
void launch_rows(const RowsArgs& a, hipStream_t st)
{
    const int tiles_m = (a.M + 16 * TM - 1) / (16 * TM), tiles_n = (a.N + 16 * TN - 1) / (16 * TN);
    const auto kernel = a.g == F8_TENSORWISE ? gemm_rows_kernel<F8_TENSORWISE, TM, TN, STAGES> : gemm_rows_kernel<F8_ROWWISE, TM, TN, STAGES>;
    kernel<<<(unsigned)(tiles_m * tiles_n), 256, 0, st>>>(a.A, a.B, a.D, a.M, a.N, a.K, a.K, a.K, a.N, a.isa, a.isb, tiles_m, tiles_n,
                                                          a.amax_bits);
}

}  // namespace

// The tile that a forward of few tokens takes here, as 10 TM + TN, or 0: another kernel is faster.
int rows_tile(int M, int N, int K, int cus)
{
    // Estimates in us, from 75 sizes of 16 to 512 tokens and good to 10 %: a round of tiles takes a little and the bytes
    // that a tile loads, in any shape.  A wave needs a K step or more to be worth its share of the sums.
    if (M <= 0 || M > 512 || N <= 0 || K < 4 * kBK) return 0;
    auto kilobytes = [&](int rows, int cols) { return ((M < rows ? M : rows) + (N < cols ? N : cols)) * (double)K / 1024.0; };
    auto tiles = [&](int rows, int cols) { return (int64_t)((M + rows - 1) / rows) * ((N + cols - 1) / cols); };
    // (as without an output amax, whatever the call: these sums are in another order, and the amax is not to change Y)
    const TilePlan plan = plan_product(M, N, K, false, false, false, 0, cus);
    double best;
    if (plan.kind == TilePlan::kSmall)
        best = 3.1 + 0.0222 * kilobytes(kSm, kSm);
    else if (plan.kind == TilePlan::kQuarter && tiles(128, 128) <= cus)
        best = 2.5 + 0.75 * ksteps_of(K, 1);  // (0.75 to 1.0 a step)
    else
        return 0;
    best *= 0.93;
    int choice = 0;
    constexpr int kShapes[][2] = {{4, 4}, {4, 2}, {2, 2}, {1, 2}, {1, 1}};
    for (auto [tm, tn] : kShapes) {
        const int64_t rounds = (tiles(16 * tm, 16 * tn) + cus - 1) / cus;
        const double us = 2.2 + (double)rounds * (0.9 + 0.0205 * kilobytes(16 * tm, 16 * tn));
        if (rounds <= 2 && us < best) best = us, choice = 10 * tm + tn;
    }
    return choice;
}

// Contiguous, validated operands; amax_bits nullable.  true: the product has been enqueued.
bool gemm_rows(int g, int M, int N, int K, const uint8_t* A, const uint8_t* B, const float* isa, const float* isb, uint16_t* D,
               uint32_t* amax_bits, hipStream_t st)
{
    const int tile = rows_tile(M, N, K, cu_count());
    if (!tile) return false;
    if (amax_bits) zero_word(amax_bits, st);
    const RowsArgs a{g, M, N, K, A, B, isa, isb, D, amax_bits};
    switch (tile) {
        case 44: launch_rows<4, 4, 2>(a, st); return true;
        case 42: launch_rows<4, 2, 3>(a, st); return true;
        case 22: launch_rows<2, 2, 4>(a, st); return true;
        case 12: launch_rows<1, 2, 6>(a, st); return true;
        default: launch_rows<1, 1, 8>(a, st); return true;
    }
}

}  // namespace f8

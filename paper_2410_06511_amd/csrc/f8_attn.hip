// Causal grouped-query attention in bf16 between the Float8 linears of a transformer block
// (Section 2.2.4 applies Float8 to the linear layers only: everything else stays in bf16).  Flash-style: scores are never
// written; bf16 MFMA (v_mfma_f32_32x32x16_bf16) with fp32 accumulation and an online softmax.
//
// Orientation.  Of a 32x32 MFMA result, a lane holds one column (the row index of the SECOND
// operand) and 16 rows (row indices of the FIRST operand: 8 * (r / 4) + 4 * (lane / 32) + r % 4
// for register r).  The kernels form S^T = K Q^T (keys along registers, one query per lane), so
// the softmax statistics of a query live in one lane (plus its partner lane + 32), and the
// probabilities are already laid out as the operand of the next product, whose contraction runs
// over keys: 8 consecutive registers are the 8 contraction slots of a lane.  The other operand
// only has to present the same keys in the same slots: it is read from a copy that is contiguous
// along tokens (V^T in the forward, which f8_transpose_bf16 writes) or from the token-major tile by
// transposing LDS reads (the backward).  No operand is transposed in registers.
// Registers 8u .. 8u + 7 of lane group g hold tokens 16u + 4g + {0..3} and 16u + 8 + 4g + {0..3} of their 32-token
// block (reg_token), which the other operand presents in two reads of four.  (An order with eight consecutive
// tokens, one 16-byte read, is 1.5 % faster; but the sums then round differently, which the fp8 casts of a block
// amplify to 1e-2 and more of its gradients, and results would not compare with earlier ones.)
#include <type_traits>
#include <utility>

#include "f8_device.hpp"
#include "f8_host.hpp"

namespace f8 {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kAttnThreads = 256;
constexpr int kHd = 128;   // head dimension of every model the paper trains
constexpr int kBk = 64;    // keys per step
// operand reads ahead of their product (deeper did not help)
constexpr int kFwdAhead = 4, kDqAhead = 4, kDkvAhead = 3;

__device__ inline f32x16 mma(uint4 first, uint4 second, f32x16 acc)
{
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, first), __builtin_bit_cast(bf16x8, second), acc,
                                                   0, 0, 0);
}

__device__ inline uint32_t pack2(float lo, float hi)
{
    // v_cvt_pk_bf16_f32: round to nearest even
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    bf16x2 r = {(__bf16)lo, (__bf16)hi};
    return __builtin_bit_cast(uint32_t, r);
}

// registers 8u .. 8u+7 of an accumulator as a bf16 operand (8 contraction slots)
__device__ inline uint4 slots(const f32x16& c, int u)
{
    return make_uint4(pack2(c[8 * u], c[8 * u + 1]), pack2(c[8 * u + 2], c[8 * u + 3]), pack2(c[8 * u + 4], c[8 * u + 5]),
                      pack2(c[8 * u + 6], c[8 * u + 7]));
}

// the token of a 32-token block that register r of lane group g holds
__device__ inline int reg_token(int r, int g) { return 8 * (r >> 2) + 4 * g + (r & 3); }

// N products use(i, frag(i)) whose LDS operand reads run AHEAD products
// ahead of their use.  Left to itself the scheduler reads each operand right before its product
// and every product waits out the LDS latency; the group barriers pin the interleaving.
// ONE: the first ONE operands take one DS read, the others two.
template <int N, int AHEAD, int ONE = N, class Frag, class Use>
__device__ inline void pipelined_products(Frag frag, Use use)
{
    uint4 f[N];
#pragma unroll
    for (int i = 0; i < AHEAD; ++i) f[i] = frag(i);
    __builtin_amdgcn_sched_group_barrier(0x100, AHEAD <= ONE ? AHEAD : 2 * AHEAD - ONE, 0);  // DS reads
    [&]<int... I>(std::integer_sequence<int, I...>) {
        (..., [&] {
            if constexpr (I + AHEAD < N) f[I + AHEAD] = frag(I + AHEAD);
            use(I, f[I]);
            if constexpr (I + AHEAD < N) __builtin_amdgcn_sched_group_barrier(0x100, I + AHEAD < ONE ? 1 : 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // one MFMA
        }());
    }(std::make_integer_sequence<int, N>{});
}
// The same with the first STARTED operands read beforehand (in the phase before), and two DS
// instructions for operand i if two(i) (transposing reads, or both operands from LDS).  frag(i) may be
// a pair of operands.
template <int N, int AHEAD, int STARTED, class Frag, class Use, class Two, class F>
__device__ inline void started_products(const F (&started)[STARTED], Frag frag, Use use, Two two)
{
    static_assert(STARTED <= AHEAD && AHEAD <= N);
    F f[N];
#pragma unroll
    for (int i = 0; i < STARTED; ++i) f[i] = started[i];
#pragma unroll
    for (int i = STARTED; i < AHEAD; ++i) f[i] = frag(i);
    if constexpr (AHEAD > STARTED) __builtin_amdgcn_sched_group_barrier(0x100, 2 * (AHEAD - STARTED), 0);
    [&]<int... I>(std::integer_sequence<int, I...>) {
        (..., [&] {
            if constexpr (I + AHEAD < N) f[I + AHEAD] = frag(I + AHEAD);
            use(I, f[I]);
            if constexpr (I + AHEAD < N) __builtin_amdgcn_sched_group_barrier(0x100, two(I + AHEAD) ? 2 : 1, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        }());
    }(std::make_integer_sequence<int, N>{});
}

// ---- staging for the staggered kernels ----------------------------------------------------
// Tiles come straight from memory into LDS (one instruction of a wave: 64 lanes x 16 bytes into 1 KB of
// consecutive LDS), with no registers in between.  Rows are not padded then; instead the 16-byte chunks
// of a row are permuted so that the rows a read touches together fall into different banks.
static __device__ __attribute__((aligned(16))) const uint32_t kZeros[4] = {0, 0, 0, 0};  // what lanes past the end load

// Written as asm, so the compiler does not count these loads: stream_wait before the barrier that
// publishes the tile.  The second form (uniform base, 32-bit lane offset in bytes) issues faster.
__device__ inline uint32_t lds_address(uint16_t* lds) { return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) uint16_t*)lds; }
__device__ inline void load_to_lds(uint16_t* lds, const uint16_t* src)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" : : "s"(lds_address(lds)), "v"(src) : "memory");
}
__device__ inline void load_to_lds(uint16_t* lds, const uint16_t* base, uint32_t offset)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" : : "s"(lds_address(lds)), "v"(offset), "s"(base) : "memory");
}
__device__ inline void stream_wait() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// A barrier between two phases: this wave's LDS reads are done, and nothing moves across it.  Unlike
// __syncthreads it leaves loads in flight.
__device__ inline void phase_barrier()
{
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
}
// Values that are complete here: arithmetic without memory operations is not held by a barrier, and the
// compiler otherwise moves a phase's vector work past it, to the products that use the result.
__device__ inline void computed(float& v) { asm volatile("" : "+v"(v)); }
__device__ inline void computed(uint4& v) { asm volatile("" : "+v"(v.x), "+v"(v.y), "+v"(v.z), "+v"(v.w)); }

// Successive tiles of a tensor, PITCH elements per tile row.  A wave's share is N pieces of 1 KB; lane i of a
// piece fills physical chunk i % CPR of row i / CPR.  FAR: rows of the tensor so far apart that a lane's
// offset within a tile does not fit 32 bits.
template <int ROWS, int PITCH, int NW, bool FAR>
struct TileStream {
    static constexpr int CPR = PITCH / 8, RPP = 64 / CPR;  // 16-byte chunks per row, rows per piece
    static constexpr int N = ROWS / RPP / NW;
    static_assert(N >= 1 && N * RPP * NW == ROWS, "the pieces divide evenly over the waves");
    const uint16_t* tile;  // first element of the next tile
    std::conditional_t<FAR, uint64_t, uint32_t> offset[N];  // of this lane's 16 bytes in it, in bytes
    int row0, chunk[N];
    // (row, logical chunk) <-> physical chunk: an involution for a given row.  For a row of 256 bytes (all of the
    // banks) a read of one chunk of 16 rows wants 16 different permutations, and the transposing read of
    // TokenFrags, four chunks of four consecutive rows, wants these to differ in bits 2 and 3.
    static __device__ int swizzle(int row, int c)
    {
        return PITCH == kHd ? c ^ ((row & 3) << 2 | (row >> 2 & 3)) : c ^ ((row >> 1) & (CPR - 1));
    }
    __device__ void start(const uint16_t* first, int64_t ld, int wave, int lane)
    {
        tile = first;
        row0 = wave * N * RPP + lane / CPR;
#pragma unroll
        for (int i = 0; i < N; ++i) {
            const int row = row0 + i * RPP;
            chunk[i] = swizzle(row, lane % CPR);
            offset[i] = (std::conditional_t<FAR, uint64_t, uint32_t>)(2 * ((int64_t)row * ld + 8 * chunk[i]));
        }
    }
    // Requests the next tile, and moves on by `along` elements.  EDGE: its tokens start at token0, those at or
    // beyond limit read as zero (TOKEN_ROWS: a row is a token; otherwise a column is).
    template <bool EDGE, bool TOKEN_ROWS>
    __device__ void request(uint16_t* lds, int wave, int64_t along, int token0, int limit)
    {
#pragma unroll
        for (int i = 0; i < N; ++i) {
            uint16_t* dst = lds + (wave * N + i) * 512;
            if constexpr (EDGE || FAR) {
                const uint16_t* p = tile + offset[i] / 2;
                if (EDGE && token0 + (TOKEN_ROWS ? row0 + i * RPP : 8 * chunk[i]) >= limit) p = reinterpret_cast<const uint16_t*>(kZeros);
                load_to_lds(dst, p);
            } else {
                load_to_lds(dst, tile, offset[i]);
            }
        }
        tile += along;
    }
};
// LDS offsets of this lane's operand reads from a [tokens][kHd] tile of a TileStream.
// Contraction over hd: chunk 2 s + g of token ln; the tile's 32-token blocks are 32 * kHd apart.
struct RowFrags {
    int at;  // of s = 0; the chunk's permutation is an XOR, so that of s is another one
    __device__ void start(int lane)
    {
        const int row = lane & 31;
        at = row * kHd + 8 * TileStream<64, kHd, 8, false>::swizzle(row, lane >> 5);
    }
    __device__ uint4 read(const uint16_t* tile, int block32, int s) const
    {
        return *reinterpret_cast<const uint4*>(tile + 32 * kHd * block32 + (at ^ (16 * s)));
    }
    // Called once a step, it keeps the compiler from holding every s's offset in a register of its own.
    __device__ void renew() { asm volatile("" : "+v"(at)); }
};
// Contraction over tokens: the operand that matches slots(c, u), rows hd 32 d + ln, tokens 16 u + 4 g + {0..3} and
// 16 u + 8 + 4 g + {0..3}, by a transposing read each: within 16 lanes, lane i gets element i % 4 of the 8-byte pieces that lanes i / 4,
// 4 + i / 4, 8 + i / 4 and 12 + i / 4 point at.  So lane i points at token i / 4 (of four), hd 4 (i % 4).
struct TokenFrags {
    int at;  // of d = 0, first of the two reads
    __device__ void start(int lane)
    {
        const int g = lane >> 5, a = (lane >> 4) & 1, i = lane & 15;
        const int row = 4 * g + i / 4, col = 16 * a + 4 * (i % 4);
        at = row * kHd + 8 * TileStream<64, kHd, 8, false>::swizzle(row, col / 8) + col % 8;
    }
    __device__ void renew() { asm volatile("" : "+v"(at)); }
    __device__ uint4 read(const uint16_t* tile, int block16, int d) const
    {
        typedef short v4s __attribute__((ext_vector_type(4)));
        typedef __attribute__((address_space(3))) v4s* lds_v4s;
        const uint16_t* p = tile + 16 * kHd * block16;
        const uint2 lo = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p + (at ^ (32 * d)))));
        // eight tokens further down: the permutation of those rows differs in bit 1
        const uint2 hi = __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_v4s)(p + 8 * kHd + (at ^ (32 * d + 16)))));
        return make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
};
// whether a tile of `rows` rows of pitch ld needs FAR
static bool far_rows(int64_t rows, int64_t ld) { return 2 * (rows * ld + kHd) >= ((int64_t)1 << 32); }

// A wave's 32 rows x 128 results (row ln, columns 32 d + 8 j + 4 g + r in acc[d][4 j + r]) to `out` (its first row), rows before
// `rows` only.  From the registers a store would touch 32 rows with 8 bytes (16 in fp32) of each lane; through `stage`, 8 KB
// of LDS of the wave's own that nobody reads any more, 16 lanes cover 256 bytes of a row.  A row's chunks are permuted by its
// number: no bank conflicts.  The eight waves of a block end together, with nothing to hide the stores behind.  us of rope,
// attention and its backward, straight / so (sequences x tokens, query / key heads): 2 x 512, 8 / 8 82 / 77, 4 x 1000, 16 / 16
// 202.5 / 196.5, 2 x 2048, 32 / 8 461 / 451, 1 x 8192, 32 / 8 2436 / 2394.
__device__ inline void store_rows(const f32x16 (&acc)[kHd / 32], float mul, uint16_t* stage, uint16_t* out, int64_t ld, int rows, int lane)
{
    const int ln = lane & 31, g = lane >> 5;
#pragma unroll
    for (int d = 0; d < kHd / 32; ++d)
#pragma unroll
        for (int j = 0; j < 4; ++j)
            *reinterpret_cast<uint2*>(stage + ln * kHd + 8 * ((4 * d + j) ^ (ln & 15)) + 4 * g) =
                make_uint2(pack2(acc[d][4 * j] * mul, acc[d][4 * j + 1] * mul), pack2(acc[d][4 * j + 2] * mul, acc[d][4 * j + 3] * mul));
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = 4 * i + lane / 16, c = lane % 16;
        const uint4 v = *reinterpret_cast<const uint4*>(stage + row * kHd + 8 * (c ^ (row & 15)));
        if (row < rows) *reinterpret_cast<uint4*>(out + row * ld + 8 * c) = v;
    }
    asm volatile("" ::: "memory");
}
__device__ inline void store_rows(const f32x16 (&acc)[kHd / 32], float mul, uint16_t* stage, float* out, int64_t ld, int rows, int lane)
{
    const int ln = lane & 31, g = lane >> 5;
    float* st = reinterpret_cast<float*>(stage);
#pragma unroll
    for (int half = 0; half < 2; ++half) {  // 64 columns fit the stage
#pragma unroll
        for (int d = 0; d < 2; ++d)
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const f32x16& a = acc[2 * half + d];
                *reinterpret_cast<float4*>(st + ln * 64 + 4 * ((8 * d + 2 * j + g) ^ (ln & 15))) =
                    make_float4(a[4 * j] * mul, a[4 * j + 1] * mul, a[4 * j + 2] * mul, a[4 * j + 3] * mul);
            }
        asm volatile("" ::: "memory");
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const int row = 4 * i + lane / 16, c = lane % 16;
            const float4 v = *reinterpret_cast<const float4*>(st + row * 64 + 4 * (c ^ (row & 15)));
            if (row < rows) *reinterpret_cast<float4*>(out + row * ld + 64 * half + 4 * c) = v;
        }
        asm volatile("" ::: "memory");
    }
}

// The same straight from the registers: where one or two waves of the block have rows, little competes with their stores, and
// the barrier before the stage, the other waves' empty stores and the way through the stage are what they would wait for.
template <typename T>
__device__ inline void store_rows_straight(const f32x16 (&acc)[kHd / 32], float mul, T* out, int64_t ld, int rows, int lane)
{
    const int ln = lane & 31, g = lane >> 5;
    if (ln >= rows) return;
    T* row = out + ln * ld + 4 * g;
#pragma unroll
    for (int d = 0; d < kHd / 32; ++d)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float v0 = acc[d][4 * j] * mul, v1 = acc[d][4 * j + 1] * mul, v2 = acc[d][4 * j + 2] * mul, v3 = acc[d][4 * j + 3] * mul;
            if constexpr (sizeof(T) == 2) *reinterpret_cast<uint2*>(row + 32 * d + 8 * j) = make_uint2(pack2(v0, v1), pack2(v2, v3));
            else *reinterpret_cast<float4*>(row + 32 * d + 8 * j) = make_float4(v0, v1, v2, v3);
        }
}
// Sequences of at most so many tokens (bf16 gradients; fp32 shares) store their rows straight, in instances of their own: as a
// branch of the others it costs longer sequences 0.8 % (4 x 1000 tokens, 16 heads 80.2 -> 80.7 us).  us of the backward, through the
// stage / straight, 64 sequences, 32 / 32 heads: 16 tokens 110.2 / 102.9, 40 127.3 / 125.5, 48 131.0 / 132.3, 56 134.5 / 138.6, 64
// 142.8 / 149.3; 32 / 8 heads (dQ by the same line) 16 tokens 124.0 / 111.1, 48 158.3 / 152.8, 64 182.0 / 179.1.
constexpr int kStraightRows = 40, kStraightShares = 64;

// ---- forward ------------------------------------------------------------------------------
// One block: 8 waves of 32 queries each of one (sequence, head), loop over 64-key steps up to the
// diagonal.  Two waves share a SIMD, and they work in opposite phases: while waves 0 .. 3 feed the matrix
// pipe (phase M: S^T of the next step and P V of this one, 32 products), waves 4 .. 7 do the vector
// work of theirs (phase V: softmax of S^T, 32 exponentials per lane), then they change over.
//   time slot:            2t        2t + 1    2t + 2
//   waves 0 .. 3:         M_t       V_t       M_t+1         M_t: S_t+1 = K_t+1 Q, O += P_t V_t
//   waves 4 .. 7:         V_t-1     M_t       V_t           V_t: P_t+1 = softmax(S_t+1)
// with a barrier between slots; the second half enters one slot late.  M_t reads the tiles K_t+1 and V_t
// in slots 2t and 2t + 1.  K_t+3 and V_t+2 are requested at the end of V_t into the third of three buffers
// (what it held was read up to slot 2t - 1) and waited for at the end of the wave's next phase M.
// Measured (1 x 8192 tokens, 32/8 heads; cycles of a slot, both phases in it): M 1300 (32 products are 1024), V
// 1400 (softmax 1080 to 1300, the four loads the rest: a wave's load holds up its next instruction until the memory
// pipe of the compute unit takes it).  All waves in step instead, tiles through registers: 550 us; this: 497
// (1000 tokens, 4 heads: 33.2 and 29.6; 256 tokens: 13.4 and 13.0; 64 tokens, a single step: 5.7 and 6.2).
template <int NW, bool FAR>
__global__ __launch_bounds__(64 * NW, 512 / (64 * NW)) void sdpa_fwd_kernel(const uint16_t* __restrict__ Q, int64_t ldq,
                                                                const uint16_t* __restrict__ K, int64_t ldk,
                                                                const uint16_t* __restrict__ Vt, int64_t M, int S, int Hq,
                                                                int group, float scale_log2e, uint16_t* __restrict__ O,
                                                                int64_t ldo, float* __restrict__ lse, int nqt,
                                                                uint32_t* __restrict__ amax_bits /* nullable */)
{
    static_assert(NW == 8, "two waves per SIMD in opposite phases");
    constexpr int QB = 32 * NW;  // queries per block
    __shared__ __attribute__((aligned(1024))) uint16_t sK[3][kBk * kHd];
    __shared__ __attribute__((aligned(1024))) uint16_t sV[3][kHd * kBk];

    // long (late) query tiles first, over all heads: the tile index varies slowest
    const int nbh = Hq * (int)(M / S), qt = nqt - 1 - (int)(blockIdx.x / nbh);
    const int bh = blockIdx.x % nbh, h = bh % Hq, b = bh / Hq, kvh = h / group;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, ln = lane & 31, g = lane >> 5;
    const bool late = wave >= NW / 2;          // the half that runs one slot behind
    const int q_first = qt * QB + wave * 32;  // of this wave
    const int q_pos = q_first + ln;            // position of this lane's query in its sequence
    const int64_t tok0 = (int64_t)b * S;
    const uint16_t* Kb = K + tok0 * ldk + (int64_t)kvh * kHd;
    const uint16_t* Vb = Vt + (int64_t)kvh * kHd * M + tok0;

    uint4 qf[kHd / 16];
    {
        const bool ok = q_pos < S;
        const uint16_t* row = Q + (tok0 + (ok ? q_pos : 0)) * ldq + (int64_t)h * kHd + 8 * g;
#pragma unroll
        for (int s = 0; s < kHd / 16; ++s) qf[s] = ok ? *reinterpret_cast<const uint4*>(row + 16 * s) : make_uint4(0, 0, 0, 0);
    }

    int key_end = (qt + 1) * QB;  // keys at or beyond it are masked for every query of the block
    if (key_end > S) key_end = S;
    const int nkt = (key_end + kBk - 1) / kBk;
    const int t_last = min(nkt - 1, (q_first + 31) / kBk);  // the last step that this wave has any query for

    f32x16 acc_o[kHd / 32];
#pragma unroll
    for (int d = 0; d < kHd / 32; ++d) acc_o[d] = f32x16{0};
    float m_run = -INFINITY, l_run = 0.0f;  // running maximum of the raw scores and this lane's share of the sum
    f32x16 sc[2];                           // S^T of the next step: [64 keys][32 queries] as two 32x32 results
    uint4 pf[4];                            // P^T of this step as operands, [2 kb + u]

    using KStream = TileStream<kBk, kHd, NW, FAR>;
    using VStream = TileStream<kHd, kBk, NW, FAR>;
    KStream ks;
    VStream vs;
    ks.start(Kb, ldk, wave, lane);
    vs.start(Vb, M, wave, lane);
    // K_t and V_t live in buffer t % 3.  Requests V_t and K_t+1, buf = t % 3; EDGE: they may reach past S or
    // past the last step
    auto request = [&](auto EDGE, int t, int buf) {
        constexpr bool edge = decltype(EDGE)::value;
        if (!edge || t < nkt) vs.template request<edge, false>(sV[buf], wave, kBk, t * kBk, S);
        if (!edge || t + 1 < nkt) ks.template request<edge, true>(sK[buf == 2 ? 0 : buf + 1], wave, kBk * ldk, (t + 1) * kBk, S);
    };
    ks.template request<true, true>(sK[0], wave, kBk * ldk, 0, S);
    request(std::true_type{}, 0, 0);

    // Every wave runs the same number of slots, whatever it has left to do in them.  One without queries (the last
    // block of a short sequence) only loads its share of the tiles: scores of zero rows and their softmax held up the
    // waves that share its SIMD (8 tokens, 4 heads 6.1 us, so 5.6; 128 tokens 8.3, 8.05; without the skip 9.1).
    auto end_of_m = [&]() {
        stream_wait();  // for what this wave requested in its last phase V
        phase_barrier();
    };
    auto end_of_slots = [&]() {  // after it nothing reads the tiles any more
        if (!late) phase_barrier();
        phase_barrier();
    };
    auto next = [](int buf) { return buf == 2 ? 0 : buf + 1; };
    if (q_first >= S) {
        end_of_m();
        if (late) phase_barrier();
        for (int t = -1, buf = 1; t < nkt - 1; ++t, buf = next(buf)) {
            end_of_m();
            request(std::true_type{}, t + 2, buf);
            phase_barrier();
        }
        end_of_slots();
        return;
    }

    // LDS offsets of this lane's operand reads: of a key's row; of hd row ln, 4 g tokens into chunk 2 v, and (the
    // permutation is an XOR) the same of chunk 2 v + 1
    RowFrags k_rd;
    k_rd.start(lane);
    int v_rd[kBk / 16];
#pragma unroll
    for (int v = 0; v < kBk / 16; ++v) v_rd[v] = ln * kBk + 8 * VStream::swizzle(ln, 2 * v) + 4 * g;

    // products [LO, HI) of M_t: 0 .. 15 S^T = K Q^T (tile K_t+1), 16 .. 31 O^T += V^T P^T (tile V_t,
    // [128 hd][32 queries], contraction over the 64 keys in four 16-slot steps).  The matrix phase goes
    // before the other wave's vector work: its instructions are few, and the pipe idles without them.
    auto products = [&](int buf /* of V_t */, auto LO, auto HI) {
        constexpr int lo = decltype(LO)::value, hi = decltype(HI)::value;
        const uint16_t *tK = sK[buf == 2 ? 0 : buf + 1], *tV = sV[buf];
        if constexpr (lo == 0) sc[0] = f32x16{0}, sc[1] = f32x16{0};
        __builtin_amdgcn_s_setprio(1);
        pipelined_products<hi - lo, kFwdAhead, 16 - lo>(
            [&](int n) {
                const int i = n + lo;
                if (i < 16) return k_rd.read(tK, i % 2, i / 2 % 8);
                const uint16_t* v = tV + 32 * kBk * (i % 4);
                const uint2 a = *reinterpret_cast<const uint2*>(v + v_rd[i / 4 % 4]), b = *reinterpret_cast<const uint2*>(v + (v_rd[i / 4 % 4] ^ 8));
                return make_uint4(a.x, a.y, b.x, b.y);
            },
            [&](int n, uint4 f) {
                const int i = n + lo;
                if (i < 16) sc[i % 2] = mma(f, qf[i / 2 % 8], sc[i % 2]);
                else acc_o[i % 4] = mma(f, pf[(i - 16) / 4], acc_o[i % 4]);
            });
        __builtin_amdgcn_s_setprio(0);
    };
    using std::integral_constant;
    using C0 = integral_constant<int, 0>;
    using C16 = integral_constant<int, 16>;
    using C32 = integral_constant<int, 32>;

    // of step t.  MASKED: the step at the diagonal, a wave's last one (32 queries from a multiple of 32 on, 64
    // keys: it is the only one with anything to mask)
    auto softmax = [&](int t, auto MASKED) {
        const int key0 = t * kBk;
        // The maximum is taken over the raw scores (the scale is positive), so the scaling and the
        // subtraction of the maximum are one fused multiply-add per score.
        if constexpr (decltype(MASKED)::value) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int r = 0; r < 16; ++r) {
                    const int key = key0 + 32 * kb + reg_token(r, g);
                    if (key > q_pos) sc[kb][r] = -INFINITY;
                }
        }
        float mx[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
#pragma unroll
        for (int r = 0; r < 16; ++r) mx[r % 4] = fmaxf(fmaxf(mx[r % 4], sc[0][r]), sc[1][r]);
        const float m_here = fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3]));
        const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(m_here), __float_as_uint(m_here), false, false);
        const float m_new = fmaxf(__uint_as_float(both[0]), __uint_as_float(both[1]));  // of the query: the pair of lanes
        const float m_next = fmaxf(m_run, m_new);  // finite: key 0 is visible to every query
        const float alpha = __builtin_amdgcn_exp2f((m_run - m_next) * scale_log2e);
        m_run = m_next;
        l_run *= alpha;
        // (Following the maximum only when it has grown by 2^8 saves 4 % of the kernel, but puts the probabilities
        // on another rounding grid: 2e-3 of the output, which the fp8 casts of a whole block turn into 5e-2.)
        if (__builtin_amdgcn_ballot_w64(alpha != 1.0f)) {
#pragma unroll
            for (int d = 0; d < kHd / 32; ++d)
#pragma unroll
                for (int r = 0; r < 16; ++r) acc_o[d][r] *= alpha;
        }
        const float neg_m = -m_run * scale_log2e;
        float psum = 0.0f;
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[kb][r], scale_log2e, neg_m));
                sc[kb][r] = p;
                psum += p;
            }
            pf[2 * kb] = slots(sc[kb], 0), pf[2 * kb + 1] = slots(sc[kb], 1);
        }
        l_run += psum;
        for (int i = 0; i < 4; ++i) computed(pf[i]);
        computed(l_run);
    };

    int buf = 2, t = -1;  // buf = t % 3
    auto step = [&](auto EDGE) {
        end_of_m();
        softmax(t + 1, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
        request(EDGE, t + 2, buf == 0 ? 2 : buf - 1);
        phase_barrier();
        buf = next(buf);
        products(buf, C0{}, C32{});
        ++t;
    };
    end_of_m();
    if (late) phase_barrier();
    products(buf, C0{}, C16{});
    const int t_inside = min(t_last - 1, min(nkt, S / kBk) - 3);  // steps t before it request whole tiles only
    while (t < t_inside) step(std::false_type{});
    while (t < t_last - 1) step(std::true_type{});
    for (; t < nkt - 1; ++t) {
        end_of_m();
        if (t == t_last - 1) softmax(t_last, std::true_type{});
        request(std::true_type{}, t + 2, buf == 0 ? 2 : buf - 1);
        phase_barrier();
        buf = next(buf);
        if (t == t_last - 1) products(buf, C16{}, C32{});
    }
    end_of_slots();

    // O: a lane has 16 pieces of 8 bytes of one row.  Stored from here they would touch 32 rows per instruction, and all
    // eight waves get here together, with nothing to hide the stores behind (7500 cycles: 2 us of every block, 256 tokens
    // 15.3 us); so they go through the LDS, which nothing reads any more, to 16-byte pieces of which 16 lanes cover a
    // row (13.0 us; a row's chunks are permuted by its number: no bank conflicts).
    const float l_tot = l_run + __shfl_xor(l_run, 32, kWave);
    uint32_t mag = 0;  // packed pair of the largest 15-bit magnitudes written
    uint16_t* stage = (wave < NW / 2 ? sK[0] : sV[0]) + (wave % (NW / 2)) * 32 * kHd;  // this wave's 32 rows
    const float inv = 1.0f / l_tot;
#pragma unroll
    for (int d = 0; d < kHd / 32; ++d)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint2 w = make_uint2(pack2(acc_o[d][4 * j] * inv, acc_o[d][4 * j + 1] * inv),
                                       pack2(acc_o[d][4 * j + 2] * inv, acc_o[d][4 * j + 3] * inv));
            *reinterpret_cast<uint2*>(stage + ln * kHd + 8 * ((4 * d + j) ^ (ln & 15)) + 4 * g) = w;
            if (q_pos < S) mag = pkmax(pkmax(mag, w.x & 0x7FFF7FFFu), w.y & 0x7FFF7FFFu);
        }
    if (q_pos < S && g == 0) lse[(int64_t)h * M + tok0 + q_pos] = (m_run * scale_log2e + __builtin_amdgcn_logf(l_tot)) * 0.69314718055994530942f;
    asm volatile("" ::: "memory");
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int row = 4 * i + lane / 16, c = lane % 16;
        const uint4 v = *reinterpret_cast<const uint4*>(stage + row * kHd + 8 * (c ^ (row & 15)));
        if (q_first + row < S) *reinterpret_cast<uint4*>(O + (tok0 + q_first + row) * ldo + (int64_t)h * kHd + 8 * c) = v;
    }
    if (amax_bits) {
        // the exact maximum magnitude of the bf16 values written, as float bits: a maximum of
        // non-negative floats is a maximum of their bit patterns, and does not depend on the order
        const uint32_t m = wave_max_u32(pk_collapse(mag)) << 16;
        if (lane == 0 && m > __atomic_load_n(amax_bits, __ATOMIC_RELAXED)) atomicMax(amax_bits, m);
    }
}

__global__ void zero_amax_kernel(uint32_t* p) { p[0] = 0; }

// ---- backward -----------------------------------------------------------------------------
// With P = exp(S / sqrt(hd) - lse) recomputed from the saved lse and delta[q] = sum_d dO O:
//   dV = P^T dO,  dP = dO V^T,  dS = P (dP - delta),  dQ = dS K / sqrt(hd),  dK = dS^T Q / sqrt(hd)
// Two kernels, neither with atomics: dQ per query tile (loop over keys, S^T orientation, which
// also produces delta), then dK and dV per key tile and query head (loop over queries, S
// orientation: one key per lane); with grouped heads the shares of a group's query heads are
// kept in fp32 and summed in head order by a small third kernel.  Where a launch of either is few blocks, both
// run in one (sdpa_bwd_kernel).

// two of the products of delta
__device__ inline float delta_term(uint32_t d, uint32_t o) { return bf16_lo(d) * bf16_lo(o) + bf16_hi(d) * bf16_hi(o); }

// dQ^T = K^T dS^T.  In two staggered halves like the forward (see there), per 64-key step:
//   M_t: dQ += K_t^T dS_t (16 products), then S^T = K_t+1 Q^T and dP^T = V_t+1 dO^T (32 products)
//   V_t: dS_t+1 = P (dP - delta)
// Tiles t live in buffer t % 4: M_t reads K_t, K_t+1 and V_t+1; K_t+3 and V_t+3 are requested at the end of V_t.
// K^T comes from the K tile itself, by transposing reads.  (All waves in step, three tiles through registers: 821 us for
// 1 x 8192 tokens, 32/8 heads; this: 700.  Phase M is what it waits for: 48 products, 1536 cycles, in about 1900.)
// The work of one block: query tile qt of (sequence, head) bh.  DELTA: delta is formed and stored here, else it is read.
// STRAIGHT: see store_rows_straight.
struct DqArgs {
    const uint16_t *Q, *K, *V, *O, *dO;
    int64_t ldq, ldk, ldv, ldo, lddo;
    const float* lse;
    int64_t M;
    int S, Hq, group;
    float scale_log2e, scale;
    uint16_t* dQ;
    int64_t lddq;
    float* delta;
};
template <int NW, bool FAR, bool DELTA, bool STRAIGHT>
__device__ __forceinline__ void sdpa_bwd_dq_work(const DqArgs& P, int qt, int bh, uint16_t (&sK)[4][kBk * kHd], uint16_t (&sV)[4][kBk * kHd])
{
    static_assert(NW == 8, "two waves per SIMD in opposite phases");
    constexpr int QB = 32 * NW;  // queries per block
    const uint16_t *__restrict__ Q = P.Q, *__restrict__ K = P.K, *__restrict__ V = P.V, *__restrict__ O = P.O, *__restrict__ dO = P.dO;
    const int64_t ldq = P.ldq, ldk = P.ldk, ldv = P.ldv, ldo = P.ldo, lddo = P.lddo, M = P.M, lddq = P.lddq;
    const float* __restrict__ lse = P.lse;
    const int S = P.S, Hq = P.Hq, group = P.group;
    const float scale_log2e = P.scale_log2e, scale = P.scale;
    uint16_t* __restrict__ dQ = P.dQ;
    float* __restrict__ delta = P.delta;

    const int h = bh % Hq, b = bh / Hq, kvh = h / group;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, ln = lane & 31, g = lane >> 5;
    const bool late = wave >= NW / 2;
    const int q_first = qt * QB + wave * 32, q_pos = q_first + ln;
    const int64_t tok0 = (int64_t)b * S;
    const bool q_ok = q_pos < S;
    const int64_t tok = tok0 + (q_ok ? q_pos : 0);

    int key_end = (qt + 1) * QB;
    if (key_end > S) key_end = S;
    const int nkt = (key_end + kBk - 1) / kBk;
    const int t_last = min(nkt - 1, (q_first + 31) / kBk);

    using Stream = TileStream<kBk, kHd, NW, FAR>;
    Stream ks, vs;
    ks.start(K + tok0 * ldk + (int64_t)kvh * kHd, ldk, wave, lane);
    vs.start(V + tok0 * ldv + (int64_t)kvh * kHd, ldv, wave, lane);
    auto request = [&](auto EDGE, int t) {  // tiles t
        constexpr bool edge = decltype(EDGE)::value;
        if (edge && t >= nkt) return;
        ks.template request<edge, true>(sK[t & 3], wave, kBk * ldk, t * kBk, S);
        vs.template request<edge, true>(sV[t & 3], wave, kBk * ldv, t * kBk, S);
    };
    request(std::true_type{}, 0);
    request(std::true_type{}, 1);

    uint4 qf[kHd / 16], dof[kHd / 16];
    float dl = 0.0f;
    {
        const uint16_t* qrow = Q + tok * ldq + (int64_t)h * kHd + 8 * g;
        const uint16_t* drow = dO + tok * lddo + (int64_t)h * kHd + 8 * g;
        const uint16_t* orow = O + tok * ldo + (int64_t)h * kHd + 8 * g;
#pragma unroll
        for (int s = 0; s < kHd / 16; ++s) {
            qf[s] = q_ok ? *reinterpret_cast<const uint4*>(qrow + 16 * s) : make_uint4(0, 0, 0, 0);
            dof[s] = q_ok ? *reinterpret_cast<const uint4*>(drow + 16 * s) : make_uint4(0, 0, 0, 0);
            if constexpr (DELTA) {
                const uint4 ov = q_ok ? *reinterpret_cast<const uint4*>(orow + 16 * s) : make_uint4(0, 0, 0, 0);
                const uint32_t dw[4] = {dof[s].x, dof[s].y, dof[s].z, dof[s].w}, ow[4] = {ov.x, ov.y, ov.z, ov.w};
#pragma unroll
                for (int j = 0; j < 4; ++j) dl += delta_term(dw[j], ow[j]);
            }
        }
    }
    if constexpr (DELTA) {
        dl += __shfl_xor(dl, 32, kWave);
        if (q_ok && g == 0) delta[(int64_t)h * M + tok] = dl;
    } else {
        dl = q_ok ? delta[(int64_t)h * M + tok] : 0.0f;
    }
    const float lse2 = q_ok ? lse[(int64_t)h * M + tok] * 1.4426950408889634074f : 0.0f;

    f32x16 acc[kHd / 32], sc[2], dp[2];
    uint4 ds[4];  // dS^T of this step as operands, one per 16 keys
#pragma unroll
    for (int d = 0; d < kHd / 32; ++d) acc[d] = f32x16{0};
    RowFrags row_rd;
    TokenFrags tok_rd;
    row_rd.start(lane);
    tok_rd.start(lane);

    // products [LO, HI) of M_t: 0 .. 15 dQ^T += K_t^T dS_t^T, 16 .. 47 S^T and dP^T of step t + 1.  The first operands
    // (of K_t, which landed a step ago) are read at the end of phase V.
    constexpr int STARTED = 2;  // (four do not fit the registers)
    uint4 started[STARTED];
    auto start_products = [&](int t) {
        tok_rd.renew();
#pragma unroll
        for (int i = 0; i < STARTED; ++i) started[i] = tok_rd.read(sK[t & 3], i / 4, i % 4);
    };
    auto score_operand = [&](int t, int i) { return row_rd.read(i & 1 ? sV[t & 3] : sK[t & 3], (i >> 1) & 1, i / 4); };
    auto score_product = [&](int i, uint4 f) {
        const int kb = (i >> 1) & 1;
        if (i & 1) dp[kb] = mma(f, dof[i / 4], dp[kb]);
        else sc[kb] = mma(f, qf[i / 4], sc[kb]);
    };
    auto products = [&](int t, auto HI) {
        constexpr int hi = decltype(HI)::value;
        row_rd.renew();
        if constexpr (hi > 16) sc[0] = sc[1] = dp[0] = dp[1] = f32x16{0};
        __builtin_amdgcn_s_setprio(1);
        started_products<hi, kDqAhead>(
            started, [&](int i) { return i < 16 ? tok_rd.read(sK[t & 3], i / 4, i % 4) : score_operand(t + 1, i - 16); },
            [&](int i, uint4 f) {
                if (i < 16) acc[i % 4] = mma(f, ds[i / 4], acc[i % 4]);
                else score_product(i - 16, f);
            },
            [](int i) { return i < 16; });
        __builtin_amdgcn_s_setprio(0);
    };
    using C16 = std::integral_constant<int, 16>;
    using C48 = std::integral_constant<int, 48>;
    auto grad_scores = [&](int t, auto MASKED) {
#pragma unroll
        for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                float p = __builtin_amdgcn_exp2f(sc[kb][r] * scale_log2e - lse2);
                if constexpr (decltype(MASKED)::value) {
                    if (t * kBk + 32 * kb + reg_token(r, g) > q_pos) p = 0.0f;
                }
                sc[kb][r] = p * (dp[kb][r] - dl);
            }
            ds[2 * kb] = slots(sc[kb], 0), ds[2 * kb + 1] = slots(sc[kb], 1);
        }
        for (int i = 0; i < 4; ++i) computed(ds[i]);
    };

    int t = -1;
    auto end_of_m = [&]() {
        stream_wait();
        phase_barrier();
    };
    auto step = [&](auto EDGE) {
        end_of_m();
        grad_scores(t + 1, std::false_type{});
        __builtin_amdgcn_sched_barrier(0);
        request(EDGE, t + 3);
        start_products(++t);
        phase_barrier();
        products(t, C48{});
    };
    stream_wait();
    phase_barrier();
    if (late) phase_barrier();
    sc[0] = sc[1] = dp[0] = dp[1] = f32x16{0};
    pipelined_products<32, kDqAhead>([&](int i) { return score_operand(0, i); }, score_product);
    const int t_inside = min(t_last - 1, min(nkt, S / kBk) - 3);
    while (t < t_inside) step(std::false_type{});
    while (t < t_last - 1) step(std::true_type{});
    for (; t < nkt; ++t) {
        end_of_m();
        if (t == t_last - 1) {
            grad_scores(t_last, std::true_type{});
            start_products(t_last);
        }
        request(std::true_type{}, t + 3);
        phase_barrier();
        if (t == t_last - 1) products(t_last, C16{});
    }
    if (!late) phase_barrier();
    if constexpr (!STRAIGHT) phase_barrier();  // after it nothing reads the tiles any more
    if (STRAIGHT && q_first >= S) return;      // (not STRAIGHT: 1 % of 1 x 2048 tokens)
    int l64 = threadIdx.x & 63;  // (formed anew: what the stores are addressed by would be held over the loop)
    asm volatile("" : "+v"(l64));
    uint16_t* out = dQ + (tok0 + q_first) * lddq + (int64_t)h * kHd;
    if constexpr (STRAIGHT) store_rows_straight(acc, scale, out, lddq, S - q_first, l64);
    else store_rows(acc, scale, &sK[0][0] + wave * 32 * kHd, out, lddq, S - q_first, l64);
}

template <int NW, bool FAR, bool STRAIGHT = false>
__global__ __launch_bounds__(64 * NW, 512 / (64 * NW)) void sdpa_bwd_dq_kernel(const DqArgs P, int nqt)
{
    __shared__ __attribute__((aligned(1024))) uint16_t sK[4][kBk * kHd];
    __shared__ __attribute__((aligned(1024))) uint16_t sV[4][kBk * kHd];
    // long (late) query tiles first, over all heads
    const int nbh = P.Hq * (int)(P.M / P.S), qt = nqt - 1 - (int)(blockIdx.x / nbh);
    sdpa_bwd_dq_work<NW, FAR, true, STRAIGHT>(P, qt, blockIdx.x % nbh, sK, sV);
}

// dV^T = dO^T P and dK^T = Q^T dS in one pass over the scores.  One block: 8 waves, 32 keys each (one key per lane),
// of one (sequence, query head); steps of 32 queries, in pairs from the end of the sequence down to the diagonal (the
// lower half of a pair first), in two staggered halves like the forward (see there):
//   M_t: dV += dO_t^T P_t, dK += Q_t^T dS_t (8 products each), then S = Q_t+1 K^T, dP = dO_t+1 V^T (8 each)
//   V_t: P_t+1 = exp(S - lse), dS_t+1 = P (dP - delta)
// Tiles t (Q, dO and their lse, delta) live in buffer t % 4; those of step t + 3 are requested at the end of V_t.
// Q^T and dO^T come from the same tiles by transposing reads.  The two accumulators (128 registers), the K
// operand (32), scores and operands leave no room for the V operand: the block's 256 rows of V stay in LDS.
// (dK and dV in a kernel each, 40 products a step instead of 32 and the exponentials twice, all waves in step: 1490 us for
// 1 x 8192 tokens, 32/8 heads; this: 1010.)
constexpr int kDkvQ = 32;  // queries per step
struct DkvArgs {
    const uint16_t *Q, *K, *V, *dO;
    int64_t ldq, ldk, ldv, lddo;
    const float *lse, *delta;
    int64_t M;
    int S, Hq, group;
    float scale_log2e, scale;
    uint16_t *dK, *dV;
    int64_t lddk, lddv;
    float *part_k, *part_v;
};
template <int NW>
struct DkvLds {
    uint16_t sQ[4][kDkvQ * kHd], sD[4][kDkvQ * kHd], sV[32 * NW * kHd];
    float sStat[4][2 * kDkvQ];  // lse, then delta
};
// The work of one block: key tile kt of (sequence, query head) bh.
template <int NW, bool FAR, bool STRAIGHT>
__device__ __forceinline__ void sdpa_bwd_dkv_work(const DkvArgs& P, int kt, int bh, uint16_t (&sQ)[4][kDkvQ * kHd], uint16_t (&sD)[4][kDkvQ * kHd],
                                                  uint16_t (&sV)[32 * NW * kHd], float (&sStat)[4][2 * kDkvQ])
{
    static_assert(NW == 8, "two waves per SIMD in opposite phases");
    constexpr int KB = 32 * NW;  // keys per block
    const uint16_t *__restrict__ Q = P.Q, *__restrict__ K = P.K, *__restrict__ V = P.V, *__restrict__ dO = P.dO;
    const int64_t ldq = P.ldq, ldk = P.ldk, ldv = P.ldv, lddo = P.lddo, M = P.M, lddk = P.lddk, lddv = P.lddv;
    const float *__restrict__ lse = P.lse, *__restrict__ delta = P.delta;
    const int S = P.S, Hq = P.Hq, group = P.group;
    const float scale_log2e = P.scale_log2e, scale = P.scale;
    uint16_t *__restrict__ dK = P.dK, *__restrict__ dV = P.dV;
    float *__restrict__ part_k = P.part_k, *__restrict__ part_v = P.part_v;

    const int hq = bh % Hq, b = bh / Hq, kvh = hq / group, gi = hq % group;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, ln = lane & 31, g = lane >> 5;
    const bool late = wave >= NW / 2;
    const int key_first = kt * KB + wave * 32, key_pos = key_first + ln;
    const int64_t tok0 = (int64_t)b * S;
    const bool k_ok = key_pos < S;
    const int64_t tok = tok0 + (k_ok ? key_pos : 0);

    const int q_start = kt * KB;
    const int pairs = (S - q_start + 2 * kDkvQ - 1) / (2 * kDkvQ);  // >= 1: the block exists only if q_start < S
    const int steps = 2 * pairs;
    const int t_last = 2 * max(0, pairs - 1 - wave / 2) + 1;  // the pair of steps t_last - 1, t_last holds this wave's diagonal
    auto q0 = [&](int t) { return q_start + (pairs - 1 - t / 2) * (2 * kDkvQ) + (t & 1) * kDkvQ; };  // step t: queries q0(t) ..

    using Stream = TileStream<kDkvQ, kHd, NW, FAR>;
    Stream qs, os;
    qs.start(Q + (tok0 + q0(0)) * ldq + (int64_t)hq * kHd, ldq, wave, lane);
    os.start(dO + (tok0 + q0(0)) * lddo + (int64_t)hq * kHd, lddo, wave, lane);
    const float *lse_b = lse + (int64_t)hq * M + tok0, *delta_b = delta + (int64_t)hq * M + tok0;
    auto request = [&](auto EDGE, int t) {  // in order.  EDGE: may lie past the last step, or (the first pair) past S
        constexpr bool edge = decltype(EDGE)::value;
        if (edge && t >= steps) return;
        const int buf = t & 3;
        const int on = (t & 1) ? -3 * kDkvQ : kDkvQ;  // rows to the next step's tile
        qs.template request<edge, true>(sQ[buf], wave, on * ldq, q0(t), S);
        os.template request<edge, true>(sD[buf], wave, on * lddo, q0(t), S);
        if (wave == NW - 1) {
            int l64 = threadIdx.x;  // (formed anew: held over the loop, the pointer costs registers that are not there)
            asm volatile("" : "+v"(l64));
            const int q = q0(t) + (l64 & 31);
            const float* p = ((l64 & 32) ? delta_b : lse_b) + q;
            if (edge && q >= S) p = reinterpret_cast<const float*>(kZeros);
            const uint32_t l = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float*)sStat[buf];
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dword %1, off" : : "s"(l), "v"(p) : "memory");
        }
    };
    {
        TileStream<KB, kHd, NW, FAR> vs;
        vs.start(V + (tok0 + q_start) * ldv + (int64_t)kvh * kHd, ldv, wave, lane);
        vs.template request<true, true>(sV, wave, 0, q_start, S);
    }
    request(std::true_type{}, 0);
    request(std::true_type{}, 1);

    uint4 kf[kHd / 16];
    {
        const uint16_t* krow = K + tok * ldk + (int64_t)kvh * kHd + 8 * g;
#pragma unroll
        for (int s = 0; s < kHd / 16; ++s) kf[s] = k_ok ? *reinterpret_cast<const uint4*>(krow + 16 * s) : make_uint4(0, 0, 0, 0);
    }
    f32x16 acc_k[kHd / 32], acc_v[kHd / 32], sc, dp;
    uint4 pf[2], ds[2];  // P and dS of this step as operands, one per 16 queries
#pragma unroll
    for (int d = 0; d < kHd / 32; ++d) acc_k[d] = acc_v[d] = f32x16{0};
    RowFrags row_rd;
    TokenFrags tok_rd;
    row_rd.start(lane);
    tok_rd.start(lane);
    int v_at = (32 * wave + ln) * kHd + 8 * Stream::swizzle(ln, g);  // chunk 2 s + g of this lane's key: s enters as an XOR

    struct Operands {
        uint4 first, second;
    };
    // products of M_t: 0 .. 7 dV, 8 .. 15 dK, 16 .. 31 S and dP of step t + 1
    auto score_operands = [&](int t, int j) {
        const int s = j / 2;
        if (j & 1) return Operands{row_rd.read(sD[t & 3], 0, s), *reinterpret_cast<const uint4*>(sV + (v_at ^ (16 * s)))};
        return Operands{row_rd.read(sQ[t & 3], 0, s), kf[s]};
    };
    auto score_product = [&](int j, const Operands& f) {
        if (j & 1) dp = mma(f.first, f.second, dp);
        else sc = mma(f.first, f.second, sc);
    };
    auto grad_operands = [&](int t, int i) {
        return Operands{tok_rd.read(i < 8 ? sD[t & 3] : sQ[t & 3], (i / 4) % 2, i % 4), i < 8 ? pf[(i / 4) % 2] : ds[(i / 4) % 2]};
    };
    constexpr int STARTED = 1;  // (two, and four operands ahead, were no faster)
    Operands started[STARTED];  // read at the end of phase V: these tiles landed a step ago
    auto start_products = [&](int t) {
        tok_rd.renew();
#pragma unroll
        for (int i = 0; i < STARTED; ++i) started[i] = grad_operands(t, i);
    };
    auto products = [&](int t, auto HI) {
        constexpr int hi = decltype(HI)::value;
        row_rd.renew();
        asm volatile("" : "+v"(v_at));
        if constexpr (hi > 16) sc = dp = f32x16{0};
        __builtin_amdgcn_s_setprio(1);
        started_products<hi, kDkvAhead>(
            started, [&](int i) { return i < 16 ? grad_operands(t, i) : score_operands(t + 1, i - 16); },
            [&](int i, const Operands& f) {
                if (i < 8) acc_v[i % 4] = mma(f.first, f.second, acc_v[i % 4]);
                else if (i < 16) acc_k[i % 4] = mma(f.first, f.second, acc_k[i % 4]);
                else score_product(i - 16, f);
            },
            [](int i) { return i < 16 || (i & 1); });
        __builtin_amdgcn_s_setprio(0);
    };
    using C16 = std::integral_constant<int, 16>;
    using C32 = std::integral_constant<int, 32>;
    // MASKED: the diagonal's pair, and the first one if it reaches past S (its queries there are zero rows with
    // lse = delta = 0, but their P is 1, or not a number for a key that is not finite).
    auto grad_scores = [&](int t, auto MASKED) {
        const float* st = sStat[t & 3];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            float ds8[8];
#pragma unroll
            for (int j = 0; j < 2; ++j) {
                const int ql = reg_token(8 * u + 4 * j, g);
                const float4 l4 = *reinterpret_cast<const float4*>(st + ql), d4 = *reinterpret_cast<const float4*>(st + kDkvQ + ql);
                const float lv[4] = {l4.x, l4.y, l4.z, l4.w}, dv[4] = {d4.x, d4.y, d4.z, d4.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const int r = 8 * u + 4 * j + i;
                    float p = __builtin_amdgcn_exp2f(sc[r] * scale_log2e - lv[i] * 1.4426950408889634074f);
                    if constexpr (decltype(MASKED)::value) {
                        // queries key_pos .. S - 1 (a key at or past S is not stored, whatever it gets)
                        if ((unsigned)(q0(t) + ql + i - key_pos) >= (unsigned)(S - key_pos)) p = 0.0f;
                    }
                    sc[r] = p;
                    ds8[4 * j + i] = p * (dp[r] - dv[i]);
                }
            }
            pf[u] = slots(sc, u);
            ds[u] = make_uint4(pack2(ds8[0], ds8[1]), pack2(ds8[2], ds8[3]), pack2(ds8[4], ds8[5]), pack2(ds8[6], ds8[7]));
        }
        for (int u = 0; u < 2; ++u) computed(pf[u]), computed(ds[u]);
    };

    int t = -1;
    auto end_of_m = [&]() {
        stream_wait();
        phase_barrier();
    };
    auto step = [&](auto EDGE, auto MASKED) {
        end_of_m();
        grad_scores(t + 1, MASKED);
        __builtin_amdgcn_sched_barrier(0);
        request(EDGE, t + 3);
        start_products(++t);
        phase_barrier();
        products(t, C32{});
    };
    stream_wait();
    phase_barrier();
    if (late) phase_barrier();
    sc = dp = f32x16{0};
#pragma unroll
    for (int j = 0; j < 16; ++j) score_product(j, score_operands(0, j));
    const int t_inside = min(t_last - 2, steps - 3);
    const int t_whole = S % (2 * kDkvQ) ? 1 : -1;  // from this t on step(t) forms scores of whole pairs
    do {
        if (t >= t_whole) {
            while (t < t_inside) step(std::false_type{}, std::false_type{});
            while (t < t_last - 2) step(std::true_type{}, std::false_type{});
        }
        step(std::true_type{}, std::true_type{});  // scores of the first pair, or of t_last - 1
    } while (t < t_last - 1);
    for (; t < steps; ++t) {
        end_of_m();
        if (t == t_last - 1) {
            grad_scores(t_last, std::true_type{});
            start_products(t_last);
        }
        request(std::true_type{}, t + 3);
        phase_barrier();
        if (t == t_last - 1) products(t_last, C16{});
    }
    if (!late) phase_barrier();
    if constexpr (!STRAIGHT) phase_barrier();  // after it nothing reads the tiles any more
    const int rows = S - key_first;
    if (STRAIGHT && rows <= 0) return;
    uint16_t* stage = sV + wave * 32 * kHd;
    int l64 = threadIdx.x & 63;  // (formed anew: what the stores are addressed by would be held over the loop)
    asm volatile("" : "+v"(l64));
    auto store = [&](const f32x16(&acc)[kHd / 32], float mul, auto* out, int64_t ld) {
        if constexpr (STRAIGHT) store_rows_straight(acc, mul, out, ld, rows, l64);
        else store_rows(acc, mul, stage, out, ld, rows, l64);
    };
    if (group == 1) {
        const int64_t first = tok0 + key_first, col = (int64_t)kvh * kHd;
        store(acc_k, scale, dK + first * lddk + col, lddk);
        store(acc_v, 1.0f, dV + first * lddv + col, lddv);
    } else {
        // this query head's share, fp32: [group][token][Hkv * hd]; summed in a fixed order afterwards
        const int64_t w = (int64_t)(Hq / group) * kHd, at = ((int64_t)gi * M + tok0 + key_first) * w + (int64_t)kvh * kHd;
        store(acc_k, scale, part_k + at, w);
        store(acc_v, 1.0f, part_v + at, w);
    }
}

template <int NW, bool FAR, bool STRAIGHT = false>
__global__ __launch_bounds__(64 * NW, 512 / (64 * NW)) void sdpa_bwd_dkv_kernel(const DkvArgs P)
{
    __shared__ __attribute__((aligned(1024))) uint16_t sQ[4][kDkvQ * kHd];
    __shared__ __attribute__((aligned(1024))) uint16_t sD[4][kDkvQ * kHd];
    __shared__ __attribute__((aligned(1024))) uint16_t sV[32 * NW * kHd];
    __shared__ __attribute__((aligned(1024))) float sStat[4][2 * kDkvQ];  // lse, then delta
    // early key tiles see the most queries: they are the slowest-varying index, so they start first
    const int nbh = P.Hq * (int)(P.M / P.S);
    sdpa_bwd_dkv_work<NW, FAR, STRAIGHT>(P, blockIdx.x / nbh, blockIdx.x % nbh, sQ, sD, sV, sStat);
}

// delta[h][token] = sum of dO O over the head, in the order of sdpa_bwd_dq_work (chunk 2 s + g of a row to lane group g,
// s ascending, then g 0 and 1): for the kernel below, whose dK/dV blocks cannot wait for its dQ blocks.  One block: 128
// rows (token, head).  The products' pair sums are formed by coalesced loads and chained through LDS.
constexpr int kDeltaRows = kAttnThreads / 2;
__global__ __launch_bounds__(kAttnThreads) void sdpa_delta_kernel(const uint16_t* __restrict__ O, int64_t ldo, const uint16_t* __restrict__ dO,
                                                                  int64_t lddo, int64_t M, int Hq, float* __restrict__ delta)
{
    constexpr int CPR = kHd / 8, PER_THREAD = kDeltaRows * CPR / kAttnThreads;
    __shared__ float4 terms[kDeltaRows][CPR + 1];  // (a padded row: the chains read one column of all rows)
    const int64_t row0 = (int64_t)blockIdx.x * kDeltaRows, rows = M * Hq;
    uint4 o[PER_THREAD], d[PER_THREAD];
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i) {
        const int rl = (i * kAttnThreads + (int)threadIdx.x) / CPR, c = threadIdx.x % CPR;
        const int64_t row = row0 + rl < rows ? row0 + rl : rows - 1, tok = row / Hq, col = row % Hq * kHd + 8 * c;
        o[i] = *reinterpret_cast<const uint4*>(O + tok * ldo + col), d[i] = *reinterpret_cast<const uint4*>(dO + tok * lddo + col);
    }
#pragma unroll
    for (int i = 0; i < PER_THREAD; ++i)
        terms[(i * kAttnThreads + (int)threadIdx.x) / CPR][threadIdx.x % CPR] =
            make_float4(delta_term(d[i].x, o[i].x), delta_term(d[i].y, o[i].y), delta_term(d[i].z, o[i].z), delta_term(d[i].w, o[i].w));
    __syncthreads();
    const int rl = threadIdx.x / 2, g = threadIdx.x % 2;
    float dl = 0.0f;
#pragma unroll
    for (int s = 0; s < CPR / 2; ++s) {
        const float4 t = terms[rl][2 * s + g];
        dl += t.x, dl += t.y, dl += t.z, dl += t.w;
    }
    dl += __shfl_xor(dl, 1, kWave);
    const int64_t row = row0 + rl;
    if (g == 0 && row < rows) delta[row % Hq * M + row / Hq] = dl;
}

// dQ and dK/dV in one launch, the blocks of both, longest first (a dK/dV block takes 1.35 times as long as a dQ block of
// as many tiles), delta beforehand.  A launch of at most one block per compute unit lasts as long as its longest block, and
// the units of the shorter ones idle: here the other kernel's blocks fill them (4 x 1000 tokens, 16 heads: 48 + 64 us in two
// launches; this 90 and delta 7).  Same device code, same bits.
template <int NW, bool STRAIGHT>
__global__ __launch_bounds__(64 * NW, 512 / (64 * NW)) void sdpa_bwd_kernel(const DqArgs Pq, const DkvArgs Pk, int tiles)
{
    constexpr size_t kDq = 2 * sizeof(uint16_t[4][kBk * kHd]), kDkv = sizeof(DkvLds<NW>);
    __shared__ __attribute__((aligned(1024))) uint8_t lds[kDq > kDkv ? kDq : kDkv];
    const int nbh = Pq.Hq * (int)(Pq.M / Pq.S), k = blockIdx.x / nbh, bh = blockIdx.x % nbh;
    if (k & 1) {
        auto* s = reinterpret_cast<uint16_t(*)[4][kBk * kHd]>(lds);
        sdpa_bwd_dq_work<NW, false, false, STRAIGHT>(Pq, tiles - 1 - k / 2, bh, s[0], s[1]);
    } else {
        auto* s = reinterpret_cast<DkvLds<NW>*>(lds);
        sdpa_bwd_dkv_work<NW, false, STRAIGHT>(Pk, k / 2, bh, s->sQ, s->sD, s->sV, s->sStat);
    }
}

// out[tok][c] = bf16(sum over the group's query heads, in order, of part[gi][tok][c]); 8 columns per thread
__global__ __launch_bounds__(kAttnThreads) void sdpa_group_sum_kernel(const float* __restrict__ part_k, const float* __restrict__ part_v,
                                                                      int64_t M, int64_t w, int group,
                                                                      uint16_t* __restrict__ dK, int64_t lddk,
                                                                      uint16_t* __restrict__ dV, int64_t lddv,
                                                                      uint32_t* __restrict__ amax_dv_bits /* nullable: max-updated */)
{
    uint32_t mag = 0;
    const int64_t chunks = M * (w / 8);
    for (int64_t c = (int64_t)blockIdx.x * kAttnThreads + threadIdx.x; c < 2 * chunks; c += (int64_t)gridDim.x * kAttnThreads) {
        const bool is_v = c >= chunks;
        const int64_t cc = is_v ? c - chunks : c, tok = cc / (w / 8), col = (cc % (w / 8)) * 8;
        const float* src = (is_v ? part_v : part_k) + tok * w + col;
        float4 a = *reinterpret_cast<const float4*>(src), b2 = *reinterpret_cast<const float4*>(src + 4);
        for (int gi = 1; gi < group; ++gi) {
            const float4 x = *reinterpret_cast<const float4*>(src + (int64_t)gi * M * w);
            const float4 y = *reinterpret_cast<const float4*>(src + (int64_t)gi * M * w + 4);
            a.x += x.x, a.y += x.y, a.z += x.z, a.w += x.w;
            b2.x += y.x, b2.y += y.y, b2.z += y.z, b2.w += y.w;
        }
        uint16_t* dst = is_v ? dV + tok * lddv + col : dK + tok * lddk + col;
        const uint4 o = make_uint4(pack2(a.x, a.y), pack2(a.z, a.w), pack2(b2.x, b2.y), pack2(b2.z, b2.w));
        *reinterpret_cast<uint4*>(dst) = o;
        if (is_v) mag = absmax_acc(mag, o);
    }
    if (amax_dv_bits) {
        const uint32_t m = wave_max_u32(pk_collapse(mag)) << 16;
        if ((threadIdx.x & (kWave - 1)) == 0 && m > __atomic_load_n(amax_dv_bits, __ATOMIC_RELAXED)) atomicMax(amax_dv_bits, m);
    }
}

// A matrix of `rows` rows of w elements of `size` bytes, a pitch of ld elements apart.
struct Rows {
    const void* p;
    int64_t rows, ld, w;
    int size;
};
static bool rows_apart(const Rows& a, const Rows& b)
{
    if (apart({a.p, ((a.rows - 1) * a.ld + a.w) * a.size}, {b.p, ((b.rows - 1) * b.ld + b.w) * b.size})) return true;
    const uintptr_t p = (uintptr_t)a.p, q = (uintptr_t)b.p;
    const int64_t pitch = a.ld * a.size;  // column slices of one matrix
    if (pitch != b.ld * b.size) return false;
    const int64_t d = (((int64_t)(q - p)) % pitch + pitch) % pitch;
    return d >= a.w * a.size && d + b.w * b.size <= pitch;
}

// Whether the backward takes one launch for dQ and dK/dV.  In two, `blocks` blocks of n, n - 1, ..., 1 tiles take the time of n
// tiles each or, with more blocks, that of their sum over the units: with less than 2 n / (n + 1) blocks per unit the former
// is longer.  us of rope, attention and its backward, two launches / one (sequences x tokens, heads): 2 x 512, 8 107 / 84,
// 1 x 2048, 16 264 / 208, 1 x 8192, 8 844 / 698, 4 x 1000, 16 213 / 197, 5 x 256, 32 131 / 129; at the line 7 x 2048, 8 452 / 443 and
// 8 x 256, 32 164 / 172, beyond it 2 x 2048, 32 454 / 453 and 1 x 8192, 32 2344 / 2354.  With one tile each, more than half a unit's
// share of blocks are a second round, which the rest of a short block's time and delta's launch make longer than a second launch.  us of
// the backward alone, two / one, 17 and 24 sequences of 8 heads: 16 tokens 14.6 / 16.1 and 14.8 / 17.6, 64 18.0 / 18.8 and 19.2 / 20.7, 96 25.5 / 26.2
// and 27.9 / 26.8, 112 27.9 / 27.7 and 30.3 / 28.0; 8 / 2 heads 48 tokens 22.5 / 22.5 and 24.0 / 24.9, 64 24.9 / 25.0 and 28.4 / 27.9; 28 and 30 sequences of 40
// tokens 23.2 / 24.0 and 23.9 / 24.0, 48 24.7 / 24.4 and 25.4 / 24.1, 56 26.5 / 24.6 and 27.2 / 25.2.
static bool one_launch(int64_t blocks, int64_t n, int64_t S, bool grouped, int cus)
{
    return blocks * (n + 1) < 2 * n * cus && (n > 1 || 2 * blocks <= cus || S >= (!grouped ? 112 : 8 * blocks < 7 * cus ? 64 : 48));
}

constexpr int kDqWaves = 8;  // 256 queries per block, one block per compute unit
constexpr int kDkvWaves = 8;             // 256 keys per block, one block per compute unit
static f8_status check_attn(const void* q, int64_t ldq, const void* k, int64_t ldk, int64_t B, int64_t S, int64_t Hq,
                            int64_t Hkv, int64_t hd)
{
    if (!q || !k) return F8_ERR_NULL;
    if (hd != kHd || B < 0 || S < 0 || (S % 8) || Hq < 1 || Hkv < 1 || (Hq % Hkv)) return F8_ERR_SHAPE;
    if (S >= (1 << 24) || Hq >= (1 << 16) || B * S >= ((int64_t)1 << 31)) return F8_ERR_SHAPE;
    if (ldq < Hq * hd || ldk < Hkv * hd || (ldq % 8) || (ldk % 8)) return F8_ERR_SHAPE;
    if (!aligned16(q) || !aligned16(k)) return F8_ERR_ALIGN;
    return F8_OK;
}

}  // namespace f8

using namespace f8;

extern "C" {

f8_status f8_sdpa_fwd(const void* q_bf16, int64_t ldq, const void* k_bf16, int64_t ldk, const void* vt_bf16, int64_t B,
                      int64_t S, int64_t Hq, int64_t Hkv, int64_t hd, void* o_bf16, int64_t ldo, float* lse, float* amax_o,
                      void* stream)
{
    f8_status s = check_attn(q_bf16, ldq, k_bf16, ldk, B, S, Hq, Hkv, hd);
    if (s != F8_OK) return s;
    if (!vt_bf16 || !o_bf16 || !lse) return F8_ERR_NULL;
    if (ldo < Hq * hd || (ldo % 8)) return F8_ERR_SHAPE;
    if (!aligned16(vt_bf16) || !aligned16(o_bf16)) return F8_ERR_ALIGN;
    if (amax_o) zero_amax_kernel<<<1, 1, 0, (hipStream_t)stream>>>(reinterpret_cast<uint32_t*>(amax_o));
    if (B == 0 || S == 0) return last_launch_status();
    constexpr int kFwdWaves = 8;  // 256 queries per block, one block per compute unit
    const int64_t nqt = (S + 32 * kFwdWaves - 1) / (32 * kFwdWaves), nb = nqt * Hq * B;
    if (nb > (int64_t)0x7FFFFFFF) return F8_ERR_SHAPE;
    const float scale_log2e = (float)(1.4426950408889634074 / sqrt((double)hd));
    const auto kernel = far_rows(kBk, ldk) || far_rows(kHd, B * S) ? sdpa_fwd_kernel<kFwdWaves, true> : sdpa_fwd_kernel<kFwdWaves, false>;
    kernel<<<(unsigned)nb, 64 * kFwdWaves, 0, (hipStream_t)stream>>>(
        (const uint16_t*)q_bf16, ldq, (const uint16_t*)k_bf16, ldk, (const uint16_t*)vt_bf16, B * S, (int)S, (int)Hq,
        (int)(Hq / Hkv), scale_log2e, (uint16_t*)o_bf16, ldo, lse, (int)nqt, reinterpret_cast<uint32_t*>(amax_o));
    return last_launch_status();
}

size_t f8_sdpa_bwd_workspace_bytes(int64_t B, int64_t S, int64_t Hq, int64_t Hkv, int64_t hd)
{
    if (B <= 0 || S <= 0 || Hq <= 0 || Hkv <= 0 || hd <= 0 || (Hq % Hkv) || Hq == Hkv) return 0;
    return (size_t)2 * (size_t)(B * S) * (size_t)(Hq * hd) * sizeof(float);  // dk and dv shares of every query head
}

static f8_status sdpa_bwd(const void* q_bf16, int64_t ldq, const void* k_bf16, int64_t ldk, const void* v_bf16, int64_t ldv, const void* o_bf16,
                          int64_t ldo, const void* do_bf16, int64_t lddo, const float* lse, int64_t B, int64_t S, int64_t Hq, int64_t Hkv,
                          int64_t hd, void* dq_bf16, int64_t lddq, void* dk_bf16, int64_t lddk, void* dv_bf16, int64_t lddv, float* delta,
                          float* amax_dv_inout, void* workspace, size_t workspace_bytes_, void* stream, bool copies_aligned = true)
{
    f8_status s = check_attn(q_bf16, ldq, k_bf16, ldk, B, S, Hq, Hkv, hd);
    if (s != F8_OK) return s;
    if (!v_bf16 || !o_bf16 || !do_bf16 || !lse || !dq_bf16 || !dk_bf16 || !dv_bf16 || !delta) return F8_ERR_NULL;
    const int64_t wq = Hq * hd, wk = Hkv * hd;
    if (ldv < wk || ldo < wq || lddo < wq || lddq < wq || lddk < wk || lddv < wk || (ldv % 8) || (ldo % 8) || (lddo % 8) ||
        (lddq % 8) || (lddk % 8) || (lddv % 8))
        return F8_ERR_SHAPE;
    if (!copies_aligned || !aligned16(v_bf16) || !aligned16(o_bf16) || !aligned16(do_bf16) || !aligned16(dq_bf16) || !aligned16(dk_bf16) || !aligned16(dv_bf16))
        return F8_ERR_ALIGN;
    const int64_t group = Hq / Hkv;
    if (amax_dv_inout && group == 1) return F8_ERR_ENUM;  // the amax of dv is taken where the heads' shares are summed
    if (group > 1 && (!workspace || workspace_bytes_ < f8_sdpa_bwd_workspace_bytes(B, S, Hq, Hkv, hd))) return F8_ERR_WORKSPACE;
    if (group > 1 && !aligned16(workspace)) return F8_ERR_ALIGN;
    if (B == 0 || S == 0) return F8_OK;
    hipStream_t st = (hipStream_t)stream;
    const int64_t M = B * S;
    if ((S + 255) / 256 * Hq * B > (int64_t)0x7FFFFFFF) return F8_ERR_SHAPE;  // one block per 256 tokens and head
    const double sc = 1.0 / sqrt((double)hd);
    const float scale = (float)sc, scale_log2e = (float)(sc * 1.4426950408889634074);
    float* part_k = group > 1 ? (float*)workspace : nullptr;
    float* part_v = group > 1 ? part_k + group * M * wk : nullptr;
    const DqArgs q{(const uint16_t*)q_bf16, (const uint16_t*)k_bf16, (const uint16_t*)v_bf16, (const uint16_t*)o_bf16, (const uint16_t*)do_bf16,
                   ldq, ldk, ldv, ldo, lddo, lse, M, (int)S, (int)Hq, (int)group, scale_log2e, scale, (uint16_t*)dq_bf16, lddq, delta};
    const DkvArgs kv{(const uint16_t*)q_bf16, (const uint16_t*)k_bf16, (const uint16_t*)v_bf16, (const uint16_t*)do_bf16, ldq, ldk, ldv, lddo,
                     lse, delta, M, (int)S, (int)Hq, (int)group, scale_log2e, scale, (uint16_t*)dk_bf16, (uint16_t*)dv_bf16, lddk, lddv, part_k, part_v};
    const int64_t nqt = (S + 32 * kDqWaves - 1) / (32 * kDqWaves), blocks = nqt * Hq * B;
    const bool dq_far = far_rows(kBk, ldk) || far_rows(kBk, ldv);
    const bool dkv_far = far_rows(kDkvQ, ldq) || far_rows(kDkvQ, lddo) || far_rows(32 * kDkvWaves, ldv);
    static_assert(kDqWaves == kDkvWaves, "as many query tiles as key tiles");
    // One after the other, dK and dV (or their shares) may lie over what only dQ's kernel still reads, or over dQ: gradients
    // that replace k and v, or one buffer for both where one is of no use.
    auto written_apart = [&](const Rows& w) {
        for (const Rows& r : {Rows{q_bf16, M, ldq, wq, 2}, Rows{k_bf16, M, ldk, wk, 2}, Rows{v_bf16, M, ldv, wk, 2}, Rows{do_bf16, M, lddo, wq, 2},
                              Rows{lse, Hq, M, M, 4}, Rows{delta, Hq, M, M, 4}, Rows{dq_bf16, M, lddq, wq, 2}})
            if (!rows_apart(w, r)) return false;
        return true;
    };
    const bool dq_straight = S <= kStraightRows, dkv_straight = group > 1 ? S <= kStraightShares : dq_straight;
    const bool one = !dq_far && !dkv_far && one_launch(blocks, nqt, S, group > 1, cu_count()) &&
                     (group > 1 ? written_apart({workspace, 2 * group, M * wk, M * wk, 4})
                                : written_apart({dk_bf16, M, lddk, wk, 2}) && written_apart({dv_bf16, M, lddv, wk, 2}));
    if (one) {
        sdpa_delta_kernel<<<(unsigned)((M * Hq + kDeltaRows - 1) / kDeltaRows), kAttnThreads, 0, st>>>(q.O, ldo, q.dO, lddo, M, (int)Hq, delta);
        (dkv_straight ? sdpa_bwd_kernel<kDqWaves, true> : sdpa_bwd_kernel<kDqWaves, false>)<<<(unsigned)(2 * blocks), 64 * kDqWaves, 0, st>>>(q, kv, (int)nqt);
    } else {
        const auto dq_kernel = dq_far ? sdpa_bwd_dq_kernel<kDqWaves, true> : dq_straight ? sdpa_bwd_dq_kernel<kDqWaves, false, true> : sdpa_bwd_dq_kernel<kDqWaves, false>;
        const auto dkv_kernel = dkv_far ? sdpa_bwd_dkv_kernel<kDkvWaves, true> : dkv_straight ? sdpa_bwd_dkv_kernel<kDkvWaves, false, true> : sdpa_bwd_dkv_kernel<kDkvWaves, false>;
        dq_kernel<<<(unsigned)blocks, 64 * kDqWaves, 0, st>>>(q, (int)nqt);
        dkv_kernel<<<(unsigned)blocks, 64 * kDkvWaves, 0, st>>>(kv);
    }
    if (group > 1) {
        int64_t nb = (2 * M * (wk / 8) + kAttnThreads - 1) / kAttnThreads;
        if (nb > 8192) nb = 8192;
        sdpa_group_sum_kernel<<<(unsigned)nb, kAttnThreads, 0, st>>>(part_k, part_v, M, wk, (int)group, (uint16_t*)dk_bf16, lddk,
                                                                   (uint16_t*)dv_bf16, lddv, reinterpret_cast<uint32_t*>(amax_dv_inout));
    }
    return last_launch_status();
}

f8_status f8_sdpa_bwd(const void* q_bf16, int64_t ldq, const void* qt_bf16, const void* k_bf16, int64_t ldk,
                      const void* kt_bf16, const void* v_bf16, int64_t ldv, const void* o_bf16, int64_t ldo,
                      const void* do_bf16, int64_t lddo, const void* dot_bf16, const float* lse, int64_t B, int64_t S,
                      int64_t Hq, int64_t Hkv, int64_t hd, void* dq_bf16, int64_t lddq, void* dk_bf16, int64_t lddk,
                      void* dv_bf16, int64_t lddv, float* delta, float* amax_dv_inout, void* workspace, size_t workspace_bytes_,
                      void* stream)
{
    f8_status s = check_attn(q_bf16, ldq, k_bf16, ldk, B, S, Hq, Hkv, hd);
    if (s != F8_OK) return s;
    if (!qt_bf16 || !kt_bf16 || !dot_bf16) return F8_ERR_NULL;
    return sdpa_bwd(q_bf16, ldq, k_bf16, ldk, v_bf16, ldv, o_bf16, ldo, do_bf16, lddo, lse, B, S, Hq, Hkv, hd, dq_bf16, lddq, dk_bf16, lddk,
                    dv_bf16, lddv, delta, amax_dv_inout, workspace, workspace_bytes_, stream,
                    aligned16(qt_bf16) && aligned16(kt_bf16) && aligned16(dot_bf16));
}

f8_status f8_sdpa_bwd_rows(const void* q_bf16, int64_t ldq, const void* k_bf16, int64_t ldk, const void* v_bf16, int64_t ldv,
                           const void* o_bf16, int64_t ldo, const void* do_bf16, int64_t lddo, const float* lse, int64_t B, int64_t S,
                           int64_t Hq, int64_t Hkv, int64_t hd, void* dq_bf16, int64_t lddq, void* dk_bf16, int64_t lddk, void* dv_bf16,
                           int64_t lddv, float* delta, float* amax_dv_inout, void* workspace, size_t workspace_bytes_, void* stream)
{
    return sdpa_bwd(q_bf16, ldq, k_bf16, ldk, v_bf16, ldv, o_bf16, ldo, do_bf16, lddo, lse, B, S, Hq, Hkv, hd, dq_bf16, lddq, dk_bf16, lddk,
                    dv_bf16, lddv, delta, amax_dv_inout, workspace, workspace_bytes_, stream);
}

}  // extern "C"

// The bf16 glue between the two Float8 linears of a Llama feed-forward block,
//   Y = W2 ( silu(W1 x) * (W3 x) ),
// with W1 and W3 stacked into one linear whose output row is [a | b]:
//   forward   h = silu(a) * b                       silu(t) = t / (1 + e^-t)
//   backward  da = dh * b * silu'(a),  db = dh * silu(a)
// Both are elementwise and HBM-bound.  Each also leaves the amax of what it wrote, taken while
// the values are in registers, so that the Float8 linear that consumes the result casts it in
// one pass (f8_linear_fwd_chained / f8_linear_bwd_chained) instead of reading it twice.
#include <type_traits>

#include "f8_device.hpp"
#include "f8_host.hpp"

namespace f8 {

constexpr int kGlueThreads = 256;
constexpr int kGlueWaves = kGlueThreads / kWave;
constexpr int kGlueMaxBlocks = 2048;
static_assert((size_t)kGlueMaxBlocks * sizeof(uint32_t) <= kMinWorkspaceBytes, "one partial per block fits the minimum workspace");

// ab [M, 2H] as 16-byte chunks: row m has 2 * hc chunks, a first; h [M, H]: hc chunks per row.
// Bound by memory.  A block takes CHUNKS chunks per thread that lie side by side, then as many a grid further on.
// STREAM (from 8 M elements of h on): loads and stores past the caches, which would keep little of the tensors until they are
// read again, and two chunks side by side, so that one front moves through each tensor (chunks of one thread a grid apart are
// streams some MB apart that meet in the same memory channels).  us plain / past the caches, with other data in between:
// 8192 x 14336 forward 130 / 118 (6.0 TB/s), backward 223 / 204, 2048 x 14336 33.1 / 30.0 and 54.5 / 49.5.  With operands that
// are still in the caches it is 8 % slower up to 2048 x 14336, and the cast that reads the result misses more (with an amax
// after it 4096 x 4096 31.8 / 30.2, 2048 x 4096 19.4 / 21.1): in a whole block of the 8B model gate and casts take 758 / 745 us
// at 8192 tokens, 429 / 438 at 4096.  Stores to the caches and only the loads past them: 428 there, but alone 8192 x 14336 134
// and 229, and whole blocks of 2048 tokens lose 1 % in their products.
// Smaller tensors: one chunk a thread, one or two of them in turn; a block of its own for every 256 chunks only while those
// are at most one per compute unit.  us in turn / all at once: 256 x 1024 4.7 / 4.3, but 1008 x 4096
// 8.9 / 9.8 and backward 10.7 / 11.7 (blocks that do little, and twice the partial maxima to read); two side by side 9.1 and
// 11.7.
constexpr int kGateMaxBlocks = 1024;  // of a streamed tensor (2048: 0.5 to 1.5 % slower)
constexpr int kGateAtOnceBlocks = 256;
constexpr int64_t kGateStreamChunks = (int64_t)1 << 20;

template <bool STREAM>
__device__ inline uint4 gate_load(const uint4* p)
{
    if constexpr (STREAM) return load_once(p);
    else return *p;
}
template <bool STREAM>
__device__ inline void gate_store(uint4* p, uint4 v)
{
    if constexpr (STREAM) store_stream(p, v);
    else *p = v;
}

template <bool STREAM, int CHUNKS = STREAM ? 2 : 1>
__global__ __launch_bounds__(kGlueThreads) void silu_mul_kernel(const uint4* __restrict__ ab, int64_t M, int64_t hc,
                                                               uint4* __restrict__ h, uint32_t* __restrict__ partial)
{
    __shared__ uint32_t red[kGlueWaves];
    const int64_t n = M * hc;
    uint32_t acc = 0;
    for (int64_t c0 = (int64_t)blockIdx.x * (CHUNKS * kGlueThreads) + threadIdx.x; c0 < n; c0 += (int64_t)gridDim.x * (CHUNKS * kGlueThreads)) {
        uint4 a[CHUNKS], b[CHUNKS];
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u) {
            const int64_t c = c0 + u * kGlueThreads < n ? c0 + u * kGlueThreads : c0, at = c + c / hc * hc;
            a[u] = gate_load<STREAM>(ab + at), b[u] = gate_load<STREAM>(ab + at + hc);
        }
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u) {
            if (c0 + u * kGlueThreads >= n) break;
            uint4 o;
            o.x = silu_mul2(a[u].x, b[u].x), o.y = silu_mul2(a[u].y, b[u].y);
            o.z = silu_mul2(a[u].z, b[u].z), o.w = silu_mul2(a[u].w, b[u].w);
            gate_store<STREAM>(h + c0 + u * kGlueThreads, o);
            acc = absmax_acc(acc, o);
        }
    }
    if (partial) {
        const uint32_t mx = block_max_u32<kGlueWaves>(pk_collapse(acc), red);
        if (threadIdx.x == 0) partial[blockIdx.x] = mx;
    }
}

template <bool STREAM, int CHUNKS = STREAM ? 2 : 1>
__global__ __launch_bounds__(kGlueThreads) void silu_mul_bwd_kernel(const uint4* __restrict__ ab, const uint4* __restrict__ dh,
                                                                   int64_t M, int64_t hc, uint4* __restrict__ dab,
                                                                   uint32_t* __restrict__ partial)
{
    __shared__ uint32_t red[kGlueWaves];
    const int64_t n = M * hc;
    uint32_t acc = 0;
    for (int64_t c0 = (int64_t)blockIdx.x * (CHUNKS * kGlueThreads) + threadIdx.x; c0 < n; c0 += (int64_t)gridDim.x * (CHUNKS * kGlueThreads)) {
        uint4 a[CHUNKS], b[CHUNKS], g[CHUNKS];
        int64_t at[CHUNKS];
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u) {
            const int64_t c = c0 + u * kGlueThreads < n ? c0 + u * kGlueThreads : c0;
            at[u] = c + c / hc * hc;
            a[u] = gate_load<STREAM>(ab + at[u]), b[u] = gate_load<STREAM>(ab + at[u] + hc), g[u] = gate_load<STREAM>(dh + c);
        }
#pragma unroll
        for (int u = 0; u < CHUNKS; ++u) {
            if (c0 + u * kGlueThreads >= n) break;
            uint4 da, db;
            silu_mul_bwd2(a[u].x, b[u].x, g[u].x, &da.x, &db.x);
            silu_mul_bwd2(a[u].y, b[u].y, g[u].y, &da.y, &db.y);
            silu_mul_bwd2(a[u].z, b[u].z, g[u].z, &da.z, &db.z);
            silu_mul_bwd2(a[u].w, b[u].w, g[u].w, &da.w, &db.w);
            gate_store<STREAM>(dab + at[u], da);
            gate_store<STREAM>(dab + at[u] + hc, db);
            acc = absmax_acc(absmax_acc(acc, da), db);
        }
    }
    if (partial) {
        const uint32_t mx = block_max_u32<kGlueWaves>(pk_collapse(acc), red);
        if (threadIdx.x == 0) partial[blockIdx.x] = mx;
    }
}

__global__ __launch_bounds__(kGlueThreads) void glue_amax_final_kernel(const uint32_t* __restrict__ partial, int n,
                                                                      float* __restrict__ amax_out)
{
    __shared__ uint32_t red[kGlueWaves];
    uint32_t m = 0;
    for (int i = threadIdx.x; i < n; i += kGlueThreads) m = partial[i] > m ? partial[i] : m;
    m = block_max_u32<kGlueWaves>(m, red);
    if (threadIdx.x == 0) amax_out[0] = mag_to_float(m);
}

// RMS normalisation, forward: y[m, :] = x[m, :] * rstd[m] * g, rstd[m] = 1 / sqrt(mean x[m, :]^2 + eps).
// One wavefront per row, rows strided over the grid; the row is read twice (the second time
// from the caches it has just been loaded into): once for the sum of squares, once to scale.
__device__ inline float sumsq_word(uint32_t w)
{
    const float a = bf16_lo(w), b = bf16_hi(w);
    return a * a + b * b;
}
__device__ inline uint32_t scale_word(uint32_t x, uint32_t g, float r)
{
    return pack_bf16((bf16_lo(x) * r) * bf16_lo(g), (bf16_hi(x) * r) * bf16_hi(g));
}

// NC > 0: a row has at most NC 16-byte chunks per lane and is kept in registers between the two
// passes; NC = 0: any row length, the second pass reads the row again (from the caches).
// STREAM: x and y past the caches (8192 x 4096 33.0 -> 29.0 us, 8192 x 8192 62.6 -> 53.2).  Tensors of less than
// kNormStreamChunks do not: the next call reads y, from the caches (a block of 1008 x 1024 loses 1 % with it).
constexpr int64_t kNormStreamChunks = (int64_t)1 << 21;
template <int NC, bool STREAM>
__global__ __launch_bounds__(kGlueThreads) void rmsnorm_kernel(const uint4* __restrict__ x, const uint4* __restrict__ g,
                                                              int64_t M, int64_t dc /* 16-byte chunks per row */,
                                                              float inv_d, float eps, uint4* __restrict__ y,
                                                              float* __restrict__ rstd, uint32_t* __restrict__ partial)
{
    __shared__ uint32_t red[kGlueWaves];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint32_t acc = 0;
    for (int64_t m = (int64_t)blockIdx.x * kGlueWaves + wave; m < M; m += (int64_t)gridDim.x * kGlueWaves) {
        const uint4* row = x + m * dc;
        float ss = 0.0f;
        uint4 keep[NC > 0 ? NC : 1];
        if constexpr (NC > 0) {
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                const int64_t c = lane + (int64_t)kWave * i;
                keep[i] = c < dc ? (STREAM ? load_once(row + c) : row[c]) : make_uint4(0, 0, 0, 0);
                ss += (sumsq_word(keep[i].x) + sumsq_word(keep[i].y)) + (sumsq_word(keep[i].z) + sumsq_word(keep[i].w));
            }
        } else {
            for (int64_t c = lane; c < dc; c += kWave) {
                const uint4 v = row[c];
                ss += (sumsq_word(v.x) + sumsq_word(v.y)) + (sumsq_word(v.z) + sumsq_word(v.w));
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) ss += __shfl_xor(ss, off, kWave);
        const float r = 1.0f / sqrtf(ss * inv_d + eps);
        if (lane == 0 && rstd) rstd[m] = r;
        auto emit = [&](int64_t c, uint4 v) {
            const uint4 w = g[c];
            uint4 o;
            o.x = scale_word(v.x, w.x, r), o.y = scale_word(v.y, w.y, r);
            o.z = scale_word(v.z, w.z, r), o.w = scale_word(v.w, w.w, r);
            if constexpr (STREAM) store_stream(y + m * dc + c, o);
            else y[m * dc + c] = o;
            acc = absmax_acc(acc, o);
        };
        if constexpr (NC > 0) {
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                const int64_t c = lane + (int64_t)kWave * i;
                if (c < dc) emit(c, keep[i]);
            }
        } else {
            for (int64_t c = lane; c < dc; c += kWave) emit(c, row[c]);
        }
    }
    if (partial) {
        const uint32_t mx = block_max_u32<kGlueWaves>(pk_collapse(acc), red);
        if (threadIdx.x == 0) partial[blockIdx.x] = mx;
    }
}

// f(which instance of a gate kernel, its blocks)
template <class F>
static int launch_gate(int64_t chunks, F&& f)
{
    if (chunks >= kGateStreamChunks) return f(std::true_type{}, kGateMaxBlocks), kGateMaxBlocks;
    static_assert(kGateStreamChunks <= 2 * kGlueThreads * kGlueMaxBlocks && kGateMaxBlocks <= kGlueMaxBlocks, "one partial maximum per block");
    const int one = (int)((chunks + kGlueThreads - 1) / kGlueThreads), nb = one <= kGateAtOnceBlocks ? one : (one + 1) / 2;
    f(std::false_type{}, nb);
    return nb;
}

static f8_status check_glue(const void* ab, const void* other, void* out, int64_t M, int64_t H, const float* amax,
                            const void* ws, size_t ws_bytes)
{
    if (!ab || !other || !out) return F8_ERR_NULL;
    if (M < 0 || H < 0 || (M % 16) || (H % 16)) return F8_ERR_SHAPE;
    if (!aligned16(ab) || !aligned16(other) || !aligned16(out)) return F8_ERR_ALIGN;
    if (amax && (!ws || ws_bytes < (size_t)kGlueMaxBlocks * sizeof(uint32_t))) return F8_ERR_WORKSPACE;
    return F8_OK;
}

}  // namespace f8

using namespace f8;

extern "C" {

f8_status f8_silu_mul(const void* ab_bf16, int64_t M, int64_t H, void* h_bf16, float* amax_h, void* workspace,
                      size_t workspace_bytes_, void* stream)
{
    f8_status s = check_glue(ab_bf16, h_bf16, h_bf16, M, H, amax_h, workspace, workspace_bytes_);
    if (s != F8_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    const int64_t hc = H / 8;
    int nb = 0;
    if (M > 0 && H > 0) {
        nb = launch_gate(M * hc, [&](auto STREAM, int blocks) {
            silu_mul_kernel<STREAM()><<<blocks, kGlueThreads, 0, st>>>((const uint4*)ab_bf16, M, hc, (uint4*)h_bf16,
                                                                                amax_h ? (uint32_t*)workspace : nullptr);
        });
    }
    if (amax_h) glue_amax_final_kernel<<<1, kGlueThreads, 0, st>>>((const uint32_t*)workspace, nb, amax_h);
    return last_launch_status();
}

f8_status f8_silu_mul_bwd(const void* ab_bf16, const void* dh_bf16, int64_t M, int64_t H, void* dab_bf16,
                          float* amax_dab, void* workspace, size_t workspace_bytes_, void* stream)
{
    f8_status s = check_glue(ab_bf16, dh_bf16, dab_bf16, M, H, amax_dab, workspace, workspace_bytes_);
    if (s != F8_OK) return s;
    hipStream_t st = (hipStream_t)stream;
    const int64_t hc = H / 8;
    int nb = 0;
    if (M > 0 && H > 0) {
        nb = launch_gate(M * hc, [&](auto STREAM, int blocks) {
            silu_mul_bwd_kernel<STREAM()><<<blocks, kGlueThreads, 0, st>>>((const uint4*)ab_bf16, (const uint4*)dh_bf16, M, hc,
                                                                                    (uint4*)dab_bf16, amax_dab ? (uint32_t*)workspace : nullptr);
        });
    }
    if (amax_dab) glue_amax_final_kernel<<<1, kGlueThreads, 0, st>>>((const uint32_t*)workspace, nb, amax_dab);
    return last_launch_status();
}

f8_status f8_rmsnorm(const void* x_bf16, const void* g_bf16, int64_t M, int64_t D, float eps, void* y_bf16,
                     float* rstd, float* amax_y, void* workspace, size_t workspace_bytes_, void* stream)
{
    if (!x_bf16 || !g_bf16 || !y_bf16) return F8_ERR_NULL;
    if (M < 0 || D < 0 || (M % 16) || (D % 16) || !(eps >= 0.0f)) return F8_ERR_SHAPE;
    if (!aligned16(x_bf16) || !aligned16(g_bf16) || !aligned16(y_bf16)) return F8_ERR_ALIGN;
    if (amax_y && (!workspace || workspace_bytes_ < (size_t)kGlueMaxBlocks * sizeof(uint32_t))) return F8_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    int nb = 0;
    if (M > 0 && D > 0) {
        int64_t b = (M + kGlueWaves - 1) / kGlueWaves;
        nb = (int)(b > kGlueMaxBlocks ? kGlueMaxBlocks : b);
        const bool stream = M * (D / 8) >= kNormStreamChunks;
        const auto kernel = D <= 8 * kWave * 8    ? (stream ? rmsnorm_kernel<8, true> : rmsnorm_kernel<8, false>)  // rows up to 4096
                            : D <= 8 * kWave * 16 ? (stream ? rmsnorm_kernel<16, true> : rmsnorm_kernel<16, false>)  // and 8192 stay in registers
                                                  : rmsnorm_kernel<0, false>;
        kernel<<<nb, kGlueThreads, 0, st>>>((const uint4*)x_bf16, (const uint4*)g_bf16, M, D / 8, 1.0f / (float)D, eps, (uint4*)y_bf16, rstd,
                                            amax_y ? (uint32_t*)workspace : nullptr);
    }
    if (amax_y) glue_amax_final_kernel<<<1, kGlueThreads, 0, st>>>((const uint32_t*)workspace, nb, amax_y);
    return last_launch_status();
}

}  // extern "C"

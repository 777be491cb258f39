// The bf16 operations that join the Float8 linears of one transformer block (Section 2.2.4
// applies Float8 to the linear layers only; everything between them stays in bf16): rotary
// position embedding (if asked, with a transposed copy), a plain bf16 transposition, the residual addition and the backward of RMSNorm.
// All HBM-bound: 16-byte accesses, fp32 arithmetic, one rounding to bf16.
#include "f8_device.hpp"
#include "f8_host.hpp"

#include <math.h>

namespace f8 {

constexpr int kBlkThreads = 256;
constexpr int kBlkWaves = kBlkThreads / kWave;
constexpr int kRt = 64;            // tile edge of the rotating / transposing kernel
constexpr int kRtStride = kRt + 2; // LDS row pitch in bf16: odd number of words

struct RopeFreq {
    double f[128];  // theta^(-2 i / hd), i < hd / 2 <= 128
};

__device__ inline uint32_t add_word(uint32_t a, uint32_t b)
{
    return pack_bf16(bf16_lo(a) + bf16_lo(b), bf16_hi(a) + bf16_hi(b));
}

// rotate the pair (lo, hi) of one word by (c, s)
__device__ inline uint32_t rotate_word(uint32_t w, float c, float s)
{
    const float x0 = bf16_lo(w), x1 = bf16_hi(w);
    return pack_bf16(x0 * c - x1 * s, x0 * s + x1 * c);
}

// x [rows, nh * hd] (row pitch ldx) -> out (row pitch ldo; ROTATE: pairs of adjacent columns turned
// by pos * freq) and out_t [nh * hd, rows] (packed).  One block: a 64x64 tile at the same place of
// `hpb` consecutive heads, one head after the other: the sines and cosines depend on the row and
// on the column inside the head only, so they are taken once and used for every head.  The next head's tile is requested
// before this one is worked on, the first before the sines: a block has one tile in flight otherwise, and its stores before
// it (4000 x 16 heads of 128: both outputs 15.2 -> 14.4 us, one 10.2 -> 9.2; 8192 x 32 47.4 -> 44.6 and 29.8 -> 28.2).  rows, hd
// and the pitches are multiples of 8.  (The plain transposition is the case of one head of width
// cols.)
struct RopePart {
    const uint16_t* x;
    uint16_t *out, *out_t;
    int64_t ldx, ldo;
    int nh, hpb;
    int tiles_c;       // per row of tiles: tiles per head x head groups
    unsigned blocks;
};
// `id`: the block's number within the part; tile: kRt * kRtStride of LDS (OUT_T)
template <bool ROTATE, bool OUT, bool OUT_T>
__device__ __forceinline__ void rope_tile_work(const RopePart& P, unsigned id, int64_t rows, int hd, int64_t S, float sign, const RopeFreq& fr,
                                               uint32_t* __restrict__ amax_bits /* nullable: max-updated */, uint16_t* tile)
{
    const uint16_t* __restrict__ x = P.x;
    uint16_t *__restrict__ out = P.out, *__restrict__ out_t = P.out_t;
    const int64_t ldx = P.ldx, ldo = P.ldo;
    const int nh = P.nh, hpb = P.hpb;
    uint32_t mag = 0;  // packed pair of the largest 15-bit magnitudes written
    const int tph = (hd + kRt - 1) / kRt;  // tiles per head
    const int tc = id % P.tiles_c;
    const int64_t r0 = (int64_t)(id / P.tiles_c) * kRt;
    const int c0 = (tc % tph) * kRt, h0 = (tc / tph) * hpb;  // column inside the head, first head
    const int cc = threadIdx.x & 7, rr = threadIdx.x >> 3;
    const int cih = c0 + cc * 8;            // this thread's column inside the head
    const bool col_ok = cih < hd;
    const int h_end = h0 + hpb < nh ? h0 + hpb : nh;
    auto request = [&](uint4(&v)[2], int h) {
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int64_t r = r0 + rr + 32 * i;
            v[i] = make_uint4(0, 0, 0, 0);
            if (col_ok && r < rows) v[i] = *reinterpret_cast<const uint4*>(x + r * ldx + (int64_t)h * hd + cih);
        }
    };
    uint4 next[2];
    request(next, h0);
    float cs[2][4], sn[2][4];
    if constexpr (ROTATE) {
        const bool short_ids = ((uint64_t)rows | (uint64_t)S) >> 32 == 0;  // a 64-bit remainder takes 0.3 us
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int64_t r = r0 + rr + 32 * i;
            const double pos = short_ids ? (double)((uint32_t)r % (uint32_t)S) : (double)(r % S);
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                // the angle reaches thousands of radians: product and reduction to
                // [-pi, pi] in fp64, sine and cosine of the remainder in fp32
                const double a = pos * fr.f[col_ok ? (cih >> 1) + j : 0];
                const double red = a - 6.283185307179586476925286766559 * rint(a * 0.15915494309189533576888376337251);
                sincosf((float)red, &sn[i][j], &cs[i][j]);
                sn[i][j] *= sign;
            }
        }
    }
    for (int h = h0; h < h_end; ++h) {
        const int64_t col = (int64_t)h * hd + cih;
        uint4 here[2] = {next[0], next[1]};
        if (h + 1 < h_end) request(next, h + 1);  // on its way while this head is rotated, turned and stored
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int rl = rr + 32 * i;
            const int64_t r = r0 + rl;
            uint4 v = here[i];
            if (col_ok && r < rows) {
                if constexpr (ROTATE)
                    v = make_uint4(rotate_word(v.x, cs[i][0], sn[i][0]), rotate_word(v.y, cs[i][1], sn[i][1]),
                                   rotate_word(v.z, cs[i][2], sn[i][2]), rotate_word(v.w, cs[i][3], sn[i][3]));
                if constexpr (OUT) *reinterpret_cast<uint4*>(out + r * ldo + col) = v;
                mag = absmax_acc(mag, v);
            }
            if constexpr (OUT_T) {
                uint32_t* t32 = reinterpret_cast<uint32_t*>(tile + rl * kRtStride + cc * 8);  // 4-byte aligned: pitch and cc*8 are even
                t32[0] = v.x, t32[1] = v.y, t32[2] = v.z, t32[3] = v.w;
            }
        }
        if constexpr (OUT_T) {
            __syncthreads();
            const int rb = threadIdx.x & 7, cb = threadIdx.x >> 3;
            const int64_t rbase = r0 + 8 * rb;
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int c = cb + 32 * i;
                uint32_t o[4];
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    o[j] = (uint32_t)tile[(8 * rb + 2 * j) * kRtStride + c] | ((uint32_t)tile[(8 * rb + 2 * j + 1) * kRtStride + c] << 16);
                if (rbase < rows && c0 + c < hd)  // rows is a multiple of 8: the piece is all in or all out
                    *reinterpret_cast<uint4*>(out_t + ((int64_t)h * hd + c0 + c) * rows + rbase) = make_uint4(o[0], o[1], o[2], o[3]);
            }
            __syncthreads();  // the tile is free for the next head
        }
    }
    if (amax_bits) {  // a maximum of non-negative floats is a maximum of their bit patterns: order-independent
        const uint32_t m = wave_max_u32(pk_collapse(mag)) << 16;
        if ((threadIdx.x & (kWave - 1)) == 0 && m > __atomic_load_n(amax_bits, __ATOMIC_RELAXED)) atomicMax(amax_bits, m);
    }
}

template <bool ROTATE, bool OUT, bool OUT_T>
__global__ __launch_bounds__(kBlkThreads) void rope_tile_kernel(const RopePart part, int64_t rows, int hd, int64_t S, float sign, const RopeFreq fr,
                                                                uint32_t* __restrict__ amax_bits)
{
    __shared__ uint16_t tile[OUT_T ? kRt * kRtStride : 1];
    rope_tile_work<ROTATE, OUT, OUT_T>(part, blockIdx.x, rows, hd, S, sign, fr, amax_bits, tile);
}

// q and k rotated and (V) v transposed in one launch: of small tensors each launch takes its own 4 us (1008 tokens, 8 / 2 /
// 2 heads: 12.5 -> 6.5 us, and turned back 10.0 -> 5.0), of large ones the smaller parts fill the ends of the larger one.  No
// transposed copies of q and k (8192 tokens, 32 / 8 / 8 heads: with them 67 us, this 37.6; back 51.7 -> 46.2).
template <bool V>
__global__ __launch_bounds__(kBlkThreads) void rope_parts_kernel(const RopePart q, const RopePart k, const RopePart v, int64_t rows, int hd, int64_t S,
                                                                 float sign, const RopeFreq fr, uint32_t* __restrict__ amax_bits)
{
    __shared__ uint16_t tile[V ? kRt * kRtStride : 1];
    if (V && blockIdx.x >= q.blocks + k.blocks) {
        rope_tile_work<false, false, true>(v, blockIdx.x - q.blocks - k.blocks, rows, hd, S, sign, fr, nullptr, tile);
    } else {
        const bool second = blockIdx.x >= q.blocks;
        rope_tile_work<true, true, false>(second ? k : q, blockIdx.x - (second ? q.blocks : 0), rows, hd, S, sign, fr, amax_bits, tile);
    }
}


__global__ __launch_bounds__(kBlkThreads) void add_kernel(const uint4* __restrict__ a, const uint4* __restrict__ b, int64_t n,
                                                          uint4* __restrict__ out)
{
    for (int64_t c = (int64_t)blockIdx.x * kBlkThreads + threadIdx.x; c < n; c += (int64_t)gridDim.x * kBlkThreads) {
        const uint4 u = a[c], v = b[c];
        out[c] = make_uint4(add_word(u.x, v.x), add_word(u.y, v.y), add_word(u.z, v.z), add_word(u.w, v.w));
    }
}

// ---- RMSNorm backward ---------------------------------------------------------------------
//   y = x * r * g, r = rsqrt(mean(x^2) + eps):
//   dx = r * (g . dy) - x * r^3 * mean(x . g . dy),   dg = sum over rows of dy . x * r

__device__ inline float xgd_word(uint32_t x, uint32_t g, uint32_t d)
{
    return bf16_lo(x) * (bf16_lo(g) * bf16_lo(d)) + bf16_hi(x) * (bf16_hi(g) * bf16_hi(d));
}
__device__ inline uint32_t dx_word(uint32_t x, uint32_t g, uint32_t d, float r, float k)
{
    return pack_bf16(r * (bf16_lo(g) * bf16_lo(d)) - bf16_lo(x) * k, r * (bf16_hi(g) * bf16_hi(d)) - bf16_hi(x) * k);
}

// one wave per row.  NC > 0: at most NC 16-byte chunks per lane, x and dy are kept in registers
// between the two passes; NC = 0: any row length, the rows are read twice (second time from the caches)
template <int NC>
__global__ __launch_bounds__(kBlkThreads) void rmsnorm_dx_kernel(const uint4* __restrict__ x, const uint4* __restrict__ g,
                                                                 const float* __restrict__ rstd, const uint4* __restrict__ dy,
                                                                 int64_t M, int64_t dc, float inv_d, uint4* __restrict__ dx,
                                                                 const uint4* __restrict__ res /* nullable: added to dx */,
                                                                 uint32_t* __restrict__ amax_bits /* nullable: max-updated */)
{
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint32_t mag = 0;
    for (int64_t m = (int64_t)blockIdx.x * kBlkWaves + wave; m < M; m += (int64_t)gridDim.x * kBlkWaves) {
        const uint4 *xr = x + m * dc, *dr = dy + m * dc;
        float t = 0.0f;
        uint4 kx[NC > 0 ? NC : 1], kd[NC > 0 ? NC : 1];
        auto term = [&](uint4 v, uint4 w, uint4 d) {
            return (xgd_word(v.x, w.x, d.x) + xgd_word(v.y, w.y, d.y)) + (xgd_word(v.z, w.z, d.z) + xgd_word(v.w, w.w, d.w));
        };
        if constexpr (NC > 0) {
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                const int64_t c = lane + (int64_t)kWave * i;
                kx[i] = c < dc ? xr[c] : make_uint4(0, 0, 0, 0);
                kd[i] = c < dc ? dr[c] : make_uint4(0, 0, 0, 0);
                if (c < dc) t += term(kx[i], g[c], kd[i]);
            }
        } else {
            for (int64_t c = lane; c < dc; c += kWave) t += term(xr[c], g[c], dr[c]);
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off, kWave);
        const float r = rstd[m];
        const float k = ((r * r) * r) * (t * inv_d);
        auto emit = [&](int64_t c, uint4 v, uint4 d) {
            const uint4 w = g[c];
            uint4 o = make_uint4(dx_word(v.x, w.x, d.x, r, k), dx_word(v.y, w.y, d.y, r, k),
                                 dx_word(v.z, w.z, d.z, r, k), dx_word(v.w, w.w, d.w, r, k));
            if (res) {  // the residual branch's gradient: the same two roundings as f8_add after this call
                const uint4 a = res[m * dc + c];
                o = make_uint4(add_word(a.x, o.x), add_word(a.y, o.y), add_word(a.z, o.z), add_word(a.w, o.w));
            }
            dx[m * dc + c] = o;
            mag = absmax_acc(mag, o);
        };
        if constexpr (NC > 0) {
#pragma unroll
            for (int i = 0; i < NC; ++i) {
                const int64_t c = lane + (int64_t)kWave * i;
                if (c < dc) emit(c, kx[i], kd[i]);
            }
        } else {
            for (int64_t c = lane; c < dc; c += kWave) emit(c, xr[c], dr[c]);
        }
    }
    if (amax_bits) {
        const uint32_t m = wave_max_u32(pk_collapse(mag)) << 16;
        if (lane == 0 && m > __atomic_load_n(amax_bits, __ATOMIC_RELAXED)) atomicMax(amax_bits, m);
    }
}

// dx and dg from one read of x and dy (D up to 1024): a wave walks rows and keeps, beside the row, the sums of
// dy * x * rstd of its own rows for its columns in registers; the block's four sets meet in LDS and leave one
// partial row, partial[block][D].  NC: 16-byte chunks of a row per lane, so that a short row pays for no more
// registers, LDS and chunks than it has (2048 x 512 with eight always 10.5 us, as two passes 9.2, so 8.1).
template <int NC>
__global__ __launch_bounds__(kBlkThreads, 2) void rmsnorm_bwd_fused_kernel(const uint4* __restrict__ x, const uint4* __restrict__ g,
                                                                           const float* __restrict__ rstd, const uint4* __restrict__ dy,
                                                                           int64_t M, int dc, float inv_d, uint4* __restrict__ dx,
                                                                           const uint4* __restrict__ res /* nullable: added to dx */,
                                                                           float* __restrict__ partial,
                                                                           uint32_t* __restrict__ amax_bits /* nullable: max-updated */)
{
    __shared__ float sum[kBlkWaves][NC * kWave * 8];
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    uint32_t mag = 0;
    float acc[NC][8];
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) acc[i][j] = 0.0f;
    for (int64_t m = (int64_t)blockIdx.x * kBlkWaves + wave; m < M; m += (int64_t)gridDim.x * kBlkWaves) {
        const uint4 *xr = x + m * dc, *dr = dy + m * dc;
        uint4 kx[NC], kd[NC];
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const int c = lane + kWave * i;
            kx[i] = c < dc ? xr[c] : make_uint4(0, 0, 0, 0);
            kd[i] = c < dc ? dr[c] : make_uint4(0, 0, 0, 0);
        }
        const float r = rstd[m];
        float t = 0.0f;
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const int c = lane + kWave * i;
            if (c < dc) {
                const uint4 v = kx[i], w = g[c], d = kd[i];
                t += (xgd_word(v.x, w.x, d.x) + xgd_word(v.y, w.y, d.y)) + (xgd_word(v.z, w.z, d.z) + xgd_word(v.w, w.w, d.w));
            }
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off, kWave);
        const float k = ((r * r) * r) * (t * inv_d);
#pragma unroll
        for (int i = 0; i < NC; ++i) {
            const int c = lane + kWave * i;
            const uint32_t vw[4] = {kx[i].x, kx[i].y, kx[i].z, kx[i].w}, dw[4] = {kd[i].x, kd[i].y, kd[i].z, kd[i].w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[i][2 * j] += bf16_lo(dw[j]) * (bf16_lo(vw[j]) * r);
                acc[i][2 * j + 1] += bf16_hi(dw[j]) * (bf16_hi(vw[j]) * r);
            }
            if (c < dc) {
                const uint4 v = kx[i], w = g[c], d = kd[i];
                uint4 o = make_uint4(dx_word(v.x, w.x, d.x, r, k), dx_word(v.y, w.y, d.y, r, k), dx_word(v.z, w.z, d.z, r, k),
                                     dx_word(v.w, w.w, d.w, r, k));
                if (res) {
                    const uint4 a = res[m * dc + c];
                    o = make_uint4(add_word(a.x, o.x), add_word(a.y, o.y), add_word(a.z, o.z), add_word(a.w, o.w));
                }
                dx[m * dc + c] = o;
                mag = absmax_acc(mag, o);
            }
        }
    }
#pragma unroll
    for (int i = 0; i < NC; ++i)
#pragma unroll
        for (int j = 0; j < 8; ++j) sum[wave][(i * 8 + j) * kWave + lane] = acc[i][j];
    __syncthreads();
    // thread (i, lane) adds the four waves' sums of its chunks in wave order
    for (int i = wave; i < NC; i += kBlkWaves) {
        const int c = lane + kWave * i;
        if (c >= dc) continue;
        float s[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int at = (i * 8 + j) * kWave + lane;
            s[j] = ((sum[0][at] + sum[1][at]) + sum[2][at]) + sum[3][at];
        }
        float4* out = reinterpret_cast<float4*>(partial + (int64_t)blockIdx.x * dc * 8 + c * 8);
        out[0] = make_float4(s[0], s[1], s[2], s[3]);
        out[1] = make_float4(s[4], s[5], s[6], s[7]);
    }
    if (amax_bits) {
        const uint32_t m = wave_max_u32(pk_collapse(mag)) << 16;
        if (lane == 0 && m > __atomic_load_n(amax_bits, __ATOMIC_RELAXED)) atomicMax(amax_bits, m);
    }
}

// The same for rows of 1040 to 8192 elements, a row per block: thread t has chunks t, t + 256, ... of it (U of them).
// Bound by memory.  With a row per wave a lane holds eight chunks of x and dy and 64 sums, which leaves no registers to
// request the next row with, and all waves load, then compute, then store: 8192 x 4096 with the residual 82 us (268 MB).
// A quarter of that per lane lets the next row be on its way while this one is worked on: 52 us; 1008 x 4096 20.8 -> 12.7,
// 1008 x 2048 11.7 -> 10.0, 8192 x 6144 (two passes before) 144 -> 89.  Shorter rows would leave threads without a chunk.
// Loads and stores past the caches at every size: both calls of a transformer block together, past / through them, 36 / 47 us
// for 2048 x 2048, 36 / 39 for 1008 x 2048, 65 / 68 for 4096 x 4096, 107 / 113 for 8192 x 4096, but 54 / 50 for 2048 x 4096.
// The sum over a row is formed by every wave from the chunks' terms in LDS, in the order in which a lane of the kernel
// above adds them, and the block takes that kernel's rows wave by wave: the same bits, of dx and of dg.
template <int U>
__global__ __launch_bounds__(kBlkThreads, 2) void rmsnorm_bwd_row_kernel(const uint4* __restrict__ x, const uint4* __restrict__ g,
                                                                      const float* __restrict__ rstd, const uint4* __restrict__ dy,
                                                                      int64_t M, int dc, float inv_d, uint4* __restrict__ dx,
                                                                      const uint4* __restrict__ res /* nullable: added to dx */,
                                                                      float* __restrict__ partial,
                                                                      uint32_t* __restrict__ amax_bits /* nullable: max-updated */)
{
    __shared__ float terms[2][kBlkWaves * U][kWave];  // of x . g . dy, by chunk / 64 and chunk % 64; of this row and the next
    const int lane = threadIdx.x & (kWave - 1), wave = threadIdx.x / kWave;
    const int64_t step = (int64_t)gridDim.x * kBlkWaves;
    uint32_t mag = 0;
    float acc[U][8] = {}, sum[U][8] = {};
    uint4 gw[U];
    bool in[U];
    struct Row {
        uint4 x[U], d[U], a[U];
        float r;
    };
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int c = (int)threadIdx.x + kBlkThreads * u;
        in[u] = c < dc;
        gw[u] = in[u] ? g[c] : make_uint4(0, 0, 0, 0);
    }
    auto request = [&](int64_t m) {
        Row row;
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int64_t at = m * dc + threadIdx.x + kBlkThreads * u;
            row.x[u] = row.d[u] = row.a[u] = make_uint4(0, 0, 0, 0);
            if (in[u]) {
                row.x[u] = load_once(x + at), row.d[u] = load_once(dy + at);
                if (res) row.a[u] = load_once(res + at);
            }
        }
        row.r = rstd[m];
        return row;
    };
    int w = 0, buf = 0;
    int64_t m = (int64_t)blockIdx.x * kBlkWaves;
    Row row = request(m);
    while (true) {
        // the row after this one: of wave w of the kernel above, then of the next wave
        int nw = w;
        int64_t nm = m + step;
        if (nm >= M) nw = w + 1, nm = (int64_t)blockIdx.x * kBlkWaves + nw;
        const bool more = nw < kBlkWaves && nm < M;
        Row next = row;
        if (more) next = request(nm);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint4 v = row.x[u], k = gw[u], d = row.d[u];
            terms[buf][wave + kBlkWaves * u][lane] =
                (xgd_word(v.x, k.x, d.x) + xgd_word(v.y, k.y, d.y)) + (xgd_word(v.z, k.z, d.z) + xgd_word(v.w, k.w, d.w));
        }
        __syncthreads();
        float t = 0.0f;
#pragma unroll
        for (int i = 0; i < kBlkWaves * U; ++i) t += terms[buf][i][lane];
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) t += __shfl_xor(t, off, kWave);
        const float r = row.r, k = ((r * r) * r) * (t * inv_d);
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const uint4 v = row.x[u], wg = gw[u], d = row.d[u], a = row.a[u];
            const uint32_t vw[4] = {v.x, v.y, v.z, v.w}, dw[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[u][2 * j] += bf16_lo(dw[j]) * (bf16_lo(vw[j]) * r);
                acc[u][2 * j + 1] += bf16_hi(dw[j]) * (bf16_hi(vw[j]) * r);
            }
            uint4 o = make_uint4(dx_word(v.x, wg.x, d.x, r, k), dx_word(v.y, wg.y, d.y, r, k), dx_word(v.z, wg.z, d.z, r, k),
                                 dx_word(v.w, wg.w, d.w, r, k));
            if (res) o = make_uint4(add_word(a.x, o.x), add_word(a.y, o.y), add_word(a.z, o.z), add_word(a.w, o.w));
            if (in[u]) {
                store_stream(dx + m * dc + threadIdx.x + kBlkThreads * u, o);
                mag = absmax_acc(mag, o);
            }
        }
        if (nw != w || !more) {  // the waves' sums in wave order
#pragma unroll
            for (int u = 0; u < U; ++u)
#pragma unroll
                for (int j = 0; j < 8; ++j) sum[u][j] = w == 0 ? acc[u][j] : sum[u][j] + acc[u][j], acc[u][j] = 0.0f;
        }
        if (!more) break;
        m = nm, w = nw, row = next, buf ^= 1;
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (!in[u]) continue;
        float4* out = reinterpret_cast<float4*>(partial + ((int64_t)blockIdx.x * dc + threadIdx.x + kBlkThreads * u) * 8);
        out[0] = make_float4(sum[u][0], sum[u][1], sum[u][2], sum[u][3]);
        out[1] = make_float4(sum[u][4], sum[u][5], sum[u][6], sum[u][7]);
    }
    if (amax_bits) {
        const uint32_t mx = wave_max_u32(pk_collapse(mag)) << 16;
        if (lane == 0 && mx > __atomic_load_n(amax_bits, __ATOMIC_RELAXED)) atomicMax(amax_bits, mx);
    }
}

// dg alone, with the sums of rmsnorm_bwd_fused_kernel and rmsnorm_dg_final_kernel in their order.  No sum over a row is
// needed here, so the rows are cut into pieces of 64 columns, and of a piece one block takes every sixteenth of the
// fused kernel's row blocks: what one of the final kernel's groups adds, which leaves 16 partial rows (read as if by
// one block each) instead of up to 512.  Thread (cl, w, rl): 8 columns of wave w's rows of row block part + 16 rl.
// 1008 x 4096 6.6 us, 2048 x 4096 9.8, 8192 x 4096 25; by the fused kernel 13, 18 and 39, as strips of rows (below) 6.4, 10.7
// and 28.
constexpr int kFinalGroups = 16;  // of the final kernel
constexpr int kDgParts = kFinalGroups, kDgPieces = 8 /* of 16 bytes */, kRowBlocks = 512;
static_assert(2 * kDgPieces * kBlkWaves == kWave, "a wave holds two row blocks");
__global__ __launch_bounds__(kDgPieces* kBlkWaves*(kRowBlocks / kDgParts)) void rmsnorm_dg_only_kernel(
    const uint4* __restrict__ x, const float* __restrict__ rstd, const uint4* __restrict__ dy, int64_t M, int dc, int row_blocks,
    float* __restrict__ partial, int parts)
{
    __shared__ float sum[kRowBlocks / kDgParts][kBlkWaves][kDgPieces * 8];
    const int cl = threadIdx.x % kDgPieces, w = threadIdx.x / kDgPieces % kBlkWaves, rl = threadIdx.x / (kDgPieces * kBlkWaves);
    const int part = (int)(blockIdx.x % (unsigned)parts), c0 = (int)(blockIdx.x / (unsigned)parts) * kDgPieces;
    const int rb = part + kDgParts * rl, c = c0 + cl;
    float acc[8] = {};
    if (rb < row_blocks && c < dc)
        for (int64_t m = (int64_t)rb * kBlkWaves + w; m < M; m += (int64_t)row_blocks * kBlkWaves) {
            const uint4 v = x[m * dc + c], d = dy[m * dc + c];
            const float r = rstd[m];
            const uint32_t vw[4] = {v.x, v.y, v.z, v.w}, dw[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[2 * j] += bf16_lo(dw[j]) * (bf16_lo(vw[j]) * r);
                acc[2 * j + 1] += bf16_hi(dw[j]) * (bf16_hi(vw[j]) * r);
            }
        }
#pragma unroll
    for (int j = 0; j < 8; ++j) sum[rl][w][8 * cl + j] = acc[j];
    __syncthreads();
    const int col = c0 * 8 + (int)threadIdx.x;
    if (threadIdx.x >= kDgPieces * 8 || col >= dc * 8) return;
    float s = 0.0f;
    for (int i = 0; part + kDgParts * i < row_blocks; ++i)
        s += ((sum[i][0][threadIdx.x] + sum[i][1][threadIdx.x]) + sum[i][2][threadIdx.x]) + sum[i][3][threadIdx.x];
    partial[(int64_t)part * dc * 8 + col] = s;
}

// partial[strip][col] = sum over the strip's rows of dy * x * rstd.  Block: 64 columns x one strip
// of rows; thread (cc, rr) owns 8 columns and every 32nd row.
__global__ __launch_bounds__(kBlkThreads) void rmsnorm_dg_partial_kernel(const uint16_t* __restrict__ x,
                                                                         const float* __restrict__ rstd,
                                                                         const uint16_t* __restrict__ dy, int64_t M,
                                                                         int64_t D, int64_t strip_rows,
                                                                         float* __restrict__ partial, int tiles_c)
{
    __shared__ float red[32][65];
    const int64_t strip = blockIdx.x / tiles_c, c0 = (int64_t)(blockIdx.x % tiles_c) * 64;
    const int cc = threadIdx.x & 7, rr = threadIdx.x >> 3;
    const int64_t col = c0 + cc * 8;
    const int64_t rbeg = strip * strip_rows, rend = rbeg + strip_rows < M ? rbeg + strip_rows : M;
    float acc[8] = {0, 0, 0, 0, 0, 0, 0, 0};
    if (col < D) {
        for (int64_t r = rbeg + rr; r < rend; r += 32) {
            const uint4 v = *reinterpret_cast<const uint4*>(x + r * D + col);
            const uint4 d = *reinterpret_cast<const uint4*>(dy + r * D + col);
            const float rs = rstd[r];
            const uint32_t vw[4] = {v.x, v.y, v.z, v.w}, dw[4] = {d.x, d.y, d.z, d.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                acc[2 * j] += bf16_lo(dw[j]) * (bf16_lo(vw[j]) * rs);
                acc[2 * j + 1] += bf16_hi(dw[j]) * (bf16_hi(vw[j]) * rs);
            }
        }
    }
#pragma unroll
    for (int j = 0; j < 8; ++j) red[rr][cc * 8 + j] = acc[j];
    __syncthreads();
    if (threadIdx.x < 64 && c0 + threadIdx.x < D) {
        float s = 0.0f;
        for (int i = 0; i < 32; ++i) s += red[i][threadIdx.x];  // fixed order: the result is reproducible
        partial[strip * D + c0 + threadIdx.x] = s;
    }
}

// dg[c] = sum over the strips, always in the same order: 32 columns per block, sixteen groups of
// threads take every sixteenth strip each, their sums are added in group order.
constexpr int kFinalCols = 32;
__global__ __launch_bounds__(kFinalGroups * kFinalCols) void rmsnorm_dg_final_kernel(const float* __restrict__ partial, int strips, int64_t D,
                                                                       float* __restrict__ dg)
{
    __shared__ float red[kFinalGroups][kFinalCols];
    const int cl = threadIdx.x % kFinalCols, part = threadIdx.x / kFinalCols;
    const int64_t c = (int64_t)blockIdx.x * kFinalCols + cl;
    float s = 0.0f;
    if (c < D) {
        constexpr int AHEAD = 8;  // loads in flight: the sum is one chain, and its loads are what it waits for
        for (int i = part; i < strips; i += kFinalGroups * AHEAD) {
            float p[AHEAD];
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) {
                const int at = i + kFinalGroups * k;
                p[k] = at < strips ? partial[(int64_t)at * D + c] : 0.0f;
            }
#pragma unroll
            for (int k = 0; k < AHEAD; ++k) s += p[k];
        }
    }
    red[part][cl] = s;
    __syncthreads();
    if (part == 0 && c < D) {
        float v = red[0][cl];
#pragma unroll
        for (int k = 1; k < kFinalGroups; ++k) v += red[k][cl];
        dg[c] = v;
    }
}
static void launch_dg_final(const float* partial, int64_t strips, int64_t D, float* dg, hipStream_t st)
{
    rmsnorm_dg_final_kernel<<<(unsigned)((D + kFinalCols - 1) / kFinalCols), kFinalGroups * kFinalCols, 0, st>>>(partial, (int)strips, D, dg);
}

static int elementwise_blocks(int64_t chunks)
{
    int64_t b = (chunks + kBlkThreads * 2 - 1) / (kBlkThreads * 2);
    if (b < 1) b = 1;
    if (b > 4096) b = 4096;
    return (int)b;
}

// Heads per block: as many as leave about four blocks per compute unit, or, since the sines and cosines bound a
// block of few heads, two where they are taken (4000 x 16 heads: one output 12.3 -> 9.6 us, both 16.4 -> 16.1).
// `heads`: those of the whole launch.  false: too many blocks.
static bool plan_rope_part(RopePart& p, int64_t rows, int64_t hd, int64_t heads, bool rotate)
{
    const int64_t tiles_r = (rows + kRt - 1) / kRt, tph = (hd + kRt - 1) / kRt;
    int64_t hpb = (tiles_r * tph * heads) / (rotate ? 512 : 1024);
    if (hpb < 1) hpb = 1;
    if (hpb > 8) hpb = 8;
    if (hpb > p.nh) hpb = p.nh;
    const int64_t tiles_c = tph * ((p.nh + hpb - 1) / hpb), nb = tiles_r * tiles_c;
    if (nb > (int64_t)0x7FFFFFFF) return false;
    p.hpb = (int)hpb, p.tiles_c = (int)tiles_c, p.blocks = (unsigned)nb;
    return true;
}

template <bool ROTATE>
static f8_status launch_rope_tiles(const void* x, int64_t rows, int64_t nh, int64_t hd, int64_t ldx, int64_t ldo, int64_t S,
                                   float sign, const RopeFreq& fr, void* out, void* out_t, float* amax, hipStream_t st)
{
    RopePart p{(const uint16_t*)x, (uint16_t*)out, (uint16_t*)out_t, ldx, ldo, (int)nh, 0, 0, 0};
    if (!plan_rope_part(p, rows, hd, nh, ROTATE)) return F8_ERR_SHAPE;
    if (p.blocks == 0) return F8_OK;
    const auto kernel = out && out_t ? rope_tile_kernel<ROTATE, true, true> : out ? rope_tile_kernel<ROTATE, true, false> : rope_tile_kernel<ROTATE, false, true>;
    kernel<<<p.blocks, kBlkThreads, 0, st>>>(p, rows, (int)hd, S, sign, fr, reinterpret_cast<uint32_t*>(amax));
    return last_launch_status();
}

static RopeFreq rope_freq(double theta, int64_t hd)
{
    RopeFreq fr;
    for (int i = 0; i < 128; ++i) fr.f[i] = i < hd / 2 ? pow(theta, -2.0 * (double)i / (double)hd) : 0.0;
    return fr;
}

static bool rope_shape_ok(int64_t M, int64_t S, int64_t n_heads, int64_t hd, double theta, int64_t ldx)
{
    return M >= 0 && S >= 1 && n_heads >= 1 && hd >= 2 && hd <= 256 && hd % 8 == 0 && M % 8 == 0 && theta > 0.0 &&
           n_heads < ((int64_t)1 << 23) && n_heads * hd < (1 << 23) && ldx >= n_heads * hd && ldx % 8 == 0;
}

}  // namespace f8

using namespace f8;

extern "C" {

f8_status f8_rope(const void* x_bf16, int64_t ldx, int64_t M, int64_t S, int64_t n_heads, int64_t hd, double theta,
                  int inverse, void* out_bf16, int64_t ldo, void* out_t_bf16, float* amax_inout, void* stream)
{
    if (!x_bf16 || (!out_bf16 && !out_t_bf16)) return F8_ERR_NULL;
    if (!rope_shape_ok(M, S, n_heads, hd, theta, ldx) || (out_bf16 && (ldo < n_heads * hd || (ldo % 8)))) return F8_ERR_SHAPE;
    if (!aligned16(x_bf16) || (out_bf16 && !aligned16(out_bf16)) || (out_t_bf16 && !aligned16(out_t_bf16))) return F8_ERR_ALIGN;
    return launch_rope_tiles<true>(x_bf16, M, n_heads, hd, ldx, ldo, S, inverse ? -1.0f : 1.0f, rope_freq(theta, hd), out_bf16, out_t_bf16,
                                   amax_inout, (hipStream_t)stream);
}

f8_status f8_rope_qkv(const void* qkv_bf16, int64_t ldqkv, int64_t M, int64_t S, int64_t Hq, int64_t Hkv, int64_t hd, double theta,
                      void* q_bf16, int64_t ldq, void* k_bf16, int64_t ldk, void* vt_bf16, void* stream)
{
    if (!qkv_bf16 || !q_bf16 || !k_bf16 || !vt_bf16) return F8_ERR_NULL;
    if (Hq < 1 || Hkv < 1 || Hq >= (1 << 20) || Hkv >= (1 << 20) || !rope_shape_ok(M, S, Hq + 2 * Hkv, hd, theta, ldqkv)) return F8_ERR_SHAPE;
    if (ldq < Hq * hd || ldk < Hkv * hd || (ldq % 8) || (ldk % 8)) return F8_ERR_SHAPE;
    if (!aligned16(qkv_bf16) || !aligned16(q_bf16) || !aligned16(k_bf16) || !aligned16(vt_bf16)) return F8_ERR_ALIGN;
    const uint16_t* x = (const uint16_t*)qkv_bf16;
    RopePart q{x, (uint16_t*)q_bf16, nullptr, ldqkv, ldq, (int)Hq, 0, 0, 0}, k{x + Hq * hd, (uint16_t*)k_bf16, nullptr, ldqkv, ldk, (int)Hkv, 0, 0, 0},
        v{x + (Hq + Hkv) * hd, nullptr, (uint16_t*)vt_bf16, ldqkv, 0, (int)Hkv, 0, 0, 0};
    if (!plan_rope_part(q, M, hd, Hq + Hkv, true) || !plan_rope_part(k, M, hd, Hq + Hkv, true) || !plan_rope_part(v, M, hd, Hq + Hkv, true))
        return F8_ERR_SHAPE;
    const int64_t blocks = (int64_t)q.blocks + k.blocks + v.blocks;
    if (blocks > (int64_t)0x7FFFFFFF) return F8_ERR_SHAPE;
    if (blocks)
        rope_parts_kernel<true><<<(unsigned)blocks, kBlkThreads, 0, (hipStream_t)stream>>>(q, k, v, M, (int)hd, S, 1.0f, rope_freq(theta, hd), nullptr);
    return last_launch_status();
}

f8_status f8_rope_qk_bwd(const void* dq_bf16, int64_t lddq, const void* dk_bf16, int64_t lddk, int64_t M, int64_t S, int64_t Hq, int64_t Hkv,
                         int64_t hd, double theta, void* dqkv_bf16, int64_t lddqkv, float* amax_inout, void* stream)
{
    if (!dq_bf16 || !dk_bf16 || !dqkv_bf16) return F8_ERR_NULL;
    if (Hq < 1 || Hkv < 1 || Hq >= (1 << 20) || Hkv >= (1 << 20) || !rope_shape_ok(M, S, Hq + Hkv, hd, theta, lddqkv)) return F8_ERR_SHAPE;
    if (lddq < Hq * hd || lddk < Hkv * hd || (lddq % 8) || (lddk % 8)) return F8_ERR_SHAPE;
    if (!aligned16(dq_bf16) || !aligned16(dk_bf16) || !aligned16(dqkv_bf16)) return F8_ERR_ALIGN;
    uint16_t* out = (uint16_t*)dqkv_bf16;
    RopePart q{(const uint16_t*)dq_bf16, out, nullptr, lddq, lddqkv, (int)Hq, 0, 0, 0},
        k{(const uint16_t*)dk_bf16, out + Hq * hd, nullptr, lddk, lddqkv, (int)Hkv, 0, 0, 0};
    if (!plan_rope_part(q, M, hd, Hq + Hkv, true) || !plan_rope_part(k, M, hd, Hq + Hkv, true)) return F8_ERR_SHAPE;
    const int64_t blocks = (int64_t)q.blocks + k.blocks;
    if (blocks > (int64_t)0x7FFFFFFF) return F8_ERR_SHAPE;
    if (blocks)
        rope_parts_kernel<false><<<(unsigned)blocks, kBlkThreads, 0, (hipStream_t)stream>>>(q, k, k, M, (int)hd, S, -1.0f, rope_freq(theta, hd),
                                                                                            reinterpret_cast<uint32_t*>(amax_inout));
    return last_launch_status();
}

f8_status f8_transpose_bf16(const void* x_bf16, int64_t ldx, int64_t rows, int64_t cols, void* out_t_bf16, void* stream)
{
    if (!x_bf16 || !out_t_bf16) return F8_ERR_NULL;
    if (rows < 0 || cols < 0 || (rows % 8) || (cols % 8) || ldx < cols || (ldx % 8)) return F8_ERR_SHAPE;
    if (!aligned16(x_bf16) || !aligned16(out_t_bf16)) return F8_ERR_ALIGN;
    RopeFreq fr = {};
    if (cols >= ((int64_t)1 << 31)) return F8_ERR_SHAPE;
    return launch_rope_tiles<false>(x_bf16, rows, 1, cols, ldx, cols, 1, 1.0f, fr, nullptr, out_t_bf16, nullptr, (hipStream_t)stream);
}

f8_status f8_add(const void* a_bf16, const void* b_bf16, int64_t n, void* out_bf16, void* stream)
{
    if (!a_bf16 || !b_bf16 || !out_bf16) return F8_ERR_NULL;
    if (n < 0 || (n % 8)) return F8_ERR_SHAPE;
    if (!aligned16(a_bf16) || !aligned16(b_bf16) || !aligned16(out_bf16)) return F8_ERR_ALIGN;
    if (n == 0) return F8_OK;
    add_kernel<<<elementwise_blocks(n / 8), kBlkThreads, 0, (hipStream_t)stream>>>((const uint4*)a_bf16, (const uint4*)b_bf16,
                                                                                   n / 8, (uint4*)out_bf16);
    return last_launch_status();
}

static f8_status rmsnorm_bwd(const void* x_bf16, const void* g_bf16, const float* rstd, const void* dy_bf16, const void* add_bf16,
                             int64_t M, int64_t D, void* dx_bf16, float* dg, float* amax_dx, void* workspace,
                             size_t workspace_bytes_, void* stream)
{
    if (!x_bf16 || !g_bf16 || !rstd || !dy_bf16 || (!dx_bf16 && !dg)) return F8_ERR_NULL;
    if (M < 0 || D < 0 || (M % 16) || (D % 16)) return F8_ERR_SHAPE;
    if (!aligned16(x_bf16) || !aligned16(g_bf16) || !aligned16(dy_bf16) || (dx_bf16 && !aligned16(dx_bf16))) return F8_ERR_ALIGN;
    // at most 64 strips of rows, each a multiple of 32 rows
    int64_t strip_rows = ((M + 63) / 64 + 31) / 32 * 32;
    if (strip_rows < 32) strip_rows = 32;
    const int64_t strips = M ? (M + strip_rows - 1) / strip_rows : 0;
    if (dg && (!workspace || workspace_bytes_ < (size_t)(strips * D) * sizeof(float))) return F8_ERR_WORKSPACE;
    hipStream_t st = (hipStream_t)stream;
    if (D == 0) return F8_OK;
    // One pass where a row fits the registers of a block and the workspace holds a partial row of every block (two per
    // compute unit; f8_workspace_bytes always does from 16 rows on, a caller's smaller one may not).
    const int64_t blocks = (M + kBlkWaves - 1) / kBlkWaves < kRowBlocks ? (M + kBlkWaves - 1) / kBlkWaves : kRowBlocks;
    // dg alone of rows above 4096 elements is faster as strips of rows, below (us: 2048 x 4608 11.1 against 13.1, 2048 x 8192
    // 17.5 / 21.3, 64 x 8192 4.5 / 5.2).
    if (dg && M && D <= 8 * kBlkThreads * (dx_bf16 ? 4 : 2) && aligned16(workspace) && workspace_bytes_ >= (size_t)(blocks * D) * sizeof(float)) {
        const int dc = (int)(D / 8), chunks = (dc + kWave - 1) / kWave;  // 16-byte chunks of a row, in all and per lane
        int strips = (int)blocks;
        if (dx_bf16) {
            const auto kernel = chunks == 1   ? rmsnorm_bwd_fused_kernel<1>
                                : chunks == 2 ? rmsnorm_bwd_fused_kernel<2>
                                : chunks <= 4 ? rmsnorm_bwd_row_kernel<1>
                                : chunks <= 8 ? rmsnorm_bwd_row_kernel<2>
                                : chunks <= 12 ? rmsnorm_bwd_row_kernel<3>
                                              : rmsnorm_bwd_row_kernel<4>;
            kernel<<<(unsigned)blocks, kBlkThreads, 0, st>>>((const uint4*)x_bf16, (const uint4*)g_bf16, rstd, (const uint4*)dy_bf16, M, dc,
                                                             1.0f / (float)D, (uint4*)dx_bf16, (const uint4*)add_bf16,
                                                             (float*)workspace, reinterpret_cast<uint32_t*>(amax_dx));
        } else {
            strips = blocks < kDgParts ? (int)blocks : kDgParts;
            const unsigned dg_threads = (unsigned)((blocks + 2 * kDgParts - 1) / (2 * kDgParts)) * 2 * kDgPieces * kBlkWaves;  // whole waves
            rmsnorm_dg_only_kernel<<<(unsigned)(strips * ((dc + kDgPieces - 1) / kDgPieces)), dg_threads, 0, st>>>(
                (const uint4*)x_bf16, rstd, (const uint4*)dy_bf16, M, dc, (int)blocks, (float*)workspace, strips);
        }
        launch_dg_final((const float*)workspace, strips, D, dg, st);
        return last_launch_status();
    }
    if (dx_bf16 && M) {
        int64_t nb = (M + kBlkWaves - 1) / kBlkWaves;
        if (nb > 8192) nb = 8192;
#define F8_DX_LAUNCH(NC)                                                                                      \
    rmsnorm_dx_kernel<NC><<<(unsigned)nb, kBlkThreads, 0, st>>>((const uint4*)x_bf16, (const uint4*)g_bf16, rstd, \
                                                                (const uint4*)dy_bf16, M, D / 8, 1.0f / (float)D, (uint4*)dx_bf16, \
                                                                (const uint4*)add_bf16, reinterpret_cast<uint32_t*>(amax_dx))
        if (D <= 8 * kWave * 8) F8_DX_LAUNCH(8);  // rows up to 4096 elements stay in registers
        else F8_DX_LAUNCH(0);
#undef F8_DX_LAUNCH
    }
    if (dg) {
        const int64_t tiles_c = (D + 63) / 64;
        if (strips * tiles_c > (int64_t)0x7FFFFFFF) return F8_ERR_SHAPE;
        if (strips)
            rmsnorm_dg_partial_kernel<<<(unsigned)(strips * tiles_c), kBlkThreads, 0, st>>>(
                (const uint16_t*)x_bf16, rstd, (const uint16_t*)dy_bf16, M, D, strip_rows, (float*)workspace, (int)tiles_c);
        launch_dg_final((const float*)workspace, strips, D, dg, st);
    }
    return last_launch_status();
}

f8_status f8_rmsnorm_bwd(const void* x_bf16, const void* g_bf16, const float* rstd, const void* dy_bf16, int64_t M,
                         int64_t D, void* dx_bf16, float* dg, void* workspace, size_t workspace_bytes_, void* stream)
{
    return rmsnorm_bwd(x_bf16, g_bf16, rstd, dy_bf16, nullptr, M, D, dx_bf16, dg, nullptr, workspace, workspace_bytes_, stream);
}

f8_status f8_rmsnorm_bwd_add(const void* x_bf16, const void* g_bf16, const float* rstd, const void* dy_bf16,
                             const void* add_bf16, int64_t M, int64_t D, void* dx_bf16, float* dg, float* amax_dx_inout,
                             void* workspace, size_t workspace_bytes_, void* stream)
{
    if (!add_bf16 || !dx_bf16) return F8_ERR_NULL;
    if (!aligned16(add_bf16)) return F8_ERR_ALIGN;
    return rmsnorm_bwd(x_bf16, g_bf16, rstd, dy_bf16, add_bf16, M, D, dx_bf16, dg, amax_dx_inout, workspace, workspace_bytes_,
                       stream);
}

}  // extern "C"

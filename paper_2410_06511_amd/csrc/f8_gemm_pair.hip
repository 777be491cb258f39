// Both products of a linear's backward in ONE launch: dX [M,K] = dY . W and dW [N,K] = dY^T . X.  The build compiles this
// file once per format of dY and granularity (-DF8_PAIR_FA=<0|1>, -DF8_PAIR_GRAN=<F8_TENSORWISE | F8_ROWWISE>).
#if !defined(F8_PAIR_FA) || !defined(F8_PAIR_GRAN)
#error "compile with -DF8_PAIR_FA=, -DF8_PAIR_GRAN= (see build.py)"
#endif
#include "f8_gemm_kernels.hpp"

namespace f8 {

// One product as its kernel takes it
struct PairSide {
    const uint8_t *A, *B;
    uint16_t* D;
    int M, N, K;
    int64_t lda, ldb, ldd;
    const float *isa, *isb;
    int tiles_m, tiles_n, ksteps;
};

// The XCDs share the products: those below x_xcds work on dX, the others on dW, each XCD as it would in a launch of its
// own (one product's tiles in its L2).  Rowwise codes are read row-major in both products, tensorwise ones where they lie.
template <int BM, int BN, int FA, int GRAN, bool RAGGED, bool AMAX>
__global__ __launch_bounds__(256) void gemm_pair_kernel(const PairSide x, const PairSide w, int x_xcds,
                                                        uint32_t* __restrict__ amax_bits /* AMAX: of dX */)
{
    __shared__ __attribute__((aligned(1024))) uint8_t st0[TileLds<BM, BN>::kStage];
    __shared__ __attribute__((aligned(1024))) uint8_t st1[TileLds<BM, BN>::kStage];
    __shared__ __attribute__((aligned(16))) uint8_t epb[TileLds<BM, BN>::kEpilogue];
    constexpr bool KM = GRAN == F8_TENSORWISE;
    const int xcd = (int)blockIdx.x % kXcds, idx = (int)blockIdx.x / kXcds, per_xcd = (int)gridDim.x / kXcds;
    if (xcd < x_xcds) {
        const int first = idx * x_xcds + xcd;
        if (first >= x.tiles_m * x.tiles_n) return;
        gemm_tile_work<BM, BN, 2, 2, FA, F8_E4M3, GRAN, AMAX, false, KM, false, RAGGED>(
            x.A, x.B, x.D, x.M, x.N, x.K, x.lda, x.ldb, x.ldd, x.isa, x.isb, x.tiles_m, x.tiles_n, amax_bits, x.ksteps, 1,
            nullptr, 0, first, per_xcd * x_xcds, x_xcds, st0, st1, epb);
    } else {
        const int xcds = kXcds - x_xcds, first = idx * xcds + (xcd - x_xcds);
        if (first >= w.tiles_m * w.tiles_n) return;
        gemm_tile_work<BM, BN, 2, 2, FA, F8_E4M3, GRAN, false, KM, KM, false, RAGGED>(
            w.A, w.B, w.D, w.M, w.N, w.K, w.lda, w.ldb, w.ldd, w.isa, w.isb, w.tiles_m, w.tiles_n, nullptr, w.ksteps, 1,
            nullptr, 0, first, per_xcd * xcds, xcds, st0, st1, epb);
    }
}

template <int FA, int GRAN>
__global__ __launch_bounds__(256) void gemm_small_pair_kernel(const PairSide x, const PairSide w,
                                                              uint32_t* __restrict__ amax_bits /* nullable: of dX */)
{
    __shared__ __attribute__((aligned(1024))) uint8_t st[4][2][2 * kSmOp];
    constexpr bool KM = GRAN == F8_TENSORWISE;
    const int nx = x.tiles_m * x.tiles_n;
    if ((int)blockIdx.x < nx)
        gemm_small_work<FA, F8_E4M3, GRAN, false, KM, 4>(x.A, x.B, x.D, x.M, x.N, x.K, x.lda, x.ldb, x.ldd, x.isa, x.isb,
                                                         x.tiles_m, x.tiles_n, amax_bits, (int)blockIdx.x, st);
    else
        gemm_small_work<FA, F8_E4M3, GRAN, KM, KM, 4>(w.A, w.B, w.D, w.M, w.N, w.K, w.lda, w.ldb, w.ldd, w.isa, w.isb,
                                                      w.tiles_m, w.tiles_n, nullptr, (int)blockIdx.x - nx, st);
}

template <int BM, int BN, int FA, int GRAN>
static void launch_pair(PairSide x, PairSide w, int x_xcds, uint32_t* amax_bits, int cus, hipStream_t st)
{
    for (PairSide* s : {&x, &w}) s->tiles_m = (s->M + BM - 1) / BM, s->tiles_n = (s->N + BN - 1) / BN, s->ksteps = ksteps_of(s->K, 1);
    const bool ragged = x.K % (2 * kBK) != 0 || w.K % (2 * kBK) != 0;
    const unsigned grid = (unsigned)(BM * BN == 128 * 128 ? 2 * cus : cus);  // two workgroups of 128 x 128 tiles fit a compute unit
    auto kernel = ragged ? gemm_pair_kernel<BM, BN, FA, GRAN, true, false> : gemm_pair_kernel<BM, BN, FA, GRAN, false, false>;
    if constexpr (GRAN == F8_TENSORWISE)
        if (amax_bits) kernel = ragged ? gemm_pair_kernel<BM, BN, FA, GRAN, true, true> : gemm_pair_kernel<BM, BN, FA, GRAN, false, true>;
    kernel<<<grid, 256, 0, st>>>(x, w, x_xcds, amax_bits);
}

// ---------------------------------------------------------------------------
// one launch or two
// ---------------------------------------------------------------------------
// Estimates in us, fitted to 236 backward passes of random linears (128 .. 16384 tokens, both granularities), each in one
// launch in every way below and in two, and good to about 10 % each: a launch, its rounds of tiles, and per tile its K
// steps and its epilogue.
struct TileTime {
    double step, epilogue;
    double tile(int k) const { return ksteps_of(k, 1) * step + epilogue; }
};
constexpr TileTime kFullTime{1.04, 7.9}, kHalfTime{0.70, 2.95}, kSmallTime{0.256, 1.9};

// 128 x 128 tiles, two on a compute unit at once where it has more than one
static double quarter_us(int64_t per_cu, int k, double alone, double two, double epilogue)
{
    const int steps = ksteps_of(k, 1);
    return (double)(per_cu / 2) * (steps * two + epilogue) + (double)(per_cu % 2) * (steps * alone + epilogue);
}
static int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
static int64_t tile_count(const PairSide& s, int bm, int bn) { return ceil_div(s.M, bm) * ceil_div(s.N, bn); }

static double alone_us(const PairSide& s, bool b_kmajor, bool may_split, size_t ws_bytes, int cus, double launch)
{
    const TilePlan p = plan_product(s.M, s.N, s.K, b_kmajor, false, may_split, ws_bytes, cus);
    switch (p.kind) {
        case TilePlan::kSmall: return 4.65 + ksteps_of(s.K, 1) * 0.244;
        case TilePlan::kSmallOnePair: return 4.65;
        case TilePlan::kSplit:  // and the pass that adds the ranges
            return 2 * launch + ksteps_of(s.K, p.ranges) * kFullTime.step + kFullTime.epilogue + (p.ranges + 0.5) * s.M * s.N * 4.0 / 5.0e6;
        case TilePlan::kFull: return launch + ceil_div((int64_t)p.tm * p.tn, cus) * kFullTime.tile(s.K);
        case TilePlan::kFullRows:
        case TilePlan::kFullCols: return 2 * launch + p.whole / cus * kFullTime.tile(s.K) + kHalfTime.tile(s.K);
        case TilePlan::kHalf: return launch + ceil_div(tile_count(s, 256, 128), cus) * kHalfTime.tile(s.K);
        case TilePlan::kQuarter: break;
    }
    return launch + quarter_us(ceil_div(tile_count(s, 128, 128), cus), s.K, 0.49, 2.5, 0.6);
}

struct PairChoice {
    int tile;    // 64, 128, 192 (256 x 128) or 256; 0: two launches
    int x_xcds;  // XCDs that work on dX (not with 64)
};

// A second set of estimates, fitted to whole passes (forward, backward and casts, tensorwise) of 144 random linears, each in
// one launch in every way and in two: within a pass a launch begins while the one before it ends, the epilogues of two 128 x
// 128 tiles on a unit hide behind each other, and the separate launches fare 0.81 times what they are above.  They rank the
// ways and are no times of a kernel: large products take longer under the lowered clock (8192 x 3584 x 8192 in one launch
// 236 us by them, 375 in a trace), and a K step of 256 x 256 tiles is less here than the matrix pipe's 0.85 us, the rest of
// it in other terms.  Beyond 64 K steps the smaller tiles' workgroups drift apart and share less in the L2 (2048 x 4096 with
// 64 / 128 steps of 128 x 128 tiles: 0.8 / 1.33 us a step).
static double in_pass_us(const PairSide& x, const PairSide& w, PairChoice c, double separately, int cus)
{
    constexpr TileTime kFull{0.82, 5.3}, kHalf{0.56, 2.3}, kQuarter{0.435, 0.52}, kQuarterTwo{0.63, 1.46}, kSmall{0.265, 1.16};
    if (!c.tile) return 0.81 * separately;
    auto drifting = [](TileTime t, int k) {
        const int steps = ksteps_of(k, 1);
        return t.tile(k) + (steps > 64 ? 0.3 * (steps - 64) * t.step : 0.0);
    };
    if (c.tile == kSm) {
        const double tx = kSmall.tile(x.K), tw = kSmall.tile(w.K), longest = tx > tw ? tx : tw;
        const double work = (tile_count(x, kSm, kSm) * tx + tile_count(w, kSm, kSm) * tw) / cus + 0.15 * longest;
        return 4.5 + (work > longest ? work : longest);
    }
    auto side_us = [&](const PairSide& s, int xcds) {
        const int64_t units = (int64_t)(cus / kXcds) * xcds;
        if (c.tile == 256) return ceil_div(tile_count(s, 256, 256), units) * kFull.tile(s.K);
        if (c.tile == 192) return ceil_div(tile_count(s, 256, 128), units) * drifting(kHalf, s.K);
        const int64_t n = ceil_div(tile_count(s, 128, 128), units);
        return (double)(n / 2) * drifting(kQuarterTwo, s.K) + (double)(n % 2) * kQuarter.tile(s.K);
    };
    const double tx = side_us(x, c.x_xcds), tw = side_us(w, kXcds - c.x_xcds);
    return (c.tile == 256 ? 5.3 : c.tile == 192 ? 3.0 : 3.5) + (tx > tw ? tx : tw);
}

#define F8_PAIR_NAME_(what, fa, g) gemm_pair_##what##fa##_##g
#define F8_PAIR_NAME(what, fa, g) F8_PAIR_NAME_(what, fa, g)

// One launch where it is estimated to be enough faster than the separate ones.  dX and dW have the same number of
// operations, so an even division of the XCDs is mostly right (others are taken only for 3 % more); it is the rounds of
// tiles that decide: 896 tiles are 3.5 rounds of a whole chip, but 7 of half of it, and the two products' epilogues
// (67 MB of dX in 14 us for 8192 x 4096) overlap with each other's arithmetic.  Over those 236 passes this rule gave 1.13
// in the mean (the best choice at hand each time: 1.157).  us of a backward, two launches / one: 256 x 512 x 1024 (tokens,
// inputs, outputs) 15.4 / 12.7, 8192 x 4096 x 1024 101 / 78, 2000 x 4096 x 4096 72 / 67, 8192 x 4096 x 6144 354 / 322,
// 16384 x 4096 x 14336 1459 / 1441.  The margin is 0.985 for the tiles that large separate launches have too, 0.95 for the
// others (with less, 192 x 2176 x 11648 takes 1.09 times as long).  Where no round is saved there is little to gain: rowwise
// 8192 x 16384 x 2048 would be 3 % slower.
// An amax of dX (tensorwise scaling only) changes nothing in the rule: separately dW may be split, and its sums are then in
// another order.
PairChoice F8_PAIR_NAME(choice_, F8_PAIR_FA, F8_PAIR_GRAN)(int M, int K, int N, bool may_split, size_t ws_bytes, int cus)
{
    PairSide x{}, w{};
    x.M = M, x.N = K, x.K = N, w.M = N, w.N = K, w.K = M;
    const int per_xcd = cus / kXcds;
    constexpr bool KM = F8_PAIR_GRAN == F8_TENSORWISE;
    auto separately = [&](double launch) {
        return alone_us(x, KM, false, 0, cus, launch) + alone_us(w, KM, may_split, ws_bytes, cus, launch);
    };
    // Where the products take long, a launch hides behind the one before it and saves nothing by itself.
    double apart = separately(4.5);
    const bool hidden = apart > 200.0;
    if (hidden) apart = separately(0.0);
    // Smaller tiles than 256 x 256 need more of the L2 per product: not with more than two rounds of work.
    const bool few = tile_count(x, 256, 256) + tile_count(w, 256, 256) <= 2 * cus;

    double best = apart;
    PairChoice c{0, 0};
    // 64 x 64 tiles, several rounds of them if need be: the other tiles' larger areas leave more of the chip idle.
    const int64_t small = tile_count(x, kSm, kSm) + tile_count(w, kSm, kSm);
    if (small <= 4 * cus) {
        const double tx = kSmallTime.tile(x.K), tw = kSmallTime.tile(w.K), longest = tx > tw ? tx : tw;
        const double work = (tile_count(x, kSm, kSm) * tx + tile_count(w, kSm, kSm) * tw) / cus + 0.22 * longest;
        const double us = 4.8 + (work > longest ? work : longest);
        if (us < 0.95 * best) best = us / 0.95, c.tile = kSm;
    }
    for (int xc : {4, 3, 5}) {
        auto side_us = [&](const PairSide& s, int xcds, int t) {
            const int64_t units = (int64_t)per_xcd * xcds;
            if (t == 256) return ceil_div(tile_count(s, 256, 256), units) * kFullTime.tile(s.K);
            if (t == 192) return ceil_div(tile_count(s, 256, 128), units) * kHalfTime.tile(s.K);
            return quarter_us(ceil_div(tile_count(s, 128, 128), units), s.K, 0.46, 1.13, 2.8);
        };
        for (int t : {256, 192, 128}) {  // 192: 256 x 128
            if (t != 256 && !few) continue;
            const double tx = side_us(x, xc, t), tw = side_us(w, kXcds - xc, t), launch = hidden ? 0.0 : t == 256 ? 2.5 : t == 192 ? 3.5 : 3.9;
            const double margin = (t == 256 ? 0.985 : 0.95) / (xc == 4 ? 1.0 : 1.03);
            const double us = (launch + (tx > tw ? tx : tw)) / margin;
            if (us < best) best = us, c = PairChoice{t, xc};
        }
    }
    // The estimates within a pass have the last word where the above stays with two launches (it takes no tiles below 256 x
    // 256 beyond two rounds of work, and knows no overlap), and choose between the ways of one launch, where they see 8 us or
    // more; up to five rounds of work, as far as they hold (512 x 15040 x 12800 rowwise by them 663 -> 827), and not for less
    // than a tile's rows of tokens or outputs (160 x 12800 x 3584 109 -> 116).  How much they have to see, by 1500 random
    // passes in the ways that the two sets rank first.  Another tile of one launch: 0.943 in the mean, four of 457 slower by
    // more than 2 % (the worst 4.3 %).  Tensorwise, predicted 0.9 times two launches or less: 0.90; 0.9 .. 0.97: the large
    // tiles on half the XCDs each, as in the separate launches, 0.98; where the product of fewer tiles is one round of its
    // units, or either contraction at most 8 steps, 0.95 (1600 x 2048 x 15360 delayed 200 -> 187), else 1.03, up to 1.10:
    // smaller tiles read their operands more often (3008 x 2928 x 4528 167 -> 184).  Rowwise, predicted 0.86 or less: 0.94,
    // and smaller tiles of more than three rounds by the card: where dX alone is 3.5 to 4 rounds, 1.02, up to 1.12, on one, and
    // 0.94, at most 1.02, on another.
    // us of a pass, before / after: 16384 x 2048 x 1024 173 / 153, 16384 x 4096 x 512 205 / 180, 11440 x 5568 x 512 207 /
    // 182, 400 x 5632 x 5760 119 / 103, 448 x 3328 x 10752 rowwise 188 / 162, 5920 x 5312 x 320 124 / 108, 8192 x 3584 x
    // 8192 delayed 604 / 598; two launches still: 1664 x 8896 x 6656, 16384 x 1024 x 1024.
    if (tile_count(x, 256, 256) + tile_count(w, 256, 256) > 5 * cus || M < 256 || N < 256) return c;
    constexpr double kLeast = 8.0;
    const double two = separately(4.5), first = in_pass_us(x, w, c, two, cus);
    PairChoice in_pass = c;
    best = first;
    auto few_reads = [&](PairChoice k) {
        if (k.tile == kSm || (k.tile == 256 && k.x_xcds == 4)) return true;
        const int bm = k.tile == 128 ? 128 : 256, bn = k.tile == 256 ? 256 : 128, at_once = k.tile == 128 ? 2 : 1;
        return tile_count(x, bm, bn) <= (int64_t)at_once * per_xcd * k.x_xcds || tile_count(w, bm, bn) <= (int64_t)at_once * per_xcd * (kXcds - k.x_xcds) ||
               (k.tile != 256 && (ksteps_of(x.K, 1) <= 8 || ksteps_of(w.K, 1) <= 8));
    };
    auto consider = [&](PairChoice k) {
        const double us = in_pass_us(x, w, k, two, cus);
        const bool clear = c.tile ? us < first - kLeast : us < first * (!KM ? 0.86 : few_reads(k) ? 0.97 : 0.90);
        if (clear && us < best) best = us, in_pass = k;
    };
    if (small <= 4 * cus) consider({kSm, 0});
    for (int xc : {4, 3, 5})
        for (int t : {256, 192, 128}) consider({t, xc});
    return in_pass;
}

bool F8_PAIR_NAME(, F8_PAIR_FA, F8_PAIR_GRAN)(const GemmArgs& gx, const GemmArgs& gw, uint32_t* amax_bits, void* ws, size_t ws_bytes,
                                              hipStream_t st)
{
    constexpr int FA = F8_PAIR_FA, GRAN = F8_PAIR_GRAN;
    if (GRAN != F8_TENSORWISE && amax_bits) return false;  // no call asks for it
    const int cus = cu_count();
    const PairChoice c = F8_PAIR_NAME(choice_, F8_PAIR_FA, F8_PAIR_GRAN)(gx.M, gx.N, gx.K, ws != nullptr, ws_bytes, cus);
    if (!c.tile) return false;
    auto side = [](const GemmArgs& a) {
        return PairSide{a.A, a.B, a.D, a.M, a.N, a.K, a.lda, a.ldb, a.ldd, a.isa, a.isb, 0, 0, 0};
    };
    const PairSide x = side(gx), w = side(gw);
    if (amax_bits) zero_word(amax_bits, st);
    switch (c.tile) {
        case kSm: {
            PairSide a = x, b = w;
            for (PairSide* s : {&a, &b}) s->tiles_m = (s->M + kSm - 1) / kSm, s->tiles_n = (s->N + kSm - 1) / kSm;
            gemm_small_pair_kernel<FA, GRAN><<<(unsigned)(a.tiles_m * a.tiles_n + b.tiles_m * b.tiles_n), 256, 0, st>>>(a, b, amax_bits);
            break;
        }
        case 128: launch_pair<128, 128, FA, GRAN>(x, w, c.x_xcds, amax_bits, cus, st); break;
        case 192: launch_pair<256, 128, FA, GRAN>(x, w, c.x_xcds, amax_bits, cus, st); break;
        default: launch_pair<256, 256, FA, GRAN>(x, w, c.x_xcds, amax_bits, cus, st);
    }
    return true;
}

}  // namespace f8

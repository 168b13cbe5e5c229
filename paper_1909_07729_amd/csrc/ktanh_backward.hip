// libktanh: gradients for training through K-TanH -- the derivative identities of TanH and Sigmoid
// on the forward outputs, the derivatives of the Swish and GELU identities from the forward inputs
// (BFloat16 and Float32 tensors), and one LSTM-cell step backwards -- and their entry points.
#include "ktanh_cell.h"

#include <type_traits>

using namespace ktanh_device;

namespace {

// Which slope multiplies dy.  TanH and Sigmoid take it from the forward OUTPUT (no table involved);
// Swish and GELU rebuild the K-TanH value from the forward INPUT with the device functions the
// forward kernels use:
//   TanH'    = 1 - y^2                      Sigmoid' = s * (1 - s)
//   Swish'   = s + x * (s * (1 - s)),                                       s = Sigmoid(x)
//   GELU'    = 0.5 * (1 + t) + (0.5 * x) * ((1 - t^2) * (c * (1 + 3a * x^2))),   t = K(c * (x + a x^3))
// Float32, one rounding per written operation.
enum Grad { GRAD_TANH = 0, GRAD_SIGMOID = 1, GRAD_SWISH = 2, GRAD_GELU = 3 };

// The slope from Float32 values: v is the forward output (TanH, Sigmoid) or the input with its
// K-TanH-derived value k already formed (s for Swish, t for GELU).
template <int GRAD>
__device__ __forceinline__ float slope_of(float v, float k)
{
    if constexpr (GRAD == GRAD_TANH) {
        const float sq = v * v;
        return 1.0f - sq;
    } else if constexpr (GRAD == GRAD_SIGMOID) {
        const float one_minus = 1.0f - v;
        return v * one_minus;
    } else if constexpr (GRAD == GRAD_SWISH) {
        const float one_minus = 1.0f - k;
        const float bell = k * one_minus;
        const float xbell = v * bell;
        return k + xbell;
    } else {
        const float a3 = 0.134145f;  // 3a
        const float c = 0.7978845608028654f;
        const float one_plus = 1.0f + k;
        const float left = 0.5f * one_plus;
        const float tsq = k * k;
        const float sech2 = 1.0f - tsq;
        const float sq = v * v;
        const float a3sq = a3 * sq;
        const float poly = 1.0f + a3sq;
        const float du = c * poly;
        const float chain = sech2 * du;
        const float half_x = 0.5f * v;
        const float right = half_x * chain;
        return left + right;
    }
}

// The argument of K inside GELU: c * (x + a * x^3).
__device__ __forceinline__ float gelu_argument(float x)
{
    const float a = 0.044715f;
    const float c = 0.7978845608028654f;
    const float sq = x * x;
    const float cube = sq * x;
    const float acube = a * cube;
    const float inner = x + acube;
    return c * inner;
}

// One 32-bit word of each stream: a packed BFloat16 pair (ELEM = uint16_t) or one Float32
// (ELEM = uint32_t, `hi` unused).  A single BFloat16 element travels in the low half of the word.
struct Slopes {
    float lo, hi;
};

template <class ELEM, int GRAD, bool WIDE>
__device__ __forceinline__ Slopes slopes_of_word(uint32_t v_w, const LaneTable &tab)
{
    if constexpr (sizeof(ELEM) == 2) {
        const float v[2] = {widen_lo(v_w), widen_hi(v_w)};
        float k[2] = {0.f, 0.f};
        if constexpr (GRAD == GRAD_SWISH) {
            ksigmoid_f32_pair<false, WIDE>(v_w, tab, k[0], k[1]);  // a NaN x reaches the slope through x itself
        } else if constexpr (GRAD == GRAD_GELU) {
            const uint32_t t2 = ktanh_pair<false, WIDE>(narrow_pair(gelu_argument(v[0]), gelu_argument(v[1])), tab);
            k[0] = widen_lo(t2);
            k[1] = widen_hi(t2);
        }
        return Slopes{slope_of<GRAD>(v[0], k[0]), slope_of<GRAD>(v[1], k[1])};
    } else {
        const float v = __uint_as_float(v_w);
        float k = 0.f;
        if constexpr (GRAD == GRAD_SWISH) {
            // 0.5 * t is exact for every K output t that can change the sum, so the multiply-add may fuse
            const float t = __uint_as_float(ktanh_f32_one<WIDE>(__float_as_uint(0.5f * v), tab));
            k = __builtin_fmaf(0.5f, t, 0.5f);
        } else if constexpr (GRAD == GRAD_GELU) {
            k = __uint_as_float(ktanh_f32_one<WIDE>(__float_as_uint(gelu_argument(v)), tab));
        }
        return Slopes{slope_of<GRAD>(v, k), 0.f};
    }
}

template <class ELEM>
__device__ __forceinline__ uint32_t grad_word(uint32_t dy_w, const Slopes &s)
{
    if constexpr (sizeof(ELEM) == 2) return narrow_pair(widen_lo(dy_w) * s.lo, widen_hi(dy_w) * s.hi);
    else return __float_as_uint(__uint_as_float(dy_w) * s.lo);
}

// Two input streams, one output stream (which may be one of the inputs): 6 bytes per BFloat16
// element, 12 per Float32 element.  One wavefront per block, one 128-bit vector per lane and stream.
// The body starts where `dx` reaches a 16-byte boundary and its tiles are cut at 1 KiB boundaries of
// `dx` (skew = index of the first vector inside its 1 KiB group); the elements before and after the
// body (n_edge < 64 of them) are taken by block 0.  IN_UNALIGNED: an input disagrees with `dx`
// modulo 16 bytes, so both are read with 16-byte loads from element-aligned addresses.  The table
// reads of Swish and GELU need every lane enabled, so bounds predicate only the loads and stores.
// The arguments a wavefront needs before its loads (the three body pointers, nvec, skew, n_edge)
// come first, as scalars: the leading scalar arguments of a kernel arrive preloaded in registers.
// KEEP: dx is small enough to stay in the last-level cache (stays_cached), where the kernel that takes
// it next finds it: kgelu_backward, three input pairs and two outputs in turn, us per launch without ->
// with: 12.3 -> 11.7 (22 MB tensors), 25.2 -> 23.9 (52 MB), 45.5 -> 42.9 (100 MB); all out of the cache:
// 12.1 -> 12.0, 25.2 -> 25.0, 45.5 -> 45.0; at 268 MB it is 118.0 -> 118.7, hence the line.
// NEAR: plain loads instead of loads with the non-temporal hint (plain_gradient_loads).  us per launch, three input pairs and two
// outputs in turn / all out of the cache, hint | plain: 12 MB tensors 6.5 / 7.8 | 6.6 / 8.2, 17 MB 9.4 / 10.1 | 8.9 / 10.7, 25 MB 13.0 / 13.7 |
// 12.1 / 14.7, 32 MB 15.9 / 17.0 | 15.3 / 18.4, 42 MB 20.0 / 21.5 | 20.3 / 23.3; Float32 25 MB 12.0 / 13.0 | 11.2 / 14.0: never plain.
// Inputs off the 16-byte grid, where neighbouring wavefronts share a cache line: 8 MB 5.1 / 6.0 | 4.9 / 6.2, 17 MB 9.6 / 10.2 |
// 9.0 / 10.7, 32 MB 16.0 / 17.2 | 15.4 / 18.2: plain up to 32 MiB of dx, and from there on with the hint in runs of tiles: 42 MB 19.6 / 22.9
// plain in the plain order, 20.0 / 21.1, kgelu_backward 27.3 -> 26.1 (52 MB), 136.6 -> 133.8 (268 MB), kswish_f32_backward 34.0 -> 28.9 (66 MB).
// DY: when dy is asked for.  A call that the memory bounds does better the less of it is on its way at once, so large calls (late_gradient_load) ask for
// dy when x has arrived (GELU on BFloat16, whose arithmetic, as long as the memory takes, then runs while dy is on its way) or when the slopes
// are formed (Swish and GELU on Float32).  us per launch, with x | late, inputs partly / all out of the cache: kgelu_backward 52 MB tensors 24.0 / 25.9 |
// 24.2 / 25.4, 80 MB 39.2 / 39.4 | 36.9 / 38.5, 120 MB 53.2 / 53.1 | 52.5 / 52.6, 134 MB 58.3 / 62.7 | 57.7 / 61.0, 268 MB 121.7 / 121.2 | 119.2 / 118.3, 537 MB 241.2 /
// 240.1 | 233.2 / 233.9, kgelu64_backward 52 MB 24.7 / 26.0 | 24.4 / 25.4, 268 MB 121.0 / 121.0 | 117.9 / 117.7; kgelu_f32_backward 200 MB 92.4 / 92.4 | 90.8 / 90.4, 268 MB
// 121.0 / 121.0 | 119.1 / 118.8, kswish_f32_backward 160 MB 73.6 / 74.0 | 73.1 / 73.1, kswish64_f32_backward 537 MB 239.6 / 239.0 | 238.2 / 237.2.  Below those lines
// a call whose inputs lie in the cache loses (kgelu_backward 34 MB 16.7 / 17.8 | 17.1 / 17.4).  The others are level, or gain on inputs out of the cache what they lose on
// others (kswish_backward 134 MB 57.2 / 62.3 | 58.7 / 62.2, ktanh_bf16_backward 57.1 / 61.7 | 57.2 / 62.0).
// With x the words are finished one after the other (DY_IN_TURN) or all slopes are formed first (DY_WITH_X), as they are in the late forms, where the late loads of
// kgelu64_backward lose 4-6 % without that.  In turn | slopes first: kgelu_backward 4.8 MB 3.87 / 4.18 | 4.00 / 4.22, 5 MB 3.79 / 4.21 | 3.92 / 4.24, 10 MB 6.13 / 6.66 | 6.26 / 6.68, kgelu64_backward 6 MB 4.35 / 4.66 |
// 4.49 / 4.75, kswish_f32_backward 1.5 MB 2.01 / 2.45 | 2.12 / 2.43, kgelu_f32_backward 1.8 MB off the grid 2.12 / 2.74 | 2.24 / 2.73; but kgelu64_backward 2.5 MB 2.78 / 3.25 | 2.72 /
// 3.14, 4.2 MB 3.30 / 3.90 | 3.17 / 3.87, BFloat16 inputs off the grid -3 to 0 % (ktanh_bf16_backward of 0.9 and 1 MB there 1.92 | 2.00, from 10 MB on -1 %).
enum DyLoad { DY_IN_TURN, DY_WITH_X, DY_BEHIND_X, DY_BEHIND_SLOPES };

template <class ELEM>
struct GradEdge {
    const ELEM *dy, *v;  // the whole tensors
    ELEM *dx;
    unsigned long long n;
    unsigned n_head;
};

template <class ELEM, int GRAD, bool WIDE, bool IN_UNALIGNED, bool KEEP, bool NEAR, DyLoad DY>
__global__ __launch_bounds__(kBlock) void grad_stream_kernel(const char *bdy0, const char *bv0,
                                                             uint4 *bdx0,  // the aligned bodies
                                                             unsigned long long nvec, unsigned skew,
                                                             unsigned n_edge,
                                                             unsigned runs,  // tile_of_block_in_runs
                                                             GradEdge<ELEM> g, KtLutPack pack)
{
    const LaneTable tab(pack);
    const unsigned tile = IN_UNALIGNED ? tile_of_block_in_runs(blockIdx.x, runs, 0, 18) : blockIdx.x;
    const unsigned long long slot = (unsigned long long)tile * kBlock + threadIdx.x;
    const unsigned long long at = slot - skew;
    const bool live = slot >= skew && at < nvec;
    const char *bdy = bdy0 + 16 * at;
    const char *bv = bv0 + 16 * at;
    uint4 a = uint4{0u, 0u, 0u, 0u}, b = uint4{0u, 0u, 0u, 0u};
    if (live) {
        if constexpr (DY == DY_IN_TURN || DY == DY_WITH_X) a = load_vec<!IN_UNALIGNED, NEAR>(bdy);
        b = load_vec<!IN_UNALIGNED, NEAR>(bv);
        if constexpr (DY == DY_BEHIND_X) {
            asm volatile("" : "+v"(b.x), "+v"(b.y), "+v"(b.z), "+v"(b.w) : : "memory");  // here before dy is asked for
            a = load_vec<!IN_UNALIGNED, NEAR>(bdy);
        }
    }
    if constexpr (DY == DY_IN_TURN) {
        const uint4 r = uint4{grad_word<ELEM>(a.x, slopes_of_word<ELEM, GRAD, WIDE>(b.x, tab)),
                              grad_word<ELEM>(a.y, slopes_of_word<ELEM, GRAD, WIDE>(b.y, tab)),
                              grad_word<ELEM>(a.z, slopes_of_word<ELEM, GRAD, WIDE>(b.z, tab)),
                              grad_word<ELEM>(a.w, slopes_of_word<ELEM, GRAD, WIDE>(b.w, tab))};
        if (live) store_stream<KEEP>(bdx0 + at, r);
    } else {
        Slopes s[4] = {slopes_of_word<ELEM, GRAD, WIDE>(b.x, tab), slopes_of_word<ELEM, GRAD, WIDE>(b.y, tab),
                       slopes_of_word<ELEM, GRAD, WIDE>(b.z, tab), slopes_of_word<ELEM, GRAD, WIDE>(b.w, tab)};
        if constexpr (DY == DY_BEHIND_SLOPES) {
#pragma unroll
            for (Slopes &one : s) asm volatile("" : "+v"(one.lo) : : "memory");  // formed before dy is asked for
            if (live) a = load_vec<!IN_UNALIGNED, NEAR>(bdy);
        }
        if (live)
            store_stream<KEEP>(bdx0 + at, uint4{grad_word<ELEM>(a.x, s[0]), grad_word<ELEM>(a.y, s[1]),
                                                grad_word<ELEM>(a.z, s[2]), grad_word<ELEM>(a.w, s[3])});
    }
    if (n_edge != 0 && blockIdx.x == 0) {  // uniform over the block
        const unsigned k = threadIdx.x;
        const bool some = k < n_edge;
        const unsigned long long i = k < g.n_head ? k : g.n - n_edge + k;
        const uint32_t d1 = some ? g.dy[i] : 0u, v1 = some ? g.v[i] : 0u;
        const uint32_t r1 = grad_word<ELEM>(d1, slopes_of_word<ELEM, GRAD, WIDE>(v1, tab));
        if (some) g.dx[i] = (ELEM)r1;
    }
}

ktanh_status_t pack_grad(const ktanh_lut_t *lut, bool f32, KtLutPack *pack)
{
    return f32 ? kt_pack_lut_f32(lut, pack) : kt_pack_lut_bf16(lut, pack);
}
ktanh_status_t pack_grad(const ktanh_lut64_t *lut, bool f32, KtLutPack *pack)
{
    return f32 ? kt_pack_lut64_f32(lut, pack) : kt_pack_lut64_bf16(lut, pack);
}
// `lut` is only read by Swish and GELU; TanH and Sigmoid pass NULL and Table 1 rides along unused.
template <class ELEM, int GRAD, class Lut>
ktanh_status_t launch_grad(const void *dy, const void *v, void *dx, size_t n, const Lut *lut,
                           ktanh_stream_t stream)
{
    constexpr bool WIDE = is_wide(static_cast<const Lut *>(nullptr));
    constexpr size_t kPerVec = 16 / sizeof(ELEM);
    if (n == 0) return KT_OK;
    if (dy == nullptr || v == nullptr || dx == nullptr) return KT_ERR_NULL;
    const uintptr_t ady = reinterpret_cast<uintptr_t>(dy), av = reinterpret_cast<uintptr_t>(v),
                    adx = reinterpret_cast<uintptr_t>(dx);
    if ((ady | av | adx) & (sizeof(ELEM) - 1)) return KT_ERR_ALIGN;
    if (n > (size_t)1 << 40) return KT_ERR_SHAPE;
    KtLutPack pack;
    const ktanh_status_t st = pack_grad(lut, sizeof(ELEM) == 4, &pack);
    if (st != KT_OK) return st;
    GradEdge<ELEM> g;
    g.dy = static_cast<const ELEM *>(dy);
    g.v = static_cast<const ELEM *>(v);
    g.dx = static_cast<ELEM *>(dx);
    g.n = n;
    size_t head = ((16 - (adx & 15)) & 15) / sizeof(ELEM);
    if (head > n) head = n;
    const size_t nvec = (n - head) / kPerVec;
    g.n_head = (unsigned)head;
    const unsigned n_edge = (unsigned)(n - nvec * kPerVec);
    const unsigned skew = (unsigned)((reinterpret_cast<uintptr_t>(g.dx + head) / 16) % kBlock);
    size_t tiles = (nvec + skew + kBlock - 1) / kBlock;
    if (tiles == 0) tiles = 1;  // edge elements only
    if (tiles > kMaxTiles) return KT_ERR_SHAPE;
    const char *bdy = reinterpret_cast<const char *>(g.dy + head);
    const char *bv = reinterpret_cast<const char *>(g.v + head);
    uint4 *bdx = reinterpret_cast<uint4 *>(g.dx + head);
    auto launch = [&](auto kernel) {
        return launch_checked(kernel, (unsigned)tiles, kBlock, stream, bdy, bv, bdx, (unsigned long long)nvec,
                              skew, n_edge, run_tiles_for(tiles), g, pack);
    };
    const bool congruent = (ady & 15) == (adx & 15) && (av & 15) == (adx & 15);
    const unsigned long long moved = 3 * n * sizeof(ELEM);
    constexpr bool kF32 = sizeof(ELEM) == 4, kReadsTable = GRAD == GRAD_GELU || GRAD == GRAD_SWISH;
    constexpr DyLoad kWithX = kF32 ? DY_IN_TURN : DY_WITH_X;
    constexpr DyLoad kLate = GRAD == GRAD_GELU && !kF32 ? DY_BEHIND_X : kReadsTable && kF32 ? DY_BEHIND_SLOPES : kWithX;
    if (plain_gradient_loads(moved, congruent)) return launch(grad_stream_kernel<ELEM, GRAD, WIDE, true, true, true, kWithX>);
    auto launch_kept = [&](auto kept, auto dy_load) {
        constexpr bool KEEP = decltype(kept)::value;
        constexpr DyLoad DY = decltype(dy_load)::value;
        return congruent ? launch(grad_stream_kernel<ELEM, GRAD, WIDE, false, KEEP, false, DY>)
                         : launch(grad_stream_kernel<ELEM, GRAD, WIDE, true, KEEP, false, DY>);
    };
    typedef std::integral_constant<DyLoad, kWithX> WithX;
    typedef std::integral_constant<DyLoad, kLate> Late;
    static_assert(late_gradient_load(3 * kLastLevelCacheBytes, kF32), "a streamed output is past the line");
    if (!stays_cached(n * sizeof(ELEM))) return launch_kept(std::false_type(), Late());
    if (late_gradient_load(moved, kF32)) return launch_kept(std::true_type(), Late());
    if constexpr (GRAD == GRAD_GELU && !kF32) {
        if (congruent && gelu_words_in_turn(moved)) return launch(grad_stream_kernel<ELEM, GRAD, WIDE, false, true, false, DY_IN_TURN>);
    }
    return launch_kept(std::true_type(), WithX());
}

// ---------------------------------------------------------------------------------------------
// LSTM cell, one step backwards: each lane owns two neighbouring cells (one packed pair per gate).
// The forward activations are rebuilt with the same device functions the forward kernel uses; the
// table reads need every lane enabled, so bounds predicate only the stores (lanes past the end work on
// pair 0 and store nothing).
//
// A stream of 30 bytes per cell with about 165 vector instructions per wavefront and 3840 bytes: bound by
// memory (the arithmetic alone is half of the time).  One wavefront per block and no wider than a pair
// per lane, as in the streaming kernels: two pairs per lane measured level, four 20-30 % slower.
// STREAMED: loads with the non-temporal hint, on calls whose inputs come from HBM; plain ones below, where
// they may still lie in the L2s and the last-level cache.  Two forms, by where the rows of a gate lie (cell_rows_fill_lines):
//
// WHOLE: where every piece of 64 pairs is made of whole cache lines, and on short calls, where it does not matter yet.  The pieces
// are taken in the plain order, and the stores write through to the last-level cache (sc1): dgates goes into a matrix product
// and dc_prev into the next step right away.  us per call, blocks of four wavefronts with plain loads and stores -> this, 3 inputs and 2 outputs in turn / all
// out of the cache: 16 MB 3.97 -> 3.25 / 4.95 -> 4.7, 31 MB 5.92 -> 5.59 / 7.78 -> 7.22, 126 MB 22.0 -> 19.5 /
// 24.9 -> 21.6, 252 MB 41.6 -> 36.7 / 44.3 -> 41.3; the other kind of load: 16 MB 4.1 / 4.3, 31 MB 6.0 / 6.5, 63 MB
// 9.8 plain against 10.7 / 12.2 against 11.5, 126 MB 20.3 / 23.0, 252 MB 41.2 / 44.4.
//
// Else neighbouring pieces share a line at either end.  In the plain order the neighbour runs on another XCD,
// which fetches the line again and writes its part of it through to memory on its own: [4000, 3000] cells took 94.8 us
// out of the cache against 61.0 of [4000, 3072], [100000, 8] 10.9 against 8.0 with four wavefronts and plain stores.  So
// each XCD takes runs of neighbouring pieces and its L2 puts the lines together.  us per call, 3 in 2 out / out of the
// cache, four wavefronts and plain loads and stores | WHOLE | this with plain loads | this with the hint:
//   [2048, 1000]   61 MB   11.3 / 14.6 | 12.6 / 16.0 |  9.9 / 13.5 | 11.3 / 12.4
//   [4096, 1000]  123 MB   22.4 / 26.0 | 23.0 / 31.5 | 20.3 / 24.0 | 20.9 / 23.3
//   [4000, 3000]  360 MB   69.8 / 69.4 | 65.7 / 94.5 | 66.0 / 64.6 | 59.3 / 65.4
//   [100000, 40]  120 MB   23.1 / 25.7 | 26.4 / 35.3 | 21.6 / 24.4 | 24.2 / 25.4
//   [700000, 8]   168 MB   35.2 / 36.1 | 50.6 / 62.5 | 32.7 / 33.9 | 38.0 / 38.6
//   [400000, 32]  384 MB   68.9 / 68.3 | 64.9 / 65.0 |             | 68.9 / 68.8   (no line is shared: WHOLE)
// Short rows (cell_rows_are_short) read a line once for several gates, so they need it in the cache: plain loads, and this
// form from 2^15 pairs on, a span of runs ([100000, 8], 24 MB, 6.9 / 8.0 | 8.1 / 10.9 | 5.5 / 7.4; [8192, 8] 2.3 / 2.5 | 2.1 / 2.5 | 2.0 / 2.4;
// [1024, 8] 2.1 / 2.1 | 1.9 / 1.9 | 2.0 / 2.0).  Of longer ones a call of up to 48 MiB is better off with WHOLE ([512, 1000] 4.1 / 5.6 | 3.3 / 5.1 |
// 3.9 / 5.3).
//
// The table reads of the gates go out together, NaN rules are a rare repair, and a 64-interval table that folds has no selects (ktanh_cell.h).
// LOADS (CellLoads in ktanh_order.h): when a lane asks for what is not a gate word.  A small call takes as long as one wavefront, which then waits for memory
// once; a large one is bound by memory, which does better the less of it is on its way at once.  us per call, in turn | at once, inputs
// partly / all out of the cache: [64, 1024] 2.14 / 2.32 | 1.96 / 2.15, [128, 1024] 2.28 / 2.54 | 2.03 / 2.31, [200, 1000] 2.47 / 3.74 | 2.26 / 3.20,
// [128, 2048] 2.53 / 3.81 | 2.43 / 3.48, [192, 2048] 3.00 / 4.21 | 2.76 / 4.24, [256, 2048] 3.28 / 4.67 | 3.03 / 4.86, [512, 2048] 5.45 / 7.11 | 5.87 / 7.44.
// In turn | late: whole lines [2048, 2048] 20.9 / 21.7 | 21.6 / 21.6, [3500, 2048] 32.8 / 36.2 | 33.1 / 35.6, [5000, 2048] 45.3 / 51.3 | 45.4 / 50.1, [6000, 2048]
// 56.8 / 61.4 | 55.5 / 59.7; rows off the lines [1800, 2040] 20.6 / 21.7 | 20.6 / 21.6, [2400, 2040] 27.5 / 28.4 | 26.4 / 27.9, [3600, 2040] 38.7 / 40.7 |
// 37.9 / 39.8, [5000, 2040] 51.5 / 57.7 | 49.4 / 55.1; rows of 32 [400000, 32] 65.1 / 65.1 | 64.4 / 64.4, of 40 level.

template <bool THROUGH, class T>
__device__ __forceinline__ void store_cell(T *base, unsigned byte_offset, T v)
{
    if constexpr (THROUGH) store_stream(base, byte_offset, v);
    else *reinterpret_cast<T *>(reinterpret_cast<char *>(base) + byte_offset) = v;
}

template <CellTable TAB, bool STREAMED, bool WHOLE, CellLoads LOADS>
__global__ __launch_bounds__(kBlock) void lstm_cell_backward_kernel(
    unsigned n_pairs, unsigned H2, unsigned row_mul, unsigned row_shift,  // row_of_pair
    const uint32_t *__restrict__ gates, const float2 *__restrict__ c_prev, const uint32_t *__restrict__ dh,
    const float2 *dc_next, uint32_t *__restrict__ dgates, float2 *dc_prev, KtLutPack pack)
{
    const LaneTable tab(pack);
    const unsigned tile = WHOLE ? blockIdx.x : tile_of_block_in_runs(blockIdx.x, cell_run_tiles(n_pairs), 0, 18);
    const unsigned p = tile * kBlock + threadIdx.x;
    const bool live = p < n_pairs;
    const unsigned p_read = live ? p : 0;
    // byte offsets, below 2^32 (checked by the caller); pair p = row * H2 + j has its i gate at word
    // row * 4 * H2 + j = p + row * 3 * H2 of [B][4H]
    const unsigned at_i = 4u * (p_read + row_of_pair(p_read, row_mul, row_shift) * (3u * H2));
    const unsigned at_f = at_i + 4u * H2, at_g = at_f + 4u * H2, at_o = at_g + 4u * H2;

    const GateWords q = {load_at<STREAMED>(gates, at_i), load_at<STREAMED>(gates, at_f),
                         load_at<STREAMED>(gates, at_g), load_at<STREAMED>(gates, at_o)};
    float2 c0 = float2{0.f, 0.f}, dcn = float2{0.f, 0.f};
    uint32_t wdh = 0u;
    if constexpr (LOADS != CELL_LOADS_LATE) c0 = load_at<STREAMED>(c_prev, 8u * p_read);
    if constexpr (LOADS == CELL_LOADS_AT_ONCE) {
        wdh = load_at<STREAMED>(dh, 4u * p_read);
        dcn = load_at<STREAMED>(dc_next, 8u * p_read);
    }

    Acts a = gate_activations<TAB>(q, tab);
    if constexpr (LOADS == CELL_LOADS_LATE) {
        asm volatile("" : "+v"(a.i_lo), "+v"(a.f_lo), "+v"(a.g2) : : "memory");  // formed before the state is asked for
        c0 = load_at<STREAMED>(c_prev, 8u * p_read);
    }
    float2 c1 = c0;
    advance_state(a, c1);
    const uint32_t tc2 = state_tanh<TAB>(c1.x, c1.y, tab);
    const float ig[2] = {a.i_lo, a.i_hi}, fg[2] = {a.f_lo, a.f_hi}, og[2] = {a.o_lo, a.o_hi};
    const float gg[2] = {widen_lo(a.g2), widen_hi(a.g2)};
    const float cp[2] = {c0.x, c0.y};
    const float tc[2] = {widen_lo(tc2), widen_hi(tc2)};
    if (!live) return;  // no table read from here on
    if constexpr (LOADS != CELL_LOADS_AT_ONCE) {
        wdh = load_at<STREAMED>(dh, 4u * p);
        dcn = load_at<STREAMED>(dc_next, 8u * p);
    }
    const float dhv[2] = {widen_lo(wdh), widen_hi(wdh)};
    const float dnx[2] = {dcn.x, dcn.y};

    float d_gi[2], d_gf[2], d_gg[2], d_go[2], dcp[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
        const float d_o = dhv[k] * tc[k];
        const float dh_o = dhv[k] * og[k];
        const float tsq = tc[k] * tc[k];
        const float tslope = 1.0f - tsq;
        const float through = dh_o * tslope;
        const float dc = dnx[k] + through;
        const float d_i = dc * gg[k], d_f = dc * cp[k], d_g = dc * ig[k];
        dcp[k] = dc * fg[k];
        const float i1 = 1.0f - ig[k], f1 = 1.0f - fg[k], o1 = 1.0f - og[k];
        const float islope = ig[k] * i1, fslope = fg[k] * f1, oslope = og[k] * o1;
        const float gsq = gg[k] * gg[k];
        const float gslope = 1.0f - gsq;
        d_gi[k] = d_i * islope;
        d_gf[k] = d_f * fslope;
        d_gg[k] = d_g * gslope;
        d_go[k] = d_o * oslope;
    }
    store_cell<WHOLE>(dgates, at_i, narrow_pair(d_gi[0], d_gi[1]));
    store_cell<WHOLE>(dgates, at_f, narrow_pair(d_gf[0], d_gf[1]));
    store_cell<WHOLE>(dgates, at_g, narrow_pair(d_gg[0], d_gg[1]));
    store_cell<WHOLE>(dgates, at_o, narrow_pair(d_go[0], d_go[1]));
    store_cell<WHOLE>(dc_prev, 8u * p, float2{dcp[0], dcp[1]});
}

}  // namespace

extern "C" ktanh_status_t ktanh_bf16_backward(const uint16_t *dy, const uint16_t *y, uint16_t *dx,
                                              size_t n, ktanh_stream_t stream)
{
    return launch_grad<uint16_t, GRAD_TANH>(dy, y, dx, n, static_cast<const ktanh_lut_t *>(nullptr), stream);
}

extern "C" ktanh_status_t ksigmoid_backward(const uint16_t *dy, const uint16_t *s, uint16_t *dx,
                                            size_t n, ktanh_stream_t stream)
{
    return launch_grad<uint16_t, GRAD_SIGMOID>(dy, s, dx, n, static_cast<const ktanh_lut_t *>(nullptr), stream);
}

extern "C" ktanh_status_t kswish_backward(const uint16_t *dy, const uint16_t *x, uint16_t *dx,
                                          size_t n, const ktanh_lut_t *lut, ktanh_stream_t stream)
{
    return launch_grad<uint16_t, GRAD_SWISH>(dy, x, dx, n, lut, stream);
}

extern "C" ktanh_status_t kgelu_backward(const uint16_t *dy, const uint16_t *x, uint16_t *dx,
                                         size_t n, const ktanh_lut_t *lut, ktanh_stream_t stream)
{
    return launch_grad<uint16_t, GRAD_GELU>(dy, x, dx, n, lut, stream);
}

extern "C" ktanh_status_t ktanh_f32_backward(const float *dy, const float *y, float *dx, size_t n,
                                             ktanh_stream_t stream)
{
    return launch_grad<uint32_t, GRAD_TANH>(dy, y, dx, n, static_cast<const ktanh_lut_t *>(nullptr), stream);
}

extern "C" ktanh_status_t ksigmoid_f32_backward(const float *dy, const float *s, float *dx, size_t n,
                                                ktanh_stream_t stream)
{
    return launch_grad<uint32_t, GRAD_SIGMOID>(dy, s, dx, n, static_cast<const ktanh_lut_t *>(nullptr), stream);
}

extern "C" ktanh_status_t kswish_f32_backward(const float *dy, const float *x, float *dx, size_t n,
                                              const ktanh_lut_t *lut, ktanh_stream_t stream)
{
    return launch_grad<uint32_t, GRAD_SWISH>(dy, x, dx, n, lut, stream);
}

extern "C" ktanh_status_t kgelu_f32_backward(const float *dy, const float *x, float *dx, size_t n,
                                             const ktanh_lut_t *lut, ktanh_stream_t stream)
{
    return launch_grad<uint32_t, GRAD_GELU>(dy, x, dx, n, lut, stream);
}

namespace {

ktanh_status_t pack_cell(const ktanh_lut_t *lut, KtLutPack *pack, bool *folds)
{
    *folds = false;
    return kt_pack_lut_bf16(lut, pack);
}
ktanh_status_t pack_cell(const ktanh_lut64_t *lut, KtLutPack *pack, bool *folds)
{
    return kt_pack_lut64_bf16(lut, pack, nullptr, folds);
}

template <class Lut>
ktanh_status_t launch_cell_backward(const uint16_t *gates, const float *c_prev, const uint16_t *dh,
                                    const float *dc_next, uint16_t *dgates, float *dc_prev, size_t B,
                                    size_t H, const Lut *lut, ktanh_stream_t stream)
{
    constexpr bool WIDE = is_wide(static_cast<const Lut *>(nullptr));
    if (B == 0 || H == 0) return KT_OK;
    if (gates == nullptr || c_prev == nullptr || dh == nullptr || dc_next == nullptr ||
        dgates == nullptr || dc_prev == nullptr)
        return KT_ERR_NULL;
    if (H % 8 != 0) return KT_ERR_SHAPE;
    if (B > ((size_t)1 << 40) || H > ((size_t)1 << 40)) return KT_ERR_SHAPE;
    // the kernel moves BFloat16 pairs (4 bytes) and Float32 pairs (8 bytes)
    const uintptr_t words = reinterpret_cast<uintptr_t>(gates) | reinterpret_cast<uintptr_t>(dh) |
                            reinterpret_cast<uintptr_t>(dgates);
    const uintptr_t states = reinterpret_cast<uintptr_t>(c_prev) | reinterpret_cast<uintptr_t>(dc_next) |
                             reinterpret_cast<uintptr_t>(dc_prev);
    if ((words & 3) || (states & 7)) return KT_ERR_ALIGN;
    KtLutPack pack;
    bool folds = false;
    const ktanh_status_t st = pack_cell(lut, &pack, &folds);
    if (st != KT_OK) return st;
    if (B > (1ull << 28) / (H / 2)) return KT_ERR_SHAPE;
    const unsigned long long n_pairs = (unsigned long long)B * (H / 2);
    if (n_pairs >= (1ull << 28)) return KT_ERR_SHAPE;  // word indices inside [B][4H] fit 32 bits
    const unsigned long long blocks = (n_pairs + kBlock - 1) / kBlock;
    const RowDivision row = row_division((unsigned)(H / 2));
    auto launch = [&](auto kernel) {
        return launch_checked(kernel, (unsigned)blocks, kBlock, stream, (unsigned)n_pairs, (unsigned)(H / 2),
                              row.mul, row.shift, reinterpret_cast<const uint32_t *>(gates),
                              reinterpret_cast<const float2 *>(c_prev), reinterpret_cast<const uint32_t *>(dh),
                              reinterpret_cast<const float2 *>(dc_next), reinterpret_cast<uint32_t *>(dgates),
                              reinterpret_cast<float2 *>(dc_prev), pack);
    };
    const CellBackward form = cell_backward_form(n_pairs, H, cell_rows_fill_lines(H, words | states));
    auto launch_with = [&](auto table) {
        constexpr CellTable TAB = decltype(table)::value;
        switch (form.loads) {
            case CELL_LOADS_AT_ONCE: return launch(lstm_cell_backward_kernel<TAB, false, true, CELL_LOADS_AT_ONCE>);
            case CELL_LOADS_LATE:
                return form.whole ? launch(lstm_cell_backward_kernel<TAB, true, true, CELL_LOADS_LATE>)
                                  : launch(lstm_cell_backward_kernel<TAB, true, false, CELL_LOADS_LATE>);
            default: break;
        }
        if (form.whole)
            return form.streamed ? launch(lstm_cell_backward_kernel<TAB, true, true, CELL_LOADS_IN_TURN>)
                                 : launch(lstm_cell_backward_kernel<TAB, false, true, CELL_LOADS_IN_TURN>);
        return form.streamed ? launch(lstm_cell_backward_kernel<TAB, true, false, CELL_LOADS_IN_TURN>)
                             : launch(lstm_cell_backward_kernel<TAB, false, false, CELL_LOADS_IN_TURN>);
    };
    if constexpr (WIDE) {
        if (folds) return launch_with(std::integral_constant<CellTable, CELL64_FOLDED>());
        return launch_with(std::integral_constant<CellTable, CELL64>());
    } else {
        return launch_with(std::integral_constant<CellTable, CELL32>());
    }
}

}  // namespace

extern "C" ktanh_status_t klstm_cell_backward(const uint16_t *gates, const float *c_prev,
                                              const uint16_t *dh, const float *dc_next,
                                              uint16_t *dgates, float *dc_prev, size_t B, size_t H,
                                              const ktanh_lut_t *lut, ktanh_stream_t stream)
{
    return launch_cell_backward(gates, c_prev, dh, dc_next, dgates, dc_prev, B, H, lut, stream);
}

extern "C" ktanh_status_t klstm_cell64_backward(const uint16_t *gates, const float *c_prev,
                                                const uint16_t *dh, const float *dc_next,
                                                uint16_t *dgates, float *dc_prev, size_t B, size_t H,
                                                const ktanh_lut64_t *lut, ktanh_stream_t stream)
{
    return launch_cell_backward(gates, c_prev, dh, dc_next, dgates, dc_prev, B, H, lut, stream);
}

extern "C" ktanh_status_t kswish64_backward(const uint16_t *dy, const uint16_t *x, uint16_t *dx,
                                            size_t n, const ktanh_lut64_t *lut, ktanh_stream_t stream)
{
    return launch_grad<uint16_t, GRAD_SWISH>(dy, x, dx, n, lut, stream);
}

extern "C" ktanh_status_t kgelu64_backward(const uint16_t *dy, const uint16_t *x, uint16_t *dx,
                                           size_t n, const ktanh_lut64_t *lut, ktanh_stream_t stream)
{
    return launch_grad<uint16_t, GRAD_GELU>(dy, x, dx, n, lut, stream);
}

extern "C" ktanh_status_t kswish64_f32_backward(const float *dy, const float *x, float *dx, size_t n,
                                                const ktanh_lut64_t *lut, ktanh_stream_t stream)
{
    return launch_grad<uint32_t, GRAD_SWISH>(dy, x, dx, n, lut, stream);
}

extern "C" ktanh_status_t kgelu64_f32_backward(const float *dy, const float *x, float *dx, size_t n,
                                               const ktanh_lut64_t *lut, ktanh_stream_t stream)
{
    return launch_grad<uint32_t, GRAD_GELU>(dy, x, dx, n, lut, stream);
}

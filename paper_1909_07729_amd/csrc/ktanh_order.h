// Internal to libktanh: the order in which the blocks of a streaming launch take their tiles.
// Plain C++ (no device headers) so that host tests can check it.
#pragma once

#ifdef __HIPCC__
#define KT_HOST_DEVICE __host__ __device__
#else
#define KT_HOST_DEVICE
#endif

namespace ktanh_device {

// Which tile a block takes.  Blocks are dispatched in index order, round-robin over the eight XCDs,
// so the tiles in flight at any moment form one window that moves through the tensor.  On large
// tensors two windows 128 or 256 MiB apart keep the memory busier than one: measured 0.8-2 % faster
// from 256 MiB of output upwards (windows closer than 64 MiB are slower by up to 9 %, and below
// 256 MiB nothing beats the plain order).  So a tensor is cut into segments of `1 << lg_seg` tiles
// (256 MiB; 512 MiB from 512 MiB of output on); inside each whole segment the blocks alternate, in
// groups of eight (one per XCD), between its two halves; what follows the last whole segment, and
// every tensor smaller than one segment, keeps the plain order.  A bijection on [0, tiles).
struct TileOrder {
    unsigned whole;   // tiles covered by whole segments (0 = plain order everywhere)
    unsigned lg_seg;  // log2 of the segment length in tiles
};

inline TileOrder tile_order_for(unsigned long long tiles)
{
    const unsigned lg = tiles >= (1ull << 19) ? 19u : 18u;
    return TileOrder{(unsigned)((tiles >> lg) << lg), lg};
}

KT_HOST_DEVICE inline unsigned tile_of_block(unsigned b, unsigned whole, unsigned lg_seg)
{
    if (b >= whole) return b;
    const unsigned mask = (1u << lg_seg) - 1u;
    const unsigned w = b & mask;
    return (b & ~mask) + (((w >> 3) & 1u) << (lg_seg - 1u)) + (((w >> 4) << 3) | (w & 7u));
}

// The same for a launch whose input starts off the 16-byte grid: a wavefront's KiB of input then touches nine
// cache lines, the ninth of which is the first of the next tile.  In the plain order the next tile runs on
// another XCD, which has to fetch that line into its own L2 again: an eighth more reads.  So blocks are taken in
// spans of 512, in which each XCD (block index modulo eight) gets a run of 64 neighbouring tiles; the two windows
// of large tensors then alternate by whole spans.  Measured on K-TanH with an input one element off, us per
// launch, plain order -> runs (each with its better kind of load): 52 MB tensors 16.8 -> 16.0, 105 MB 34.8 -> 30.4,
// 268 MB 85.4 -> 81.7, 537 MB 170.4 -> 165.9 (runs of 16 and of 1024 up to 3 % more, shorter ones more than the plain
// order).  Below 32 MiB the spans are too few to keep the XCDs level (8.4 MB 3.5 -> 3.9).
constexpr unsigned kRun = 64, kSpan = 8 * kRun;

inline unsigned run_tiles_for(unsigned long long tiles)
{
    return tiles >= (1ull << 15) ? (unsigned)(tiles / kSpan * kSpan) : 0u;
}

// runs: tiles covered by whole spans (run_tiles_for); `whole` is then a multiple of kSpan below it.
KT_HOST_DEVICE inline unsigned tile_of_block_in_runs(unsigned b, unsigned runs, unsigned whole, unsigned lg_seg)
{
    if (b >= runs) return b;
    const unsigned tile = (b & ~(kSpan - 1u)) + (b & 7u) * kRun + ((b & (kSpan - 1u)) >> 3);
    if (tile >= whole) return tile;
    const unsigned mask = (1u << lg_seg) - 1u;
    const unsigned w = tile & mask, span = w / kSpan;
    return (tile & ~mask) + ((span & 1u) << (lg_seg - 1u)) + (span >> 1) * kSpan + (w & (kSpan - 1u));
}

// Which calls read their input with plain loads and which with the non-temporal hint, by the bytes that the call reads and
// writes (figures at load_vec in ktanh_device.h and at grad_stream_kernel).  `aligned`: inputs congruent to the output modulo 16.
inline bool plain_elementwise_loads(unsigned long long moved, bool aligned)
{
    return aligned ? moved < 64ull << 20 : moved <= 96ull << 20;
}
inline bool plain_gradient_loads(unsigned long long moved, bool aligned) { return !aligned && moved <= 96ull << 20; }
// From where on GELU on aligned BFloat16 tensors finishes its words one after the other (as far as dy is not late).
constexpr bool gelu_words_in_turn(unsigned long long moved) { return moved >= 13ull << 20; }
// Which gradients ask for dy behind x or behind the slopes, where the kernel gains by it (figures at grad_stream_kernel).
constexpr bool late_gradient_load(unsigned long long moved, bool f32) { return moved >= (f32 ? 448ull : 144ull) << 20; }

// Row of a pair in an LSTM state of `d` pairs per row: p / d for p < 2^30 and 4 <= d <= 2^30, as one
// high-half multiplication and a shift by numbers that the host forms once per call (division by an
// invariant integer, Granlund and Montgomery 1994).  With l = ceil(log2 d) and mul = floor(2^(30+l) / d) + 1
// we have 2^(30+l) < mul * d <= 2^(30+l) + 2^l, so that p * mul / 2^(30+l) exceeds p / d by less than 1 / d
// and both have the same whole part; mul < 2^32.  (The compiler's 32-bit division by a value it does not
// know is about thirty vector instructions in every lane.)
struct RowDivision {
    unsigned mul, shift;
};

inline RowDivision row_division(unsigned d)
{
    unsigned l = 2;
    while ((1ull << l) < d) ++l;
    return RowDivision{(unsigned)((1ull << (30 + l)) / d + 1u), l - 2u};
}

KT_HOST_DEVICE inline unsigned row_of_pair(unsigned p, unsigned mul, unsigned shift)
{
    return (unsigned)(((unsigned long long)p * mul) >> 32) >> shift;
}

// The LSTM kernels that take one time step give every wavefront a piece of 64 neighbouring pairs.  Whether the pieces of all four
// gates are made of whole 128-byte cache lines that no other piece touches: rows that are a multiple of a line (or, 32 cells, half
// of one: a piece is then four whole rows), and tensors that start on one.  `pointers`: the addresses of the tensors or'ed together.
inline bool cell_rows_fill_lines(unsigned long long H, unsigned long long pointers)
{
    return (H % 64 == 0 || H == 32) && pointers % 128 == 0;
}

// Where they are not, an XCD takes runs of neighbouring pieces: the tiles that tile_of_block_in_runs covers.
KT_HOST_DEVICE inline unsigned cell_run_tiles(unsigned n_pairs) { return (n_pairs + 63u) / 64u / kSpan * kSpan; }

// Rows of less than a line (and other than half of one) put several gates' parts into one line, which a wavefront then reads once per
// gate: such a line has to stay in the cache, so large calls keep plain loads.
inline bool cell_rows_are_short(unsigned long long H) { return H < 64 && H % 32 != 0; }

// The form of the backward step (lstm_cell_backward_kernel, where the figures are): with non-temporal loads, and with
// pieces in the plain order whose stores write through.  `lines` is cell_rows_fill_lines.
// loads: the state and the gradients that come in are asked for with the gate words (calls that take as long as one wavefront), the gradients
// when K of the state is formed, or the state too when the gates are (calls that are bound by memory; short rows are level).
enum CellLoads { CELL_LOADS_AT_ONCE, CELL_LOADS_IN_TURN, CELL_LOADS_LATE };

struct CellBackward {
    bool streamed, whole;
    CellLoads loads;
};

inline CellBackward cell_backward_form(unsigned long long n_pairs, unsigned long long H, bool lines)
{
    const unsigned long long moved = 60 * n_pairs, MiB = 1ull << 20;
    if (cell_rows_are_short(H) && n_pairs >= 1u << 15) return CellBackward{false, false, CELL_LOADS_IN_TURN};
    const CellLoads loads = n_pairs <= 3u << 16                   ? CELL_LOADS_AT_ONCE
                            : moved <= (lines ? 256 : 128) * MiB ? CELL_LOADS_IN_TURN
                                                                 : CELL_LOADS_LATE;
    if (lines) return CellBackward{moved > 48 * MiB, true, loads};
    return moved <= 48 * MiB ? CellBackward{false, true, loads} : CellBackward{moved > 96 * MiB, false, loads};
}

// The form of a single forward step (lstm_step_kernel, where the figures are).
enum CellStep { STEP_ONE_WAVE, STEP_FOUR_WAVES, STEP_SHORT_ROWS, STEP_STREAMED };

inline CellStep cell_step_form(unsigned long long n_pairs, unsigned long long H)
{
    if (36 * n_pairs > 72ull << 20) return cell_rows_are_short(H) ? STEP_SHORT_ROWS : STEP_STREAMED;
    return n_pairs > 1u << 16 && n_pairs <= 1u << 19 ? STEP_FOUR_WAVES : STEP_ONE_WAVE;
}

// How many time steps the LSTM cell takes at a time where the pairs of cells are too few to fill the chip with one lane each
// (chunks of time, ktanh_lstm_chunks.hip): up to this many pairs, by the number of steps.  Beyond them, and with two steps, the kernels that take the
// steps one by one win: steps written out below eight steps, the ring of ring_stages from there on.  The line lies lowest where the last chunk of four holds
// a single step (T = 5, 9, 13, ...).  us per launch, inputs partly / all out of the cache, chunks | step by step, rows of 2048 cells:
// T = 2 49152 pairs 2.82 / 3.03 | 2.53 / 2.62; T = 3 49152 2.89 / 3.06 | 3.00 / 3.12, 131072 3.52 / 3.98 | 3.52 / 3.93; T = 4 131072 3.67 / 4.26 | 4.08 / 4.49; T = 5 40960 3.38 / 3.60 | 3.52 /
// 3.85, 57344 3.66 / 3.95 | 3.59 / 4.00, 131072 5.33 / 5.84 | 4.69 / 5.11; T = 6 98304 4.81 / 5.25 | 4.93 / 5.37, 106496 4.98 / 5.46 | 4.98 / 5.42, 131072 5.45 / 5.94 | 5.17 / 5.51; T = 7 131072
// 6.15 / 6.25 | 6.21 / 6.12; T = 8 131072 6.01 / 6.09 | 6.83 / 6.53; T = 9 98304 6.28 / 6.64 | 6.57 / 6.80, 106496 6.91 / 6.92 | 7.12 / 6.84, 131072 7.49 / 7.66 | 7.42 / 7.09; T = 10 114688 7.04 /
// 7.09 | 7.85 / 7.57, 131072 8.01 / 8.11 | 8.23 / 7.98; T = 11 131072 7.77 / 7.83 | 8.84 / 8.61; T = 13 98304 7.97 / 8.01 | 8.64 / 8.38, 131072 9.73 / 9.85 | 9.24 / 9.03; T = 16 114688 8.82 / 8.89 | 9.78 /
// 9.80, 131072 10.1 / 10.1 | 10.3 / 10.1; T = 20 98304 9.57 / 9.67 | 11.1 / 10.9, 106496 11.0 / 10.8 | 11.6 / 11.5; T = 33 98304 15.3 / 15.8 | 16.1 / 16.4, 106496 16.7 / 16.5 | 16.3 / 16.3.  64
// intervals alike.  Rows off the cache lines gain less (of 2000, T = 9 98304 6.63 / 7.21 | 6.70 / 7.17, T = 16 114688 9.91 / 10.4 | 9.98 / 10.1), and of a few hundred cells least: the kernels
// step by step pass the chunks at 50000 to 90000 pairs (of 200, T = 16 114688 12.1 / 12.4 | 10.5 / 10.7, T = 20 98304 12.2 / 12.3 | 11.9 / 12.0, T = 6 98304 5.26 / 6.03 | 5.19 / 5.79), below these lines.
inline unsigned most_pairs_in_chunks(unsigned T)
{
    switch (T) {
        case 0: case 1: case 2: return 0;
        case 3: return 49152;
        case 4: case 8: return 131072;
        case 5: return 40960;
        case 6: return 98304;
        default: break;
    }
    if (T > 16 || T % 4 == 1) return 98304;
    return T % 4 == 3 ? 131072 : 114688;
}

// The steps of a chunk: 4 to 64, a power of two; 0 where there are no chunks.  A step of a chunk times its pairs is at most 2^19, so that 16 bytes of gate
// words for each keep the offsets inside a chunk up to 2^23.
inline unsigned chunk_steps(unsigned T, unsigned n_pairs)
{
    if (n_pairs > most_pairs_in_chunks(T)) return 0;
    unsigned steps = 4;
    while (steps < 64 && steps < T) steps *= 2;
    // 64 steps | 32, inputs partly / all out of the cache: T = 40 5120 pairs 4.44 / 5.14 | 4.63 / 4.83, T = 64 5.51 / 6.50 | 5.32 / 5.60, T = 90 7.96 / 8.79 | 7.14 / 7.32,
    // 8192 pairs T = 64 6.40 / 7.38 | 5.15 / 5.81
    if (steps == 64 && n_pairs > 4096) steps = 32;
    while (steps > 4 && n_pairs * steps > 1u << 19) steps /= 2;
    return steps;
}

// Whether a chunk of four steps asks for the next chunk's gate words together with its own (lstm_chunk_kernel).  us per launch, before the walk / together, inputs
// partly in the cache: T = 17 81920 pairs 8.67 / 8.99, 98304 9.51 / 9.68; T = 24 98304 11.5 / 11.8; T = 40 98304 17.2 / 17.9, rows of 2000 cells 19.6 / 19.7; T = 64 81920 23.1 /
// 23.1, of 2000 26.2 / 25.7; T = 90 81920 32.4 / 31.7, of 2000 36.4 / 35.3, of 200 41.6 / 40.0.
inline bool chunk_words_at_once(unsigned T) { return T > 40; }

// How many stages the kernel for cells that do not fill the chip works with (ktanh_lstm_ring.hip), behind chunk_steps; 0: the kernels for many
// cells.  Four stages read three steps ahead, three two: the more wavefronts share the memory, the fewer steps should be read at once.  us per
// launch, T = 64, kernel for many cells / four stages / three: 131072 pairs 35.8 / 29.6 / 32.3, 163840 41.1 / 38.4 / 39.1, 180224 42.5 / 40.4 / 41.3,
// 212992 50.5 / 52.6 / 48.9, 262144 56.2 / 57.3 / 55.9, 286720 65.4 / 67.7 / 65.7; T = 16 163840 12.9 / 12.0 / 12.0, 204800 15.3 / 15.3 / 14.5, 262144
// 16.9 / 16.6 / 16.3.  Rows off the cache lines (and half lines, 32 cells) make a wavefront read more lines per step: 131072 pairs of rows of 2000 cells 37.3 /
// 31.6 / 33.9, of 32 35.8 / 31.0 / 32.8; 144000 of 32 T = 40 27.8 / 28.3 / 27.4, of 72 T = 64 46.4 / 48.8 / 47.0, 150000 of 200 T = 32 23.9 / 24.7 / 24.0, 170000 of
// 16 T = 20 21.5 / 20.8 / 20.9, 200000 of 2000 T = 64 55.5 / 59.1 / 56.0, T = 16 16.0 / - / 15.7: there three stages gain on few steps only.
// Whole rows that start off the lines (`aligned` is false) lose where the steps are many, with four stages sooner: rows of 2048, kernel for many cells / four stages 145000 pairs T = 42 30.9 / 31.1,
// T = 48 33.3 / 34.4, T = 96 63.9 / 67.9, 157000 T = 33 25.5 / 25.0, T = 64 45.9 / 47.8; with three T = 39 215000 38.4 / 37.1, T = 64 230000 62.6 / 64.2, rows of 512 T = 80 208000 71.6 / 74.3, of 1024 T = 92
// 215000 88.0 / 90.3 (means of 40 to 100 sizes: T = 40 -2 %, 64 level, 80 and more +1 %, rows of 64 cells -1.5 %).  A 64-interval table that folds goes to three there,
// four / three T = 48 151000 34.9 / 33.1, T = 64 157000 48.1 / 45.2, T = 96 133000 64.9 / 59.8.
inline unsigned ring_stages(unsigned T, unsigned n_pairs, unsigned long long H, bool aligned)
{
    if (T < 8) return 0;
    if (H % 64 == 0) {
        if (n_pairs > 5u << 15) return n_pairs < 1u << 18 && (aligned || T < 80) ? 3 : 0;
        return aligned || T < 44 || n_pairs <= 1u << 17 ? 4 : 0;
    }
    return n_pairs <= 1u << 17 ? 4 : n_pairs <= 3u << 16 && T <= 24 ? 3 : 0;
}

// The same kernel where the cells fill the chip, with the 64-interval tables that it takes instead of the multi-step kernel: three stages, and two on calls
// that move more than twice the last-level cache (20 bytes per pair and step).  us per launch, multi-step kernel / four stages / three / two:
// 262144 pairs T = 64 65.0 / 58.6 / 57.2 / -, T = 16 19.3 / 17.2 / 16.6 / -; 614400 T = 32 77.6 / 74.9 / 73.5 / -; 2^20 T = 16 61.9 / - / 57.1 / 58.3,
// T = 24 91.3 / - / 84.7 / 86.5, T = 32 129.7 / - / 128.1 / 125.0; 2^21 T = 12 93.6 / - / 86.2 / 86.3, T = 14 114.7 / - / 114.2 / 109.5, T = 16 130.1 / - / 135.5 / 128.7;
// 2^19 T = 64 132.0 / - / 120.3 / 120.9; rows of 2000 cells 400000 T = 32 59.6 / 56.6 / 52.9 / -, 1500000 T = 20 133.0 / - / 129.3 / 122.7.
// Rows of 64 cells and more off the cache lines, whose steps read more lines each, are better with two from 3 * 2^18 pairs on: two / three 790000 pairs of 200 cells T = 8 29.0 / 29.9,
// 1200000 of 104 T = 11 62.5 / 66.6, of 2000 T = 13 63.5 / 67.3, 2097152 of 200 T = 9 81.5 / 85.9, of 72 T = 10 93.8 / 98.4; 700000 of 200 T = 11 35.5 / 36.1, 600000 31.6 / 31.5,
// 540000 T = 9 +7 %; rows of 16 level, of 2048 T = 11 79.3 / 79.3.  (The multi-step kernel: 62.8 for the 1200000 of 104, 83.0 for the 2097152 of 200.)
inline unsigned full_ring_stages(unsigned T, unsigned n_pairs, unsigned long long H)
{
    if (H % 64 != 0 && H >= 64 && n_pairs >= 3u << 18) return 2;
    return (unsigned long long)T * n_pairs < 7ull << 22 ? 3 : 2;
}

// Where the sixteen wavefronts of a large block go in step (lstm_ring_kernel).  A block is 1024 pairs and a round of one block per compute unit 2^18: a round takes
// the same however few its blocks are, so that what a block gains it loses again in a last round that is mostly empty.  In the first round the other kernels, whose blocks are
// 256 pairs, have three of them on a compute unit up to 192 * 1024 pairs and take a fifth longer beyond.  Rows off the cache lines (H % 64) gain the
// most, from one round on; short ones gain less in a round and need more of the last.  Whole lines gain in two rounds and more, and up to eleven steps in one.  us per
// launch, other kernels / this, inputs partly in the cache:
//   rows of 2000 cells  T = 9   192 blocks 9.12 / 10.1, 196 11.5 / 9.98, 220 11.9 / 10.3, 256 13.0 / 11.3
//                       T = 12  420 21.6 / 22.4, 465 24.9 / 24.3, 512 26.5 / 25.8, 586 31.4 / 32.6, 635 34.4 / 33.2, 879 42.1 / 43.9, 938 45.4 / 44.4, 1075 52.9 / 53.2
//                       T = 16  440 28.7 / 29.4, 635 45.2 / 43.0, 879 55.9 / 56.8, 1075 70.9 / 69.7, 1563 100.1 / 98.3
//                       T = 20  633 57.7 / 55.3, 672 60.2 / 55.8, 732 63.1 / 58.7
//                       T = 40  192 31.5 / 34.5, 196 35.7 / 33.8, 220 38.5 / 35.0, 293 49.8 / 59.2, 469 76.8 / 68.5, 586 108.1 / 97.9, 879 156.5 / 147.5, 1172 215.8 / 197.1
//   of 104              T = 20  633 65.1 / 60.2, 1054 101.3 / 97.3, 1184 119.5 / 104.6
//   of 96               T = 20  1295 103.9 / 107.8, 1332 105.1 / 109.5, 1415 117.5 / 113.2, 1557 146.1 / 140.1
//   of 56               T = 18  644 58.9 / 55.5     T = 16  1065 82.5 / 83.9, 1281 98.6 / 88.7
//   of 48               T = 18  635 57.2 / 54.9     T = 20  1087 99.0 / 100.4, 1121 104.8 / 102.6     T = 16  1319 96.5 / 97.4, 1341 99.2 / 97.5, 1824 147.1 / 140.9
//   of 40               T = 20  633 65.1 / 65.7, 672 70.6 / 69.1, 1054 104.9 / 109.2, 1134 116.9 / 113.8, 1184 125.7 / 115.4, 1282 130.2 / 127.2, 1301 131.3 / 131.7, 1826 205.9 / 199.6
//   of 32               T = 18  1153 85.0 / 86.3     T = 20  1179 98.3 / 98.9, 1284 102.2 / 110.0, 1336 105.9 / 115.0, 1620 142.3 / 144.6, 2587 220.8 / 220.4     T = 16  1386 92.3 / 92.7
//   of 24               T = 18  683 73.1 / 72.1     T = 16  1163 110.6 / 106.5, 1300 117.7 / 122.9, 1379 125.3 / 124.9, 1597 143.9 / 144.9, 2579 241.3 / 241.8
//   of 16               T = 12  192 14.8 / 17.7, 196 18.9 / 17.8, 256 20.2 / 19.1     T = 40  192 44.0 / 50.4, 196 54.8 / 50.5, 256 59.5 / 54.7
//                       T = 16  633 59.1 / 64.0, 702 65.4 / 65.4, 732 68.7 / 66.1, 929 86.7 / 85.2, 1054 95.9 / 102.4, 1134 102.0 / 104.9, 1184 107.7 / 106.5, 1641 153.2 / 153.0
//                       T = 20  1329 148.9 / 157.3, 1406 163.7 / 164.7, 1566 178.2 / 186.8, 2610 317.8 / 319.1
//   of 2048             T = 8   224 9.3 / 8.8, 256 10.3 / 9.2, 512 16.4 / 17.7      T = 9  224 9.6 / 9.6, 248 10.2 / 9.8, 256 11.6 / 10.0
//                       T = 16  248 15.8 / 16.2, 256 16.5 / 16.3, 512 30.1 / 29.9, 640 38.6 / 40.4, 700 41.5 / 40.9, 768 44.4 / 43.1, 960 55.3 / 55.2, 1100 62.8 / 66.4
//                       T = 40  256 35.7 / 35.3, 432 61.5 / 61.7, 464 66.0 / 63.7, 512 71.0 / 68.1, 640 92.1 / 94.8, 700 101.5 / 96.6, 1024 157.5 / 153.3
//                       T = 96  470 174.6 / 175.1, 490 181.9 / 183.4 (the blocks of a round drift apart), 512 184.9 / 178.0
// The lines hold for all numbers of steps, at the price of long calls that would gain below them (T = 40, 586 and 879 blocks).  Folding 64-interval tables alike.
// Rows off the lines from five full rounds on, this to the others, means of 1500 to 3000 calls for each number of rounds, by the blocks in the last (1 to 31, 32 to 63, 64 to 95, 96 to 127): rows
// of 8 to 32 cells, five rounds 1.04, 1.04, 1.01, 0.99, six 1.02, 1.02, 1.00, 0.99, seven 1.01, 1.00, 1.00, 0.99, ten 1.00, 0.99, 0.99, 0.97; of 40 five 0.99, 0.98, 0.94, 0.93; of 96 1.00, 0.98, 0.95, 0.93.
inline bool rows_together(unsigned T, unsigned n_pairs, unsigned long long H)
{
    if (T < 8 || n_pairs == 0) return false;
    const unsigned blocks = (n_pairs + 1023u) / 1024u, full = (blocks - 1u) / 256u, last = blocks - 256u * full;
    if (H % 64 == 0) {
        if (full == 0) return T < 12 && last >= 240;
        return full == 1 ? T >= 24 && T <= 80 && last >= 208 : T >= 16 && last >= (full == 2 ? 188u : 240u);
    }
    if (full == 0) return last > 192;
    if (full > 4) return T >= 16 && last >= (H >= 40 ? 1u : full == 5 ? 96u : full == 6 ? 64u : 1u);
    if (full == 4) return T >= 16 && last >= (H < 40 ? 120u : H < 56 ? 64u : 1u);
    if (full == 2) return T >= 12 && last >= (H < 40 ? 176u : H < 48 ? 128u : 120u);
    return T >= 12 && last >= (full == 1 ? 208u : 160u);
}

// Whether the kernels for several steps of many cells work with two stages instead of four (ktanh_lstm_impl.h says why either).  The chip
// holds 2^19 pairs at a time (eight wavefronts per SIMD).  Two stages need it full, from six wavefronts on, and lose in a last
// round that is mostly empty: there a wavefront has few others beside it.  us per launch, four stages / two, all out of the
// cache: T = 32 393728 pairs 49.3 / 46.5, 435200 52.3 / 50.2, 2^19 59.6 / 59.5, 527360 61.9 / 75.3, 614400 75.3 / 79.7,
// 786432 92.6 / 91.6, 870400 107.1 / 102.4, 2^20 139.2 / 123.3; T = 16 1075200 63.4 / 63.8, 1280000 74.6 / 75.2, 1536000
// 92.4 / 89.0, 2^21 144.9 / 128.5.  With the 64-interval table, whose selects make a step longer, two gain only
// where a single round is nearly full and the steps are few (512000 pairs T = 10 25.5 / 23.2, T = 16 35.3 / 35.6, T = 32 64.1 / 69.3;
// 563200 pairs T = 12 28.8 / 31.7), or where a call moves more than twice the last-level cache (20 bytes per pair and
// step make 640 MiB at 2^25 pairs and steps: 2^19 pairs T = 64 136.5 / 127.6, 2^21 T = 16 142.8 / 129.1, 1536000 T = 32 197.7 / 193.5; but 665600 T = 64 175.5 / 182.7).
// Rows that do not fill lines make a wavefront's loads wait for more of them, which the other wavefronts have to cover as well: two
// stages do not gain on short rows (400000 pairs of rows of 8 cells T = 40 95.6 / 103.5, 524288 of 56 T = 16 39.2 / 42.8), nor in a full
// round on rows of 32 or below 160 cells (524288 of 72 39.3 / 42.3, of 104 38.9 / 40.6, of 184 38.7 / 38.1; 460000 of 72 38.4 / 38.1;
// 1000000 of 72 75.6 / 79.0).
// Behind a full round they need less of a last one to gain (rows of 1000: 560000 pairs T = 16 +12 %, 614400 -3 %, 720000 -4 %; rows of 1024:
// 614400 +5 %, 716800 +2 %).
// Ten and eleven steps leave four stages a tail of six or seven with loads that wait for each other (870000 pairs of rows of 1000,
// 64 intervals, T = 10 43.8 / 41.2).
// Up to seven steps have kernels of their own (lstm_short_kernel), for which the last round counts less.
inline bool shallow_ring(bool wide, unsigned T, unsigned n_pairs, unsigned long long H)
{
    constexpr unsigned round = 1u << 19, some = 5u << 14;
    if (T < 8) return n_pairs >= (wide ? round : 3u << 17);
    const unsigned full = (n_pairs - 1u) / round, last = n_pairs - full * round;  // rounds before the last, pairs in it
    const bool large = (unsigned long long)T * n_pairs >= 1ull << 25;
    if (wide && full == 0) return last > 15u << 15 && (T < 16 || large);
    if (cell_rows_are_short(H)) return false;
    if (full != 0 && last >= some && (T == 10 || T == 11)) return true;
    if (wide) return n_pairs >= 3u << 18 && large;
    if (full < 2 && last > 29u << 14 && (H == 32 || (H < 160 && H % 32 != 0))) return false;
    if (full == 0) return last >= 3u << 17;
    return full > 2 || last >= (H % 32 == 0 ? round / (2 * full) : some);
}

// The table that the cell reads: 32 intervals, 64, or 64 of a table that folds (ktanh_cell.h).
enum CellTable { CELL32, CELL64, CELL64_FOLDED };

// Which kernel takes a call of the cell: a single step (cell_step_form); chunks of time, of `n` steps; the ring of ktanh_lstm_ring.hip in lockstep, or
// with `n` stages; steps written out, or the multi-step kernel, with `n` stages.
enum CellKernel { CELL_ONE_STEP, CELL_CHUNKS, CELL_RING_TOGETHER, CELL_RING, CELL_WRITTEN_OUT, CELL_MULTI_STEP };

struct CellForm {
    CellKernel kernel;
    unsigned n;
};

constexpr unsigned kDeepStages = 4, kShallowStages = 2;  // of the kernels for several steps of many cells (ktanh_lstm_impl.h)
constexpr unsigned kTogetherStages = 3;

// `aligned`: the tensors start on a 128-byte cache line.
inline CellForm cell_form(CellTable table, unsigned T, unsigned n_pairs, unsigned long long H, bool aligned = true)
{
    if (T == 1) return CellForm{CELL_ONE_STEP, 0};
    const unsigned steps = chunk_steps(T, n_pairs);
    if (steps != 0) return CellForm{CELL_CHUNKS, steps};
    // a table that does not fold has no form of the lockstep kernel
    if (table != CELL64 && rows_together(T, n_pairs, H)) return CellForm{CELL_RING_TOGETHER, kTogetherStages};
    const unsigned stages = ring_stages(T, n_pairs, H, aligned);
    if (stages != 0) return CellForm{CELL_RING, stages};
    const bool shallow = shallow_ring(table == CELL64, T, n_pairs, H);
    if (T < (shallow ? 6u : 8u)) return CellForm{CELL_WRITTEN_OUT, shallow ? kShallowStages : kDeepStages};
    // a table that folds has no form of the multi-step kernel: the ring is ahead of it everywhere
    if (table == CELL64_FOLDED) return CellForm{CELL_RING, full_ring_stages(T, n_pairs, H)};
    return CellForm{CELL_MULTI_STEP, shallow ? kShallowStages : kDeepStages};
}

}  // namespace ktanh_device

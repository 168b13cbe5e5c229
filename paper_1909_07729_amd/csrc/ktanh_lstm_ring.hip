// libktanh: the fused LSTM cell over many time steps, one lane per pair of cells: where the cells do not fill the chip, and in lockstep where they do.
#include "ktanh_lstm_impl.h"

namespace ktanh_device {

// The multi-step kernel (lstm_cell_kernel) for two to four wavefronts per SIMD, where nothing but the wavefront itself hides
// a latency: its time is the number of steps times what one wavefront needs for a step.  So a step here
//   waits for its table reads once instead of five times (ktanh_cell.h);
//   asks for the words of the step STAGES ahead before it does anything else, into the registers that the step before has
//   emptied: a whole step more of lead than a refill behind the step, with the same registers (in the first step of the unrolled body the
//   compiler puts them behind the step's table reads);
//   stores its outputs where the compiler can count them (store_counted), with no branch around a load or store, so that it waits for its own
//   four words and not for the stores before them and younger words.
// us per launch, multi-step kernel -> the first of these alone -> all: 64 steps of [128, 2048] cells 35.8 -> 32.0 -> 29.6 (the bytes
// take 26), [112, 2048] 34.6 -> 30.9 -> 27.9, [160, 2048] 41.1 -> 39.1 -> 38.4, [192, 2048] 44.7 -> 43.5 -> 43.3; 24 of [128, 2048] 15.6 -> 12.7; 16 of
// [160, 2048] 12.9 -> 12.0, [256, 2048] 16.9 -> 16.3; rows off the cache lines 64 of [128, 2000] 37.3 -> 31.6, 9 of [250, 2000] 12.0 -> 10.7.
// Blocks of 64 and 128 threads are level on whole lines and up to 18 % slower elsewhere ([176, 2048] 40.6 / 47.3 / 42.1).
// Stages and range: ring_stages in ktanh_order.h.
//
// THREADS = 1024: the same where the chip is full, in blocks of sixteen wavefronts, one or two on a compute unit, that wait for each
// other after every step.  Left alone, neighbouring wavefronts drift steps apart, so that a line that two of them share is read twice (rows of 2000 cells, 500 of them T = 40:
// the kernel for many cells reads 1.17 times the bytes, this 1.05 times) and more steps' matrices, megabytes apart, are read at once; the same accesses with
// no arithmetic take 56.5 us alone and 52.2 together (262144 pairs, T = 64, whole lines, where both read each byte once; with it 57.7 and 57.2), 78.7 and 69.7 (the rows of 2000, 85.0 and 72.3).  us per launch, kernels for many cells -> this: rows of 2000 cells 250 of them T = 40 40.0 -> 37.0,
// 500 T = 16 31.9 -> 30.5, T = 40 78.8 -> 70.5, 1000 T = 40 176 -> 155; of 104 4923 T = 40 46.4 -> 39.4; of 40 24064 T = 40 98.7 -> 83.8; whole lines [512, 2048]
// T = 40 72.6 -> 68.2, [768, 2048] 111.7 -> 103.6, [256, 2048] T = 8 10.3 -> 9.2; 64 intervals 500 rows of 2000 T = 32 68.8 -> 56.6.  Two stages with a barrier
// per two steps 3-8 % slower, four stages 0-2 %; counted stores level, 4 % slower on 2^21 pairs.  Blocks are too large to balance a round that is
// not nearly full: rows_together in ktanh_order.h.  (A barrier waits for the wavefronts of the block that are still running, so that the ones that
// returned at the start do not hold it up, and all others take it as often as T says.)
template <CellTable TAB, int STAGES, int THREADS>
__global__ __launch_bounds__(THREADS) void lstm_ring_kernel(const uint32_t *__restrict__ gates, const float2 *c_in,
                                                             float2 *c_out,  // may be c_in
                                                             uint32_t *__restrict__ h_out, unsigned T, unsigned n_pairs,
                                                             unsigned H2, unsigned row_mul,
                                                             unsigned row_shift,  // row_of_pair
                                                             unsigned always_checked, KtLutPack pack)
{
    const LaneTable tab(pack);
    const unsigned mine = blockIdx.x * THREADS + threadIdx.x;
    if ((unsigned)__builtin_amdgcn_readfirstlane((int)mine) >= n_pairs) return;  // the whole wavefront is past the end
    // Lanes past the end repeat the last pair, which is in their own wavefront, and store the same words to the
    // same place, so that no access has a branch around it.
    const unsigned p = mine < n_pairs ? mine : n_pairs - 1;
    const unsigned long long row_step = 4ull * n_pairs;  // gate words per time step
    GateOffsets at = gate_offsets(p, H2, row_mul, row_shift);
    unsigned h_at = 4u * p;  // byte offset of this lane's output word inside one step of h

    float2 c = c_in[p];
    GateWords stage[STAGES];
    const uint32_t *ahead = gates;  // the next step to fetch
    uint32_t *h_row = h_out;        // the next step to store
#pragma unroll
    for (int s = 0; s < STAGES; ++s) {
        stage[s] = load_gates(ahead, at);
        ahead += row_step;
    }
    bool watch = true;
    Acts a = gate_activations<TAB>(stage[0], tab);
    const bool always = always_checked != 0;
    auto store = [&](uint32_t *row, uint32_t h) {
        if constexpr (THREADS == kLargeBlock) store_stream(row, h_at, h);
        else store_counted(row, h_at, h);
    };

    unsigned t = 0;
    for (; t + 2u * STAGES <= T; t += STAGES) {
#pragma unroll
        for (int s = 0; s < STAGES; ++s) {
            stage[s] = load_gates(ahead, at);
            ahead += row_step;
            const uint32_t h = step_and_look_up<TAB>(a, watch, stage[(s + 1) % STAGES], c, always, tab);
            store(h_row, h);
            h_row += n_pairs;
            if constexpr (THREADS == kLargeBlock) __builtin_amdgcn_s_barrier();
        }
    }
    // the last steps, fewer than twice the ring: stage k % STAGES holds step t + k
#pragma unroll
    for (int k = 0; k < 2 * STAGES - 1; ++k) {
        if (t + k < T) {
            if (k < STAGES && t + k + STAGES < T) {
                stage[k % STAGES] = load_gates(ahead, at);
                ahead += row_step;
            }
            uint32_t h;
            if (t + k + 1 < T) h = step_and_look_up<TAB>(a, watch, stage[(k + 1) % STAGES], c, always, tab);
            else h = closing_step<TAB>(a, c, tab);
            store(h_row, h);
            h_row += n_pairs;
        }
    }
    store_stream(c_out, 8u * p, c);
}

template <CellTable TAB>
ktanh_status_t launch_cell_ring(const CellCall &a, CellForm form, bool within_unit, const KtLutPack &pack,
                                ktanh_stream_t stream)
{
    auto launch = [&](auto kernel, unsigned threads) {
        return launch_checked(kernel, (a.n_pairs + threads - 1) / threads, threads, stream, a.gates, a.c_in, a.c_out, a.h_out,
                              a.T, a.n_pairs, a.H2, a.row.mul, a.row.shift, within_unit ? 0u : 1u, pack);
    };
    if (form.kernel == CELL_RING_TOGETHER) {
        if constexpr (TAB != CELL64) return launch(lstm_ring_kernel<TAB, kTogetherStages, kLargeBlock>, kLargeBlock);
        else return KT_ERR_SHAPE;  // cell_form gives it to the other tables only
    }
    if constexpr (TAB == CELL64_FOLDED) {
        if (form.n == 2) return launch(lstm_ring_kernel<TAB, 2, kCellBlock>, kCellBlock);
    }
    return form.n == 4 ? launch(lstm_ring_kernel<TAB, 4, kCellBlock>, kCellBlock)
                       : launch(lstm_ring_kernel<TAB, 3, kCellBlock>, kCellBlock);
}

template ktanh_status_t launch_cell_ring<CELL32>(const CellCall &, CellForm, bool, const KtLutPack &, ktanh_stream_t);
template ktanh_status_t launch_cell_ring<CELL64>(const CellCall &, CellForm, bool, const KtLutPack &, ktanh_stream_t);
template ktanh_status_t launch_cell_ring<CELL64_FOLDED>(const CellCall &, CellForm, bool, const KtLutPack &, ktanh_stream_t);

}  // namespace ktanh_device

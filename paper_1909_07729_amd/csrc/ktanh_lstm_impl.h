// Internal to libktanh: the fused LSTM-cell kernel and its launcher, shared by the entry points
// (ktanh_lstm.hip) and by the measurement yardstick (ktanh_probe.hip), so that the yardstick is the
// very same launch with the arithmetic taken out.
#pragma once
#include "ktanh_cell.h"

namespace ktanh_device {

// ---------------------------------------------------------------------------------------------
// LSTM cell: each lane owns two neighbouring cells of one batch row (one packed BFloat16 pair per
// gate) and carries their state through all T steps.  The work per cell is about forty vector
// instructions against ten bytes of traffic, so the kernel wants many wavefronts per SIMD to overlap
// arithmetic with memory rather than wide accesses; a wavefront's loads still cover 256 contiguous
// bytes each.  The steps of one lane are sequential, so the gate words of the next few steps are
// already on their way while a step is computed (a ring of register stages): without that the loop
// would pay one full memory latency per step.  The gate non-linearities of a step are formed one step
// early, under the wait for the previous step's K(c').
//
// How many stages: shallow_ring in ktanh_order.h decides.  Four cover the latency by themselves.  Two do not: a step's words are asked for at
// the end of the step before, so each step waits for memory and only the other wavefronts of the SIMD fill the
// time.  Where there are enough of those, two are better all the same, because the steps' gate matrices lie megabytes apart and
// the fewer of them are being read at once the better the memory does.  us per launch with 4 / 3 / 2 stages: 262144 pairs T = 8
// 10.2 / 11.6 / 11.1, T = 64 56.3 / 68.6 / 71.3; 524288 pairs T = 8 18.7 / 18.6 / 17.3, T = 12 25.6 / 25.2 / 24.0,
// T = 32 60.7 / 59.4 / 58.0; 2^20 pairs T = 8 32.1 / 33.0 / 31.2, T = 16 59.5 / 58.9 / 57.9; 393216 pairs T = 8 14.6 / 14.9 /
// 13.9, T = 32 45.4 / 46.2 / 45.6.  Four stages with half the wavefronts kept off the chip are no better (T = 32 58.0, T = 8 19.4).
constexpr int kCellBlock = 256, kLargeBlock = 1024;  // four and sixteen wavefronts per block

// Byte offsets of a lane's four gate words inside one time step's [B][4H] gate matrix: 32-bit, so
// that each load is "uniform 64-bit base + 32-bit lane offset" and needs no address arithmetic.
struct GateOffsets {
    unsigned i, f, g, o;
};

// Pair p = row * H2 + j has its i gate at word row * 4 * H2 + j = p + row * 3 * H2 of [B][4H].  The byte
// offsets stay below 16 * n_pairs <= 2^32 (checked by the caller).
__device__ __forceinline__ GateOffsets gate_offsets(unsigned p, unsigned H2, unsigned row_mul, unsigned row_shift)
{
    GateOffsets at;
    at.i = 4u * (p + row_of_pair(p, row_mul, row_shift) * (3u * H2));
    at.f = at.i + 4u * H2;
    at.g = at.f + 4u * H2;
    at.o = at.g + 4u * H2;
    return at;
}

// Gate words are read once: with many steps the non-temporal hint measured 4-6 % faster than a plain load.
template <bool STREAMED = true>
__device__ __forceinline__ GateWords load_gates(const uint32_t *step_base, GateOffsets &at)
{
    // The empty statement re-defines the four 32-bit offsets right where they are used, so that
    // each access is selected as "scalar base + 32-bit vector offset"; otherwise their 64-bit
    // extensions are hoisted out of the loop and every access pays a 64-bit vector add.
    asm volatile("" : "+v"(at.i), "+v"(at.f), "+v"(at.g), "+v"(at.o));
    GateWords q;
    q.i = load_at<STREAMED>(step_base, at.i);
    q.f = load_at<STREAMED>(step_base, at.f);
    q.g = load_at<STREAMED>(step_base, at.g);
    q.o = load_at<STREAMED>(step_base, at.o);
    return q;
}

// NANS = false is the same arithmetic without the NaN rules of K-TanH; it is exact whenever no gate
// word holds a NaN.
template <bool NANS, bool WIDE>
__device__ __forceinline__ Acts activations(const GateWords &q, const LaneTable &tab)
{
    Acts a;
    ksigmoid_f32_pair<NANS, WIDE, true>(q.i, tab, a.i_lo, a.i_hi);
    ksigmoid_f32_pair<NANS, WIDE, true>(q.f, tab, a.f_lo, a.f_hi);
    ksigmoid_f32_pair<NANS, WIDE, true>(q.o, tab, a.o_lo, a.o_hi);
    a.g2 = whole_pair<WIDE>(ktanh_pair<NANS, WIDE>(q.g, tab));
    return a;
}

// The state update and the hidden outputs of one step from its activations, with the full NaN rules
// (exact for any input).
template <bool WIDE>
__device__ __forceinline__ uint32_t finish_step_checked(const Acts &a, float2 &c, const LaneTable &tab)
{
    advance_state(a, c);
    const uint32_t tc2 = whole_pair<WIDE>(ktanh_pair<true, WIDE>(narrow_pair(c.x, c.y), tab));
    return narrow_pair(a.o_lo * widen_lo(tc2), a.o_hi * widen_hi(tc2));
}

// True for the whole wavefront when some lane holds a NaN in one of its four gate words.
__device__ __forceinline__ bool gates_hold_nan(const GateWords &q)
{
    const uint32_t worst = max_pair(max_pair(q.i & kMag2, q.f & kMag2),
                                    max_pair(q.g & kMag2, q.o & kMag2));
    return __builtin_amdgcn_ballot_w64(nan_bits_pair(worst) != 0u) != 0;
}

// One time step, and the activations of the next one.  `a` holds the activations of this step and
// is replaced by those of the step whose gate words are `next`; `a_checked` says (for the whole
// wavefront) whether `a` was formed under the NaN rules, i.e. may hold a NaN.
//
// The steps of a lane form one dependent chain (state -> K(state) -> output), and each K costs a
// round trip through the cross-lane unit.  With only four wavefronts per SIMD that latency is not
// hidden by other wavefronts, so it is hidden inside the wavefront: the table reads for K(c') are
// put in flight, the next step's activations (four independent K evaluations) are formed while they
// travel, and only then is K(c') finished.
//
// NaNs are rare: the fast path drops the NaN rules and runs only when no lane of the wavefront needs
// them (wavefront-uniform branches, so that the cross-lane table reads still run with every lane
// enabled).  The step of ktanh_cell.h in its place is level with the 32-interval table and up to 4 % faster with a 64-interval one (us per launch, this / that:
// [256, 2048] cells T = 64 60.5 / 59.2, [512, 2048] T = 16 30.8 / 31.0, 8437 rows of 64 T = 64 64.9 / 65.6; 64 intervals [512, 2048] T = 16 35.3 / 33.8).  `suspect` is a per-lane flag word (non-zero = this lane's state may not be finite);
// always_checked: the caller's table lets |K| exceed 1, so the state may overflow on the way.
template <bool WIDE>
__device__ __forceinline__ uint32_t step_and_look_ahead(Acts &a, bool &a_checked, const GateWords &next,
                                                        float2 &c, uint32_t &suspect,
                                                        uint32_t always_checked, const LaneTable &tab)
{
    const bool next_checked = gates_hold_nan(next);
    const bool now_checked = a_checked || __builtin_amdgcn_ballot_w64(suspect != 0u) != 0;
    uint32_t h;
    if (!now_checked && !next_checked) {
        // exact here: no gate is a NaN, the incoming state is finite and |K| <= 1, so the state
        // stays finite (|c'| <= |c| + 1)
        advance_state(a, c);
        const uint32_t cb = narrow_pair(c.x, c.y);
        const uint32_t mag2 = cb & kMag2;
        const SlotPair sp = fetch_slots<WIDE>(mag2, tab);
        const Acts ahead = activations<false, WIDE>(next, tab);
        const uint32_t tc2 = whole_pair<WIDE>(bitsel(kMag2, finish_mag_pair<WIDE>(mag2, sp), cb));
        h = narrow_pair(a.o_lo * widen_lo(tc2), a.o_hi * widen_hi(tc2));
        a = ahead;
    } else {
        h = finish_step_checked<WIDE>(a, c, tab);
        suspect = always_checked | not_finite(c.x) | not_finite(c.y);
        a = activations<true, WIDE>(next, tab);
    }
    a_checked = next_checked;
    return h;
}

// The last step of a call: no next gate words to look at.
template <bool WIDE>
__device__ __forceinline__ uint32_t last_step(const Acts &a, float2 &c, const LaneTable &tab)
{
    return finish_step_checked<WIDE>(a, c, tab);
}

// ARITH = false is the measurement form of the kernel: the same loads, stores, waits and loop with
// the arithmetic taken out.  A step's output word is then the XOR of its four gate words and the
// bits of the lane's first state value (so that no load can be dropped), formed one step ahead like
// the activations, and the state passes through unchanged.
__device__ __forceinline__ uint32_t fold(const GateWords &q) { return q.i ^ q.f ^ q.g ^ q.o; }

template <bool WIDE, bool ARITH>
__device__ __forceinline__ uint32_t one_step(Acts &a, bool &a_checked, const GateWords &next, float2 &c,
                                             uint32_t &suspect, uint32_t always_checked,
                                             const LaneTable &tab)
{
    if constexpr (ARITH) {
        return step_and_look_ahead<WIDE>(a, a_checked, next, c, suspect, always_checked, tab);
    } else {
        const uint32_t h = a.g2 ^ __float_as_uint(c.x);
        a.g2 = fold(next);
        return h;
    }
}

template <bool WIDE, bool ARITH>
__device__ __forceinline__ uint32_t final_step(const Acts &a, float2 &c, const LaneTable &tab)
{
    if constexpr (ARITH) return last_step<WIDE>(a, c, tab);
    else return a.g2 ^ __float_as_uint(c.x);
}

template <bool WIDE, bool ARITH, int STAGES>
__global__ __launch_bounds__(kCellBlock) void lstm_cell_kernel(const uint32_t *__restrict__ gates,
                                                           const float2 *c_in, float2 *c_out,  // may be equal
                                                           uint32_t *__restrict__ h_out, unsigned T,
                                                           unsigned n_pairs, unsigned H2,
                                                           unsigned row_mul, unsigned row_shift,  // row_of_pair
                                                           unsigned always_checked, KtLutPack pack)
{
    const LaneTable tab(pack);
    const unsigned p = blockIdx.x * kCellBlock + threadIdx.x;
    const bool live = p < n_pairs;
    // Lanes past the end work on pair 0 and store nothing: every lane then issues every load, with
    // no branch around it, which lets each step wait for exactly its own gate words (a load that
    // only some paths issue makes the wait cover everything in flight).
    const unsigned p_read = live ? p : 0;
    const unsigned long long row_step = 4ull * n_pairs;  // gate words per time step
    GateOffsets at = gate_offsets(p_read, H2, row_mul, row_shift);
    const unsigned h_at = 4u * p;  // byte offset of this lane's output word inside one step of h

    float2 c = c_in[p_read];  // first in the queue: its wait leaves the gate words in flight
    GateWords stage[STAGES];
    const uint32_t *ahead = gates;  // the next step to fetch
    uint32_t *h_row = h_out;        // the next step to store
    unsigned t = 0;

    const bool ring = T >= 2u * STAGES;
#pragma unroll
    for (int s = 0; s < STAGES; ++s) {
        stage[s] = GateWords{0u, 0u, 0u, 0u};
        if (ring || s < (int)T) {  // uniform over the grid
            stage[s] = load_gates(ahead, at);
            ahead += row_step;
        }
    }
    uint32_t suspect = always_checked | not_finite(c.x) | not_finite(c.y);
    // the activations of step 0, under the full rules (once per call)
    Acts a = Acts{};
    if constexpr (ARITH) a = activations<true, WIDE>(stage[0], tab);
    else a.g2 = fold(stage[0]);
    bool a_checked = true;

    if (ring) {
        // Steady state: stage s holds the gate words of the current step, stage s + 1 those of the
        // next; each stage is refilled right after the step that consumed it, in place (the refill
        // follows the step's last use of the old words, so that no register copies -- which would
        // have to wait for every load in flight -- are needed at the end of the body).
        for (; t + 2u * STAGES <= T; t += STAGES) {
#pragma unroll
            for (int s = 0; s < STAGES; ++s) {
                const uint32_t h = one_step<WIDE, ARITH>(a, a_checked, stage[(s + 1) % STAGES], c,
                                                         suspect, always_checked, tab);
                if (live) store_stream(h_row, h_at, h);
                h_row += n_pairs;
                stage[s] = load_gates(ahead, at);
                ahead += row_step;
            }
        }
    }

    // The last steps (fewer than 2 * STAGES): stage k % STAGES holds step t + k.  Written out step
    // by step with the stages named statically, like the steady loop: moving the ring up through
    // register copies instead would make every one of these steps wait for all loads in flight,
    // a full memory latency each.  All conditions are uniform over the grid.
#pragma unroll
    for (int k = 0; k < 2 * STAGES - 1; ++k) {
        if (t + k < T) {
            constexpr int kRing = STAGES;
            const int s = k % kRing;
            uint32_t h;
            if (t + k + 1 < T)
                h = one_step<WIDE, ARITH>(a, a_checked, stage[(s + 1) % kRing], c, suspect,
                                          always_checked, tab);
            else
                h = final_step<WIDE, ARITH>(a, c, tab);
            if (live) store_stream(h_row, h_at, h);
            h_row += n_pairs;
            if (k < kRing && t + k + kRing < T) {
                stage[s] = load_gates(ahead, at);
                ahead += row_step;
            }
        }
    }
    if (live) c_out[p] = c;
}

// One time step per call, the form a recurrent network makes: nothing to prefetch or to carry, so the
// kernel is a plain stream of 18 bytes per cell, one pair per lane, written through to the last-level cache for
// the matrix product and the step that come next.  (Two pairs per lane measured 2-5 % slower, four 20-40 %.)
// What it gains over the multi-step kernel lies in inputs that come from that cache: [256, 2048] cells 3.06 -> 2.24 us per launch
// with three inputs in turn, 3.63 -> 3.69 with all of them out of the cache ([512, 2048] 4.24 -> 3.38, 5.21 -> 5.21; [1024, 2048]
// 8.22 -> 6.75, 8.97 -> 8.30).  The form is chosen by cell_step_form.
// NEAR: plain loads; the others carry the non-temporal hint, without which calls that move more than 72 MiB are 10-17 % slower.
// us per launch; the three figures of a form are for three inputs and two outputs in turn, sixteen, and sixty-four:
//                    64 threads, hint     64 threads, plain    256 threads, plain
//   [8, 1024] cells  1.72  1.72  1.75     1.72  1.72  1.72     1.76  1.76  1.75   (an empty launch 1.7)
//   [64, 1024]       1.84  2.06  2.11     1.76  1.77  1.94     1.79  1.79  1.98
//   [128, 2048]      2.26  2.49  2.48     2.24  2.21  2.21     1.89  2.20  2.27
//   [256, 2048]      2.66  3.46  3.45     2.67  2.79  3.46     2.37  2.65  3.15
//   [512, 2048]      4.45  4.80  4.80     4.08  4.11  4.82     3.43  3.84  4.86
//   [1024, 2048]     6.66  7.29  7.29     6.63  7.30  7.32     5.85  7.76  7.86
//   [4096, 1024]    12.22 12.26 12.25    11.85 12.28 12.26    11.58 12.97 13.03
// so blocks of 256 threads serve the middle (2^16 to 2^19 pairs), where a quarter of the dispatches counts for more than a
// wavefront's place being free at once, and blocks of one wavefront the rest.
// RUNS, on calls that move more than 72 MiB: each XCD takes runs of neighbouring pieces (tile_of_block_in_runs), because rows that do
// not fill cache lines make neighbours share one, which a load with the hint fetches twice.  us per launch, three in turn / out of
// the cache, 256 threads in the multi-step kernel | 64 threads in the plain order | in runs:
//   [3000, 3000]   27.4 / 29.7 | 28.6 / 31.9 | 24.8 / 26.7      [8000, 4000]   93.9 / 93.8 | 101.6 / 101.8 | 88.4 / 88.4
//   [3000, 3072]   27.6 / 29.1 | 24.9 / 26.7 | 25.1 / 26.7 (whole lines: level)
//   [700000, 8]    20.7 / 23.0 | 21.5 / 22.3 | with plain loads (short rows) 16.2 / 18.7
//   [200000, 40]   25.8 / 27.9 | 27.3 / 28.9 | 22.5 / 25.3
//   [400000, 32]   38.6 / 40.8 | 35.6 / 37.8 | 39.8 / 40.4 (half lines: not short)
template <CellTable TAB, int THREADS, bool NEAR, bool RUNS>
__global__ __launch_bounds__(THREADS) void lstm_step_kernel(unsigned n_pairs, unsigned H2, unsigned row_mul,
                                                          unsigned row_shift,  // row_of_pair
                                                          const uint32_t *__restrict__ gates,
                                                          const float2 *c_in, float2 *c_out,  // may be equal
                                                          uint32_t *__restrict__ h_out, KtLutPack pack)
{
    static_assert(!RUNS || THREADS == kBlock, "a tile of the runs is one wavefront");
    const LaneTable tab(pack);
    const unsigned tile = RUNS ? tile_of_block_in_runs(blockIdx.x, cell_run_tiles(n_pairs), 0, 18) : blockIdx.x;
    const unsigned p = tile * THREADS + threadIdx.x;
    const bool live = p < n_pairs;
    const unsigned p_read = live ? p : 0;  // lanes past the end work on pair 0 and store nothing
    GateOffsets at = gate_offsets(p_read, H2, row_mul, row_shift);
    const GateWords q = load_gates<!NEAR>(gates, at);
    float2 c = load_at<!NEAR>(c_in, 8u * p_read);
    const uint32_t h = closing_step<TAB>(gate_activations<TAB>(q, tab), c, tab);
    if (live) {
        store_stream(h_out, 4u * p, h);
        store_stream(c_out, 8u * p, c);
    }
}

// A few time steps of many cells, their number T known to the compiler: the steps are written out, STAGES of them
// ahead, so that each waits for exactly its own words.  In the multi-step kernel a call with fewer steps than
// twice its ring has conditional loads, whose waits cover everything in flight.  T = 2 to 7 with four stages, 2 to 5
// with two.  us per launch, multi-step kernel with four stages -> all words at once -> this: 262144 pairs T = 4
// 6.6 -> 5.8 -> 5.7, T = 7 10.8 -> 9.2 -> 8.8; 524288 pairs T = 3 9.1 -> 8.9 -> 8.2, T = 4 11.8 -> 10.9 -> 10.1, T = 5
// 14.8 -> 13.5 -> 12.1 (multi-step kernel with two stages 10.8 and 12.7, from T = 6 on level or ahead).
template <CellTable TAB, int T, int STAGES>
__global__ __launch_bounds__(kCellBlock) void lstm_short_kernel(const uint32_t *__restrict__ gates, const float2 *c_in,
                                                             float2 *c_out,  // may be c_in
                                                             uint32_t *__restrict__ h_out, unsigned n_pairs,
                                                             unsigned H2, unsigned row_mul,
                                                             unsigned row_shift,  // row_of_pair
                                                             unsigned always_checked, KtLutPack pack)
{
    const LaneTable tab(pack);
    const unsigned p = blockIdx.x * kCellBlock + threadIdx.x;
    const bool live = p < n_pairs;
    const unsigned p_read = live ? p : 0;  // lanes past the end work on pair 0 and store nothing
    GateOffsets at = gate_offsets(p_read, H2, row_mul, row_shift);
    float2 c = load_at<true>(c_in, 8u * p_read);
    GateWords q[T];
#pragma unroll
    for (int t = 0; t < T && t < STAGES; ++t) q[t] = load_gates(gates + 4ull * n_pairs * t, at);
    bool watch = true;
    Acts a = gate_activations<TAB>(q[0], tab);
#pragma unroll
    for (int t = 0; t < T; ++t) {
        uint32_t h;
        if (t + 1 < T) h = step_and_look_up<TAB>(a, watch, q[(t + 1) % T], c, always_checked != 0, tab);
        else h = closing_step<TAB>(a, c, tab);
        if (live) store_stream(h_out + (unsigned long long)n_pairs * t, 4u * p, h);
        if (t + STAGES < T) q[(t + STAGES) % T] = load_gates(gates + 4ull * n_pairs * (t + STAGES), at);
    }
    if (live) store_stream(c_out, 8u * p, c);
}

// A checked call, as the launchers take it.
struct CellCall {
    const uint32_t *gates;
    const float2 *c_in;
    float2 *c_out;
    uint32_t *h_out;
    unsigned T, n_pairs, H2;
    RowDivision row;
    bool aligned;  // the tensors start on a cache line
};

// Chunks of time (ktanh_lstm_chunks.hip).
template <CellTable TAB>
ktanh_status_t launch_cell_chunks(const CellCall &call, unsigned steps, const KtLutPack &pack, ktanh_stream_t stream);

// CELL_RING_TOGETHER and CELL_RING (ktanh_lstm_ring.hip).
template <CellTable TAB>
ktanh_status_t launch_cell_ring(const CellCall &call, CellForm form, bool within_unit, const KtLutPack &pack,
                                ktanh_stream_t stream);

// CELL_WRITTEN_OUT.
template <CellTable TAB, int STAGES>
ktanh_status_t launch_cell_written_out(const CellCall &a, bool within_unit, const KtLutPack &pack, ktanh_stream_t stream)
{
    auto launch = [&](auto kernel) {
        return launch_checked(kernel, (a.n_pairs + kCellBlock - 1) / kCellBlock, kCellBlock, stream, a.gates, a.c_in, a.c_out,
                              a.h_out, a.n_pairs, a.H2, a.row.mul, a.row.shift, within_unit ? 0u : 1u, pack);
    };
    switch (a.T) {
        case 2: return launch(lstm_short_kernel<TAB, 2, STAGES>);
        case 3: return launch(lstm_short_kernel<TAB, 3, STAGES>);
        case 4: return launch(lstm_short_kernel<TAB, 4, STAGES>);
        case 5: return launch(lstm_short_kernel<TAB, 5, STAGES>);
        default: break;
    }
    if constexpr (STAGES == kDeepStages) {
        if (a.T == 6) return launch(lstm_short_kernel<TAB, 6, STAGES>);
        if (a.T == 7) return launch(lstm_short_kernel<TAB, 7, STAGES>);
    }
    return KT_ERR_SHAPE;  // cell_form gives this kernel no other number of steps
}

// CELL_MULTI_STEP; the yardstick (ARITH = false) takes this kernel whatever the size.
template <bool WIDE, bool ARITH>
ktanh_status_t launch_cell_multi_step(const CellCall &a, unsigned stages, bool within_unit, const KtLutPack &pack,
                                      ktanh_stream_t stream)
{
    auto launch = [&](auto kernel) {
        return launch_checked(kernel, (a.n_pairs + kCellBlock - 1) / kCellBlock, kCellBlock, stream, a.gates, a.c_in, a.c_out,
                              a.h_out, a.T, a.n_pairs, a.H2, a.row.mul, a.row.shift, within_unit ? 0u : 1u, pack);
    };
    return stages == kDeepStages ? launch(lstm_cell_kernel<WIDE, ARITH, kDeepStages>)
                                 : launch(lstm_cell_kernel<WIDE, ARITH, kShallowStages>);
}

inline ktanh_status_t pack_cell(const ktanh_lut_t *lut, KtLutPack *pack, bool *within_unit, bool *folds)
{
    *folds = false;
    return kt_pack_lut_bf16(lut, pack, within_unit);
}
inline ktanh_status_t pack_cell(const ktanh_lut64_t *lut, KtLutPack *pack, bool *within_unit, bool *folds)
{
    return kt_pack_lut64_bf16(lut, pack, within_unit, folds);
}

// A single step.
template <CellTable TAB>
ktanh_status_t launch_cell_step(const CellCall &a, const KtLutPack &pack, ktanh_stream_t stream)
{
    auto launch = [&](auto kernel, unsigned threads) {
        return launch_checked(kernel, (a.n_pairs + threads - 1) / threads, threads, stream, a.n_pairs, a.H2, a.row.mul,
                              a.row.shift, a.gates, a.c_in, a.c_out, a.h_out, pack);
    };
    switch (cell_step_form(a.n_pairs, 2 * a.H2)) {
        case STEP_STREAMED: return launch(lstm_step_kernel<TAB, kBlock, false, true>, kBlock);
        case STEP_SHORT_ROWS: return launch(lstm_step_kernel<TAB, kBlock, true, true>, kBlock);
        case STEP_FOUR_WAVES: return launch(lstm_step_kernel<TAB, kCellBlock, true, false>, kCellBlock);
        default: return launch(lstm_step_kernel<TAB, kBlock, true, false>, kBlock);
    }
}

template <CellTable TAB>
ktanh_status_t launch_cell_with(const CellCall &a, bool within_unit, const KtLutPack &pack, ktanh_stream_t stream)
{
    const CellForm form = cell_form(TAB, a.T, a.n_pairs, 2 * a.H2, a.aligned);
    switch (form.kernel) {
        case CELL_ONE_STEP: return launch_cell_step<TAB>(a, pack, stream);
        case CELL_CHUNKS: return launch_cell_chunks<TAB>(a, form.n, pack, stream);
        case CELL_RING_TOGETHER:
        case CELL_RING: return launch_cell_ring<TAB>(a, form, within_unit, pack, stream);
        case CELL_WRITTEN_OUT:
            return form.n == kDeepStages ? launch_cell_written_out<TAB, kDeepStages>(a, within_unit, pack, stream)
                                         : launch_cell_written_out<TAB, kShallowStages>(a, within_unit, pack, stream);
        case CELL_MULTI_STEP:
            if constexpr (TAB != CELL64_FOLDED)
                return launch_cell_multi_step<TAB == CELL64, true>(a, form.n, within_unit, pack, stream);
    }
    return KT_ERR_SHAPE;  // cell_form gives no such kernel to this table
}

template <bool WIDE, bool ARITH = true, class Lut>
ktanh_status_t launch_cell(const uint16_t *gates, const float *c_in, float *c_out, uint16_t *h_out,
                           size_t T, size_t B, size_t H, const Lut *lut, ktanh_stream_t stream)
{
    if (T == 0 || B == 0 || H == 0) return KT_OK;
    if (gates == nullptr || c_in == nullptr || c_out == nullptr || h_out == nullptr)
        return KT_ERR_NULL;
    if (H % 8 != 0) return KT_ERR_SHAPE;
    // one time step holds fewer than 2^28 lane pairs (byte offsets inside a step fit 32 bits), and
    // T*B*4H elements stay far below 2^63; every bound is tested by division, so nothing wraps
    if (T > 0x7FFFFFFFull || B >= ((size_t)1 << 28) || H >= ((size_t)1 << 29) ||
        B > (((size_t)1 << 28) - 1) / (H / 2))
        return KT_ERR_SHAPE;
    // the kernel moves BFloat16 pairs (4 bytes) and Float32 pairs (8 bytes)
    const uintptr_t words = reinterpret_cast<uintptr_t>(gates) | reinterpret_cast<uintptr_t>(h_out);
    const uintptr_t states = reinterpret_cast<uintptr_t>(c_in) | reinterpret_cast<uintptr_t>(c_out);
    if ((words & 3) || (states & 7)) return KT_ERR_ALIGN;
    KtLutPack pack;
    bool within_unit = true, folds = false;
    const ktanh_status_t st = pack_cell(lut, &pack, &within_unit, &folds);
    if (st != KT_OK) return st;

    const unsigned n_pairs = (unsigned)(B * (H / 2));  // < 2^28, checked above
    const CellCall a = {reinterpret_cast<const uint32_t *>(gates), reinterpret_cast<const float2 *>(c_in),
                        reinterpret_cast<float2 *>(c_out), reinterpret_cast<uint32_t *>(h_out),
                        (unsigned)T, n_pairs, (unsigned)(H / 2), row_division((unsigned)(H / 2)), (words | states) % 128 == 0};
    if constexpr (!ARITH) {
        const unsigned stages = shallow_ring(WIDE, a.T, a.n_pairs, H) ? kShallowStages : kDeepStages;
        return launch_cell_multi_step<WIDE, false>(a, stages, within_unit, pack, stream);
    } else if constexpr (WIDE) {
        return folds ? launch_cell_with<CELL64_FOLDED>(a, within_unit, pack, stream)
                     : launch_cell_with<CELL64>(a, within_unit, pack, stream);
    } else {
        return launch_cell_with<CELL32>(a, within_unit, pack, stream);
    }
}

}  // namespace ktanh_device

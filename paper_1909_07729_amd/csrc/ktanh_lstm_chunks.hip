// libktanh: the fused LSTM cell over many time steps of few cells, chunk by chunk of time.
#include "ktanh_lstm_impl.h"

namespace ktanh_device {

// With all gate pre-activations given, only  c' = f * c + i * g  ties one time step to the next; the four
// gate activations and the output of a step (about 130 of its 135 vector instructions) do not.  The
// multi-step kernel gives every pair of cells one lane for all T steps, which is the right thing when the
// pairs fill the chip; with few pairs its time is T times the 0.4 us that a lone wavefront needs for a step,
// whatever the size.  Here a block of 64 * WAVES lanes takes GROUP pairs and a chunk of STEPS time steps at
// once, one lane per pair and step: all lanes form their step's activations and leave f and i * g in LDS;
// GROUP lanes walk through the chunk with the two products and sums that each step still needs and leave
// the states in LDS; all lanes form their step's output from the state.  The gate words of the next chunk are
// loaded before the walk.  Operations and their order are those of the multi-step kernel, so the results are
// the same bits.
template <CellTable TAB, int GROUP, int WAVES>
__global__ __launch_bounds__(64 * WAVES) void lstm_chunk_kernel(const uint32_t *__restrict__ gates,
                                                               const float2 *c_in, float2 *c_out,  // may be equal
                                                               uint32_t *__restrict__ h_out, unsigned T,
                                                               unsigned n_pairs, unsigned H2, unsigned row_mul,
                                                               unsigned row_shift,  // row_of_pair
                                                               KtLutPack pack)
{
    constexpr unsigned STEPS = 64 * WAVES / GROUP;
    constexpr unsigned BATCH = STEPS < 8 ? STEPS : 8;
    __shared__ float4 held[STEPS][GROUP];  // f and i * g of both cells; then the new state in x and y

    const LaneTable tab(pack);
    const unsigned j = threadIdx.x % GROUP, s = threadIdx.x / GROUP;
    const unsigned p = blockIdx.x * GROUP + j;
    const bool live = p < n_pairs;
    const unsigned p_read = live ? p : 0;  // lanes past the end work on pair 0 and store nothing
    const unsigned long long row_step = 4ull * n_pairs;  // gate words per time step
    GateOffsets at = gate_offsets(p_read, H2, row_mul, row_shift);
    const bool walks = threadIdx.x < GROUP;  // these lanes have s = 0 and their own pair

    // lanes past the last step work on the last one and store nothing
    auto fetch = [&](unsigned t) { return load_gates(gates + row_step * (t < T ? t : T - 1), at); };
    GateWords q = fetch(s);
    float2 c = float2{0.f, 0.f};
    if (walks) c = c_in[p_read];
    for (unsigned t0 = 0; t0 < T; t0 += STEPS) {
        const Acts a = gate_activations<TAB>(q, tab);
        held[s][j] = float4{a.f_lo, a.f_hi, a.i_lo * widen_lo(a.g2), a.i_hi * widen_hi(a.g2)};
        if (t0 + STEPS < T) q = fetch(t0 + STEPS + s);  // uniform over the grid
        __syncthreads();
        if (walks) {
            const unsigned last = T - t0 < STEPS ? T - t0 : STEPS;  // steps past it are walked on c1 and dropped
            float2 c1 = c;
#pragma unroll 1
            for (unsigned k0 = 0; k0 < last; k0 += BATCH) {
                float4 v[BATCH];
#pragma unroll
                for (unsigned k = 0; k < BATCH; ++k) v[k] = held[k0 + k][j];
#pragma unroll
                for (unsigned k = 0; k < BATCH; ++k) {
                    const float keep_lo = v[k].x * c1.x, keep_hi = v[k].y * c1.y;
                    c1.x = keep_lo + v[k].z;
                    c1.y = keep_hi + v[k].w;
                    *reinterpret_cast<float2 *>(&held[k0 + k][j]) = c1;
                    if (k0 + k + 1 == last) c = c1;
                }
            }
        }
        __syncthreads();
        // only this lane reads this slot until the next barrier, so the next chunk may overwrite it
        const float4 now = held[s][j];
        const uint32_t h = hidden_of<TAB>(a, now.x, now.y, tab);
        if (live && t0 + s < T) store_stream(h_out + ((unsigned long long)n_pairs * (t0 + s) + p), h);
    }
    if (walks && live) c_out[p] = c;
}

// The chunk is as long as the call's steps or as the lanes that the chip holds at once allow (2^19 at the
// eight wavefronts per SIMD that these kernels' registers leave): shorter chunks walk less of their time with
// most lanes waiting but load and start more often, longer ones queue for the chip.  A group of 16 pairs puts
// few pairs on four times as many compute units as one of 64.  us per launch at 512 / 8192 / 16384 / 32768 /
// 65536 / 98304 pairs:
//   T = 64   multi-step kernel 25.1 / 25.6 / 27.1 / 27.8 / 29.1 / 33.9
//            64 steps, group 16, 4.7 / 6.5 / 12.7 / 22.3 / 40.0 / 59.1    32 steps, group 32, 5.8 / 5.9 / 7.5 / 15.4 / 25.7 / 37.6
//            16 steps, group 32, 6.9 / 6.9 / 8.8 / 11.6 / 22.2 / 32.4     8 steps, group 64, 10.5 / 10.4 / 10.6 / 13.7 / 19.4 / 29.1
//   T = 20   multi-step kernel 9.3 / 9.5 / 9.5 / 10.1 / 10.9 / 12.4; chosen 3.0 / 3.5 / 4.2 / 6.0 / 8.2 / 10.7
//   T = 8    5.5 / 5.6 / 5.6 / 5.7 / 5.6 / 6.5; chosen 2.4 / 2.5 / 2.6 / 3.2 / 4.0 / 5.2
template <CellTable TAB>
ktanh_status_t launch_cell_chunks(const CellCall &a, const KtLutPack &pack, ktanh_stream_t stream)
{
    auto launch = [&](auto kernel, unsigned group, unsigned waves) {
        return launch_checked(kernel, (a.n_pairs + group - 1) / group, 64 * waves, stream, a.gates, a.c_in, a.c_out,
                              a.h_out, a.T, a.n_pairs, a.H2, a.row.mul, a.row.shift, pack);
    };
    switch (chunk_steps(TAB != CELL32, a.T, a.n_pairs)) {
        case 64: return launch(lstm_chunk_kernel<TAB, 16, 16>, 16, 16);
        case 32:
            // one chunk of up to 32 steps, 512 pairs 3.0 against 3.2, 12288 pairs 3.8 against 4.3; from 16384 on slower
            if (a.T <= 32 && a.n_pairs <= 12288) return launch(lstm_chunk_kernel<TAB, 16, 8>, 16, 8);
            return launch(lstm_chunk_kernel<TAB, 32, 16>, 32, 16);
        case 16: return launch(lstm_chunk_kernel<TAB, 32, 8>, 32, 8);
        case 8: return launch(lstm_chunk_kernel<TAB, 64, 8>, 64, 8);
        default: return launch(lstm_chunk_kernel<TAB, 64, 4>, 64, 4);
    }
}

template ktanh_status_t launch_cell_chunks<CELL32>(const CellCall &, const KtLutPack &, ktanh_stream_t);
template ktanh_status_t launch_cell_chunks<CELL64>(const CellCall &, const KtLutPack &, ktanh_stream_t);
template ktanh_status_t launch_cell_chunks<CELL64_FOLDED>(const CellCall &, const KtLutPack &, ktanh_stream_t);

}  // namespace ktanh_device

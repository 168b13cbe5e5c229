// libktanh: the fused LSTM cell over many time steps of few cells, chunk by chunk of time.
#include "ktanh_lstm_impl.h"

namespace ktanh_device {

// With all gate pre-activations given, only  c' = f * c + i * g  ties one time step to the next; the four
// gate activations and the output of a step (all but four of the about ninety vector instructions for two cells) do not.  The
// multi-step kernel gives every pair of cells one lane for all T steps, which is the right thing when the
// pairs fill the chip; with few pairs its time is T times the 0.4 us that a lone wavefront needs for a step,
// whatever the size.  Here a block of 64 * WAVES lanes takes GROUP pairs and a chunk of STEPS time steps at
// once, one lane per pair and step: all lanes form their step's activations and leave f and i * g in LDS;
// GROUP lanes walk through the chunk with the two products and sums that each step still needs and leave
// the states in LDS; all lanes form their step's output from the state.  Operations and their order are those of the multi-step kernel, so the results are
// the same bits.
//
// The gate words of the next chunk are asked for before the walk, when this chunk's have been used.  AT_ONCE: together with this chunk's, which gains
// where chunks are short and many (chunk_words_at_once); there the outputs are stored where the compiler counts them, without a branch, so that the wait for the words
// is not one for the stores of the chunk before (T = 64 98304 pairs 28.4 -> 26.1; the other form is level).  In between, as soon as this chunk's are here, is
// worse than either (more words on their way when a chunk's are asked for; rows that share cache lines lose up to 8 %).  us per launch, inputs partly / all out of the
// cache, in between | before the walk: T = 20 65536 pairs 7.94 / 8.12 | 7.68 / 7.86, rows of 2000 cells 9.01 / 9.29 | 8.56 / 8.85; T = 64 32768 11.7 / 11.9 | 10.8 / 11.0, 49152
// 15.4 / 15.4 | 14.7 / 14.8; T = 90 65536 25.6 / 25.6 | 24.6 / 24.8; T = 15 131072 10.1 / 10.2 | 9.41 / 9.69, rows of 2000 122880 10.9 / 11.3 | 10.5 / 11.1.
template <CellTable TAB, int GROUP, int WAVES, bool AT_ONCE>
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
    const unsigned mine = blockIdx.x * GROUP + j;
    // Lanes past the end repeat the last pair, which is in their own block, and store the same words to the same
    // place, so that no access has a branch around it.
    const unsigned p = mine < n_pairs ? mine : n_pairs - 1;
    const GateOffsets at = gate_offsets(p, H2, row_mul, row_shift);
    const bool walks = threadIdx.x < GROUP;  // these lanes have s = 0 and their own pair

    // The gate words of this lane's step in the chunk that starts at t0, of the last step where that is past it.  Byte offsets
    // inside a chunk stay below 16 * n_pairs * STEPS <= 2^23 (chunk_steps).
    auto fetch = [&](unsigned t0) {
        const unsigned k = T - t0 - 1 < s ? T - t0 - 1 : s;
        const unsigned from = 16u * n_pairs * k;
        GateOffsets here = {at.i + from, at.f + from, at.g + from, at.o + from};
        return load_gates(gates + 4ull * n_pairs * t0, here);
    };
    GateWords q = fetch(0);
    float2 c = float2{0.f, 0.f};
    if (walks) c = c_in[p];
    unsigned t0 = 0;
    unsigned h_at = 4u * (n_pairs * s + p);  // byte offset of this lane's output word inside a chunk
    // chunks with another one behind them
    for (; T - t0 > STEPS; t0 += STEPS) {
        GateWords next;
        if constexpr (AT_ONCE) next = fetch(t0 + STEPS);
        const Acts a = gate_activations<TAB>(q, tab);
        held[s][j] = float4{a.f_lo, a.f_hi, a.i_lo * widen_lo(a.g2), a.i_hi * widen_hi(a.g2)};
        if constexpr (!AT_ONCE) next = fetch(t0 + STEPS);
        __syncthreads();
        if (walks) {
#pragma unroll 1
            for (unsigned k0 = 0; k0 < STEPS; k0 += BATCH) {
                float4 v[BATCH];
#pragma unroll
                for (unsigned k = 0; k < BATCH; ++k) v[k] = held[k0 + k][j];
#pragma unroll
                for (unsigned k = 0; k < BATCH; ++k) {
                    const float keep_lo = v[k].x * c.x, keep_hi = v[k].y * c.y;
                    c.x = keep_lo + v[k].z;
                    c.y = keep_hi + v[k].w;
                    *reinterpret_cast<float2 *>(&held[k0 + k][j]) = c;
                }
            }
        }
        __syncthreads();
        // only this lane reads this slot until the next barrier, so the next chunk may overwrite it
        const float4 now = held[s][j];
        store_counted(h_out + (unsigned long long)n_pairs * t0, h_at, hidden_of<TAB>(a, now.x, now.y, tab));
        q = next;
    }
    // the last chunk, whole or not
    const Acts a = gate_activations<TAB>(q, tab);
    held[s][j] = float4{a.f_lo, a.f_hi, a.i_lo * widen_lo(a.g2), a.i_hi * widen_hi(a.g2)};
    __syncthreads();
    if (walks) {
        const unsigned last = T - t0;  // steps past it are walked on c1 and dropped
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
        c_out[p] = c;
    }
    __syncthreads();
    const float4 now = held[s][j];
    const uint32_t h = hidden_of<TAB>(a, now.x, now.y, tab);
    if (t0 + s < T) store_stream(h_out + (unsigned long long)n_pairs * t0, h_at, h);
}

// The chunk is as long as the call's steps or as the lanes that the chip holds at once allow (2^19 at the
// eight wavefronts per SIMD that these kernels' registers leave): shorter chunks walk less of their time with
// most lanes waiting but load and start more often, longer ones queue for the chip.  A group of 16 pairs puts
// few pairs on four times as many compute units as one of 64.  us per launch, inputs out of the cache, chunks of half the steps | as chosen | of twice the steps:
//   T = 64   8192 pairs  6.38 | 5.67 | 7.44     24576 11.7 | 9.38 | 11.1     32768 12.1 | 11.0 | 15.3     57344 20.2 | 17.1 | 18.6     81920 - | 23.1 | 24.4
//            512 pairs 5.03, 4096 5.66; the multi-step kernel took 25.1 for 512 pairs, 27.1 for 16384, 29.1 for 65536
//   T = 20   32768 5.85 | 6.16 | 7.95     40960 7.06 | 6.49 | 7.84     65536 8.05 | 7.86 | 10.9
//   T = 16   40960 6.10 | 5.10 | 5.99     65536 6.88 | 6.18 | 7.71     81920 - | 7.58 | 7.99
template <CellTable TAB>
ktanh_status_t launch_cell_chunks(const CellCall &a, unsigned steps, const KtLutPack &pack, ktanh_stream_t stream)
{
    auto launch = [&](auto kernel, unsigned group, unsigned waves) {
        return launch_checked(kernel, (a.n_pairs + group - 1) / group, 64 * waves, stream, a.gates, a.c_in, a.c_out,
                              a.h_out, a.T, a.n_pairs, a.H2, a.row.mul, a.row.shift, pack);
    };
    switch (steps) {
        case 64: return launch(lstm_chunk_kernel<TAB, 16, 16, false>, 16, 16);
        case 32:
            // one chunk of up to 32 steps, 512 pairs 3.0 against 3.2, 12288 pairs 3.8 against 4.3; from 16384 on slower
            if (a.T <= 32 && a.n_pairs <= 12288) return launch(lstm_chunk_kernel<TAB, 16, 8, false>, 16, 8);
            return launch(lstm_chunk_kernel<TAB, 32, 16, false>, 32, 16);
        case 16: return launch(lstm_chunk_kernel<TAB, 32, 8, false>, 32, 8);
        case 8: return launch(lstm_chunk_kernel<TAB, 64, 8, false>, 64, 8);
        default:
            return chunk_words_at_once(a.T) ? launch(lstm_chunk_kernel<TAB, 64, 4, true>, 64, 4)
                                            : launch(lstm_chunk_kernel<TAB, 64, 4, false>, 64, 4);
    }
}

template ktanh_status_t launch_cell_chunks<CELL32>(const CellCall &, unsigned, const KtLutPack &, ktanh_stream_t);
template ktanh_status_t launch_cell_chunks<CELL64>(const CellCall &, unsigned, const KtLutPack &, ktanh_stream_t);
template ktanh_status_t launch_cell_chunks<CELL64_FOLDED>(const CellCall &, unsigned, const KtLutPack &, ktanh_stream_t);

}  // namespace ktanh_device

// Internal to libktanh: the arithmetic of one LSTM-cell step for the two cells of a lane, as the kernels for a
// single step, for a few steps, for chunks of time and for many steps of few cells (or of a table that folds) use it.
//
// A step is five evaluations of K for two cells.  Each costs two cross-lane table reads, about a hundred cycles away,
// and about a dozen vector instructions, and few wavefronts per SIMD leave little else to fill the wait.  So the reads of
// all gates go out together (look_up_gates) before the first is needed, and the NaN rules of K-TanH, a quarter of the instructions,
// are no part of every K and no second copy of the step, but a repair of its results on a wavefront-uniform path that only a NaN
// takes.  us per launch before -> with it: chunks of time, 64 steps of [64, 1024] cells 11.5 -> 11.1, of [64, 2048] 19.8 -> 18.5, of
// [96, 2048] 28.8 -> 27.1, 8 of [128, 2048] 5.95 -> 5.68, 64 intervals 64 steps of [64, 2048] 22.6 -> 21.1; steps written out, 4 of [256, 2048]
// 6.06 -> 5.77; a single step of [256, 2048] 2.46 -> 2.38.
#pragma once
#include "ktanh_device.h"

namespace ktanh_device {

// Gate words of a lane: one packed pair of cells per gate.
struct GateWords {
    uint32_t i, f, g, o;
};

// CellTable (ktanh_order.h): 32 intervals, 64, or 64 of a table that folds (kt_pack_lut64_bf16).
// In a table that folds the two regions around it need no selects of their own.  Its first entry takes 4.0, whose index is that
// of 0.25, to 1.0, so that magnitudes clamped to 4.0 come out saturated; and no output exceeds its input, so that the smaller of the
// input and the output for max(|x|, 0.25) is the pass-through region.  89 instead of 114 vector instructions per step of the ring; us per
// launch, selects -> folded, both otherwise as here: chunks of time, 64 steps of [64, 1024] cells 12.3 -> 11.4, of [64, 2048] 21.3 -> 19.6, many steps, 64 of
// [128, 2048] 35.6 -> 30.9, of [192, 2048] 50.3 -> 44.8, of [256, 2048] 65.5 -> 57.2; steps written out, 5 of [512, 2048] 12.9 -> 11.6; a single
// step of [256, 2048] 2.50 -> 2.45.  The fitted table folds; a caller's table that does not keeps CELL64.

// One K of a pair with its table reads in flight.
struct Look {
    uint32_t mag2;
    SlotPair sp;
};

template <CellTable TAB>
__device__ __forceinline__ Look look_up(uint32_t mag2, const LaneTable &tab)
{
    if constexpr (TAB == CELL64_FOLDED) {
        const u16x2 capped = __builtin_elementwise_min(as_u16x2(mag2), splat(0x4080));
        const uint32_t key2 = as_u32(__builtin_elementwise_max(capped, splat(0x3E80)));
        return Look{mag2, SlotPair{key2, tab.get(key2 >> 1), tab.get(key2 >> 17)}};  // index bits as for 64 intervals
    } else {
        return Look{mag2, fetch_slots<TAB == CELL64>(mag2, tab)};
    }
}

// K without the NaN rule (a NaN comes out as +-1), signs from w.
template <CellTable TAB>
__device__ __forceinline__ uint32_t finish_look(const Look &k, uint32_t w)
{
    if constexpr (TAB == CELL64_FOLDED) {
        const u16x2 base2 = as_u16x2(__builtin_amdgcn_perm(k.sp.e_hi, k.sp.e_lo, 0x07060302u));
        const u16x2 r2 = as_u16x2(__builtin_amdgcn_perm(k.sp.e_hi, k.sp.e_lo, 0x05040100u));
        const u16x2 lut2 = base2 + (as_u16x2(k.sp.key2) >> r2);
        return bitsel(kMag2, as_u32(__builtin_elementwise_min(lut2, as_u16x2(k.mag2))), w);
    } else {
        return bitsel(kMag2, finish_mag_pair<TAB == CELL64>(k.mag2, k.sp), w);
    }
}

// The NaN rule on a result of finish_look.
__device__ __forceinline__ uint32_t with_nans(uint32_t t2, uint32_t w)
{
    return bitsel(nan_mask_pair(w & kMag2), w | 0x00400040u, t2);
}

struct GateLooks {
    Look i, f, g, o;
};

template <CellTable TAB>
__device__ __forceinline__ GateLooks look_up_gates(const GateWords &q, const LaneTable &tab)
{
    return GateLooks{look_up<TAB>(sigmoid_half_mag_pair(q.i), tab), look_up<TAB>(sigmoid_half_mag_pair(q.f), tab),
                     look_up<TAB>(q.g & kMag2, tab), look_up<TAB>(sigmoid_half_mag_pair(q.o), tab)};
}

// The K values of the gates: K(x / 2) for i, f, o and K(x) for g.
template <CellTable TAB>
__device__ __forceinline__ GateWords finish_gates(const GateLooks &k, const GateWords &q)
{
    return GateWords{finish_look<TAB>(k.i, q.i), finish_look<TAB>(k.f, q.f), finish_look<TAB>(k.g, q.g),
                     finish_look<TAB>(k.o, q.o)};
}
__device__ __forceinline__ GateWords with_nans(const GateWords &t, const GateWords &q)
{
    return GateWords{with_nans(t.i, q.i), with_nans(t.f, q.f), with_nans(t.g, q.g), with_nans(t.o, q.o)};
}

// True for the whole wavefront when `flag` is non-zero in some lane.
__device__ __forceinline__ bool any_lane(uint32_t flag) { return __builtin_amdgcn_ballot_w64(flag != 0u) != 0; }

// Non-zero where one of the lane's gate words holds a NaN.
__device__ __forceinline__ uint32_t gate_nans(const GateWords &q)
{
    return nan_bits_pair(max_pair(max_pair(q.i & kMag2, q.f & kMag2), max_pair(q.g & kMag2, q.o & kMag2)));
}

// Non-zero where x is an infinity or a NaN.
__device__ __forceinline__ uint32_t not_finite(float x)
{
    return (__float_as_uint(x) & 0x7F800000u) == 0x7F800000u ? 1u : 0u;
}

// The gate non-linearities of one time step for the two cells of a lane.  They depend on the gate
// words alone, not on the state, so they can be formed one step ahead.
struct Acts {
    float i_lo, i_hi, f_lo, f_hi, o_lo, o_hi;
    uint32_t g2;  // K(g) as a BFloat16 pair
};

// Sigmoids from their K values: 0.5 * t is exact for every K output t that can change the sum, so the multiply-add may fuse.
template <CellTable TAB>
__device__ __forceinline__ Acts acts_from(const GateWords &t)
{
    const uint32_t i2 = whole_pair<TAB == CELL64>(t.i), f2 = whole_pair<TAB == CELL64>(t.f),
                   o2 = whole_pair<TAB == CELL64>(t.o);
    Acts a;
    a.i_lo = __builtin_fmaf(0.5f, widen_lo(i2), 0.5f);
    a.i_hi = __builtin_fmaf(0.5f, widen_hi(i2), 0.5f);
    a.f_lo = __builtin_fmaf(0.5f, widen_lo(f2), 0.5f);
    a.f_hi = __builtin_fmaf(0.5f, widen_hi(f2), 0.5f);
    a.o_lo = __builtin_fmaf(0.5f, widen_lo(o2), 0.5f);
    a.o_hi = __builtin_fmaf(0.5f, widen_hi(o2), 0.5f);
    a.g2 = whole_pair<TAB == CELL64>(t.g);
    return a;
}

template <CellTable TAB>
__device__ __forceinline__ Acts gate_activations(const GateWords &q, const LaneTable &tab)
{
    const GateLooks k = look_up_gates<TAB>(q, tab);
    const bool rare = any_lane(gate_nans(q));
    GateWords t = finish_gates<TAB>(k, q);
    if (rare) t = with_nans(t, q);
    return acts_from<TAB>(t);
}

// c' = (f * c) + (i * g): two products and one sum, each rounded on its own.
__device__ __forceinline__ void advance_state(const Acts &a, float2 &c)
{
    const float keep_lo = a.f_lo * c.x, keep_hi = a.f_hi * c.y;
    const float add_lo = a.i_lo * widen_lo(a.g2), add_hi = a.i_hi * widen_hi(a.g2);
    c.x = keep_lo + add_lo;
    c.y = keep_hi + add_hi;
}

// K of a state as a BFloat16 pair, exact for any input.
template <CellTable TAB>
__device__ __forceinline__ uint32_t state_tanh(float c_lo, float c_hi, const LaneTable &tab)
{
    const uint32_t cb = narrow_pair(c_lo, c_hi);
    const Look k = look_up<TAB>(cb & kMag2, tab);
    return whole_pair<TAB == CELL64>(with_nans(finish_look<TAB>(k, cb), cb));
}

// The hidden outputs of a step from K of its new state, a whole_pair.
__device__ __forceinline__ uint32_t hidden_from(const Acts &a, uint32_t tc2)
{
    return narrow_pair(a.o_lo * widen_lo(tc2), a.o_hi * widen_hi(tc2));
}

// The hidden outputs of a step whose new state is given.
template <CellTable TAB>
__device__ __forceinline__ uint32_t hidden_of(const Acts &a, float c_lo, float c_hi, const LaneTable &tab)
{
    return hidden_from(a, state_tanh<TAB>(c_lo, c_hi, tab));
}

// State update and hidden outputs of a step with no step after it.
template <CellTable TAB>
__device__ __forceinline__ uint32_t closing_step(const Acts &a, float2 &c, const LaneTable &tab)
{
    advance_state(a, c);
    return hidden_of<TAB>(a, c.x, c.y, tab);
}

// One time step, and the activations of the next one: `a` holds this step's and is replaced by those of the step whose gate
// words are `next`.  The ten table reads are in flight together.  `watch`, the same in the whole wavefront, says that this step's
// activations or its incoming state may not be finite: without it, and with no NaN in `next`, no K here can meet a NaN (no gate is one,
// the incoming state is finite and |K| <= 1, so |c'| <= |c| + 1).  always: the caller's table lets |K| exceed 1, so the
// state may overflow on the way.
template <CellTable TAB>
__device__ __forceinline__ uint32_t step_and_look_up(Acts &a, bool &watch, const GateWords &next, float2 &c, bool always,
                                                     const LaneTable &tab)
{
    const GateLooks k = look_up_gates<TAB>(next, tab);
    advance_state(a, c);
    const uint32_t cb = narrow_pair(c.x, c.y);
    const Look kc = look_up<TAB>(cb & kMag2, tab);
    const uint32_t nans = gate_nans(next);
    const bool rare = watch || any_lane(nans);
    GateWords t = finish_gates<TAB>(k, next);
    uint32_t tc2 = finish_look<TAB>(kc, cb);
    watch = false;
    if (rare) {
        t = with_nans(t, next);
        tc2 = with_nans(tc2, cb);
        watch = always || any_lane(nans | not_finite(c.x) | not_finite(c.y));
    }
    const uint32_t h = hidden_from(a, whole_pair<TAB == CELL64>(tc2));
    a = acts_from<TAB>(t);
    return h;
}

}  // namespace ktanh_device

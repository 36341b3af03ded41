// Atomic row-adds of the backward kernels: a wave adds one gradient row, scaled, to a list of
// destination rows.
#pragma once

#include "fsa_device.hip.h"

#include <type_traits>

namespace fsa {

struct g_f32 { using T = float; };
struct g_bf16 { using T = uint16_t; };
struct g_f16 { using T = uint16_t; };

template <typename GT, typename XG> struct Epl { static constexpr int value = 2; };
template <typename GT> struct Epl<GT, g_f32> { static constexpr int value = 1; };

typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));

// The EPL elements at `at` += v, by hardware atomics without a return value.
template <typename XG, int EPL>
__device__ __forceinline__ void atomic_add_row(void* at, const float (&v)[EPL]) {
    if constexpr (std::is_same<XG, g_f32>::value) {
        float* p = static_cast<float*>(at);
#pragma unroll
        for (int e = 0; e < EPL; ++e) unsafeAtomicAdd(p + e, v[e]);          // global_atomic_add_f32
    } else {
        static_assert(EPL == 2, "16-bit grad_x takes packed pairs");
        const f32x2_t f = {v[0], v[1]};
        if constexpr (std::is_same<XG, g_bf16>::value) {
            const bf16x2_t b = __builtin_convertvector(f, bf16x2_t);
            __builtin_amdgcn_global_atomic_fadd_v2bf16(static_cast<bf16x2_t*>(at), b);
        } else {
            const f16x2_t h = __builtin_convertvector(f, f16x2_t);
            __builtin_amdgcn_global_atomic_fadd_v2f16(static_cast<f16x2_t*>(at), h);
        }
    }
}

// How the lanes of a wave lie over the rows of grad_x, in units of 4 bytes (an fp32 element or a pair
// of 16-bit ones).
struct RowLanes {
    int units;                 // units per row
    int width_shift;           // log2 of the lanes that take a row together: 6, or less for narrow rows
    int base;                  // unit of its 64-byte segment at which grad_x starts, or -1: lanes start where rows start
};
constexpr int kSegment = 16;   // units of a 64-byte segment
inline int rows_an_instruction(const RowLanes& l) { return kWave >> l.width_shift; }

inline RowLanes row_lanes(const void* grad_x, int64_t units) {
    const int at = (int)((reinterpret_cast<uintptr_t>(grad_x) >> 2) & (kSegment - 1));
    RowLanes l;
    l.units = (int)units;
    // a row within one instruction touches no segment twice
    l.base = units <= kWave || (units % kSegment == 0 && at == 0) ? -1 : at;
    l.width_shift = units <= 16 ? 4 : units <= 32 ? 5 : 6;
    return l;
}

// The values are here when this returns.  Without it the compiler puts the wait for a load that is first used
// in a loop into the loop, where it waits for every atomic of the loop as well.
template <int EPL> __device__ __forceinline__ void arrived(float (&g)[EPL]) {
#pragma unroll
    for (int c = 0; c < EPL; ++c) asm volatile("" : "+v"(g[c]));
}

// grad_x[rows[e], :] += factor[e] * g for e < n, where load(d, v) reads the EPL elements of g from element d
// on; of `parts` callers with the same list each takes its share of it.  `rows` and `factor` lie in LDS.
// Called by a whole wave.
//
// What bounds it: the memory side takes an atomic instruction apart into 64-byte segments and serves
// 20.8 G of them a second, 19 to 20 G in tables of a gigabyte and more, whether 1 or 16 lanes fall into one and in
// whatever order (150,000 rows of 128 floats: 61 us with all lanes, with every second and with every fourth; the same
// from 128 CUs on as on 256).  A launch and its IDs add 6 us: 150,000 / 1,200,000 distinct rows of 64 floats 34 / 235 us, of
// 100 57 / 411, of 128 64 / 468, of 256 123 / 934, of 128 bf16 elements 34 / 236.  So a row that starts inside a segment is
// not cut every 64 elements, where
// both pieces touch the segment of the cut, but at the last segment's start before that: the lanes behind
// the cut go along with the next instruction (150,000 rows of 100 floats 59.5 -> 53.8 us, of 150 91 -> 78;
// 37,500 of 602 87 -> 75).  Rows of two segments or one share an instruction, because an instruction costs
// at least as much as two segments (150,000 rows of 16 floats 19.2 -> 10.1 us, of 32 20.4 -> 16.7).
template <typename XG, int EPL, typename Load>
__device__ __forceinline__ void add_scaled_rows(void* grad_x, const RowLanes& l, const int* rows, const float* factor,
                                                int n, int part, int parts, int lane, Load load) {
    char* const base = static_cast<char*>(grad_x);
    if (l.width_shift < 6) {                                         // kernel-uniform
        const int u = lane & ((1 << l.width_shift) - 1);
        if (u >= l.units) return;
        float g[EPL];
        load((int64_t)u * EPL, g);
        arrived(g);
        const int each = kWave >> l.width_shift;
        for (int e = part * each + (lane >> l.width_shift); e < n; e += parts * each) {
            float v[EPL];
#pragma unroll
            for (int c = 0; c < EPL; ++c) v[c] = g[c] * factor[e];
            atomic_add_row<XG, EPL>(base + ((int64_t)rows[e] * l.units + u) * 4, v);
        }
        return;
    }
    if (l.base < 0) {                                                // kernel-uniform
        for (int u = lane; u < l.units; u += kWave) {
            float g[EPL];
            load((int64_t)u * EPL, g);
            arrived(g);
            for (int e = part; e < n; e += parts) {
                float v[EPL];
#pragma unroll
                for (int c = 0; c < EPL; ++c) v[c] = g[c] * factor[e];
                atomic_add_row<XG, EPL>(base + ((int64_t)rows[e] * l.units + u) * 4, v);
            }
        }
        return;
    }
    float prev[EPL];
#pragma unroll
    for (int c = 0; c < EPL; ++c) prev[c] = 0.0f;
    for (int t0 = 0; t0 < l.units + kSegment - 1; t0 += kWave) {
        const int u = t0 + lane;
        float cur[EPL];
#pragma unroll
        for (int c = 0; c < EPL; ++c) cur[c] = 0.0f;
        if (u < l.units) load((int64_t)u * EPL, cur);
        arrived(cur);
        for (int e = part; e < n; e += parts) {
            const int row = rows[e];
            // lanes from the cut on: the elements that the instruction before left
            const int cut = kWave - (int)(((uint32_t)l.base + (uint32_t)row * (uint32_t)l.units) & (kSegment - 1));
            const int d = lane < cut ? u : u - kWave;
            float v[EPL];
#pragma unroll
            for (int c = 0; c < EPL; ++c) v[c] = (lane < cut ? cur[c] : prev[c]) * factor[e];
            if ((unsigned)d < (unsigned)l.units) atomic_add_row<XG, EPL>(base + ((int64_t)row * l.units + d) * 4, v);
        }
#pragma unroll
        for (int c = 0; c < EPL; ++c) prev[c] = cur[c];
    }
}

}  // namespace fsa

// Backward into a gradient of its own (fsa_mean_bwd_dense): every row of grad_x is written once, rows that
// no leaf names as zeros, so a caller that wants the whole gradient of the table -- torch.autograd does --
// neither clears it first nor adds to it with atomics.  The paper describes no backward kernel (Sec. 3.3
// "Reproducibility" only asks that the saved IDs are replayed).
//
// What bounds it: the rows written (N*D elements, once).  Clearing first and adding with atomics wrote them all, read
// the named ones back and paid a 64-byte segment's atomic (20.8 G/s) for every 64 bytes of every leaf.
//
// Three launches on the caller's stream, all state in the caller's workspace:
//   clear   zero the bins' counters (a fill kernel: a memset node must not end up in a captured graph);
//   bin     grad_x is cut into bins of consecutive rows; every live leaf slot appends an entry to its row's bin;
//           a full bin sends its entries to the overflow list;
//   write   a workgroup per bin sums the gradients of its rows' entries in registers, in fp32, and writes every row.
//           A bin that overflowed picks its entries out of the overflow list as well, so hub rows take no atomics in
//           memory either.
// The order of additions follows the places that the entries got, which varies from run to run, as with atomics.
#include "fsa_atomic_rows.hip.h"
#include "fsa_device.hip.h"
#include "fsa_internal.h"

#include <type_traits>

namespace fsa {

constexpr int kDenseThreads = 256;
// Elements of a bin, and its rows: enough entries per workgroup to pay for its steps (clear counter to last store, 75,000
// entries in 169,343 rows of 128 floats: 4096 elements 38.6 us, 8192 33.2, 16384 33.9; 590,000 entries 174 / 157 / 182),
// and several rows per group of lanes where rows are wide (49,000 in 30,000 rows of 301 floats: 8 / 16 / 32 rows
// 77 / 54 / 38).  Several bins per workgroup, the next one's entries requested ahead: 2 to 8 % slower on large tables.
constexpr int kDenseBinElements = 8192;
constexpr int kDenseRowsMin = 32;                                    // (bins start at multiples of 16 bytes of grad_x, whatever D)
constexpr int kDenseRowsMax = 256;
constexpr int64_t kDenseMinSegments = 768 * 1024;                   // see dense_pays
constexpr int64_t kDenseMaxRowsPerSlot = 16;
constexpr int64_t kDenseMaxD = 1024;                                 // 16 KB of LDS at four groups

struct DenseParams {
    const void* grad_out; const void* grad_h1;
    const int32_t* ids1;                  // two hops: [slots], a negative entry switches the slot off; one hop: NULL
    const int32_t* leaf;                  // [slots, k2]
    void* grad_x;
    int64_t slots, N;
    int D, k1, k2;                        // a root has k1 slots, a slot k2 leaves (one hop: k1 = 1, a seed is a slot)
    int slots_per_wg;                     // binning: whole roots
    int row_shift, bins, room, stride;    // rows of a bin (log2), bins, entries a bin holds, ints between two counters
    int* counter; int* overflow_count; unsigned long long* entries; unsigned long long* overflow; int* overflow_bin;
};

// A leaf slot in a bin: its row of the bin, its root and slot, and how many slots of the root and leaf slots of the slot
// take part -- all that its share of the gradient follows from.
struct Entry {
    unsigned long long v;
    __device__ static Entry of(int row, int64_t root, int slot, int c1, int c2) {
        return {(unsigned long long)row << 56 | (unsigned long long)(c1 - 1) << 50 | (unsigned long long)(c2 - 1) << 44 |
                (unsigned long long)slot << 38 | (unsigned long long)root};
    }
    __device__ int row() const { return (int)(v >> 56); }            // < kDenseRowsMax
    __device__ int c1() const { return (int)(v >> 50 & 63) + 1; }    // at most FSA_KMAX, as is c2
    __device__ int c2() const { return (int)(v >> 44 & 63) + 1; }
    __device__ int slot() const { return (int)(v >> 38 & 63); }
    __device__ int64_t root() const { return (int64_t)(v & 0x3fffffffffull); }
};

struct DensePlan { int row_shift, room, stride; int64_t bins; size_t off[5], total; };

static DensePlan dense_plan(int64_t slots, int k2, int64_t D, int64_t N) {
    DensePlan q{};
    while ((2ll << q.row_shift) <= kDenseRowsMax && (2ll << q.row_shift) * D <= kDenseBinElements) ++q.row_shift;
    while ((1 << q.row_shift) < kDenseRowsMin) ++q.row_shift;
    q.bins = (N + (1ll << q.row_shift) - 1) >> q.row_shift;
    // room for four times the mean with every slot full; a skewed batch's hubs go to the overflow list
    const int64_t mean = slots * k2 / q.bins;
    q.room = 32;
    while (q.room < 4096 && q.room < 4 * mean) q.room *= 2;
    q.stride = q.bins <= 16384 ? kSegment * 2 : 4;                   // few counters: a 128-byte line each, over all L2 channels
    auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
    size_t o = 0;
    q.off[0] = o; o += up((size_t)q.bins * q.stride * sizeof(int));
    q.off[1] = o; o += up(sizeof(int));
    q.off[2] = o; o += up((size_t)q.bins * q.room * sizeof(unsigned long long));
    q.off[3] = o; o += up((size_t)slots * k2 * sizeof(unsigned long long));
    q.off[4] = o; o += up((size_t)slots * k2 * sizeof(int));
    q.total = o;
    return q;
}

__global__ __launch_bounds__(256) void dense_clear_kernel(int* counter, int bins, int stride, int* overflow_count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < bins) counter[(size_t)i * stride] = 0;
    if (i == 0) *overflow_count = 0;
}

// A workgroup takes whole roots (one with two hops, as many seeds as have 256 leaf slots with one hop).  Bound by the
// chain IDs -> place (a returning atomic) -> entry; four leaf slots per thread go through it together, and the slots are
// counted while the places are on their way.
__global__ __launch_bounds__(kDenseThreads) void dense_bin_kernel(const DenseParams p) {
    __shared__ int on[kDenseThreads];                                // slots_per_wg <= kDenseThreads
    __shared__ int cnt[kDenseThreads];
    const int tid = threadIdx.x;
    const int64_t slot0 = (int64_t)blockIdx.x * p.slots_per_wg;
    const int n_slots = (int)(p.slots - slot0 < p.slots_per_wg ? p.slots - slot0 : p.slots_per_wg);
    const int32_t* leaf = p.leaf + slot0 * p.k2;
    const int n_ent = n_slots * p.k2;                                // at most 64 * 64
    if (tid < n_slots) on[tid] = p.ids1 ? p.ids1[slot0 + tid] : 0;
    cnt[tid] = 0;
    __syncthreads();
    constexpr int U = 4;
    int id[U], slot[U], at[U];
    auto look = [&](int e0) {
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int e = e0 + k * kDenseThreads;
            slot[k] = (e < n_ent ? e : 0) / p.k2;
            id[k] = leaf[e < n_ent ? e : 0];
            if (e >= n_ent || on[slot[k]] < 0) id[k] = -1;
        }
    };
    auto place = [&] {
#pragma unroll
        for (int k = 0; k < U; ++k) at[k] = id[k] >= 0 ? atomicAdd(&p.counter[(size_t)(id[k] >> p.row_shift) * p.stride], 1) : 0;
    };
    look(tid);
    place();
#pragma unroll
    for (int k = 0; k < U; ++k) { if (id[k] >= 0) atomicAdd(&cnt[slot[k]], 1); }
    for (int e = tid + U * kDenseThreads; e < n_ent; e += kDenseThreads) {
        const int j = e / p.k2;
        if (on[j] >= 0 && leaf[e] >= 0) atomicAdd(&cnt[j], 1);
    }
    __syncthreads();
    const int lane = tid & (kWave - 1);                              // two hops: the root's slots that take part (k1 <= 64)
    const int c1 = p.ids1 ? __popcll(__ballot(lane < n_slots && cnt[lane] > 0)) : 1;
    for (int e0 = tid;;) {
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (id[k] < 0) continue;
            const int bin = id[k] >> p.row_shift;
            const int64_t root = p.ids1 ? (int64_t)blockIdx.x : slot0 + slot[k];
            const Entry e = Entry::of(id[k] & ((1 << p.row_shift) - 1), root, p.ids1 ? slot[k] : 0, c1, cnt[slot[k]]);
            if (at[k] < p.room) {
                p.entries[(size_t)bin * p.room + at[k]] = e.v;
            } else {
                const int o = atomicAdd(p.overflow_count, 1);        // an entry lands once: below slots * k2
                p.overflow[o] = e.v;
                p.overflow_bin[o] = bin;
            }
        }
        e0 += U * kDenseThreads;
        if (e0 - tid >= n_ent) break;                                // workgroup-uniform
        look(e0);
        place();
    }
}

template <typename GT> struct TableOf;
template <> struct TableOf<g_f32> { using T = f32_t; };
template <> struct TableOf<g_bf16> { using T = bf16_t; };
template <> struct TableOf<g_f16> { using T = f16_t; };

// A workgroup per bin.  Its entries are sorted by row in LDS, 256 at a time, by
// counting; groups of `1 << group_shift` lanes, VE elements each, take a row each, sum its entries in registers and write
// it.  Rows of more than kHubEntries entries are summed by all groups together.  Entries beyond the first 256 of a bin
// are added to the rows that are written already, by the lanes that wrote them.
// (Bound by instructions before it was by the rows written: with the sums in LDS, cleared, added to and copied out, 46 us for
// 75,000 entries in 169,343 rows of 128 floats, and 110 us where LDS took them with atomics, at 3 to 7 clocks a lane.)
constexpr int kHubEntries = 32;
template <typename GT, int VE, bool SLOT_GRADS>
__global__ __launch_bounds__(kDenseThreads) void dense_write_kernel(const DenseParams p, int group_shift) {
    using Row = Chunk<typename TableOf<GT>::T, VE * (std::is_same<GT, g_f32>::value ? 4 : 2)>;
    using Raw = typename Row::Raw;
    extern __shared__ __align__(16) float partial[];                 // [groups][D], rows of many entries
    __shared__ int count[kDenseRowsMax], start[kDenseRowsMax];
    __shared__ int4 sorted[kDenseThreads];                           // root, slot, their coefficients
    __shared__ int wave_total[kDenseThreads / kWave];
    __shared__ int hubs[kDenseThreads / kHubEntries];
    __shared__ int n_hubs, picked;
    unsigned long long* const chosen = reinterpret_cast<unsigned long long*>(sorted);   // entries from the overflow list
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const int D = p.D;
    const uint32_t row_bytes = (uint32_t)D * (uint32_t)(sizeof(Raw) / VE);
    const int grp = tid >> group_shift, sl = tid & ((1 << group_shift) - 1), lanes = 1 << group_shift;
    const int n_grp = kDenseThreads >> group_shift;
    const char* const go = static_cast<const char*>(p.grad_out);
    const char* const gh = static_cast<const char*>(p.grad_h1);

    // acc += the gradients of the U sorted entries e, e + step, ... at byte `at` of their rows
    auto gather = [&](auto u_, float (&acc)[VE], int e, int step, uint32_t at) {
        constexpr int U = decltype(u_)::value;
        Raw a[U], b[U];
        int4 s[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            s[u] = sorted[e + u * step];
            a[u] = *reinterpret_cast<const Raw*>(go + ((uint64_t)(uint32_t)s[u].x * row_bytes + at));
            if constexpr (SLOT_GRADS) b[u] = *reinterpret_cast<const Raw*>(gh + ((uint64_t)(uint32_t)s[u].y * row_bytes + at));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            Row::fma(acc, a[u], __int_as_float(s[u].z));
            if constexpr (SLOT_GRADS) Row::fma(acc, b[u], __int_as_float(s[u].w));
        }
    };
    auto sum = [&](float (&acc)[VE], int e, int end, int step, uint32_t at) {
        for (; e + 3 * step < end; e += 4 * step) gather(std::integral_constant<int, 4>{}, acc, e, step, at);
        for (; e < end; e += step) gather(std::integral_constant<int, 1>{}, acc, e, step, at);
    };
    // The rows of a bin at `out`: n entries of theirs, thread tid has the tid-th; `more`: the rows are written already.
    auto add = [&](int n, Entry mine, char* out, int rows, bool more) {
        if (tid < rows) count[tid] = 0;
        if (tid == 0) n_hubs = 0;
        __syncthreads();
        const int place = tid < n ? atomicAdd(&count[mine.row()], 1) : 0;
        __syncthreads();
        const int c = tid < rows ? count[tid] : 0;
        int at = wave_inclusive_scan(c, lane);
        if (lane == kWave - 1) wave_total[wave] = at;
        if (c > kHubEntries) hubs[atomicAdd(&n_hubs, 1)] = tid;
        __syncthreads();
        for (int w = 0; w < wave; ++w) at += wave_total[w];
        if (tid < rows) start[tid] = at - c;
        __syncthreads();
        if (tid < n) {
            const float c1 = (float)mine.c1(), c2 = (float)mine.c2();
            sorted[start[mine.row()] + place] = make_int4((int)mine.root(), (int)(mine.root() * p.k1 + mine.slot()),
                                                          __float_as_int(1.0f / (c1 * c2)), __float_as_int(1.0f / c2));
        }
        __syncthreads();
        for (int r = grp; r < rows; r += n_grp) {
            const int m = count[r], e = start[r];
            if (m > kHubEntries || (more && m == 0)) continue;
            char* const row = out + (uint32_t)r * row_bytes;
            for (int d = sl * VE; d < D; d += lanes * VE) {
                const uint32_t by = (uint32_t)d * (uint32_t)(sizeof(Raw) / VE);
                float acc[VE] = {};
                if (more) Row::add(acc, *reinterpret_cast<const Raw*>(row + by));
                sum(acc, e, e + m, 1, by);
                *reinterpret_cast<Raw*>(row + by) = Row::pack(acc);
            }
        }
        const int nh = n_hubs;
        for (int h = 0; h < nh; ++h) {                               // workgroup-uniform
            const int r = hubs[h], e = start[r], end = e + count[r];
            for (int d = sl * VE; d < D; d += lanes * VE) {
                float acc[VE] = {};
                sum(acc, e + grp, end, n_grp, (uint32_t)d * (uint32_t)(sizeof(Raw) / VE));
#pragma unroll
                for (int k = 0; k < VE; ++k) partial[grp * D + d + k] = acc[k];
            }
            __syncthreads();
            if (grp == r % n_grp) {                                  // the lanes that write row r whenever it is written
                char* const row = out + (uint32_t)r * row_bytes;
                for (int d = sl * VE; d < D; d += lanes * VE) {
                    const uint32_t by = (uint32_t)d * (uint32_t)(sizeof(Raw) / VE);
                    float acc[VE] = {};
                    if (more) Row::add(acc, *reinterpret_cast<const Raw*>(row + by));
                    for (int g = 0; g < n_grp; ++g) {
#pragma unroll
                        for (int k = 0; k < VE; ++k) acc[k] += partial[g * D + d + k];
                    }
                    *reinterpret_cast<Raw*>(row + by) = Row::pack(acc);
                }
            }
            __syncthreads();
        }
        __syncthreads();
    };

    const int bin = blockIdx.x;
    const int64_t row0 = (int64_t)bin << p.row_shift;
    const int rows = (int)(p.N - row0 < (1ll << p.row_shift) ? p.N - row0 : 1ll << p.row_shift);
    char* const out = static_cast<char*>(p.grad_x) + row0 * row_bytes;
    // the counter and the first entries are requested together (places behind the counter hold anything)
    const int asked = p.counter[(size_t)bin * p.stride];
    const unsigned long long* const entries = p.entries + (size_t)bin * p.room;
    unsigned long long key = tid < p.room ? entries[tid] : 0ull;
    if (asked == 0) {                                                // zeros: the rows lie one after the other
        const uint32_t bytes = (uint32_t)rows * row_bytes;
        for (uint32_t i = tid * 16u; i + 16u <= bytes; i += kDenseThreads * 16u) *reinterpret_cast<uint4*>(out + i) = make_uint4(0u, 0u, 0u, 0u);
        for (uint32_t i = (bytes & ~15u) + 2u * tid; i < bytes; i += 2u * kDenseThreads) *reinterpret_cast<uint16_t*>(out + i) = 0;
        return;
    }
    const int held = asked < p.room ? asked : p.room;
    for (int i0 = 0; i0 < held; i0 += kDenseThreads) {               // workgroup-uniform, as every branch below
        const int n = held - i0 < kDenseThreads ? held - i0 : kDenseThreads;
        if (i0 > 0 && tid < n) key = entries[i0 + tid];
        add(n, Entry{key}, out, rows, i0 > 0);
    }
    if (asked <= p.room) return;
    const int n_over = *p.overflow_count;
    for (int i0 = 0; i0 < n_over; i0 += kDenseThreads) {
        if (tid == 0) picked = 0;
        __syncthreads();
        if (i0 + tid < n_over && p.overflow_bin[i0 + tid] == bin) chosen[atomicAdd(&picked, 1)] = p.overflow[i0 + tid];
        __syncthreads();
        const int n = picked;
        if (tid < n) key = chosen[tid];
        __syncthreads();
        if (n > 0) add(n, Entry{key}, out, rows, true);
    }
}

static bool dense_shape_ok(int64_t B, int k1, int k2, int64_t D, int64_t N) {
    const int64_t leaves = B * k1 * (k2 > 0 ? k2 : 1);
    if (B <= 0 || D > kDenseMaxD || N <= 0 || leaves > INT32_MAX) return false;
    if (k2 > 0 && B * kDenseThreads > (int64_t)UINT32_MAX) return false;             // a workgroup per root
    const DensePlan q = k2 > 0 ? dense_plan(B * k1, k2, D, N) : dense_plan(B, k1, D, N);
    return q.bins * kDenseThreads <= (int64_t)UINT32_MAX;
}

size_t dense_workspace_bytes(int64_t B, int k1, int k2, int64_t D, int64_t N) {
    if (!dense_shape_ok(B, k1, k2, D, N)) return 0;
    return (k2 > 0 ? dense_plan(B * k1, k2, D, N) : dense_plan(B, k1, D, N)).total;
}

// Against clearing and atomics, which take 48 ps per 64-byte segment of a leaf's row (20.8 G/s), with the dearer launches of
// this one to be made up for, and the rows of a table that is hardly touched, which a fill writes at 6.6 TB/s and this
// at 5.2.  Both ways, backward alone, by leaf slots and the share of them that has an ID: 169,343 rows of 128 floats,
// 256,000 slots (29 %) 58 -> 33 us, 16,000 21.4 / 20-22, 2 M 320 -> 157; of 128 bf16 elements 256,000 slots 38 -> 30; 500,000 rows of
// 64 floats, 300,000 slots (80 %) 79 -> 47; 2.4 M rows of 100 floats, 153,600 slots 233 -> 203; not taken: 10,000 rows of 64 floats,
// 10,240 slots 9 / 15; 1 M rows of 640 floats, 30,720 slots 428 / 496; of 32 fp16 elements, 307,200 slots 31 / 35.
bool dense_pays(int64_t B, int k1, int k2, int64_t D, int elem_bytes, int64_t N) {
    if (!dense_shape_ok(B, k1, k2, D, N)) return false;
    const int64_t leaves = B * k1 * (k2 > 0 ? k2 : 1);
    const int64_t segments = leaves * ((D * elem_bytes + 63) / 64);
    return segments >= kDenseMinSegments && leaves * kDenseMaxRowsPerSlot >= N;
}

template <typename GT> static hipError_t launch_dense(const DenseParams& p, hipStream_t stream) {
    constexpr int EB = std::is_same<GT, g_f32>::value ? 4 : 2;
    auto al = [](const void* q) { return reinterpret_cast<uintptr_t>(q) % (4 * EB) == 0; };
    const bool quads = p.D % 4 == 0 && al(p.grad_out) && al(p.grad_h1);
    const int units = quads ? p.D / 4 : p.D;
    int group_shift = 2;
    while (group_shift < 6 && (1 << group_shift) < units) ++group_shift;
    const size_t lds = sizeof(float) * (size_t)(kDenseThreads >> group_shift) * p.D;
    auto go = [&](auto ve, auto slots) {
        hipLaunchKernelGGL((dense_write_kernel<GT, decltype(ve)::value, decltype(slots)::value>), dim3((unsigned)p.bins), dim3(kDenseThreads),
                           lds, stream, p, group_shift);
    };
    auto with = [&](auto ve) { p.grad_h1 ? go(ve, std::true_type{}) : go(ve, std::false_type{}); };
    quads ? with(std::integral_constant<int, 4>{}) : with(std::integral_constant<int, 1>{});
    return hipGetLastError();
}

hipError_t launch_backward_dense(const BwdArgs& a, int64_t N, void* workspace, size_t workspace_bytes, hipStream_t stream) {
    if (!dense_shape_ok(a.B, a.k1, a.k2, a.D, N)) return hipErrorInvalidValue;
    const bool two = a.ids2 != nullptr;
    DenseParams p{};
    p.grad_out = a.grad_out; p.grad_h1 = a.grad_h1;
    p.ids1 = two ? a.ids1 : nullptr; p.leaf = two ? a.ids2 : a.ids1;
    p.grad_x = a.grad_x; p.slots = two ? a.B * a.k1 : a.B; p.N = N; p.D = (int)a.D;
    p.k1 = two ? a.k1 : 1; p.k2 = two ? a.k2 : a.k1;
    p.slots_per_wg = two ? a.k1 : kDenseThreads / a.k1;
    const DensePlan q = dense_plan(p.slots, p.k2, a.D, N);
    if (workspace_bytes < q.total) return hipErrorInvalidValue;
    char* w = static_cast<char*>(workspace);
    p.row_shift = q.row_shift; p.bins = (int)q.bins; p.room = q.room; p.stride = q.stride;
    p.counter = reinterpret_cast<int*>(w + q.off[0]);
    p.overflow_count = reinterpret_cast<int*>(w + q.off[1]);
    p.entries = reinterpret_cast<unsigned long long*>(w + q.off[2]);
    p.overflow = reinterpret_cast<unsigned long long*>(w + q.off[3]);
    p.overflow_bin = reinterpret_cast<int*>(w + q.off[4]);
    hipLaunchKernelGGL(dense_clear_kernel, dim3((p.bins + 255) / 256), dim3(256), 0, stream, p.counter, p.bins, p.stride, p.overflow_count);
    hipLaunchKernelGGL(dense_bin_kernel, dim3((unsigned)((p.slots + p.slots_per_wg - 1) / p.slots_per_wg)), dim3(kDenseThreads), 0, stream, p);
    if (hipError_t e = hipGetLastError()) return e;
    switch (a.grad_kind) {
        case 0:  return launch_dense<g_f32>(p, stream);
        case 1:  return launch_dense<g_bf16>(p, stream);
        default: return launch_dense<g_f16>(p, stream);
    }
}

}  // namespace fsa

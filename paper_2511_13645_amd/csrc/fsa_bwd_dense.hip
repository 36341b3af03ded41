// Backward into a gradient of its own (fsa_mean_bwd_dense): every row of grad_x is written once, rows that
// no leaf names as zeros, so a caller that wants the whole gradient of the table -- torch.autograd does --
// neither clears it first nor adds to it with atomics.  The paper describes no backward kernel (Sec. 3.3
// "Reproducibility" only asks that the saved IDs are replayed).
//
// What bounds it: the rows written (N*D elements, once).  Clearing first and adding with atomics wrote them all, read
// the named ones back and paid a 64-byte segment's atomic (20.8 G/s) for every 64 bytes of every leaf.
//
// Four launches on the caller's stream, all state in the caller's workspace:
//   clear   zero the bins' counters (a fill kernel: a memset node must not end up in a captured graph);
//   bin     grad_x is cut into bins of consecutive rows; every live leaf slot appends an entry to its row's bin.
//           A full bin gets a tile, its rows in fp32, and further entries go to lists;
//   rest    the workgroups of a list share its entries out by rows, up to 4096 at a time, sum them and add one row per
//           distinct row to its bin's tile: however a batch's leaves are skewed, no more row atomics than leaf by leaf;
//   write   a workgroup per bin sums the gradients of its rows' entries in registers, in fp32, adds the tile if there
//           is one, and writes every row.
// The order of additions follows the places that the entries got, which varies from run to run, as with atomics.
#include "fsa_atomic_rows.hip.h"
#include "fsa_device.hip.h"
#include "fsa_internal.h"

#include <type_traits>

namespace fsa {

constexpr int kDenseThreads = 256;
constexpr int kBinTile = 1024;                                       // leaf slots of a binning workgroup, or one root's
constexpr int kBinWorkgroups = 256;                                  // one to a compute unit before any takes more than a root
// Elements of a bin, and its rows: enough entries per workgroup to pay for its steps (the whole call, 256,000 slots on 169,343
// rows of 128 floats: 4096 elements 38.6 us, 8192 36.8, 16384 36.9; 300,000 on 500,000 of 64 46.7 / 44.3 / 44.3; 1.2 M on 2.4 M of
// 100 441 / 380 / 330), and several rows per group of lanes where rows are wide (50,000 on 30,000 rows of 300 floats: 8 / 16 / 32
// rows 35 / 36 / 29).  Several bins per workgroup, the next one's entries requested ahead: 2 to 8 % slower on large tables.
constexpr int kDenseBinElements = 8192;
constexpr int kDenseRowsMin = 32;
constexpr int kDenseRowsMax = 256;
// Fewer rows where a bin would have more leaf slots: a workgroup's 256 entries are one pass, and rows that meet again in
// the next one are read back, one trip to memory after the other.  20,000 rows of 64 floats, 256,000 slots (68 % live): 128 rows
// to a bin 65 us, 16 28; 1.25 M slots 270, 89; 8 rows are slower where hub rows lie side by side (169,343 rows sorted by
// degree, 2 M slots: 146 us with 16, 209 with 8).  With half the line nearly empty tables lose: 2 M rows of 64 floats, 2 M
// slots, a tenth live: 150 us at 64 rows to a bin, 182 at 32.
constexpr int64_t kDenseLoad = 128;
constexpr int kDenseRowsLoaded = 16;
// Room of a bin at most: longer is a longer chain for one workgroup, shorter leaves more of an evenly loaded batch to the
// lists (16 M leaf slots, 28 % live, on 169,343 rows of 128 floats: 512 1260 us, 1024 974, 2048 788, the longest bin 82 us).
constexpr int kDenseMostRoom = 2048;
constexpr int kRestLists = 32;                                       // of entries that found their bins full: a wave's append is an
                                                                     // atomic on its list's length, one per 11 ns on one address
constexpr int kCountStride = 2 * kSegment;                           // ints between their lengths: a 128-byte line each
constexpr int64_t kDenseMinSegments = 768 * 1024;                   // see dense_pays
constexpr int64_t kDenseMinSegmentsSingles = 8 * 1024 * 1024;
constexpr int64_t kDenseMaxRowsPerSlot = 2;
constexpr int64_t kDenseMinRowBytes = 256;
constexpr int64_t kDenseMinBins = 512;
constexpr int64_t kDenseMostLoad = 4096;                            // leaf slots to a bin
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
    int* counter; int* rest_count; int* tile_count;
    unsigned long long* entries;          // [bins][room]
    unsigned long long* rest; int* rest_bin;                         // [kRestLists][rest_room]: entries and their bins
    int64_t rest_room;
    int* tile_of; float* tiles;           // [bins], full bins only; [tiles][rows of a bin][D]
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

struct DensePlan { int row_shift, room, stride; int64_t bins, rest_room; size_t off[7], total; };

static DensePlan dense_plan(int64_t slots, int k2, int slots_per_wg, int64_t D, int64_t N) {
    DensePlan q{};
    while ((2ll << q.row_shift) <= kDenseRowsMax && (2ll << q.row_shift) * D <= kDenseBinElements) ++q.row_shift;
    while ((1 << q.row_shift) < kDenseRowsMin) ++q.row_shift;
    while ((1 << q.row_shift) > kDenseRowsLoaded && slots * k2 / ((N >> q.row_shift) + 1) > kDenseLoad) --q.row_shift;
    q.bins = (N + (1ll << q.row_shift) - 1) >> q.row_shift;
    // room for four times the mean with every slot full, while that is no long chain for the bin's workgroup (twice / four /
    // eight times: 256,000 slots on 169,343 rows of 128 floats 39.8 / 36.8 / 36.9 us, 2 M 119 / 117 / 125)
    const int64_t leaves = slots * k2, mean = leaves / q.bins;
    q.room = 32;
    while (q.room < kDenseMostRoom && q.room < 4 * mean) q.room *= 2;
    q.stride = q.bins <= 16384 ? kSegment * 2 : 4;                   // few counters: a 128-byte line each, over all L2 channels
    const int64_t full = (leaves - 1) / q.room < q.bins ? (leaves - 1) / q.room : q.bins;   // bins that can get a tile
    const int64_t wgs = (slots + slots_per_wg - 1) / slots_per_wg;                          // of the binning
    q.rest_room = full > 0 ? (wgs + kRestLists - 1) / kRestLists * slots_per_wg * k2 : 0;
    size_t o = 0;
    auto take = [&](int i, size_t bytes) { q.off[i] = o; o += (bytes + 255) & ~(size_t)255; };
    take(0, (size_t)q.bins * q.stride * sizeof(int));
    take(1, kRestLists * kCountStride * sizeof(int) + sizeof(int));
    take(2, (size_t)q.bins * q.room * sizeof(unsigned long long));
    take(3, kRestLists * (size_t)q.rest_room * sizeof(unsigned long long));
    take(4, kRestLists * (size_t)q.rest_room * sizeof(int));
    take(5, full > 0 ? (size_t)q.bins * sizeof(int) : 0);
    take(6, ((size_t)full << q.row_shift) * D * sizeof(float));
    q.total = o;
    return q;
}

__global__ __launch_bounds__(256) void dense_clear_kernel(int* counter, int bins, int stride, int* rest_count, int* tile_count) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < bins) counter[(size_t)i * stride] = 0;
    if (i < kRestLists) rest_count[i * kCountStride] = 0;
    if (i == 0) *tile_count = 0;
}

// A workgroup takes whole roots, as many as have kBinTile leaf slots while there are workgroups enough.  Bound by the chain
// IDs -> place (a returning atomic) -> entry, which four leaf slots per thread go through together; the slots are counted
// on the way.  Leaf slots of one bin are merged in LDS before they ask for places: atomics on one address go through at
// one per 11 ns, and a hub's bin is asked by every root (153,600 leaves of one row, the kernel alone: 1720 -> 11 us; without
// hubs 9 us either way).  A bin that finds its two places of the table taken by others is asked directly.
constexpr int kBinTable = 2048;
__global__ __launch_bounds__(kDenseThreads) void dense_bin_kernel(const DenseParams p) {
    __shared__ int on[kBinTile], cnt[kBinTile];                      // by slot: takes part; leaf slots that do
    __shared__ int live[kBinTile];                                   // by root: slots that take part
    __shared__ int tag[kBinTable], asked[kBinTable], got[kBinTable]; // bin; entries of it; the first one's place
    const int tid = threadIdx.x;
    const int64_t slot0 = (int64_t)blockIdx.x * p.slots_per_wg;
    const int n_slots = (int)(p.slots - slot0 < p.slots_per_wg ? p.slots - slot0 : p.slots_per_wg);
    const int32_t* leaf = p.leaf + slot0 * p.k2;
    const int n_ent = n_slots * p.k2;                                // at most kBinTile, or one root's 64 * 64
    for (int s = tid; s < n_slots; s += kDenseThreads) {
        on[s] = p.ids1 ? p.ids1[slot0 + s] : 0;
        cnt[s] = live[s] = 0;
    }
    __syncthreads();
    constexpr int U = kBinTile / kDenseThreads;
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
    // the places of these entries, in two halves between which the table is complete
    int h[U];
    auto ask = [&] {
        for (int i = tid; i < kBinTable; i += kDenseThreads) { tag[i] = -1; asked[i] = 0; }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < U; ++k) {
            h[k] = -1;
            at[k] = 0;
            if (id[k] < 0) continue;
            const int bin = id[k] >> p.row_shift;
            int t = (int)(((uint32_t)bin * 2654435761u) >> 21), was = atomicCAS(&tag[t], -1, bin);
            if (was != -1 && was != bin) { t ^= 1; was = atomicCAS(&tag[t], -1, bin); }
            if (was != -1 && was != bin) {
                at[k] = atomicAdd(&p.counter[(size_t)bin * p.stride], 1);
            } else {
                h[k] = was == -1 ? t | kBinTable : t;                // the one that claimed it asks for all
                at[k] = atomicAdd(&asked[t], 1);
            }
        }
    };
    auto place = [&] {
        __syncthreads();
#pragma unroll
        for (int k = 0; k < U; ++k) {
            if (h[k] >= kBinTable) {
                const int t = h[k] & (kBinTable - 1);
                got[t] = atomicAdd(&p.counter[(size_t)(id[k] >> p.row_shift) * p.stride], asked[t]);
            }
        }
        __syncthreads();
#pragma unroll
        for (int k = 0; k < U; ++k) { if (h[k] >= 0) at[k] += got[h[k] & (kBinTable - 1)]; }
    };
    look(tid);
    ask();
#pragma unroll
    for (int k = 0; k < U; ++k) { if (id[k] >= 0) atomicAdd(&cnt[slot[k]], 1); }
    for (int e = tid + U * kDenseThreads; e < n_ent; e += kDenseThreads) {
        const int j = e / p.k2;
        if (on[j] >= 0 && leaf[e] >= 0) atomicAdd(&cnt[j], 1);
    }
    __syncthreads();
    for (int s = tid; s < n_slots; s += kDenseThreads) { if (cnt[s] > 0) atomicAdd(&live[s / p.k1], 1); }
    place();
    const int lane = tid & (kWave - 1);
    const int64_t root0 = slot0 / p.k1;
    for (int e0 = tid;;) {
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int bin = id[k] >> p.row_shift;
            const int of = slot[k] / p.k1;                           // its root
            const Entry e = Entry::of(id[k] & ((1 << p.row_shift) - 1), root0 + of, slot[k] - of * p.k1, live[of], cnt[slot[k]]);
            if (id[k] >= 0 && at[k] < p.room) p.entries[(size_t)bin * p.room + at[k]] = e.v;
            const bool over = id[k] >= 0 && at[k] >= p.room;
            const uint64_t all = __ballot(over);
            if (all == 0) continue;                                  // wave-uniform
            const int list = blockIdx.x % kRestLists;                // has room for all entries of its workgroups
            int n_before = 0;
            if (lane == 0) n_before = atomicAdd(&p.rest_count[list * kCountStride], __popcll(all));
            const int64_t o = list * p.rest_room + __shfl(n_before, 0) + __popcll(all & lanemask_lt(lane));
            if (over) { p.rest[o] = e.v; p.rest_bin[o] = bin; }
            // the bin's first entry too many gets it a tile, which this wave clears
            for (uint64_t first = __ballot(over && at[k] == p.room); first; first &= first - 1) {
                const int from = __ffsll((unsigned long long)first) - 1;
                int t = 0;
                if (lane == from) {
                    t = atomicAdd(p.tile_count, 1);
                    p.tile_of[bin] = t;
                }
                t = __shfl(t, from);
                const size_t n = (size_t)p.D << p.row_shift;         // a multiple of 16
                float4* const tile = reinterpret_cast<float4*>(p.tiles + (size_t)t * n);
                for (size_t i = lane; i < n / 4; i += kWave) tile[i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
            }
        }
        e0 += U * kDenseThreads;
        if (e0 - tid >= n_ent) break;                                // workgroup-uniform
        look(e0);
        __syncthreads();                                             // the table's last readers
        ask();
        place();
    }
}

template <typename GT> struct TableOf;
template <> struct TableOf<g_f32> { using T = f32_t; };
template <> struct TableOf<g_bf16> { using T = bf16_t; };
template <> struct TableOf<g_f16> { using T = f16_t; };

// Rows of more than kHubEntries of a workgroup's 256 entries are summed by all of its groups together.
constexpr int kHubEntries = 32;

// What a workgroup of the two kernels below knows of 256 entries sorted by rows, which groups of `1 << group_shift`
// lanes, VE elements each, sum in registers: a row each, or a hub row all together.
template <typename GT, int VE, bool SLOT_GRADS> struct RowSums {
    using Row = Chunk<typename TableOf<GT>::T, VE * (std::is_same<GT, g_f32>::value ? 4 : 2)>;
    using Raw = typename Row::Raw;
    const DenseParams& p;
    const int group_shift;
    const int4* const sorted;                                        // LDS: root, slot, their coefficients
    const int *const count, *const start;                            // LDS, by row: entries, the first one's place
    const int* const hubs;                                           // LDS: rows of more than kHubEntries
    float* const partial;                                            // LDS: [groups][D]

    __device__ static int4 sorted_entry(const Entry e, int k1) {
        const float c1 = (float)e.c1(), c2 = (float)e.c2();
        return make_int4((int)e.root(), (int)(e.root() * k1 + e.slot()), __float_as_int(1.0f / (c1 * c2)), __float_as_int(1.0f / c2));
    }

    // acc += the gradients of the U sorted entries e, e + step, ... at byte `at` of their rows
    template <int U> __device__ __forceinline__ void gather(float (&acc)[VE], int e, int step, uint32_t at) const {
        const uint32_t row_bytes = (uint32_t)p.D * (uint32_t)(sizeof(Raw) / VE);
        Raw a[U], b[U];
        int4 s[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            s[u] = sorted[e + u * step];
            a[u] = *reinterpret_cast<const Raw*>(static_cast<const char*>(p.grad_out) + ((uint64_t)(uint32_t)s[u].x * row_bytes + at));
            if constexpr (SLOT_GRADS)
                b[u] = *reinterpret_cast<const Raw*>(static_cast<const char*>(p.grad_h1) + ((uint64_t)(uint32_t)s[u].y * row_bytes + at));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            Row::fma(acc, a[u], __int_as_float(s[u].z));
            if constexpr (SLOT_GRADS) Row::fma(acc, b[u], __int_as_float(s[u].w));
        }
    }
    __device__ __forceinline__ void sum(float (&acc)[VE], int e, int end, int step, uint32_t at) const {
        for (; e + 3 * step < end; e += 4 * step) gather<4>(acc, e, step, at);
        for (; e < end; e += step) gather<1>(acc, e, step, at);
    }

    // out(r, d, acc) for every row r < rows and its elements d, always by the same lanes for one r; rows without entries
    // only if `empty`.  All threads of the workgroup, between two barriers.
    template <typename F> __device__ __forceinline__ void operator()(int rows, bool empty, int n_hubs, F out) const {
        const int tid = threadIdx.x, grp = tid >> group_shift, n_grp = kDenseThreads >> group_shift;
        const int lanes = 1 << group_shift, D = p.D, d0 = (tid & (lanes - 1)) * VE;
        constexpr uint32_t EB = sizeof(Raw) / VE;
        for (int r = grp; r < rows; r += n_grp) {
            const int m = count[r], e = start[r];
            if (m > kHubEntries || (!empty && m == 0)) continue;
            for (int d = d0; d < D; d += lanes * VE) {
                float acc[VE] = {};
                sum(acc, e, e + m, 1, (uint32_t)d * EB);
                out(r, d, acc);
            }
        }
        for (int h = 0; h < n_hubs; ++h) {                           // workgroup-uniform
            const int r = hubs[h], e = start[r], end = e + count[r];
            for (int d = d0; d < D; d += lanes * VE) {
                float acc[VE] = {};
                sum(acc, e + grp, end, n_grp, (uint32_t)d * EB);
#pragma unroll
                for (int k = 0; k < VE; ++k) partial[grp * D + d + k] = acc[k];
            }
            __syncthreads();
            if (grp == r % n_grp) {
                for (int d = d0; d < D; d += lanes * VE) {
                    float acc[VE] = {};
                    for (int g = 0; g < n_grp; ++g) {
#pragma unroll
                        for (int k = 0; k < VE; ++k) acc[k] += partial[g * D + d + k];
                    }
                    out(r, d, acc);
                }
            }
            __syncthreads();
        }
    }
};

// The entries that found their bins full.  The workgroups of a list read up to 4096 of them together and share them out by
// row classes, so that a row's entries meet in one workgroup; a class that a hub fills is shared out by place instead.  Each
// takes its share up to 256 entries at a time: rows are told apart in an LDS table, and each distinct row's sum is added to its
// tile.  Bound by these adds (20.8 G 64-byte segments/s) where many rows take part, else by a group's trips to memory,
// one row after the other.  Shares by place alone left rows of a dense front apart: nine tenths of 153,600 leaves on 1000 of
// 100,000 rows of 128 floats 69 us, this way 35; all on one row 25 and 29.  Short lists have little to bring together
// and reading all of them costs 2 us.
constexpr int kRestTable = 2 * kDenseThreads;
constexpr int kRestLeast = 32;                                       // entries a workgroup takes at least, in the mean; at most:
constexpr int kRestMost = kDenseThreads;                             // (192 2 % ahead on some fronts, 4 % behind on hubs)
constexpr int kRestShort = 64;                                       // up to this mean the shares go by place alone
constexpr int kRestEach = 16;                                        // workgroups to a list
constexpr int kRestClasses = 4 * kRestEach;
constexpr int kRestLoads = kRestEach * kRestMost / kDenseThreads;    // entries that a thread reads of those shared out
constexpr int kRestShare = (kRestClasses / kRestEach / 2 + 1) * kRestMost;   // classes of up to half a mean share, and places
template <typename GT, int VE, bool SLOT_GRADS>
__global__ __launch_bounds__(kDenseThreads) void dense_rest_kernel(const DenseParams p, int group_shift) {
    using Sums = RowSums<GT, VE, SLOT_GRADS>;
    extern __shared__ __align__(16) float partial[];
    __shared__ uint32_t tag[kRestTable];
    __shared__ int seen[kRestTable], first[kRestTable];              // by table place: entries; the first one's place
    __shared__ uint32_t row[kDenseThreads];                          // distinct rows, of all tiles
    __shared__ int count[kDenseThreads], start[kDenseThreads];
    __shared__ int4 sorted[kDenseThreads];
    __shared__ int wave_total[kDenseThreads / kWave];
    __shared__ int hubs[kDenseThreads / kHubEntries];
    __shared__ int n_rows, n_hubs;
    __shared__ int of_class[kRestClasses];                           // entries
    __shared__ unsigned long long share[kRestShare];
    __shared__ int share_bin[kRestShare], n_share;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const Sums sums{p, group_shift, sorted, count, start, hubs, partial};
    const int list = blockIdx.x % kRestLists, turn = blockIdx.x / kRestLists;
    const unsigned total = (unsigned)p.rest_count[list * kCountStride];
    unsigned each = (total + kRestEach - 1) / kRestEach;
    each = each < kRestLeast ? kRestLeast : each < kRestMost ? each : kRestMost;
    for (unsigned i0 = 0; i0 < total; i0 += kRestEach * each) {      // workgroup-uniform, as the passes below
        const unsigned here = total - i0 < kRestEach * each ? total - i0 : kRestEach * each;
        const int64_t at0 = list * p.rest_room + i0;
        int shared;
        if (each <= kRestShort) {
            const unsigned from = turn * each;
            shared = here > from ? (int)(here - from < each ? here - from : each) : 0;
            if (tid < shared) { share[tid] = p.rest[at0 + from + tid]; share_bin[tid] = p.rest_bin[at0 + from + tid]; }
        } else {
            for (int c = tid; c < kRestClasses; c += kDenseThreads) of_class[c] = 0;
            if (tid == 0) n_share = 0;
            __syncthreads();
            Entry of[kRestLoads];
            int bin[kRestLoads], cls[kRestLoads];
#pragma unroll
            for (int k = 0; k < kRestLoads; ++k) {
                const unsigned i = k * kDenseThreads + tid;
                of[k].v = p.rest[at0 + (i < here ? i : 0)];
                bin[k] = p.rest_bin[at0 + (i < here ? i : 0)];
            }
            int run = -1, n_run = 0;                                 // a hub's entries are counted once per thread
#pragma unroll
            for (int k = 0; k < kRestLoads; ++k) {
                const uint32_t r = (uint32_t)bin[k] << p.row_shift | (uint32_t)of[k].row();
                cls[k] = k * kDenseThreads + tid < here ? (int)((r * 0x9e3779b1u ^ r >> 3) * 0x85ebca6bu >> 26) : -1;
                if (cls[k] != run) {
                    if (run >= 0) atomicAdd(&of_class[run], n_run);
                    run = cls[k];
                    n_run = 0;
                }
                ++n_run;
            }
            if (run >= 0) atomicAdd(&of_class[run], n_run);
            __syncthreads();
#pragma unroll
            for (int k = 0; k < kRestLoads; ++k) {
                const unsigned i = k * kDenseThreads + tid;
                const bool mine = cls[k] >= 0 && (of_class[cls[k]] <= (int)each / 2 ? cls[k] % kRestEach == turn : i / each == (unsigned)turn);
                const uint64_t all = __ballot(mine);
                int n_before = 0;
                if (lane == 0 && all) n_before = atomicAdd(&n_share, __popcll(all));
                const int o = __shfl(n_before, 0) + __popcll(all & lanemask_lt(lane));   // < kRestShare
                if (mine) { share[o] = of[k].v; share_bin[o] = bin[k]; }
            }
            __syncthreads();
            shared = n_share;
        }
        for (int j0 = 0; j0 < shared; j0 += kDenseThreads) {
            const int n = shared - j0 < kDenseThreads ? shared - j0 : kDenseThreads;
            Entry mine{0};
            uint32_t to = ~0u;                                       // (no row's number: there are fewer than 2^24 bins)
            if (tid < n) {
                mine.v = share[j0 + tid];
                to = (uint32_t)p.tile_of[share_bin[j0 + tid]] << p.row_shift | (uint32_t)mine.row();
            }
            for (int h = tid; h < kRestTable; h += kDenseThreads) { tag[h] = ~0u; seen[h] = 0; }
            if (tid == 0) { n_rows = 0; n_hubs = 0; }
            __syncthreads();
            int h = 0, place = 0;
            bool owner = false;
            if (tid < n) {                                           // twice as many places as rows: one is found
                for (h = (int)((to * 2654435761u) >> 23);; h = (h + 1) & (kRestTable - 1)) {
                    const uint32_t was = atomicCAS(&tag[h], ~0u, to);
                    owner = was == ~0u;
                    if (owner || was == to) break;
                }
                place = atomicAdd(&seen[h], 1);
            }
            __syncthreads();
            const int c = owner ? seen[h] : 0;
            int at = wave_inclusive_scan(c, lane);
            if (lane == kWave - 1) wave_total[wave] = at;
            __syncthreads();
            for (int w = 0; w < wave; ++w) at += wave_total[w];
            if (owner) {
                const int r = atomicAdd(&n_rows, 1);
                row[r] = to; count[r] = c; start[r] = first[h] = at - c;
                if (c > kHubEntries) hubs[atomicAdd(&n_hubs, 1)] = r;
            }
            __syncthreads();
            if (tid < n) sorted[first[h] + place] = Sums::sorted_entry(mine, p.k1);
            __syncthreads();
            sums(n_rows, false, n_hubs, [&](int r, int d, const float (&acc)[VE]) {
                // the lanes trade elements, so that each atomic instruction covers consecutive ones
                const int lanes = 1 << group_shift, sl = tid & (lanes - 1), d0 = d - sl * VE;
                const int on = (p.D - d0) / VE < lanes ? (p.D - d0) / VE : lanes;     // lanes that are here
                float* const mine = partial + (tid >> group_shift) * p.D + d0;
                float* const to = p.tiles + (size_t)row[r] * p.D + d0;
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int k = 0; k < VE; ++k) mine[sl * VE + k] = acc[k];
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int k = 0; k < VE; ++k) atomicAdd(to + sl + k * on, mine[sl + k * on]);
            });
            __syncthreads();
        }
        __syncthreads();
    }
}

// A workgroup per bin.  Its entries are sorted by row in LDS, 256 at a time, by counting.  Entries beyond the first 256
// of a bin are added to the rows that are written already, by the lanes that wrote them.
// (Bound by instructions before it was by the rows written: with the sums in LDS, cleared, added to and copied out, 46 us for
// 75,000 entries in 169,343 rows of 128 floats, and 110 us where LDS took them with atomics, at 3 to 7 clocks a lane.)
template <typename GT, int VE, bool SLOT_GRADS>
__global__ __launch_bounds__(kDenseThreads) void dense_write_kernel(const DenseParams p, int group_shift) {
    using Sums = RowSums<GT, VE, SLOT_GRADS>;
    using Row = typename Sums::Row;
    using Raw = typename Sums::Raw;
    extern __shared__ __align__(16) float partial[];
    __shared__ int count[kDenseRowsMax], start[kDenseRowsMax];
    __shared__ int4 sorted[kDenseThreads];
    __shared__ int wave_total[kDenseThreads / kWave];
    __shared__ int hubs[kDenseThreads / kHubEntries];
    __shared__ int n_hubs;
    const int tid = threadIdx.x, lane = tid & (kWave - 1), wave = tid >> 6;
    const Sums sums{p, group_shift, sorted, count, start, hubs, partial};
    const uint32_t row_bytes = (uint32_t)p.D * (uint32_t)(sizeof(Raw) / VE);

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
    const float* const tile = asked > p.room ? p.tiles + (((size_t)p.tile_of[bin] << p.row_shift) * p.D) : nullptr;
    for (int i0 = 0; i0 < held; i0 += kDenseThreads) {               // workgroup-uniform, as every branch below
        const bool more = i0 > 0;                                    // the rows are written already
        const int n = held - i0 < kDenseThreads ? held - i0 : kDenseThreads;
        if (more && tid < n) key = entries[i0 + tid];
        const Entry mine{key};
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
        if (tid < n) sorted[start[mine.row()] + place] = Sums::sorted_entry(mine, p.k1);
        __syncthreads();
        sums(rows, !more, n_hubs, [&](int r, int d, float (&acc)[VE]) {
            Raw* const to = reinterpret_cast<Raw*>(out + ((uint32_t)r * row_bytes + (uint32_t)d * (uint32_t)(sizeof(Raw) / VE)));
            if (more) Row::add(acc, *to);
            if (!more && tile) {
#pragma unroll
                for (int k = 0; k < VE; ++k) acc[k] += tile[r * p.D + d + k];
            }
            *to = Row::pack(acc);
        });
        __syncthreads();
    }
}

// Slots that a binning workgroup takes: those of whole roots (one hop: k1 = 1, a seed is a slot).
static int slots_of_workgroup(int64_t B, int k1, int k2) {
    const int64_t most = kBinTile / (k1 * k2), fair = B / kBinWorkgroups, roots = most < fair ? most : fair;
    return k1 * (int)(roots > 1 ? roots : 1);
}

static DensePlan dense_plan_of(int64_t B, int k1, int k2, int64_t D, int64_t N) {
    return k2 > 0 ? dense_plan(B * k1, k2, slots_of_workgroup(B, k1, k2), D, N) : dense_plan(B, k1, slots_of_workgroup(B, 1, k1), D, N);
}

static bool dense_shape_ok(int64_t B, int k1, int k2, int64_t D, int64_t N) {
    const int64_t leaves = B * k1 * (k2 > 0 ? k2 : 1);
    if (B <= 0 || D > kDenseMaxD || N <= 0 || leaves > INT32_MAX) return false;
    if (k2 > 0 && B * kDenseThreads > (int64_t)UINT32_MAX) return false;             // a workgroup per root
    return dense_plan_of(B, k1, k2, D, N).bins * kDenseThreads <= (int64_t)UINT32_MAX;
}

size_t dense_workspace_bytes(int64_t B, int k1, int k2, int64_t D, int64_t N) {
    return dense_shape_ok(B, k1, k2, D, N) ? dense_plan_of(B, k1, k2, D, N).total : 0;
}

// Against clearing and atomics, which take 48 ps per 64-byte segment of a leaf's row (20.8 G/s), with the dearer launches of
// this one to be made up for, and the rows of a table that is hardly touched, which a fill writes at 6.6 TB/s and this
// at 5.2.  Both ways, backward alone, by leaf slots and the share of them that has an ID: 169,343 rows of 128 floats,
// 256,000 slots (29 %) 57 / 37 us, 100,000 33 / 27, 2 M 305 / 114; as bf16 256,000 36 / 34; 2.4 M rows of 100 floats, 1.2 M slots
// (96 %) 599 / 380; not taken: 50,000 slots on the 169,343 rows 26 / 25.
// Rows that nothing names are the line of the rows: with 256,000 slots on rows of 128 floats and 13 / 30 / 100 % of them live,
// two rows a slot 52 / 70 / 140 against 51 / 57 / 66 us, four 105 / 124 / 191 against 121 / 121 / 121.  (Below a tenth live
// it is behind whatever the rows: 5 % on half a row, one and two rows a slot 22 / 29 / 45 against 23 / 32 / 53.  And the host
// does not see a crowded run of the table so large that its rows seldom meet in a list: nine tenths of 300,000 slots, 80 %
// live, on 5000 of 500,000 rows of 64 floats 73 / 102, where the same slots without order are 75 / 44.)
// Few bins leave the chip idle, long ones are a chain, and narrow rows cost the atomics least: 300 rows of 128 floats, 153,600
// slots (80 %) 59 / 81 us, 2100 of 64, 256,000 65 / 67; 4000 of 32, 2 M slots, 8192 to a bin, 260 / 404, at 4096 8000 rows 265 / 261,
// of 64 floats 449 / 255; 200,000 rows of 16 floats, 1.2 M slots 57 / 74, 1 M of 24, 512,000 34 / 45.
// Rows that are not made of quads go through the write kernel one element a lane, so a bin of hub rows is a chain four times as
// long, which only a large call hides.  With rows sorted by degree, 301 floats on 30,000 rows, 1.6 / 3.4 / 13.5 M segments
// 65 / 116 / 386 against 121 / 112 / 416 us; 602 floats on 60,000 1.5 / 6.4 / 12.8 M 75 / 202 / 358 against 135 / 276 / 307;
// in no order (602 on 232,965, 9.5 M) 590 / 258.
// One hop is left to the atomics, which sum the rows that seeds of a workgroup share in LDS: 15,000 entities x 128 floats,
// 16,384 x 15 leaf slots of a knowledge graph (46 % live) 57 us that way and 85 this, all leaves on one row 35 / 49, where a
// graph without such hubs (500,000 x 64, 30,000 x 10, 80 % live) would be 79 / 49.
bool dense_pays(int64_t B, int k1, int k2, int64_t D, int elem_bytes, int64_t N) {
    if (k2 == 0 || !dense_shape_ok(B, k1, k2, D, N)) return false;
    const int64_t leaves = B * k1 * k2;
    const int64_t segments = leaves * ((D * elem_bytes + 63) / 64);
    const int64_t bins = dense_plan_of(B, k1, k2, D, N).bins;
    return segments >= (D % 4 == 0 ? kDenseMinSegments : kDenseMinSegmentsSingles) && leaves * kDenseMaxRowsPerSlot >= N &&
           D * elem_bytes >= kDenseMinRowBytes && bins >= kDenseMinBins && leaves <= bins * kDenseMostLoad;
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
        if (p.rest_room > 0)                                         // else no bin is ever full
            hipLaunchKernelGGL((dense_rest_kernel<GT, decltype(ve)::value, decltype(slots)::value>), dim3(kRestLists * kRestEach),
                               dim3(kDenseThreads), lds, stream, p, group_shift);
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
    p.slots_per_wg = two ? slots_of_workgroup(a.B, a.k1, a.k2) : slots_of_workgroup(a.B, 1, a.k1);
    const DensePlan q = dense_plan_of(a.B, a.k1, two ? a.k2 : 0, a.D, N);
    if (workspace_bytes < q.total) return hipErrorInvalidValue;
    char* w = static_cast<char*>(workspace);
    p.row_shift = q.row_shift; p.bins = (int)q.bins; p.room = q.room; p.stride = q.stride; p.rest_room = q.rest_room;
    p.counter = reinterpret_cast<int*>(w + q.off[0]);
    p.rest_count = reinterpret_cast<int*>(w + q.off[1]);
    p.tile_count = p.rest_count + kRestLists * kCountStride;
    p.entries = reinterpret_cast<unsigned long long*>(w + q.off[2]);
    p.rest = reinterpret_cast<unsigned long long*>(w + q.off[3]);
    p.rest_bin = reinterpret_cast<int*>(w + q.off[4]);
    p.tile_of = reinterpret_cast<int*>(w + q.off[5]);
    p.tiles = reinterpret_cast<float*>(w + q.off[6]);
    hipLaunchKernelGGL(dense_clear_kernel, dim3((p.bins + 255) / 256), dim3(256), 0, stream, p.counter, p.bins, p.stride, p.rest_count, p.tile_count);
    hipLaunchKernelGGL(dense_bin_kernel, dim3((unsigned)((p.slots + p.slots_per_wg - 1) / p.slots_per_wg)), dim3(kDenseThreads), 0, stream, p);
    if (hipError_t e = hipGetLastError()) return e;
    switch (a.grad_kind) {
        case 0:  return launch_dense<g_f32>(p, stream);
        case 1:  return launch_dense<g_bf16>(p, stream);
        default: return launch_dense<g_f16>(p, stream);
    }
}

}  // namespace fsa

// Backward kernels: the adjoint of the replay forward with respect to the feature table
// (Sec. 3.3 "Reproducibility" of arXiv 2511.13645: backward replays the saved IDs so that
// gradients reach the same sampled neighborhoods).  The paper does not describe a kernel.
//
// Mapping: the same ownership as the forward (wave per seed; workgroup per root with waves
// owning interleaved hop-1 slots).  For each owned slot the wave first aggregates inside
// itself: equal IDs within the slot (parallel edges) are merged into one entry with a
// multiplicity, so each distinct row receives one atomic per element.  Lanes then lie over 256
// consecutive bytes of a row (fsa_atomic_rows.hip.h).
#include "fsa_atomic_rows.hip.h"
#include "fsa_device.hip.h"
#include "fsa_internal.h"

#include <type_traits>

namespace fsa {

struct BwdParams {
    const void* grad_out; const void* grad_h1; const int32_t* ids1; const int32_t* ids2;
    void* grad_x; int64_t B; int64_t D; int k1, k2;
    const float* w1;                     // 1-hop weighted mean: [B,k1] weights of the sampled edges, else unused
    const int32_t* root_valid;           // 2-hop, nullable: [B], a negative entry switches root b off
    RowLanes lanes;                      // how the lanes of a wave lie over destination rows
};

// ---------------------------------------------------------------------------------------
// Element types of the incoming gradients (GT) and of grad_x (XG).  With an fp32 grad_x a
// lane owns one element of the row (EPL = 1), whatever the type of the incoming gradients, so
// that one wave instruction of global_atomic_add_f32 covers 256 contiguous bytes (pairs per
// lane would leave every instruction striding over twice as many cache lines: measured 1.7x
// slower).  With a 16-bit grad_x a lane owns two consecutive elements (EPL = 2; D is even)
// and adds the pair in ONE packed atomic (global_atomic_pk_add_bf16 / _f16), which halves the
// 64-byte segments per row -- their rate, not bandwidth, bounds this kernel.  Products and sums before the atomic are fp32; the value is rounded to the 16-bit
// type once (nearest-even) and every packed atomic rounds the running sum again.
// ---------------------------------------------------------------------------------------

// EPL consecutive gradient elements starting at element index `idx` (even when EPL == 2).
template <typename GT, int EPL>
__device__ __forceinline__ void load_grad(const void* base, int64_t idx, float (&g)[EPL]) {
    if constexpr (std::is_same<GT, g_f32>::value) {
        const float* p = static_cast<const float*>(base) + idx;
#pragma unroll
        for (int e = 0; e < EPL; ++e) g[e] = p[e];
    } else if constexpr (EPL == 1) {
        const uint16_t w = static_cast<const uint16_t*>(base)[idx];
        if constexpr (std::is_same<GT, g_bf16>::value) {
            g[0] = __uint_as_float((uint32_t)w << 16);
        } else {
            _Float16 h;
            __builtin_memcpy(&h, &w, sizeof h);
            g[0] = (float)h;
        }
    } else {
        const uint32_t w = *reinterpret_cast<const uint32_t*>(static_cast<const uint16_t*>(base) + idx);
        if constexpr (std::is_same<GT, g_bf16>::value) {
            g[0] = __uint_as_float(w << 16);
            g[1] = __uint_as_float(w & 0xffff0000u);
        } else {
            f16x2_t h;
            __builtin_memcpy(&h, &w, sizeof h);
            const f32x2_t f = __builtin_convertvector(h, f32x2_t);
            g[0] = f[0];
            g[1] = f[1];
        }
    }
}

// Merge equal IDs inside a segment of `k` lanes starting at seg_base.  Returns how many
// times this lane's ID occurs in the segment and whether this lane is its first occurrence.
__device__ __forceinline__ void merge_equal_ids(int id, int k, int li, int seg_base, int& mult,
                                                bool& first) {
    mult = 0;
    first = true;
    for (int m0 = 0; m0 < k; m0 += 8) {                 // eight shuffles in flight at a time
        int other[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) other[j] = __shfl(id, seg_base + m0 + j);
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            if (m0 + j < k && other[j] == id) { ++mult; if (m0 + j < li) first = false; }
        }
    }
}

// ---------------------------------------------------------------------------------------
// 1-hop backward.  A workgroup of nw (16) waves takes nw*spw consecutive seeds (wave w the
// seeds w, w+nw, ...).  Rows that many seeds of the workgroup share -- the hub rows of a skewed
// graph, which would otherwise serialise thousands of atomics on one L2 channel -- are first
// summed in LDS and reach grad_x with ONE atomic row-add per workgroup:
//   pass 1  every sampled ID claims the bucket at hash(id) of an LDS table or the one beside it (first
//           claimant wins; an ID that finds both taken stays on the direct path) and bumps its counter;
//   pass 2  buckets that count kHotMin IDs take an LDS row each; when there are fewer rows than such
//           buckets, they are handed out again to those that reach the lowest kHotMin * 2^i that no more do;
//   pass 3  per seed: equal IDs of the seed are merged (multiplicity), then each distinct row
//           receives grad_out[b,:] * mult/cnt -- into its LDS row if it has one, else
//           straight into grad_x with hardware atomics;
//   flush   LDS rows are added to grad_x.
// When no counter reaches kHotMin (uniform graphs) pass 2 and flush are skipped.
//
// A small call is bound by its chain of dependent steps, a large one by each wave's trips to memory,
// one seed after the other.  So a seed's IDs and the first tile of its gradient are requested
// together, for the first seed before the LDS is cleared and for every further one before the adds of
// the seed before it (a load behind atomics waits for them).  Backward alone, before and after: 1024 seeds x 10
// of 64 floats 7.1 -> 6.4 us, KG shape B=1024 10.1 -> 8.3, B=16384 31 -> 29; 64 seeds x 15 of 128 floats 9.5 -> 6.8;
// with the rows cut at their segments 4096 seeds x 15 of 300 floats 74 -> 63 us.  Asking for four seeds at a time
// was slower everywhere (B=4096 13 -> 16 us).
// ---------------------------------------------------------------------------------------
constexpr int kHotBuckets = 2048;
constexpr int kHotMin = 3;
constexpr int kHotRowsMax = 64;
constexpr int kHotLevels = 16;                                       // kHotMin * 2^15 exceeds any count (at most 2^15)
constexpr int kBwd1MaxSeeds = 32;                                    // seeds per wave: at most a bit for each of a lane's entries

__device__ __forceinline__ int hot_hash(int id) {
    return (int)(((uint32_t)id * 2654435761u) >> 21);              // 11 bits -> kHotBuckets
}

// The bucket that `id` owns, or -1.  An ID that finds its bucket taken has the one beside it.
__device__ __forceinline__ int hot_bucket(const int* tag, int id) {
    const int h = hot_hash(id);
    return tag[h] == id ? h : tag[h ^ 1] == id ? h ^ 1 : -1;
}

// LDS ints of the 1-hop kernel without the hot rows: tags and counters, levels, flags, node of each hot row, and
// per wave 64 rows with their factors.
FSA_HD inline int bwd1_fixed_ints(int nw) { return 2 * kHotBuckets + kHotLevels + 4 + kHotRowsMax + nw * 2 * kWave; }

template <typename GT, typename XG, bool WEIGHTED>
__global__ __launch_bounds__(1024) void bwd1_kernel(const BwdParams p, int spw, int hot_rows) {
    constexpr int EPL = Epl<GT, XG>::value;
    extern __shared__ __align__(16) int smem[];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int nw = blockDim.x >> 6;
    int* tag = smem;
    uint32_t* count = reinterpret_cast<uint32_t*>(tag + kHotBuckets);  // IDs | 1 + LDS row << 16
    int* level = tag + 2 * kHotBuckets;
    int* flags = level + kHotLevels;                                 // [0] any hot, [1] hot buckets, [2] rows of the second round
    int* row_node = flags + 4;
    int* rows = row_node + kHotRowsMax + wave * 2 * kWave;
    float* factor = reinterpret_cast<float*>(rows + kWave);
    float* hot = reinterpret_cast<float*>(smem + bwd1_fixed_ints(nw));
    const int64_t b0 = (int64_t)blockIdx.x * nw * spw;
    const RowLanes l = p.lanes;
    const int u0 = lane & ((1 << l.width_shift) - 1);

    // seed s of this wave: its IDs (lane < k1), their weights, the first tile of its gradient
    int next_id;
    float next_w = 0.0f;
    float next_g[EPL];
    auto request = [&](int s) {
        const int64_t b = b0 + wave + (int64_t)s * nw;
        const bool there = b < p.B && lane < p.k1;
        next_id = there ? p.ids1[b * p.k1 + lane] : -1;
        if constexpr (WEIGHTED) next_w = there ? p.w1[b * p.k1 + lane] : 0.0f;
        if (b < p.B) load_grad<GT, EPL>(p.grad_out, b * p.D + (int64_t)(u0 < l.units ? u0 : 0) * EPL, next_g);
    };
#pragma unroll
    for (int c = 0; c < EPL; ++c) next_g[c] = 0.0f;
    request(0);

    bool any_hot = false;
    int n_rows = 0;
    if (hot_rows > 0) {
        for (int i = threadIdx.x; i < kHotBuckets; i += blockDim.x) { tag[i] = -1; count[i] = 0; }
        if (threadIdx.x < kHotLevels + 4) level[threadIdx.x] = 0;    // and the flags behind the levels
        __syncthreads();
        // the workgroup's IDs: with one seed per wave those that are here already, else all of them in order
        const int64_t first_entry = b0 * p.k1;
        const int n_ent = (int)(((b0 + (int64_t)nw * spw < p.B ? b0 + (int64_t)nw * spw : p.B) - b0) * p.k1);
        const int turns = spw == 1 ? 1 : (n_ent + (int)blockDim.x - 1) / (int)blockDim.x;
        auto entry = [&](int i) {
            if (spw == 1) return next_id;
            const int e = i * (int)blockDim.x + (int)threadIdx.x;
            return e < n_ent ? p.ids1[first_entry + e] : -1;
        };
        uint32_t owner = 0u;                                         // bit i: this lane claimed a bucket for its entry i
        bool saw_hot = false;
        for (int i = 0; i < turns; ++i) {
            const int id = entry(i);
            if (id >= 0) {
                int h = hot_hash(id);
                int was = atomicCAS(&tag[h], -1, id);
                if (was != -1 && was != id) { h ^= 1; was = atomicCAS(&tag[h], -1, id); }
                if (was == -1) owner |= 1u << i;
                if (was == -1 || was == id) saw_hot = (atomicAdd(&count[h], 1u) + 1 >= kHotMin) || saw_hot;
            }
        }
        if (saw_hot) flags[0] = 1;
        __syncthreads();
        any_hot = flags[0] != 0;                                     // workgroup-uniform
        if (any_hot) {
            for (int i = 0; i < turns; ++i) {
                if (!((owner >> i) & 1u)) continue;
                const int id = entry(i);
                const int h = hot_bucket(tag, id);
                const uint32_t c = count[h];
                if (c < kHotMin) continue;
                const int r = atomicAdd(&flags[1], 1);
                if (r < hot_rows) { row_node[r] = id; count[h] = c | (uint32_t)(r + 1) << 16; }
            }
            for (int i = threadIdx.x; i < hot_rows * (int)p.D; i += blockDim.x) hot[i] = 0.0f;
            __syncthreads();
            n_rows = flags[1];
            if (n_rows > hot_rows) {                                 // workgroup-uniform
                for (int i = 0; i < turns; ++i) {
                    if (!((owner >> i) & 1u)) continue;
                    const uint32_t c = count[hot_bucket(tag, entry(i))] & 0xffffu;
                    if (c >= kHotMin) atomicAdd(&level[31 - __clz(c / kHotMin)], 1);
                }
                __syncthreads();
                int at = kHotLevels, over = 0;                       // buckets of level `at` and above
                while (at > 0 && over + level[at - 1] <= hot_rows) over += level[--at];
                n_rows = over;
                for (int i = 0; i < turns; ++i) {
                    if (!((owner >> i) & 1u)) continue;
                    const int id = entry(i);
                    const int h = hot_bucket(tag, id);
                    uint32_t c = count[h] & 0xffffu;
                    if (c >= (uint32_t)kHotMin << at) {
                        const int r = atomicAdd(&flags[2], 1);
                        row_node[r] = id;
                        c |= (uint32_t)(r + 1) << 16;
                    }
                    count[h] = c;
                }
                __syncthreads();
            }
        }
    }

    // pass 3: one seed at a time per wave
    for (int s = 0; s < spw; ++s) {
        const int64_t b = b0 + wave + (int64_t)s * nw;
        if (b >= p.B) break;                                         // wave-uniform
        const int id = next_id;
        // share of the seed's gradient that this lane's row receives: multiplicity / count, or,
        // for the weighted mean, the summed weight of its occurrences / the seed's weight sum
        // (a seed whose weights sum to zero contributes nothing)
        float share;
        bool first;
        bool live_seed = true;
        if constexpr (WEIGHTED) {
            const float w = id >= 0 ? next_w : 0.0f;
            float total = w;
            for (int off = 1; off < kWave; off <<= 1) total += __shfl_xor(total, off);
            float wsum;
            merge_equal_ids_w(id, w, p.k1, lane, 0, wsum, first);
            live_seed = total > 0.0f;
            share = live_seed ? wsum / total : 0.0f;
        } else {
            const int cnt = __popcll(__ballot(id >= 0));
            int mult;
            merge_equal_ids(id, p.k1, lane, 0, mult, first);
            share = (float)mult / (float)cnt;
        }
        // the list: rows of grad_x from the front, LDS rows from the back
        const bool keep = id >= 0 && first && live_seed;
        int to = id;
        if (any_hot && keep) {
            const int h = hot_bucket(tag, id);
            if (h >= 0 && count[h] >> 16) to = -(int)(count[h] >> 16);  // ~LDS row
        }
        const uint64_t direct = __ballot(keep && to >= 0), shared = __ballot(keep && to < 0);
        const int n = __popcll(direct), n_shared = __popcll(shared);
        if (keep) {
            const int slot = to >= 0 ? __popcll(direct & lanemask_lt(lane)) : kWave - 1 - __popcll(shared & lanemask_lt(lane));
            rows[slot] = to;
            factor[slot] = share;
        }
        float held[EPL];
#pragma unroll
        for (int c = 0; c < EPL; ++c) held[c] = next_g[c];
        if (s + 1 < spw) request(s + 1);
        __builtin_amdgcn_wave_barrier();
        add_scaled_rows<XG, EPL>(p.grad_x, l, rows, factor, n, 0, 1, lane, [&](int64_t d, float (&g)[EPL]) {
            if (d < kWave * EPL) {
#pragma unroll
                for (int c = 0; c < EPL; ++c) g[c] = held[c];
            } else {
                load_grad<GT, EPL>(p.grad_out, b * p.D + d, g);
            }
            arrived(g);                                              // (and after these, for the atomics on rows)
            for (int e = kWave - n_shared; e < kWave; ++e) {         // (narrow rows: for the first group of lanes)
                if (lane >> l.width_shift) break;
                float* at = hot + ~rows[e] * (int)p.D + d;
#pragma unroll
                for (int c = 0; c < EPL; ++c) atomicAdd(at + c, g[c] * factor[e]);
            }
        });
        __builtin_amdgcn_wave_barrier();
    }

    if (any_hot) {                                                   // workgroup-uniform
        __syncthreads();
        char* const base = static_cast<char*>(p.grad_x);
        for (int r = wave; r < n_rows; r += nw) {
            const int64_t row = row_node[r];
            const int shift = l.base >= 0 ? (int)(((uint32_t)l.base + (uint32_t)row * (uint32_t)l.units) & (kSegment - 1)) : 0;
            for (int d = lane - shift; d < l.units; d += kWave) {    // from the start of the row's first segment
                if (d < 0) continue;
                float v[EPL];
#pragma unroll
                for (int c = 0; c < EPL; ++c) v[c] = hot[r * (int)p.D + d * EPL + c];
                atomic_add_row<XG, EPL>(base + (row * l.units + d) * 4, v);
            }
        }
    }
}

template <typename GT, typename XG>
__global__ __launch_bounds__(512) void bwd2_kernel(const BwdParams p) {
    constexpr int EPL = Epl<GT, XG>::value;
    extern __shared__ int smem[];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int nw = blockDim.x >> 6;
    const int64_t b = blockIdx.x;
    const int k1 = p.k1, k2 = p.k2;
    const int nq_max = (k1 + nw - 1) / nw;
    // per wave: leaf rows, multiplicities, per-slot total count and distinct count
    const int per_wave = 2 * nq_max * k2 + 2 * nq_max;
    int* leaf = smem + wave * per_wave;
    float* mul = reinterpret_cast<float*>(leaf + nq_max * k2);
    int* cnt2 = leaf + 2 * nq_max * k2;
    int* uniq = cnt2 + nq_max;
    int* live_slots = smem + nw * per_wave;

    if (p.root_valid && p.root_valid[b] < 0) return;    // workgroup-uniform, before any barrier
    const int u_mine = lane < k1 ? p.ids1[b * k1 + lane] : -1;
    const int nq = wave < k1 ? (k1 - wave + nw - 1) / nw : 0;
    const int spw = kWave / k2;
    const int g = lane / k2;
    const int li = lane - g * k2;
    for (int q0 = 0; q0 < nq; q0 += spw) {              // wave-uniform trip count
        const int q = q0 + g;
        const bool valid = g < spw && q < nq;
        const int j = wave + q * nw;
        const int u = __shfl(u_mine, valid ? j : 0);
        const int seg_base = valid ? g * k2 : 0;
        int id = valid ? p.ids2[(b * k1 + j) * k2 + li] : -1;         // travels with ids1
        if (u < 0) id = -1;
        const uint64_t seg = (k2 == 64 ? ~0ull : ((1ull << k2) - 1ull)) << seg_base;
        const int c2 = __popcll(__ballot(id >= 0) & seg);
        int mult; bool first;
        merge_equal_ids(id, k2, li, seg_base, mult, first);
        const bool keep = id >= 0 && first;
        const uint64_t kept = __ballot(keep) & seg;
        if (keep) {
            const int slot = __popcll(kept & lanemask_lt(lane));
            leaf[q * k2 + slot] = id;
            mul[q * k2 + slot] = (float)mult;
        }
        if (valid && li == 0) { cnt2[q] = c2; uniq[q] = __popcll(kept); }
    }
    __builtin_amdgcn_wave_barrier();
    {
        const int mine = lane < nq ? cnt2[lane] : 0;
        const int n_live = __popcll(__ballot(mine > 0));
        if (lane == 0) live_slots[wave] = n_live;
    }
    __syncthreads();
    int c1 = 0;
    for (int w = 0; w < nw; ++w) c1 += live_slots[w];
    if (c1 == 0) return;
    const float fc1 = (float)c1;

    for (int q = 0; q < nq; ++q) {
        const int c = cnt2[q];
        if (c == 0) continue;
        const int64_t j = wave + q * nw;
        const float fc = (float)c;
        add_scaled_rows<XG, EPL>(p.grad_x, p.lanes, leaf + q * k2, mul + q * k2, uniq[q], blockIdx.y, gridDim.y, lane, [&](int64_t d, float (&gsum)[EPL]) {
            load_grad<GT, EPL>(p.grad_out, b * p.D + d, gsum);
#pragma unroll
            for (int c = 0; c < EPL; ++c) gsum[c] = gsum[c] / fc1;
            if (p.grad_h1) {
                float gh[EPL];
                load_grad<GT, EPL>(p.grad_h1, (b * k1 + j) * p.D + d, gh);
#pragma unroll
                for (int c = 0; c < EPL; ++c) gsum[c] += gh[c];
            }
#pragma unroll
            for (int c = 0; c < EPL; ++c) gsum[c] = gsum[c] / fc;
        });
    }
}

// ---------------------------------------------------------------------------------------
// Three-hop backward, first step: the gradient that reaches each hop-1 slot's nested mean.
//   work[b,j,:] = (slot j took part ? grad_out[b,:] / c_b : 0) + grad_h1[b,j,:]
// where slot j took part iff ids1[b,j] >= 0 and some i has ids2[b,j,i] >= 0 and a non-negative
// ids3[b,j,i,:], and c_b counts such slots.
// One workgroup per root; the two-hop backward then runs over the B*k1 slots as its roots.  Bound by the
// IDs' latency, then by the rows written: all threads look at IDs side by side, four of each level in
// flight per thread, where a wave that went through the slots one after the other waited once per slot
// (products, 15/10/5, B=1024: 21.1 -> 5.5 us).
// ---------------------------------------------------------------------------------------
template <int VE>
__global__ __launch_bounds__(256) void deep_grad_kernel(const float* __restrict__ grad_out,
                                                        const float* __restrict__ grad_h1,
                                                        const int32_t* __restrict__ ids1,
                                                        const int32_t* __restrict__ ids2,
                                                        const int32_t* __restrict__ ids3, float* __restrict__ work,
                                                        int k1, int k2, int k3, int64_t D) {
    using Row = Chunk<f32_t, VE * 4>;
    using Raw = typename Row::Raw;
    __shared__ int took_part[64];                                    // k1 <= 64
    const int tid = threadIdx.x;
    const int64_t b = blockIdx.x;
    const int per_slot = k2 * k3, n_ent = k1 * per_slot;
    const int32_t* q1 = ids1 + b * k1;
    const int32_t* q2 = ids2 + b * k1 * k2;
    const int32_t* q3 = ids3 + b * n_ent;
    if (tid < 64) took_part[tid] = 0;
    __syncthreads();
    for (int e0 = tid; e0 < n_ent; e0 += 4 * 256) {
        int v[4], slot[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const int e = e0 + u * 256 < n_ent ? e0 + u * 256 : e0;  // past the end: the first one again
            slot[u] = e / per_slot;
            v[u] = q3[e] | q2[e / k3] | q1[slot[u]];                 // negative if any of the three is
        }
#pragma unroll
        for (int u = 0; u < 4; ++u) if (v[u] >= 0) took_part[slot[u]] = 1;
    }
    __syncthreads();
    const uint64_t part = __ballot(took_part[tid & 63] != 0);        // bit j: slot j took part
    const int c = __popcll(part);
    const float inv = c > 0 ? 1.0f / (float)c : 0.0f;
    const int chunks = (int)(D / VE);
    const int64_t row0 = b * k1 * D;
    for (int64_t i = tid; i < (int64_t)k1 * chunks; i += 256) {      // the slots' rows lie one after the other
        const int j = (int)(i / chunks);
        float v[VE], g[VE];
#pragma unroll
        for (int k = 0; k < VE; ++k) { v[k] = 0.0f; g[k] = 0.0f; }
        if ((part >> j) & 1ull) {
            Row::add(g, *reinterpret_cast<const Raw*>(grad_out + b * D + (i - (int64_t)j * chunks) * VE));
#pragma unroll
            for (int k = 0; k < VE; ++k) v[k] = g[k] * inv;
        }
        if (grad_h1) Row::add(v, *reinterpret_cast<const Raw*>(grad_h1 + row0 + i * VE));
        *reinterpret_cast<Raw*>(work + row0 + i * VE) = Row::pack(v);
    }
}

hipError_t launch_deep_grad(const float* grad_out, const float* grad_h1, const int32_t* ids1, const int32_t* ids2,
                            const int32_t* ids3, float* work, int64_t B, int k1, int k2, int k3, int64_t D,
                            hipStream_t stream) {
    auto al = [](const void* q) { return reinterpret_cast<uintptr_t>(q) % 16 == 0; };
    const bool quads = D % 4 == 0 && al(grad_out) && al(grad_h1) && al(work);
    for (int64_t b = 0; b < B; b += kMostRoots) {
        const dim3 grid((unsigned)(B - b < kMostRoots ? B - b : kMostRoots)), block(256);
        const float* go = grad_out + b * D;
        const float* gh = grad_h1 ? grad_h1 + b * k1 * D : nullptr;
        const int32_t* q1 = ids1 + b * k1;
        const int32_t* q2 = ids2 + b * k1 * k2;
        const int32_t* q3 = ids3 + b * k1 * k2 * k3;
        float* w = work + b * k1 * D;
        if (quads) hipLaunchKernelGGL(deep_grad_kernel<4>, grid, block, 0, stream, go, gh, q1, q2, q3, w, k1, k2, k3, D);
        else       hipLaunchKernelGGL(deep_grad_kernel<1>, grid, block, 0, stream, go, gh, q1, q2, q3, w, k1, k2, k3, D);
    }
    return hipGetLastError();
}

template <typename GT, typename XG, bool WEIGHTED>
static hipError_t launch_bwd1(const BwdArgs& a, const BwdParams& p, hipStream_t stream) {
    // The more seeds a workgroup sees the fewer atomic row-adds reach a hub row, and 16 waves work through them
    // side by side; a small batch is spread over the CUs in workgroups of 4 or 8 waves instead.  Seeds per wave
    // grow with the batch so that the launch keeps a few hundred workgroups.  Measured, KG shape: B=4096
    // 20.4 / 14.7 us with 4 / 16 waves, B=1024 8.3 / 8.0; product graph, 64 seeds of 300 floats 12.5 / 13.7.
    const int forced_spw = tune_int("FSA_BWD1_SEEDS_PER_WAVE", 0);
    const int forced_nw = tune_int("FSA_BWD1_WAVES", 0);
    int nw = 4;
    while (nw < 16 && a.B > (int64_t)nw * 256) nw *= 2;
    if (forced_nw >= 1 && forced_nw <= 16) nw = forced_nw;
    int spw = 1;
    while (spw < 16 && a.B / ((int64_t)nw * spw * 2) >= 256) spw *= 2;
    if (forced_spw >= 1 && forced_spw <= kBwd1MaxSeeds) spw = forced_spw;
    // LDS: the fixed part (hash tables, per-wave strips) plus as many fp32 rows as fit in 64 KB
    const size_t lds_fixed = sizeof(int) * bwd1_fixed_ints(nw);
    int hot_rows = (int)((65536 - lds_fixed) / (sizeof(float) * (size_t)a.D));
    if (hot_rows > kHotRowsMax) hot_rows = kHotRowsMax;
    if (tune_int("FSA_BWD1_NO_HOT", 0)) hot_rows = 0;
    const unsigned grid = (unsigned)((a.B + nw * spw - 1) / (nw * spw));
    const size_t lds = lds_fixed + sizeof(float) * (size_t)hot_rows * a.D;
    BwdParams q = p;
    q.lanes = row_lanes(a.grad_x, a.D / Epl<GT, XG>::value);
    hipLaunchKernelGGL((bwd1_kernel<GT, XG, WEIGHTED>), dim3(grid), dim3(nw * kWave), lds, stream, q, spw, hot_rows);
    return hipGetLastError();
}

template <typename GT, typename XG>
static hipError_t launch_backward_typed(const BwdArgs& a, const BwdParams& p, hipStream_t stream) {
    if (!a.ids2) {
        return launch_bwd1<GT, XG, false>(a, p, stream);
    } else {
        const int forced = tune_int("FSA_BWD2_WAVES", 0);
        int nw = (forced >= 1 && forced <= 8) ? forced : (a.k1 < 8 ? a.k1 : 8);
        const int nq_max = (a.k1 + nw - 1) / nw;
        const size_t lds = sizeof(int) * ((size_t)nw * (2 * nq_max * a.k2 + 2 * nq_max) + nw);
        BwdParams q = p;
        q.lanes = row_lanes(a.grad_x, a.D / Epl<GT, XG>::value);
        hipLaunchKernelGGL((bwd2_kernel<GT, XG>), dim3((unsigned)a.B, backward_parts(a.B, a.k2, rows_an_instruction(q.lanes))), dim3(nw * kWave), lds, stream, q);
    }
    return hipGetLastError();
}

hipError_t launch_backward(const BwdArgs& a, hipStream_t stream) {
    if (const int64_t most = most_at_a_time(a.ids2 ? 2 : 1); a.B > most) {
        for (int64_t b = 0; b < a.B; b += most)
            if (hipError_t e = launch_backward(backward_part(a, b, a.B - b < most ? a.B - b : most), stream)) return e;
        return hipSuccess;
    }
    BwdParams p;
    p.grad_out = a.grad_out; p.grad_h1 = a.grad_h1; p.ids1 = a.ids1; p.ids2 = a.ids2;
    p.grad_x = a.grad_x; p.B = a.B; p.D = a.D; p.k1 = a.k1; p.k2 = a.k2; p.root_valid = a.root_valid; p.w1 = nullptr;
    // kinds: 0 fp32, 1 bfloat16, 2 fp16.  A 16-bit grad_x takes gradients of its own type or fp32.
    switch (a.grad_kind * 3 + a.grad_x_kind) {
        case 0 * 3 + 0: return launch_backward_typed<g_f32, g_f32>(a, p, stream);
        case 1 * 3 + 0: return launch_backward_typed<g_bf16, g_f32>(a, p, stream);
        case 2 * 3 + 0: return launch_backward_typed<g_f16, g_f32>(a, p, stream);
        case 0 * 3 + 1: return launch_backward_typed<g_f32, g_bf16>(a, p, stream);
        case 1 * 3 + 1: return launch_backward_typed<g_bf16, g_bf16>(a, p, stream);
        case 0 * 3 + 2: return launch_backward_typed<g_f32, g_f16>(a, p, stream);
        case 2 * 3 + 2: return launch_backward_typed<g_f16, g_f16>(a, p, stream);
        default: return hipErrorInvalidValue;
    }
}

// 1-hop weighted-mean backward (fp32): the 1-hop kernel with weight shares.
hipError_t launch_backward1_weighted(const BwdArgs& a, const float* w1, hipStream_t stream) {
    BwdParams p;
    p.grad_out = a.grad_out; p.grad_h1 = nullptr; p.ids1 = a.ids1; p.ids2 = nullptr;
    p.grad_x = a.grad_x; p.B = a.B; p.D = a.D; p.k1 = a.k1; p.k2 = 0; p.root_valid = nullptr; p.w1 = w1;
    return launch_bwd1<g_f32, g_f32, true>(a, p, stream);
}

}  // namespace fsa

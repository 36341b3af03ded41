// Backward that gives every destination row one owner, for calls with enough row updates that are
// handed a workspace: such a call may not share grad_x with other work while it runs.  The paper describes no backward kernel (Sec. 3.3 "Reproducibility" only asks that the
// saved IDs are replayed).
//
// Why: a hardware atomic is one 4-byte operation per L2 channel and clock (about 1.1 TB/s of row
// payload however the rows lie), and in the atomic backward every sampled leaf costs a whole row of
// them.  A plain read-add-write of a random row runs at 1.8-2.2 TB/s of payload (147,000 rows of
// 400 bytes: 32 us against 60 us of atomics), so a row is updated once per call, by one wave, with
// ordinary loads and stores, wherever it can be known that nobody else touches it.
//
// Three launches on the caller's stream, all state in the caller's workspace:
//   clear   zero the bucket counters (a fill kernel: a memset node must not end up in a captured
//           graph);
//   mark    every live leaf slot appends (leaf slot, row) to the bucket its row hashes to, and every
//           slot gets its two coefficients;
//   add     every live leaf slot looks its bucket up.  The smallest leaf slot of a row owns the row:
//           its wave adds the gradients of all leaf slots of the row, in ascending order, to the old
//           row and writes it back; the others do nothing.  A row's leaf slots all hash to one
//           bucket, so two owners never meet on a row.  Rows named more than kRowMax times, and rows
//           of a bucket that was asked for more than it holds (hubs), are left to atomics by all of
//           their leaf slots, so plain and atomic updates never meet on a row either.  Without such
//           rows the result is bit-reproducible.
//
// Most rows are sampled once in a batch (69 % of the leaves of a 1024-seed batch on the product
// graph, 83 % of a 4096-seed batch on the citation graph) and need no sum.
#include "fsa_device.hip.h"
#include "fsa_internal.h"

namespace fsa {

constexpr int kBucketCap = 64;            // entries a bucket holds
constexpr int kBucketFill = 4;            // leaf slots per bucket: an owner sees its bucket in one go of 8 entries, and
                                          // 64 against 4 leave room for rows sampled more than once
constexpr int kRowMax = 16;               // leaf slots of a row that its owner adds up, one after the other
constexpr int kTile = 1024;               // leaf slots a mark workgroup takes at a time
constexpr int kTileThreads = 256;
constexpr int kTilePer = kTile / kTileThreads;
constexpr int kHash = 1024;               // LDS table that merges the appends of rows shared inside a tile
constexpr int kList = 128;                // contributions a wave lists at a time
static_assert(kList >= kRowMax && kList == 2 * kWave, "one row always fits; two ballots cover the list");
static_assert(kBucketCap % 8 == 0, "a bucket is read 8 entries at a time");

struct OwnedParams {
    const char* grad_out; const char* grad_h1;
    const int32_t* ids1;                  // [B,k1]
    const int32_t* ids2;                  // [B,k1,k2] leaf slots
    const int32_t* root_valid;            // nullable: [B], a negative entry switches root b off
    const float* w1; const float* w2;     // weighted mean only
    char* grad_x; int64_t B; int64_t D;
    int k1, k2, n_leaf;
    int chunks, sub, sub_shift, tiles;    // row chunks of VE elements, lanes over a row, passes over a row
    int roots_per_tile;
    int* cnt;                             // [n_buckets] entries asked of each bucket (may exceed the capacity)
    float2* coef;                         // [B*k1] per slot: factor of grad_out, and 1/rows (weighted: weight sum);
                                          // y <= 0: the slot has no part
    uint2* entries;                       // [n_buckets][kBucketCap] (leaf slot, row)
    uint32_t n_buckets;
    int lpw;                              // leaf slots per wave of the add kernel
};

__global__ __launch_bounds__(256) void owned_clear_kernel(int4* cnt, int n) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) cnt[i] = make_int4(0, 0, 0, 0);
}

__device__ __forceinline__ uint32_t row_hash(int row) { return (uint32_t)row * 2654435761u; }

// A workgroup takes roots_per_tile whole roots (at most kTile leaf slots, or one root of up to 4096).
// Leaf slots of a tile that name the same row are merged in LDS first: one returning atomic per
// distinct row and tile, because atomics on one address go through at one per 11 ns (4000 of them:
// 47 us) and a hub row of a skewed graph is named by every tenth leaf slot.  Bound by its chain of
// dependent steps, so the loads of a thread's four leaf slots go out together.
template <bool WEIGHTED>
__global__ __launch_bounds__(kTileThreads) void owned_mark_kernel(const OwnedParams p) {
    __shared__ int slot_cnt[kTile];                                   // rows of each slot (weighted: bits of the weight sum)
    __shared__ float root_sum[kTile];                                 // per root: slots that take part (weighted: their weight)
    __shared__ int t_row[kHash], t_cnt[kHash], t_base[kHash];
    const int tid = threadIdx.x;
    const int k1 = p.k1, k2 = p.k2;
    const int64_t b0 = (int64_t)blockIdx.x * p.roots_per_tile;
    const int n_roots = (int)(p.B - b0 < p.roots_per_tile ? p.B - b0 : p.roots_per_tile);
    const int n_slots = n_roots * k1;                                 // <= kTile
    const int n_ent = n_slots * k2;
    const int slot0 = (int)(b0 * k1);
    const int e0 = slot0 * k2;

    for (int s = tid; s < n_slots; s += kTileThreads) {
        if constexpr (WEIGHTED) {
            float tot = 0.0f;                                         // in slot order
            const bool on = p.ids1[slot0 + s] >= 0;
            for (int i = 0; i < k2; ++i) {
                const int e = (slot0 + s) * k2 + i;
                const float w = p.w2[e];
                if (p.ids2[e] >= 0 && on) tot += w;
            }
            slot_cnt[s] = __float_as_int(tot);
        } else {
            slot_cnt[s] = 0;
        }
    }
    for (int r = tid; r < n_roots; r += kTileThreads) root_sum[r] = 0.0f;
    for (int c0 = 0; c0 < n_ent; c0 += kTile) {                       // one pass unless a root has more than kTile
        int id[kTilePer], pos[kTilePer], base[kTilePer], slot[kTilePer];
        bool member[kTilePer];
#pragma unroll
        for (int u = 0; u < kTilePer; ++u) {
            const int i = c0 + u * kTileThreads + tid;
            const int at = i < n_ent ? i : n_ent - 1;                 // past the end: a leaf slot of the tile again, not used
            slot[u] = at / k2;
            id[u] = p.ids2[e0 + at];
            if constexpr (!WEIGHTED) {
                int on = p.ids1[slot0 + slot[u]];
                if (p.root_valid) on |= p.root_valid[b0 + slot[u] / k1];      // either negative: the slot has no part
                member[u] = on >= 0;
            }
        }
        for (int i = tid; i < kHash; i += kTileThreads) { t_row[i] = -1; t_cnt[i] = 0; }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kTilePer; ++u) {
            if constexpr (WEIGHTED) member[u] = __int_as_float(slot_cnt[slot[u]]) > 0.0f;
            if (!member[u] || c0 + u * kTileThreads + tid >= n_ent) id[u] = -1;
            member[u] = false;
            pos[u] = 0;
            if (id[u] >= 0) {
                if constexpr (!WEIGHTED) atomicAdd(&slot_cnt[slot[u]], 1);
                const int h = (int)(row_hash(id[u]) >> 22);           // 10 bits -> kHash
                const int was = atomicCAS(&t_row[h], -1, id[u]);
                member[u] = was == -1 || was == id[u];
                if (member[u]) pos[u] = atomicAdd(&t_cnt[h], 1);
            }
        }
        __syncthreads();
        // one append per distinct row (its first leaf slot here), or per leaf slot that found its LDS place taken
#pragma unroll
        for (int u = 0; u < kTilePer; ++u) {
            base[u] = 0;
            if (id[u] >= 0 && pos[u] == 0) {
                const uint32_t h = row_hash(id[u]);
                base[u] = atomicAdd(&p.cnt[__umulhi(h, p.n_buckets)], member[u] ? t_cnt[h >> 22] : 1);
            }
        }
#pragma unroll
        for (int u = 0; u < kTilePer; ++u) {
            if (member[u] && pos[u] == 0) t_base[row_hash(id[u]) >> 22] = base[u];
        }
        __syncthreads();
#pragma unroll
        for (int u = 0; u < kTilePer; ++u) {
            if (id[u] >= 0) {
                const uint32_t h = row_hash(id[u]);
                const int at = member[u] ? t_base[h >> 22] + pos[u] : base[u];
                if (at < kBucketCap)
                    p.entries[(size_t)__umulhi(h, p.n_buckets) * kBucketCap + at] =
                        make_uint2((uint32_t)(e0 + c0 + u * kTileThreads + tid), (uint32_t)id[u]);
            }
        }
        __syncthreads();                                              // t_* are reset by the next pass
    }

    if constexpr (WEIGHTED) {
        for (int r = tid; r < n_roots; r += kTileThreads) {
            float outer = 0.0f;
            for (int j = 0; j < k1; ++j)
                if (__int_as_float(slot_cnt[r * k1 + j]) > 0.0f) outer += p.w1[slot0 + r * k1 + j];
            root_sum[r] = outer;
        }
        __syncthreads();
        for (int s = tid; s < n_slots; s += kTileThreads) {
            const float outer = root_sum[s / k1];
            p.coef[slot0 + s] = make_float2(outer > 0.0f ? p.w1[slot0 + s] / outer : 0.0f, __int_as_float(slot_cnt[s]));
        }
    } else {
        for (int s = tid; s < n_slots; s += kTileThreads) {
            if (slot_cnt[s] > 0) atomicAdd(&root_sum[s / k1], 1.0f);  // small whole numbers: exact in any order
        }
        __syncthreads();
        for (int s = tid; s < n_slots; s += kTileThreads) {
            const int c2 = slot_cnt[s];
            p.coef[slot0 + s] = c2 > 0 ? make_float2(1.0f / root_sum[s / k1], 1.0f / (float)c2) : make_float2(0.0f, 0.0f);
        }
    }
}

template <typename T> constexpr int kElemBytes = (int)sizeof(T);

// grad_x[idx .. idx+EPL) += v by hardware atomics without a return value (EPL 1: fp32, 2: a packed pair)
template <typename XT, int EPL>
__device__ __forceinline__ void add_elements(char* base, int64_t idx, const float (&v)[EPL]) {
    if constexpr (EPL == 1) {
        unsafeAtomicAdd(reinterpret_cast<float*>(base) + idx, v[0]);
    } else {
        typedef float f32x2 __attribute__((ext_vector_type(2)));
        const f32x2 f = {v[0], v[1]};
        uint16_t* at = reinterpret_cast<uint16_t*>(base) + idx;
        if constexpr (__is_same(XT, bf16_t)) {
            typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_global_atomic_fadd_v2bf16(reinterpret_cast<bf16x2*>(at), __builtin_convertvector(f, bf16x2));
        } else {
            typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
            __builtin_amdgcn_global_atomic_fadd_v2f16(reinterpret_cast<f16x2*>(at), __builtin_convertvector(f, f16x2));
        }
    }
}

// A wave's list of contributions to the rows it owns, in LDS, row by row, ascending leaf slots.
struct WaveStrip {
    longlong2 at[kList];                  // byte offsets in grad_x (bit 63: the row's last contribution) and grad_out
    int4 more[kList];                     // byte offset in grad_h1, bits of the two factors
    int leaf[kList];                      // leaf slots, those of a row as its bucket has them
    int lane[kList];                      // the lane that owns the row
};

// A lane per leaf slot looks its row up, lpw leaf slots per wave; then sub-groups of lanes walk the
// list with U contributions in flight each.  Bound by the rows' traffic (old row in, new row out) after
// a chain of four dependent look-ups (one trip fewer, with the counter beside its entries, changes
// nothing).  Three contributions in flight: products, forward and backward, 84 / 82 / 81 / 84 us with
// 1 / 2 / 3 / 4; 800-byte rows 118 / 113 / 108 / 107 us; three hops 323 / 318 / 320 / 327 us.  The lanes of a leaf slot's own gradient rows hit the wave's cache lines, because
// consecutive leaf slots share them: a pass over the rows in table order would read them once more per
// leaf.
template <typename GT, typename XT, int VE, int U, bool H1, bool WEIGHTED>
__global__ __launch_bounds__(256) void owned_add_kernel(const OwnedParams p) {
    using G = Chunk<GT, VE * kElemBytes<GT>>;
    using X = Chunk<XT, VE * kElemBytes<XT>>;
    using GRaw = typename G::Raw;
    using XRaw = typename X::Raw;
    __shared__ WaveStrip strips[4];
    const int lane = threadIdx.x & 63;
    WaveStrip& st = strips[threadIdx.x >> 6];
    const int64_t first = ((int64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * p.lpw;
    if (first >= p.n_leaf) return;                                    // wave-uniform; no block barrier below
    const int k1 = p.k1, k2 = p.k2;

    const bool valid = lane < p.lpw && first + lane < p.n_leaf;
    const int e = valid ? (int)first + lane : (int)first;
    const int id = p.ids2[e];
    const int slot = e / k2;
    const float2 cf = p.coef[slot];
    const bool live = valid && id >= 0 && cf.y > 0.0f;
    if (!__any(live)) return;                                         // wave-uniform
    const uint32_t bucket = live ? __umulhi(row_hash(id), p.n_buckets) : 0u;
    const uint4* const two = reinterpret_cast<const uint4*>(p.entries + (size_t)bucket * kBucketCap);
    const int asked = p.cnt[bucket];
    bool hub = live && asked > kBucketCap;
    const int n_ent = live && !hub ? asked : 0;
    int same = 0;                                                     // other leaf slots of the row
    bool lowest = true;
    if (n_ent > 1) {
        for (int j = 0; j < n_ent; j += 8) {
            uint4 t[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) t[k] = two[(j >> 1) + k];
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const bool h0 = j + 2 * k < n_ent && t[k].y == (uint32_t)id;
                const bool h1 = j + 2 * k + 1 < n_ent && t[k].w == (uint32_t)id;
                same += (int)(h0 && t[k].x != (uint32_t)e) + (int)(h1 && t[k].z != (uint32_t)e);
                lowest = lowest && !(h0 && t[k].x < (uint32_t)e) && !(h1 && t[k].z < (uint32_t)e);
            }
        }
    }
    hub = hub || same >= kRowMax;                                     // all leaf slots of the row see the same number
    bool todo = live && !hub && lowest;

    // hub rows: atomics, the wave's leaf slots of one row summed first
    uint64_t hubs = __ballot(hub);
    if (hubs) {                                                       // wave-uniform
        float f = cf.y;
        if constexpr (WEIGHTED) f = hub ? p.w2[e] / cf.y : 0.0f;
        while (hubs) {
            const int row = __builtin_amdgcn_readlane(id, __builtin_ctzll(hubs));
            const uint64_t mine = __ballot(hub && id == row);
            hubs &= ~mine;
            constexpr int EPL = __is_same(XT, f32_t) ? 1 : 2;
            using GE = Chunk<GT, EPL * kElemBytes<GT>>;
            for (int64_t d = (int64_t)lane * EPL; d < p.D; d += kWave * EPL) {
                float v[EPL] = {};
                for (uint64_t m = mine; m; m &= m - 1) {
                    const int l = __builtin_ctzll(m);
                    const int s = __builtin_amdgcn_readlane(slot, l);
                    const float a = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(cf.x), l));
                    const float w = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(f), l));
                    float t[EPL] = {};
                    GE::fma(t, *reinterpret_cast<const typename GE::Raw*>(p.grad_out + ((int64_t)(s / k1) * p.D + d) * kElemBytes<GT>), a);
                    if constexpr (H1) GE::add(t, *reinterpret_cast<const typename GE::Raw*>(p.grad_h1 + ((int64_t)s * p.D + d) * kElemBytes<GT>));
#pragma unroll
                    for (int c = 0; c < EPL; ++c) v[c] = fmaf(w, t[c], v[c]);
                }
                add_elements<XT, EPL>(p.grad_x, (int64_t)row * p.D + d, v);
            }
        }
    }

    // owned rows, in rounds of as many as the list can take (nearly always one)
    const int sub = p.sub;
    const int sg = lane >> p.sub_shift;
    const int sl = lane & (sub - 1);
    const int nsg = kWave >> p.sub_shift;
    for (;;) {
        const int want = todo ? 1 + same : 0;
        const int upto = wave_inclusive_scan(want, lane);
        const int at = upto - want;
        const bool now = todo && upto <= kList;
        const uint64_t chosen = __ballot(now);
        if (chosen == 0) break;                                       // wave-uniform: the first one left always fits
        const int total = __builtin_amdgcn_readlane(upto, 63 - __builtin_clzll(chosen));
        todo = todo && !now;
        if (now) {
            st.leaf[at] = e;
            st.lane[at] = lane;
            if (same > 0) {
                int put = at;
                for (int j = 0; j < n_ent; j += 8) {
                    uint4 t[4];
#pragma unroll
                    for (int k = 0; k < 4; ++k) t[k] = two[(j >> 1) + k];
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        if (j + 2 * k < n_ent && t[k].y == (uint32_t)id && t[k].x != (uint32_t)e) { ++put; st.leaf[put] = (int)t[k].x; st.lane[put] = lane; }
                        if (j + 2 * k + 1 < n_ent && t[k].w == (uint32_t)id && t[k].z != (uint32_t)e) { ++put; st.leaf[put] = (int)t[k].z; st.lane[put] = lane; }
                    }
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
        // a lane per contribution: its place in the row's ascending order, where its rows are, its factors
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int i = h * kWave + lane;
            const bool have = i < total;
            const int who = have ? st.lane[i] : lane;
            const int r = __shfl(id, who), r_at = __shfl(at, who), r_same = __shfl(same, who);
            if (have) {
                const int x = st.leaf[i];
                const int s = x / k2;
                float2 c = p.coef[s];
                if constexpr (WEIGHTED) c.y = p.w2[x] / c.y;
                int to = r_at;
                for (int j = 0; j < r_same; ++j) to += st.leaf[r_at + 1 + j] < x;
                if (i != r_at) ++to;                                  // the owner is the lowest, and not among those counted
                const int64_t row_off = (int64_t)r * p.D * kElemBytes<XT>;
                const int64_t h1_off = (int64_t)s * p.D * kElemBytes<GT>;
                st.at[to] = make_longlong2((long long)(row_off | ((int64_t)(to == r_at + r_same) << 63)),
                                           (long long)(s / k1) * p.D * kElemBytes<GT>);
                st.more[to] = make_int4((int)(uint32_t)h1_off, (int)(h1_off >> 32), __float_as_int(c.x), __float_as_int(c.y));
            }
        }
        __builtin_amdgcn_wave_barrier();
        uint64_t ends[2];
#pragma unroll
        for (int h = 0; h < 2; ++h) ends[h] = __ballot(h * kWave + lane < total && st.at[h * kWave + lane].x < 0);

        // Even split of the list over the sub-groups, whole rows: a sub-group starts at the first row
        // that begins at or after its share.
        auto row_start = [&](int share) {
            const int i = share * total / nsg;
            if (i == 0) return 0;
            const uint64_t lo = i - 1 < 64 ? ends[0] >> (i - 1) << (i - 1) : 0ull;
            if (lo) return __builtin_ctzll(lo) + 1;
            const uint64_t hi = i - 1 < 64 ? ends[1] : ends[1] >> (i - 65) << (i - 65);
            return hi ? __builtin_ctzll(hi) + 65 : total;
        };
        const int start = row_start(sg);
        const int stop = sg == nsg - 1 ? total : row_start(sg + 1);

        for (int tile = 0; tile < p.tiles; ++tile) {
            const int chunk = tile * sub + sl;
            const bool there = chunk < p.chunks;
            const int64_t d = there ? chunk * VE : 0;                 // lanes past the row read its first piece
            char* const gx = p.grad_x + d * kElemBytes<XT>;
            const char* const g0 = p.grad_out + d * kElemBytes<GT>;
            const char* const g1 = H1 ? p.grad_h1 + d * kElemBytes<GT> : nullptr;
            float acc[VE];
#pragma unroll
            for (int c = 0; c < VE; ++c) acc[c] = 0.0f;
            for (int i0 = start; i0 < stop; i0 += U) {
                long long at_x[U];
                float fa[U], fw[U];
                XRaw old[U];
                GRaw go[U], gh[U];
#pragma unroll
                for (int u = 0; u < U; ++u) {                         // past the end: the last one again, not used
                    const int i = i0 + u < stop ? i0 + u : stop - 1;
                    const longlong2 a = st.at[i];
                    const int4 m = st.more[i];
                    at_x[u] = a.x;
                    fa[u] = __int_as_float(m.z);
                    fw[u] = __int_as_float(m.w);
                    old[u] = *reinterpret_cast<const XRaw*>(gx + (a.x & 0x7fffffffffffffffll));
                    go[u] = *reinterpret_cast<const GRaw*>(g0 + a.y);
                    if constexpr (H1) gh[u] = *reinterpret_cast<const GRaw*>(g1 + (int64_t)(((uint64_t)(uint32_t)m.y << 32) | (uint32_t)m.x));
                }
#pragma unroll
                for (int u = 0; u < U; ++u) {
                    if (i0 + u < stop) {
                        float t[VE];
#pragma unroll
                        for (int c = 0; c < VE; ++c) t[c] = 0.0f;
                        G::fma(t, go[u], fa[u]);
                        if constexpr (H1) G::add(t, gh[u]);
#pragma unroll
                        for (int c = 0; c < VE; ++c) acc[c] = fmaf(fw[u], t[c], acc[c]);
                        if (at_x[u] < 0) {
                            X::add(acc, old[u]);
                            if (there) *reinterpret_cast<XRaw*>(gx + (at_x[u] & 0x7fffffffffffffffll)) = X::pack(acc);
#pragma unroll
                            for (int c = 0; c < VE; ++c) acc[c] = 0.0f;
                        }
                    }
                }
            }
        }
        if (!__any(todo)) break;
        __builtin_amdgcn_wave_barrier();                              // the list is refilled by the next round
    }
}

// ---------------------------------------------------------------------------------------
// host side
// ---------------------------------------------------------------------------------------
struct OwnedLayout { size_t cnt, coef, entries, total; uint32_t n_buckets; };

static OwnedLayout owned_layout(int64_t slots, int64_t leaves) {
    auto up = [](size_t v) { return (v + 255) & ~(size_t)255; };
    OwnedLayout L;
    L.n_buckets = (uint32_t)((leaves + kBucketFill - 1) / kBucketFill);
    size_t o = 0;
    L.cnt = o;     o += up((size_t)L.n_buckets * sizeof(int));
    L.coef = o;    o += up((size_t)slots * sizeof(float2));
    L.entries = o; o += up((size_t)L.n_buckets * kBucketCap * sizeof(uint2));
    L.total = o;
    return L;
}

// Where the route pays.  Clear and mark are a fixed cost per leaf slot, which short rows do not earn
// back, and the plain updates feel the forward's traffic, which the atomics do not.  Forward and
// backward together, product graph, fanouts 15/10, atomics against this route: rows of 256 bytes equal
// at 154 k and 614 k leaf slots (backward alone 36 -> 40 and 121 -> 119 us); 400 bytes 85.5 -> 80.6 us and
// 512 bytes 89 -> 80 us at 154 k (61 and 79 MB of row updates), 512 bytes at 77 k equal (39 MB); 800 bytes
// 82 -> 68 us at 77 k; three hops, 400 bytes at 768 k, 409 -> 320 us; bf16 rows of 512 bytes 309 -> 239 us
// and of 1024 bytes 594 -> 382 us at 614 k; 1024-byte fp32 rows at 38 k (39 MB) 38 -> 30 us alone.
// Since the atomics are cut at the rows' 64-byte segments, products 78.3 / 80.2 us a pass with atomics / with this
// route, weighted 81.4 / 82.9, three hops 366 / 302, so calls just above the lines pay up to 2 %.  The lines stay because
// callers size their workspace by them and rely on what it buys: sums in a fixed order in every row that is named
// up to 16 times (include/fsa.h; rows named more often, as hubs are, go in by atomics here as well).
// The line counts leaf slots, because the call knows no more; on graphs whose slots are mostly empty or whose
// rows are mostly shared the two are equal (512-byte rows, backward alone: 169 k nodes, 256 k slots of which 73 k
// hold 31 k distinct rows, 44 -> 43 us; hubs, 307 k slots of which 36 k hold 5.7 k distinct rows, 79 -> 83 us).
constexpr int64_t kOwnedMinRowBytes = 384;
constexpr int64_t kOwnedWideRowBytes = 1024;
constexpr int64_t kOwnedMinPayload = 48ll << 20;
constexpr int64_t kOwnedMinPayloadWide = 32ll << 20;

static bool owned_backward_pays(int64_t B, int k1, int k2, int64_t D, int x_bytes) {
    const int64_t leaves = B * k1 * k2, row = D * x_bytes;
    if (k2 <= 0 || leaves > (int64_t)INT32_MAX - kTile || row < kOwnedMinRowBytes) return false;
    return leaves * row >= (row < kOwnedWideRowBytes ? kOwnedMinPayload : kOwnedMinPayloadWide);
}

size_t owned_workspace_bytes(int64_t B, int k1, int k2, int64_t D, int x_bytes) {
    return owned_backward_pays(B, k1, k2, D, x_bytes) ? owned_layout(B * k1, B * k1 * k2).total : 0;
}

template <typename GT, typename XT, int VE, bool WEIGHTED>
static void launch_owned_ve(OwnedParams& p, hipStream_t stream) {
    p.chunks = (int)(p.D / VE);
    int sub = 1, shift = 0;
    while (sub < p.chunks && sub < kWave) { sub <<= 1; ++shift; }
    p.sub = sub; p.sub_shift = shift; p.tiles = (p.chunks + sub - 1) / sub;
    // leaf slots per wave: few enough for a wave in every slot of the chip, many enough to share the look-up's
    // dependent steps (backward after its forward, 400-byte rows: 154 k leaf slots 61 / 85 with 16 / 32 per wave,
    // less the forward's 20 us; 768 k leaf slots 346 / 320)
    p.lpw = p.n_leaf >= 288000 ? 32 : 16;
#define FSA_LAUNCH_OWNED(H1_)                                                                                             \
    hipLaunchKernelGGL((owned_add_kernel<GT, XT, VE, 3, H1_, WEIGHTED>), dim3((unsigned)(((int64_t)p.n_leaf + 4 * p.lpw - 1) / (4 * p.lpw))), \
                       dim3(256), 0, stream, p)
    if (p.grad_h1) FSA_LAUNCH_OWNED(true); else FSA_LAUNCH_OWNED(false);
#undef FSA_LAUNCH_OWNED
}

template <typename GT, typename XT, bool WEIGHTED>
static hipError_t launch_owned_typed(OwnedParams& p, int ve, hipStream_t stream) {
    switch (ve) {
        case 4: launch_owned_ve<GT, XT, 4, WEIGHTED>(p, stream); break;
        case 2: launch_owned_ve<GT, XT, 2, WEIGHTED>(p, stream); break;
        case 8: if constexpr (sizeof(GT) == 2 && sizeof(XT) == 2) { launch_owned_ve<GT, XT, 8, WEIGHTED>(p, stream); break; } return hipErrorInvalidValue;
        case 1: if constexpr (sizeof(XT) == 4) { launch_owned_ve<GT, XT, 1, WEIGHTED>(p, stream); break; } return hipErrorInvalidValue;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// Elements per lane: the widest piece, 16 bytes at most, that divides the row and the alignment of
// every array of rows; 0 if a 16-bit grad_x cannot be taken in pairs.
static int owned_elements(const BwdArgs& a) {
    const int gb = a.grad_kind == 0 ? 4 : 2, xb = a.grad_x_kind == 0 ? 4 : 2;
    auto al = [](const void* q, int m) { return reinterpret_cast<uintptr_t>(q) % (uintptr_t)m == 0; };
    for (int ve = gb == 2 && xb == 2 ? 8 : 4; ve >= (xb == 2 ? 2 : 1); ve >>= 1)
        if (a.D % ve == 0 && al(a.grad_out, ve * gb) && al(a.grad_h1, ve * gb) && al(a.grad_x, ve * xb)) return ve;
    return 0;
}

// Runs the owning backward when the call is worth it and the workspace is large enough and 256-byte
// aligned; otherwise launches nothing and sets *used = false (the caller takes the atomics).
hipError_t launch_backward_owned(const BwdArgs& a, const WeightArgs* w, void* workspace, size_t workspace_bytes,
                                 hipStream_t stream, bool* used) {
    *used = false;
    const int k1 = a.k1, k2 = a.k2;
    const int x_bytes = a.grad_x_kind == 0 ? 4 : 2;
    if (!workspace || reinterpret_cast<uintptr_t>(workspace) % 256 != 0) return hipSuccess;
    if (!a.ids2 || !owned_backward_pays(a.B, k1, k2, a.D, x_bytes)) return hipSuccess;
    const OwnedLayout L = owned_layout(a.B * k1, a.B * k1 * k2);
    if (workspace_bytes < L.total) return hipSuccess;
    const int ve = owned_elements(a);
    if (ve == 0) return hipSuccess;

    char* ws = static_cast<char*>(workspace);
    OwnedParams p{};
    p.grad_out = static_cast<const char*>(a.grad_out); p.grad_h1 = static_cast<const char*>(a.grad_h1);
    p.ids1 = a.ids1; p.ids2 = a.ids2; p.root_valid = a.root_valid;
    if (w) { p.w1 = w->w1; p.w2 = w->w2; }
    p.grad_x = static_cast<char*>(a.grad_x); p.B = a.B; p.D = a.D;
    p.k1 = k1; p.k2 = k2; p.n_leaf = (int)(a.B * k1 * k2);
    const int per_root = k1 * k2;
    p.roots_per_tile = per_root < kTile ? kTile / per_root : 1;
    // smaller tiles keep 512 workgroups in a smaller call
    while (p.roots_per_tile > 1 && (a.B + p.roots_per_tile - 1) / p.roots_per_tile < 512) p.roots_per_tile = (p.roots_per_tile + 1) / 2;
    p.cnt = reinterpret_cast<int*>(ws + L.cnt);
    p.coef = reinterpret_cast<float2*>(ws + L.coef);
    p.entries = reinterpret_cast<uint2*>(ws + L.entries);
    p.n_buckets = L.n_buckets;

    const int quads = (int)((L.n_buckets + 3) / 4);                   // the counters' area is padded to 256 bytes
    hipLaunchKernelGGL(owned_clear_kernel, dim3((quads + 255) / 256), dim3(256), 0, stream, reinterpret_cast<int4*>(p.cnt), quads);
    const dim3 mark_grid((unsigned)((a.B + p.roots_per_tile - 1) / p.roots_per_tile));
    if (w) hipLaunchKernelGGL(owned_mark_kernel<true>, mark_grid, dim3(kTileThreads), 0, stream, p);
    else   hipLaunchKernelGGL(owned_mark_kernel<false>, mark_grid, dim3(kTileThreads), 0, stream, p);
    *used = true;
    if (w) return launch_owned_typed<f32_t, f32_t, true>(p, ve, stream);  // the weighted backward is fp32 on both sides
    switch (a.grad_kind * 3 + a.grad_x_kind) {
        case 0 * 3 + 0: return launch_owned_typed<f32_t, f32_t, false>(p, ve, stream);
        case 1 * 3 + 0: return launch_owned_typed<bf16_t, f32_t, false>(p, ve, stream);
        case 2 * 3 + 0: return launch_owned_typed<f16_t, f32_t, false>(p, ve, stream);
        case 0 * 3 + 1: return launch_owned_typed<f32_t, bf16_t, false>(p, ve, stream);
        case 1 * 3 + 1: return launch_owned_typed<bf16_t, bf16_t, false>(p, ve, stream);
        case 0 * 3 + 2: return launch_owned_typed<f32_t, f16_t, false>(p, ve, stream);
        case 2 * 3 + 2: return launch_owned_typed<f16_t, f16_t, false>(p, ve, stream);
        default: return hipErrorInvalidValue;
    }
}

}  // namespace fsa

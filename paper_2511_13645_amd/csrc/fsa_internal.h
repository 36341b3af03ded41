// Host-side launch interface between the C ABI (fsa_api.hip) and the kernel files.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "fsa_layout.h"

#ifdef FSA_TUNING
#include <cstdlib>
#endif

namespace fsa {

// Launch-shape overrides for sweeps.  Only a library built with -DFSA_TUNING (a separately
// named build that is never shipped) reads the environment; the product returns the default.
#ifdef FSA_TUNING
inline int tune_int(const char* name, int fallback) {
    const char* v = std::getenv(name);
    return v ? std::atoi(v) : fallback;
}
#else
constexpr int tune_int(const char*, int fallback) { return fallback; }
#endif

#ifdef FSA_TRACE
// Debug builds only (-DFSA_TRACE): per-root time stamps of the 2-hop forward go to this
// device buffer, set through fsa_debug_set_trace().
extern long long* g_trace;
#endif

// How a feature row is cut into per-lane chunks and how lanes are grouped over rows.
struct RowGeom {
    int vec_bytes;     // 16, 8, 4 or 2: bytes one lane loads per instruction
    int chunks;        // chunks per row = D * elem_bytes / vec_bytes
    int sub;           // lanes that cover one row together: min(64, pow2 >= chunks)
    int tiles;         // passes of `sub` lanes needed to cover a row
};

struct FwdArgs {
    const void* indptr; int indptr_is64; const int32_t* indices;
    const void* x; int x_kind; int64_t D;      // x_kind: 0 fp32, 1 bfloat16, 2 fp16
    const int32_t* seeds; int64_t B; int k1; int k2; int hops; uint64_t seed;
    const int32_t* ids1; const int32_t* ids2;   // replay inputs (indptr == nullptr selects replay)
    void* out; void* out_h1; int32_t* out_ids1; int32_t* out_ids2;
    RowGeom geom;
    // chained (deeper-hop) calls
    uint32_t hop_base = 0;                      // hop counter of the seeds' own rows; negative seeds = empty rows
    int32_t* out_live = nullptr;                // 2-hop: [B] number of hop-1 slots that took part
    const int32_t* slot_cnt = nullptr;          // non-null selects the slot-mean kernel: out[b] = mean of the
                                                // rows x[b*k1+j] with slot_cnt[b,j] > 0
};

struct BwdArgs {
    const void* grad_out; const void* grad_h1; const int32_t* ids1; const int32_t* ids2;
    int64_t B; int k1; int k2; int64_t D; void* grad_x;
    int grad_kind = 0;      // element type of grad_out / grad_h1: 0 fp32, 1 bfloat16, 2 fp16
    int grad_x_kind = 0;    // element type of grad_x
    const int32_t* root_valid = nullptr;   // 2-hop, chained calls: [B], a negative entry switches root b off
};

// A launch of 2^32 threads or more is cut off without an error.  So the 2-hop kernels, which take a workgroup of up
// to 512 threads per root, are launched on this many roots at a time, the others, at most a wave per seed, on
// this many seeds.
constexpr int64_t kMostRoots = 1 << 22;
constexpr int64_t kMostSeeds = 1 << 25;
inline int64_t most_at_a_time(int hops) { return hops == 2 ? kMostRoots : kMostSeeds; }

// Workgroups per root of the atomic 2-hop backwards (fsa_layout.h), whose atomic instructions take `each` rows.
inline unsigned backward_parts(int64_t B, int k2, int each) {
    const int forced = tune_int("FSA_BWD2_PARTS", 0);
    return (unsigned)(forced > 0 ? forced : parts_of_root(B, k2, each));
}

// Roots [b, b + n) of a call.
inline BwdArgs backward_part(const BwdArgs& a, int64_t b, int64_t n) {
    const int gb = a.grad_kind == 0 ? 4 : 2;
    BwdArgs c = a;
    c.B = n;
    c.grad_out = static_cast<const char*>(a.grad_out) + b * a.D * gb;
    if (a.grad_h1) c.grad_h1 = static_cast<const char*>(a.grad_h1) + b * a.k1 * a.D * gb;
    c.ids1 = a.ids1 + b * a.k1;
    if (a.ids2) c.ids2 = a.ids2 + b * a.k1 * a.k2;
    if (a.root_valid) c.root_valid = a.root_valid + b;
    return c;
}

// Weighted mean: the same launches with per-edge weights (edge_w aligned with indices) and
// the sampled weights emitted / taken back next to the IDs.
struct WeightArgs {
    const float* edge_w;                        // sampling forward
    const float* w1; const float* w2;           // replay / backward inputs
    float* out_w1; float* out_w2;               // sampling forward outputs (nullable)
};

// Roots [b, b + n) of a call; `w` is cut along with it.
inline FwdArgs forward_part(const FwdArgs& a, int64_t b, int64_t n, WeightArgs& w) {
    const int64_t row = a.D * (a.x_kind == 0 ? 4 : 2), slots = b * a.k1, leaves = slots * a.k2;
    auto at = [](auto*& q, int64_t by) { if (q) q += by; };
    auto at_row = [row](void*& q, int64_t by) { if (q) q = static_cast<char*>(q) + by * row; };
    FwdArgs c = a;
    c.B = n;
    at(c.seeds, b); at(c.ids1, slots); at(c.ids2, leaves); at(c.out_ids1, slots); at(c.out_ids2, leaves); at(c.out_live, b);
    at_row(c.out, b); at_row(c.out_h1, slots);
    if (a.slot_cnt) { c.slot_cnt += slots; c.x = static_cast<const char*>(a.x) + slots * row; }   // x is the slots' own table
    at(w.w1, slots); at(w.w2, leaves); at(w.out_w1, slots); at(w.out_w2, leaves);
    return c;
}

hipError_t launch_forward(const FwdArgs& a, hipStream_t stream);
hipError_t launch_forward_weighted(const FwdArgs& a, const WeightArgs& w, hipStream_t stream);
hipError_t launch_backward_weighted(const BwdArgs& a, const WeightArgs& w, hipStream_t stream);
hipError_t launch_backward(const BwdArgs& a, hipStream_t stream);
// 2-hop backward that owns each destination row (sorted, no atomics on full rows): needs a caller
// workspace; `*used` tells whether it ran (false: not eligible, nothing was launched).
size_t sorted_workspace_bytes(int64_t B, int k1, int k2, int64_t D);
hipError_t launch_backward_sorted(const BwdArgs& a, void* workspace, size_t workspace_bytes, hipStream_t stream,
                                  bool* used);
// Backward that owns each destination row for every element type, weighted or not: needs a caller
// workspace; `*used` as above.
size_t owned_workspace_bytes(int64_t B, int k1, int k2, int64_t D, int x_bytes);
hipError_t launch_backward_owned(const BwdArgs& a, const WeightArgs* w, void* workspace, size_t workspace_bytes,
                                 hipStream_t stream, bool* used);
// Backward that writes every row of grad_x once, whatever it held (N rows; ids2 or one hop; grad_x of the
// gradients' type).  dense_workspace_bytes is 0 where it does not run, dense_pays says
// where it is faster than clearing and atomics.
bool dense_pays(int64_t B, int k1, int k2, int64_t D, int elem_bytes, int64_t N);
size_t dense_workspace_bytes(int64_t B, int k1, int k2, int64_t D, int64_t N);
hipError_t launch_backward_dense(const BwdArgs& a, int64_t N, void* workspace, size_t workspace_bytes, hipStream_t stream);
hipError_t launch_backward1_weighted(const BwdArgs& a, const float* w1, hipStream_t stream);   // 1-hop, fp32
// work[b,j,:] = (slot j took part ? grad_out[b,:] / #such slots : 0) + grad_h1[b,j,:]  (grad_h1 nullable)
hipError_t launch_deep_grad(const float* grad_out, const float* grad_h1, const int32_t* ids1, const int32_t* ids2,
                            const int32_t* ids3, float* work, int64_t B, int k1, int k2, int k3, int64_t D,
                            hipStream_t stream);

}  // namespace fsa

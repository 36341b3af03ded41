// Index arithmetic of the forward kernels' LDS strips and of the 2-hop backward's parts, shared by the kernels and
// the host launch code, and written without HIP types so that a plain C++ compiler can build it: the
// CPU tests sweep every fanout / waves-per-root combination through these functions and
// check that every offset a kernel can form stays inside the strip the host sizes.
#pragma once

#if defined(__HIPCC__)
#define FSA_HD __host__ __device__
#else
#define FSA_HD
#endif

namespace fsa {

// Draw staging of the duplicate test: 64 lanes plus the overshoot of reading it in fours.
constexpr int kDrawStripInts = 68;

FSA_HD inline int round_up4(int v) { return (v + 3) & ~3; }

// One wave's strip of the 2-hop forward, offsets in ints from the strip base.  n = nq_max * k2
// is the most leaf rows the wave's nq_max hop-1 slots can name.
struct Fwd2Layout {
    int flat;       // int2[n]   row byte offsets of the leaf rows, slot by slot; bit 63 = last row of its slot
    int meta;       // int[n]    at a slot's last row: hop-1 slot j | owned index q << 8 | count << 16
    int flat_w;     // float[n]  weighted mean only: edge weight of each listed row
    int leaf;       // int[n]    replay only: saved leaf IDs squeezed to the front of each slot
    int leaf_w;     // float[n]  weighted replay only: their weights
    int cnt2;       // int[nq_max] replay: rows per owned slot; sampling: hop-1 node of each owned slot
    int empty_q;    // int[nq_max] owned slots without rows
    int rec;        // int4[nq_max] per owned slot: row start (lo, hi), degree (replay: count), place in flat
    int slot_a;     // float[nq_max] weighted mean only: weight of the hop-0 edge of each owned slot
    int draws;      // int[kDrawStripInts] Floyd draws of the lanes, for the duplicate test
    int per_wave;   // strip size, a multiple of 4 ints so that every strip starts 16-byte aligned
};

FSA_HD inline Fwd2Layout fwd2_layout(int nq_max, int k2, bool weighted) {
    Fwd2Layout L;
    const int n = nq_max * k2;
    int o = 0;
    L.flat = o;    o += round_up4(2 * n);
    L.meta = o;    o += round_up4(n);
    L.flat_w = o;  o += weighted ? round_up4(n) : 0;
    L.leaf = o;    o += round_up4(n);
    L.leaf_w = o;  o += weighted ? round_up4(n) : 0;
    L.cnt2 = o;    o += round_up4(nq_max);
    L.empty_q = o; o += round_up4(nq_max);
    L.rec = o;     o += 4 * nq_max;
    L.slot_a = o;  o += weighted ? round_up4(nq_max) : 0;
    L.draws = o;   o += kDrawStripInts;
    L.per_wave = o;
    return L;
}

// Hop-1 slots a wave owns when `nw` waves share a root with fanout k1: j = wave + q * nw.
FSA_HD inline int owned_slots(int k1, int nw, int wave) { return wave < k1 ? (k1 - wave + nw - 1) / nw : 0; }

// Dynamic LDS of one 2-hop forward workgroup, in bytes: the strips, one live-slot count (or
// outer weight) per strip, and the floats of the cross-wave reduction (used when nw > 1).
FSA_HD inline long long fwd2_lds_bytes(int k1, int k2, int nw, int roots_per_wg, bool weighted, int sub, int ve) {
    const Fwd2Layout L = fwd2_layout((k1 + nw - 1) / nw, k2, weighted);
    const long long strips = (long long)nw * roots_per_wg;
    return 4 * (strips * L.per_wave + round_up4((int)strips)) + 4LL * nw * sub * ve;
}

// Workgroups that share out the leaves of one root in the atomic 2-hop backwards; an atomic instruction of theirs takes
// `each` rows, so of P parts part p starts at leaf p * each of a slot.  A CU issues an atomic instruction every 40
// clocks or so, so a batch of fewer roots than CUs would leave most of the chip idle; each workgroup goes through the
// root's IDs again, so every part has an instruction of its own, and two leaves of a full slot at least.  That makes up to
// 4 parts for k2 = 10, 8 for 25, 32 for 64.  Backward alone, 1 / 2 / 4 / 8 / 16 / 32 parts: fanouts 15/10, 8 roots of 100 floats
// 10.5 / 8.2 / 7.2 / 6.8 / 6.4 / 6.5 us, 64 roots 10.5 / 8.9 / 8.3 / 8.4 / 10.0 / 16, 128 roots of 602 floats 49 / 44 / 44 / 46 / 58 / 78;
// 15/25, 8 roots of 100 floats 18.2 / 12.6 / 9.8 / 8.4 / 7.7 / 7.4; 10/64, one root of 602 floats 163 / 90 / 55 / 37 / 28 / 23, 64 roots
// 169 / 118 / 101 / 96 / 94 / 102.  Rows of 16 floats take four an instruction and gain nothing from more parts at 15/10 (all
// 5.8 .. 6.0 at 8 roots).  256 and more roots gain nothing (256 of 100 floats 17.6 / 17.7 / 17.5 with 1 / 2 / 4) and lose with
// many (300 k leaves of 64 floats 67 -> 70 with 4).
FSA_HD inline int parts_of_root(long long B, int k2, int each) {
    int parts = 1;
    while (B * parts < 256 && parts * 2 * (each > 2 ? each : 2) <= k2) parts *= 2;
    return parts;
}

// 1-hop forward: per wave 64 staged IDs (the draws of the duplicate test use the same ints
// first) and 64 staged weights.
constexpr int kFwd1StripInts = 72 + 64;

}  // namespace fsa

// The training kernel: Algorithm 1, one wavefront per clause.
// Included by tm_train_launch.hpp; its forms are compiled in tm_train_part.hip.
#ifndef TM_KERNELS_TRAIN_HPP_
#define TM_KERNELS_TRAIN_HPP_
#include <type_traits>

namespace tsetlin {

// ------------------------------------------------------------------------
// k_train: Algorithm 1, one wavefront per clause
// ------------------------------------------------------------------------

struct TrainArgs {
    Dims d;
    SatConst sat;
    uint32_t *planes;
    uint32_t *inc;
    int32_t *tally;
    const int32_t *vhat; // [q][m] snapshot the gate reads instead of the live tally, or null
    const int32_t *y_regr; // regression mode: targets [q] in 0..T; null for classification
    uint32_t *ostar;
    int32_t *fresh; // [C][4] per clause: examples whose stored output may be outdated lie in [plo,phi) or [slo,qp)
    const int32_t *order; // [C] clause handled by each wavefront of the launch
    unsigned long long *counters;
    int32_t q, qp, Qw, i_begin, i_end; // example counts fit 31 bits (checked at bind)
    uint32_t epoch;
    int lds_mask_words; // W rounded up to a multiple of 4
    int lds_off_words;  // Wf + EVAL_PAD rounded up to a multiple of 4
    int lds_wave_words; // LDS words per wavefront
    int lds_draw_off;   // where the Type I draws made ahead start among them (DEEP)
    int QW;             // words per row of XB
    int slot_lo, slot_hi; // positions of `order` this launch covers
};

// Which literal word register slot r of a lane holds.  With an even number of slots, slots 2k and 2k + 1 hold
// the plain and the negated literals of feature word 64 k + lane: one word of the example then serves both slots
// (half the registers and loads for the rows), the sign of a slot is known at compile time, and the entries
// of the evaluation list come out of one lane.  With an odd number (1 or 3) the literal words follow one
// another, lw = 64 r + lane, which wastes no lanes where a clause has few of them.
// What bounds a wide clause is the register file, i.e. how many wavefronts a SIMD holds to hide the latency
// of each other's multiplies, LDS trips and scalar loads.  With paired slots and the planes of a slot finished in
// its turn (see the feedback loop) 10 slots take 161 to 168 instead of 235 registers (three wavefronts per SIMD instead
// of two) and 20 slots 256 and 11 (thresholds of one or two Philox blocks) or 25 spilled ones instead of 462 (two instead of one).  Measured: a batch of 3,328 documents on 20,000
// clauses of 10,000 features 45.2 -> 32.2 ms, 832 examples on 16,384 clauses of 20,000 features 50.8 -> 28.2 ms.
// Narrow clauses (at most 16 literal words, one slot): lane f holds the plain literals of feature word f, lane 8 + f
// the negated ones, so that the masks of a feature word sit at fixed lanes.
template <int WPL, bool NARROW = false>
struct SlotMap {
    static constexpr bool PAIRED = WPL % 2 == 0;
    static constexpr int NX = PAIRED ? WPL / 2 : WPL; // words of an example row per lane
    static __device__ __forceinline__ bool held(int r, int lane, int Wf)
    {
        if (NARROW) return lane < 16 && (lane & 7) < Wf;
        return PAIRED ? (r / 2) * 64 + lane < Wf : r * 64 + lane < 2 * Wf;
    }
    static __device__ __forceinline__ int word(int r, int lane, int Wf) // literal word of the slot
    {
        if (NARROW) return (lane & 7) + (lane >> 3) * Wf;
        return PAIRED ? (r / 2) * 64 + lane + (r & 1) * Wf : r * 64 + lane;
    }
};

constexpr int EVAL_PAD = 16; // empty entries after the list: a group may read that far past its end

// Include mask of a register slot: plane 7 of its automata, or the mask itself.
__device__ __forceinline__ uint32_t include_mask(const u32x8 &planes) { return planes[7]; }
__device__ __forceinline__ uint32_t include_mask(const uint32_t &mask) { return mask; }

// The clause as the evaluation loop wants it: one entry per feature word whose
// plain or negated mask word is non-zero, compacted in LDS: eoff[k] = byte
// offset of that word's row in XT, emask[k] = {mask of plain literals, mask of
// negated literals}; padded with EVAL_PAD empty entries.  Rebuilt whenever plane 7
// changes.
template <int WPL, class Slot>
__device__ __forceinline__ int build_entries(const Slot (&p)[WPL], uint32_t *lmask, uint32_t *eoff,
                                             uint2 *emask, int lane, int Wf, int W, uint32_t row_bytes)
{
    int n = 0;
    auto append = [&](int fw, uint32_t mp, uint32_t mn) {
        const bool nzf = (mp | mn) != 0u;
        const uint64_t b = ballot(nzf);
        const int pre = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
        if (nzf) {
            eoff[n + pre] = (uint32_t)fw * row_bytes;
            emask[n + pre] = make_uint2(mp, mn);
        }
        n += __builtin_popcountll(b);
    };
    if constexpr (SlotMap<WPL>::PAIRED) { // both masks of a feature word sit in one lane (0 where the lane holds no word)
#pragma unroll
        for (int k = 0; k < WPL / 2; ++k) append(k * 64 + lane, include_mask(p[2 * k]), include_mask(p[2 * k + 1]));
    } else {
#pragma unroll
        for (int r = 0; r < WPL; ++r) {
            const int lw = r * 64 + lane;
            if (lw < W) lmask[lw] = include_mask(p[r]);
        }
        wave_lds_sync();
        for (int f0 = 0; f0 < Wf; f0 += 64) {
            const int fw = f0 + lane;
            const bool ok = fw < Wf;
            append(fw, ok ? lmask[fw] : 0u, ok ? lmask[Wf + fw] : 0u);
        }
    }
    if (lane < EVAL_PAD) {
        eoff[n + lane] = 0u;
        emask[n + lane] = make_uint2(0u, 0u);
    }
    wave_lds_sync();
    return n;
}

// Clause outputs for 64 examples, lane = example: bit l of the result is
// C(X_{i0+l}).  xt_block points at XT[0][i0].  An entry costs one coalesced
// 256-byte load, an LDS broadcast of its masks and two bit operations.
// Entries are taken in groups (that many loads in flight; 8 and 24 measured
// slower where the registers allow 16); a dense (young) clause violates all 64 examples
// within the first group and the loop stops.  From 6 slots on the masks of a group are read four entries at a
// time behind its loads (32 registers less); above 10 slots a group of 8 spills 27 registers and one of 16
// spills 60: 832 examples on 16,384 clauses of 20,000 features 27.2 against 28.5 ms.
__host__ __device__ constexpr int eval_group(int wpl) { return wpl > 10 ? 8 : 16; }

template <int WPL, int GROUP = eval_group(WPL)>
__device__ __forceinline__ uint64_t eval64(const uint32_t *eoff, const uint2 *emask, int nent,
                                           const uint32_t *__restrict__ xt_block, int lane)
{
    uint32_t viol = 0;
    const char *base = reinterpret_cast<const char *>(xt_block);
    const uint32_t lane4 = (uint32_t)lane * 4u;
    for (int k = 0; k < nent; k += GROUP) {
        uint32_t off[GROUP], x[GROUP];
#pragma unroll
        for (int j = 0; j < GROUP; j += 4) {
            const uint4 o = *reinterpret_cast<const uint4 *>(eoff + k + j);
            off[j] = o.x; off[j + 1] = o.y; off[j + 2] = o.z; off[j + 3] = o.w;
        }
#pragma unroll
        for (int j = 0; j < GROUP; ++j) x[j] = *reinterpret_cast<const uint32_t *>(base + (off[j] + lane4));
        const uint4 *mq = reinterpret_cast<const uint4 *>(emask + k);
#pragma unroll
        for (int j = 0; j < GROUP / 2; ++j) {
            if (WPL >= 6 && j % 2 == 0) __builtin_amdgcn_sched_barrier(0); // masks of four entries at a time
            const uint4 m = mq[j]; // {plain, negated} masks of entries 2j and 2j+1
            // a plain literal is violated where x = 0, a negated one where x = 1
            viol |= bitselect(x[2 * j], m.y, m.x) | bitselect(x[2 * j + 1], m.w, m.z);
        }
        if (ballot(viol == 0u) == 0) break;
    }
    return ballot(viol == 0u);
}

// The feedback update comes in two forms.  ROOMY: a loop over the slots for Type I events and one for Type II events; what
// an event costs a wavefront is least, but the registers of the slots are live together.  Otherwise one loop serves
// both types (a branch per slot, two more steps of latency), which needs the fewest registers.  Fewer registers are more
// wavefronts per SIMD, so the second form pays as soon as the launch has wavefronts for them, and only then.  Thresholds
// of more than two Philox blocks (DEEP) take two loops where the form is roomy (up to a SIMD per clause) or has 4 slots, else
// one: with the draws out of the way two loops gain 2 to 6 % with up to 2,000 clauses and lose 10 to 25 % with 5,000.
// Other thresholds, time with one loop divided by time with two:
//   1 slot: two loops (s = 2: 0.97 of one)
//   2 slots: one loop (1,000 to 16,000 clauses: 0.96 to 0.97 of two), roomy up to a SIMD per clause: nothing laundered, no
//     floor of five wavefronts (800 clauses of 1,500 features, s = 2: 1,052 / 998 us)
//   3 slots: two loops (0.93 to 0.99 of one at every clause count)
//   4 slots: two loops; for many clauses held to four wavefronts by the launch bound (16,000 clauses: 0.90 to 0.97 of the
//     time with three wavefronts, 0.94 to 0.99 of one loop; 3,000 clauses: 1.18 to 1.27)
//   6 to 10 slots: 1.15 with 500 to 1,000 clauses, 0.85 to 0.97 with many
//   12 to 20 slots: one loop; two would not leave room for two wavefronts
// train_min_waves: the wavefronts per SIMD that a form is held to.  DEEP, time without the bound divided by time with
// it: 1 slot (4 wavefronts instead of 5), 20,000 clauses 1.05; 10 slots (2 instead of 3) 1.25.  With spans the bound costs one slot
// spilled registers (12 when this was measured, now 17: 40 bytes of scratch per lane) and still pays: four wavefronts without any, 8,000 to 40,000
// clauses of 300 and 784 features 1.05 to 1.09, up to 4,000 clauses 0.99 to 1.0.
__host__ __device__ constexpr bool train_split(int wpl, bool roomy, bool deep) { return (roomy && (wpl != 2 || deep)) || wpl == 4 || (!deep && (wpl == 1 || wpl == 3)); }
__host__ __device__ constexpr int train_min_waves(int wpl, bool roomy) { return roomy ? 1 : wpl <= 2 ? 5 : wpl <= 6 ? 4 : wpl <= 10 ? 3 : 2; }

// Lowest Philox block that a form without draws made ahead (not DEEP) may have to draw: thresholds of more than two blocks
// reach it in regression of one slot only (launch_train_slots).
__host__ __device__ constexpr int train_least_block(int wpl, bool roomy, bool regr) { return wpl == 1 && roomy && regr ? 0 : 2; }

// train_max_waves: roomy forms of 2 and 3 slots are for launches of one wavefront per SIMD; without a ceiling the compiler
// schedules for five (1,000 clauses of 2,500 features, s = 2: 0.91 of the speed).  The roomy form of 4 slots is for up to three
// wavefronts per SIMD: where registers leave room for a fourth, some SIMDs get four and others two, and the launch takes as long
// as the fullest (3,000 clauses, s = 2, without a ceiling / with: 3,300 features 752 / 641 us, documents of 3,929 features 758 / 666).
__host__ __device__ constexpr int train_max_waves(int wpl, bool roomy) { return !roomy ? 8 : wpl == 2 || wpl == 3 ? 2 : wpl == 4 ? 3 : 8; }

// Literals a clause's list in LDS can hold for the sweeps over outdated outputs; clauses
// with more (untrained ones) are swept block by block with eval64.  Trained clauses of the
// image-like workload have 17 literals on average, but a few dozen of 20,000 grow past 64 within
// 30 epochs and past 128 within 100 (always-true negated literals of pixels that are never set
// cost nothing to include); block by block such a clause took 0.45 ms alone when it changed.
constexpr int TRAIN_LIT_MAX = 256;
constexpr int LIT_PAD = 8;       // entries of the all-ones row after the list
constexpr int SWEEP_WORDS = 2; // words of 32 examples per lane and pass of a sweep through the literal list

// Number of included literals of the clause held in p: the per-lane counts are summed bit by
// bit with ballots, a loop-free wave sum.  (An atomic add on one LDS word would do, but the
// compiler expands it into a 64-step scalar loop over the lanes.)
template <int WPL, class Slot>
__device__ __forceinline__ int count_literals(const Slot (&p)[WPL])
{
    uint32_t cnt = 0;
#pragma unroll
    for (int r = 0; r < WPL; ++r) cnt += (uint32_t)__builtin_popcount(include_mask(p[r])); // 0 where a lane holds no word
    int total = 0;
#pragma unroll
    for (int bit = 0; bit < 8; ++bit) // cnt <= 32 * WPL <= 128 for the narrow clauses this is used for
        total += __builtin_popcountll(ballot(((cnt >> bit) & 1u) != 0u)) << bit;
    return total;
}

// List of the included literals of the clause held in p (lane = literal word), as byte
// offsets of their rows in XB, padded to a multiple of PAD with the all-ones row; returns
// the number of included literals.  Only called for clauses with at most TRAIN_LIT_MAX.
// The order of the list does not matter (the output is their conjunction): a round takes one
// literal of every word that has one left, compacted over the lanes by ballot, so that a slot costs
// as many rounds as its fullest word has literals.
template <int WPL, bool NARROW, int PAD = LIT_PAD, class Slot>
__device__ __forceinline__ int build_literals(const Slot (&p)[WPL], uint32_t *llist, int lane, int Wf, int o,
                                              uint32_t xb_row_bytes)
{
    int base = 0;
#pragma unroll
    for (int r = 0; r < WPL; ++r) {
        int lw = SlotMap<WPL, NARROW>::word(r, lane, Wf);
        asm volatile("" : "+v"(lw)); // recomputed here, not kept for every slot
        uint32_t m = include_mask(p[r]); // 0 where the lane holds no word
        const uint32_t k0 = lw >= Wf ? (uint32_t)o + (uint32_t)(lw - Wf) * 32u : (uint32_t)lw * 32u; // literal of bit 0
        for (uint64_t bal; (bal = ballot(m != 0u)) != 0;) { // one literal of every word that has one left
            const int pos = base + (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(bal >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bal, 0u));
            if (m && pos < TRAIN_LIT_MAX) llist[pos] = (k0 + (uint32_t)__builtin_ctz(m)) * xb_row_bytes;
            m &= m - 1u; // stays 0 once it is 0
            base += __builtin_popcountll(bal);
        }
    }
    if (lane < PAD) llist[min(base, TRAIN_LIT_MAX) + lane] = 2u * (uint32_t)o * xb_row_bytes;
    wave_lds_sync();
    return base;
}

// The planes of a slot are final here: the compiler may not move their update behind this point.
__device__ __forceinline__ void pin_planes(uint32_t (&sp)[8], uint32_t &changed)
{
    asm volatile("" : "+v"(sp[0]), "+v"(sp[1]), "+v"(sp[2]), "+v"(sp[3]), "+v"(sp[4]), "+v"(sp[5]), "+v"(sp[6]),
                 "+v"(sp[7]), "+v"(changed));
}

constexpr int TRAIN_WAVES_MAX = 4; // most clauses (wavefronts) per workgroup of the training kernel; the launch chooses

// Type I draws of thresholds that need more than two Philox blocks (DEEP) are made ahead of the events, for up to
// this many Type I events of a round of gate entries at a time: with few register slots several events share the
// Philox calls for what the first two blocks leave undecided.  4 to 16 events with one slot measured within 2 % of
// one another up to 10, 16 slower (LDS).
__host__ __device__ constexpr int train_draw_events(int wpl) { return wpl == 1 ? 8 : wpl == 2 ? 4 : wpl <= 4 ? 2 : 1; }
constexpr int DRAW_RING = 128; // words of literals waiting for their last two blocks: at most 31 left over and 64 new ones
// Launches of one wavefront per SIMD, one slot, DEEP (which takes every threshold then): other wavefronts of the workgroup draw the
// gates and the Type I events of a round of gate entries while the first works through the round before.  A wavefront alone on its
// SIMD leaves two thirds of the issue slots empty, and its time is the length of its own chain, of which the draws are almost half.
// They meet at one barrier per round; what is handed over lies in LDS twice.
// Four wavefronts with train_spans, two with train_clause.
__host__ __device__ constexpr bool train_team(int wpl, bool roomy, bool deep, bool narrow) { return wpl == 1 && roomy && deep && !narrow; }
// Forms that come with train_spans as well, for classification.  Spans gain most where masks change seldom; where they change at every second
// event, as on bag-of-words data, spans are short and taken row by row.  Speed with against without, first eight epochs of 60 to 20,000 clauses with
// s = 2 to 10, noisy images / bags of words: one slot, teams 1.6 to 1.8 / 1.2, wavefronts DEEP 1.3 / 1.05, not DEEP 1.1 / 0.86 to 0.9 (1.2 settled);
// two slots, DEEP and few clauses 1.08 / 0.97; three slots 1.16 to 1.27 / 0.97 to 1.15.  Two slots, DEEP and many clauses 0.88 to 0.92 on images,
// not DEEP 1.04 to 1.11 / 0.77 to 0.84 (measured when a block was evaluated for every short span): without.
__host__ __device__ constexpr bool train_has_spans(int wpl, bool roomy, bool deep, bool narrow)
{
    return wpl <= 3 && !narrow && (wpl != 2 || (deep && roomy));
}
// Least gate entries per class and launch, as the host expects them (every gate open), for which they take it.  Short launches mean
// young machines, whose masks change at every second or third event, and then an open block is the cheaper place for the outputs.
// Speed with spans, by expected entries (200 to 5,000 clauses per class of 400 to 2,500 features, s = 2 and 10): 400 0.85 to 0.97, 800 0.93
// to 1.05, 1,600 1.0 to 1.3, 4,000 1.06 to 1.4, 8,000 1.1 to 1.8; teams 400 0.98, 800 1.05, 1,600 1.16 to 1.4; two slots 1,600 0.97, 4,000 1.03.
__host__ __device__ constexpr int train_spans_from(int wpl, bool roomy, bool deep)
{
    return train_team(wpl, roomy, deep, false) ? 800 : wpl == 2 ? 3000 : 1500;
}
constexpr int TEAM_ROUND = 32;     // gate entries per round
constexpr int TEAM_DRAWERS = 2;    // wavefronts that draw Type I events
constexpr int TEAM_HANDED = 36;    // words handed over per round beside rows and draws
constexpr int PAIR_ROUND = 64 + 8; // words handed over per round of 64 entries: examples, masks of fired and target-1 lanes, open gates
__host__ __device__ constexpr int train_draw_words(int wpl, bool team) // without spans
{
    return 4 * DRAW_RING + 64 * wpl * (team ? 2 * 64 : train_draw_events(wpl)) + (team ? 2 * PAIR_ROUND : 0);
}

// A clause whose class has many open gates in this launch is all but certain to get feedback: its
// automata are loaded up front and the loop carries no check for them (the check and the pointers it
// keeps alive cost the feedback-bound regime 3-10 %).  With few open gates - a trained machine - most
// clauses get none, and the lazy version saves moving their automata (16 % of a quiet epoch).
constexpr int TRAIN_EAGER_CANDIDATES = 256;

// Event counters of one clause: 64 interleaved sets, because thousands of wavefronts ending at the
// same time on one address serialise in the L2 atomic unit (measured: ~1.7 ms per launch)
__device__ __forceinline__ void store_counters(const TrainArgs &a, int g, int lane, uint32_t n_listed_blocks, uint32_t n_fired,
                                               uint32_t n_type1, uint32_t n_changes, uint32_t n_type2, uint32_t n_eval,
                                               uint32_t n_draw, bool moved)
{
    if (lane < 10) { // slot 4 (trained pairs) is counted by the launch preparation; slot 8: examples this clause
                     // walked; slot 9: 1 if its automata were fetched (and written back)
        const uint32_t v = lane == 0 ? n_listed_blocks : lane == 1 ? n_fired : lane == 2 ? n_type1 : lane == 3 ? n_changes
                         : lane == 4 ? 0u : lane == 5 ? n_type2 : lane == 6 ? n_eval : lane == 7 ? n_draw
                         : lane == 8 ? (uint32_t)(a.i_end - a.i_begin) : (moved ? 1u : 0u);
        if (v) atomicAdd(&a.counters[(g & (COUNTER_SETS - 1)) * COUNTER_WIDTH + lane], (unsigned long long)v);
    }
}

} // namespace tsetlin
#include "tm_kernels_train_spans.hpp"
namespace tsetlin {

// One wavefront = one clause of class c.  The examples whose gate can open for this
// clause are those of the gate list of c for this launch (label c: trained towards 1;
// drawn negative class c: trained towards 0); their gates are drawn 64 at a time, lane =
// list entry.  Blocks of 64 consecutive examples are evaluated (lane = example) only
// when a gate in them fired or their stored outputs may be outdated; all other blocks
// of the pass are never touched.
// LAZY: the automata (all planes but the include masks) are fetched only when the first feedback
// is due and written back only if there was one; otherwise they are loaded up front.  The kernel
// holds both versions of the loop and picks per clause (see k_train).
template <int WPL, bool FULL, bool REGR, bool LAZY, bool NARROW, bool ROOMY, bool DEEP, bool TINY>
__device__ __forceinline__ void train_clause(const uint32_t *__restrict__ X, const uint32_t *__restrict__ XT,
                                             const uint32_t *__restrict__ XB, const int32_t *__restrict__ gate,
                                             const int k_hi, const TrainArgs &a, uint32_t *lds, const int g,
                                             const int lane, const int wave, const bool helper)
{
    constexpr bool TEAM = train_team(WPL, ROOMY, DEEP, NARROW);
    using Map = SlotMap<WPL, NARROW>;
    const Dims &d = a.d;
    uint32_t *lmask = lds + (TEAM ? 0 : wave) * a.lds_wave_words; // [W] include masks, literal-word order
    uint32_t *eoff = lmask + a.lds_mask_words;              // [Wf + EVAL_PAD] (rounded to 4 words)
    uint2 *emask = reinterpret_cast<uint2 *>(eoff + a.lds_off_words);
    uint32_t *llist = lmask + a.lds_wave_words - (TRAIN_LIT_MAX + LIT_PAD); // [TRAIN_LIT_MAX + LIT_PAD] literal list for the sweeps

    const int c = g / d.n;
    constexpr bool regr = REGR;                   // regression mode: every clause votes +1 (a compile-time
                                                  // switch: as a run-time one it cost wide clauses 36 registers)
    // Key and threshold are laundered in front of the draws of kernels that many clauses share a SIMD in: the constants
    // derived from them (20 round keys, comparator masks) are then computed by scalar instructions where they are used.  Kept for
    // the whole kernel they overflow the scalar registers and come back through readlane, a vector instruction each
    // (20,000 clauses of 784 features: 2 % of a loaded epoch, 7 % of a quiet one).  A wavefront alone on its SIMD waits for
    // the scalar additions instead (90 clauses of 297 features, quiet: 29 us kept, 35 us laundered).
    constexpr bool LAUNDER = TINY || (!NARROW && !ROOMY);
    const bool pos = ((g - c * d.n) & 1) != 0 || regr; // odd index within the class: positive polarity
    const int sign = pos ? 1 : -1;
    const int T = d.T;
    const uint32_t row_bytes = (uint32_t)a.qp * 4u;
    const int i_begin = a.i_begin, i_end = a.i_end, q = a.q;

    // The automata of the clause.  Until the first gate fires only the include masks (plane 7, of
    // which `inc` holds a compact copy) are needed - for evaluation and sweeps -, so the other seven
    // planes are fetched when the first feedback is due and written back only if there was one: in a
    // trained machine most clauses get no feedback in an epoch and move 200 bytes instead of 3.2 KB.
    u32x8 p[WPL];
#pragma unroll
    for (int r = 0; r < WPL; ++r) {
        const int lw = Map::word(r, lane, d.Wf);
        u32x8 t = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
        if (Map::held(r, lane, d.Wf)) t[7] = a.inc[(int64_t)g * d.W + lw];
        p[r] = t;
    }
    bool have_planes = false;
    // Clauses of one feature word (TINY): lane l < 32 holds the state of literal l, lane 32 + l that of its negation, as a
    // number; include masks, the word of an example and draws are masks over the lanes in scalar registers.  An event is a handful of scalar operations and four vector ones (add, subtract, clamp,
    // compare) instead of the fifty dependent ones of the bit planes, and what an epoch of so small a machine costs is its
    // events' latency.  Outputs of the open block are taken when the masks change and when it is closed.
    // Noisy XOR (20 clauses, 5,000 examples) 958 -> 545 us; with two words the planes are as fast (0.91 to 0.94 of their
    // speed), with four faster (0.63 to 0.78).
    uint32_t st = 0u;                    // stored states
    uint64_t inc64 = 0, valid64 = 0;
    if constexpr (TINY) {
        inc64 = (uint64_t)readlane(p[0][7], 0) | ((uint64_t)readlane(p[0][7], 8) << 32);
        valid64 = (uint64_t)d.tailmask | ((uint64_t)d.tailmask << 32);
    }
    auto load_planes = [&]() {
        if constexpr (TINY) {
            const uint4 *src = reinterpret_cast<const uint4 *>(a.planes + ((int64_t)g * 2 + (lane >> 5)) * 8);
            const uint4 v0 = src[0], v1 = src[1];
            const uint32_t pl[8] = {v0.x, v0.y, v0.z, v0.w, v1.x, v1.y, v1.z, v1.w};
            st = 0u;
#pragma unroll
            for (int b = 0; b < 8; ++b) st |= ((pl[b] >> (lane & 31)) & 1u) << b;
            have_planes = true;
            return;
        }
#pragma unroll
        for (int r = 0; r < WPL; ++r) {
            int ln = lane;
            asm volatile("" : "+v"(ln)); // addresses are formed here, not kept for every slot
            const int lw = Map::word(r, ln, d.Wf);
            if (Map::held(r, ln, d.Wf)) {
                const uint4 *src = reinterpret_cast<const uint4 *>(a.planes + ((int64_t)g * d.W + lw) * 8);
                const uint4 v0 = src[0], v1 = src[1];
                u32x8 t;
                t[0] = v0.x; t[1] = v0.y; t[2] = v0.z; t[3] = v0.w;
                t[4] = v1.x; t[5] = v1.y; t[6] = v1.z; t[7] = v1.w; // equals the include mask held so far
                p[r] = t;
            }
        }
        have_planes = true;
    };
    if ((!LAZY || k_hi >= TRAIN_EAGER_CANDIDATES) && !helper) load_planes();
    int nent = 0;
    bool list_ok = true; // the entries are those of the current masks
    if constexpr (!NARROW) {
        if (!helper) nent = build_entries<WPL>(p, lmask, eoff, emask, lane, d.Wf, d.W, row_bytes);
    }

    // Narrow clauses.  An epoch of so small a machine is the chain of one clause's feedback events and block
    // changes, and costs their latency and nothing else.  So the words of the open block of 64 examples stay in
    // registers (lane = example, at most eight words), the next block's are requested a block ahead, and an event
    // touches neither LDS lists nor memory.  Measured per epoch: noisy XOR (20 clauses of 2 literal words, 5,000
    // examples) 1.27 -> 0.96 ms, regression (1,280 clauses of 16 words, 13,911 examples) 0.673 -> 0.654 ms.
    uint32_t bw[NARROW ? 8 : 1] = {}, bw_next[NARROW ? 8 : 1] = {}, os_next0 = 0u, os_next1 = 0u;
    int block_next = -1; // block that bw_next holds
    auto narrow_load = [&](int b, uint32_t (&dst)[NARROW ? 8 : 1]) {
        if constexpr (NARROW) {
#pragma unroll
            for (int f = 0; f < (TINY ? 1 : 8); ++f)
                dst[f] = XT[(uint32_t)min(f, d.Wf - 1) * (uint32_t)a.qp + (uint32_t)(b << 6) + (uint32_t)lane];
        }
    };
    auto narrow_eval = [&](const uint32_t (&x)[NARROW ? 8 : 1]) { // outputs of the clause on the block held in x
        uint32_t viol = 0u;
        if constexpr (TINY) {
            viol = bitselect(x[0], (uint32_t)(inc64 >> 32), (uint32_t)inc64);
        } else if constexpr (NARROW) {
            const uint32_t m7 = p[0][7];
            auto word = [&](int f) { viol |= bitselect(x[f], readlane(m7, 8 + f), readlane(m7, f)); };
            word(0);
            word(1);
            if (d.Wf > 2) { // masks beyond the last word are 0
                word(2);
                word(3);
                if (d.Wf > 4) {
#pragma unroll
                    for (int f = 4; f < 8; ++f) word(f);
                }
            }
        }
        return ballot(viol == 0u);
    };
    auto narrow_keep = [&]() { // more than two words: the block also goes to LDS, from where an event takes its row
        if constexpr (NARROW && !TINY) {
            if (d.Wf > 2) {
#pragma unroll
                for (int f = 0; f < 8; ++f) lmask[f * 64 + lane] = bw[f];
                wave_lds_sync();
            }
        }
    };
    auto narrow_row = [&](int bl) { // word lane & 7 of example bl of the open block
        uint32_t v = 0u;
        if constexpr (NARROW) {
            if (d.Wf > 2) {
                v = lmask[(lane & 7) * 64 + bl];
            } else {
                const uint32_t v0 = readlane(bw[0], bl), v1 = readlane(bw[1], bl);
                v = (lane & 7) == 0 ? v0 : v1;
            }
        }
        return v;
    };

    // lowest Philox block of the Type I comparator that can matter: bits of the
    // uniform below the lowest set bit of thr never decide u < thr
    const int tz = d.thr ? __builtin_ctz(d.thr) : 16;
    const int first_blk = min(tz >> 2, 4);
    const uint32_t ge_init = d.thr >= 65536u ? 0u : ~0u;
    // Narrow clauses leave most lanes idle while their word lanes draw up to four blocks each, one after the
    // other, for every Type I event.  Their draws depend on nothing but the example, so they are made ahead and
    // side by side: lane = (event, block t, half h, feature word f), with the words of a half rounded up to wp = 1, 2, 4
    // or 8, i.e. 8 / wp events per Philox call.  The four partial
    // comparisons of a word are folded at once for all events; an event takes its lanes with one shuffle.
    const int wps = TINY ? 0 : d.Wf <= 2 ? 1 : d.Wf <= 4 ? 2 : 3; // wp = 1 << wps
    const int dr_f = lane & ((1 << wps) - 1), dr_h = (lane >> wps) & 1, dr_t = (lane >> (wps + 1)) & 3, dr_e = lane >> (wps + 3);
    // complement of the four thr bits of this lane's block; 65536 (s = 1) as 65535: with ge_init = 0 nothing stays "at least"
    const uint32_t thr_nibble_n = NARROW ? ~(min(d.thr, 65535u) >> (4 * dr_t)) : 0u;
    const uint32_t dr_ctr = 4u * (uint32_t)(dr_f + dr_h * d.Wf) + (uint32_t)dr_t;
    const int dr_src = ((lane >> 3) & 1) * (1 << wps) + (lane & ((1 << wps) - 1)); // draw lane (event 0) of this state lane
    uint32_t ge_ahead = 0u;
    int t1_done = 0; // TINY: Type I events of the round drawn so far
    int n_ahead = 0; // events drawn ahead and not used yet; they are consecutive Type I events of the round
    auto narrow_draw = [&](uint64_t t1, int iv) { // t1: Type I events of the round still to come, iv: example of each gate lane
        if constexpr (NARROW) {
            const int per_call = 8 >> wps;
            uint32_t ii = 0u;
            if constexpr (TINY) { // the examples of the round's Type I events lie side by side in LDS
                n_ahead = min(per_call, __builtin_popcountll(t1));
                ii = lmask[t1_done + dr_e];
                t1_done += n_ahead;
            } else {
                for (n_ahead = 0; n_ahead < per_call && t1; ++n_ahead) {
                    const uint32_t id = readlane((uint32_t)iv, __builtin_ctzll(t1));
                    t1 &= t1 - 1;
                    ii = dr_e == n_ahead ? id : ii;
                }
            }
            // Over the four planes of one block the comparison is "the value that went in if the four bits
            // equal those of thr, else decided": two runs of the chain, from 0 and from 1, give what is
            // decided (d0) and where the input passes (d0 ^ d1).
            RngKey key = d.key;
            if (TINY) asm volatile("" : "+s"(key.seed_lo), "+s"(key.seed_hi)); // the scalar registers are wanted for the masks
            const U4 R = draw(key, STREAM_TYPE1, dr_ctr, (uint32_t)g, (uint64_t)ii, a.epoch);
            const uint32_t w[4] = {R.x, R.y, R.z, R.w};
            uint32_t d0 = 0u, d1 = ~0u;
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const uint32_t K = (uint32_t)__builtin_amdgcn_sbfe((int)thr_nibble_n, j, 1); // thr bit 1: 0, 0: ~0
                d0 = majority3(w[j], d0, K);
                d1 = majority3(w[j], d1, K);
            }
            const uint32_t pass = d0 ^ d1;
            ge_ahead = ge_init;
#pragma unroll
            for (int t = 0; t < 4; ++t) { // least significant block first
                const int src = (lane & ~(3 << (wps + 1))) | (t << (wps + 1));
                const uint32_t dt = (uint32_t)__shfl((int)d0, src, 64), pt = (uint32_t)__shfl((int)pass, src, 64);
                ge_ahead = dt | (pt & ge_ahead);
            }
        }
    };
    int n_used = 0; // of the events drawn ahead

    // Type I draws ahead, clauses of any width.  A uniform is compared with thr from its most significant bits: after the
    // eight bits of blocks 3 and 2 all but one literal in 256 are decided, and only the words that hold one of the others
    // draw their last two blocks, gathered from all the words of a batch: item k of a call is drawn by lane k (block 1)
    // and lane k + 32 (block 0).  Same counters and bits as drawing every block.  What bounds the loop is vector issue, most
    // of it Philox rounds: a word costs 2 blocks and a share of a call instead of 4 blocks.  Vector instructions per
    // pass and time: 20,000 clauses of 784 features -14 %, 29.2 -> 25.2 ms; 16,384 clauses of 20,000 features -23 %, 30.5 -> 26.1 ms.
    uint4 *ring = reinterpret_cast<uint4 *>(lmask + a.lds_draw_off); // {4 lw, undecided literals, example, index in draws}
    uint32_t *draws = lmask + a.lds_draw_off + 4 * DRAW_RING;        // [event][slot][lane]: u >= thr
    auto deep_rest = [&](int head, int cnt) { // items head .. head + cnt - 1 of the ring, at most 32
        const uint4 it = ring[(head + (lane & 31)) & (DRAW_RING - 1)];
        const bool low = lane >= 32;
        RngKey key = d.key;
        if (LAUNDER) asm volatile("" : "+s"(key.seed_lo), "+s"(key.seed_hi));
        const U4 R = draw(key, STREAM_TYPE1, it.x + (low ? 0u : 1u), (uint32_t)g, (uint64_t)it.z, a.epoch);
        const uint32_t w[4] = {R.x, R.y, R.z, R.w};
        const uint32_t nib = ~(low ? d.thr : d.thr >> 4);
        uint32_t d0 = 0u, d1 = ~0u; // above, not below: see narrow_draw
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t K = (uint32_t)__builtin_amdgcn_sbfe((int)nib, k, 1);
            d0 = majority3(w[k], d0, K);
            d1 = majority3(w[k], d1, K);
        }
        const uint32_t ge_low = (uint32_t)__shfl_xor((int)d1, 32, 64); // block 0: not below
        if (lane < cnt) draws[it.w] |= it.y & (d0 | (d1 & ge_low));
        wave_lds_sync();
    };
    auto deep_draw = [&](uint64_t t1, int iv, int most, int place) { // at most `most` events, results from draws[place] on; t1: Type I events of the round still to come, iv: example of each gate lane
        int head = 0, cnt = 0;
        RngKey key = d.key;
        uint32_t nthr = ~d.thr;
        if (LAUNDER) asm volatile("" : "+s"(key.seed_lo), "+s"(key.seed_hi), "+s"(nthr));
        const int slots = SlotMap<WPL>::PAIRED ? 2 * ((d.Wf + 63) >> 6) : WPL;
        for (n_ahead = 0; n_ahead < most && t1; ++n_ahead) {
            const uint32_t id = readlane((uint32_t)iv, __builtin_ctzll(t1));
            t1 &= t1 - 1;
#pragma unroll 1
            for (int r = 0; r < slots; ++r) {
                const uint32_t c4 = 4u * (uint32_t)Map::word(r, lane, d.Wf);
                const U4 A = draw(key, STREAM_TYPE1, c4 + 2u, (uint32_t)g, (uint64_t)id, a.epoch);
                const U4 B = draw(key, STREAM_TYPE1, c4 + 3u, (uint32_t)g, (uint64_t)id, a.epoch);
                const uint32_t w[8] = {A.x, A.y, A.z, A.w, B.x, B.y, B.z, B.w};
                uint32_t d0 = 0u, d1 = ~0u;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const uint32_t K = (uint32_t)__builtin_amdgcn_sbfe((int)nthr, 8 + k, 1);
                    d0 = majority3(w[k], d0, K);
                    d1 = majority3(w[k], d1, K);
                }
                const uint32_t undecided = Map::held(r, lane, d.Wf) ? d0 ^ d1 : 0u;
                const uint32_t at = (uint32_t)(place + (n_ahead * WPL + r) * 64 + lane);
                draws[at] = d0;
                const uint64_t b = ballot(undecided != 0u);
                const int pre = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                if (undecided) ring[(head + cnt + pre) & (DRAW_RING - 1)] = make_uint4(c4, undecided, id, at);
                cnt += __builtin_popcountll(b);
                wave_lds_sync();
                while (cnt >= 32) {
                    deep_rest(head, 32);
                    head += 32;
                    cnt -= 32;
                }
            }
        }
        if (cnt) deep_rest(head, cnt);
    };

    // per-wavefront event counts of one launch fit 32 bits (at most 2^30 examples per launch)
    uint32_t n_fired = 0, n_type1 = 0, n_changes = 0, n_type2 = 0, n_eval = 0, n_draw = 0, n_listed_blocks = 0;

    // Which stored previous outputs o* can differ from the clause's current output: only
    // those not re-evaluated since the include mask last changed.  Kept per clause as two
    // example ranges, a prefix part [plo, phi) and a suffix [slo, qp), multiples of 64 where this form has left them and
    // any examples where train_spans has, so that whoever reads them rounds outwards to whole blocks; a
    // block outside both needs no evaluation and no refresh unless one of its gates fires
    // (the result is the same as refreshing every visited pair: o != o* would be false).
    int plo, phi, slo;
    {
        const int4 f = *reinterpret_cast<const int4 *>(a.fresh + (int64_t)g * 4);
        plo = __builtin_amdgcn_readfirstlane(f.x);
        phi = __builtin_amdgcn_readfirstlane(f.y);
        slo = __builtin_amdgcn_readfirstlane(f.z);
    }
    auto next_stale = [&](int b) { // first block index >= b that may hold outdated outputs
        int r = max(b, slo >> 6);
        if (plo < phi && b < ((phi + 63) >> 6)) r = min(r, max(b, plo >> 6));
        return r;
    };

    // the gate list of this class for this launch
    const int32_t *list = gate + (int64_t)c * a.qp;
    const int k_lo = 0;
    const int32_t *tally_c = a.tally + (int64_t)c * a.qp;

    // state of the block of 64 examples that is currently open (cb < 0: none)
    const int end_block = (i_end + 63) >> 6;
    int cb = -1, next_block = i_begin >> 6;
    uint64_t obits = 0, ost = 0, rmask = 0;
    bool mask_changed = false;

    auto range_mask = [&](int b0) { return ballot(b0 + lane >= i_begin && b0 + lane < i_end); };
    auto pack64 = [&](uint32_t lo, uint32_t hi) {
        return (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)lo) |
               ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)hi) << 32);
    };
    // Refresh of tally and previous-output bits (last lines of Algorithm 1) for the 64
    // examples of block b at once: ob = outputs with the current masks, os = stored ones,
    // rm = examples of the block that belong to this launch.
    auto refresh_block = [&](int b, uint64_t ob, uint64_t os, uint64_t rm) {
        const int b0 = b << 6;
        const uint64_t diff = (ob ^ os) & rm;
        if (diff) {
            if ((diff >> lane) & 1ull) {
                const int delta = ((ob >> lane) & 1ull) ? sign : -sign;
                atomicAdd(&a.tally[(int64_t)c * a.qp + b0 + lane], delta);
            }
            const uint64_t nw = os ^ diff;
            if (lane == 0) {
                uint32_t *op = a.ostar + (int64_t)g * a.Qw + (b0 >> 5);
                op[0] = (uint32_t)nw;
                op[1] = (uint32_t)(nw >> 32);
            }
            n_changes += __builtin_popcountll(diff);
        }
    };
    // Narrow clauses: the refresh of a closed block is held back until the next gate entries have arrived.  Loads
    // and atomics of a wavefront complete in order, and where all clauses correct the same few tallies at the same
    // time an atomic takes microseconds: a load issued behind it would wait for it.
    int held_block = -1;
    uint64_t held_ob = 0, held_os = 0, held_rm = 0;
    auto refresh_held = [&]() {
        if (NARROW && held_block >= 0) {
            refresh_block(held_block, held_ob, held_os, held_rm);
            held_block = -1;
        }
    };
    // ... followed by the bookkeeping of which stored outputs may be outdated
    auto close_block = [&](int b, uint64_t ob, uint64_t os, uint64_t rm, bool changed) {
        if constexpr (NARROW) {
            refresh_held();
            held_block = b;
            held_ob = ob;
            held_os = os;
            held_rm = rm;
        } else {
            refresh_block(b, ob, os, rm);
        }
        const int b0 = b << 6, b1 = b0 + 64;
        const bool whole = b0 >= i_begin && (b1 <= i_end || i_end == q);
        if (whole) { // this block is up to date again
            if (b0 <= plo) plo = max(plo, b1);
            if (b0 <= slo) slo = max(slo, b1);
        }
        if (changed) { // everything not visited after the change is outdated now
            plo = 0;
            phi = b1;
            slo = b1;
        }
    };
    // Refresh of every block in [from, to) that may hold outdated outputs; no gate fired in
    // them, so the masks stay as they are.  After a mask change these are all the blocks up
    // to the next fired gate, most of what an epoch of a trained machine has to evaluate.
    // A trained clause has few literals, so the sweep walks its literal list over the rows
    // of XB, lane = SWEEP_WORDS words of 32 examples: 4096 examples per pass and one load per literal and word.
    int n_listed = -1;          // literals of the current masks (list built if <= TRAIN_LIT_MAX), -1: not counted since the last change
    uint32_t n_changes_v = 0;   // tally changes found by the passes, per lane
    const char *xb_base = reinterpret_cast<const char *>(XB);
    uint32_t *ostar_row = a.ostar + (int64_t)g * a.Qw;
    auto sweep_listed = [&](int bs, int be) { // blocks [bs, be), all of them possibly outdated
        // SWEEP_WORDS words per lane and pass, eight literals per round: 16 independent loads in flight.
        // What a sweep costs is the number of dependent trips to the L2 - a clause whose mask changed
        // walks the rest of the epoch alone, and the last such clause is the tail of the launch
        // (measured per wavefront: 2.6 us per pass of 2,048 examples and 28 literals before, one word
        // per lane).  Four words per lane halve the trips again but cost 24 registers and with them a
        // wavefront per SIMD: 6-8 % on feedback-bound epochs, so two it is.
        const int w_end = 2 * be;
        for (int w0 = 2 * bs; w0 < w_end; w0 += 64 * SWEEP_WORDS) {
            uint32_t rm[SWEEP_WORDS], woff[SWEEP_WORDS], ost[SWEEP_WORDS], accv[SWEEP_WORDS];
#pragma unroll
            for (int u = 0; u < SWEEP_WORDS; ++u) {
                const int w = w0 + u * 64 + lane;
                const bool act = w < w_end;
                const int e0 = w << 5;
                const int lo = min(max(i_begin - e0, 0), 32), hi = min(max(i_end - e0, 0), 32);
                rm[u] = 0u; // examples of the word that belong to this launch
                if (act && hi > lo) rm[u] = (hi == 32 ? ~0u : (1u << hi) - 1u) & ~((1u << lo) - 1u);
                woff[u] = act ? (uint32_t)w * 4u : 0u;
                ost[u] = act ? ostar_row[w] : 0u;
                accv[u] = rm[u];
            }
            for (int k = 0; k < n_listed; k += 8) { // the list is padded to a multiple of 8 with the all-ones row
                const uint4 e = *reinterpret_cast<const uint4 *>(llist + k), e2 = *reinterpret_cast<const uint4 *>(llist + k + 4);
                uint32_t x[SWEEP_WORDS][8];
#pragma unroll
                for (int u = 0; u < SWEEP_WORDS; ++u) {
                    x[u][0] = *reinterpret_cast<const uint32_t *>(xb_base + (e.x + woff[u]));
                    x[u][1] = *reinterpret_cast<const uint32_t *>(xb_base + (e.y + woff[u]));
                    x[u][2] = *reinterpret_cast<const uint32_t *>(xb_base + (e.z + woff[u]));
                    x[u][3] = *reinterpret_cast<const uint32_t *>(xb_base + (e.w + woff[u]));
                    x[u][4] = *reinterpret_cast<const uint32_t *>(xb_base + (e2.x + woff[u]));
                    x[u][5] = *reinterpret_cast<const uint32_t *>(xb_base + (e2.y + woff[u]));
                    x[u][6] = *reinterpret_cast<const uint32_t *>(xb_base + (e2.z + woff[u]));
                    x[u][7] = *reinterpret_cast<const uint32_t *>(xb_base + (e2.w + woff[u]));
                }
                uint32_t any = 0u;
#pragma unroll
                for (int u = 0; u < SWEEP_WORDS; ++u) {
                    accv[u] &= x[u][0] & x[u][1] & x[u][2] & x[u][3] & x[u][4] & x[u][5] & x[u][6] & x[u][7];
                    any |= accv[u];
                }
                // a clause of many literals is false on all examples of the pass after a few rounds
                if (n_listed > 32 && ballot(any != 0u) == 0) break;
            }
#pragma unroll
            for (int u = 0; u < SWEEP_WORDS; ++u) {
                const int w = w0 + u * 64 + lane;
                uint32_t diff = (accv[u] ^ ost[u]) & rm[u];
                if (diff) ostar_row[w] = ost[u] ^ diff;
                n_changes_v += (uint32_t)__builtin_popcount(diff);
                while (diff) { // one tally correction per changed example
                    const int bit = __builtin_ctz(diff);
                    diff &= diff - 1u;
                    atomicAdd(&a.tally[(int64_t)c * a.qp + (w << 5) + bit], ((accv[u] >> bit) & 1u) ? sign : -sign);
                }
            }
        }
        n_eval += (uint32_t)(be - bs);
        n_listed_blocks += (uint32_t)(be - bs);
        // the whole blocks among them are up to date again
        const int fs = max(bs, (i_begin + 63) >> 6), fe = (i_end == q) ? be : min(be, i_end >> 6);
        if (fs < fe) {
            const int b0 = fs << 6, b1 = fe << 6;
            if (b0 <= plo) plo = max(plo, b1);
            if (b0 <= slo) slo = max(slo, b1);
        }
    };
    auto list_outputs = [&](int b) { // outputs of the clause on block b from the entries, rebuilt if the masks changed
        if (!list_ok) {
            nent = build_entries<WPL>(p, lmask, eoff, emask, lane, d.Wf, d.W, row_bytes);
            list_ok = true;
        }
        return eval64<WPL>(eoff, emask, nent, XT + (b << 6), lane);
    };
    auto sweep = [&](int from, int to) {
        if (next_stale(from) >= to) return;
        // the outdated blocks are those of [plo, phi) and of [slo, qp), in this order
        int s1 = from, e1 = from;
        if (plo < phi) {
            s1 = max(from, plo >> 6);
            e1 = max(s1, min(to, (phi + 63) >> 6));
        }
        const int s2 = max(max(from, slo >> 6), e1);
        const int n_blocks = (e1 - s1) + max(to - s2, 0);
        // The list pays for runs of blocks: a few blocks, or a list that the last mask change
        // left to be rebuilt for a short run, are cheaper block by block below; so are wide
        // clauses (their registers hold the automata) and untrained ones (hundreds of literals).
        if (WPL <= 4 && n_blocks >= (n_listed < 0 ? 8 : 3)) {
            if (n_listed < 0) {
                if constexpr (TINY) p[0][7] = lane == 0 ? (uint32_t)inc64 : lane == 8 ? (uint32_t)(inc64 >> 32) : 0u;
                n_listed = count_literals<WPL>(p);
                if (n_listed <= TRAIN_LIT_MAX) build_literals<WPL, NARROW>(p, llist, lane, d.Wf, d.o, (uint32_t)a.QW * 4u);
            }
            if (n_listed <= TRAIN_LIT_MAX) {
                if (s1 < e1) sweep_listed(s1, e1);
                if (s2 < to) sweep_listed(s2, to);
                return;
            }
        }
        for (int b = next_stale(from); b < to; b = next_stale(b + 1)) { // closing b does not change which later blocks are outdated
            const uint32_t *op = ostar_row + (b << 1);
            const uint32_t o0 = op[0], o1 = op[1];
            uint64_t ob;
            if constexpr (NARROW) {
                uint32_t x[8];
                narrow_load(b, x);
                ob = narrow_eval(x);
            } else {
                ob = list_outputs(b);
            }
            close_block(b, ob, pack64(o0, o1), range_mask(b << 6), false);
            ++n_eval;
        }
    };

    // Candidate data are fetched ahead: entry words two candidate blocks ahead, tallies (which
    // need the entry's example index) one block ahead of the visit.  Reading a tally early is within the
    // method's premise of outdated tallies.  The helper draws a round while the one before is worked through, so it reads
    // tallies when it draws and not a round before that: the older they are, the further machines swing in which all clauses step
    // together (live regression, 800 clauses of 400 features, s = 1.5, one launch: mean error 0.33 of T with tallies two rounds
    // ahead of the visit, 0.08 with one).
    auto load_ent = [&](int k0) { // packed (example << 1 | target), or -1 beyond the range
        const int k = k0 + lane;
        return k < k_hi ? list[k] : -1;
    };
    auto load_v = [&](int ent) {
        if (ent < 0) return 0;
        const int i = ent >> 1;
        return a.vhat ? a.vhat[(int64_t)i * d.m + c]
                      : __hip_atomic_load(&tally_c[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto load_y = [&](int ent) {
        if constexpr (REGR) return ent >= 0 ? a.y_regr[ent >> 1] : 0;
        else return 0;
    };
    // Paired slots: which bits of a feature word exist (0 in lanes that hold no word), one register per pair.
    constexpr bool PAIRED = SlotMap<WPL>::PAIRED;
    constexpr int NX = SlotMap<WPL>::NX;
    // With 20 slots the registers for that are not there: all pairs but the one that holds the last word are
    // whole or empty, which is a scalar.
    constexpr bool HOLD_VALID = PAIRED && WPL <= 16;
    uint32_t word_valid[HOLD_VALID ? NX : 1];
    const int last_pair = (d.Wf - 1) >> 6;
    const uint32_t narrow_valid = Map::held(0, lane, d.Wf) ? ((lane & 7) == d.Wf - 1 ? d.tailmask : ~0u) : 0u;
    if constexpr (PAIRED) {
#pragma unroll
        for (int k = 0; k < (HOLD_VALID ? NX : 1); ++k) {
            const int fw = (HOLD_VALID ? k : last_pair) * 64 + lane;
            word_valid[k] = fw < d.Wf ? (fw == d.Wf - 1 ? d.tailmask : ~0u) : 0u;
        }
    }
    // words of an example in lane = literal-word layout.  Slot geometry (which half, which bits exist) is recomputed from a
    // laundered index wherever it is needed: it is example-independent, and the compiler would otherwise keep it in VGPRs
    // for every slot.
    auto load_row = [&](int ii, uint32_t (&dst)[NX]) {
        const uint32_t *xrow = X + (int64_t)ii * d.Wf;
#pragma unroll
        for (int r = 0; r < NX; ++r) {
            uint32_t lw = (uint32_t)(r * 64 + lane);
            asm volatile("" : "+v"(lw));
            if constexpr (PAIRED) {
                dst[r] = xrow[min(lw, (uint32_t)d.Wf - 1u)];
            } else {
                const bool act = lw < (uint32_t)d.W;
                const uint32_t fw = act ? (lw >= (uint32_t)d.Wf ? lw - (uint32_t)d.Wf : lw) : 0u;
                dst[r] = xrow[fw];
            }
        }
    };
    // Where the masks change at most events (wide clauses: at nine of ten on the text-like workload), evaluating the
    // block's remaining examples after each change is most of the latency, and all but the few up to the next change is
    // thrown away.  There (hot) the outputs are taken one example at a time, lane = literal word, with the masks as they
    // stand in the registers: the outputs of the open block are known below position `known`, those of the examples
    // between two events are taken when the second one comes up (the first one's words are requested an event ahead),
    // and after a change the update loop leaves the violated literals of its own example.  Longer runs, and blocks
    // between rare changes, go through the entry list.  Where changes are neither frequent nor rare this loses (image-like data of
    // 3,300 features, s = 2: 0.96 of the speed; planted conjunctions, 5,500 features, s = 2: 0.97 to 1.0; calling changes frequent after one
    // at the last event or the one before only: 0.97, but s = 5 1.27 instead of 1.32).  Measured, before / now: 3,328 documents on 20,000 clauses of 10,000
    // features (116 entries) 32.6 / 21.4 ms; 1,600 on 1,000 clauses of them 1.93 / 1.20 ms; 832 on 16,000 of 20,000 features
    // 34.9 / 22.8 ms.  With 2 slots the entries are too few (14 to 20: 0.91 to 0.98 of the speed); with 3 slots it pays only
    // with a threshold of many blocks, where events take longer (s = 5 1.14 to 1.30, s = 2 0.89 to 0.98).  Never in regression,
    // whose masks change less often (speed with it / without, 4 to 10 slots, 60 to 5,000 clauses: s = 2 0.78 to 0.92 / 0.95 to 1.06 of the block
    // by block version before, s = 1.5 and 5 0.85 to 1.09 / 0.94 to 1.15).
    constexpr bool DIRECT = !REGR && (WPL >= 4 || (WPL == 3 && DEEP));
    // LATER: the outputs after a change, and those of a block just opened, are taken when the next event or the end of the
    // block needs them, whether changes are frequent or not: then every mask change goes one way.  Above 10 slots, where the registers of
    // the example would have to be kept through the update, the update gathers the violated literals and calm blocks are
    // evaluated at once.
    constexpr bool LATER = WPL <= 10;
    constexpr int DIRECT_ENTRIES = 12; // entries that cost a block about the latency of one example taken directly
    constexpr int DIRECT_CALM = 3;  // active events without a change after which changes count as rare
    std::conditional_t<LATER, int, bool> hot = 0; // changes are frequent
    int known = 64, calm = DIRECT_CALM + 1;
    auto direct_output = [&](const uint32_t (&x)[NX]) { // output of the clause on the example whose words are x
        uint32_t viol = 0u;
        if constexpr (PAIRED) {
#pragma unroll
            for (int k = 0; k < WPL / 2; ++k) viol |= bitselect(x[k], p[2 * k + 1][7], p[2 * k][7]);
        } else {
#pragma unroll
            for (int r = 0; r < WPL; ++r) viol |= p[r][7] & ~(r * 64 + lane >= d.Wf ? ~x[r] : x[r]);
        }
        return ballot(viol != 0u) == 0;
    };
    constexpr bool GAP_AHEAD = DIRECT && WPL <= 16; // with 20 slots the registers are not there
    uint32_t gap_row[NX]; // words of an example between two events, requested ahead
    int gap_example = -1;
    auto below = [](int bit) { return bit < 64 ? (1ull << bit) - 1ull : ~0ull; };
    auto know = [&](int upto) { // outputs of the open block below `upto`, or all of them, with the current masks
        if (!LATER && known >= upto) return;
        if (!hot || (upto - known - 1) * DIRECT_ENTRIES > nent) {
            obits = (obits & below(known)) | (list_outputs(cb) & ~below(known));
            known = 64;
            return;
        }
        for (; known < upto; ++known) {
            const int ii = (cb << 6) + known;
            if (!GAP_AHEAD || ii != gap_example) load_row(ii, gap_row);
            if (direct_output(gap_row)) obits |= 1ull << known;
        }
    };
    uint32_t xe = 0u, xe_cur = 0u; // TINY: words of the examples of the round's entries, and of the next round's
    auto load_xe = [&](int ent) {
        if constexpr (TINY) xe_cur = X[max(ent, 0) >> 1];
    };
    int ent_cur = load_ent(k_lo);
    load_xe(ent_cur);
    int v_cur = TEAM ? 0 : load_v(ent_cur);
    int y_cur = load_y(ent_cur);
    int ent_nxt = load_ent(k_lo + 64);

    auto draw_gates = [&](int k0, int &iv, uint64_t &fmask, uint64_t &tmask) { // the round of gate entries from k0 on
        const int ent = ent_cur, yv = y_cur;
        int v = v_cur;
        ent_cur = ent_nxt;
        if constexpr (TEAM) v = load_v(ent);
        else v_cur = load_v(ent_cur);
        y_cur = load_y(ent_cur);
        if constexpr (TINY) {
            xe = xe_cur;
            asm volatile("" : "+v"(xe)); // requested anew into the register that this round leaves
            load_xe(ent_cur);
        }
        ent_nxt = load_ent(k0 + 128);
        if constexpr (NARROW) { // everything requested so far arrives here, ahead of the atomics
            asm volatile("" : "+v"(bw_next[0]), "+v"(bw_next[1]), "+v"(bw_next[2]), "+v"(bw_next[3]), "+v"(bw_next[4]),
                         "+v"(bw_next[5]), "+v"(bw_next[6]), "+v"(bw_next[7]), "+v"(os_next0), "+v"(os_next1));
        }
        refresh_held();
        const bool valid = ent >= 0;
        iv = ent >> 1;
        bool target = (ent & 1) != 0;
        bool fire = false, open = false;
        if (valid) {
            int e, span;
            if (regr) {
                // regression: error of the clipped vote sum against the target, probability e/T;
                // below the target the clause is trained towards 1, above it towards 0
                const int vc = min(max(v, 0), T);
                target = vc < yv;
                e = target ? yv - vc : vc - yv;
                span = T;
            } else {
                const int vc = min(max(v, -T), T);
                e = target ? T - vc : T + vc; // Algorithm 1: error of the recorded vote sum
                span = 2 * T;
            }
            open = e > 0;
            if (open) {
                RngKey key = d.key;
                if (LAUNDER) asm volatile("" : "+s"(key.seed_lo), "+s"(key.seed_hi));
                const U4 r = draw(key, STREAM_GATE, 0, (uint32_t)g, (uint64_t)(uint32_t)iv, a.epoch);
                fire = (uint64_t)r.x * (uint64_t)span < ((uint64_t)e << 32);
            }
        }
        fmask = ballot(fire);
        tmask = ballot(target);
        n_draw += __builtin_popcountll(ballot(open));
        n_fired += __builtin_popcountll(fmask);
    };
    uint32_t *handed = draws + 2 * 64 * WPL * 64;
    if constexpr (TEAM) {
        if (helper) { // round k + 1 is drawn between barriers k and k + 1, in which the first wavefront works through round k
            for (int k0 = k_lo; k0 < k_hi; k0 += 64) {
                const int parity = (k0 >> 6) & 1;
                int iv = 0;
                uint64_t fmask = 0, tmask = 0;
                draw_gates(k0, iv, fmask, tmask);
                uint32_t *h = handed + parity * PAIR_ROUND;
                h[lane] = (uint32_t)iv;
                if (lane < 5)
                    h[64 + lane] = lane == 0 ? (uint32_t)fmask : lane == 1 ? (uint32_t)(fmask >> 32) : lane == 2 ? (uint32_t)tmask
                                 : lane == 3 ? (uint32_t)(tmask >> 32) : n_draw;
                deep_draw(fmask & (pos ? tmask : ~tmask), iv, 64, parity * 64 * WPL * 64);
                __syncthreads();
            }
            return;
        }
    }

    for (int k0 = k_lo;; k0 += 64) {
        const bool last = k0 >= k_hi; // all candidates done: one more round sweeps the remaining blocks
        uint64_t fmask = 0, tmask = 0;
        int iv = 0;
        if (!last) {
            if constexpr (TEAM) {
                __syncthreads();
                const uint32_t *h = handed + ((k0 >> 6) & 1) * PAIR_ROUND;
                iv = (int)h[lane];
                fmask = pack64(h[64], h[65]);
                tmask = pack64(h[66], h[67]);
                n_draw = (uint32_t)__builtin_amdgcn_readfirstlane((int)h[68]);
                n_fired += __builtin_popcountll(fmask);
            } else {
                draw_gates(k0, iv, fmask, tmask);
            }
        }

        // the row of the next fired example is requested while the current one is processed
        uint32_t xnext[NX];
        if (!NARROW && fmask) load_row(__builtin_amdgcn_readlane(iv, __builtin_ctzll(fmask)), xnext);
        n_ahead = n_used = 0;
        if constexpr (TINY) {
            const uint64_t t1 = fmask & (pos ? tmask : ~tmask);
            wave_lds_sync();
            if ((t1 >> lane) & 1ull) lmask[__builtin_amdgcn_mbcnt_hi((uint32_t)(t1 >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)t1, 0u))] = (uint32_t)iv;
            wave_lds_sync();
            t1_done = 0;
        }

        for (;;) {
            // next event: a fired candidate, or (after the last candidate) the end of the range
            const bool have = fmask != 0;
            int l = 0, ii = 0, B;
            if (have) {
                l = __builtin_ctzll(fmask);
                fmask &= fmask - 1;
                ii = __builtin_amdgcn_readlane(iv, l);
                B = ii >> 6;
            } else if (last) {
                B = end_block;
            } else {
                break;
            }

            // bring block B up: close the open block, refresh the outdated blocks in between
            if (cb != B) {
                uint32_t os_b0 = 0u, os_b1 = 0u;
                const bool ahead = NARROW && B == block_next;
                if (TINY && cb >= 0) obits = (obits & below(known)) | (narrow_eval(bw) & ~below(known));
                if constexpr (NARROW) {
                    if (ahead) {
#pragma unroll
                        for (int f = 0; f < 8; ++f) bw[f] = bw_next[f];
                        os_b0 = os_next0;
                        os_b1 = os_next1;
                    }
                }
                if (cb >= 0) {
                    if constexpr (DIRECT) {
                        const int end = min(64, i_end - (cb << 6));
                        if (!LATER || known < end) know(end);
                    }
                    close_block(cb, obits, ost, rmask, mask_changed);
                    next_block = cb + 1;
                    cb = -1;
                }
                const int lim = min(B, end_block);
                sweep(next_block, lim);
                next_block = max(next_block, lim);
                if (B < end_block) {
                    // open block B: previous outputs, range mask, evaluation with the current masks
                    cb = B;
                    const int b0 = B << 6;
                    rmask = range_mask(b0);
                    if constexpr (NARROW) {
                        if (!ahead) {
                            narrow_load(B, bw);
                            os_b0 = ostar_row[B << 1];
                            os_b1 = ostar_row[(B << 1) + 1];
                        }
                        narrow_keep();
                        if constexpr (TINY) known = 0; // outputs are taken when the masks change and when the block is closed
                        else obits = narrow_eval(bw);
                        ost = pack64(os_b0, os_b1);
                        block_next = -1;
                        if (B + 1 < end_block) { // nothing but the wavefront itself writes the stored outputs, and those of a
                            block_next = B + 1;  // later block only when it gets there
                            narrow_load(B + 1, bw_next);
                            os_next0 = ostar_row[(B << 1) + 2];
                            os_next1 = ostar_row[(B << 1) + 3];
                        }
                    } else {
                        const uint32_t *op = a.ostar + (int64_t)g * a.Qw + (b0 >> 5);
                        const uint32_t o0 = op[0], o1 = op[1];
                        ost = pack64(o0, o1);
                        if (DIRECT && (LATER || hot)) {
                            obits = 0;
                            known = max(0, i_begin - b0);
                        } else {
                            obits = list_outputs(B);
                            known = 64;
                        }
                    }
                    mask_changed = false;
                    ++n_eval;
                }
            }
            if (!have) break; // the range is finished

            const int bl = ii & 63;                  // position of the example in the open block
            const bool tgt = (tmask >> l) & 1;
            if constexpr (DIRECT) {
                if (!LATER || __builtin_expect(known <= bl, 0)) {
                    know(bl);
                    if (known == bl) {
                        if (direct_output(xnext)) obits |= 1ull << bl;
                        known = bl + 1;
                    }
                }
            }
            if constexpr (TINY) { // this event and those that follow in the open block
                for (;;) {
                    const uint32_t x = readlane(xe, l);
                    const bool target = (tmask >> l) & 1;
                    const uint64_t lit64 = (uint64_t)x | ((uint64_t)~x << 32);
                    const bool out = (inc64 & ~lit64) == 0, t1 = target == pos;
                    if (t1 || out) { // Type II feedback to a clause whose output is 0 changes nothing (Table 2)
                        if (LAZY && !have_planes) load_planes();
                        uint64_t up, dn;
                        if (t1) { // Type I feedback (Table 1)
                            ++n_type1;
                            if (n_used == n_ahead) {
                                narrow_draw((fmask | (1ull << l)) & (pos ? tmask : ~tmask), iv);
                                n_used = 0;
                            }
                            const int at = n_used << 3;
                            ++n_used;
                            const uint64_t ge = (uint64_t)readlane(ge_ahead, at) | ((uint64_t)readlane(ge_ahead, at + 1) << 32);
                            const uint64_t weak = valid64 & ~ge, boost = (uint64_t)d.boost | ((uint64_t)d.boost << 32);
                            const uint64_t fed = out ? lit64 : 0;
                            up = fed & valid64 & (ge | boost);
                            dn = weak & ~fed;
                        } else {  // Type II feedback (Table 2)
                            ++n_type2;
                            up = valid64 & ~lit64 & ~inc64;
                            dn = 0;
                        }
                        const int v = (int)sub_lanes(add_lanes(st, up), dn);
                        // ends of the state range as constants pay in regression only (N = 128: noisy XOR 536 us, with constants 552)
                        st = (uint32_t)min(max(v, FULL && REGR ? 0 : 128 - d.N), FULL && REGR ? 255 : 127 + d.N);
                        const uint64_t now = ballot(st >= 128u); // padding automata stay below
                        if (now != inc64) { // the conjunction changed: the examples before this one have the outputs of the old masks
                            obits = (obits & below(known)) | (narrow_eval(bw) & ~below(known));
                            known = ii & 63;
                            mask_changed = true;
                            n_listed = -1;
                            inc64 = now;
                        }
                    }
                    if (REGR || fmask == 0) break; // few events per block in regression: 400 clauses of 24 features 238 us, with the loop 247
                    const int next = __builtin_ctzll(fmask), in = __builtin_amdgcn_readlane(iv, next);
                    if (in >> 6 != cb) break;
                    l = next;
                    ii = in;
                    fmask &= fmask - 1;
                }
                continue;
            }
            const bool Cout = (obits >> bl) & 1;     // clause output on the state before the update
            // Type II feedback to a clause whose output is 0 changes nothing (Table 2): no automata needed
            if (LAZY && !have_planes && (tgt == pos || Cout)) load_planes();
            uint32_t changed = 0, viol = 0; // viol: included literals that are 0, after the update
            uint32_t xw[NX];
#pragma unroll
            for (int r = 0; r < NX; ++r) {
                xw[r] = NARROW ? 0u : xnext[r];
                // the next example is requested into the registers that this one leaves: where the compiler takes others and
                // copies them, the copies wait for the request.  200 to 3,000 clauses of 4,000 to 10,000 features,
                // time with that wait / without: 1.0 to 1.09
                if (DIRECT && LATER) asm volatile("" : "+v"(xw[r]));
            }
            if (!NARROW && fmask) {
                const int next = __builtin_amdgcn_readlane(iv, __builtin_ctzll(fmask));
                load_row(next, xnext);
                if constexpr (GAP_AHEAD) {
                    gap_example = -1;
                    if (hot && next > ii + 1) {
                        gap_example = ii + 1;
                        load_row(gap_example, gap_row);
                    }
                }
            }
            auto literal = [&](int r, uint32_t lw, uint32_t &valid) { // 0 on padding bits and idle lanes
                if constexpr (NARROW) {
                    valid = narrow_valid;
                    return (xw[0] ^ (lane & 8 ? ~0u : 0u)) & valid;
                } else if constexpr (PAIRED) {
                    if constexpr (HOLD_VALID) {
                        valid = word_valid[r / 2];
                    } else {
                        const int k = r / 2;
                        valid = (word_valid[0] & (k == last_pair ? ~0u : 0u)) | (k < last_pair ? ~0u : 0u);
                    }
                    return ((r & 1) ? ~xw[r / 2] : xw[r / 2]) & valid;
                } else {
                    const bool act = lw < (uint32_t)d.W;
                    const bool neg = lw >= (uint32_t)d.Wf;
                    const uint32_t fw = neg ? lw - (uint32_t)d.Wf : lw;
                    valid = act ? (fw == (uint32_t)d.Wf - 1u ? d.tailmask : ~0u) : 0u;
                    return (xw[r] ^ (neg ? ~0u : 0u)) & valid;
                }
            };
            const bool type1 = tgt == pos;
            if (!type1 && !Cout) continue; // Type II feedback to a clause whose output is 0 changes nothing (Table 2)
            if (type1) ++n_type1;
            else ++n_type2;
            if constexpr (NARROW) {
                xw[0] = narrow_row(bl);
                if (type1 && n_used == n_ahead) {
                    narrow_draw((fmask | (1ull << l)) & (pos ? tmask : ~tmask), iv);
                    n_used = 0;
                }
            }
            if constexpr (DEEP) {
                if (!TEAM && type1 && n_used == n_ahead) {
                    deep_draw((fmask | (1ull << l)) & (pos ? tmask : ~tmask), iv, train_draw_events(WPL), 0);
                    n_used = 0;
                }
            }
            constexpr bool SPLIT = !NARROW && train_split(WPL, ROOMY, DEEP);
            if (SPLIT && !type1) { // Type II feedback (Table 2): where the clause is 1 and the literal 0, push Exclude towards Include
#pragma unroll
                for (int r = 0; r < WPL; ++r) {
                    uint32_t lw = (uint32_t)Map::word(r, lane, d.Wf);
                    asm volatile("" : "+v"(lw));
                    uint32_t valid;
                    const uint32_t lit = literal(r, lw, valid);
                    uint32_t sp[8];
                    get_slot(p[r], sp);
                    const uint32_t old7 = sp[7];
                    ripple_inc(sp, ~lit & ~old7 & valid); // excluded automata (below the top bit) cannot overflow
                    changed |= sp[7] ^ old7;
                    if (DIRECT && !LATER) {
                        viol |= sp[7] & ~lit;
                        asm volatile("" : "+v"(viol));
                    }
                    if (WPL == 1) pin_planes(sp, changed);
                    put_slot(p[r], sp);
                }
            } else {
#pragma unroll
                for (int r = 0; r < WPL; ++r) {
                    uint32_t sp[8];
                    get_slot(p[r], sp);
                    const uint32_t old7 = sp[7];
                    uint32_t up, wk; // the automata that move towards Include and towards Exclude (disjoint)
                    // The literal-word index is laundered through an empty asm so that the
                    // compiler does not hoist the example-independent first Philox round of
                    // every slot and block out of the example loop (dozens of live VGPRs per slot).
                    uint32_t lw = (uint32_t)Map::word(r, lane, d.Wf);
                    asm volatile("" : "+v"(lw));
                    uint32_t valid;
                    const uint32_t lit = literal(r, lw, valid);
                    if (SPLIT || type1) { // Type I feedback (Table 1)
                    // bit-sliced comparison of 32 16-bit uniforms with thr, least significant bit first:
                    // ge = [u >= thr]; bit b of literal j's uniform is bit j of random word b;
                    // thr bit 1: ge &= w, thr bit 0: ge |= w, i.e. majority(w, ge, ~thr bit)
                    uint32_t ge = ge_init;
                    RngKey key = d.key;
                    uint32_t thr = d.thr;
                    if (WPL <= 2) asm volatile("" : "+s"(key.seed_lo), "+s"(key.seed_hi), "+s"(thr));
                    if constexpr (NARROW) {
                        ge = (uint32_t)__shfl((int)ge_ahead, dr_src + (n_used << (wps + 3)), 64);
                        ++n_used;
                    } else if constexpr (DEEP) {
                        ge = draws[((TEAM ? (k0 & 64) : 0) + n_used) * WPL * 64 + r * 64 + lane];
                        if (r == WPL - 1) ++n_used;
                    } else {
#pragma unroll
                        for (int t = train_least_block(WPL, ROOMY, REGR); t < 4; ++t) {
                            if (t >= first_blk) {
                                // With one or two slots, key and threshold are laundered as well (above):
                                // their derived constants (20 round keys, 16 comparator masks) are then
                                // computed by scalar instructions per slot instead of being kept for the
                                // whole kernel - kept, they overflow the scalar registers and come back
                                // through readlane, a vector instruction each, in the loop that is bound by
                                // vector issue (-5 % per epoch of an untrained machine).  With many slots the
                                // scalar work per slot costs more than the spills (measured +8 .. +20 %).
                                const U4 R = draw(key, STREAM_TYPE1, 4u * lw + (uint32_t)t, (uint32_t)g,
                                                  (uint64_t)(uint32_t)ii, a.epoch);
                                const uint32_t w[4] = {R.x, R.y, R.z, R.w};
#pragma unroll
                                for (int k = 0; k < 4; ++k) {
                                    const uint32_t K = ((thr >> (4 * t + k)) & 1u) ? 0u : ~0u;
                                    ge = majority3(w[k], ge, K);
                                }
                            }
                        }
                    }
                    up = 0u; // strong: literals that are 1 move towards Include with probability (s-1)/s (1 if boosted)
                    if (Cout) up = lit & (ge | d.boost) & ~at_value<FULL>(sp, a.sat.kmax, true);
                    // weak: everything else moves towards Exclude with probability 1/s
                    wk = (Cout ? ~lit : ~0u) & ~ge & valid & ~at_value<FULL>(sp, a.sat.kmin, false);
                    } else { // Type II feedback, as above
                        up = ~lit & ~old7 & valid;
                        wk = 0u;
                    }
                    ripple_updown(sp, up, wk);
                    changed |= sp[7] ^ old7;
                    if (DIRECT && !LATER) {
                        viol |= sp[7] & ~lit;
                        asm volatile("" : "+v"(viol));
                    }
                    // the planes are final here: without this the compiler moves the updates of all slots behind
                    // the last slot's draw, and old planes, direction masks and carries of every slot stay in
                    // registers until then
                    pin_planes(sp, changed);
                    put_slot(p[r], sp);
                    // keep the slots apart in the instruction schedule: interleaving them
                    // multiplies the live registers by the number of slots
                    if (WPL > 2) __builtin_amdgcn_sched_barrier(0);
                }
            }
            const bool moved = ballot(changed != 0u) != 0;
            if constexpr (DIRECT) {
                if constexpr (LATER) {
                    hot = moved ? (calm <= DIRECT_CALM ? 1 : 0) : (calm < DIRECT_CALM ? hot : 0);
                    calm = moved ? 0 : min(calm, DIRECT_CALM) + 1;
                } else if (moved) {
                    hot = calm <= DIRECT_CALM;
                    calm = 0;
                } else if (++calm > DIRECT_CALM) {
                    hot = 0;
                }
            }
            if (moved) { // the conjunction changed: re-evaluate this and the later examples of the block
                mask_changed = true;
                list_ok = false;
                n_listed = -1;
                if (DIRECT && (LATER || hot)) {
                    obits = (obits & below(bl)) | ((LATER ? direct_output(xw) : ballot(viol != 0u) == 0) ? 1ull << bl : 0ull);
                    known = bl + 1;
                } else {
                    uint64_t nb;
                    if constexpr (NARROW) nb = narrow_eval(bw);
                    else nb = list_outputs(cb);
                    obits = (obits & below(bl)) | (nb & ~below(bl));
                    known = 64;
                }
            }
        }
        if (last) break;
    }
    refresh_held();
    if (plo >= phi) plo = phi = 0;
    if (lane == 0) *reinterpret_cast<int4 *>(a.fresh + (int64_t)g * 4) = make_int4(plo, phi, slo, 0);

    if (TINY && (!LAZY || have_planes)) {
        uint32_t w = 0u; // lane b: plane b of the plain word, lane 8 + b of the negated one
#pragma unroll
        for (int b = 0; b < 8; ++b) {
            const uint64_t pl = ballot(((st >> b) & 1u) != 0u);
            w = lane == b ? (uint32_t)pl : lane == 8 + b ? (uint32_t)(pl >> 32) : w;
        }
        const int64_t lw = (int64_t)g * 2 + ((lane >> 3) & 1);
        if (lane < 16) a.planes[lw * 8 + (lane & 7)] = w;
        if (lane == 7 || lane == 15) a.inc[lw] = w;
    } else if (!LAZY || have_planes) { // a gate fired: the automata may have moved
#pragma unroll
        for (int r = 0; r < WPL; ++r) {
            const int lw = Map::word(r, lane, d.Wf);
            if (Map::held(r, lane, d.Wf)) {
                uint4 *dst = reinterpret_cast<uint4 *>(a.planes + ((int64_t)g * d.W + lw) * 8);
                const u32x8 t = p[r];
                dst[0] = make_uint4(t[0], t[1], t[2], t[3]);
                dst[1] = make_uint4(t[4], t[5], t[6], t[7]);
                a.inc[(int64_t)g * d.W + lw] = t[7];
            }
        }
    }
    for (int sh = 32; sh > 0; sh >>= 1) n_changes_v += __shfl_xor(n_changes_v, sh, 64);
    n_changes += n_changes_v;
    if (lane < 10) { // as store_counters, written out: called, it costs this kernel scalar registers (1 to 5 % of short launches)
        const uint32_t v = lane == 0 ? n_listed_blocks : lane == 1 ? n_fired : lane == 2 ? n_type1 : lane == 3 ? n_changes
                         : lane == 4 ? 0u : lane == 5 ? n_type2 : lane == 6 ? n_eval : lane == 7 ? n_draw
                         : lane == 8 ? (uint32_t)(i_end - i_begin) : ((!LAZY || have_planes) ? 1u : 0u);
        if (v) atomicAdd(&a.counters[(g & (COUNTER_SETS - 1)) * COUNTER_WIDTH + lane], (unsigned long long)v);
    }
}

template <int WPL, bool FULL, bool REGR, bool ROOMY, bool NARROW, bool DEEP, bool SPANS, bool TINY>
__global__ __launch_bounds__(64 * TRAIN_WAVES_MAX) __attribute__((amdgpu_waves_per_eu(train_min_waves(WPL, ROOMY || NARROW), train_max_waves(WPL, ROOMY)))) void k_train(const uint32_t *__restrict__ X, const uint32_t *__restrict__ XT,
                                                            const uint32_t *__restrict__ XB,
                                                            const int32_t *__restrict__ gate,
                                                            const int32_t *__restrict__ ngate, const TrainArgs a)
{
    extern __shared__ uint32_t lds[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    constexpr bool TEAM = train_team(WPL, ROOMY, DEEP, NARROW); // one clause per workgroup
    const int slot = a.slot_lo + (TEAM ? (int)blockIdx.x : (int)(blockIdx.x * (blockDim.x >> 6)) + wave);
    if (slot >= a.slot_hi) return; // whole wavefront (TEAM: all of them, and all walk the same rounds with one barrier in each)
    const int g = __builtin_amdgcn_readfirstlane(a.order[slot]);
    const int k_hi = __builtin_amdgcn_readfirstlane(ngate[g / a.d.n]);
    const bool many = k_hi >= TRAIN_EAGER_CANDIDATES;
    if constexpr (SPANS) {
        if (many) train_spans<WPL, FULL, false, ROOMY, DEEP>(X, XT, XB, gate, k_hi, a, lds, g, lane, wave);
        else train_spans<WPL, FULL, true, ROOMY, DEEP>(X, XT, XB, gate, k_hi, a, lds, g, lane, wave);
    } else {
        // From 6 slots on one version serves both, which loads up front where the gates are many: the check per event is
        // nothing beside the event, and a quiet pass moves no automata (16,000 clauses of 20,000 features, T = n / 40: 430 -> 300 us)
        const bool helper = TEAM && wave != 0;
        if (WPL <= 4 && many) train_clause<WPL, FULL, REGR, false, NARROW, ROOMY, DEEP, TINY>(X, XT, XB, gate, k_hi, a, lds, g, lane, wave, helper);
        else train_clause<WPL, FULL, REGR, true, NARROW, ROOMY, DEEP, TINY>(X, XT, XB, gate, k_hi, a, lds, g, lane, wave, helper);
    }
}

} // namespace tsetlin

#endif

// Launch of the training kernel: one function per form of it.  The forms are compiled in several translation units
// (tm_train_part.hip), because together they take minutes.
#ifndef TM_TRAIN_LAUNCH_HPP_
#define TM_TRAIN_LAUNCH_HPP_
#include "tm_dims.hpp"
#include "tm_kernels_prep.hpp"
#include "tm_kernels_train.hpp"

namespace tsetlin {

constexpr int ONE_PER_SIMD = 1536; // most clauses for which "about one per SIMD" holds (256 CUs of four)

struct TrainPtrs {
    const uint32_t *X, *XT, *XB;
    const int32_t *gate, *ngate;
};

// Live classification passes with T below a quarter of n.  An error of one vote moves the expected feedback of a class by n / 2T
// clauses; where that is several, a machine swings about its margin, the more the further its clauses walk in step, reading
// tallies that all of them are about to correct alike.  How far they do depends on how long the clauses take between two looks at the
// tallies, and the span forms, in which they take much the same time, do worse (test accuracy of late epochs, block by block / span by span;
// T / n = 1 / 20: 2 x 2,000 clauses of 900 bag-of-words features 0.995 / 0.93, 2 x 1,000 of 2,500 0.92 / 0.75, 10 x 400 of 784 noisy pixels
// 0.994 / 0.987, 4 x 1,000 of 2,500 0.61 / 0.95; 1 / 5, 2 x 100 of 64 features, which a team would take, 0.985 / 0.981).  From a tenth of n on they
// are alike elsewhere (24 machines of 700 to 10,000 features: within 0.002, gates fired within 5 %), from a quarter on everywhere.
inline bool train_swings(const TrainArgs &a) { return !a.vhat && !a.y_regr && 4 * (int64_t)a.d.T < a.d.n; }

// With clauses_per_group nothing is launched; it receives how many clauses a workgroup of the launch would hold.
template <int WPL, bool ROOMY, bool DEEP, bool NARROW>
void launch_train_form(const TrainPtrs &p, TrainArgs a, bool full, hipStream_t st, int *clauses_per_group)
{
    const bool regr = a.y_regr != nullptr;
    constexpr bool HAS_SPANS = train_has_spans(WPL, ROOMY, DEEP, NARROW), team = train_team(WPL, ROOMY, DEEP, NARROW);
    const int64_t entries = 2 * (int64_t)(a.i_end - a.i_begin) / a.d.m; // of a class's gate list where every gate is open
    const bool spans = HAS_SPANS && !regr && !train_swings(a) && entries >= train_spans_from(WPL, ROOMY, DEEP);
    if (!NARROW) {
        if (SlotMap<WPL>::PAIRED) a.lds_mask_words = 0; // the masks come out of the slots
        a.lds_draw_off = (a.lds_mask_words + a.lds_off_words + 2 * (a.d.Wf + EVAL_PAD) + 3) & ~3;
        if (spans) { // the literal list takes the place of the entries; then the events of a round, their rows and draws
            a.lds_draw_off = a.lds_draw_off > TRAIN_LIT_MAX + SPAN_LIT_PAD ? a.lds_draw_off : TRAIN_LIT_MAX + SPAN_LIT_PAD;
            a.lds_wave_words = a.lds_draw_off + span_lds_words(WPL, team, DEEP);
        } else {
            a.lds_wave_words = a.lds_draw_off + (DEEP ? train_draw_words(WPL, team) : 0) + (WPL <= 4 ? TRAIN_LIT_MAX + LIT_PAD : 0);
        }
    }
    // Clauses per workgroup: one of several wavefronts (team), else one per wavefront, and these do not interact.  A workgroup's
    // slots are handed on only when its slowest clause is done, so one is best once every SIMD holds several wavefronts (speed against
    // two: 3,000 to 20,000 clauses of 20,000 features 1.09 to 1.2, of 10,000 features 1.0 to 1.06; 3,000 and 8,000 of 300 to 784 features 1.15 and
    // 1.09, 20,000 of them 1.0), and two
    // where clauses have few gate entries to work through and few slots (20,000 clauses of 300 to 784 features, 200 entries: one 0.98 of
    // two).  With about one clause per SIMD four are better: they land on the four SIMDs of a CU, while two workgroups of two may share a
    // pair of SIMDs (1,000 clauses: 4.0 ms per epoch against 5.0 ms).  Live passes that swing hold two: neighbours, one of either polarity,
    // then walk side by side (T = 0.05 and 0.075 n, 2 x 3,000 clauses of 4,100 bag-of-words features: test accuracy 0.944 and 0.917, one
    // clause per workgroup 0.815 and 0.901).
    // Single wavefronts spread unevenly over the SIMDs, depending on what ran before: one too many on some costs little where a SIMD
    // gets three or more than four, but not where it gets two or four, which pairs fill evenly (speed of one against two, best and worst after
    // different work: 2,000 clauses of 5,000 to 10,000 features 1.04 and 0.82; 4,000 of 1,500 1.0 and 0.84; 3,000 of 300 to 2,500 1.1 to 1.2).  That
    // goes for forms of which a SIMD holds as many.
    const int clauses = a.slot_hi - a.slot_lo;
    const bool even = (WPL <= 10 && clauses <= 2 * 1024) || (WPL <= 4 && clauses > 3 * 1024 && clauses <= 4 * 1024);
    const int tw = team ? 1 : a.d.C <= ONE_PER_SIMD ? TRAIN_WAVES_MAX : even || train_swings(a) || (WPL <= 2 && entries < 600) ? 2 : 1;
    if (clauses_per_group) {
        *clauses_per_group = tw;
        return;
    }
    const size_t lds = (size_t)a.lds_wave_words * tw * 4;
    const dim3 grid((unsigned)((a.slot_hi - a.slot_lo + tw - 1) / tw)), block(64 * (team ? (spans ? 2 + TEAM_DRAWERS : 2) : tw));
    constexpr bool CLASSES_ONLY = WPL == 1 && !ROOMY && !NARROW; // regression of one slot takes the roomy forms (launch_train_slots)
    auto launch = [&](auto kernel) { hipLaunchKernelGGL(kernel, grid, block, lds, st, p.X, p.XT, p.XB, p.gate, p.ngate, a); };
    auto choose = [&](auto spans_too, auto tiny) {
        constexpr bool SPANS = decltype(spans_too)::value;
        constexpr bool TINY = decltype(tiny)::value;
        if (!regr) return full ? launch(k_train<WPL, true, false, ROOMY, NARROW, DEEP, SPANS, TINY>) : launch(k_train<WPL, false, false, ROOMY, NARROW, DEEP, SPANS, TINY>);
        if constexpr (!CLASSES_ONLY && !SPANS)
            return full ? launch(k_train<WPL, true, true, ROOMY, NARROW, DEEP, false, TINY>) : launch(k_train<WPL, false, true, ROOMY, NARROW, DEEP, false, TINY>);
    };
    if constexpr (HAS_SPANS) {
        if (spans) return choose(std::true_type{}, std::false_type{});
    }
    if constexpr (NARROW) {
        if (a.d.Wf <= 1) return choose(std::false_type{}, std::true_type{});
    }
    choose(std::false_type{}, std::false_type{});
}

// The forms there are: F(part, register slots, roomy, deep, narrow)
#define TM_TRAIN_FORMS(F)                                                                                                      \
    F(1, 1, false, false, true) F(1, 1, true, false, false) F(1, 1, false, false, false) F(1, 1, true, true, false)            \
    F(1, 1, false, true, false)                                                                                                \
    F(2, 2, true, false, false) F(2, 2, false, false, false) F(2, 2, true, true, false) F(2, 2, false, true, false)                                        \
    F(2, 3, true, false, false) F(2, 3, false, false, false)                                                                   \
    F(3, 3, true, true, false) F(3, 3, false, true, false) F(3, 4, true, false, false) F(3, 4, false, false, false)            \
    F(4, 4, false, true, false) F(4, 6, true, false, false) F(4, 6, false, false, false) F(4, 6, true, true, false)            \
    F(4, 6, false, true, false)                                                                                                \
    F(5, 8, true, false, false) F(5, 8, false, false, false) F(5, 8, true, true, false) F(5, 8, false, true, false)            \
    F(6, 10, true, false, false) F(6, 10, false, false, false) F(6, 10, true, true, false) F(6, 10, false, true, false)        \
    F(7, 12, false, false, false) F(7, 12, false, true, false) F(7, 16, false, false, false)                                   \
    F(8, 16, false, true, false) F(8, 20, false, false, false) F(8, 20, false, true, false)

} // namespace tsetlin

#endif

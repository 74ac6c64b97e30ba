// The training kernel for clauses of up to three register slots: outputs taken span by span.
// Included by tm_kernels_train.hpp.
#ifndef TM_KERNELS_TRAIN_SPANS_HPP_
#define TM_KERNELS_TRAIN_SPANS_HPP_

namespace tsetlin {

constexpr int SPAN_LIT_PAD = 16; // entries of the all-ones row after the literal list

// Rows of fired examples that a wavefront takes into LDS at a time.
__host__ __device__ constexpr int span_rows(int wpl) { return wpl == 1 ? 16 : 8; }

// LDS words of a wavefront (a team: of the workgroup) beside what evaluates spans.
__host__ __device__ constexpr int span_lds_words(int wpl, bool team, bool deep)
{
    return team ? 4 * TEAM_HANDED + 2 * TEAM_ROUND * 32 + (2 * TEAM_ROUND + 1) * 64 + TEAM_DRAWERS * 4 * DRAW_RING
                : 64 + span_rows(wpl) * 32 * wpl + (deep ? train_draw_events(wpl) * wpl * 64 + 4 * DRAW_RING : 0);
}

// Outputs that wait for a change of the masks are taken anyway once so many examples wait at the end of a round of gate entries (2,048 are one
// pass of a sweep); their tallies wait as long.  A round covers as many examples as its entries are apart - with 64 of ten classes' entries
// 320 where every gate is open, thousands where few are -, so up to that many more may wait.  Looking before every event
// instead holds live training back (10 x 400 clauses of 784 features, T = 20: epoch 0.38 ms, with a bound of 512 examples 0.46, of 64
// 0.64) and it learns no better for it (test accuracy 0.98, 0.98 and 0.90).
constexpr int SPAN_MOST = 2048;
// Most examples of a span that are taken row by row.  Where masks change at every second event, as young machines' and those of bags of words
// do, a span is a handful of examples, and a list of literals or entries for a block of 64 is not worth making for it: the rows come eight
// (four) at a time, and a row costs what a row in LDS does.  First epoch and sum of the first eight, a block for every span / row by row: 2 x 400
// clauses of 1,000 bag-of-words features, s = 5 2.14, 12.4 / 1.54, 9.4 ms; 2 x 8,000, s = 2 7.5, 35.8 / 6.4, 31.6; 2 x 200 of 1,500 5.5, 34.7 /
// 4.5, 29.7; 2 x 6,000 of 3,000, s = 5 9.6, 75.0 / 8.2, 59.9; machines of noisy images 0.99 to 1.03 of the time.  24 instead of 16: the same
// within 2 %.  The other way, a clause whose masks change often taken block by block by the same
// kernel, costs settled machines up to 3 % with one slot and 19 % with three (scalar registers).
constexpr int SPAN_DIRECT = 16;

// One wavefront = one clause of class c, as train_clause below, but no block of examples is ever opened.  The rows of the fired
// examples of a round go into LDS a handful at a time, and the output that an example's feedback needs comes from there: the
// included literals that are 0 in it cost one operation per slot and a ballot, for eight rows side by side, so that Type II events
// of a clause whose output is 0 (nearly all of them) are dropped before the loop over the events.  The outputs of all
// examples since the last change of the masks (`pend`) are taken when the masks change next, at the end of the launch, or when SPAN_MOST
// of them wait after a round: one walk of the literal list over the rows of XB, lane = word of 32 examples, or up to SPAN_DIRECT of them from their
// rows.  Masks change at 2 to 3 % of
// the feedback events of an image-like machine with every gate open: 60 to 90 walks of 18 literals take the place of 1,000
// evaluations of blocks of 64 examples, which were a sixth of the vector instructions of such a pass.
// What bounds it is vector issue (0.85 of the peak rate).  20,000 clauses of 784 features, 60,000 examples, s = 10: vector
// instructions 12.2e9 -> 9.4e9, scalar 8.3e9 -> 6.0e9, 24.4 -> 16.9 ms.
// With about one clause per SIMD a team of four wavefronts takes a clause (TEAM below): 1,000 clauses of 784 features 2.72 -> 1.21 ms.
template <int WPL, bool FULL, bool LAZY, bool ROOMY, bool DEEP>
__device__ __forceinline__ void train_spans(const uint32_t *__restrict__ X, const uint32_t *__restrict__ XT,
                                            const uint32_t *__restrict__ XB, const int32_t *__restrict__ gate,
                                            const int k_hi, const TrainArgs &a, uint32_t *lds, const int g,
                                            const int lane, const int wave)
{
    constexpr bool TEAM = train_team(WPL, ROOMY, DEEP, false);
    using Map = SlotMap<WPL>;
    constexpr bool PAIRED = Map::PAIRED;
    constexpr int NX = Map::NX;
    const Dims &d = a.d;
    // LDS of the wavefront (TEAM: of the workgroup): what evaluates spans - the literal list or, for clauses of more literals than
    // it holds, entries for eval64 - and then the events of a round, rows and draws.
    uint32_t *lds_w = lds + (TEAM ? 0 : wave) * a.lds_wave_words;
    uint32_t *llist = lds_w, *lmask = lds_w;   // [TRAIN_LIT_MAX + SPAN_LIT_PAD]; [W] include masks, literal-word order
    uint32_t *eoff = lmask + a.lds_mask_words; // [Wf + EVAL_PAD] (rounded to 4 words)
    uint2 *emask = reinterpret_cast<uint2 *>(eoff + a.lds_off_words);
    uint32_t *lds_draw = lds_w + a.lds_draw_off;

    const int c = g / d.n;
    constexpr bool LAUNDER = !ROOMY; // key and threshold, see train_clause
    const bool pos = ((g - c * d.n) & 1) != 0; // odd index within the class: positive polarity
    const int sign = pos ? 1 : -1;
    const int T = d.T;
    const int i_begin = a.i_begin, i_end = a.i_end;
    const int32_t *list = gate + (int64_t)c * a.qp;
    const int32_t *tally_c = a.tally + (int64_t)c * a.qp;
    uint32_t n_fired = 0, n_type1 = 0, n_type2 = 0, n_draw = 0, n_changes = 0;

    // ---- gates: 64 entries of the gate list at a time (TEAM: 32, see below), lane = entry ----
    auto load_ent = [&](int k) { return k < k_hi ? list[k] : -1; };
    auto load_v = [&](int ent) {
        if (ent < 0) return 0;
        const int i = ent >> 1;
        return a.vhat ? a.vhat[(int64_t)i * d.m + c]
                      : __hip_atomic_load(&tally_c[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto gate_of = [&](int ent, int v, bool &target) { // draws the gates of a round
        target = (ent & 1) != 0;
        bool fire = false, open = false;
        if (ent >= 0) { // Algorithm 1: error of the recorded vote sum, probability e/2T
            const int vc = min(max(v, -T), T), e = target ? T - vc : T + vc;
            open = e > 0;
            if (open) {
                RngKey key = d.key;
                if (LAUNDER) asm volatile("" : "+s"(key.seed_lo), "+s"(key.seed_hi));
                const U4 r = draw(key, STREAM_GATE, 0, (uint32_t)g, (uint64_t)(uint32_t)(ent >> 1), a.epoch);
                fire = (uint64_t)r.x * (uint64_t)(2 * T) < ((uint64_t)e << 32);
            }
        }
        n_draw += __builtin_popcountll(ballot(open));
        return fire;
    };

    // ---- Type I draws ahead of the events (DEEP), see train_clause ----
    constexpr int ROUND = TEAM ? TEAM_ROUND : 64;
    constexpr int PITCH = 32 * WPL;                                         // words of a row
    constexpr int STAGED = TEAM ? TEAM_ROUND : span_rows(WPL);              // rows in LDS at a time
    uint32_t *handed = lds_draw;                                            // TEAM: [round & 3][TEAM_HANDED], otherwise [64]: {example << 1 | Type I} of the fired entries; TEAM: then their number, open gates, end of the round
    uint32_t *rows = handed + (TEAM ? 4 * TEAM_HANDED : 64);                // TEAM: [round parity] of [STAGED][PITCH]: words of the fired examples
    uint32_t *draws = rows + (TEAM ? 2 : 1) * STAGED * PITCH;               // [event][slot][lane]: u >= thr (TEAM: [round parity] of these)
    uint4 *ring = reinterpret_cast<uint4 *>(draws + (TEAM ? 2 * TEAM_ROUND + 1 : train_draw_events(WPL)) * WPL * 64) // {4 lw, undecided literals, example, index in draws}
                  + (TEAM ? max(wave - 2, 0) * DRAW_RING : 0);
    int head = 0, cnt = 0; // of the ring
    auto deep_rest = [&](int n) { // the next n words of the ring, at most 32
        const uint4 it = ring[(head + (lane & 31)) & (DRAW_RING - 1)];
        const bool low = lane >= 32;
        RngKey key = d.key;
        if (LAUNDER) asm volatile("" : "+s"(key.seed_lo), "+s"(key.seed_hi));
        const U4 R = draw(key, STREAM_TYPE1, it.x + (low ? 0u : 1u), (uint32_t)g, (uint64_t)it.z, a.epoch);
        const uint32_t w[4] = {R.x, R.y, R.z, R.w};
        const uint32_t nib = ~(low ? d.thr : d.thr >> 4);
        uint32_t d0 = 0u, d1 = ~0u; // block 1: above, not below; block 0: d1, not below
#pragma unroll
        for (int k = 0; k < 4; ++k) {
            const uint32_t K = (uint32_t)__builtin_amdgcn_sbfe((int)nib, k, 1);
            d0 = majority3(w[k], d0, K);
            d1 = majority3(w[k], d1, K);
        }
        const uint32_t ge_low = (uint32_t)__shfl_xor((int)d1, 32, 64);
        if (lane < n) draws[it.w] |= it.y & (d0 | (d1 & ge_low));
        wave_lds_sync();
        head += n;
        cnt -= n;
    };
    // With one slot what the first two rounds make of a block number is the same for every example and stays in registers.
    PhiloxStart start2 = {0, 0, 0}, start3 = {0, 0, 0};
    const uint32_t word_held = Map::held(0, lane, d.Wf) ? ~0u : 0u;
    if constexpr (WPL == 1) {
        const uint32_t c4 = 4u * (uint32_t)Map::word(0, lane, d.Wf);
        start2 = philox_start(c4 + 2u, STREAM_TYPE1, a.epoch, d.key);
        start3 = philox_start(c4 + 3u, STREAM_TYPE1, a.epoch, d.key);
    }
    // Upper two blocks of the events t1 (bits: lanes of ev) on the examples ev >> 1, at most `most` of them, every stride-th of them
    // beginning with the first-th; results of the k-th from draws[place + 64 k WPL] on.  Returns how many events that were.
    auto deep_draw = [&](uint64_t t1, int ev, int most, int first, int stride, int place) {
        RngKey key = d.key;
        uint32_t nthr = ~d.thr;
        if (LAUNDER) asm volatile("" : "+s"(key.seed_lo), "+s"(key.seed_hi), "+s"(nthr));
        const int slots = PAIRED ? 2 * ((d.Wf + 63) >> 6) : WPL;
        int n = 0;
        for (; n < most && t1; ++n) {
            const uint32_t id = readlane((uint32_t)ev, __builtin_ctzll(t1)) >> 1;
            t1 &= t1 - 1;
            if (TEAM) {
                if (n != first) continue;
                first += stride;
            }
#pragma unroll 1
            for (int r = 0; r < slots; ++r) {
                const uint32_t c4 = 4u * (uint32_t)Map::word(r, lane, d.Wf);
                U4 A, B;
                if constexpr (WPL == 1) {
                    A = draw_from(start2, key, (uint32_t)g, id);
                    B = draw_from(start3, key, (uint32_t)g, id);
                } else {
                    A = draw(key, STREAM_TYPE1, c4 + 2u, (uint32_t)g, (uint64_t)id, a.epoch);
                    B = draw(key, STREAM_TYPE1, c4 + 3u, (uint32_t)g, (uint64_t)id, a.epoch);
                }
                const uint32_t w[8] = {A.x, A.y, A.z, A.w, B.x, B.y, B.z, B.w};
                uint32_t d0 = 0u, d1 = ~0u;
#pragma unroll
                for (int k = 0; k < 8; ++k) {
                    const uint32_t K = (uint32_t)__builtin_amdgcn_sbfe((int)nthr, 8 + k, 1);
                    d0 = majority3(w[k], d0, K);
                    d1 = majority3(w[k], d1, K);
                }
                const uint32_t held = WPL == 1 ? word_held : Map::held(r, lane, d.Wf) ? ~0u : 0u;
                const uint32_t undecided = (uint32_t)__builtin_amdgcn_bitop3_b32(d0, d1, held, 0x28); // (d0 ^ d1) & held
                const uint32_t at = (uint32_t)(place + (n * WPL + r) * 64 + lane);
                draws[at] = d0;
                const uint64_t b = ballot(undecided != 0u);
                const int pre = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                if (undecided) ring[(head + cnt + pre) & (DRAW_RING - 1)] = make_uint4(c4, undecided, id, at);
                cnt += __builtin_popcountll(b);
                wave_lds_sync();
                while (cnt >= 32) deep_rest(32);
            }
        }
        if (cnt) deep_rest(cnt);
        return n;
    };

    // ---- the other wavefronts of a team ----
    // One barrier per round of 32 gate entries.  While the first wavefront works through round t, the second draws the gates of round
    // t + 2 and brings the rows of the fired examples of round t + 1 into LDS, and the others share the Type I draws of round t + 1.
    const int rounds = (k_hi + ROUND - 1) / ROUND;
    if constexpr (TEAM) {
        // A SIMD gives way to its oldest wavefront: with four teams on a CU the youngest one's first wavefront waited for everybody's
        // draws and its clause took 1.5 instead of 0.9 ms, and so did the launch.
        if (wave == 0) __builtin_amdgcn_s_setprio(3);
        else if (wave == 1) __builtin_amdgcn_s_setprio(2);
        if (wave == 1 && rounds) {
            const int half = lane >> 5, word = min(lane & 31, d.Wf - 1);
            const int32_t *vsrc = a.vhat ? a.vhat + c : tally_c;
            const int64_t vstride = a.vhat ? d.m : 1;
            int ent = list[min(lane, k_hi - 1)]; // of the next round, past the end the last one
            for (int t = -2; t < rounds - 1; ++t) {
                const int k = (t + 2) * ROUND + lane;
                const bool live = lane < ROUND && k < k_hi;
                const int ent_now = ent;
                const int v = __hip_atomic_load(&vsrc[(int64_t)(ent >> 1) * vstride], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                ent = list[min(k + ROUND, k_hi - 1)];
                const uint32_t *h1 = handed + ((t + 1) & 3) * TEAM_HANDED;
                const int nf = t >= -1 ? __builtin_amdgcn_readfirstlane((int)h1[ROUND]) : 0;
                uint32_t x[ROUND / 2];
#pragma unroll
                for (int u = 0; u < ROUND / 2; ++u) // two rows a load
                    if (2 * u < nf) x[u] = X[(int64_t)(h1[min(2 * u + half, nf - 1)] >> 1) * d.Wf + word];
                if (t + 2 < rounds) {
                    bool target;
                    const bool fire = gate_of(live ? ent_now : -1, v, target);
                    const uint64_t f = ballot(fire);
                    const int pre = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(f >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)f, 0u));
                    uint32_t *h = handed + ((t + 2) & 3) * TEAM_HANDED;
                    if (fire) h[pre] = (uint32_t)(ent_now & ~1) | (target == pos ? 1u : 0u);
                    const uint32_t end = (readlane((uint32_t)ent_now, min(ROUND, k_hi - (t + 2) * ROUND) - 1) >> 1) + 1u;
                    if (lane < 3) h[ROUND + lane] = lane == 0 ? (uint32_t)__builtin_popcountll(f) : lane == 1 ? n_draw : end;
                }
                uint32_t *to = rows + ((t + 1) & 1) * STAGED * PITCH;
#pragma unroll
                for (int u = 0; u < ROUND / 2; ++u)
                    if (2 * u < nf) to[u * 64 + lane] = x[u];
                __syncthreads();
            }
        } else if (wave >= 2 && rounds) {
            for (int t = -2; t < rounds - 1; ++t) {
                if (t >= -1) {
                    const uint32_t *h = handed + ((t + 1) & 3) * TEAM_HANDED;
                    const uint32_t ev = h[lane & (ROUND - 1)];
                    const int nf = __builtin_amdgcn_readfirstlane((int)h[ROUND]);
                    deep_draw(ballot((ev & 1u) != 0u && lane < nf), (int)ev, 64, wave - 2, TEAM_DRAWERS, ((t + 1) & 1) * ROUND * 64);
                }
                __syncthreads();
            }
        }
        if (wave != 0) return;
    }

    // ---- the clause ----
    u32x8 p[WPL];
#pragma unroll
    for (int r = 0; r < WPL; ++r) {
        const int lw = Map::word(r, lane, d.Wf);
        u32x8 t = {0u, 0u, 0u, 0u, 0u, 0u, 0u, 0u};
        if (Map::held(r, lane, d.Wf)) t[7] = a.inc[(int64_t)g * d.W + lw];
        p[r] = t;
    }
    bool have_planes = false;
    auto load_planes = [&]() { // until the first feedback the include masks are all that is needed
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
    if (!LAZY) load_planes();
    // sign and existing bits of the literal words a lane holds
    uint32_t neg[WPL], valid[WPL];
#pragma unroll
    for (int r = 0; r < WPL; ++r) {
        const int lw = Map::word(r, lane, d.Wf), fw = lw >= d.Wf ? lw - d.Wf : lw;
        neg[r] = PAIRED ? ((r & 1) ? ~0u : 0u) : lw >= d.Wf ? ~0u : 0u;
        valid[r] = Map::held(r, lane, d.Wf) ? (fw == d.Wf - 1 ? d.tailmask : ~0u) : 0u;
    }
    uint32_t row_at[NX]; // where a lane finds its words in a row: the feature words of its literal words
#pragma unroll
    for (int r = 0; r < NX; ++r) {
        const int slot = PAIRED ? 2 * r : r, lw = Map::word(slot, lane, d.Wf);
        row_at[r] = Map::held(slot, lane, d.Wf) ? (uint32_t)(lw >= d.Wf ? lw - d.Wf : lw) : 0u;
    }
    // ---- outputs, tallies and stored outputs of a span of examples ----
    // Stored outputs that may differ from the clause's present ones lie in [plo, phi) and [slo, q); everything else needs neither
    // evaluation nor refresh (o = o* there).
    int plo, phi, slo;
    {
        const int4 f = *reinterpret_cast<const int4 *>(a.fresh + (int64_t)g * 4);
        plo = __builtin_amdgcn_readfirstlane(f.x);
        phi = __builtin_amdgcn_readfirstlane(f.y);
        slo = __builtin_amdgcn_readfirstlane(f.z);
    }
    int n_listed = 0, nent = 0; // literals in the list, entries for eval64
    enum { NOTHING, LIST, ENTRIES } have = NOTHING; // which of them LDS holds, of the present masks
    uint32_t n_eval = 0, n_listed_blocks = 0, n_changes_v = 0; // the first two in examples until they are stored
    const char *xb_base = reinterpret_cast<const char *>(XB);
    uint32_t *ostar_row = a.ostar + (int64_t)g * a.Qw;
    // Examples [lo, hi) from the literal list, 16 loads in flight: two words of 32 examples per lane with eight literals at a
    // time, or, for a span of up to 2,048 examples, one word with sixteen.
    auto sweep = [&](int lo, int hi) {
        const int w_end = (hi + 31) >> 5;
        const bool one = w_end - (lo >> 5) <= 64;
        const int step = one ? 64 : 128, group = one ? 16 : 8;
        const uint32_t *second = llist + (one ? 8 : 0);
        for (int w0 = lo >> 5; w0 < w_end; w0 += step) {
            uint32_t rm[2], woff[2], ost[2], accv[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int w = w0 + (one ? 0 : u * 64) + lane, e0 = w << 5;
                const bool act = w < w_end;
                const int from = min(max(lo - e0, 0), 32), to = min(max(hi - e0, 0), 32);
                rm[u] = 0u; // examples of the word that belong to the span
                if (act && to > from) rm[u] = (to == 32 ? ~0u : (1u << to) - 1u) & ~((1u << from) - 1u);
                woff[u] = act ? (uint32_t)w * 4u : 0u;
                ost[u] = act ? ostar_row[w] : 0u;
                accv[u] = rm[u];
            }
            for (int k = 0; k < n_listed; k += group) { // the list is padded with the all-ones row
                uint32_t x[2][8];
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const uint32_t *at = (u ? second : llist) + k;
#pragma unroll
                    for (int j = 0; j < 8; j += 4) {
                        const uint4 e = *reinterpret_cast<const uint4 *>(at + j);
                        x[u][j] = *reinterpret_cast<const uint32_t *>(xb_base + (e.x + woff[u]));
                        x[u][j + 1] = *reinterpret_cast<const uint32_t *>(xb_base + (e.y + woff[u]));
                        x[u][j + 2] = *reinterpret_cast<const uint32_t *>(xb_base + (e.z + woff[u]));
                        x[u][j + 3] = *reinterpret_cast<const uint32_t *>(xb_base + (e.w + woff[u]));
                    }
                }
#pragma unroll
                for (int u = 0; u < 2; ++u) accv[u] &= x[u][0] & x[u][1] & x[u][2] & x[u][3] & x[u][4] & x[u][5] & x[u][6] & x[u][7];
                // a clause of many literals is false on all examples of the pass after a few rounds
                if (n_listed > 32 && ballot((one ? accv[0] & accv[1] : accv[0] | accv[1]) != 0u) == 0) break;
            }
            if (one) {
                accv[0] &= accv[1];
                rm[1] = 0u;
            }
#pragma unroll
            for (int u = 0; u < 2; ++u) {
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
    };
    auto blocks = [&](int lo, int hi) { // examples [lo, hi) block by block: clauses of more literals than the list holds
        for (int b = lo >> 6; b < (hi + 63) >> 6; ++b) {
            const int b0 = b << 6;
            const uint32_t *op = ostar_row + (b << 1);
            const uint32_t o0 = op[0], o1 = op[1];
            const uint64_t ob = eval64<WPL, WPL == 1 && !ROOMY ? 8 : 16>(eoff, emask, nent, XT + b0, lane);
            const uint64_t os = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)o0) |
                                ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)o1) << 32);
            const uint64_t diff = (ob ^ os) & ballot(b0 + lane >= lo && b0 + lane < hi);
            if (diff) {
                if ((diff >> lane) & 1ull) atomicAdd(&a.tally[(int64_t)c * a.qp + b0 + lane], ((ob >> lane) & 1ull) ? sign : -sign);
                const uint64_t nw = os ^ diff;
                if (lane == 0) {
                    ostar_row[b << 1] = (uint32_t)nw;
                    ostar_row[(b << 1) + 1] = (uint32_t)(nw >> 32);
                }
                n_changes += __builtin_popcountll(diff);
            }
        }
    };
    // Examples [lo, hi), at most SPAN_DIRECT, from their rows, a few of them in flight at a time.
    auto direct = [&](int lo, int hi, const uint32_t (&m7)[WPL]) {
        constexpr int GROUP = NX == 1 ? 8 : 4;
        const int w = lo >> 5, w_last = (hi - 1) >> 5;
        const uint32_t o0 = ostar_row[w], o1 = ostar_row[w_last];
        uint32_t out = 0u; // bit k: output on example lo + k
        uint32_t in_row[NX];
        int ln = lane;
        // Addresses are formed here, not kept for every slot.  They are where registers are left (three slots, roomy, DEEP: 1.03 of the speed), and
        // with one slot, where it makes 1.03 as well.
        constexpr bool FORMED = WPL == 2 || (WPL == 3 && !(ROOMY && DEEP));
        if (FORMED) asm volatile("" : "+v"(ln));
#pragma unroll
        for (int r = 0; r < NX; ++r) {
            in_row[r] = row_at[r] * 4u;
            if (FORMED) asm volatile("" : "+v"(in_row[r]));
        }
#pragma unroll 1
        for (int i = lo; i < hi; i += GROUP) {
            uint32_t x[GROUP][NX], bits = 0u;
#pragma unroll
            for (int u = 0; u < GROUP; ++u) { // past the end: the last one again, which counts no more below
                const char *row = reinterpret_cast<const char *>(X + (int64_t)min(i + u, hi - 1) * d.Wf);
#pragma unroll
                for (int r = 0; r < NX; ++r) x[u][r] = *reinterpret_cast<const uint32_t *>(row + in_row[r]);
            }
#pragma unroll
            for (int u = 0; u < GROUP; ++u) {
                uint32_t viol = 0u;
#pragma unroll
                for (int r = 0; r < NX; ++r) viol |= PAIRED ? bitselect(x[u][r], m7[PAIRED ? 2 * r + 1 : 0], m7[PAIRED ? 2 * r : 0]) : m7[r] & ~(x[u][r] ^ neg[r]);
                bits |= ballot(viol != 0u) == 0 ? 1u << u : 0u;
            }
            out |= bits << (i - lo);
        }
        const uint64_t os = (uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)o0) |
                            ((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)o1) << 32); // o1 counts where there are two words
        const uint32_t diff = ((uint32_t)(os >> (lo & 31)) ^ out) & ((1u << (hi - lo)) - 1u);
        if (diff) {
            if (ln < 32 && ((diff >> ln) & 1u)) atomicAdd(&a.tally[(int64_t)c * a.qp + lo + ln], ((out >> ln) & 1u) ? sign : -sign);
            const uint64_t nw = os ^ ((uint64_t)diff << (lo & 31));
            if (ln == 0) {
                ostar_row[w] = (uint32_t)nw;
                if (w_last > w) ostar_row[w_last] = (uint32_t)(nw >> 32);
            }
            n_changes += (uint32_t)__builtin_popcount(diff);
        }
    };
    // Refresh (last lines of Algorithm 1) of the examples [from, to) under the masks m7, and the note that they are current.
    auto refresh = [&](int from, int to, const uint32_t (&m7)[WPL]) {
        if (from >= to) return;
        int s1 = from, e1 = from;
        if (plo < phi) {
            s1 = max(from, plo);
            e1 = max(s1, min(to, phi));
        }
        int s2 = max(max(from, slo), e1);
        if ((s1 < e1 || s2 < to) && have == NOTHING && to - from <= SPAN_DIRECT) {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); // as below
            n_eval += (uint32_t)(to - from);
            direct(from, to, m7);
        } else if (s1 < e1 || s2 < to) {
            // One block is evaluated from entries: building the list costs as much as that does.
            const bool brief = ((to + 63) >> 6) - (from >> 6) <= 1;
            if (have == NOTHING || (have == ENTRIES && !brief)) {
                bool dense = false; // a word of more than 20 literals: not worth counting
#pragma unroll
                for (int r = 0; r < WPL; ++r) dense |= __builtin_popcount(m7[r]) > 20;
                wave_lds_sync();
                have = ENTRIES;
                if (!brief && ballot(dense) == 0) {
                    n_listed = count_literals<WPL>(m7);
                    if (n_listed <= TRAIN_LIT_MAX) {
                        have = LIST;
                        build_literals<WPL, false, SPAN_LIT_PAD>(m7, llist, lane, d.Wf, d.o, (uint32_t)a.QW * 4u);
                    }
                }
                if (have == ENTRIES) nent = build_entries<WPL>(m7, lmask, eoff, emask, lane, d.Wf, d.W, (uint32_t)a.qp * 4u);
            }
            const bool listed = have == LIST;
            // words at the ends of a span may have been written by another lane of this wavefront a span before
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            if (s1 < e1 && e1 == s2) { // one run, as after every change of the masks
                s2 = s1;
                s1 = e1;
            }
#pragma unroll 1
            for (int part = 0; part < 2; ++part) {
                const int lo = part ? s2 : s1, hi = part ? to : e1;
                if (lo >= hi) continue;
                n_eval += (uint32_t)(hi - lo);
                if (listed) {
                    n_listed_blocks += (uint32_t)(hi - lo);
                    sweep(lo, hi);
                } else {
                    blocks(lo, hi);
                }
            }
        }
        if (from <= plo) plo = max(plo, to);
        if (from <= slo) slo = max(slo, to);
    };
    int pend = i_begin; // examples of the range from here on wait for their outputs under the present masks
    const int tz = d.thr ? __builtin_ctz(d.thr) : 16; // blocks below hold no bit that decides u < thr
    const int first_blk = min(tz >> 2, 4);
    const uint32_t ge_init = d.thr >= 65536u ? 0u : ~0u;

    // Feedback to the clause, whose output is Cout, on example ii, whose words are xw; drawn(r, ii): u >= thr of the literals of
    // slot r.  True if the masks changed, by flip.
    auto event = [&](int ii, bool type1, bool Cout, const uint32_t (&xw)[NX], uint32_t (&flip)[WPL], auto drawn) {
        if (LAZY && !have_planes) load_planes();
        if (!type1) ++n_type2;
        uint32_t changed = 0u;
#pragma unroll
        for (int r = 0; r < WPL; ++r) {
            uint32_t sp[8], move, up;
            get_slot(p[r], sp);
            const uint32_t lit = xw[PAIRED ? r / 2 : r] ^ neg[r]; // padding bits and idle lanes: not valid
            if (!type1) { // Type II feedback (Table 2): where the clause is 1 and the literal 0, push Exclude towards Include
                move = up = ~lit & ~sp[7] & valid[r]; // excluded automata (below the top bit) cannot overflow
            } else {      // Type I feedback (Table 1)
                const uint32_t ge = drawn(r, ii);
                // weak: towards Exclude with probability 1/s; strong, clause and literal 1: towards Include with (s-1)/s (1 if boosted)
                move = ~ge & valid[r] & ~at_value<FULL>(sp, a.sat.kmin, false);
                up = 0u;
                if (Cout) {
                    up = lit & valid[r] & (ge | d.boost) & ~at_value<FULL>(sp, a.sat.kmax, true);
                    move = (move & ~lit) | up;
                }
            }
            flip[r] = ripple_flip(sp, move, up);
            changed |= flip[r];
            if (WPL > 1) pin_planes(sp, changed);
            put_slot(p[r], sp);
        }
        return ballot(changed != 0u) != 0;
    };

    // One round of gate entries after the other; the last turn takes what waits for its outputs.
    int ent_cur = -1, v_cur = 0, ent_nxt = -1;
    if constexpr (TEAM) {
        if (rounds) __syncthreads();
    } else { // entries are fetched two rounds ahead, tallies (which need the entry) one: reading a tally early is within the method's premise
        ent_cur = load_ent(lane);
        v_cur = load_v(ent_cur);
        ent_nxt = load_ent(64 + lane);
    }
    for (int k0 = 0;; k0 += ROUND) {
        const bool last = k0 >= k_hi;
        int end = i_end;     // outputs may wait beyond this example of the range
        int ev = 0, nf = 0;  // {example << 1 | Type I} of the fired entries, their number
        uint64_t t1mask = 0; // which of them mean Type I feedback
        if (!last) {
            const uint32_t *h = handed;
            if constexpr (TEAM) {
                __syncthreads();
                h += ((k0 / ROUND) & 3) * TEAM_HANDED;
                nf = __builtin_amdgcn_readfirstlane((int)h[ROUND]);
                n_draw = (uint32_t)__builtin_amdgcn_readfirstlane((int)h[ROUND + 1]);
                end = __builtin_amdgcn_readfirstlane((int)h[ROUND + 2]);
            } else {
                const int ent = ent_cur, v = v_cur;
                ent_cur = ent_nxt;
                v_cur = load_v(ent_cur);
                ent_nxt = load_ent(k0 + 128 + lane);
                bool target;
                const bool fire = gate_of(ent, v, target);
                const uint64_t f = ballot(fire);
                const int pre = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(f >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)f, 0u));
                wave_lds_sync();
                if (fire) handed[pre] = (uint32_t)(ent & ~1) | (target == pos ? 1u : 0u);
                wave_lds_sync();
                nf = __builtin_popcountll(f);
                end = (__builtin_amdgcn_readlane(ent, min(64, k_hi - k0) - 1) >> 1) + 1;
            }
            ev = (int)h[lane & (ROUND - 1)];
            t1mask = ballot((ev & 1) != 0 && lane < nf);
            n_fired += nf;
            n_type1 += __builtin_popcountll(t1mask);
        }
        const uint32_t *rows_now = rows + (TEAM ? ((k0 / ROUND) & 1) * STAGED * PITCH : 0);
        const uint32_t *ge_at = draws + (TEAM ? ((k0 / ROUND) & 1) * ROUND * 64 : 0) + lane;
        uint64_t t1left = t1mask;    // whose draws are still to come (not TEAM)
        int n_ahead = 0, n_used = 0; // events drawn ahead, those of them used
        int at = 0, from = 0, to = 0; // next event; those whose rows are in LDS
        uint32_t act = 0u, outs = 0u; // of these, beginning with the from-th: to be worked on; the clause's outputs
        bool wide = true;             // the masks may hold for a while: outputs on all of these at once
        for (;;) {
            uint32_t flip[WPL] = {};
            bool moved = false;
            int upto = pend; // outputs are taken up to here
            // one event after the other until the masks change
            while (at < nf) {
                if (at == to) { // the rows of the next fired examples into LDS
                    from = at;
                    to = TEAM ? nf : min(at + STAGED, nf);
                    if constexpr (!TEAM && WPL == 1) { // two rows a load
                        const int half = lane >> 5, word = lane & 31;
                        uint32_t x[STAGED / 2];
#pragma unroll
                        for (int u = 0; u < STAGED / 2; ++u) {
                            if (from + 2 * u < to) {
                                const uint32_t i = handed[min(from + 2 * u + half, to - 1)] >> 1;
                                x[u] = *reinterpret_cast<const uint32_t *>(reinterpret_cast<const char *>(X) + (i * (uint32_t)d.Wf + (uint32_t)min(word, d.Wf - 1)) * 4u);
                            }
                        }
#pragma unroll
                        for (int u = 0; u < STAGED / 2; ++u)
                            if (from + 2 * u < to) rows[u * 2 * PITCH + lane] = x[u];
                        wave_lds_sync();
                    } else if constexpr (!TEAM) {
                        uint32_t x[STAGED][(PITCH + 63) / 64];
#pragma unroll
                        for (int u = 0; u < STAGED; ++u) {
                            if (from + u < to) {
                                const uint32_t *row = X + (int64_t)(readlane((uint32_t)ev, from + u) >> 1) * d.Wf;
#pragma unroll
                                for (int w = 0; w < (PITCH + 63) / 64; ++w) x[u][w] = row[min(w * 64 + lane, d.Wf - 1)];
                            }
                        }
#pragma unroll
                        for (int u = 0; u < STAGED; ++u) {
                            if (from + u < to) {
#pragma unroll
                                for (int w = 0; w < (PITCH + 63) / 64; ++w)
                                    if (w * 64 + lane < PITCH) rows[u * PITCH + w * 64 + lane] = x[u][w];
                            }
                        }
                        wave_lds_sync();
                    }
                }
                // outputs of the clause on the events to come, the state before each of them being the present one: all of those in LDS, or
                // after a change, which another may follow soon, the next eight at most (with two and three slots there are no more; with two the
                // compiler makes 3 % faster code if it is not told)
                const int first = (at - from) & ~7, n = wide || WPL == 3 ? to - from : min(to - from, first + 8);
                outs = 0u;
                for (int j = first; j < n; j += 8) {
                    uint32_t viol[8];
#pragma unroll
                    for (int u = 0; u < 8; ++u) {
                        viol[u] = 0u;
#pragma unroll
                        for (int r = 0; r < NX; ++r) {
                            const uint32_t x = rows_now[(j + u) * PITCH + row_at[r]];
                            viol[u] |= PAIRED ? bitselect(x, p[PAIRED ? 2 * r + 1 : 0][7], p[PAIRED ? 2 * r : 0][7]) : p[r][7] & ~(x ^ neg[r]);
                        }
                    }
                    uint32_t byte = 0u;
#pragma unroll
                    for (int u = 0; u < 8; ++u) byte |= ballot(viol[u] != 0u) == 0 ? 1u << u : 0u;
                    outs |= byte << j;
                }
                // Type II feedback to a clause whose output is 0 changes nothing (Table 2)
                act = ((uint32_t)(t1mask >> from) | outs) & (n < 32 ? (1u << n) - 1u : ~0u) & ~((1u << (at - from)) - 1u);
                uint32_t xnext[NX], genext = 0u; // of the next event: words, and where they are there (TEAM) the draws of the next Type I event
                int j = act ? __builtin_ctz(act) : 0;
#pragma unroll
                for (int r = 0; r < NX; ++r) xnext[r] = rows_now[j * PITCH + row_at[r]];
                if constexpr (TEAM) genext = *ge_at;
                while (act) {
                    act &= act - 1u;
                    const uint32_t s = readlane((uint32_t)ev, from + j);
                    const bool type1 = (s & 1u) != 0u, Cout = ((outs >> j) & 1u) != 0u;
                    upto = (int)(s >> 1);
                    at = from + j + 1;
                    uint32_t xw[NX], g0 = genext;
#pragma unroll
                    for (int r = 0; r < NX; ++r) xw[r] = xnext[r];
                    j = act ? __builtin_ctz(act) : j;
#pragma unroll
                    for (int r = 0; r < NX; ++r) xnext[r] = rows_now[j * PITCH + row_at[r]];
                    if constexpr (TEAM) {
                        if (type1) ge_at += 64;
                        genext = *ge_at;
                    }
                    if constexpr (DEEP && !TEAM) {
                        if (type1 && n_used == n_ahead) {
                            n_ahead = deep_draw(t1left, ev, train_draw_events(WPL), 0, 1, 0);
                            for (int k = 0; k < n_ahead; ++k) t1left &= t1left - 1;
                            n_used = 0;
                        }
                    }
                    moved = event(upto, type1, Cout, xw, flip, [&](int r, int i) {
                        if constexpr (TEAM) {
                            return g0;
                        } else if constexpr (DEEP) {
                            return ge_at[(n_used * WPL + r) * 64];
                        } else {
                            // the bits of blocks below first_blk cannot decide, see train_clause
                            uint32_t lw = (uint32_t)Map::word(r, lane, d.Wf), ge = ge_init, thr = d.thr;
                            asm volatile("" : "+v"(lw)); // the first Philox round of every slot is not to be kept
                            RngKey key = d.key;
                            if (WPL == 1) asm volatile("" : "+s"(key.seed_lo), "+s"(key.seed_hi), "+s"(thr)); // see LAUNDER
#pragma unroll
                            for (int t = 2; t < 4; ++t) {
                                if (t >= first_blk) {
                                    uint32_t tm[4];
#pragma unroll
                                    for (int k = 0; k < 4; ++k) tm[k] = (uint32_t)__builtin_amdgcn_sbfe((int)thr, 4 * t + k, 1);
                                    const PhiloxStart start = WPL > 1 ? philox_start(4u * lw + (uint32_t)t, STREAM_TYPE1, a.epoch, key) : t == 2 ? start2 : start3;
                                    ge = compare_nibble(draw_from(start, key, (uint32_t)g, (uint32_t)i, tm[0], tm[2]), tm, ge);
                                }
                            }
                            return ge;
                        }
                    });
                    if (DEEP && !TEAM && type1) n_used = uniform(n_used + 1);
                    if (moved) break;
                }
                if (moved) break;
                at = from + n;
                wide = true;
            }
            if (!moved) upto = last ? i_end : end - pend >= SPAN_MOST ? end & ~31 : pend;
            uint32_t m7[WPL]; // the masks those examples were visited with
#pragma unroll
            for (int r = 0; r < WPL; ++r) m7[r] = moved ? p[r][7] ^ flip[r] : p[r][7];
            refresh(pend, upto, m7);
            pend = max(pend, upto);
            if (!moved) break;
            plo = 0; // the conjunction changed: whatever was visited before is outdated, and so is all that comes
            phi = slo = upto;
            have = NOTHING;
            wide = TEAM; // eight at a time costs a team 2 % on noisy images (1,000 clauses of 784 features) and gains 3 % on bags of words
        }
        if (last) break;
    }
    if (plo >= phi) plo = phi = 0;
    if (lane == 0) *reinterpret_cast<int4 *>(a.fresh + (int64_t)g * 4) = make_int4(plo, phi, slo >= a.q ? a.qp : slo, 0);

    if (!LAZY || have_planes) { // a gate fired: the automata may have moved
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
    // outputs taken: those of spans, and one per fired gate from its row
    store_counters(a, g, lane, (n_listed_blocks + 63) >> 6, n_fired, n_type1, n_changes, n_type2, (n_eval + n_fired + 63) >> 6, n_draw, !LAZY || have_planes);
}

} // namespace tsetlin

#endif

// Clause outputs from include masks and literal rows in LDS, lane = 64 examples (interpretation of a trained machine).
// Part of tm_kernels.hip (included there).
#ifndef TM_KERNELS_EVAL_BITS_HPP_
#define TM_KERNELS_EVAL_BITS_HPP_

namespace tsetlin {

// ------------------------------------------------------------------------
// k_eval_bits: outputs of every clause on a range of examples, without a workspace
// ------------------------------------------------------------------------
//
// The lane = clause kernels do one operation per feature WORD and example whatever the masks hold; a trained clause
// includes a few dozen literals, and its outputs are the AND of that many bit rows over the examples.  The call has
// no workspace for such rows, but those of a range of examples fit the LDS of a CU: a workgroup of 16 wavefronts
// transposes 32 * RW examples into one row per feature (RW words; a negated literal is the complement), and each
// wavefront then takes clauses of the workgroup's share.  Lane = literal word finds the included literals, the lowest of
// every word per step, into a list of the wavefront; 64 / (RW / 2) groups of lanes AND the rows of different
// literals, a lane holding 64 examples.  The steps end when no example is left.  Literals that are true on the whole
// range (blank pixels, rare words: a trained clause may hold hundreds of them) are dropped from the masks first.
// Pair p of row k stands at place p ^ (k mod (RW / 2)), so that the 32 rows a transposition writes at once
// spread over the banks, and a list entry is the address of its row with that folded in: an exclusive or with
// the lane's pair finds the word (seven operations an entry with row numbers).  Lists are filled up to 64 entries with a row
// of ones, so that reading them takes neither a clamp nor an address of its own per entry.
// What bounds it is the issue of the list and row steps of every (clause, range) and, with few clauses per share, the
// transposition.  Measured: 10,000 examples on 20,000 trained clauses of 784 features 250 -> 98 (row numbers) -> 72 us; clauses
// of 100 literals of 2,400 features, false on every example, are the one form measured slower (2,000 of them 35 -> 42 us).

constexpr int BITS_WAVES = 16; // wavefronts per workgroup

// RW = words of examples per row, WF = most feature words
template <int RW, int WF>
__global__ __launch_bounds__(64 * BITS_WAVES) void k_eval_bits(const uint32_t *__restrict__ inc,
                                                               const uint32_t *__restrict__ X, uint32_t *__restrict__ bits,
                                                               const EvalArgs a, int share)
{
    constexpr int PAIRS = RW / 2, GROUPS = 64 / PAIRS, NW = (2 * WF + 63) / 64, AHEAD = 8;
    static_assert(BITS_WAVES % PAIRS == 0, "wavefronts per pair of words");
    __shared__ uint2 rows[(WF * 32 + 1) * PAIRS]; // the last one: ones
    __shared__ uint32_t always[2 * WF]; // literals that are true on every example of the range
    __shared__ uint32_t lists[BITS_WAVES][64];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int64_t e0 = (int64_t)blockIdx.x * (RW * 32);

    for (int w = (int)threadIdx.x; w < 2 * WF; w += 64 * BITS_WAVES) always[w] = ~0u;
    if (threadIdx.x < PAIRS) rows[WF * 32 * PAIRS + threadIdx.x] = make_uint2(~0u, ~0u);
    __syncthreads();
    { // rows: this wavefront's 64 examples, every (BITS_WAVES / PAIRS)-th feature word
        constexpr int STEP = BITS_WAVES / PAIRS;
        const int p = wave & (PAIRS - 1);
        const uint32_t *xr = X + min(e0 + p * 64 + lane, a.q - 1) * a.Wf; // past the end: the last example again
        uint32_t *out = reinterpret_cast<uint32_t *>(rows) + (lane >> 5);
        for (int f0 = wave / PAIRS; f0 < a.Wf; f0 += AHEAD * STEP) {
            uint32_t x[AHEAD];
#pragma unroll
            for (int t = 0; t < AHEAD; ++t) x[t] = xr[min(f0 + t * STEP, a.Wf - 1)];
#pragma unroll
            for (int t = 0; t < AHEAD; ++t) {
                const int fw = f0 + t * STEP;
                if (fw >= a.Wf) break;
                uint32_t v = x[t]; // 32 x 32 bits over each half of the wavefront: lane b, bit k -> lane k, bit b
                const uint32_t keep[5] = {0x0000ffffu, 0x00ff00ffu, 0x0f0f0f0fu, 0x33333333u, 0x55555555u};
#pragma unroll
                for (int s = 0; s < 5; ++s) {
                    const int sh = 16 >> s;
                    const uint32_t w = __shfl_xor(v, sh, 64);
                    v = (lane & sh) ? bitselect(keep[s], w >> sh, v) : bitselect(keep[s], v, w << sh);
                }
                const uint64_t ones = ballot(v == ~0u), zeros = ballot(v == 0u);
                if (lane == 0) {
                    atomicAnd(&always[fw], (uint32_t)ones & (uint32_t)(ones >> 32));
                    atomicAnd(&always[a.Wf + fw], (uint32_t)zeros & (uint32_t)(zeros >> 32));
                }
                const int k = fw * 32 + (lane & 31);
                out[(k * PAIRS + (p ^ (k & (PAIRS - 1)))) * 2] = v;
            }
        }
    }
    __syncthreads();

    const int t = lane & (PAIRS - 1), grp = lane / PAIRS;
    uint32_t *list = lists[wave];
    const char *row_bytes = reinterpret_cast<const char *>(rows);
    constexpr uint32_t ROW = 8u * PAIRS, NEGATED = 0x80000000u; // bytes of a row; bit 31 of an entry: the literal is negated
    constexpr uint32_t ONES = (uint32_t)(WF * 32) * ROW; // WF * 32 mod PAIRS is 0: nothing to fold in
    const uint32_t t8 = 8u * (uint32_t)t;
    const int64_t words = (a.q + 31) >> 5;
    const int g_end = min(a.C, ((int)blockIdx.y + 1) * share);
    uint32_t mk[NW], next[NW], skip[NW];
    const int g0 = (int)blockIdx.y * share + wave;
    if (g0 >= g_end) return;
#pragma unroll
    for (int r = 0; r < NW; ++r) skip[r] = r * 64 + lane < a.W ? always[r * 64 + lane] : 0u;
#pragma unroll
    for (int r = 0; r < NW; ++r) next[r] = r * 64 + lane < a.W ? inc[(int64_t)g0 * a.W + r * 64 + lane] : 0u;
    for (int g = g0; g < g_end; g += BITS_WAVES) {
        const int gn = min(g + BITS_WAVES, g_end - 1); // requested a clause ahead
#pragma unroll
        for (int r = 0; r < NW; ++r) {
            mk[r] = next[r] & ~skip[r];
            next[r] = r * 64 + lane < a.W ? inc[(int64_t)gn * a.W + r * 64 + lane] : 0u;
        }
        uint2 acc = make_uint2(~0u, ~0u);
        bool left = true;
#pragma unroll
        for (int r = 0; r < NW; ++r) {
            const int lw = r * 64 + lane;
            const uint32_t first = lw >= a.Wf ? (uint32_t)(lw - a.Wf) * (32u * ROW) | NEGATED : (uint32_t)lw * (32u * ROW);
            while (left) {
                const uint64_t b = ballot(mk[r] != 0u);
                if (b == 0) break;
                const int cnt = __builtin_popcountll(b);
                const int pre = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u));
                const bool has = mk[r] != 0u;
                uint32_t entry = ONES;
                if (has) { // a word's rows begin at a multiple of PAIRS
                    const uint32_t bit = (uint32_t)__builtin_ctz(mk[r]);
                    entry = first + (bit * ROW | (bit & (PAIRS - 1)) * 8u);
                }
                list[has ? pre : cnt + lane - pre] = entry;
                mk[r] &= mk[r] - 1u; // stays 0 once it is 0
                wave_lds_sync();
                for (int j = 0; j < cnt; j += 4 * GROUPS) {
                    uint32_t ent[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) ent[u] = list[j + u * GROUPS + grp];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const uint32_t neg = (uint32_t)((int32_t)ent[u] >> 31);
                        const uint2 v = *reinterpret_cast<const uint2 *>(row_bytes + ((ent[u] & ~NEGATED) ^ t8));
                        acc.x &= v.x ^ neg;
                        acc.y &= v.y ^ neg;
                    }
                }
                left = ballot((acc.x | acc.y) != 0u) != 0;
                wave_lds_sync(); // the list is written again
            }
        }
        if (left) { // otherwise every lane holds zeros
#pragma unroll
            for (int s = PAIRS; s < 64; s <<= 1) {
                acc.x &= __shfl_xor(acc.x, s, 64);
                acc.y &= __shfl_xor(acc.y, s, 64);
            }
        }
        if (grp == 0) {
            const int64_t w = (int64_t)blockIdx.x * RW + 2 * t;
            const uint32_t tail = (a.q & 31) ? (1u << (a.q & 31)) - 1u : ~0u; // bits of the last word that are examples
            if (w < words) bits[(int64_t)g * a.bits_stride + w] = acc.x & (w == words - 1 ? tail : ~0u);
            if (w + 1 < words) bits[(int64_t)g * a.bits_stride + w + 1] = acc.y & (w + 1 == words - 1 ? tail : ~0u);
        }
    }
}

} // namespace tsetlin

#endif

// Clause evaluation for a few examples, lane = literal word (inference with a workspace, small calls).
// Part of tm_kernels.hip (included there).
#ifndef TM_KERNELS_EVAL_FEW_HPP_
#define TM_KERNELS_EVAL_FEW_HPP_

namespace tsetlin {

// ------------------------------------------------------------------------
// k_eval_few / k_few_finish: class sums of a few examples straight from the include masks
// ------------------------------------------------------------------------
//
// The list path (k_rows_and_lists + k_eval_sparse) evaluates 2,048 examples at a time and costs the same for one
// example as for all of them: building the lists and bit rows, then the chain of list rounds.  A few examples need
// only the masks: lane = literal word, the words of E examples in registers (or the L1), FEW_U clauses in flight per
// wavefront.  With more than FEW_E examples the groups of a share of clauses are workgroups that follow one
// another on the same XCD (workgroups are dealt out to the eight XCDs in turn), so that the masks come from
// memory once and to the later groups from that XCD's L2.  What bounds it is launch latency and the passes over
// the masks, on large machines the L2 and the issue of the bit operations.  Every workgroup writes its own partial sums, so
// nothing has to be cleared first, and the second kernel adds them up, clamps and decides.
// Measured per call of 1 / 32 examples, us: 20,000 clauses of 784 features 11 / 19 (list path 31 / 35), 65,536 of 20,000
// features 64 / 235 (337 / 347; 489 for 32 examples with the groups of four in the slowest grid dimension, the masks
// read from memory eight times).

constexpr int FEW_E = 8;        // examples of a workgroup, most
constexpr int FEW_U = 4;        // clauses a wavefront walks in step
constexpr int FEW_WAVES = 4;    // wavefronts per workgroup
constexpr int FEW_CHUNK = 32;   // clauses of a class per workgroup, a multiple of FEW_U * FEW_WAVES
constexpr int FEW_EXAMPLES = 32; // most examples of a call that takes this path

struct FewArgs {
    int q, Wf, W, n, m, S; // S = shares of FEW_CHUNK clauses per class
    int all_pos;           // regression mode: every clause votes +1
    int Tlo, T;
    int rows_y;            // grid dimension y of k_eval_few
};

// partial[(c * S + s) * q + i] = votes of the clauses of share s of class c for example i.  Grid: x = 8 * groups of E
// examples, (y, z) = shares of all classes by eights; the XCD of a workgroup is its x modulo 8.
template <int E>
__global__ __launch_bounds__(64 * FEW_WAVES) void k_eval_few(const uint32_t *__restrict__ inc, const uint32_t *__restrict__ X,
                                                             int32_t *__restrict__ partial, const FewArgs a)
{
    __shared__ int32_t votes[FEW_WAVES][E];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
    const int share = (int)((blockIdx.z * (unsigned)a.rows_y + blockIdx.y) * 8 + (blockIdx.x & 7)); // at most half the 2^30 clauses
    if (share >= a.m * a.S) return; // the whole workgroup
    const int c = share / a.S, s = share - c * a.S;
    const int i0 = (int)(blockIdx.x >> 3) * E;
    const int j_end = min(a.n, (s + 1) * FEW_CHUNK);
    int sum[E];
#pragma unroll
    for (int e = 0; e < E; ++e) sum[e] = 0;
    for (int j0 = s * FEW_CHUNK + wave * FEW_U; j0 < j_end; j0 += FEW_U * FEW_WAVES) {
        uint32_t viol[FEW_U][E];
#pragma unroll
        for (int u = 0; u < FEW_U; ++u)
#pragma unroll
            for (int e = 0; e < E; ++e) viol[u][e] = 0u;
        for (int lw0 = 0; lw0 < a.W; lw0 += 64) {
            const int lw = lw0 + lane;
            const bool act = lw < a.W;
            const bool neg = lw >= a.Wf;
            const int fw = act ? (neg ? lw - a.Wf : lw) : 0;
            uint32_t lit[E], mk[FEW_U];
#pragma unroll
            for (int u = 0; u < FEW_U; ++u) { // clauses past the end are read as the last one and not counted
                const int64_t g = (int64_t)c * a.n + min(j0 + u, j_end - 1);
                mk[u] = act ? inc[g * a.W + lw] : 0u;
            }
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const uint32_t x = X[(int64_t)min(i0 + e, a.q - 1) * a.Wf + fw];
                lit[e] = neg ? ~x : x;
            }
#pragma unroll
            for (int u = 0; u < FEW_U; ++u)
#pragma unroll
                for (int e = 0; e < E; ++e) viol[u][e] |= mk[u] & ~lit[e];
        }
#pragma unroll
        for (int u = 0; u < FEW_U; ++u) {
            const int vote = j0 + u < j_end ? (((u & 1) || a.all_pos) ? 1 : -1) : 0; // odd index within the class: positive
#pragma unroll
            for (int e = 0; e < E; ++e) sum[e] += ballot(viol[u][e] != 0u) == 0 ? vote : 0;
        }
    }
    if (lane == 0) {
#pragma unroll
        for (int e = 0; e < E; ++e) votes[wave][e] = sum[e];
    }
    __syncthreads();
    if ((int)threadIdx.x < E && i0 + (int)threadIdx.x < a.q) {
        int v = 0;
#pragma unroll
        for (int w = 0; w < FEW_WAVES; ++w) v += votes[w][threadIdx.x];
        partial[(int64_t)share * a.q + i0 + threadIdx.x] = v;
    }
}

// One workgroup per example: sums[i][c] = clamped sum of the partial sums, pred[i] (if wanted) = lowest class index
// with the largest of them, in regression mode the clamped sum itself.  2^per_log lanes add up the shares of a class (S
// rounded up to a power of two, at most 64), so that a wavefront takes several classes at once: with one class at a time 3,000
// classes of two clauses took 264 us per call instead of 11.
__global__ __launch_bounds__(256) void k_few_finish(const int32_t *__restrict__ partial, int32_t *sums, int32_t *pred,
                                                    const FewArgs a, int per_log)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = blockIdx.x;
    int best = 0x7fffffff, bv = (int)0x80000000; // no class yet
    const int per = 1 << per_log, step = 256 >> per_log;
    for (int c0 = 0; c0 < a.m; c0 += step) { // every lane takes part in the shuffles of every round
        const int c = c0 + ((int)threadIdx.x >> per_log);
        int v = 0;
        if (c < a.m)
            for (int s = lane & (per - 1); s < a.S; s += per) v += partial[((int64_t)c * a.S + s) * a.q + i];
#pragma unroll
        for (int sh = 32; sh > 0; sh >>= 1)
            if (sh < per) v += __shfl_xor(v, sh, 64);
        if (c < a.m) {
            v = min(max(v, a.Tlo), a.T);
            if ((lane & (per - 1)) == 0) sums[(int64_t)i * a.m + c] = v;
            if (v > bv) { // ascending classes: the lowest index of equals stays
                bv = v;
                best = c;
            }
        }
    }
    if (!pred) return;
    __shared__ int wbest[4], wval[4];
    for (int sh = 32; sh >= per; sh >>= 1) { // the lanes of a class hold the same
        const int ov = __shfl_xor(bv, sh, 64), ob = __shfl_xor(best, sh, 64);
        if (ov > bv || (ov == bv && ob < best)) {
            bv = ov;
            best = ob;
        }
    }
    if (lane == 0) {
        wbest[wave] = best;
        wval[wave] = bv;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < 4; ++w)
            if (wval[w] > bv || (wval[w] == bv && wbest[w] < best)) {
                bv = wval[w];
                best = wbest[w];
            }
        pred[i] = a.all_pos ? bv : best;
    }
}

} // namespace tsetlin

#endif

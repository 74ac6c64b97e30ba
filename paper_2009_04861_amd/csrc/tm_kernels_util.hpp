// Small kernels around the main ones: fills, state conversion, transposes, label check,
// negative class, clamp / argmax, copies.
// Part of tm_kernels.hip (included there).
#ifndef TM_KERNELS_UTIL_HPP_
#define TM_KERNELS_UTIL_HPP_

namespace tsetlin {

// ------------------------------------------------------------------------
// small utility kernels
// ------------------------------------------------------------------------

__global__ void k_fill_u32(uint32_t *p, int64_t nwords, uint32_t v)
{
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < nwords; i += stride) p[i] = v;
}

// Initial TA states: state N or N+1 with probability 1/2, i.e. stored value
// 127 or 128.  One thread per (clause, literal word).
__global__ void k_init_state(Dims d, uint32_t *planes, uint32_t *inc)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= (int64_t)d.C * d.W) return;
    const int g = (int)(t / d.W);
    const int lw = (int)(t - (int64_t)g * d.W);
    const int fw = lw >= d.Wf ? lw - d.Wf : lw;
    const uint32_t valid = (fw == d.Wf - 1) ? d.tailmask : ~0u;
    const U4 r = draw(d.key, STREAM_INIT, 4u * (uint32_t)lw, (uint32_t)g, 0, 0);
    const uint32_t top = r.x & valid;
    uint32_t *p = planes + t * 8;
#pragma unroll
    for (int b = 0; b < 7; ++b) p[b] = ~top;
    p[7] = top;
    inc[t] = top;
}

// Automata as bytes (state - 1) <-> bit planes; one thread per (clause, literal word).  The bytes of consecutive literal words
// follow one another (the last word of a half is shorter), also from clause to clause, so a workgroup's are one run, which
// moves between memory and LDS in whole 32-bit words whatever its alignment (the ends byte by byte).  20,000
// clauses of 784 features, each thread its own bytes / this: set 57 / 26 us, get 31 / 16; of 783 features 57 / 30, 32 / 18.
constexpr int STATE_WORDS = 256; // literal words per workgroup

__device__ __forceinline__ int64_t state_byte(const Dims &d, int64_t t) // where the bytes of literal word t start
{
    const int64_t g = t / d.W;
    const int lw = (int)(t - g * d.W);
    return g * 2 * d.o + (lw >= d.Wf ? d.o + (lw - d.Wf) * 32 : lw * 32);
}

// Four automata of a 32-bit word (bytes) and four bits of a plane: the multiplication brings bit 0 of the four bytes side by
// side without carries, and its counterpart spreads four bits over four bytes.
__device__ __forceinline__ uint32_t bytes_to_nibble(uint32_t bytes) { return ((bytes & 0x01010101u) * 0x01020408u) >> 24; }
__device__ __forceinline__ uint32_t nibble_to_bytes(uint32_t nibble) { return (nibble * 0x00204081u) & 0x01010101u; }

__global__ __launch_bounds__(STATE_WORDS) void k_set_state(Dims d, const uint8_t *in, uint32_t *planes, uint32_t *inc)
{
    __shared__ uint32_t run[STATE_WORDS * 8 + 2];
    const int64_t words = (int64_t)d.C * d.W, t0 = (int64_t)blockIdx.x * STATE_WORDS, t = t0 + threadIdx.x;
    const int64_t b0 = state_byte(d, t0), b1 = state_byte(d, min(t0 + STATE_WORDS, words));
    const int skew = (int)((uintptr_t)(in + b0) & 3), end = skew + (int)(b1 - b0); // the run lies at [skew, end) of LDS
    const uint8_t *src = in + b0 - skew;
    uint8_t *run8 = reinterpret_cast<uint8_t *>(run);
    for (int w = threadIdx.x; 4 * w < end; w += STATE_WORDS) {
        if (4 * w >= skew && 4 * w + 4 <= end) {
            run[w] = reinterpret_cast<const uint32_t *>(src)[w];
        } else {
            for (int k = max(4 * w, skew); k < min(4 * w + 4, end); ++k) run8[k] = src[k];
        }
    }
    __syncthreads();
    if (t >= words) return;
    const int lw = (int)(t % d.W), fw = lw >= d.Wf ? lw - d.Wf : lw;
    const uint32_t most = (uint32_t)(2 * d.N - 1), shift = (uint32_t)(128 - d.N);
    const int left = d.o - fw * 32, at = skew + (int)(state_byte(d, t) - b0); // automata from here to the end of the half
    uint32_t p[8] = {0, 0, 0, 0, 0, 0, 0, 0};
#pragma unroll
    for (int k = 0; k < 8; ++k) {
        uint32_t v = 0u, stored = 0u;
        if ((at & 3) == 0) {
            v = run[min((at >> 2) + k, STATE_WORDS * 8 + 1)];
        } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) v |= (uint32_t)run8[min(at + 4 * k + j, STATE_WORDS * 32 + 7)] << (8 * j);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) { // padding automata: excluded (127), never touched
            const uint32_t b = (v >> (8 * j)) & 255u;
            stored |= (4 * k + j < left ? min(b, most) + shift : 127u) << (8 * j);
        }
#pragma unroll
        for (int b = 0; b < 8; ++b) p[b] |= bytes_to_nibble(stored >> b) << (4 * k);
    }
    uint4 *dst = reinterpret_cast<uint4 *>(planes + t * 8);
    dst[0] = make_uint4(p[0], p[1], p[2], p[3]);
    dst[1] = make_uint4(p[4], p[5], p[6], p[7]);
    inc[t] = p[7];
}

__global__ __launch_bounds__(STATE_WORDS) void k_get_state(Dims d, const uint32_t *planes, uint8_t *out)
{
    __shared__ uint32_t run[STATE_WORDS * 8 + 2];
    const int64_t words = (int64_t)d.C * d.W, t0 = (int64_t)blockIdx.x * STATE_WORDS, t = t0 + threadIdx.x;
    const int64_t b0 = state_byte(d, t0), b1 = state_byte(d, min(t0 + STATE_WORDS, words));
    const int skew = (int)((uintptr_t)(out + b0) & 3), end = skew + (int)(b1 - b0);
    uint8_t *dst = out + b0 - skew, *run8 = reinterpret_cast<uint8_t *>(run);
    if (t < words) {
        const int lw = (int)(t % d.W), fw = lw >= d.Wf ? lw - d.Wf : lw;
        const int left = d.o - fw * 32, at = skew + (int)(state_byte(d, t) - b0);
        const uint4 *src = reinterpret_cast<const uint4 *>(planes + t * 8);
        const uint4 a = src[0], c = src[1];
        const uint32_t p[8] = {a.x, a.y, a.z, a.w, c.x, c.y, c.z, c.w};
        const uint32_t shift = (uint32_t)(128 - d.N) * 0x01010101u; // no stored value is below it: no borrow between bytes
#pragma unroll
        for (int k = 0; k < 8; ++k) {
            uint32_t v = 0u;
#pragma unroll
            for (int b = 0; b < 8; ++b) v |= nibble_to_bytes((p[b] >> (4 * k)) & 15u) << b;
            v -= shift;
            if ((at & 3) == 0 && 4 * k + 4 <= left) {
                run[(at >> 2) + k] = v;
            } else {
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if (4 * k + j < left) run8[at + 4 * k + j] = (uint8_t)(v >> (8 * j));
            }
        }
    }
    __syncthreads();
    for (int w = threadIdx.x; 4 * w < end; w += STATE_WORDS) {
        if (4 * w >= skew && 4 * w + 4 <= end) {
            reinterpret_cast<uint32_t *>(dst)[w] = run[w];
        } else {
            for (int k = max(4 * w, skew); k < min(4 * w + 4, end); ++k) dst[k] = run8[k];
        }
    }
}

// labels must lie in [0, m) (regression mode: targets in [0, T], m = T + 1)
__global__ void k_check_labels(const int32_t *y, int64_t q, int m, int32_t *flag)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < q && (y[i] < 0 || y[i] >= m)) *flag = 1;
}

// sums[i][c] = clamp(sums[i][c], lo, T): lo = -T, or 0 in regression mode
__global__ void k_clamp(int32_t *sums, int64_t n, int lo, int T)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) sums[t] = min(max(sums[t], lo), T);
}

// pred[i] = lowest class index with the largest (already clamped) sum; in regression mode
// the clamped vote sum itself
__global__ void k_argmax(const int32_t *sums, int32_t *pred, int64_t q, int m, int regr)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= q) return;
    if (regr) {
        pred[i] = sums[i];
        return;
    }
    int best = 0;
    int32_t bv = sums[i * m];
    for (int c = 1; c < m; ++c) {
        const int32_t v = sums[i * m + c];
        if (v > bv) {
            bv = v;
            best = c;
        }
    }
    pred[i] = best;
}

// both of the above in one pass over the unclamped sums
__global__ void k_clamp_argmax(int32_t *sums, int32_t *pred, int64_t q, int m, int lo, int T, int regr)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= q) return;
    int best = 0;
    int32_t bv = 0;
    for (int c = 0; c < m; ++c) {
        const int32_t v = min(max(sums[i * m + c], lo), T);
        sums[i * m + c] = v;
        if (c == 0 || v > bv) {
            bv = v;
            best = c;
        }
    }
    pred[i] = regr ? bv : best;
}

// out[i][c] = tally[c][i]
__global__ void k_tally_out(const int32_t *tally, int32_t *out, int64_t q, int64_t qp, int m)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= q * m) return;
    const int64_t i = t / m;
    const int c = (int)(t - i * m);
    out[t] = tally[(int64_t)c * qp + i];
}

// dst[g][0..words) = src[g][0..words) for row strides that differ
__global__ void k_copy_rows(const uint32_t *src, int64_t src_stride, uint32_t *dst, int64_t dst_stride,
                            int64_t rows, int64_t words)
{
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= rows * words) return;
    const int64_t r = t / words, w = t - r * words;
    dst[r * dst_stride + w] = src[r * src_stride + w];
}

// fresh[g] = {plo, phi, slo, 0}: nothing outdated (0, 0, qp) or everything outdated (0, qp, qp)
__global__ void k_fresh_set(int32_t *fresh, int C, int qp, int all_stale)
{
    const int g = blockIdx.x * blockDim.x + threadIdx.x;
    if (g < C) *reinterpret_cast<int4 *>(fresh + (int64_t)g * 4) = make_int4(0, all_stale ? qp : 0, qp, 0);
}

} // namespace tsetlin

#endif

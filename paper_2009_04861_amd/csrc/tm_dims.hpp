// Sizes and settings of a machine as the kernels take them.
#ifndef TM_DIMS_HPP_
#define TM_DIMS_HPP_
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "tm_device.hpp"

namespace tsetlin {

struct Dims {
    int m, n, o, N, T, C, Wf, W;
    uint32_t thr;      // 16-bit threshold: P(u < thr) = 1/s
    uint32_t boost;    // ~0 if true positives are boosted (strong Type I event certain), else 0
    int regr;          // 1: regression mode (one bank of clauses that all vote +1, targets 0..T)
    uint32_t tailmask; // valid bits of the last feature word
    RngKey key;
};

} // namespace tsetlin

#endif

// The greedy choice: a (logit, vocabulary id) pair and the order that decides between two, shared by
// the LM-head kernels.
#pragma once
#include "device.h"

struct ArgMax {
    float v;
    int32_t i;
};

// a better than b: larger value, or equal value and lower id; NaN never wins
__device__ __forceinline__ bool better(float av, int ai, float bv, int bi) {
    return av > bv || (av == bv && ai < bi);
}

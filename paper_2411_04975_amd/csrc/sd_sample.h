// How large a sample of the tokens the intervals of the sort by codes come from, and what it may overlook. Host code without any
// HIP call, so that it can be held to its promises without a GPU.
#pragma once
#include <stdint.h>

constexpr int64_t SAMPLE_MIN = 4096;   // runs of 64 tokens: a bin of a 256-way split sees 1000 of their tokens
constexpr int SAMPLE_ONE_IN = 64;      // a token that goes unseen has a few hundred occurrences at most
constexpr int64_t SAMPLE_MAX = 32768;  // 16 * 64 * SAMPLE_MAX + 4 * 2^24, the weights' total, is below 2^27

constexpr uint32_t SIGHTING = 16;      // weight of a token that the sample has seen once
constexpr uint32_t UNSEEN = SIGHTING / 4;

// runs of 64 tokens that are looked at
static inline int64_t sd_sample_runs(int64_t n_tokens) {
    const int64_t runs = (n_tokens + 63) / 64;
    int64_t C = runs / SAMPLE_ONE_IN > SAMPLE_MIN ? runs / SAMPLE_ONE_IN : SAMPLE_MIN;
    if (C > SAMPLE_MAX) C = SAMPLE_MAX;
    return C > runs ? runs : C;
}

// How far above twice its block's average a token's weight may be where the block's tokens get equal parts of its interval: three
// sightings, 192 tokens, as long as one token in SAMPLE_ONE_IN is looked at.  A sighting of a thinner sample stands for more
// tokens, 1024 of 2^31, and a bucket of twice that many besides its own 2047 entries would not fit a workgroup: so it is
// as much less as the sample is thinner, and what a token has too much of stays at some two hundred entries.
static inline uint32_t sd_even_slack(int64_t n_tokens) {
    const int64_t most = 3 * SIGHTING, seen = sd_sample_runs(n_tokens) * 64;
    if (n_tokens <= seen * SAMPLE_ONE_IN) return (uint32_t)most;
    return (uint32_t)(most * SAMPLE_ONE_IN * seen / n_tokens);
}

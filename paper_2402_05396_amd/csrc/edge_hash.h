// Hash of an edge index for a table of a power of two of slots, of which the low bits are taken.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

// Batches are often regular (every 2048th edge, a run of them): the low bits of a product alone send edges a
// multiple of the table's size apart to one slot, its high bits those a Fibonacci number apart. Two products with
// the high bits folded down before, between and behind them leave a handful of probes in either case (1 024 edges
// 2 048 apart, one block's update: 250 us with one product's low bits, 3.4 so). The factors are 2^32 times the
// fractions of the golden ratio and of sqrt(3), rounded to odd numbers.
__host__ __device__ inline uint32_t edge_hash(uint32_t e) {
    e ^= e >> 16;
    e *= 0x9E3779B1u;
    e ^= e >> 15;
    e *= 0xBB67AE85u;
    return e ^ (e >> 16);
}

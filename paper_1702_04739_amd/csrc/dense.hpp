// dense.hpp -- interface of dense.hip (the tree of few points from all their exact distances).
#pragma once

#include <cstddef>
#include <cstdint>

#include <hip/hip_runtime.h>

namespace iso {

constexpr int DENSE_MAX_N = 4096;

struct DenseState {
    int32_t ncomp, edges, rounds;
    int32_t joined;   // components before the last round
    int32_t arrived;  // workgroups of the running round that have finished their rows
    int32_t bad;      // a D^2 out of range, or no tree: the caller screens instead
};

struct DenseArgs {
    const float *X;
    int64_t n, d, ld;
    bool f64;         // the recheck whose arithmetic orders the edges
    void *buf;        // dense_bytes(n, f64) bytes
    int32_t *comp;    // [n]
    int32_t *eu, *ev; // [n] the n - 1 edges
    DenseState *st;
};

size_t dense_bytes(int64_t n, bool f64);
// The edges, and st: the tree is whole when ncomp is 1 and bad is 0.
void launch_dense_tree(const DenseArgs &A, hipStream_t s);
// Rooted at vertex 0 (elen: the edges' lengths).
void launch_dense_root(const DenseArgs &A, const double *elen, int32_t *parent, double *length, hipStream_t s);

}  // namespace iso

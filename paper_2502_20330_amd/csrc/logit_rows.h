// Loads of fp32 logit rows, shared by the accept kernels.
#pragma once
#include <hip/hip_runtime.h>

typedef float floatx4 __attribute__((ext_vector_type(4)));

// Rows of logits start at any multiple of 4 bytes (a vocabulary that is not a multiple of four leaves three rows of
// four unaligned); 128-bit global loads need no more than that.  (Scalar loads for such rows: an odd vocabulary of
// 50257, eight sequences, took 22 us in accept_rows alone.)
typedef floatx4 floatx4_any __attribute__((aligned(4)));
__device__ __forceinline__ floatx4 load4_full(const float* p) { return *reinterpret_cast<const floatx4_any*>(p); }

// Four consecutive logits of a row from index i on, where the row may end: entries at or past V come back as -inf.
// Threads at the end load the row's last four entries and shift them.  Load and shift are two steps, so that a caller
// has all its loads in flight before it waits for the first (V >= 4; shorter rows: load4).
__device__ __forceinline__ floatx4 load4_tail(const float* row, int i, int V) { return load4_full(row + min(i, V - 4)); }
__device__ __forceinline__ floatx4 shift_tail(floatx4 x, int i, int V)
{
    const int s = i - (V - 4);                            // entries of the load that lie before i
    if (s > 0) {
        if (s & 1) x = floatx4{x[1], x[2], x[3], -INFINITY};
        if (s & 2) x = floatx4{x[2], x[3], -INFINITY, -INFINITY};
        if (s > 3) x = floatx4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    }
    return x;
}
__device__ __forceinline__ floatx4 load4(const float* row, int i, int V)
{
    if (V >= 4) return shift_tail(load4_tail(row, i, V), i, V);
    floatx4 r = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
    for (int j = 0; j < 3; ++j)
        if (i + j < V) r[j] = row[i + j];
    return r;
}
// N runs of four, `step` entries apart, the first at index i; `full`: the row holds all of them for every thread.
// ONCE: nobody reads the row again (streaming hint; rows that the draw reads again lose by it, 64 sequences 115 -> 119 us).
template <int N, bool ONCE = false>
__device__ __forceinline__ void load_runs(floatx4 (&r)[N], const float* row, int i, int step, int V, bool full)
{
    if (full) {
#pragma unroll
        for (int v = 0; v < N; ++v) {
            const float* p = row + v * step + (unsigned)i;                                 // uniform base + 32-bit offset
            r[v] = ONCE ? __builtin_nontemporal_load(reinterpret_cast<const floatx4_any*>(p)) : load4_full(p);
        }
    } else if (V >= 4) {
#pragma unroll
        for (int v = 0; v < N; ++v) {
            r[v] = floatx4{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
            if (i + v * step < V) r[v] = load4_tail(row, i + v * step, V);
        }
    } else {
#pragma unroll
        for (int v = 0; v < N; ++v) r[v] = load4(row, i + v * step, V);
    }
}
template <int N>
__device__ __forceinline__ void shift_runs(floatx4 (&r)[N], int i, int step, int V, bool full)
{
    if (full || V < 4) return;
#pragma unroll
    for (int v = 0; v < N; ++v)
        if (i + v * step < V) r[v] = shift_tail(r[v], i + v * step, V);      // (past the end: load_runs left -inf)
}
